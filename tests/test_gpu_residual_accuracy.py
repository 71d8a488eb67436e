"""The Newton residual and the gradient projection on elongated voxels: what
is left of an equilibrated stress is its rounding, eps |P| whatever the voxel's
shape (a divergence differenced in real space rounds by eps |P| / h of the
shortest side, which the projection amplifies on the long waves).

Tolerance 8e-16 |P|: three transforms of at most 8 butterfly levels each,
two roundings of eps / 2 per level, rms sqrt(48) eps / 2.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import spectral
from paper_2411_16583_amd import make_opts
from tests.gpu_util import DEV, dt, host, plan_for

pytestmark = pytest.mark.gpu

# planes transformed in LDS, grids that take the separate passes (N0 and N1 in
# parts, a long axis of each kind) and a plane grid; spacings (h0, h1, h2)
CASES = [((16, 64, 64), (32.0, 1.0, 1.0)), ((16, 64, 64), (1.0, 1.0, 32.0)), ((16, 64, 64), (1.0, 1.0, 1.0)),
         ((128, 96, 16), (1.0, 1.0, 32.0)), ((128, 96, 16), (1.0, 32.0, 1.0)), ((24, 256, 64), (32.0, 1.0, 1.0)),
         ((1, 64, 64), (1.0, 1.0, 16.0)), ((6, 96, 96), (16.0, 1.0, 4.0)), ((256, 8, 4), (1.0, 24.0, 1.0))]
TOL = 8e-16


def workload(shape, spacing):
    h = np.array(spacing) / max(shape)
    return synth.homogeneous_workload(shape, tuple(float(n * x) for n, x in zip(shape, h)))


@pytest.mark.parametrize("shape,spacing", CASES)
def test_projection_of_an_equilibrated_field(shape, spacing):
    print(f"equilibrated {shape} {spacing}", flush=True)
    work = workload(shape, spacing)
    x = np.random.default_rng(3).standard_normal((3, 3) + shape)
    for _ in range(2):
        x = x - spectral.project(x, work["spacing"])
    plan = plan_for(work)
    y = torch.empty((9,) + shape, dtype=torch.float64, device=DEV)
    plan.project_grad(dt(x.reshape((9,) + shape)), y)
    assert np.linalg.norm(host(y)) <= TOL * np.linalg.norm(x)
    plan.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape,spacing", [CASES[0], CASES[1], CASES[3]])
def test_residual_of_an_equilibrated_cell(shape, spacing, precision):
    """err_res of a state that Newton cannot improve = the oracle's projection
    of the same stress."""
    print(f"residual {shape} {spacing} {precision}", flush=True)
    work = workload(shape, spacing)
    work["E"] = np.where(np.random.default_rng(5).random(shape) < 0.3, 10.5e9, 10e9)
    Fbar = np.diag([1.0, 1.4, 1.0])
    plan = plan_for(work, precision)
    F = dt(np.broadcast_to(Fbar.reshape(3, 3, 1, 1, 1), (3, 3) + shape).copy())
    P = torch.empty((9,) + shape, dtype=torch.float64, device=DEV)
    plan.set_state(F)
    plan.stress(P)
    den = np.linalg.norm(spectral.project(host(P, (3, 3) + shape), work["spacing"]))
    plan.newton_solve(Fbar, make_opts(1e-30, 1e-8, max_newton=6), raise_on_error=False)
    plan.stress(P)
    Pn = host(P, (3, 3) + shape)
    exact = np.linalg.norm(spectral.project(Pn, work["spacing"]))
    assert abs(plan.residual(Fbar) * den - exact) <= TOL * np.linalg.norm(Pn)
    plan.close()
