"""CG iterates of the mixed form on elongated voxels:
no further from the oracle's than single-precision storage of the potentials
makes them.  Storing a potential U rounds D U by eps |r|_rms |U|, with
|U| = |D U| / |r|: the tolerance is 8 (the vectors stored in an iteration, and
some room) times eps / 2 times the amplification rms(|r|) rms(1 / |r|) of the
grid.  (With the divergence of an iteration in single precision the errors were
ten times larger, up to 1.9 times the tolerance.)
"""
import numpy as np
import pytest

import synth
from oracle import constitutive as cm
from oracle import krylov, mechanics, spectral
from tests.gpu_util import dt, host, plan_for, rel

pytestmark = pytest.mark.gpu

# planes transformed in LDS and separate passes; long along N0, N1, N2, a plane
CASES = [((4, 24, 96), (24, 4, 1)), ((32, 32, 32), (4, 1, 16)), ((16, 16, 16), (1, 1, 4)), ((48, 48, 48), (10, 1, 1)),
         ((128, 96, 16), (1, 1, 8)), ((128, 96, 6), (2, 1, 1)), ((16, 64, 64), (32, 1, 32)), ((1, 16, 64), (1, 1, 4)),
         ((12, 8, 16), (1, 16, 1))]


def amplification(shape, h):
    c, s = zip(*[spectral.half_angle_sin_cos(np.arange(n), n)[::-1] for n in shape])
    c = np.meshgrid(*c, indexing="ij", sparse=True)
    s = np.meshgrid(*[2 * a / x for a, x in zip(s, h)], indexing="ij", sparse=True)
    r2 = (s[0] * c[1] * c[2]) ** 2 + (c[0] * s[1] * c[2]) ** 2 + (c[0] * c[1] * s[2]) ** 2
    return float(np.sqrt(r2.mean() * np.where(r2 > 0, 1 / np.where(r2 > 0, r2, 1), 0).mean()))


@pytest.mark.parametrize("law", ["neo_hookean", "svk"])
@pytest.mark.parametrize("shape,voxel", CASES)
def test_mixed_iterates_on_elongated_voxels(shape, voxel, law):
    print(f"mixed {shape} {voxel} {law}", flush=True)
    h = np.array(voxel, dtype=float) / max(shape)
    work = synth.homogeneous_workload(shape, tuple(float(n * x) for n, x in zip(shape, h)))
    # (blobs: white noise would be smoothed less by the projection)
    x = np.random.default_rng(5).standard_normal(shape)
    for ax in range(3):
        x = x + np.roll(x, 1, ax)
    work["E"] = np.where(x > np.quantile(x, 0.7), 100e9, 10e9)
    work["law"] = law
    Fbar = np.eye(3)
    Fbar[1, 1] += 0.004
    Fbar[2, 1] += 0.003
    F0 = mechanics.uniform_field(Fbar, shape)
    GP, _ = mechanics.residual_rhs(F0, work["c0"], work["d0"], work, work["spacing"])
    b = -spectral.project(GP, work["spacing"])
    K = cm.tangent(F0, work["c0"], work["d0"], work["E"], work["nu"], work["Omega"], law=law)
    dF, _, _ = krylov.cg(lambda X: mechanics.operator(K, X, work["spacing"]), b, 1e-10, 100, fixed_iters=6)
    plan = plan_for(work, "mixed")
    F = dt(F0)
    plan.set_state(F)
    plan.newton_linear_begin(Fbar)
    plan.cg_iterate(6, apply=True)
    err, tol = rel(host(F, (3, 3) + shape) - F0, dF), 8 * 2.0 ** -24 * amplification(shape, work["spacing"])
    plan.close()
    print(f"error {err:.1e}, allowed {tol:.1e}", flush=True)
    assert err <= tol
