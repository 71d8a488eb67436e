"""The divergence form of the CG (q = D^T K : (D pi) formed by patches of 8
lines x 16 or 32 voxels whose edges are stored apart and added by the N2 pass,
runs of node planes along N0, the block layout of the N0 pass) at the sizes
where its splits can go wrong, against the CPU oracle.

Tolerances as for the other grids: the projection 1e-13 (FP64 rounding of
the transforms), CG iterates 1e-11 in double and 1e-5 in single precision.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import constitutive as cm
from oracle import krylov, mechanics, spectral
from tests.gpu_util import dt, host, plan_for, rel

pytestmark = pytest.mark.gpu

# partial blocks of lines (N1 = 6, 12), half and one-and-a-half patches along
# N2 (8, 24, 48), one block exactly (8), a plane, node-plane runs that do not
# divide N0 (48 and 96 planes), blocks padded in the block layout (N0 >= 64)
SHAPES = [(4, 6, 8), (6, 12, 24), (8, 8, 16), (1, 12, 48), (48, 4, 12), (96, 6, 8), (64, 8, 32),
          (4, 24, 96)]
# largest (N0, N1) planes transformed in LDS as one (96 x 96), the first ones
# that are not (128 x 96), lines of every shape on both axes; cubic voxels
PLANES = [(96, 96, 4), (128, 96, 4), (32, 16, 6), (48, 64, 8), (128, 12, 8), (256, 8, 4), (24, 256, 4), (1, 512, 8)]


@pytest.mark.parametrize("shape", SHAPES)
def test_projection_by_divergence(shape):
    print(f"projection by divergence {shape}", flush=True)
    work = synth.homogeneous_workload(shape, (1.0, 0.7, 1.3))
    plan = plan_for(work)
    x = np.random.default_rng(11).standard_normal((3, 3) + shape)
    y = torch.empty((9,) + shape, dtype=torch.float64, device="cuda:0")
    plan.project_grad(dt(x.reshape((9,) + shape)), y)
    ref = spectral.project(x, work["spacing"])
    assert rel(host(y, (3, 3) + shape), ref, x) <= 1e-13
    plan.close()


# (without (4, 24, 96) in single precision: with voxels 24 times longer along
# one axis the potentials of the modes whose gradient nearly vanishes are 3e3
# times larger than their gradients, and their single-precision storage moves
# the fourth iterate by 2e-5, whichever way the operator is applied)
@pytest.mark.parametrize("law", ["neo_hookean", "svk"])
@pytest.mark.parametrize("shape,precision,tol", [(s, "fp64", 1e-11) for s in SHAPES + PLANES] +
                         [(s, "mixed", 1e-5) for s in SHAPES[:-1] + PLANES])
def test_cg_iterates_by_divergence(shape, precision, tol, law):
    """Four CG iterations (2, then 2 more) of the first Newton system of a
    random two-phase cell = the oracle's 9-component CG."""
    check_cg_iterates(shape, precision, tol, law, tuple(float(n) for n in shape) if shape in PLANES else 1.0)


def check_cg_iterates(shape, precision, tol, law, lengths, parts=(2, 2)):
    print(f"cg {shape} {precision} {law}", flush=True)
    work = synth.homogeneous_workload(shape, lengths)
    rng = np.random.default_rng(5 + shape[2])
    phase = rng.random(shape) < 0.3
    work["E"] = np.where(phase, 100e9, 10e9)
    work["law"] = law
    Fbar = np.eye(3)
    Fbar[1, 1] += 0.004
    Fbar[2, 1] += 0.003
    F0 = mechanics.uniform_field(Fbar, shape)
    c0, d0 = work["c0"], work["d0"]
    GP, _ = mechanics.residual_rhs(F0, c0, d0, work, work["spacing"])
    b = -spectral.project(GP, work["spacing"])
    K = cm.tangent(F0, c0, d0, work["E"], work["nu"], work["Omega"], law=law)
    dF, _, _ = krylov.cg(lambda X: mechanics.operator(K, X, work["spacing"]), b, 1e-10, 100, fixed_iters=sum(parts))
    plan = plan_for(work, precision)
    F = dt(F0)
    plan.set_state(F, dt(c0), dt(d0))
    plan.newton_linear_begin(Fbar)
    for k, n in enumerate(parts):
        st = plan.cg_iterate(n, apply=k == len(parts) - 1)
    assert st["iters"] == sum(parts)
    assert rel(host(F, (3, 3) + shape) - F0, dF) <= tol
    plan.close()


@pytest.mark.parametrize("shape,precision", [((12, 8, 16), "fp64"), ((64, 8, 32), "mixed"), ((128, 96, 12), "fp64"),
                                             ((128, 96, 16), "mixed"), ((256, 8, 64), "fp64")])
def test_cg_ends_alike_wherever_its_scalars_are_read(shape, precision):
    """r.r and beta are formed by the pass after the N0 pass between iterations
    (in every workgroup of it, or in one of them), and by a kernel of their own
    before the host reads them: the same bits, so 9 iterations in one call and
    in calls of 1, 3 and 5 give the same solution."""
    print(f"cg in parts {shape} {precision}", flush=True)
    work = synth.homogeneous_workload(shape, 1.0)
    phase = np.random.default_rng(3).random(shape) < 0.3
    work["E"] = np.where(phase, 100e9, 10e9)
    Fbar = np.eye(3)
    Fbar[0, 1] += 0.004
    out = []
    for parts in ((9,), (1, 3, 5)):
        plan = plan_for(work, precision)
        F = dt(mechanics.uniform_field(Fbar, shape))
        plan.set_state(F, dt(work["c0"]), dt(work["d0"]))
        plan.newton_linear_begin(Fbar)
        for k, n in enumerate(parts):
            plan.cg_iterate(n, apply=k == len(parts) - 1)
        out.append(host(F, (3, 3) + shape))
        plan.close()
    assert np.array_equal(out[0], out[1])


# the largest grid whose iteration runs as lines (32^3 voxels, 64-long lines) and
# the first ones that take the passes; odd counts of lines and blocks of lines;
# more planes than CUs
LINES = [(32, 32, 32), (32, 32, 48), (1, 12, 64), (4, 6, 64), (24, 4, 64), (64, 96, 6), (48, 48, 24), (6, 96, 96),
         (8, 12, 192)]


@pytest.mark.parametrize("law", ["neo_hookean", "svk"])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-11), ("mixed", 1e-5)])
@pytest.mark.parametrize("shape", LINES)
def test_cg_iterates_as_lines_or_passes(shape, precision, tol, law):
    """Both sides of the choice between the one-kernel front of a CG iteration
    and its passes, against the oracle (cubic voxels; the tolerances above)."""
    check_cg_iterates(shape, precision, tol, law, tuple(float(n) for n in shape))


@pytest.mark.parametrize("parts", [(1,), (2,), (1, 2), (3, 2)])
@pytest.mark.parametrize("shape,precision,tol", [((128, 96, 4), "fp64", 1e-11), ((128, 96, 4), "mixed", 1e-5),
                                                 ((32, 32, 48), "fp64", 1e-11), ((8, 8, 16), "fp64", 1e-11)])
def test_solution_after_any_count_of_iterations(shape, precision, tol, parts):
    """The solution takes its steps late, two at a time where the direction has
    two buffers and the passes run: the steps still due are added with the
    result, after odd and even counts (against the oracle, the tolerances above)."""
    check_cg_iterates(shape, precision, tol, "neo_hookean", tuple(float(n) for n in shape), parts)
