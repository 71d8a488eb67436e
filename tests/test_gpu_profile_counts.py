"""Launch counts of the profiler for the three forms of a CG iteration: n
iterations and the residual passes of a Newton solve, nothing for the launches
behind the end of a solve."""
import numpy as np
import pytest

import synth
from oracle import mechanics
from paper_2411_16583_amd import make_opts
from tests.gpu_util import dt, plan_for

pytestmark = pytest.mark.gpu

# lines and planes in one kernel each; planes; separate passes
FORMS = [((16, 16, 16), "lines"), ((64, 64, 16), "planes"), ((128, 96, 8), "passes")]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape,form", FORMS)
def test_counted_launches_of_a_newton_solve(shape, form, precision):
    print(f"profile {shape} {precision}", flush=True)
    work = synth.homogeneous_workload(shape, tuple(float(n) for n in shape))
    work["E"] = np.where(np.random.default_rng(5).random(shape) < 0.3, 100e9, 10e9)
    Fbar = np.eye(3)
    Fbar[1, 1] += 0.004
    plan = plan_for(work, precision)
    plan.set_state(dt(mechanics.uniform_field(np.eye(3), shape)))
    plan.profile_begin()
    st = plan.newton_solve(Fbar, make_opts(1e-8, 1e-8))
    n = {k: c for k, (_, c) in plan.profile_end().items()}
    plan.close()
    its = st["lin_iters_total"]
    residuals = st["newton_iters"] + 2  # of the macroscopic state, of every iterate
    assert its > 10
    assert n["front"] == its
    assert n["zproj"] == its + residuals
    assert n["r2c"] == (0 if form == "lines" else its) + residuals
    assert n["c2r3"] == (0 if form == "lines" else its)
    assert n["axis"] == (its if form == "passes" else 0) + residuals
    assert n["axis3"] == (its if form == "passes" else 0)
    assert all(c >= 0 for c in n.values())
