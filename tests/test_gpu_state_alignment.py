"""A state field that starts on any double (a view into a larger tensor): the
solver gives the same bits as for one that starts on a wider boundary."""
import numpy as np
import pytest
import torch

import synth
from oracle import mechanics
from paper_2411_16583_amd import make_opts
from tests.gpu_util import DEV, dt, host, plan_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", [(8, 8, 8), (64, 64, 8), (128, 96, 4)])
def test_state_on_an_odd_double(shape, precision):
    print(f"state alignment {shape} {precision}", flush=True)
    work = synth.homogeneous_workload(shape, tuple(float(n) for n in shape))
    work["E"] = np.where(np.random.default_rng(9).random(shape) < 0.3, 100e9, 10e9)
    Fbar = np.eye(3)
    Fbar[1, 1] += 0.004
    F0 = dt(mechanics.uniform_field(np.eye(3), shape)).reshape(-1)
    out = []
    for shift in (0, 1):
        big = torch.zeros(F0.numel() + 2, dtype=torch.float64, device=DEV)
        F = big[shift:shift + F0.numel()]
        F.copy_(F0)
        assert (F.data_ptr() // 8) % 2 == shift
        plan = plan_for(work, precision)
        plan.set_state(F)
        plan.newton_solve(Fbar, make_opts(1e-8, 1e-8))
        out.append(host(F))
        assert big[shift + F0.numel():].count_nonzero() == 0 and big[:shift].count_nonzero() == 0
        plan.close()
    assert np.array_equal(out[0], out[1])
