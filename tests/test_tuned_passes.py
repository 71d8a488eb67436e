"""What the tile tuner measures: the passes that a plan runs, and a cache that
knows which kernels its entries were measured on."""
import json
import re

import pytest

from paper_2411_16583_amd import autotune
from tests.fake_hip import run_with_fake_hip
from tests.test_host_logic import FakeLib

BODY = """
out = []
for grid, prec in GRIDS:
    p = HostPlan(grid, prec)
    for which in range(4 if prec else 2):
        log()
        ms = ctypes.c_double()
        assert lib.fg_plan_time_pass(p.h, which, 0, 1, ctypes.byref(ms)) == 0
        out.append([l[1] for l in log() if l[0] == "launch" and "k_fill" not in l[1]])
result = out
"""
# a grid whose CG has the passes, and one whose planes are transformed in LDS
LARGE, SMALL = [128, 96, 16], [16, 16, 16]


def kernels(names):
    """Kernel names without their namespace, e.g. 'k_n0<...mangled arguments'."""
    return [re.sub(r"^_ZN2fg\d+", "", n) for n in names]


def test_the_tuner_times_the_passes_that_the_plan_runs(tmp_path):
    got = run_with_fake_hip(tmp_path, f"GRIDS = {[(LARGE, 0), (LARGE, 1), (SMALL, 0), (SMALL, 1)]}" + BODY)
    got = [kernels(g) for g in got]
    large64, large_mixed, small64, small_mixed = got[0:2], got[2:6], got[6:8], got[8:12]

    def only(run, name):
        assert run and all(k.startswith(name) for k in run), run

    for axis, zproj, t in [(large64[0], large64[1], "d"), (large_mixed[2], large_mixed[3], "f")]:
        only(axis, f"k_n1I{t}")
        # the CG's own mode and symbol, the last two arguments
        only(zproj, f"k_n0I{t}{t}")
        assert all(re.match(r"k_n0I..Li128ELi\dELi0ELi0EE", k) for k in zproj), zproj
    for axis, zproj in [large_mixed[0:2], small64, small_mixed[0:2]]:
        only(axis, "k_rows_n1I")
        only(zproj, "k_rows_n0I")
    only(small_mixed[2], "k_fft_axisIf")
    assert all(k.startswith(("k_fft_z_projIf", "k_fft_z_dcIf")) for k in small_mixed[3]) and small_mixed[3]


@pytest.mark.parametrize("entry", [{"tile": 2}, {"tile": 2, "kernels": autotune.KERNELS - 1}])
def test_entries_of_other_kernels_are_timed_again(tmp_path, entry):
    path = str(tmp_path / "tiles.json")
    key = "gfx950|8x8x8|items=1|axis_f64"
    json.dump({key: entry}, open(path, "w"))
    lib = FakeLib({0: [1, 2], 1: [1]}, {(0, 1): 1.0, (0, 2): 2.0, (1, 1): 1.0})
    autotune.tune_handle(None, (8, 8, 8), 1, 0, path, lib=lib, arch="gfx950")
    assert lib.set[0] == 1 and (0, 1) in lib.timed
    assert json.load(open(path))[key]["kernels"] == autotune.KERNELS
