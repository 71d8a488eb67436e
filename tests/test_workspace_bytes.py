"""Workspace of a plan and of a batch: no more memory per voxel than the
solver has always asked for, so that the largest problem that fits stays the
same."""
import pytest

from tests.fake_hip import run_with_fake_hip

GRIDS = [(16, 16, 16), (64, 64, 64), (96, 96, 96), (128, 128, 128), (256, 256, 256), (48, 96, 192), (4, 24, 96),
         (128, 96, 8), (256, 256, 4), (1, 64, 64), (1, 256, 256), (1, 512, 512), (256, 512, 32), (4, 4, 4)]

BODY = """
def plan_bytes(grid, prec, law):
    h = ctypes.c_void_p()
    assert lib.fg_plan_create((ctypes.c_int * 3)(*grid), (ctypes.c_double * 3)(1.0, 1.0, 1.0), prec, None,
                              ctypes.byref(h)) == 0
    assert lib.fg_set_law(h, law) == 0
    return lib.fg_plan_workspace_bytes(h)


def batch_bytes(grid, prec, cases):
    h = ctypes.c_void_p()
    assert lib.fg_batch_create(1, (ctypes.c_int * 3)(*grid), (ctypes.c_double * 3)(1.0, 1.0, 1.0), cases, prec, None,
                               ctypes.byref(h)) == 0
    return lib.fg_batch_workspace_bytes(h)


result = [[[plan_bytes(g, p, law) for law in (0, 1)] + [batch_bytes(g, p, 6)] for p in (0, 1)] for g in GRIDS]
"""


def allowed(grid, prec, law, items):
    """Nine-component stress in double, stress, three CG vectors and the tangent
    state in the working precision, the kx = 0 column of nine components, the
    scalar solvers' 16 fields (a batch: one, and 13 of its items' state and
    material), 9 partial sums per 256 voxels in two buffers, the tables and
    padding."""
    n0, n1, n2 = grid
    N = n0 * n1 * n2 * items
    t = 8 if prec == 0 else 4
    fields = (36 if prec == 0 else 36 + 18) * t + (12, 18)[law] * t + 8 * (16 if items == 1 else 14)
    return (N * fields + 18 * 8 * n0 * n1 * items + 2 * 8 * (9 * items * (N // items // 256 + 2) + 8192) +
            400 * (n0 + n1 + n2) + 64 * 1024)


@pytest.mark.parametrize("k", range(len(GRIDS)), ids=[str(g) for g in GRIDS])
def test_no_more_bytes_than_before(got, k):
    for prec in (0, 1):
        for j, (law, items) in enumerate([(0, 1), (1, 1), (0, 6)]):
            assert got[k][prec][j] <= allowed(GRIDS[k], prec, law, items), (prec, law, items)


@pytest.fixture(scope="module")
def got(tmp_path_factory):
    return run_with_fake_hip(tmp_path_factory.mktemp("fake"), f"GRIDS = {GRIDS}" + BODY)
