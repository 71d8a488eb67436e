"""Every tile of the passes that the CG runs gives the same bits: grids whose
iteration takes the separate N1 and N0 passes, so that the partial sums of
r.r come in groups of every size (several columns per group, one, a width that
is no power of two, and more groups than threads of the summing workgroup)."""
import ctypes

import numpy as np
import pytest

import synth
from oracle import mechanics
from paper_2411_16583_amd import Batch, make_opts
from paper_2411_16583_amd.autotune import candidates
from tests.gpu_util import dt, host, plan_for

pytestmark = pytest.mark.gpu

GRIDS = [((128, 96, 16), "fp64"), ((128, 96, 16), "mixed"), ((128, 96, 24), "fp64"), ((128, 96, 24), "mixed"),
         ((24, 512, 48), "fp64"), ((24, 512, 48), "mixed")]


@pytest.mark.parametrize("shape,precision", GRIDS)
def test_every_tile_gives_identical_iterates(shape, precision):
    work = synth.homogeneous_workload(shape, tuple(float(n) for n in shape))
    work["E"] = np.where(np.random.default_rng(6).random(shape) < 0.3, 100e9, 10e9)
    Fbar = np.eye(3)
    Fbar[1, 1] += 0.004
    F0 = mechanics.uniform_field(Fbar, shape)
    plan = plan_for(work, precision)

    def run(tiles):
        print(f"tiles {shape} {precision} {tiles}", flush=True)
        plan.set_tiles(tiles)
        F = dt(F0)
        plan.set_state(F)
        plan.newton_linear_begin(Fbar)
        st = plan.cg_iterate(3, apply=True)
        return np.append(host(F), st["relres"])

    ref = run([0, 0, 0, 0])
    assert 0 < ref[-1] < 1 and not np.array_equal(ref[:-1], F0.ravel())
    for w in range(2 if precision == "fp64" else 4):
        for b in candidates(plan.handle, w):
            tiles = [0, 0, 0, 0]
            tiles[w] = b
            assert np.array_equal(run(tiles), ref), (w, b)
    plan.close()


def test_every_tile_gives_an_identical_batch():
    """The same for several items through the passes, solved to the end."""
    shape = (128, 96, 4)
    E = np.where(np.random.default_rng(7).random(shape) < 0.3, 100e9, 10e9)
    b = Batch([shape], [(1.0, 1.0, 1.0)], 2)
    b.set_material(0, dt(E), dt(np.full(shape, 0.3)), dt(np.zeros(shape)))
    loads = synth.six_load_cases(1e-3)[:2]
    h = ctypes.c_void_p(b.lib.fg_batch_plan(b.handle, 0))
    out = []
    for w, tile in [(0, 0)] + [(w, t) for w in (0, 1) for t in candidates(h, w)]:
        print(f"batch tiles {w} {tile}", flush=True)
        tiles = [0, 0, 0, 0]
        tiles[w] = tile
        assert b.lib.fg_plan_set_tiles(h, (ctypes.c_int * 4)(*tiles)) == 0
        P, stats, _ = b.newton_solve(loads, make_opts(1e-8, 1e-10), graph_ticks=4)
        out.append(P)
    assert len(out) > 4 and all(np.array_equal(p, out[0]) for p in out)
    b.close()
