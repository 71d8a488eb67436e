"""The dynamic-LDS limit of the plane kernels is process-wide: plans of
different planes, whose launches may interleave in different threads, all set
the same one, and no launch asks for more."""
from tests.fake_hip import run_with_fake_hip

BODY = """
opts = fgfft.SolverOpts(1e-8, 1e-10, 10, 100, 0)
stats = fgfft.Stats()
fake.fake_fail_waits(1)  # the stand-in never converges: the solve ends at its first wait
out = []
for grid in [(96, 96, 8), (64, 64, 8), (64, 96, 8), (16, 16, 8)]:
    p = HostPlan(grid)
    assert lib.pff_solve(p.h, ctypes.byref(opts), ctypes.byref(stats)) == fgfft.FG_E_HIP
    out += log()
result = out
"""


def test_every_launch_sets_the_same_limit(tmp_path):
    log = run_with_fake_hip(tmp_path, BODY)
    limits, launches = {}, {}
    for what, name, n, *_ in log:
        if "k_plane" in name:
            (limits if what == "limit" else launches).setdefault(name, set()).add(n)
    assert len(launches) == 2  # the start and the iteration
    for name, asked in launches.items():
        assert len(asked) == 4 and min(asked) <= 65536 < max(asked)
        assert len(limits[name]) == 1 and max(asked) <= max(limits[name]) <= 160 * 1024
