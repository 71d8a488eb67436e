"""The byte model that the benchmark reports: words per voxel of the passes
of a CG iteration."""
import pytest

import bench


def test_words_of_an_iteration():
    assert sum(bench.WORDS_MOVED.values()) == 61.5
    # the kernel classes of an iteration on the separate passes, and no others
    assert set(bench.WORDS_MOVED) == {"front", "r2c", "axis", "zproj", "axis3", "c2r3"}


def test_roofline_of_the_operator():
    N = 256 ** 3
    prof = {k: (0.0, 0) for k in list(bench.WORDS_MOVED) + ["finalize", "constitutive", "grad"]}
    prof["front"] = (0.535 * 20, 20)
    prof["zproj"] = (0.294 * 20, 20)
    prof["finalize"] = (0.01 * 3, 3)
    r = bench.roofline(dict(prof=prof, words=bench.WORDS_MOVED), N, 8)
    assert r["kernel"] == "front" and r["bytes_per_launch"] == 18 * 8 * N
    assert r["achieved"] == pytest.approx(18 * 8 * N / 535e-6 / 1e9, rel=1e-3)
    assert set(r["per_class"]) == {"front", "zproj", "finalize"}
    assert r["per_class"]["zproj"]["GB/s"] == pytest.approx(12 * 8 * N / 294e-6 / 1e9, rel=1e-2)
    assert "GB/s" not in r["per_class"]["finalize"]
