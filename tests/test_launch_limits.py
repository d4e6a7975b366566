"""Host functions that size the launches of the quotient kernels
(quotient_tables.cpp, launch_limits.hpp), checked on the CPU against the hardware's limits.
"""
import ctypes as C
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1201_0499_amd", "csrc")
LDS = 160 * 1024


@pytest.fixture(scope="module")
def probe():
    d = tempfile.mkdtemp(prefix="pe_launch_")
    so = os.path.join(d, "liblaunch.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}",
                    os.path.join(ROOT, "tests", "cpp", "launch_probe.cpp"),
                    os.path.join(CSRC, "quotient_tables.cpp"), "-o", so], check=True)
    L = C.CDLL(so)
    L.lp_chunk.argtypes = [C.c_int, C.c_int, C.c_int, C.c_int64, C.c_int]
    L.lp_lds.restype = C.c_int64
    for name in ("lp_small_lds", "lp_single"):
        getattr(L, name).argtypes = [C.c_int64] * (2 if name == "lp_small_lds" else 3)
    L.lp_small_lds.restype = C.c_int64
    L.lp_max_workgroups.restype = L.lp_strided_grid.restype = C.c_int64
    L.lp_strided_grid.argtypes = [C.c_int64, C.c_int]
    return L


@pytest.mark.parametrize("words,n,d,m", [
    (4, 1024, 3, 1024), (4, 512, 7, 1024), (4, 512, 8, 512), (4, 1264, 3, 64), (4, 256, 15, 1024),
    (2, 1024, 8, 1024), (8, 512, 2, 1024), (8, 256, 5, 1024), (8, 384, 3, 1024), (8, 512, 3, 512),
])
def test_single_launch_with_tables_that_fill_the_lds(probe, words, n, d, m):
    """Tables of exactly 160 KiB leave no room for the single launch's flag:
    such calls take two launches, however few pairs they have."""
    ch = probe.lp_chunk(n, d, 0, m, words)
    quot = probe.lp_lds(n, d, 0, ch, int(ch < m), 1, words)
    assert ch and quot == LDS
    assert probe.lp_small_lds(1000, quot) > LDS
    assert not probe.lp_single(1, 1000, quot)


@pytest.mark.parametrize("words", [2, 4, 8])
def test_single_launch_fits_the_lds(probe, words):
    """What one launch asks for is within the LDS, over sizes up to its edge."""
    taken = refused = 0
    for n in list(range(1, 1300, 37)) + [256, 512, 1024]:
        for d in (1, 2, 3, 5, 8, 15, 31):
            for m in (1, 64, 300, 1024, 3000):
                for pad in (0, 1):
                    ch = probe.lp_chunk(n, d, pad, m, words)
                    if not ch:
                        continue
                    quot = probe.lp_lds(n, d, pad, ch, int(ch < m), 1, words)
                    for general in (0, quot, LDS):
                        if probe.lp_single(1280, general, quot):
                            taken += 1
                            assert probe.lp_small_lds(general, quot) <= LDS
                            assert probe.lp_small_lds(general, quot) >= max(general, quot + 4)
                        else:
                            refused += 1
                            assert quot > LDS - 16
                    assert not probe.lp_single(1281, 0, quot)
    assert taken and refused


@pytest.mark.parametrize("threads", [64, 128, 192, 256, 512, 1024])
def test_grids_stay_below_the_work_item_limit(probe, threads):
    assert probe.lp_max_workgroups(threads) * threads < 2 ** 32 <= (probe.lp_max_workgroups(threads) + 1) * threads
    for work in (8, 800, 2 ** 22, 2 ** 24, 2 ** 26, 2 ** 30, 2 ** 33):
        g = probe.lp_strided_grid(work, threads)
        assert g % 8 == 0 and 0 < g <= work and g * threads < 2 ** 32
        assert g == work or work * threads >= 2 ** 32
