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
    L.lp_single_units.restype = C.c_int64
    L.lp_single_units.argtypes = [C.c_int, C.c_int, C.c_int64, C.c_int, C.c_int]
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
                            assert quot > LDS - 80
                    assert not probe.lp_single(1281, 0, quot)
    assert taken and refused


@pytest.mark.parametrize("threads", [64, 128, 192, 256, 512, 1024])
def test_grids_stay_below_the_work_item_limit(probe, threads):
    assert probe.lp_max_workgroups(threads) * threads < 2 ** 32 <= (probe.lp_max_workgroups(threads) + 1) * threads
    for work in (8, 800, 2 ** 22, 2 ** 24, 2 ** 26, 2 ** 30, 2 ** 33):
        g = probe.lp_strided_grid(work, threads)
        assert g % 8 == 0 and 0 < g <= work and g * threads < 2 ** 32
        assert g == work or work * threads >= 2 ** 32


def test_single_launch_units(probe):
    """Only with the Jacobian, and for systems of many variables of which most
    outputs have no or one term."""
    for n, k, m, units in ((99, 2, 8, 1280), (100, 2, 8, 4096), (199, 2, 900, 4096), (200, 2, 900, 16384),
                           (199, 4, 2, 1280), (200, 4, 12, 16384), (200, 4, 13, 4096), (200, 4, 25, 4096),
                           (200, 4, 26, 1280), (300, 4, 75, 4096), (300, 4, 76, 1280), (299, 4, 74, 1280),
                           (400, 4, 199, 4096), (400, 4, 200, 1280), (449, 2, 900, 16384), (450, 2, 113, 4096),
                           (450, 2, 112, 16384)):
        assert probe.lp_single_units(n, k, m, 4, 1) == units
        assert probe.lp_single_units(n, k, m, 2, 1) == (16384 if (n, k, m) == (450, 2, 113) else units)
        for words, jac in ((2, 0), (4, 0), (8, 1)):
            assert probe.lp_single_units(n, k, m, words, jac) == 1280


def test_coefficients_that_the_quotients_take(probe):
    """Within 2^+-300 or exactly zero, and finite in every word."""
    inf, nan = float("inf"), float("nan")
    for c, ok in (((1, 0, 0, 0), 1), ((0, 0, 0, 0), 1), ((0, 0, -1, 1e-20), 1), ((0, 1e-20, 0, 0), 0),
                  ((2.0 ** 299, 0, 0, 0), 1), ((2.0 ** 300, 0, 0, 0), 0), ((0, 0, 2.0 ** -299, 0), 1),
                  ((0, 0, 2.0 ** -300, 0), 0), ((nan, 0, 1, 0), 0), ((1, 0, nan, 0), 0), ((1, nan, 1, 0), 0),
                  ((inf, 0, 1, 0), 0), ((1, 0, -inf, 0), 0), ((1, 0, 1, inf), 0), ((nan, 0, nan, 0), 0)):
        assert probe.lp_coef_ok((C.c_double * 4)(*c)) == ok, c


def test_window_of_the_points(probe):
    """Every |x_i| < 2^(b + 1/2 + 1/2): quads of factors within 2^400, or, where
    they are checked, powers within 2^300; never narrower than 2^+-8."""
    check = C.c_int()
    last = 61
    for d in range(1, 32):
        b = probe.lp_window(d, C.byref(check))
        top = b + 1.5  # log2 of the modulus, at most
        assert 8 <= b <= 59
        if check.value:
            assert d * top <= 300 and d >= 6
        else:
            assert 4 * d * top <= 400 and b >= 16 and d <= 5
            assert b <= last
            last = b


def test_words_of_the_waves_fit(probe):
    """16 words after a workgroup's tables, only where they cost no workgroup."""
    probe.lp_add_skip_words.restype = C.c_int64
    probe.lp_add_skip_words.argtypes = [C.c_int64]
    for per_cu in range(1, 40):
        most = LDS // per_cu
        for lds in (most, most - 63, most - 64, most - 65):
            if LDS // lds != per_cu:
                continue
            got = probe.lp_add_skip_words(lds)
            assert got == (lds + 64 if lds + 64 <= most else -1)
