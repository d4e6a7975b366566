"""The reciprocals that the quotients multiply with (dd.hpp), compiled for the
host, against exact rationals.

Every derivative by x_i carries the error of 1 / x_i whole, so it has to be
below that of one product: in double-double at most 2.5 u^2 of the modulus (the
last rounding of both parts, u^2, and six roundings of terms of order u, u^2 / 2
each at most, which never all meet) and 0.3 u^2 root mean square; in FP64 u
(1 + 2^-40) (the rounding of both parts, and terms of order u^2), 0.5 u root mean square
(u = 2^-53).  ArithDD::inv and Arith64::inv exceed all four.
"""
import ctypes as C
import os
import subprocess
import tempfile
from fractions import Fraction as Fr

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1201_0499_amd", "csrc")
_D = C.POINTER(C.c_double)


@pytest.fixture(scope="module")
def lib():
    d = tempfile.mkdtemp(prefix="pe_recip_")
    so = os.path.join(d, "librecip.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-ffp-contract=off", "-fno-fast-math",
                    f"-I{CSRC}", os.path.join(ROOT, "tests", "cpp", "recip_probe.cpp"), "-o", so], check=True)
    L = C.CDLL(so)
    L.rp_dd.argtypes = L.rp_f64.argtypes = [_D, _D]
    return L


def _draw(rng, words, scale):
    a = rng.uniform(0, 2 * np.pi)
    h = np.ldexp(np.array([np.cos(a), np.sin(a)]) * rng.uniform(1, 2), scale)
    b = np.zeros((2, words))
    b[:, 0] = h
    if words == 2:
        b[:, 1] = h * 2.0 ** -53 * rng.uniform(-0.5, 0.5, 2)
    return np.ascontiguousarray(b.reshape(-1))


def _exact(b):
    w = len(b) // 2
    return [sum((Fr(float(v)) for v in b[k * w:(k + 1) * w]), Fr(0)) for k in (0, 1)]


def _mul(a, b):
    return a[0] * b[0] - a[1] * b[1], a[0] * b[1] + a[1] * b[0]


def _errors(fn, words, n, scale, seed):
    rng = np.random.default_rng(seed)
    err = np.zeros(n)
    for i in range(n):
        b, o = _draw(rng, words, scale), np.zeros(2 * words)
        fn(b.ctypes.data_as(_D), o.ctypes.data_as(_D))
        d = _mul(_exact(o), _exact(b))  # |y - 1/b| / |1/b| = |y b - 1|
        err[i] = float((d[0] - 1) ** 2 + d[1] ** 2) ** 0.5
    return err


@pytest.mark.parametrize("scale", [0, 18, -60])
def test_double_double(lib, scale):
    e = _errors(lib.rp_dd, 2, 4000, scale, 41 + abs(scale)) * 2.0 ** 106
    assert e.max() <= 2.5 and np.sqrt(np.mean(e * e)) <= 0.3


@pytest.mark.parametrize("scale", [0, 18, -60])
def test_fp64(lib, scale):
    e = _errors(lib.rp_f64, 1, 4000, scale, 51 + abs(scale)) * 2.0 ** 53
    assert e.max() <= 1 + 2.0 ** -40 and np.sqrt(np.mean(e * e)) <= 0.5
