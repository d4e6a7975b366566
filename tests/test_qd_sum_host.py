"""Quad-double sums (qd.hpp), compiled for the host, against exact rationals.

All eight words enter a sum and nothing is rounded before the last four words
are cut off, so that
  - a sum errs by at most about the last word's last bit: u^4 |a + b| where the
    four words are normalised, and at most twice that (u = 2^-53);
  - a sum whose operands cancel to 2^-80 of their size or less is exact: what is
    left spans at most 212 - 80 + 53 bits, which four words hold.
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
U4 = Fr(1, 2 ** 212)
_D = C.POINTER(C.c_double)


@pytest.fixture(scope="module")
def add():
    d = tempfile.mkdtemp(prefix="pe_qdsum_")
    so = os.path.join(d, "libqd.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-ffp-contract=off", "-fno-fast-math",
                    f"-I{CSRC}", os.path.join(ROOT, "tests", "cpp", "qd_probe.cpp"), "-o", so], check=True)
    L = C.CDLL(so)
    L.qp_add.argtypes = [_D, _D, _D]

    def f(a, b):
        o = np.zeros(4)
        L.qp_add(a.ctypes.data_as(_D), b.ctypes.data_as(_D), o.ctypes.data_as(_D))
        return o
    return f


def _rand(rng, scale=1.0):
    w = [rng.uniform(-1, 1) * scale]
    for _ in range(3):
        w.append(w[-1] * 2.0 ** -53 * rng.uniform(-1, 1))
    return np.array(w)


def _fr(w):
    return sum((Fr(float(v)) for v in w), Fr(0))


def test_sums_of_different_sizes(add):
    rng = np.random.default_rng(31)
    for _ in range(2000):
        a, b = _rand(rng), _rand(rng, 2.0 ** rng.integers(-20, 20))
        exact = _fr(a) + _fr(b)
        assert abs(_fr(add(a, b)) - exact) <= 2 * U4 * max(abs(exact), U4)


@pytest.mark.parametrize("bits", [80, 106, 120, 159])
def test_cancelling_sums_are_exact(add, bits):
    rng = np.random.default_rng(32 + bits)
    for _ in range(500):
        a = _rand(rng)
        b = -a
        # words that differ from 2^-bits of the size downwards
        for i in range(1, 4):
            if 53 * i >= bits - 53:
                b[i] += a[0] * 2.0 ** -max(bits, 53 * i) * rng.uniform(-1, 1)
        assert _fr(add(a, b)) == _fr(a) + _fr(b)
