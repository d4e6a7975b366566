"""Host packer of the quotient kernels (quotient_tables.cpp), checked on the CPU.

f and J are evaluated in numpy by walking the tables the way the kernels do
(monomial values from the slices' words, then every output's run), and
compared with the definition; on the way every index is checked against the
size of what it reads.  The systems have empty polynomials, constants, ragged
monomials, several chunks per polynomial and sizes next to a slice of 64
monomials and a block of 16 outputs.
"""
import ctypes as C
import os
import subprocess
import tempfile

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1201_0499_amd", "csrc")
QUAD, PARTS, BLOCK, BITS = 4, 4, 16, 11
DT = [np.uint16, np.int32, np.int32, np.int32, np.int32, np.int32, np.uint16, np.uint16]
NAMES = ["words", "mono", "slice", "chunk", "poly", "block", "runs", "out"]


@pytest.fixture(scope="module")
def probe():
    d = tempfile.mkdtemp(prefix="pe_quot_")
    so = os.path.join(d, "libquot.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}",
                    os.path.join(ROOT, "tests", "cpp", "quotient_probe.cpp"),
                    os.path.join(CSRC, "quotient_tables.cpp"), "-o", so], check=True)
    L = C.CDLL(so)
    L.qt_build.restype = C.c_void_p
    L.qt_build.argtypes = [C.c_int32, C.c_int32, C.c_int64] + [C.c_void_p] * 4 + [
        C.c_int, C.POINTER(C.c_int), C.POINTER(C.c_int64)]
    L.qt_table.restype = C.c_int64
    L.qt_table.argtypes = [C.c_void_p, C.c_int, C.c_void_p]
    L.qt_free.argtypes = [C.c_void_p]
    L.qt_chunk.argtypes = [C.c_int, C.c_int, C.c_int, C.c_int64, C.c_int]
    L.qt_lds.restype = C.c_int64
    return L


def _tables(L, s, CH):
    a = [np.ascontiguousarray(v, t) for v, t in ((s.poly_start, np.int64), (s.mono_start, np.int64),
                                                 (s.pos, np.int32), (s.exp, np.int32))]
    pad, max_m = C.c_int(), C.c_int64()
    h = L.qt_build(s.n_vars, s.n_polys, s.n_monos, *[v.ctypes.data for v in a], CH, C.byref(pad),
                   C.byref(max_m))
    assert h
    t = dict(pad=pad.value, max_m=max_m.value)
    for w, (name, dt) in enumerate(zip(NAMES, DT)):
        t[name] = np.zeros(L.qt_table(h, w, None), dt)
        L.qt_table(h, w, t[name].ctypes.data)
    t["n_blk"], t["multi"] = L.qt_table(h, 8, None), L.qt_table(h, 9, None)
    L.qt_free(h)
    return t


def _walk(s, t, CH, x, coef):
    """f and J as the kernels form them."""
    n, d = s.n_vars, s.max_exp
    u = np.concatenate([x ** e for e in range(1, d + 1)] + ([[1.0]] if t["pad"] else []))
    f = np.zeros(s.n_polys, complex)
    J = np.zeros((n, s.n_polys), complex)
    n_rank = t["n_blk"] * BLOCK
    runs = t["runs"].reshape(-1, BLOCK, PARTS)
    seen = []
    for p in range(s.n_polys):
        c0, c1, fold, _ = t["poly"][4 * p:4 * p + 4]
        if fold:
            assert s.mono_start[fold] == s.mono_start[fold - 1]
            f[p] += coef[fold - 1]
            seen.append(fold - 1)
        assert t["multi"] or c1 - c0 <= 1
        for c in range(c0, c1):
            first, cnt, sl0, blk0 = t["chunk"][4 * c:4 * c + 4]
            assert 0 < cnt <= CH
            V = np.full(CH, 7.0 + 0j)
            V[cnt:] = np.nan
            for i in range(cnt):
                w0, quads = t["slice"][2 * (sl0 + i // 64):2 * (sl0 + i // 64) + 2]
                sc = min(64, cnt - i // 64 * 64)
                idx = (w0 + np.arange(quads) * sc + i % 64)[:, None] * QUAD + np.arange(QUAD)
                assert quads == 0 or idx.max() < t["words"].size
                w = t["words"][idx.astype(int)].reshape(-1)
                assert w.size == 0 or w.max() < u.size
                V[i] = coef[t["mono"][first + i]] * np.prod(u[w])
                seen.append(t["mono"][first + i])
            f[p] += V[:cnt].sum()
            outs = t["out"][c * n_rank:(c + 1) * n_rank]
            assert sorted(outs[:n]) == list(range(n)) and np.all(outs[n:] == 0xFFFF)
            last = None
            for b in range(t["n_blk"]):
                row0, rows = t["block"][2 * (blk0 + b):2 * (blk0 + b) + 2]
                assert row0 + rows <= runs.shape[0] and (last is None or rows <= last)
                last = rows
                for r in range(BLOCK):
                    e = runs[row0:row0 + rows, r].reshape(-1).astype(int)
                    v = e & ((1 << BITS) - 1)
                    assert v.size == 0 or v.max() < cnt
                    live = v[e >> BITS > 0]
                    assert np.unique(live).size == live.size
                    o = outs[b * BLOCK + r]
                    if o == 0xFFFF:
                        assert live.size == 0
                    else:
                        J[o, p] += np.sum((e >> BITS) * V[v]) / x[o]
    assert sorted(seen) == list(range(s.n_monos))
    return f, J


def _define(s, x, coef):
    f = np.zeros(s.n_polys, complex)
    J = np.zeros((s.n_vars, s.n_polys), complex)
    for p in range(s.n_polys):
        for q in range(int(s.poly_start[p]), int(s.poly_start[p + 1])):
            pos, ex = s.monomial(q)
            f[p] += coef[q] * np.prod(x[pos] ** ex)
            for j, i in enumerate(pos):
                e = ex.copy()
                e[j] -= 1
                J[i, p] += coef[q] * ex[j] * np.prod(x[pos] ** e)
    return f, J


def _ragged(n, ms, k, d, seed):
    rng = np.random.RandomState(seed)
    polys, coefs = [], []
    for m in ms:
        monos = []
        for _ in range(m):
            size = rng.randint(0, k + 1)
            monos.append([(int(v), int(rng.randint(1, d + 1)))
                          for v in sorted(rng.choice(n, size, replace=False))])
        polys.append(monos)
        coefs.append([complex(a) for a in np.exp(2j * np.pi * rng.uniform(size=m))])
    return synth.system_from_lists(n, polys, coefs)


@pytest.mark.parametrize("n,ms,k,d,CH", [
    (5, (0, 1, 3, 64, 65), 4, 3, 64),
    (15, (130, 63, 128), 9, 2, 64),
    (16, (200, 2), 16, 5, 128),
    (17, (191, 193), 13, 31, 192),
    (40, (100,), 33, 4, 128),
])
def test_tables_evaluate_to_the_definition(probe, n, ms, k, d, CH):
    s = _ragged(n, ms, k, d, seed=n)
    t = _tables(probe, s, CH)
    rng = np.random.RandomState(n + 1)
    x = np.exp(2j * np.pi * rng.uniform(size=n))
    coef = s.coef[0] + 1j * s.coef[2]
    assert t["max_m"] == max(np.diff(s.poly_start) - [any(s.mono_start[q + 1] == s.mono_start[q]
                             for q in range(s.poly_start[p], s.poly_start[p + 1])) for p in range(len(ms))])
    f, J = _walk(s, t, CH, x, coef)
    f0, J0 = _define(s, x, coef)
    # sums of at most max(ms) terms of modulus <= d, each with at most k + d roundings
    tol = 2.0 ** -52 * (max(ms) + k + d) * max(ms) * d * 4
    assert np.max(np.abs(f - f0)) < tol and np.max(np.abs(J - J0)) < tol
    assert np.all(J[J0 == 0] == 0)


def test_regular_quads_need_no_pad(probe):
    """A regular system whose monomials have a multiple of four variables
    (and one constant each) has no entry 1 in its power table."""
    s = synth.known_root_system(20, 70, 8, (1, 3), seed=5)[0]
    t = _tables(probe, s, 128)
    assert not t["pad"] and t["max_m"] == 70
    x = np.exp(2j * np.pi * np.random.RandomState(6).uniform(size=20))
    coef = s.coef[0] + 1j * s.coef[2]
    f, J = _walk(s, t, 128, x, coef)
    f0, J0 = _define(s, x, coef)
    assert max(np.max(np.abs(f - f0)), np.max(np.abs(J - J0))) < 2.0 ** -52 * 4 * 82 * 71 * 3


@pytest.mark.parametrize("words", [2, 4, 8])
def test_chunks_fit_the_lds(probe, words):
    """The chunk is a multiple of 64 that fits (at most 1024), and 0 where
    not even 64 monomials fit or the system is outside the packing."""
    for n, d, m in ((1, 1, 1), (8, 2, 8), (128, 3, 256), (128, 3, 257), (512, 5, 1024), (300, 4, 5000),
                    (512, 9, 1024), (40, 31, 100)):
        ch = probe.qt_chunk(n, d, 1, m, words)
        if ch:
            assert ch % 64 == 0 and 64 <= ch <= 1024 and ch >= min(m, 64)
            assert probe.qt_lds(n, d, 1, ch, int(ch < m), 1, words) <= 160 * 1024
        else:
            assert probe.qt_lds(n, d, 1, 64, int(64 < m), 1, words) > 160 * 1024
    # two buffers of the largest system's values fill the LDS exactly
    assert probe.qt_lds(512, 5, 0, 1024, 0, 2, 4) == 160 * 1024
    assert probe.qt_chunk(40, 32, 1, 100, words) == 0     # exponents past the entry's five bits
    assert probe.qt_chunk(70000, 1, 1, 100, words) == 0   # table entries past 16 bits
    for d in range(1, 32):
        b = probe.qt_point_exp(d)
        assert 2 <= b <= 60 and 4 * d * (b + 0.5) <= 400
