"""Both sides of the rules that choose between the evaluation's kernels, against
the oracle with the bars of the other evaluation tests (scaled: 1e-28 in
double-double, 1e-13 in FP64), and calls captured before their tables exist.
"""
import numpy as np
import pytest

import synth
from oracle import ddoracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1201_0499_amd as pe  # noqa: E402
from gpu_helpers import alloc, dev, host, run_eval, scaled_err  # noqa: E402


def _check(s, pts, f, J, prec):
    Sf, SJ = O.scales(s, pts[0], pts[2])
    if prec == 1:
        rf, rJ = O.eval_dd(s, pts)
    else:
        rf, rJ = O.eval_f64(s, pts[0], pts[2])
        f, J = (f[0], f[2]), (J[0], J[2])
    ef, zf = scaled_err(f, rf, Sf)
    eJ, zJ = scaled_err(J, rJ, SJ)
    assert zf and zJ and max(ef, eJ) < (1e-28 if prec == 1 else 1e-13), (ef, eJ)


@pytest.mark.parametrize("prec,n,n_polys,m,k,P", [
    (0, 23, 5, 300, 6, 300),   # FP64, runs of more than 64 terms: few variables,
    (0, 24, 5, 300, 6, 300),   # and one more
    (0, 32, 9, 64, 32, 20),    # a small call, runs of 64, in one pass,
    (0, 33, 9, 64, 33, 20),    # and one variable more
    (1, 11, 5, 520, 8, 300),   # double-double, many monomials, few variables,
    (1, 12, 5, 520, 8, 300),   # and one more
    (1, 16, 4, 256, 16, 1),    # runs of 256 in one pass,
    (1, 18, 4, 256, 16, 1),    # and two variables more
    (1, 20, 40, 12, 4, 32),    # 1280 pairs: one launch,
    (1, 20, 40, 12, 4, 33),    # and two
    (1, 60, 64, 40, 2, 96),    # two variables per monomial, 6144 pairs,
    (1, 60, 64, 40, 2, 97),    # and more
    (0, 260, 260, 3, 4, 40),   # fewer factors than entries of J in a row
    (0, 300, 3, 40, 6, 500),   # two points do not leave four workgroups on a CU
])
def test_rules_match_the_oracle(prec, n, n_polys, m, k, P):
    s = synth.regular_system(n, m, k, (1, 4), seed=n + m, n_polys=n_polys)
    pts = synth.points(P, n, 7 * n)
    print(f"[case] rules prec={prec} n={n} m={m} k={k} P={P}", flush=True)
    S = pe.System.from_csr(s)
    f, J = run_eval(S, pts, prec)
    fv, _ = run_eval(S, pts, prec, with_jac=False)
    S.close()
    _check(s, pts, f, J, prec)
    for q in (0, 1, 2, 3) if prec == 1 else (0, 2):
        assert np.array_equal(fv[q], f[q])


@pytest.mark.parametrize("first", [1, 0], ids=["fp64-captured-first", "dd-captured-first"])
def test_first_call_of_a_precision_under_capture(first):
    """Polynomials of 2600 monomials, whose chunks (and tables) differ between
    the precisions: the second precision is first called while a stream is
    being captured, and may neither allocate nor upload there."""
    s = synth.regular_system(40, 2600, 3, (1, 3), seed=77, n_polys=3)
    pts = synth.points(30, 40, 78)
    S = pe.System.from_csr(s)
    run_eval(S, pts, first)  # packs the schedule and this precision's tables
    prec = 1 - first
    x, f, J = dev(pts), alloc((30, 3)), alloc((30, 40, 3))
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(g, stream=side):
        pe.eval_jac(S.handle, 30, x, f, J, prec, side.cuda_stream)
    for _ in range(3):
        for a in f + J:
            a.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        _check(s, pts, host(f), host(J), prec)
        run_eval(S, pts, prec)  # eager work between the replays, by quotients
    S.close()


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
def test_batch_takes_the_same_side(prec):
    """Bitwise the same from a batch as from each system under the batch's
    schedule, for systems on either side of the rules."""
    systems = [synth.regular_system(n, m, k, (1, 3), seed=300 + n, n_polys=6)
               for n, m, k in [(16, 64, 16), (33, 64, 16), (11, 600, 8), (40, 30, 2)]]
    pps = np.array([3, 3, 40, 5], np.int64)
    pts = [synth.points(int(P), s.n_vars, 17) for P, s in zip(pps, systems)]
    handles = [pe.System.from_csr(s) for s in systems]
    B = pe.Batch(handles)
    _, fo, jo = B.layout(pps)
    x = dev(tuple(np.concatenate([p[q].reshape(-1) for p in pts]) for q in range(4)))
    f, J = alloc((int(fo[-1]),)), alloc((int(jo[-1]),))
    B.eval_jac(pps, x, f, J, prec)
    torch.cuda.synchronize()
    f, J = host(f), host(J)
    for i, (S, s) in enumerate(zip(handles, systems)):
        lanes = max(1, 1 << (-(-s.max_k // 4) - 1).bit_length())
        S.set_schedule(lanes=lanes, chunk_vars=4, threads=256, groups=1)
        fs, Js = run_eval(S, pts[i], prec)
        for q in (0, 1, 2, 3) if prec == 1 else (0, 2):
            assert np.array_equal(fs[q].reshape(-1), f[q][fo[i]:fo[i + 1]])
            assert np.array_equal(Js[q].reshape(-1), J[q][jo[i]:jo[i + 1]])
    B.close()
    for S in handles:
        S.close()
