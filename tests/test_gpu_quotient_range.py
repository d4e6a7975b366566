"""The range rules of the quotient kernels refuse the same (polynomial, point)
pairs however a call is launched: values and Jacobians of one point equal those
of the same point among many, bit for bit, and meet the oracle's bars (scaled:
1e-28 in double-double, 1e-13 in FP64).
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
from gpu_helpers import run_eval, scaled_err  # noqa: E402


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
@pytest.mark.parametrize("scale", [17, -17], ids=["large", "small"])
def test_single_quads_near_the_limit(scale, prec):
    """Monomials of four variables (one quad) with products of 2^272 to
    2^340: four lanes per monomial at one point, one lane at 200."""
    s = synth.regular_system(8, 16, 4, (4, 5), seed=401)
    pts = tuple(np.ldexp(a, scale) for a in synth.points(1, 8, 402))
    many = tuple(np.repeat(a, 200, axis=0) for a in pts)
    print(f"[case] single quads 2^{scale} prec={prec}", flush=True)
    S = pe.System.from_csr(s)
    f, J = run_eval(S, pts, prec)
    fm, Jm = run_eval(S, many, prec)
    S.close()
    for q in (0, 1, 2, 3) if prec == 1 else (0, 2):
        assert np.array_equal(np.repeat(f[q], 200, axis=0), fm[q])
        assert np.array_equal(np.repeat(J[q], 200, axis=0), Jm[q])
    Sf, SJ = O.scales(s, pts[0], pts[2])
    if prec == 1:
        rf, rJ = O.eval_dd(s, pts)
    else:
        rf, rJ = O.eval_f64(s, pts[0], pts[2])
        f, J = (f[0], f[2]), (J[0], J[2])
    ef, _ = scaled_err(f, rf, Sf)
    eJ, zJ = scaled_err(J, rJ, SJ)
    assert zJ and max(ef, eJ) < (1e-28 if prec == 1 else 1e-13), (ef, eJ)


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
@pytest.mark.parametrize("P", [6, 150], ids=["one-launch", "two-launches"])
@pytest.mark.parametrize("k,d,lo,hi", [
    (4, 31, -6, 8),    # quads from 2^-744 to 2^992
    (8, 31, -3, 4),    # pairs of quads that leave the range and come back
    (16, 16, -3, 3),
    (2, 31, -8, 9),    # pairs; magnitudes up to and past the window
    (9, 6, -16, 16),   # the smallest exponent with checked quads
])
def test_high_exponents_at_spread_magnitudes(k, d, lo, hi, P, prec):
    """Exponents with checked quads, at coordinates of magnitudes 2^lo to 2^hi,
    one of them zero."""
    s = synth.regular_system(20, 24, k, (1, d), seed=410 + k, n_polys=11)
    rng = np.random.RandomState(411)
    e = rng.randint(lo, hi + 1, (P, 20))
    pts = [np.ldexp(a, e) for a in synth.points(P, 20, 412)]
    for a in pts:
        a[P // 2, 3] = 0.0
    pts = tuple(pts)
    print(f"[case] spread magnitudes k={k} d={d} P={P} prec={prec}", flush=True)
    S = pe.System.from_csr(s)
    f, J = run_eval(S, pts, prec)
    fv, _ = run_eval(S, pts, prec, with_jac=False)
    S.close()
    for q in (0, 1, 2, 3) if prec == 1 else (0, 2):
        assert np.array_equal(fv[q], f[q])
    Sf, SJ = O.scales(s, pts[0], pts[2])
    # outputs whose terms could overflow or lose their low words to underflow
    # in any evaluation are left out
    okf = (Sf < 2.0 ** 1000) & (Sf > 2.0 ** -700)
    okJ = ((SJ < 2.0 ** 1000) & (SJ > 2.0 ** -700)) | (SJ == 0)
    assert okf.mean() > 0.5 and okJ.mean() > 0.5
    if prec == 1:
        rf, rJ = O.eval_dd(s, pts)
    else:
        rf, rJ = O.eval_f64(s, pts[0], pts[2])
        f, J = (f[0], f[2]), (J[0], J[2])
    ef, _ = scaled_err(tuple(a[okf] for a in f), tuple(a[okf] for a in rf), Sf[okf])
    eJ, zJ = scaled_err(tuple(a[okJ] for a in J), tuple(a[okJ] for a in rJ), SJ[okJ])
    assert zJ and max(ef, eJ) < (1e-28 if prec == 1 else 1e-13), (ef, eJ)
