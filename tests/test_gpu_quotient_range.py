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
