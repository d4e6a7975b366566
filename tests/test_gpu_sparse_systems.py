"""Systems with few terms per polynomial: workgroups that build the power table
of the polynomial's own variables only, monomials of at most two variables (no
products by the padding's 1), and the rules beside them, against the oracle
with the bars of the other evaluation tests (scaled: 1e-28 in double-double,
1e-13 in FP64); structural zeros exactly zero, values without the Jacobian bit
for bit the same.
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


def _ragged(n, n_polys, m, k, d, seed):
    """Polynomials of 0 to m monomials of 0 to k variables."""
    rng = np.random.RandomState(seed)
    polys, coefs = [], []
    for p in range(n_polys):
        monos = []
        for _ in range(m if p % 3 else rng.randint(0, m)):
            size = rng.randint(0, k + 1)
            monos.append([(int(v), int(rng.randint(1, d + 1)))
                          for v in sorted(rng.choice(n, size, replace=False))])
        polys.append(monos)
        coefs.append([complex(a) for a in np.exp(2j * np.pi * rng.uniform(size=len(monos)))])
    return synth.system_from_lists(n, polys, coefs)


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
@pytest.mark.parametrize("n,n_polys,m,k,d,P", [
    (50, 7, 5, 5, 4, 9),        # terms half the variables, one launch
    (51, 300, 5, 5, 2, 11),     # and two launches, an odd number of points
    (200, 170, 10, 5, 2, 24),   # many variables: one launch up to 4096 pairs,
    (200, 170, 10, 5, 2, 25),   # and two
    (203, 127, 10, 5, 3, 129),  # up to 16384 pairs,
    (203, 127, 10, 5, 3, 130),  # and two
    (33, 17, 1, 1, 3, 90),      # single linear or power terms
    (16, 60, 70, 2, 31, 30),    # pairs, the largest exponents, slices of 64 and 6
    (300, 3, 1100, 2, 2, 5),    # pairs, two chunks
    (450, 37, 120, 2, 2, 3),    # pairs where the general kernel is the faster
    (449, 37, 120, 2, 2, 3),    # one in double-double, and one variable fewer
])
def test_sparse_systems_match_the_oracle(n, n_polys, m, k, d, P, prec):
    s = _ragged(n, n_polys, m, k, d, seed=n + m)
    pts = [a.copy() for a in synth.points(P, n, 3 * n)]
    for a in pts:
        a[P // 2, n // 3] = 0.0   # refused where a monomial contains it
        a[P - 1, :n // 2] = 0.0
    pts = tuple(pts)
    print(f"[case] sparse n={n} polys={n_polys} m={m} k={k} d={d} P={P} prec={prec}", flush=True)
    S = pe.System.from_csr(s)
    f, J = run_eval(S, pts, prec)
    fv, _ = run_eval(S, pts, prec, with_jac=False)
    S.close()
    for q in (0, 1, 2, 3) if prec == 1 else (0, 2):
        assert np.array_equal(fv[q], f[q])
    Sf, SJ = O.scales(s, pts[0], pts[2])
    if prec == 1:
        rf, rJ = O.eval_dd(s, pts)
    else:
        rf, rJ = O.eval_f64(s, pts[0], pts[2])
        f, J = (f[0], f[2]), (J[0], J[2])
    ef, zf = scaled_err(f, rf, Sf)
    eJ, zJ = scaled_err(J, rJ, SJ)
    assert zf and zJ and max(ef, eJ) < (1e-28 if prec == 1 else 1e-13), (ef, eJ)


@pytest.mark.parametrize("P", [4, 300], ids=["one-launch", "two-launches"])
def test_non_finite_coordinates_of_other_polynomials(P):
    """A coordinate that is NaN changes no polynomial without it."""
    s = synth.regular_system(60, 3, 3, (1, 3), seed=61, n_polys=40)
    pts = [a.copy() for a in synth.points(P, 60, 62)]
    S = pe.System.from_csr(s)
    f0, J0 = run_eval(S, tuple(pts), 1)
    pts[0][1, 7] = np.nan
    f, J = run_eval(S, tuple(pts), 1)
    S.close()
    has = np.array([any(7 in s.monomial(q)[0] for q in range(int(s.poly_start[p]), int(s.poly_start[p + 1])))
                    for p in range(40)])
    assert has.any() and not has.all()
    for a, b in zip(f + J, f0 + J0):
        assert np.array_equal(a[1][..., ~has], b[1][..., ~has]) and np.array_equal(a[0], b[0])
    assert np.all(np.isnan(f[0][1][has]))
