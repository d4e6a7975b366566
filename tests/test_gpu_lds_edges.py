"""Systems whose quotient tables fill the 160 KiB of LDS exactly, in calls of
few (polynomial, point) pairs: no room for the single launch's flag, so they
take two launches.  Against the oracle (scaled: 1e-28 in double-double, 1e-58
in quad-double; in FP64 the general kernel's staging, sized for double-double,
refuses such systems).
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
from gpu_helpers import dev, run_eval, scaled_err  # noqa: E402


@pytest.mark.parametrize("n,d,m,k", [(512, 8, 512, 8), (1024, 3, 1024, 4), (1264, 3, 64, 4)])
def test_tables_that_fill_the_lds(n, d, m, k):
    s = synth.regular_system(n, m, k, (1, d), seed=n + d, n_polys=3)
    assert s.max_exp == d
    pts = [a.copy() for a in synth.points(2, n, 7)]
    for a in pts:
        a[1, 5] = 0.0  # refused where a monomial contains it
    pts = tuple(pts)
    print(f"[case] full LDS n={n} d={d} m={m}", flush=True)
    S = pe.System.from_csr(s)
    f, J = run_eval(S, pts, pe.PE_DD)
    fv, _ = run_eval(S, pts, pe.PE_DD, with_jac=False)
    S.close()
    Sf, SJ = O.scales(s, pts[0], pts[2])
    rf, rJ = O.eval_dd(s, pts)
    ef, zf = scaled_err(f, rf, Sf)
    eJ, zJ = scaled_err(J, rJ, SJ)
    assert zf and zJ and max(ef, eJ) < 1e-28, (ef, eJ)
    for a, b in zip(f, fv):
        assert np.array_equal(a, b)


def test_quad_double_tables_that_fill_the_lds():
    from test_gpu_qd import _check, _qd_points
    s = synth.regular_system(512, 512, 12, (1, 3), seed=515, n_polys=2)
    _check(s, _qd_points(1, 512, 516), polys=[1], tag="full LDS")


def test_corrector_with_one_start():
    """The all-dd corrector from one start of such a system (n = 256, d = 18)."""
    s, xstar = synth.known_root_system(256, 256, 4, (1, 18), seed=18)
    assert s.max_exp == 18
    x = dev(synth.perturbed_starts(xstar, 1, 1e-9, seed=19))
    res = torch.zeros(1, dtype=torch.float64, device="cuda")
    it = torch.zeros(1, dtype=torch.int32, device="cuda")
    st = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    print("[case] full LDS corrector", flush=True)
    S = pe.System.from_csr(s)
    code = S.newton(1, x, res, it, st, tol=1e-24, max_iter=8, mode=pe.PE_NEWTON_DD)
    torch.cuda.synchronize()
    S.close()
    assert code == 0 and int(st[0]) == 0, (res, it)
    err = O.dd_diff_abs(tuple(t.cpu().numpy() for t in x), tuple(a.reshape(1, -1) for a in xstar))
    assert np.max(err) < 1e-20
