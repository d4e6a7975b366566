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


def _oracle(s, pts, f, J):
    Sf, SJ = O.scales(s, pts[0], pts[2])
    rf, rJ = O.eval_dd(s, pts)
    ef, zf = scaled_err(f, rf, Sf)
    eJ, zJ = scaled_err(J, rJ, SJ)
    assert zf and zJ and max(ef, eJ) < 1e-28, (ef, eJ)


def long_run_system(n, m, k, d, n_polys, seed):
    """Monomials that all contain variable 0: the general kernel's row tables
    are as long as its chunks."""
    rng = np.random.RandomState(seed)
    polys, coefs = [], []
    for _ in range(n_polys):
        polys.append([[(0, int(rng.randint(1, 4)))] +
                      [(int(v), int(rng.randint(1, d + 1))) for v in sorted(rng.choice(n - 1, k - 1, replace=False) + 1)]
                      for _ in range(m)])
        coefs.append([complex(a) for a in np.exp(2j * np.pi * rng.uniform(size=m))])
    s = synth.system_from_lists(n, polys, coefs)
    assert s.max_exp == d
    return s


def test_general_stages_that_fill_the_lds():
    """163,812 of 163,840 bytes for the general kernel that serves what the
    quotients refuse: it has no static LDS."""
    s = long_run_system(382, 64, 8, 12, 4, 900)
    P = 330
    pts = [a.copy() for a in synth.points(P, 382, 902)]
    for a in pts:
        a[3, 11] = a[7, 0] = 0.0
    pts = tuple(pts)
    print("[case] full LDS general", flush=True)
    S = pe.System.from_csr(s)
    S.set_schedule(lanes=1, chunk_vars=8, threads=64, groups=1)
    f, J = run_eval(S, pts, pe.PE_DD)
    S.close()
    keep = [0, 3, 7, P - 1]
    _oracle(s, tuple(a[keep] for a in pts), tuple(a[keep] for a in f), tuple(a[keep] for a in J))


def test_batch_that_fills_the_lds():
    """163,748 bytes for a system of a batch under the default configuration."""
    s = long_run_system(337, 256, 4, 12, 5, 901)
    pts = [a.copy() for a in synth.points(3, 337, 903)]
    for a in pts:
        a[1, 0] = 0.0
    S = pe.System.from_csr(s)
    B = pe.Batch([S])
    cfg = B.config()
    assert (cfg["chunk_vars"], cfg["threads"], cfg["lanes_mult"]) == (4, 256, 1)
    f = tuple(torch.full((15,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(4))
    J = tuple(torch.full((3 * 337 * 5,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(4))
    print("[case] full LDS batch", flush=True)
    B.eval_jac(np.array([3], np.int64), dev(tuple(a.reshape(-1) for a in pts)), f, J, pe.PE_DD)
    torch.cuda.synchronize()
    B.close()
    S.close()
    _oracle(s, tuple(pts), tuple(t.cpu().numpy().reshape(3, 5) for t in f),
            tuple(t.cpu().numpy().reshape(3, 337, 5) for t in J))


def test_residual_that_fills_the_lds():
    """All 163,840 bytes for the power table of the quad-double residual (n =
    255, d = 10), whose kernel has no static LDS either."""
    from test_gpu_newton_qd import _run
    s, xstar = synth.known_root_system(255, 12, 4, (1, 10), seed=904, coef_grid=40)
    assert s.max_exp == 10
    print("[case] full LDS residual", flush=True)
    _, res, _, st, code = _run(s, synth.perturbed_starts(xstar, 2, 1e-9, seed=905), tol=1e-50, max_iter=12)
    assert code == 0 and np.all(st == 0) and np.all(res <= 1e-50)
