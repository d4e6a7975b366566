"""GPU parity of the quotient kernels and of their hand-over to the general
kernel (needs an MI355X).

The quotient kernels refuse polynomials that contain a coordinate of zero, of
a magnitude outside a window or not finite, or a product outside its range;
the general kernel evaluates those, under every schedule.  Each case mixes
ordinary points with such points, in calls of few (polynomial, point) pairs
(one launch) and of many (two launches), and compares every output with the
oracle: 1e-28 scaled in double-double, 1e-13 in FP64, 1e-58 in quad-double;
structural zeros exactly zero.
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
from gpu_helpers import dev, host, run_eval, scaled_err  # noqa: E402

BAR = {pe.PE_DD: 1e-28, pe.PE_FP64: 1e-13}


def _ragged(n, n_polys, m, k, d, seed):
    rng = np.random.RandomState(seed)
    polys, coefs = [], []
    for p in range(n_polys):
        monos = []
        for _ in range(m if p % 5 else max(1, m // 3)):
            size = rng.randint(0, k + 1)
            monos.append([(int(v), int(rng.randint(1, d + 1)))
                          for v in sorted(rng.choice(n, size, replace=False))])
        polys.append(monos)
        coefs.append([complex(a) for a in np.exp(2j * np.pi * rng.uniform(size=len(monos)))])
    return synth.system_from_lists(n, polys, coefs)


def _points(n, P, seed, d):
    """Unit-circle points; every third has a coordinate of zero, every
    seventh one far below and every fifth one far above the window."""
    pts = [a.copy() for a in synth.points(P, n, seed)]
    rng = np.random.RandomState(seed)
    for p in range(P):
        i = rng.randint(n)
        if p % 3 == 1:
            for a in pts:
                a[p, i] = 0.0
        if p % 7 == 2:
            for a in pts:
                a[p, i] = np.ldexp(a[p, i], -70)
        if p % 5 == 3:
            for a in pts:
                a[p, i] = np.ldexp(a[p, i], 70 if d <= 3 else 24)
    return tuple(pts)


def _check(s, pts, f, J, prec, tag):
    Sf, SJ = O.scales(s, pts[0], pts[2])
    if prec == pe.PE_DD:
        rf, rJ = O.eval_dd(s, pts)
    else:
        rf, rJ = O.eval_f64(s, pts[0], pts[2])
        f, J = (f[0], f[2]), (J[0], J[2])
    ef, zf = scaled_err(f, rf, Sf)
    eJ, zJ = scaled_err(J, rJ, SJ)
    print(f"[err] quotient {tag}: f {ef:.3e}, J {eJ:.3e}", flush=True)
    assert zJ and ef < BAR[prec] and eJ < BAR[prec], (ef, eJ)


SCHEDULES = [None, dict(lanes=4, chunk_vars=2, threads=64, groups=1),
             dict(lanes=2, chunk_vars=4, threads=128, groups=2),
             dict(lanes=1, chunk_vars=8, threads=64, groups=3, tile_points=2, stage_buffers=2)]


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
@pytest.mark.parametrize("n,n_polys,m,k,d,P", [
    (9, 7, 30, 7, 3, 11),       # few pairs: one launch
    (20, 40, 70, 8, 2, 31),     # many pairs, slices of 64 and 6 monomials, an odd number of points
    (33, 17, 150, 6, 31, 40),   # largest exponents: the narrowest window
    (16, 9, 1100, 5, 4, 60),    # two chunks per polynomial
])
def test_refused_points_match_the_oracle(n, n_polys, m, k, d, P, prec):
    s = _ragged(n, n_polys, m, k, d, seed=n + m)
    pts = _points(n, P, 31 * n, d)
    for sched in SCHEDULES:
        print(f"[case] quotient n={n} m={m} d={d} P={P} prec={prec} schedule={sched}", flush=True)
        S = pe.System.from_csr(s)
        if sched:
            S.set_schedule(**sched)
        f, J = run_eval(S, pts, prec)
        fv, _ = run_eval(S, pts, prec, with_jac=False)
        S.close()
        _check(s, pts, f, J, prec, f"n={n} d={d} {sched}")
        for q in (0, 1, 2, 3) if prec == pe.PE_DD else (0, 2):
            assert np.array_equal(fv[q], f[q])  # the same sums without the Jacobian


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
@pytest.mark.parametrize("P", [3, 90], ids=["one-launch", "two-launches"])
def test_products_out_of_range(P, prec):
    """Coordinates inside the window whose products leave +-2^300: magnitudes
    of 2^13 and 2^-13 in monomials of 30 variables."""
    s = synth.regular_system(40, 20, 30, (1, 2), seed=91, n_polys=12)
    pts = [a.copy() for a in synth.points(P, 40, 92)]
    for p in range(P):
        e = {0: 13, 1: -9, 2: 0}[p % 3]
        for q, a in enumerate(pts):
            a[p] = np.ldexp(a[p], e)
    pts = tuple(pts)
    S = pe.System.from_csr(s)
    f, J = run_eval(S, pts, prec)
    S.close()
    _check(s, pts, f, J, prec, f"products P={P}")


def test_non_finite_coordinates():
    """NaN and infinity reach the polynomials that contain the coordinate and
    no others; other points are unaffected."""
    s = _ragged(12, 60, 20, 4, 3, seed=5)
    for P in (5, 40):
        pts = [a.copy() for a in synth.points(P, 12, 6)]
        pts[0][1, 3], pts[2][P - 1, 7] = np.nan, np.inf
        S = pe.System.from_csr(s)
        f, J = run_eval(S, tuple(pts), pe.PE_DD)
        S.close()
        has = np.zeros((60, 12), bool)
        for p in range(60):
            for q in range(int(s.poly_start[p]), int(s.poly_start[p + 1])):
                has[p, s.monomial(q)[0]] = True
        for pt, i in ((1, 3), (P - 1, 7)):
            assert np.array_equal(np.isfinite(f[0][pt]) & np.isfinite(f[2][pt]), ~has[:, i])
            for p in np.nonzero(~has[:, i])[0]:
                assert np.all(np.isfinite(J[0][pt, :, p])) and np.all(J[0][pt, i, p] == 0)
        good = np.array([p for p in range(P) if p not in (1, P - 1)])
        sub = tuple(a[good] for a in pts)
        _check(s, sub, tuple(a[good] for a in f), tuple(a[good] for a in J), pe.PE_DD, f"finite P={P}")


def test_batch_with_refused_points():
    """A batch of three systems, one of them with exponents outside the
    quotient kernels, at points of which some are refused."""
    shapes = [(9, 8, 40, 6, 3), (14, 14, 90, 5, 40), (25, 20, 130, 8, 2)]
    syss = [_ragged(*sh, seed=7 + i) for i, sh in enumerate(shapes)]
    P = [5, 3, 8]
    pts = [_points(s.n_vars, p, 50 + i, 4) if i != 1 else synth.points(p, s.n_vars, 51)
           for i, (s, p) in enumerate(zip(syss, P))]
    handles = [pe.System.from_csr(s) for s in syss]
    B = pe.Batch(handles)
    for prec in (pe.PE_DD, pe.PE_FP64):
        pps = np.array(P, np.int64)
        _, fo, jo = B.layout(pps)
        x = dev(tuple(np.concatenate([p[q].reshape(-1) for p in pts]) for q in range(4)))
        f = tuple(torch.full((int(fo[-1]),), float("nan"), dtype=torch.float64, device="cuda") for _ in range(4))
        J = tuple(torch.full((int(jo[-1]),), float("nan"), dtype=torch.float64, device="cuda") for _ in range(4))
        B.eval_jac(pps, x, f, J, prec)
        torch.cuda.synchronize()
        fh, Jh = host(f), host(J)
        for i, s in enumerate(syss):
            _check(s, pts[i], tuple(a[fo[i]:fo[i + 1]].reshape(P[i], s.n_polys) for a in fh),
                   tuple(a[jo[i]:jo[i + 1]].reshape(P[i], s.n_vars, s.n_polys) for a in Jh), prec,
                   f"batch system {i} prec={prec}")
    B.close()
    for h in handles:
        h.close()


@pytest.mark.parametrize("P", [2, 60], ids=["one-launch", "two-launches"])
def test_quad_double_refused_points(P):
    """Quad-double with zero coordinates, against the exact evaluation."""
    from test_gpu_qd import _check as check_qd, _qd_points
    s = _ragged(10, 9, 25, 6, 4, seed=77)
    planes = [a.copy() for a in _qd_points(P, 10, 78)]
    for a in planes:
        a[1::2, 4] = 0.0
    check_qd(s, planes, polys=[1, 5], tag=f"refused P={P}", points=sorted({0, 1, P - 1}))
