"""Points with a coordinate out of the quotients' window, in systems whose
polynomials contain every variable (refused before the work on them), most or
few: against the oracle (scaled: 1e-28 in double-double, 1e-13 in FP64), values
bit for bit the same without the Jacobian and in calls of other sizes, and the
other points bit for bit what they are without them.
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


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
@pytest.mark.parametrize("n,n_polys,m,k,P", [
    (20, 9, 40, 8, 7),       # one launch
    (20, 30, 40, 8, 71),     # two launches
    (21, 130, 8, 8, 140),    # some polynomials without some variable
    (8, 2040, 9, 3, 70),     # more than 64 points per repairing workgroup
    (20, 11, 1100, 5, 200),  # two chunks
    (70, 20, 100, 3, 1),     # more than one wave of coordinates
    (70, 20, 100, 3, 150),
])
def test_refused_points(n, n_polys, m, k, P, prec):
    s = synth.regular_system(n, m, k, (1, 3), seed=n + m, n_polys=n_polys)
    good = synth.points(P, n, 501)
    pts = [a.copy() for a in good]
    bad = sorted({0, P // 3, P - 1} | set(range(4, P, 5)))
    for p in bad:
        for a in pts:
            a[p, (7 * p) % n] = 0.0
    pts = tuple(pts)
    print(f"[case] refused points n={n} polys={n_polys} m={m} P={P} prec={prec}", flush=True)
    S = pe.System.from_csr(s)
    S.set_schedule(lanes=1, chunk_vars=8, threads=256, groups=1)
    f, J = run_eval(S, pts, prec)
    fv, _ = run_eval(S, pts, prec, with_jac=False)
    f0, J0 = run_eval(S, good, prec)
    f1, J1 = run_eval(S, tuple(a[:1] for a in pts), prec)
    S.close()
    rest = [p for p in range(P) if p not in bad]
    for q in (0, 1, 2, 3) if prec == 1 else (0, 2):
        assert np.array_equal(fv[q], f[q])
        assert np.array_equal(f1[q][0], f[q][0]) and np.array_equal(J1[q][0], J[q][0])
        assert np.array_equal(f[q][rest], f0[q][rest]) and np.array_equal(J[q][rest], J0[q][rest])
    sel = bad[:6] + bad[-2:]
    pts = tuple(a[sel] for a in pts)
    f, J = tuple(a[sel] for a in f), tuple(a[sel] for a in J)
    Sf, SJ = O.scales(s, pts[0], pts[2])
    if prec == 1:
        rf, rJ = O.eval_dd(s, pts)
    else:
        rf, rJ = O.eval_f64(s, pts[0], pts[2])
        f, J = (f[0], f[2]), (J[0], J[2])
    ef, zf = scaled_err(f, rf, Sf)
    eJ, zJ = scaled_err(J, rJ, SJ)
    assert zf and zJ and max(ef, eJ) < (1e-28 if prec == 1 else 1e-13), (ef, eJ)


@pytest.mark.parametrize("mode", [0, 1], ids=["mixed", "dd"])
def test_starts_with_a_zero_coordinate(mode):
    """One Newton step from 90 starts, some of them with a zero coordinate and
    some converged already (masked), against each start alone."""
    s, xstar = synth.known_root_system(24, 40, 6, (1, 3), seed=502)
    x0 = [a.copy() for a in synth.perturbed_starts(xstar, 90, 1e-3, seed=503)]
    for p in range(0, 90, 7):
        for a in x0:
            a[p, p % 24] = 0.0
    for p in range(3, 90, 10):
        for q in range(4):
            x0[q][p] = xstar[q]

    def run(S, idx):
        x = dev(tuple(a[idx] for a in x0))
        res = torch.zeros(len(idx), dtype=torch.float64, device="cuda")
        it = torch.zeros(len(idx), dtype=torch.int32, device="cuda")
        st = torch.zeros(len(idx), dtype=torch.int32, device="cuda")
        S.newton(len(idx), x, res, it, st, tol=1e-26, max_iter=1, mode=mode)
        torch.cuda.synchronize()
        return host(x), it.cpu().numpy(), st.cpu().numpy()

    S = pe.System.from_csr(s)
    S.set_schedule(lanes=1, chunk_vars=8, threads=64, groups=1)
    x, it, st = run(S, list(range(90)))
    print(f"[case] starts with a zero coordinate mode={mode}: iterations {np.bincount(it).tolist()}", flush=True)
    for p in (0, 1, 3, 7, 13, 84, 89):
        x1, it1, st1 = run(S, [p])
        assert it1[0] == it[p] and st1[0] == st[p]
        for a, b in zip(x1, x):
            assert np.array_equal(a[0], b[p])
    S.close()
