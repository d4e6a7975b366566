"""pe_eval_jac_noalloc takes the kernels that pe_eval_jac takes for the same
call, whatever was called before: bit for bit the same results."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1201_0499_amd as pe  # noqa: E402
from gpu_helpers import alloc, dev, host, run_eval  # noqa: E402


def _noalloc(S, s, pts, prec):
    P = pts[0].shape[0]
    x, f, J = dev(pts), alloc((P, s.n_polys)), alloc((P, s.n_vars, s.n_polys))
    pe.eval_jac_noalloc(S.handle, P, x, f, J, prec)
    torch.cuda.synchronize()
    return host(f), host(J)


def _same(a, b, prec):
    for u, v in zip(a[0] + a[1], b[0] + b[1]):
        if prec == pe.PE_FP64 and np.all(np.isnan(v)):
            continue  # planes of low words
        assert np.array_equal(u.view(np.uint64), v.view(np.uint64))


@pytest.mark.parametrize("first", [1, 0], ids=["dd-first", "fp64-first"])
def test_after_a_call_in_the_other_precision(first):
    """Polynomials of 2600 monomials, whose chunks differ by precision."""
    s = synth.regular_system(40, 2600, 3, (1, 3), seed=77, n_polys=3)
    pts = synth.points(30, 40, 79)
    print(f"[case] noalloc after precision {first}", flush=True)
    S = pe.System.from_csr(s)
    run_eval(S, pts, first)
    got = _noalloc(S, s, pts, 1 - first)
    ref = run_eval(S, pts, 1 - first)
    S.close()
    _same(got, ref, 1 - first)


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
def test_after_a_call_of_fewer_points(prec):
    """Runs of 256 terms: one point goes by the general kernel, 200 in
    double-double by the quotients, under one pinned schedule."""
    s = synth.regular_system(16, 256, 16, (1, 3), seed=80)
    S = pe.System.from_csr(s)
    S.set_schedule(lanes=2, chunk_vars=8, threads=512, groups=1)
    pts = synth.points(200, 16, 81)
    print(f"[case] noalloc after one point prec={prec}", flush=True)
    run_eval(S, tuple(a[:1] for a in pts), prec)
    got = _noalloc(S, s, pts, prec)
    ref = run_eval(S, pts, prec)
    again = _noalloc(S, s, pts, prec)
    S.close()
    _same(got, ref, prec)
    _same(again, ref, prec)
