"""The general kernel's tiles of points, staging buffers, splits over workgroups
and static scratch, in systems that the quotient kernels do not take: one
coefficient of 2^301, or an exponent of 33, is out of their range.  (Systems
within it use none of these, so that tests on those compare the quotients with
themselves.)  That this kernel ran is seen from its results: they depend on the
schedule, the quotients' do not.  Against the oracle with the bars of the other
evaluation tests.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1201_0499_amd as pe  # noqa: E402
from gpu_helpers import dev, host, run_eval  # noqa: E402
from test_gpu_tiles import _bitwise, _sweep  # noqa: E402


def _outside(s, mono=0):
    """The system with one coefficient scaled by 2^301."""
    coef = tuple(c.copy() for c in s.coef)
    for c in coef:
        c[mono] = np.ldexp(c[mono], 301)
    return synth.System(s.n_vars, s.n_polys, s.poly_start, s.mono_start, s.pos, s.exp, coef, meta=s.meta)


def _differ(s, pts, a, b, prec):
    """Whether two schedules give other bits somewhere: the general kernel ran."""
    out = []
    for sched in (a, b):
        S = pe.System.from_csr(s)
        S.set_schedule(**sched)
        f, J = run_eval(S, pts, prec)
        S.close()
        out.append((f[0], f[2], J[0], J[2]) if prec == pe.PE_FP64 else f + J)
    return not _bitwise(*out)


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
def test_tiles(prec):
    """Two chunks per polynomial, one ragged, 7 points (a ragged last tile)."""
    s = _outside(synth.regular_system(20, 37, 4, (1, 3), seed=701, n_polys=11))
    pts = synth.points(7, 20, 702)
    base = dict(lanes=2, chunk_vars=2, threads=64, groups=1)
    _sweep(s, pts, base, prec, "outside ragged")
    assert _differ(s, pts, base, dict(lanes=1, chunk_vars=4, threads=256, groups=1), prec)


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
def test_tiles_many_summation_rounds(prec):
    s = _outside(synth.regular_system(300, 40, 8, (1, 3), seed=704, n_polys=4))
    _sweep(s, synth.points(3, 300, 705), dict(lanes=2, chunk_vars=4, threads=64, groups=1), prec,
           "outside rounds", shapes=[(1, 1), (2, 2), (4, 2)])


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
def test_polynomials_split_over_workgroups(prec):
    """Partial rows and the combination, with tiles and without."""
    s = _outside(synth.paper_scale_workload()[0])
    pts = synth.points(5, s.n_vars, 703)
    base = dict(lanes=4, chunk_vars=4, threads=256)
    for groups in (2, 3, 4):
        _sweep(s, pts, dict(base, groups=groups), prec, f"outside split {groups}",
               polys=[0, 1, 63, 64, 100, 127], shapes=[(1, 1), (2, 2), (4, 1)])
    assert _differ(s, pts, dict(base, groups=1), dict(base, groups=2), prec)


def test_newton_mask_under_tiles():
    """A constant folded into the value's accumulator and Newton's start mask:
    an exponent of e + 32 leaves the root at fourth roots of unity."""
    s, xstar = synth.known_root_system(24, 40, 5, (1, 3), seed=706)
    s.exp[3] += 32
    assert s.max_exp >= 33
    starts = synth.perturbed_starts(xstar, 13, 1e-7, seed=707)
    outs = []
    for T, nbuf in ((1, 1), (4, 2), (3, 1)):
        S = pe.System.from_csr(s)
        S.set_schedule(lanes=2, chunk_vars=4, threads=64, groups=1, tile_points=T, stage_buffers=nbuf)
        x = dev(starts)
        res = torch.zeros(13, dtype=torch.float64, device="cuda")
        it = torch.zeros(13, dtype=torch.int32, device="cuda")
        st = torch.zeros(13, dtype=torch.int32, device="cuda")
        code = S.newton(13, x, res, it, st, tol=1e-28, max_iter=12, mode=pe.PE_NEWTON_MIXED)
        torch.cuda.synchronize()
        outs.append((host(x), it.cpu().numpy(), st.cpu().numpy()))
        S.close()
        print(f"[case] outside newton T={T} nbuf={nbuf}: code {code}, iterations "
              f"{np.bincount(outs[-1][1]).tolist()}", flush=True)
        assert code == 0 and np.all(outs[-1][2] == 0)
    for x, it, st in outs[1:]:
        assert _bitwise(x, outs[0][0]) and np.array_equal(it, outs[0][1])


@pytest.mark.parametrize("P", [1, 48], ids=["split", "whole"])
def test_quad_double(P):
    """At one point three polynomials are split over four workgroups each."""
    from test_gpu_qd import _check, _qd_points
    s = _outside(synth.regular_system(10, 600, 6, (1, 3), seed=710, n_polys=3), mono=650)
    _check(s, _qd_points(P, 10, 711), polys=[0, 1], tag=f"outside P={P}", points=[0, P - 1])


@pytest.mark.parametrize("prec", [1, 0], ids=["dd", "fp64"])
def test_partial_rows_in_the_static_scratch(prec):
    """The allocation-free call with a split schedule: 3 points, then 1."""
    from test_zz_no_alloc import _case
    s = _outside(synth.paper_scale_workload()[0])
    S = pe.System.from_csr(s)
    S.set_schedule(lanes=4, chunk_vars=4, threads=512, groups=2)
    for P, seed in ((3, 77), (1, 78)):
        _case(S, s, synth.points(P, s.n_vars, seed), prec, f"outside groups=2 P={P}")
    S.close()
