"""Calls of more points than one grid has work-items: the kernels' workgroups
stride over them, or the launch is cut in pieces.  Against torch in FP64, with
errors of a few roundings of the magnitudes.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1201_0499_amd as pe  # noqa: E402


def test_points_past_the_grid():
    """f = c0 x + c1 x^3 in FP64 at 2^27 + 2^11 + 3 points: two points a
    workgroup of 64 lanes, more than 2^32 work-items."""
    P = 2 ** 27 + 2 ** 11 + 3
    c0, c1 = 0.6 + 0.8j, -0.8 + 0.6j
    S = pe.System.from_csr(synth.system_from_lists(1, [[[(0, 1)], [(0, 3)]]], [[c0, c1]]))
    a = torch.rand(P, 1, dtype=torch.float64, device="cuda") * 6.28
    x = (torch.cos(a), None, torch.sin(a), None)
    del a
    f = tuple(torch.full((P, 1), 7.0, dtype=torch.float64, device="cuda") if q % 2 == 0 else None for q in range(4))
    J = tuple(torch.full((P, 1, 1), 7.0, dtype=torch.float64, device="cuda") if q % 2 == 0 else None for q in range(4))
    print(f"[case] grid limit P={P}", flush=True)
    S.eval_jac(P, x, f, J, pe.PE_FP64)
    torch.cuda.synchronize()
    S.close()
    u = 2.0 ** -53
    step = 2 ** 24
    for i in range(0, P, step):
        z = torch.complex(x[0][i:i + step], x[2][i:i + step])
        got = torch.complex(f[0][i:i + step], f[2][i:i + step])
        assert float((got - (c0 * z + c1 * z ** 3)).abs().max()) < 64 * u
        got = torch.complex(J[0][i:i + step], J[2][i:i + step])[:, 0]
        assert float((got - (c0 + 3 * c1 * z ** 2)).abs().max()) < 128 * u


def test_starts_past_the_grid_of_the_elimination():
    """c0 x + c1 = 0 by the all-dd corrector from 2^23 + 5 starts: the
    elimination's workgroups of 512 lanes take more than 2^32 work-items."""
    P = 2 ** 23 + 5
    c0, c1 = 0.6 + 0.8j, 1.0 + 0.5j
    S = pe.System.from_csr(synth.system_from_lists(1, [[[(0, 1)], []]], [[c0, c1]]))
    g = torch.Generator(device="cuda").manual_seed(5)
    x = tuple(torch.rand(P, 1, dtype=torch.float64, device="cuda", generator=g) if q % 2 == 0
              else torch.zeros(P, 1, dtype=torch.float64, device="cuda") for q in range(4))
    res = torch.zeros(P, dtype=torch.float64, device="cuda")
    it = torch.zeros(P, dtype=torch.int32, device="cuda")
    st = torch.full((P,), 7, dtype=torch.int32, device="cuda")
    print(f"[case] grid limit of the elimination, {P} starts", flush=True)
    code = S.newton(P, x, res, it, st, tol=1e-24, max_iter=3, mode=pe.PE_NEWTON_DD)
    torch.cuda.synchronize()
    S.close()
    assert code == 0 and int(st.abs().max()) == 0 and int(it.max()) == 1
    root = -c1 / c0
    assert float((torch.complex(x[0], x[2]) - root).abs().max()) < 8 * 2.0 ** -53
