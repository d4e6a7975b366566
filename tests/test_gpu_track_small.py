"""GPU tracker of small systems (one wave per path) at the edges of its range
(needs an MI355X).

Systems of 1 to 16 variables with monomials of up to 8 take one wave per
path; a schedule that splits monomials over lanes, or 17 variables, takes
the lockstep rounds.  Both must end every path at the oracle's root, as in
the tracker's other tests.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1201_0499_amd as pe  # noqa: E402
from test_gpu_track import GAMMA, _compare, _gpu_track, _residual  # noqa: E402


def _system(n, k, extra, d, seed):
    """x_i^d, `extra` products of k variables, a constant in the middle and
    one at the end per polynomial (d >= k: no roots at infinity for generic
    coefficients)."""
    rng = synth.rng_for(seed)
    polys, coefs = [], []
    for i in range(n):
        monos = [[(i, d)], []]
        for _ in range(extra):
            monos.append([(int(v), 1) for v in sorted(rng.choice(n, size=k, replace=False))])
        monos.append([])
        polys.append(monos)
        coefs.append([complex(np.cos(a), np.sin(a)) for a in rng.uniform(0, 2 * np.pi, size=len(monos))])
    return synth.system_from_lists(n, polys, coefs)


@pytest.mark.parametrize("n,k,extra,d,P", [
    (4, 2, 3, 2, 16),    # four rows, two variables per slot
    (9, 3, 2, 3, 5),     # twelve rows, four per slot
    (8, 5, 1, 5, 3),     # eight per slot
    (16, 2, 3, 2, 4),    # as many rows as the kernel has
    (17, 2, 3, 2, 4),    # lockstep
])
def test_every_path_reaches_the_oracles_root(n, k, extra, d, P):
    g = _compare(_system(n, k, extra, d, seed=400 + n), P)
    assert np.all(g["status"] == 0)


def test_wave_and_lockstep_reach_the_same_roots():
    """The same system under its automatic schedule (one wave per path) and
    under one with two lanes per monomial (lockstep)."""
    s = _system(6, 2, 20, 2, seed=431)
    a = _gpu_track(s, 64)
    S = pe.System.from_csr(s)
    S.set_schedule(lanes=2, chunk_vars=2, threads=64, groups=1)
    x = tuple(torch.zeros((64, 6), dtype=torch.float64, device="cuda") for _ in range(4))
    t, res = (torch.zeros(64, dtype=torch.float64, device="cuda") for _ in range(2))
    steps, st = (torch.zeros(64, dtype=torch.int32, device="cuda") for _ in range(2))
    S.start_solutions(0, 64, x)
    code = S.track(64, x, t, steps, st, res, gamma=GAMMA)
    torch.cuda.synchronize()
    S.close()
    assert code == a["code"] == 0 and np.all(st.cpu().numpy() == 0)
    for q in (0, 2):
        assert np.max(np.abs(x[q].cpu().numpy() - a["x"][q])) < 1e-12
    assert np.max(_residual(s, a["x"], np.arange(64))) < 1e-28


def test_step_limit_and_rounds():
    """A path that ends at its step limit, in either kernel."""
    s = _system(3, 2, 2, 2, seed=441)
    g = _gpu_track(s, 8, max_steps=3)
    assert g["code"] == 5 and np.all(g["status"] == 4) and np.all(g["steps"] == 3)
    assert np.all(g["t"] < 1.0)
