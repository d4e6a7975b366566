"""The double-double elimination of the corrector at the edges of its kernels.

On a linear system one Newton step is one solve, so the residual after the
first update shows the solve's accuracy: at most n eps growth |A| |x|, times
the condition number where the elimination is not backward stable, is below
103 * 1.2e-32 * 10 * 10 * 1e6 < 1e-22, while a solve in FP64 leaves 1e-14.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1201_0499_amd as pe  # noqa: E402
from gpu_helpers import dev, host  # noqa: E402


@pytest.mark.parametrize("n", [1, 7, 8, 63, 64, 96, 103, 104])
def test_linear_system_in_one_step(n):
    rng = np.random.default_rng(5000 + n)
    polys = [[[(j, 1)] for j in range(n)] + [[]] for _ in range(n)]
    coefs = [list(rng.uniform(-1, 1, n) + 1j * rng.uniform(-1, 1, n)) + [1.0 + 0.5j] for _ in range(n)]
    S = pe.System.from_csr(synth.system_from_lists(n, polys, coefs))
    P = 5
    x = dev((rng.uniform(0.5, 1, (P, n)), np.zeros((P, n)), rng.uniform(0.5, 1, (P, n)), np.zeros((P, n))))
    res = torch.zeros(P, dtype=torch.float64, device="cuda")
    it = torch.zeros(P, dtype=torch.int32, device="cuda")
    st = torch.zeros(P, dtype=torch.int32, device="cuda")
    print(f"[case] linear dd n={n}", flush=True)
    code = S.newton(P, x, res, it, st, tol=1e-22, max_iter=3, mode=1)
    torch.cuda.synchronize()
    S.close()
    assert code == 0 and torch.all(st == 0)
    assert torch.all(it == 1), (it, res)
    xs = host(x)
    A = np.array([c[:n] for c in coefs])
    z = (xs[0] + 1j * xs[2]).T
    assert np.max(np.abs(A @ z + coefs[0][n])) < 1e-16 * 64 * n * np.max(np.abs(z))
