"""What hqr_cholesky leaves when S is not positive definite: R in the block
rows before the failing one and, from it on, S updated by them (the Schur
complement), as a factorization that works block by block stops; the same bits
on every run.  Bound: 50 n u kappa of the part factored, times max |S|."""
import numpy as np
import pytest

from tests.gpu_util import U, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bad", [(200, 70), (200, 199), (300, 128), (700, 64), (50, 20)])
def test_partial_factor(n, bad):
    import torch
    import paper_2506_09463_amd as hqr
    rng = np.random.default_rng(1500 + n + bad)
    G = rng.standard_normal((n + 10, n))
    S = G.T @ G + 0.05 * n * np.eye(n)
    S[bad, bad] = -1.0
    k = bad // 64 * 64
    want = np.triu(S)
    if k:
        R = np.linalg.cholesky(S[:k, :k]).T
        top = np.linalg.solve(R.T, S[:k, k:])
        want[:k, :k], want[:k, k:] = R, top
        want[k:, k:] = np.triu(S[k:, k:] - top.T @ top)
    tol = 50 * n * U * (np.linalg.cond(S[:k, :k]) if k else 1.0) * np.abs(S).max()
    first = None
    for run in range(5):
        print("[case] cholesky partial", n, bad, run, flush=True)
        dS = to_dev(np.triu(S), ld=n + 1)
        _, info = hqr.cholesky(dS)
        torch.cuda.synchronize()
        assert int(info.item()) == bad + 1
        F = to_host(dS)
        assert np.abs(F - want).max() <= tol
        first = F if first is None else first
        assert np.array_equal(F, first)
