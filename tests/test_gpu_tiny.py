"""The one-wave kernel of the smallest problems at the edges of its row and
column classes (64/65/128 rows, 16/17/32 columns with the right-hand sides),
against the oracle; scaled norms and a zero R[k][k] inside it."""
import numpy as np
import pytest

from tests.gpu_util import U, factor_tol, lsq_forward_bound, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,r", [(1, 1, 0), (1, 1, 31), (16, 16, 0), (20, 8, 1), (64, 15, 1), (64, 16, 1), (65, 16, 0),
                                   (128, 15, 1), (32, 32, 0), (64, 31, 1), (65, 17, 15), (128, 32, 0), (128, 16, 16)])
@pytest.mark.parametrize("scale", [1.0, 1e-140, 1e150])
def test_tiny(oracle_mod, m, n, r, scale):
    import torch
    import paper_2506_09463_amd as hqr
    rng = np.random.default_rng(1100 + m + n)
    A = np.asfortranarray(rng.standard_normal((m, n)) * scale)
    B = np.asfortranarray(rng.standard_normal((m, max(r, 1))))
    print("[case] tiny", (m, n, r), scale, flush=True)
    dA, dB = to_dev(A, ld=m + 3), to_dev(B, ld=m + 2)
    it = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    up, res, info, _ = hqr.qr_lsq_solve(dA, dB[:, :r] if r else dB[:, :0], iters=it)
    torch.cuda.synchronize()
    assert int(info.item()) == 0 and int(it.item()) == 0
    Xo, Fo, upo, reso, _ = oracle_mod.lsq_solve(A, B)
    tol = factor_tol(A)
    assert np.abs(to_host(dA) - Fo).max() <= tol
    assert np.abs(to_host(up)[:n] - upo).max() <= tol
    assert np.array_equal(to_host(up)[:n] == 0.0, upo == 0.0)
    X = to_host(dB)
    for c in range(r):
        rr = B[:, c] - A @ Xo[:, c]
        bound = 2 * lsq_forward_bound(A, Xo[:, c] * scale, rr / scale) if scale == 1.0 else 1e-10
        assert np.linalg.norm(X[:n, c] - Xo[:, c]) <= bound * np.linalg.norm(Xo[:, c])
        assert abs(to_host(res)[c] - reso[c]) <= 50 * m * U * np.linalg.norm(B[:, c])


@pytest.mark.parametrize("m,n,k", [(10, 6, 3), (100, 20, 19)])
def test_tiny_zero_diagonal(oracle_mod, m, n, k):
    import torch
    import paper_2506_09463_amd as hqr
    rng = np.random.default_rng(1200 + m)
    A = np.asfortranarray(rng.standard_normal((m, n)))
    A[:, k] = 0.0
    B = np.asfortranarray(rng.standard_normal((m, 2)))
    dA, dB = to_dev(A), to_dev(B)
    print("[case] tiny singular", (m, n, k), flush=True)
    up, res, info, _ = hqr.qr_lsq_solve(dA, dB)
    torch.cuda.synchronize()
    assert int(info.item()) == k + 1
    F, u = to_host(dA), to_host(up)
    assert u[k] == 0.0
    assert np.abs(to_host(dB) - oracle_mod.apply_qt(F, u, B)).max() <= 50 * m * U * np.abs(B).max() * 10
