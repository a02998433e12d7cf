"""The one-wave rank-one update of at most 15 rows, and the sizes beside it,
against the oracle: dense and sparse v, both signs on the diagonal, values
whose squares leave the range, a leading dimension with rows to spare that stay
as they are."""
import numpy as np
import pytest

from tests.gpu_util import U, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 7, 14, 15, 16, 17])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -530, 2.0 ** 530])
@pytest.mark.parametrize("sparse", [False, True])
def test_small_update(oracle_mod, n, scale, sparse):
    import torch
    import paper_2506_09463_amd as hqr
    rng = np.random.default_rng(2600 + n)
    G = rng.standard_normal((n + 10, n))
    R = np.linalg.cholesky(G.T @ G / n + np.eye(n)).T
    R[n // 2] *= -1.0
    v = rng.standard_normal(n)
    if sparse:
        v[: n // 2] = 0.0
        v[n - 1:] = 0.0
    low = np.tril(rng.standard_normal((n, n)), -1)
    print("[case] chol_update small", n, scale, sparse, flush=True)
    dR, dv = to_dev(R * scale + low, ld=n + 2), to_dev((v * scale).reshape(-1, 1))[:, 0]
    hqr.chol_update(dR, dv)
    torch.cuda.synchronize()
    F = to_host(dR)
    Ro = oracle_mod.chol_update(R, v)
    kappa = np.linalg.cond(R.T @ R + np.outer(v, v)) ** 0.5
    assert np.array_equal(np.tril(F, -1), low)
    assert np.abs(np.triu(F) / scale - np.triu(Ro)).max() <= 100 * n * U * kappa * np.abs(Ro).max()
    assert not to_host(dv).any()
