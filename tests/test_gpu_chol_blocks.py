"""Block edges of the Cholesky factorization and of the rank-one update, and
the update's range handling (rotations whose squares leave the normal range
are redone with hypot), against the oracle with the tolerances of
test_gpu_cholesky."""
import numpy as np
import pytest

from tests.gpu_util import U, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [63, 127, 128, 129, 193])
def test_cholesky_block_edges(oracle_mod, n):
    import torch
    import paper_2506_09463_amd as hqr
    rng = np.random.default_rng(800 + n)
    G = rng.standard_normal((n + 10, n))
    S = G.T @ G + 0.01 * n * np.eye(n)
    print("[case] hqr_cholesky", n, flush=True)
    dS = to_dev(np.triu(S), ld=n + 3)
    _, info = hqr.cholesky(dS)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    F = to_host(dS)
    assert np.array_equal(np.tril(F, -1), np.zeros((n, n)))
    Ro, _ = oracle_mod.cholesky(S)
    assert np.abs(F - Ro).max() <= 50 * n * U * np.linalg.cond(S) * np.abs(Ro).max()


@pytest.mark.parametrize("n,bad", [(40, 0), (64, 63), (200, 64), (200, 199)])
def test_cholesky_first_bad_pivot(oracle_mod, n, bad):
    import torch
    import paper_2506_09463_amd as hqr
    rng = np.random.default_rng(820 + bad)
    G = rng.standard_normal((n + 10, n))
    S = G.T @ G
    S[bad, bad] = -1.0
    print("[case] hqr_cholesky bad pivot", n, bad, flush=True)
    _, info = hqr.cholesky(to_dev(S))
    torch.cuda.synchronize()
    assert int(info.item()) == bad + 1 == oracle_mod.cholesky(S)[1]


@pytest.mark.parametrize("n,scale", [(63, 1.0), (64, 1.0), (65, 1.0), (129, 1.0), (200, 1e-160), (200, 1e160)])
def test_chol_update_blocks_and_range(oracle_mod, n, scale):
    import torch
    import paper_2506_09463_amd as hqr
    rng = np.random.default_rng(840 + n)
    G = rng.standard_normal((n + 10, n))
    R = np.linalg.cholesky(G.T @ G / n + np.eye(n)).T
    v = rng.standard_normal(n)
    v[n // 2] = 0.0
    R1, v1 = R * scale, v * scale          # exact powers of ten are not needed: both sides see the same arrays
    print("[case] hqr_chol_update", n, scale, flush=True)
    dR, dv = to_dev(R1, ld=n + 1), to_dev(v1.reshape(-1, 1))[:, 0]
    hqr.chol_update(dR, dv)
    torch.cuda.synchronize()
    R2 = to_host(dR)
    Ro = oracle_mod.chol_update(R1, v1)
    kappa = np.linalg.cond(R.T @ R + np.outer(v, v)) ** 0.5
    assert np.abs(R2 - Ro).max() <= 100 * n * U * kappa * np.abs(Ro).max()
    assert not to_host(dv).any()


def test_chol_update_zero_rows(oracle_mod):
    """Zero diagonal entries with zero and nonzero v: (c, s) = (1, 0) and (0, 1)."""
    import torch
    import paper_2506_09463_amd as hqr
    n = 70
    rng = np.random.default_rng(860)
    R = np.triu(rng.standard_normal((n, n)))
    R[3, 3] = R[66, 66] = 0.0
    v = rng.standard_normal(n)
    v[:3] = 0.0
    R[:3] *= 0.0
    dR, dv = to_dev(R), to_dev(v.reshape(-1, 1))[:, 0]
    print("[case] hqr_chol_update zero rows", flush=True)
    hqr.chol_update(dR, dv)
    torch.cuda.synchronize()
    S2 = R.T @ R + np.outer(v, v)
    R2 = to_host(dR)
    assert np.linalg.norm(S2 - R2.T @ R2) <= 50 * n * U * np.linalg.norm(S2)
    assert np.abs(R2[:4] - oracle_mod.chol_update(R, v)[:4]).max() <= 50 * n * U * np.abs(R).max()
