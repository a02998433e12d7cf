"""Applying a stored factorization at the edges of its two paths: up to 16
columns go panel by panel in one launch each, more take the wide update; the
parts of the first hold several row tiles past 8192 rows.  Against the
oracle's application of the same reflectors, within 50 n u max|B| sqrt(m)."""
import numpy as np
import pytest

from tests.gpu_util import U, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,nrhs", [(1100, 65, 1), (1100, 128, 15), (1100, 129, 16), (1100, 129, 17),
                                      (1030, 1030, 5), (8200, 130, 3), (17000, 70, 2)])
def test_stored_columns(oracle_mod, m, n, nrhs):
    import torch
    import paper_2506_09463_amd as hqr
    rng = np.random.default_rng(900 + n + nrhs)
    A = np.asfortranarray(rng.standard_normal((m, n)))
    B = np.asfortranarray(rng.standard_normal((m, nrhs)))
    print("[case] stored", (m, n, nrhs), flush=True)
    dA = to_dev(A, ld=m + 1)
    up, _ = hqr.qr_factor(dA)
    torch.cuda.synchronize()
    F, u = to_host(dA), to_host(up)
    tol = 50 * n * U * np.abs(B).max() * np.sqrt(m)
    for dev, ref in ((hqr.qr_apply_qt, oracle_mod.apply_qt), (hqr.qr_apply_q, oracle_mod.apply_q)):
        dB = to_dev(B, ld=m + 3)
        dev(dA, up, dB)
        torch.cuda.synchronize()
        assert np.abs(to_host(dB) - ref(F, u, B)).max() <= tol
    Q = hqr.qr_form_q(dA, up, k=nrhs)
    torch.cuda.synchronize()
    assert np.abs(to_host(Q) - oracle_mod.apply_q(F, u, np.eye(m, nrhs))).max() <= tol


def test_stored_nan_stays_in_its_column(oracle_mod):
    """Rows above a panel and other columns do not enter its products."""
    import torch
    import paper_2506_09463_amd as hqr
    m, n = 1100, 130
    rng = np.random.default_rng(950)
    A = np.asfortranarray(rng.standard_normal((m, n)))
    A[:, :64] = 0.0
    A[np.arange(64), np.arange(64)] = 2.0          # 64 identity reflectors: b's first rows stay as they are
    B = np.asfortranarray(rng.standard_normal((m, 3)))
    B[10, 1], B[20, 2] = np.nan, np.inf
    dA = to_dev(A)
    up, _ = hqr.qr_factor(dA)
    torch.cuda.synchronize()
    F, u = to_host(dA), to_host(up)
    assert not u[:64].any()
    dB = to_dev(B)
    print("[case] stored nan", flush=True)
    hqr.qr_apply_qt(dA, up, dB)
    torch.cuda.synchronize()
    X = to_host(dB)
    good = oracle_mod.apply_qt(F, u, np.where(np.isfinite(B), B, 0.0))
    assert np.isfinite(X[:, 0]).all()
    assert np.abs(X[:, 0] - good[:, 0]).max() <= 50 * n * U * 5 * np.sqrt(m)
