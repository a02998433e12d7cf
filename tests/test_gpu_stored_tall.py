"""Applying a stored factorization where few panels have many rows (T from as
many row splits as there are tiles, reduced first), where a single panel meets
more than 16 columns (T in the pass of V^T B), and the leading columns of Q of a
small problem, against the oracle's application of the same reflectors within
50 n u max|B| sqrt(m)."""
import numpy as np
import pytest

from tests.gpu_util import U, to_dev, to_host

pytestmark = pytest.mark.gpu


def _factor(m, n, seed):
    import torch
    import paper_2506_09463_amd as hqr
    A = np.random.default_rng(seed).standard_normal((m, n))
    dA = to_dev(A, ld=m + 1)
    up, _ = hqr.qr_factor(dA)
    torch.cuda.synchronize()
    return hqr, dA, up, to_host(dA), to_host(up)


# 33 tiles: two a split is not yet many; 2100 x 64 and up take the reduction
@pytest.mark.parametrize("m,n,nrhs", [(2048, 64, 2), (2112, 64, 1), (2113, 60, 16), (3000, 130, 3), (9001, 200, 20),
                                      (33000, 70, 2), (1100, 64, 17), (2200, 64, 64), (9000, 50, 65), (20000, 64, 17)])
def test_tall_factor(oracle_mod, m, n, nrhs):
    import torch
    hqr, dA, up, F, u = _factor(m, n, 2400 + m)
    B = np.random.default_rng(m + nrhs).standard_normal((m, nrhs))
    tol = 50 * n * U * np.abs(B).max() * np.sqrt(m)
    for fn, ref in ((hqr.qr_apply_qt, oracle_mod.apply_qt), (hqr.qr_apply_q, oracle_mod.apply_q)):
        print("[case] tall", (m, n, nrhs), fn.__name__, flush=True)
        dB = to_dev(B, ld=m + 3)
        fn(dA, up, dB)
        torch.cuda.synchronize()
        assert np.abs(to_host(dB) - ref(F, u, B)).max() <= tol


@pytest.mark.parametrize("m,n", [(130, 129), (200, 150), (256, 256), (256, 200)])
@pytest.mark.parametrize("k", [1, 16, 17, 32, 33, 100])
def test_leading_columns_of_q(oracle_mod, m, n, k):
    import torch
    hqr, dA, up, F, u = _factor(m, n, 2500 + m + n)
    print("[case] form_q", (m, n, k), flush=True)
    Q = hqr.qr_form_q(dA, up, k=k)
    torch.cuda.synchronize()
    assert np.abs(to_host(Q) - oracle_mod.apply_q(F, u, np.eye(m, k))).max() <= 50 * n * U * np.sqrt(m)
