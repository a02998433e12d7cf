"""W' = T^T X and T X for wide right-hand sides at ragged last panels and
column counts on both sides of a workgroup's 16 columns and of the narrow
form's 64: Q^T A = R and Q Q^T B = B, both within 50 n u of the norm."""
import numpy as np
import pytest

from tests.gpu_util import U, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 79, 80, 81, 127, 128, 150])
@pytest.mark.parametrize("k", [17, 31, 33, 64, 65, 130])
def test_wide_apply(n, k):
    import torch
    import paper_2506_09463_amd as hqr
    m = 1100
    rng = np.random.default_rng(1000 * n + k)
    A = rng.standard_normal((m, n))
    B = rng.standard_normal((m, k))
    print("[case] wide apply", n, k, flush=True)
    dA = to_dev(A)
    up, _ = hqr.qr_factor(dA)
    R = np.triu(to_host(dA)[:n])
    C = np.concatenate([A, B], axis=1)[:, :max(n, k)]
    dC = to_dev(C, ld=m + 1)
    hqr.qr_apply_qt(dA, up, dC)
    q = to_host(dC)
    want = np.zeros((m, n))
    want[:n] = R
    assert np.linalg.norm(q[:, :n] - want) <= 50 * n * U * np.linalg.norm(A)
    dB = to_dev(B)
    hqr.qr_apply_qt(dA, up, dB)
    hqr.qr_apply_q(dA, up, dB)
    torch.cuda.synchronize()
    assert np.linalg.norm(to_host(dB) - B) <= 50 * n * U * np.linalg.norm(B)
