"""hqr_chol_update where its rotations are exact or not finite: rows whose v is
zero keep their bits, and values that are not finite spread as in the oracle."""
import numpy as np
import pytest

from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def _run(R, v):
    import torch
    import paper_2506_09463_amd as hqr
    dR, dv = to_dev(R, ld=R.shape[0] + 1), to_dev(v.reshape(-1, 1))[:, 0]
    hqr.chol_update(dR, dv)
    torch.cuda.synchronize()
    return to_host(dR)


@pytest.mark.parametrize("n,first", [(1, 1), (50, 50), (64, 30), (200, 200), (200, 64), (200, 100), (300, 299)])
def test_rows_before_v_starts_keep_their_bits(n, first):
    """v = 0 in its first `first` entries: the rotation is (1, 0), the row stays."""
    rng = np.random.default_rng(1900 + n + first)
    R = np.triu(rng.standard_normal((n, n)))
    R[np.arange(n), np.arange(n)] *= 3.0        # both signs
    v = rng.standard_normal(n)
    v[:first] = 0.0
    v[: first // 2] *= -1.0                     # -0.0 as well
    print("[case] chol_update leading zeros", n, first, flush=True)
    F = _run(R, v)
    assert np.array_equal(F[:first], R[:first])
    assert first == n or not np.array_equal(F[first], R[first])


@pytest.mark.parametrize("n,k", [(40, 3), (200, 3), (200, 70)])
@pytest.mark.parametrize("rkk,vk", [(0.0, np.inf), (0.0, np.nan), (np.inf, 1.0), (2.0, -np.inf), (np.nan, 0.0)])
def test_not_finite(oracle_mod, n, k, rkk, vk):
    rng = np.random.default_rng(1950 + n + k)
    R = np.triu(rng.standard_normal((n, n)) + 0.5)
    v = rng.standard_normal(n)
    R[k, k], v[k] = rkk, vk
    print("[case] chol_update not finite", n, k, rkk, vk, flush=True)
    F = _run(R, v)
    with np.errstate(all="ignore"):
        Ro = oracle_mod.chol_update(R, v)
    assert np.array_equal(np.isfinite(F), np.isfinite(Ro))
