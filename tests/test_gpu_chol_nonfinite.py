"""hqr_cholesky at the ends of the number range, against the oracle: an
infinite pivot gives R_jj = inf with zeros to its right and leaves the other
rows as they are (x / inf = 0), NaN and -inf pivots end it with their own
index, and scaling S by powers of four scales R by powers of two exactly."""
import numpy as np
import pytest

from tests.gpu_util import U, to_dev, to_host

pytestmark = pytest.mark.gpu


def _spd(n, seed):
    G = np.random.default_rng(seed).standard_normal((n + 10, n))
    return G.T @ G + 0.05 * n * np.eye(n)


def _run(S):
    import torch
    import paper_2506_09463_amd as hqr
    dS = to_dev(np.triu(S), ld=S.shape[0] + 1)
    _, info = hqr.cholesky(dS)
    torch.cuda.synchronize()
    return to_host(dS), int(info.item())


@pytest.mark.parametrize("n,js", [(1, [0]), (40, [0]), (40, [39]), (64, [17, 18]), (200, [0, 63]), (200, [70]), (200, [199]),
                                  (300, [64, 127, 130])])
def test_infinite_pivot(oracle_mod, n, js):
    S = _spd(n, 1600 + n)
    S[js, js] = np.inf
    print("[case] cholesky infinite pivot", n, js, flush=True)
    F, info = _run(S)
    Ro, io = oracle_mod.cholesky(S)
    assert info == io == 0
    assert np.array_equal(np.isinf(F), np.isinf(Ro)) and np.array_equal(np.isnan(F), np.isnan(Ro))
    for j in js:
        assert F[j, j] == np.inf and not F[j, j + 1:].any()
    fin = np.isfinite(Ro)
    keep = np.setdiff1d(np.arange(n), js)
    kappa = np.linalg.cond(S[np.ix_(keep, keep)]) if keep.size else 1.0
    assert np.abs(F[fin] - Ro[fin]).max(initial=0.0) <= 50 * n * U * kappa * np.abs(Ro[fin]).max(initial=0.0)


@pytest.mark.parametrize("n,j", [(40, 5), (200, 0), (200, 100), (200, 199)])
@pytest.mark.parametrize("value", [np.nan, -np.inf, 0.0])
def test_bad_pivot_value(oracle_mod, n, j, value):
    S = _spd(n, 1700 + n)
    S[j, j] = value
    print("[case] cholesky pivot", value, n, j, flush=True)
    assert _run(S)[1] == j + 1 == oracle_mod.cholesky(S)[1]


@pytest.mark.parametrize("k", [-480, -250, 250, 480])
def test_power_of_four_scales(k):
    S = _spd(150, 1800)
    print("[case] cholesky scale 4^%d" % k, flush=True)
    F, info = _run(S)
    G, infog = _run(np.ldexp(S, 2 * k))
    assert info == infog == 0
    assert np.array_equal(np.ldexp(F, k), G)
