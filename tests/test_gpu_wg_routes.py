"""What the smallest-problem kernel took over from the one-workgroup kernel's
other tests: the 128-row variants with one column (more than 32 columns with
B, so the variant itself runs), and the patterns of values that are not finite
on both kernels, equal to the one-column loop's as long as the matrix is one
16-column panel."""
import numpy as np
import pytest

from tests.gpu_util import U, factor_tol, lsq_forward_bound, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture
def hqr():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2506_09463_amd as h
    h.load()
    yield h
    h.tune_clear()
    h.load_tune_db()


def _force(hqr, name):
    hqr.tune_clear()
    hqr.tune_set(hqr.HQR_TUNE_SINGLE, 0, 1 << 40, 0, 1 << 40, hqr.tune_variants().index(name))


def _solve(hqr, A, B):
    import torch
    dA, dB = to_dev(A), to_dev(B)
    up, res, info, _ = hqr.qr_lsq_solve(dA, dB)
    torch.cuda.synchronize()
    return to_host(dA), to_host(up)[: A.shape[1]], to_host(dB), to_host(res), int(info.item())


@pytest.mark.parametrize("name", ["wg64x2", "wg128x1", "wg256x1", "wg256x1p8"])
@pytest.mark.parametrize("m,n,r", [(128, 1, 32), (1, 1, 40), (128, 16, 17), (100, 17, 16), (33, 33, 0)])
def test_few_columns_on_the_variant(hqr, oracle_mod, name, m, n, r):
    _force(hqr, name)
    rng = np.random.default_rng(2000 + m + n)
    A, B = rng.standard_normal((m, n)), rng.standard_normal((m, r))
    print("[case] few columns", name, (m, n, r), flush=True)
    F, up, X, res, info = _solve(hqr, A, B)
    Xo, Fo, upo, reso, _ = oracle_mod.lsq_solve(A, B)
    tol = factor_tol(A)
    assert info == 0
    assert np.abs(F - Fo).max() <= tol and np.array_equal(up == 0.0, upo == 0.0)
    for c in range(r):
        rr = B[:, c] - A @ Xo[:, c]
        assert np.linalg.norm(X[:n, c] - Xo[:, c]) <= 2 * lsq_forward_bound(A, Xo[:, c], rr) * np.linalg.norm(Xo[:, c])
        assert abs(res[c] - reso[c]) <= 50 * m * U * np.linalg.norm(B[:, c])


# (20, 6): one wave; the others: the panel kernel (more than 128 rows)
@pytest.mark.parametrize("m,n,name", [(20, 6, "wg64x2"), (128, 15, "wg64x2"), (200, 12, "wg64x4"), (200, 12, "wg256x1"),
                                      (300, 16, "wg128x4"), (700, 9, "wg256x4p8")])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("row", [0, 3, -1])
def test_not_finite_pattern(hqr, oracle_mod, m, n, name, value, row):
    _force(hqr, name)
    rng = np.random.default_rng(2100 + m + n)
    A, B = rng.standard_normal((m, n)), rng.standard_normal((m, 2))
    A[row, n // 2] = value
    B[row, 1] = value
    print("[case] not finite", (m, n), name, value, row, flush=True)
    F, up, X, res, info = _solve(hqr, A, B)
    with np.errstate(all="ignore"):
        Xo, Fo, upo, reso, infoo = oracle_mod.lsq_solve(A, B)
    assert info == infoo
    assert np.array_equal(np.isfinite(F), np.isfinite(Fo))
    assert np.array_equal(np.isfinite(up), np.isfinite(upo))
    assert np.array_equal(np.isfinite(X[:n]), np.isfinite(Xo)) and np.array_equal(np.isfinite(res), np.isfinite(reso))


@pytest.mark.parametrize("m,n,r", [(20, 8, 1), (64, 31, 1), (65, 17, 15), (128, 16, 16), (128, 15, 1)])
@pytest.mark.parametrize("scale", [2.0 ** -465, 2.0 ** 498])
def test_tiny_scaled_solution(hqr, oracle_mod, m, n, r, scale):
    """Columns whose squares leave the range: A's condition number and the
    solution's bound are those of the unscaled problem (scaling by a power of
    two changes neither, x only by its inverse)."""
    rng = np.random.default_rng(2200 + m + n)
    A, B = rng.standard_normal((m, n)), rng.standard_normal((m, r))
    print("[case] tiny scaled", (m, n, r), scale, flush=True)
    F, up, X, res, info = _solve(hqr, A * scale, B)
    Xo, Fo, upo, reso, _ = oracle_mod.lsq_solve(A, B)
    assert info == 0
    assert np.abs(F / scale - Fo).max() <= factor_tol(A) and np.abs(up / scale - upo).max() <= factor_tol(A)
    for c in range(r):
        rr = B[:, c] - A @ Xo[:, c]
        assert np.linalg.norm(X[:n, c] * scale - Xo[:, c]) <= 2 * lsq_forward_bound(A, Xo[:, c], rr) * np.linalg.norm(Xo[:, c])
        assert abs(res[c] - reso[c]) <= 50 * m * U * np.linalg.norm(B[:, c])


@pytest.mark.parametrize("nrhs", [3, 16, 17, 40])
def test_stored_columns_do_not_see_each_other(hqr, oracle_mod, nrhs):
    """A stored factor applied beside columns that are not finite, above, in
    and below the panels: the other columns keep their bits."""
    import torch
    rng = np.random.default_rng(2300 + nrhs)
    m, n = 1100, 130
    F, u = oracle_mod.qr_factor(rng.standard_normal((m, n)))
    dF, du = to_dev(F), to_dev(u.reshape(-1, 1))[:, 0]
    B = rng.standard_normal((m, nrhs))
    bad = {0: (10, np.nan), nrhs - 1: (100, np.inf), nrhs // 2: (1099, -np.inf)}
    Bn = B.copy()
    for c, (i, v) in bad.items():
        Bn[i, c] = v
    keep = [c for c in range(nrhs) if c not in bad]
    for fn in (hqr.qr_apply_qt, hqr.qr_apply_q):
        out = []
        for M in (B, Bn):
            print("[case] stored columns", nrhs, fn.__name__, flush=True)
            dB = to_dev(M)
            fn(dF, du, dB)
            torch.cuda.synchronize()
            out.append(to_host(dB))
        assert np.array_equal(out[0][:, keep], out[1][:, keep])
        assert not np.isfinite(out[1][:, list(bad)]).all(axis=0).any()
