"""The panel algebra's 16-column block steps (Cholesky with its inverse, LU
with both inverses) at every kind of panel width: the last panel of n = 64 + w
columns, w on both sides of each block edge, against the oracle's
factorization within factor_tol (50 n u kappa ||A||_2)."""
import numpy as np
import pytest

from tests.gpu_util import check_reflector_invariants, factor_tol, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("graded", [False, True])
def test_last_panel_width(oracle_mod, w, graded):
    import torch
    import paper_2506_09463_amd as hqr
    m, n = 1100, 64 + w
    rng = np.random.default_rng(700 + w)
    A = np.asfortranarray(rng.standard_normal((m, n)))
    if graded:   # panels beyond the near-identity bound of the second pass
        V, _ = np.linalg.qr(rng.standard_normal((n, n)))
        A = np.asfortranarray((A * np.geomspace(1.0, 1e-5, n)) @ V)
    print("[case] panel width", (m, n), "graded" if graded else "gaussian", flush=True)
    dA = to_dev(A)
    up, info = hqr.qr_factor(dA)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    F, u = to_host(dA), to_host(up)
    Fo, uo = oracle_mod.qr_factor(A)
    tol = factor_tol(A)
    assert np.abs(F - Fo).max() <= tol
    assert np.abs(u - uo).max() <= tol
    check_reflector_invariants(A, F, u)
