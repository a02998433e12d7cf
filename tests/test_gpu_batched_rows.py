"""The 512-thread batched kernels at the edges of their row classes (257,
512/513, 1024 rows), of their 16-row blocks and of ragged panels, factoring
and with stored factors, against the oracle (factor_tol, lsq_forward_bound);
an instance alone and in the batch is bitwise the same."""
import numpy as np
import pytest

from tests.gpu_util import U, factor_tol, lsq_forward_bound, to_dev, to_host

pytestmark = pytest.mark.gpu

SHAPES = [(257, 1, 1), (257, 33, 2), (258, 250, 1), (300, 300, 3), (511, 100, 8), (512, 64, 1), (513, 40, 2),
          (515, 17, 16), (700, 129, 1), (1023, 48, 4), (1024, 31, 33), (1024, 16, 0)]


def _solve(hqr, probs, keep=None):
    import torch
    As = [to_dev(A, ld=A.shape[0] + (i % 3)) for i, (A, _) in enumerate(probs)]
    Bs = [to_dev(B, ld=B.shape[0] + (i % 2)) for i, (_, B) in enumerate(probs)]
    ups, res, info = hqr.qr_lsq_solve_batched(As, Bs)
    torch.cuda.synchronize()
    assert not to_host(info).any()
    return As, ups, Bs, res


def test_rows_kernel_edges(oracle_mod):
    import torch
    import paper_2506_09463_amd as hqr
    rng = np.random.default_rng(1000)
    probs = [(np.asfortranarray(rng.standard_normal((m, n))), np.asfortranarray(rng.standard_normal((m, r))))
             for m, n, r in SHAPES]
    print("[case] batched rows", SHAPES, flush=True)
    As, ups, Bs, res = _solve(hqr, probs)
    for i, (A, B) in enumerate(probs):
        m, n = A.shape
        Xo, Fo, upo, reso, _ = oracle_mod.lsq_solve(A, B)
        tol = factor_tol(A)
        assert np.abs(to_host(As[i]) - Fo).max() <= tol, i
        assert np.abs(to_host(ups[i])[:n] - upo).max() <= tol, i
        X = to_host(Bs[i])[:n]
        for c in range(B.shape[1]):
            r = B[:, c] - A @ Xo[:, c]
            assert np.linalg.norm(X[:, c] - Xo[:, c]) <= 2 * lsq_forward_bound(A, Xo[:, c], r) * np.linalg.norm(Xo[:, c])
            assert abs(to_host(res[i])[c] - reso[c]) <= 50 * m * U * reso[c] + tol
    # the stored factors applied to new right-hand sides, beside a new problem
    news = [np.asfortranarray(rng.standard_normal(B.shape)) for _, B in probs]
    dn = [to_dev(B) for B in news]
    extra, eb = to_dev(probs[3][0]), to_dev(probs[3][1])
    before = [to_host(a).copy() for a in As]
    _, _, info = hqr.qr_lsq_solve_batched(As + [extra], dn + [eb], ups=list(ups) + [torch.zeros(300, dtype=torch.float64, device="cuda")],
                                          factored=[1] * len(As) + [0])
    torch.cuda.synchronize()
    assert not to_host(info).any()
    assert np.array_equal(to_host(extra), before[3])         # alone or beside others: the same bits
    for i, ((A, _), B) in enumerate(zip(probs, news)):
        n = A.shape[1]
        assert np.array_equal(to_host(As[i]), before[i])
        Xo = oracle_mod.lsq_solve(A, B)[0]
        X = to_host(dn[i])[:n]
        for c in range(B.shape[1]):
            r = B[:, c] - A @ Xo[:, c]
            assert np.linalg.norm(X[:, c] - Xo[:, c]) <= 2 * lsq_forward_bound(A, Xo[:, c], r) * np.linalg.norm(Xo[:, c])
    # each alone
    for i, p in enumerate(probs):
        A1, u1, B1, _ = _solve(hqr, [p])
        assert np.array_equal(to_host(A1[0]), before[i])
