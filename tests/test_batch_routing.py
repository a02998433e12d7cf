"""Which kernel a batched instance takes depends on its own shape alone: what
else is in the batch, and which tuning rules match the batch's largest
instance, changes nothing (the kernels round differently, so the route decides
an instance's bits).  The routes are read from the host dispatch without a GPU;
the GPU test holds the bits themselves."""
import re

import numpy as np
import pytest

BIG = 1 << 40
# rules as an earlier autotuner saved them: by the batch's largest rows
RULES = [[], [("wg256x2p8", 257, 512)], [("wg256x4p8", 513, 1024)], [("wg256x1", 1, 256)],
         [("wg256x1p2", 1, 256), ("wg256x2p8", 257, 512), ("wg256x4p8", 513, 1024)], [("wg256x4p2", 0, BIG)]]
BATCHES = [[(400, 200, 3)], [(400, 200, 3), (500, 30, 1)], [(400, 200, 3), (1000, 40, 1)], [(400, 200, 3), (20, 8, 1)],
           [(400, 200, 3), (1000, 40, 1), (256, 100, 2), (1024, 16, 0), (3000, 5, 1)]]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    from tests.host_lib import HostLib
    return HostLib(tmp_path_factory.mktemp("host"))


def _threads(log):
    """rows -> threads of the workgroup that takes the instance."""
    out = {}
    for line in log:
        hit = re.match(r"launch (\S*wg_batched\S*)<.* block=(\d+) rows=([\d,]+)", line)
        if hit:
            out.update({int(r): int(hit.group(2)) for r in hit.group(3).split(",")})
    return out


@pytest.mark.parametrize("rules", range(len(RULES)))
def test_route_depends_on_own_rows(host, rules):
    host.lib.hqr_tune_clear()
    for name, lo, hi in RULES[rules]:
        assert host.lib.hqr_tune_set(1, lo, hi, 0, BIG, 0, host.variant(name)) == 0
    for shapes in BATCHES:
        for stored in (0, 1):
            host.log()
            assert host.batched(shapes, [stored] * len(shapes)) == 0
            got = _threads(host.log())
            assert got == {m: 512 if m > 256 else 256 for m, _, _ in shapes if m <= 1024}, (shapes, stored)
    host.lib.hqr_tune_clear()


@pytest.mark.gpu
def test_bits_do_not_depend_on_the_batch_or_rules():
    """A 400 x 200 instance alone, beside a 500-row and beside a 1000-row one,
    without rules and with one that covers only one of their largest sizes."""
    import torch
    import paper_2506_09463_amd as hqr
    from tests.gpu_util import to_dev, to_host
    rng = np.random.default_rng(1400)
    probs = {m: (rng.standard_normal((m, n)), rng.standard_normal((m, 3))) for m, n in ((400, 200), (500, 30), (1000, 40))}
    ref = None
    try:
        for rule in (None, ("wg256x2p8", 257, 512), ("wg256x4p8", 513, 1024)):
            hqr.tune_clear()
            if rule:
                hqr.tune_set(hqr.HQR_TUNE_BATCHED, rule[1], rule[2], 0, BIG, hqr.tune_variants().index(rule[0]))
            for rows in ((400,), (400, 500), (400, 1000)):
                print("[case] batch", rule, rows, flush=True)
                As, Bs = ([to_dev(probs[m][j]) for m in rows] for j in (0, 1))
                ups, _, info = hqr.qr_lsq_solve_batched(As, Bs)
                torch.cuda.synchronize()
                assert not to_host(info).any()
                out = [to_host(t) for t in (As[0], ups[0], Bs[0])]
                ref = ref or out
                assert all(np.array_equal(a, b) for a, b in zip(out, ref)), (rule, rows)
    finally:
        hqr.tune_clear()
        hqr.load_tune_db()


ALL = [(400, 200, 2), (300, 20, 1), (100, 20, 1), (2000, 10, 1), (20, 8, 2), (1024, 16, 1)]


def test_every_group_has_a_queue_of_its_own(host):
    """New and stored instances above 256 rows, smaller ones and streamed ones
    in one call: four launches, four queue heads, every instance in one."""
    host.log()
    assert host.batched(ALL, [0, 1, 0, 0, 1, 1]) == 0
    log = [l for l in host.log() if "head=" in l]
    assert len(log) == 4 and len({l.split("head=")[1] for l in log}) == 4
    assert sum(l.startswith("launch batched_lsq_kernel") for l in log) == 1
    rows = sorted(int(r) for l in log if "rows=" in l for r in l.split("rows=")[1].split()[0].split(","))
    assert rows == sorted(m for m, _, _ in ALL if m <= 1024)


@pytest.mark.gpu
@pytest.mark.parametrize("lookahead", ["1", "0"])
@pytest.mark.parametrize("copies", [1, 60])
def test_all_groups_in_one_batch(oracle_mod, monkeypatch, lookahead, copies):
    import torch
    import paper_2506_09463_amd as hqr
    from tests.gpu_util import factor_tol, lsq_forward_bound, to_dev, to_host
    monkeypatch.setenv("HQR_LOOKAHEAD", lookahead)
    rng = np.random.default_rng(1450)
    shapes = [(400, 200, 2), (300, 20, 1), (100, 20, 1), (2000, 10, 1), (20, 8, 2), (1024, 16, 1), (1500, 12, 1)] * copies
    stored = [0, 1, 0, 0, 1, 1, 1] * copies
    probs = [(rng.standard_normal((m, n)), rng.standard_normal((m, r))) for m, n, r in shapes]
    print("[case] all groups", copies, lookahead, flush=True)
    As = [to_dev(A) for A, _ in probs]
    ups, _, _ = hqr.qr_lsq_solve_batched(As, [to_dev(B) for _, B in probs])
    torch.cuda.synchronize()
    for a, (A, _), s in zip(As, probs, stored):
        if not s:
            a.copy_(to_dev(A))
    Bs = [to_dev(B) for _, B in probs]
    info = torch.full((len(probs),), -5, dtype=torch.int32, device="cuda")
    hqr.qr_lsq_solve_batched(As, Bs, ups=ups, info=info, factored=stored)
    torch.cuda.synchronize()
    assert not to_host(info).any()
    for (A, B), a, b in zip(probs, As, Bs):
        n = A.shape[1]
        Xo, Fo = oracle_mod.lsq_solve(A, B)[:2]
        assert np.abs(to_host(a) - Fo).max() <= factor_tol(A)
        for c in range(B.shape[1]):
            r = B[:, c] - A @ Xo[:, c]
            x = to_host(b)[:n, c]
            assert np.linalg.norm(x - Xo[:, c]) <= 2 * lsq_forward_bound(A, Xo[:, c], r) * np.linalg.norm(Xo[:, c])
