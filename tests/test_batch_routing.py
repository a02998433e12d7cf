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
