"""Which kernel a smallest problem takes: the one-wave kernel where it was
faster than the panel kernel, the panel kernel where many right-hand sides make
the wave's serial solve the longer part.  The ratios are the panel kernel's
time over the one-wave kernel's on MI355X, the smallest and largest over
m = 16, 32, 64, 65 and 128."""
import pytest

MEASURED = {(1, 1): (2.22, 2.69), (1, 31): (1.06, 1.15), (2, 24): (1.07, 1.14), (4, 16): (1.09, 1.15), (4, 24): (0.95, 1.02),
            (8, 8): (1.35, 1.38), (8, 16): (0.93, 0.96), (8, 24): (0.80, 0.84), (12, 4): (1.47, 1.49), (12, 6): (1.07, 1.11),
            (12, 12): (0.89, 0.92), (15, 1): (1.68, 1.74), (15, 4): (1.04, 1.09), (15, 8): (0.91, 0.94), (15, 16): (0.74, 0.77),
            (16, 0): (1.19, 1.31), (16, 2): (1.01, 1.04), (16, 4): (0.92, 0.95), (16, 16): (0.64, 0.67), (20, 6): (1.07, 1.14),
            (20, 12): (0.90, 0.97), (24, 6): (1.00, 1.06), (24, 8): (0.93, 1.00), (28, 3): (1.04, 1.11), (31, 1): (1.09, 1.18),
            (32, 0): (0.90, 0.98)}


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    from tests.host_lib import HostLib
    return HostLib(tmp_path_factory.mktemp("host"))


@pytest.mark.parametrize("n,r", sorted(MEASURED))
def test_route_follows_the_faster_kernel(host, n, r):
    lo, hi = MEASURED[(n, r)]
    for m in (max(n, 16), 64, 65, 128):
        host.log()
        assert (host.lsq(m, n, r) if r else host.factor(m, n)) == 0
        tiny = any(l.startswith("launch wg_tiny_kernel") for l in host.log())
        assert tiny or hi <= 1.02, (m, n, r)
        assert not tiny or lo >= 1.0, (m, n, r)


def test_rows_and_columns_the_wave_holds(host):
    for m, n, r in [(129, 8, 1), (128, 30, 3), (128, 33, 0)]:
        host.log()
        assert (host.lsq(m, n, r) if r else host.factor(m, n)) == 0
        assert not any("wg_tiny" in l for l in host.log()), (m, n, r)
