"""Work forked to the side stream is joined to the caller's stream whatever
happens in between: when a launch fails, what already runs on the side stream
still reads the call's workspace, so the caller's stream has to wait for it
before the workspace is freed in its order.  Read from the host dispatch
without a GPU, one launch after the other made to fail."""
import pytest

BATCH = [(400, 200, 3), (300, 40, 1), (100, 50, 1), (3000, 5, 1)]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    from tests.host_lib import HostLib
    return HostLib(tmp_path_factory.mktemp("host"))


CALLS = {"batched": lambda h: h.batched(BATCH, [0, 1, 0, 0]), "factor": lambda h: h.factor(300, 200)}


def _joined(log):
    """Every side stream with a launch on it is waited for by stream 0, by an
    event recorded after its last launch, before the workspace is freed."""
    end = next((i for i, l in enumerate(log) if l.startswith("free stream=0")), len(log))
    side = {l.split("stream=")[1].split()[0] for l in log if l.startswith("launch")} - {"0"}
    for s in side:
        last = max(i for i, l in enumerate(log) if l.startswith("launch") and "stream=%s " % s in l + " ")
        events = {l.split("event=")[1]: i for i, l in enumerate(log) if l.startswith("record stream=%s " % s) and i > last}
        if not any(l.startswith("wait stream=0 ") and l.split("event=")[1] in events and events[l.split("event=")[1]] < i < end
                   for i, l in enumerate(log)):
            return False
    return True


@pytest.mark.parametrize("call", sorted(CALLS))
def test_side_stream_is_joined_when_a_launch_fails(host, call):
    host.fail()
    host.log()
    assert CALLS[call](host) == 0
    log = host.log()
    assert any(l.startswith("launch") and "stream=0 " not in l for l in log) and _joined(log)
    total = sum(l.startswith("launch") for l in log)
    unjoined = []
    for nth in range(1, total + 1):
        host.fail("", nth)
        rc = CALLS[call](host)
        host.fail()
        log = host.log()
        assert rc == -1002 and sum(l.startswith("failed") for l in log) == 1
        assert any(l.startswith("free stream=0") for l in log)
        if not _joined(log):
            unjoined.append(next(l for l in log if l.startswith("failed")))
    assert unjoined == []


@pytest.mark.parametrize("call", sorted(CALLS))
def test_lookahead_switch_keeps_one_stream(host, call, monkeypatch):
    monkeypatch.setenv("HQR_LOOKAHEAD", "0")
    host.log()
    assert CALLS[call](host) == 0
    log = host.log()
    assert any(l.startswith("launch") for l in log)
    assert all("stream=0 " in l for l in log if l.startswith("launch"))
    assert not any(l.startswith("wait") for l in log)
