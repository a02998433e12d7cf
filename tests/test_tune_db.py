"""The tuning database agrees with itself: at every shape whose candidates it
holds timings of, the rule that a call of that shape meets first names a path
within 10 % of the fastest one (a bucket's paths may cross inside it by that
much), and every corner of the rules' ranges between 129 and 256 rows and
columns, where the two paths cross, was timed."""
import json

from paper_2506_09463_amd.hqr import TUNE_DB_PATH


def _db():
    with open(TUNE_DB_PATH) as f:
        return json.load(f)


def _first(rules, m, n):
    for r in rules:
        if r["op"] == "single" and r["m"][0] <= m <= r["m"][1] and r["n"][0] <= n <= r["n"][1]:
            if not r.get("square") or m == n:
                return r
    return None


def test_rules_agree_with_their_timings():
    db = _db()
    worse = []
    for t in db["measurements"]:
        if t["op"] != "single":
            continue
        r = _first(db["rules"], *t["shape"])
        if t["ms"][r["choice"]] > 1.10 * min(t["ms"].values()):
            worse.append((t["shape"], r["choice"], t["ms"][r["choice"]], min(t["ms"].values())))
    assert worse == []


def test_crossing_range_is_timed_at_its_corners():
    db = _db()
    timed = {tuple(t["shape"]) for t in db["measurements"] if t["op"] == "single"}
    for r in db["rules"]:
        if r["op"] != "single" or r["m"][0] < 129 or r["n"][0] < 129 or r["m"][1] > 256:
            continue
        for n in r["n"]:
            for m in ([n] if r.get("square") else r["m"]):
                m = m if r.get("square") else max(m, n + 1)
                assert m > r["m"][1] or (m, n) in timed, (r, m, n)
    for k in (129, 160, 192, 256):
        assert (k, k) in timed


def test_loaded_rules_route_squares(tmp_path, monkeypatch):
    """load_tune_db's rules, put into the host dispatch: squares follow their
    own rule, their neighbours the range's."""
    from paper_2506_09463_amd import hqr
    from tests.host_lib import HostLib
    host = HostLib(tmp_path)
    monkeypatch.setattr(hqr, "tune_clear", lambda: None)
    monkeypatch.setattr(hqr, "tune_set", lambda op, a, b, c, d, choice, prec=0: host.lib.hqr_tune_set(
        op, a, b, c, d, prec, choice))
    hqr.load_tune_db()
    db = _db()
    for m, n in [(129, 129), (140, 130), (161, 160), (176, 176), (192, 192), (193, 192), (256, 160), (256, 200), (256, 256)]:
        host.log()
        assert host.factor(m, n) == 0
        one = any(l.startswith("launch wg_single_kernel") for l in host.log())
        assert one == (_first(db["rules"], m, n)["choice"] != "blocked"), (m, n)
        # a stored factor of more than 128 columns: panel by panel, whatever the rule
        host.log()
        assert host.apply(m, n, 3) == 0
        assert any(l.startswith("launch stored_step_kernel") for l in host.log()), (m, n)
