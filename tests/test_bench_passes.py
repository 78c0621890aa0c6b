"""bench.py on the host: bytes from the passes the library reports, and the
committed counter profile of the two-step pass."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_crossings_per_step():
    sys.path.insert(0, ROOT)
    import bench
    assert bench.crossings((0, 20)) == 1.0
    assert bench.crossings((10, 0)) == 0.5
    assert bench.crossings((10, 1)) == 11 / 21     # the last odd step
    assert bench.crossings((20, 2)) == 11 / 21     # the same in two q-waves


def test_pass_profile_matches_source_and_launch():
    sys.path.insert(0, ROOT)
    import bench
    key = ("cfg3a", "k_pair")
    sha = bench.source_hash(bench.PAIR_SRC)
    with open(bench.TRAFFIC_FILES[key]) as fh:
        t = json.load(fh)
    v = bench.traffic_for(key, sha, t["launch"])
    assert v is not None and 1.0 <= v / t["algorithmic_bytes_per_step"] < 1.5
    assert bench.traffic_for(key, "0" * 16, t["launch"]) is None
    assert bench.traffic_for(key, sha, {"tile": 3, "zc": 16, "xcd": 2}) is None
