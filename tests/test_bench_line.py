"""The benchmark's result line leaves tables to the detail lines."""
import json

import bench


def test_brief_keeps_figures_and_drops_tables():
    rec = {"ms": 1.23456789, "n": 12, "ok": True, "rate": 184000.4, "bound": "hbm",
           "workload": "a sentence about the matrix, its levels and its probes",
           "eps": [1e-3, 1e-4], "sizes": list(range(32)),
           "log": {"time_s": {"0.001": 2.0 / 3}, "per_matrix": [{"n": i} for i in range(3)]}}
    got = bench.brief(rec)
    assert got == {"ms": 1.2346, "n": 12, "ok": True, "rate": 184000, "bound": "hbm",
                   "eps": [1e-3, 1e-4],
                   "log": {"time_s": {"0.001": 0.66667}}}
    assert json.loads(json.dumps(got)) == got
