"""The last line of bench.py, on the CPU: the metric's figures in a few
kilobytes, the tables of the paper's own tests beside it."""
import json

import bench


def test_the_line_is_short_and_keeps_the_metric():
    run = {"C_d": 1.0 / 3.0, "stable": True, "note": "x" * 200}
    out = {"metric": bench.METRIC, "value": 34793.123456789, "unit": "MLUPS", "n_gpus": 1,
           "vs_baseline": None, "config": {"cells": 256 ** 3},
           "forms_3d": {"fp32": {"ms_per_step": 0.48212345678901, "errors": [1e-6 / 3] * 100}},
           "ergun": {"runs": [run] * 40}, "packing": {"runs": [run] * 10}, "drag": {"runs": [run]}}
    assert len(json.dumps(out)) > 12000
    details, line = bench.split_line(out)
    got, more = json.loads(line), json.loads(details)
    assert len(line) < 4000 and "\n" not in line
    assert set(got) == set(out) - set(bench.DETAILS) and set(more) == set(bench.DETAILS)
    assert abs(got["value"] / out["value"] - 1) < 1e-6 and got["config"] == out["config"]
    assert more["ergun"]["runs"][39]["stable"] is True
