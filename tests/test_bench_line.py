"""The benchmark's printed line (no GPU): short enough to be kept whole, the headline untouched."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def test_compact_line():
    third = 1.0 / 3.0
    state = {f"key_{i}": third * i for i in range(26)}
    line = {"metric": bench.METRIC, "value": 1e3 * third, "ms_per_step": third, "steps": 3,
            "config": {"box_l": third}, "roofline": {"achieved": third},
            "step_configurations": {f"c{i}": dict(state) for i in range(3)},
            "kernels": {"tile_product": {"avg_us": third}},
            "forms": {**{f"f{i}": {"a": dict(state), "n": 30} for i in range(9)},
                      "theta_statics": {"states": [dict(state) for _ in range(12)], "tol": 0.01}},
            "eigen": {"scaling_with_N": {"states": [dict(state) for _ in range(18)], "fit": {"p": third}}}}
    assert len(json.dumps(line)) > 16000
    out = bench.compact(line)
    assert len(json.dumps(out)) < 12000
    for k in ("metric", "value", "ms_per_step", "steps", "config", "roofline"):
        assert out[k] == line[k]
    assert out["forms"]["theta_statics"] == {"states": 12, "tol": 0.01}
    assert out["eigen"]["scaling_with_N"] == {"states": 18, "fit": {"p": 0.333333}}
    assert out["kernels"]["tile_product"]["avg_us"] == 0.333333
    assert out["forms"]["f0"]["n"] == 30
    assert line["forms"]["theta_statics"]["states"][0]["key_1"] == third   # the input is left alone
