"""The benchmark's JSON line (CPU): valid JSON, short enough that the last 8,000
characters of the output hold all of it, the headline's fields untouched."""
import json
import math
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


def section(parts):
    """A further workload as the benchmark records it, 1.4 KB each."""
    one = {"workload": "w" * 200, "edges": 294017, "precision": "fp32+fp64 re-test", "cell_size": math.inf,
           "edges_per_s": 4922353525.736267, "ms_per_update": 0.059730980000267664, "latency_p50_us": 72.95949995977935,
           "latency_p99_us": 103.96987002764114, "stage_ms_per_update": {f"stage{k}": 1 / 3 for k in range(20)},
           "status_ok": True, "cpu_baseline": {"value": 1 / 3, "labels_match_gpu_on_sample": True, "sample": "s" * 100}}
    return {p: dict(one) for p in parts}


def test_line_is_short_and_complete(capsys):
    import bench
    rates = [{"offered_rate": 10.0 ** k, "achieved_rate": 1 / 3, "latency_p50_us": 1 / 3, "requests": 7} for k in range(3)]
    line = {"metric": "m" * 80, "value": 4.123456789e9, "unit": "edges/s", "n_gpus": 1, "steps": 20, "warmup": 5,
            "ms_per_step": 1 / 3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32+f64",
            "data": "synthetic",
            "config": {"workload": "w" * 200, "cell_size": math.inf,
                       "autotune": {"item_edges": 288, "candidates": [{"us": 1 / 3}] * 60}},
            "roofline": {"frac": 1 / 3, "kernel": "k"}, "second_forms": section("abcd"), "other_workloads": section("abcdef"),
            "batched_planar": section(("plain", "batched", "batched_graph")),
            "serving": {"rates": rates, "non_lazy": rates[0], "status_ok": True}}
    text = json.dumps(bench.headline(line), allow_nan=False)
    assert len(json.dumps(line)) > 12000 and len(text) < 7000
    out = json.loads(text)
    for k in line:
        assert k in out
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "dtype", "data", "vs_baseline"):
        assert out[k] == line[k]
    assert out["config"]["cell_size"] is None and out["config"]["autotune"] == {"item_edges": 288}
    assert out["other_workloads"]["f"]["edges_per_s"] == 4.92235e9
    assert out["second_forms"]["a"]["cpu_baseline"]["oracle_equal"] is True
    assert [r["offered_rate"] for r in out["serving"]["rates"]] == [1.0, 10.0, 100.0]
    assert "\"stage19\"" in capsys.readouterr().err    # the sections in full on stderr
    assert line["serving"]["rates"][0]["requests"] == 7 and "candidates" in line["config"]["autotune"]
