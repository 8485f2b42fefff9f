"""The benchmark's printed line: what a reader needs is on it, and it is short."""
import json

import bench


def test_short_line():
    kern = {f"k{i}": {"avg_ms": 0.123456789, "algorithmic_bytes": 1} for i in range(40)}
    out = {"metric": "m", "value": 308204996575.7076, "unit": "edges/s", "n_gpus": 1, "steps": 50,
           "warmup": 3, "ms_per_step": 0.21281608581542968, "higher_is_better": True,
           "scaling": "weak", "vs_baseline": None, "dtype": "int32", "data": "synthetic",
           "config": {"workload": "w", "n": 4194304}, "parity": True, "breakdown": kern,
           "roofline": {"kernel": "k", "frac": 0.0243907056, "traffic": None},
           "sampling": {"edge": [{"ratio": 0.1, "m": 5, "ac6": {"ms": 0.15118099, "n_live": 3}}]},
           "explicit26": {"ms": 0.8331234567, "kernels": kern, "stats": {"n_live": 7}}}
    s = short_line = bench.short_line(out)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step",
              "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config", "parity"):
        assert s[k] == out[k], k
    assert s["sampling"] == {"edge": [{"ratio": 0.1, "m": 5, "ac6": 0.151181}]}
    assert s["explicit26"] == {"ms": 0.833123} and "breakdown" not in s
    assert s["roofline"]["frac"] == 0.0243907 and s["roofline"]["traffic"] is None
    assert len(json.dumps(short_line)) < 1000
