"""bench.py's result line keeps the value and its time as measured, every key, and a
length that a log holds whole.  No GPU."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_short_line():
    sys.path.insert(0, ROOT)
    import bench
    run = {"form": "fp32", "observable": "averaged", "nu": 0.1, "seed": 1, "target": 1e-3,
           "status": "BFI_OK", "rel_err": 0.0010196367390727492, "seconds": 9.978813697999996,
           "evals": 1099504287744, "device_seconds": 9.912459714127705}
    line = {"metric": bench.METRIC, "value": 91263845723.27509, "unit": "evals/s", "n_gpus": 1,
            "ms_per_step": 11.76524850000007, "higher_is_better": True, "vs_baseline": None,
            "forms": {"fp64": {"kernel_ms": 11.750929927825927, "step_ms_each": [11.7] * 100}},
            "adaptive": [run] * 6, "adaptive_to_target": [run] * 18}
    short = bench.short_line(line)
    assert list(short) == list(line)
    for k in ("metric", "value", "unit", "n_gpus", "ms_per_step", "higher_is_better", "vs_baseline"):
        assert short[k] == line[k] and type(short[k]) is type(line[k])
    assert short["forms"] == {"fp64": {"kernel_ms": 11.7509}}
    assert short["adaptive"][0] == {"form": "fp32", "observable": "averaged", "nu": 0.1, "seed": 1,
                                    "target": 1e-3, "status": "BFI_OK", "rel_err": 0.00101964,
                                    "seconds": 9.97881}
    assert len(json.dumps(short["adaptive_to_target"])) <= 18 * 160
