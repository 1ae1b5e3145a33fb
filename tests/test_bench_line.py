"""bench.py's line on stdout: the contract's fields whole, and short enough for a reader of the last kilobytes whatever
the complete record holds."""
import json

import bench


def test_line_is_short_and_complete():
    leg = {"value": 123456.789012345, "unit": "samples/s", "ms_per_step": 1.2345678901234567, "dtype": "bf16", "data": "synthetic",
           "config": {"workload": "some_array_B8_bf16", "B": 8}, "kernels": {f"kernel_{k}": {"ms_per_step": 0.1} for k in range(200)}}
    out = dict(metric="m", n_gpus=1, steps=20, warmup=5, higher_is_better=True, scaling="weak", vs_baseline=None, **leg,
               workloads={n: dict(leg) for n in ("c0", "c2", "c3", "c4")}, operators=[{"op": "x" * 100}] * 60, operators_note="n" * 500)
    line = bench.brief_line(out)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
              "dtype", "data", "config"):
        assert line[k] == out[k], k
    assert {n: w["value"] for n, w in line["workloads"].items()} == {n: leg["value"] for n in out["workloads"]}
    text = json.dumps(line)
    assert len(text) < 2000 and "\n" not in text
    assert "kernels" in out and "operators" in out                       # the record itself keeps everything
