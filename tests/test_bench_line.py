"""bench.py's one line on standard output: complete, and short enough for a reader that keeps the last
2000 characters."""
import argparse
import json

import bench


def test_the_line_is_short_and_complete():
    legs = {"%s/%s" % (k, l): {"ms": 1234.56789, "GBps": 4567.890123} for k in ("fp16", "plain_fp16", "fp8", "plain_fp8") for l in ("packed", "rowmajor")}
    roofline = {"kernel": "small_gemm_kernel, NestedFP16 over rowmajor planes (FP16-mode streaming GEMM, 128 launches/step)",
                "bound": "hbm", "achieved": 5123.456789, "peak": 8000.0, "unit": "GB/s", "frac": 0.6404321, "traffic": None,
                "avg_launch_us": 21.23456789, "algorithmic_bytes_per_launch": 109051904.0}
    cpu = {"value": 5.123456789, "unit": "GB/s", "cores": 128, "passes": 16, "what": "a sentence about the oracle " * 20}
    args = argparse.Namespace(steps=20, warmup=5, layers=32, no_graph=False)
    line, details = bench.report(args, 16, "rowmajor", 5123.456789, 4.123456789, roofline, cpu, {"legs_interleaved": legs, "prefill": [1.0] * 1000})
    got = json.loads(line)
    assert len(line) < 2000 and "\n" not in line
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
                "dtype", "data", "config"):
        assert key in got
    assert got["value"] == 5123.456789 and got["ms_per_step"] == 4.123456789
    assert json.loads(details)["extra"]["legs_interleaved"].keys() == legs.keys()
