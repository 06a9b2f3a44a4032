"""The bench's printed record (no GPU): one line of a few kilobytes with every
field that identifies the run, the tables left to the file."""
import json

import bench


def record():
    per = [dict(op=op, dtype=dt, M=M, N=N, kernel="k" * 60, us=12345.67, us_min=12345.67, us_max=12345.67, GBps=6543.2,
                GFLOPs=54321.0, roof_frac=0.8765, roof_frac_bs=0.9876, bound="hbm")
           for dt in "DZ" for op in ("tsmttsm", "tsmm") for M, N in bench.WIDTHS]
    legs = {op: {f: {"speedup_vs_fp64": 1.234, "error_arithmetic": {"normwise": 1e-15}} for f in ("fp32_acc64", "fp32_acc32")}
            for op in ("tsmttsm", "tsmm")}
    return {
        "metric": bench.METRIC, "value": 5480.4, "unit": "GB/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 49.079,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64", "source_hash": "0" * 16,
        "data": "synthetic", "config": {"workload": "w" * 200, "calls_per_step": 36},
        "roofline": {"bound": "mfma", "achieved": 68.68, "kernel": "k" * 60, "kernel_symbol": "s" * 200, "frac": 0.87},
        "b_s": {"read_GBps": 7052.9, "copy_GBps": 5475.6, "note": "n" * 200}, "widths": per,
        "precision_form": {"note": "n" * 500, "widths": [dict(dtype=dt, M=M, N=M, uniform=legs) for dt in "DZ"
                                                         for M in (8, 16, 32, 64)]},
        "batched_form": {k: 5986.8 for k in ("us_persistent_graph", "us_128_launches", "us_orth_batched", "speedup_vs_launches",
                                             "roof_frac_persistent", "flops")},
        "small_k": {"us": 18.6, "us_graph": 16.8, "roof_frac_graph": 0.5, "note": "n" * 200},
        "autograd_form": [{"dtype": dt, "forward_us": 323.9, "backward_us": 893.6} for dt in "DZ"],
        "cpu_baseline": {"value": 14.97, "unit": "GB/s", "cores": 16, "kind": "oracle", "calls": [{}] * 100},
    }


def test_line_is_short_and_whole():
    out = record()
    line = bench.line_of(out, "detail.json")
    assert "\n" not in line and len(line) < 6000
    got = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config"):
        assert got[k] == out[k]
    assert len(got["calls"]) == 36 and got["calls"]["Z tsmm 32x8"] == [12345.67, 0.8765]
    assert len(got["speedup_vs_fp64"]) == 8 and got["detail"] == "detail.json"
    for leg in ("precision_form", "batched_form", "small_k", "autograd_form", "cpu_baseline"):
        del out[leg]
    assert json.loads(bench.line_of(out, "x"))["value"] == 5480.4
