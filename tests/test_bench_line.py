"""The line bench.py prints on stdout: every field that rates a run, within what fits the end of a kept output (2000 characters)."""
import gc
import json
import types

import bench


def test_the_line_is_short_and_complete():
    long = {"list": ["x" * 200] * 200}
    out = {"metric": "Conv3D fwd+bwd TFLOP/s (bf16, % MFMA peak); 192^3 U-Net train-step ms", "value": 705.1234567891234, "unit": "TFLOP/s",
           "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 27.123456789123456, "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
           "config": {"workload": "w" * 500, "budget_bytes": 17179869184, "instance_norm": True, "conv_flop_per_step": 19264123456789.0},
           "pct_mfma_peak": 28.20493827156494,
           "swap": {"budget_gib": 16.0, "n_swapped": 0, "bytes_out": 0, "measured_peak_device_bytes": 9876543210, "measured_peak_within_budget": True, **long},
           "loss": 0.9463769197463989, "kernels": long, "unet_step": long, "level0_192": long, "fp32": long,
           "roofline": {"bound": "mfma", "achieved": 1157.123456789, "peak": 2500.0, "unit": "TFLOP/s", "frac": 0.46284938271, "launches_per_step": 13,
                        "ms_per_launch": 0.37701234567, "kernel": "mfma_plane_stream[contracted channels >=96]", **long},
           "targets": {"swap_hidden_ge_0.8_at_16GiB": {"fp32_N2": {"met": True, "volume": "192^3", "hidden_frac": 0.9977814188234408, "bytes_out": 2038431744}}},
           "cpu_baseline": {"value": 0.011453152367262628, "unit": "TFLOP/s", "cores": 16, "kind": "oracle", "per_config": long}}
    line = bench.summary(out)
    assert len(json.dumps(line)) < 1800, len(json.dumps(line))
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config"):
        assert k in line
    assert abs(line["value"] / out["value"] - 1) < 1e-5 and line["config"]["global_batch"] == 2
    for k in ("targets", "cpu_baseline", "unet_step", "fp32"):      # a run of the headline alone
        out.pop(k)
    assert "cpu_baseline" not in bench.summary(out)


def test_timed_calls_start_behind_a_full_collection():
    """The call recorder begins with the collector's work done: none of the generations that it would walk in the first
    timed calls is due (a full collection inside a call's event pair has read as 37 ms of that kernel)."""
    mc = types.SimpleNamespace(**{name: None for name in bench.CallRecorder.NAMES})
    gc.collect(1)
    assert gc.get_count()[2] > 0
    with bench.CallRecorder(mc):
        assert gc.get_count()[1:] == (0, 0)
