"""The line that bench.py prints is short enough for a caller that keeps the last 8 KB of the output, is JSON, and has the headline's
fields as they were measured."""
import json

import bench


def _stream(blocks):
    lat = {"first": 50.91234567, "min": 43.1234567, "median": 44.1234567, "max": 47.1234567, "max_over_median": 1.0123456789,
           "slope_us_per_block": -0.00123456789}
    return {"workload": "block_480p_h20d112", "rope": "table", "blocks": blocks, "tokens_per_block": 10800, "us_per_block_stream": 36.123456789,
            "us_per_block_graph_replay": 37.123456789, "tokens_per_s": 289570123.456789, "hbm_GBps": 4744.123456789,
            "hbm_frac": 0.593123456789, "latency_us": lat, "latency_us_per_block": [44.12] * blocks,
            "latency_us_per_block_worst_of_3_passes": [44.12] * blocks, "library_bytes": 18120992,
            "peak_new_device_bytes_during_stream": 0, "allocated_bytes_after_block": [20894213120] * blocks,
            "device_bytes_in_use_after_block": [23148363776] * blocks, "memory_constant_over_stream": True,
            "roofline": {"bound": "hbm", "kernel": "block_step_mfma", "achieved": 4744.123456789, "peak": 8000.0, "unit": "GB/s",
                         "frac": 0.593123456789, "traffic": None, "algorithmic_bytes_per_launch": 176947200},
            "stream_ceiling": {"read_us": 17.0123456, "copy_us": 19.6123456}, "frac_of_stream_ceiling": 0.983123456789}


def test_line_is_short_and_keeps_the_headline():
    out = {"metric": "linear-attention tokens/s per layer (fwd)", "value": 363744262.1868666, "unit": "tokens/s", "n_gpus": 1, "steps": 20,
           "warmup": 5, "ms_per_step": 0.41567665999999726, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
           "dtype": "bf16", "data": "synthetic", "config": {"workload": "w" * 110, "B": 2, "H": 32, "N": 75600, "d": 64, "buffer_sets": 2},
           "roofline": {"bound": "hbm", "kernel": "apply", "achieved": 5477.551015611313, "peak": 8000.0, "unit": "GB/s",
                        "frac": 0.6846938769514141, "traffic": 123456789, "traffic_source": "s" * 90},
           "block_stream": [_stream(10), _stream(80)] * 4 + [_stream(80)]}
    line = bench.printed_line(out)
    assert "\n" not in line and len(line) < 4000        # the other workloads' entries take about 3.4 KB more
    got = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype",
              "data", "config", "roofline"):
        assert got[k] == out[k]
    assert len(got["block_stream"]) == 9
    assert got["block_stream"][1]["latency_us"]["max_over_median"] == 1.0123 and got["block_stream"][1]["memory_constant_over_stream"] is True
