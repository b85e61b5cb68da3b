"""The benchmark's line: the fields it has to carry, in a length that the tail of a log holds (a record with every layer of
every workload had grown past 27000 characters and was cut)."""
import json

import bench


def test_short_record():
    roofline = {"bound": "hbm", "achieved": 3042.1018749413906, "peak": 8000.0, "unit": "GB/s", "frac": 0.3802627343676738}
    layer = {"layer": "blk0.qkv", "T": 50432, "K": 768, "O": 2304, "level": "1:16", "ms": 0.11788449808955193,
             "useful_tflops": 94.62441346211783, "hbm_gbs": 2630.801276045699, "bound": "hbm", "parity_pass": True}
    out = {"metric": "m", "value": 433.2378975398313, "unit": "TFLOP/s", "n_gpus": 1, "steps": 20, "warmup": 5,
           "ms_per_step": 5.364042650000034, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16",
           "data": "synthetic", "config": {"workload": "w" * 200, "tokens": 50432, "layers": 48}, "roofline": roofline,
           "layers": [layer] * 48}
    for name in ("a", "b", "c", "d", "e", "f"):
        out[name] = {"workload": "w" * 300, "note": "n" * 100, "ms": 0.1488010007880, "roofline": roofline, "layers": [layer] * 16}
    line = json.dumps(bench.short_record(out))
    assert "\n" not in line and len(line) < 6000
    back = json.loads(line)
    for key in ("metric", "unit", "n_gpus", "steps", "warmup", "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config"):
        assert back[key] == out[key], key
    assert abs(back["value"] / out["value"] - 1) < 1e-4 and abs(back["ms_per_step"] / out["ms_per_step"] - 1) < 1e-4
    assert len(back["a"]["layer_ms"]) == 16 and back["roofline"]["bound"] == "hbm"
