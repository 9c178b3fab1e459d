"""bench.py names the kernel it timed (no GPU): counter summaries of the
pair-symmetric evaluation are used for that evaluation only."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_kernel_of_a_size(monkeypatch):
    for v in ("NBODY_FORCE_TILE", "NBODY_TUNE_CACHE"):
        monkeypatch.delenv(v, raising=False)
    keys = {"traffic_bytes_per_launch": "1e9", "ds_executed_flop_per_interaction": "33",
            "fp32_executed_flop_per_interaction": "43"}
    monkeypatch.setattr(bench, "profile_keys", lambda path: keys)
    assert bench.pair_symmetric("ds", 1 << 20) and bench.pair_symmetric("ds", 24576)
    assert not bench.pair_symmetric("ds", 24575) and not bench.pair_symmetric("fp32", 1 << 20)
    assert bench.traffic_per_launch("ds", 1 << 20) == 1e9
    assert bench.traffic_per_launch("ds", 1 << 19) is None and bench.traffic_per_launch("fp32", 1 << 20) is None
    assert bench.executed_flops("ds", 1 << 20, 1000.0)["TFLOP_s"] == 33.0
    assert bench.executed_flops("ds", 16384, 1000.0) is None
    assert bench.executed_flops("fp32", 16384, 1000.0)["TFLOP_s"] == 43.0
    monkeypatch.setenv("NBODY_FORCE_TILE", "256,2,256")
    assert not bench.pair_symmetric("ds", 1 << 20) and bench.traffic_per_launch("ds", 1 << 20) is None
