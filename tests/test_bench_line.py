"""The benchmark's line on stdout: everything that names the headline value, short enough to survive where only the end of
an output is kept."""
import json

import bench


def _result(text=""):
    head = {"name": "cfg2", "workload": "cfg2: single-layer LSTM I=256 H=1024 B=64 t=1000, BPTT-HSM budget m=50, seed 2" + text,
            "budget_m": 50, "ms_per_step": 10.472613912345678, "kernel_classes": {f"class {i}": {"net_us": 1 / 3} for i in range(400)}}
    config = {"model": "LSTM 256->1024", "global_batch": 64, "seq_len": 1000, "parallelism": "one GPU", "workload": head["workload"],
              "launch": "HIP graph replay", "budget_m": 50, "forward_ops": 2963, "peak_slots": 50, "slot_pool_bytes": 26214400,
              "workspace_bytes": 176543232}
    return {"metric": bench.METRIC, "value": 95487.123456789, "unit": "time-steps/s", "n_gpus": 1, "steps": 20, "warmup": 5,
            "ms_per_step": 10.472613912345678, "host_enqueue_ms": 0.8123456789, "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": "bf16", "data": "synthetic", "config": config,
            "cost_ratio_vs_store_all": {"measured": 1.5012345678, "theoretical": 1.6543333333, "store_all_ms": 6.9812345678},
            "kernel_classes": head["kernel_classes"], "memory": {str(i): i for i in range(300)},
            "roofline": {"bound": "mfma", "kernel": "forward_chain_kernel", "achieved": 381.23456789, "peak": 2500.0, "unit": "TFLOP/s",
                         "frac": 0.152493827, "traffic": 2861298.7120287684, "flops_per_launch": 671088640, "note": "x" * 300},
            "cpu_baseline": {"value": 167.0263231722436, "unit": "time-steps/s", "cores": 16, "kind": "oracle",
                             "sample": "first 908 of 1000 steps of cfg2 (float64 store-everything BPTT, numpy), 12.3 s"},
            "configs": [dict(head, name=f"cfg{i}", budget_m=b, ms_per_step=123.456789) for i in range(1, 6) for b in (50, 1000)]}


def test_the_line_is_short_and_complete():
    result = _result()
    line = json.dumps(bench.summary(result))
    assert len(line) <= bench.LINE_BYTES and "\n" not in line
    back = json.loads(line)
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
                "dtype", "data", "config"):
        assert back[key] == result[key]
    assert back["configs_ms_per_step"]["cfg3 m=50"] == 123.5 and back["roofline"]["frac"] == 0.1525
    assert back["cost_ratio_vs_store_all"]["measured"] == 1.501 and back["cpu_baseline"]["value"] == 167.0


def test_the_line_stays_short_when_names_are_long():
    line = json.dumps(bench.summary(_result("y" * 700)))
    assert len(line) <= bench.LINE_BYTES and json.loads(line)["ms_per_step"] == 10.472613912345678
