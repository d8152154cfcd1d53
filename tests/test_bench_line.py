"""The line bench.py prints is one JSON object with the fixed keys, short enough to survive in the last 2000 characters of an output."""
import json

import bench


def _record(cpu=True):
    rec = {k: None for k in bench.HEADLINE_KEYS}
    rec.update(metric="m" * 141, value=6985695776.948456, unit="chunks/s", n_gpus=1, steps=20, warmup=3, ms_per_step=0.27060540000007904,
               higher_is_better=True, scaling="weak", dtype="d" * 50, data="s" * 59,
               config={"workload": "w" * 140, "rows": 33554432, "chunks": 1890367, "instances": 256}, timing="t" * 400,
               roofline={"kernel": "k" * 90, "bound": "hbm", "achieved": 5802.910616569018, "peak": 8000.0, "unit": "GB/s",
                         "frac": 0.7253638270711272, "traffic": 1396483031},
               makespan_over_lower_bound={"max": 1.0189732142857142, "max_exact": "239337472/234881024"})
    if cpu:
        rec["cpu_baseline"] = {"cores": 16, "matches_gpu": True, "gpu_over_cpu": 2178.1700000000001, "sample": "x" * 200}
    return rec


def test_the_printed_line_is_short_and_keeps_the_fixed_keys():
    out = _record()
    out["workloads"] = {n: _record() for n in ("c3", "c4", "c5")}
    line = json.dumps(bench.headline(out, "/somewhere/bench_details.json"))
    assert len(line) <= bench.HEADLINE_BYTES and "\n" not in line
    got = json.loads(line)
    assert all(got[k] == out[k] for k in bench.HEADLINE_KEYS if k not in ("value", "ms_per_step"))
    assert abs(got["value"] / out["value"] - 1) < 1e-5 and abs(got["ms_per_step"] / out["ms_per_step"] - 1) < 1e-5
    assert set(got["workloads"]) == {"c3", "c4", "c5"} and got["workloads"]["c4"]["matches_cpu_oracle"] is True


def test_the_printed_line_without_cpu_baseline_and_with_a_failed_workload():
    out = _record(cpu=False)
    out["workloads"] = {"c3": _record(cpu=False), "c4": {"error": "RuntimeError: " + "e" * 500, "wall_s": 1.0}}
    line = json.dumps(bench.headline(out, ""))
    assert len(line) <= bench.HEADLINE_BYTES
    got = json.loads(line)
    assert got["details"] is None and got["workloads"]["c4"]["error"].startswith("RuntimeError")
