"""The line that bench.py prints: every key that a reader of the line relies on,
in a length that a captured tail of the output holds (host only)."""
import json

import bench

KEYS = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
        "vs_baseline", "dtype", "data", "config")


def _form():
    return {k: 12345.678901234 for k in
            ("ms_per_step", "serial_ms_per_step", "p50_ms", "p99_ms", "converged_solves_per_s", "solves_per_s",
             "max_rel_cost_vs_fp64", "iterate_ms", "mean_iters")}


def test_line_is_short_and_complete():
    # four workloads of eight forms, two serving forms of six rates
    forms = {f"mixed_tol1e-{i}_umax10": _form() for i in range(8)}
    rate = {"rate": 50000.0, "solves_per_s": 46490.123, "p50_ms": 6.312345, "p99_ms": 37.012345, "launches": 12345}
    entry = {"best_form": "mixed_tol1e-4", "forms": forms, "roofline": {"bound": "hbm", "frac": 0.28578},
             "cpu_baseline": {"value": 30180.75, "sample": "x" * 100}, "max_iter_calibration": {"p99": 8}}
    line = {**dict.fromkeys(KEYS, 0), "config": {"workload": "w" * 90, "form": "mixed_tol1e-4"}, "serial": {"value": 1.0},
            **{k: entry[k] for k in ("forms", "roofline", "cpu_baseline", "max_iter_calibration")},
            "workloads": {w: entry for w in ("pm64", "arm4k", "quad1k")},
            "serving": {"workload": "s" * 300, "forms": {f: {"rates": [rate] * 6, "server_stats": {"a": 1}}
                                                         for f in ("fp64_tol1e-10", "mixed_tol1e-7")}},
            "bic_pipeline": {"workload": "b" * 200, "ms_per_batch": 0.595, "select_ms": 0.0764, "steps": 10}}
    short = bench.summary(line)
    assert all(k in short for k in KEYS) and len(json.dumps(short)) < 8000
    assert short["workloads"]["arm4k"]["forms"].keys() == forms.keys()
    assert short["bic_pipeline"] == {"ms_per_batch": 0.595, "select_ms": 0.0764}
    line["serving"] = line["bic_pipeline"] = None  # a run of one workload
    line["workloads"] = {}
    json.dumps(bench.summary(line))
