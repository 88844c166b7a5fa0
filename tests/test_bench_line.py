"""bench.py's result line stays under 2 kB whatever the run's records hold, and keeps
the fields its readers look for; the records in full go to the line of details."""
import json

import bench


def test_result_line_is_short_and_complete():
    curve = [[k, 1.0 / (k + 1), 0.1 * k] for k in range(400)]
    kernel = {"ms": 0.0925, "launches": 40, "achieved": 10.412, "frac": 0.2648, "traffic": 43720000.0,
              "valu_issue": {"instr_per_launch": 26780000.0, "frac": 0.4711},
              "l1_accesses": {"per_launch": 57030000.0, "per_cu_per_cycle": 1.01}}
    out = {"metric": "m" * 90, "value": 3100.0, "unit": "iterations/s", "n_gpus": 1, "steps": 100, "warmup": 5,
           "ms_per_step": 0.3226, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
           "dtype": "d" * 80, "data": "d" * 80,
           "config": {"workload": "512x512 " + "w" * 130, "iterations": 100, "timed_loop": "t" * 40},
           "roofline": {"bound": "alu", "kernel": "project", "achieved": 10.412, "peak": 39.3216, "unit": "u" * 50,
                        "frac": 0.2648, "traffic": 43720000.0, "kernels": {"project": kernel, "backproject": kernel},
                        "nnz": 240840802, "counters_measured_at": "c" * 40},
           "in_solve_ms": {"project": 0.0925}, "operators_ms": {"project": 0.0866},
           "stored_matrix_equivalent": {"bytes_per_call": 1929862992, "project_GBps": 20857.9,
                                        "backproject_GBps": 29294.1},
           "solve": {"k": 21},
           "time_to_target": {"workload": "w" * 80, "plain_ms_median": 7.044, "learned_ms_to_both_median": 11.79,
                              "learned_reached_f_and_tv_within_400": "19/32"},
           "batched": {"workload": "w" * 200, "slice_iterations_per_s": 1436.05},
           "cpu_baseline": {"value": 7.7217, "unit": "iterations/s", "cores": 16, "kind": "oracle",
                            "sample": "s" * 350, "single_core": {"value": 1.8, "sample": "s" * 90}},
           "quality_curves": {"curve": curve}, "stored_matrix": {"sizes": curve}, "large": {"curve": curve}}
    line, details = bench.result_lines(out)
    assert "\n" not in line and len(line) < 2000
    assert "\n" not in details and json.loads(details) == out
    d = json.loads(line)
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data"):
        assert d[key] == out[key]
    assert d["config"]["workload"] == out["config"]["workload"]
    for key in ("bound", "kernel", "achieved", "peak", "unit", "frac", "traffic"):
        assert d["roofline"][key] == out["roofline"][key]
    for name in ("project", "backproject"):
        assert d["roofline"]["kernels"][name]["valu_issue"]["frac"] == kernel["valu_issue"]["frac"]
    for key in ("value", "unit", "cores", "kind", "sample"):
        assert d["cpu_baseline"][key] == out["cpu_baseline"][key]
    # a run without its optional parts
    short = {k: out[k] for k in ("metric", "value", "config", "roofline")}
    assert set(json.loads(bench.result_lines(short)[0])) == set(short)
