"""The benchmark's line on stdout: the headline's keys as they are, the main figures of the
other sections, and short enough for a reader that keeps the last 8 KB of the output."""
import importlib.util
import json
import os


def bench():
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "bench.py")
    spec = importlib.util.spec_from_file_location("bench", path)
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def test_line_keeps_the_headline_and_stays_short():
    b = bench()
    run = {"requests": 16, "completed": 16, "all_converged": False, "solves_per_s": 9.6095, "latency_p50_s": 0.7751,
           "latency_p99_s": 1.6454, "peak_bytes": 30312810496,
           "by_size": {str(2 ** q): {"completed": 4, "converged": 2, "mean_iterations": 40.0, "latency_p50_s": 1.3259,
                                     "worst_ev": 1.9726545807767976e-08} for q in range(7, 13)}}
    mode = {name: run for name in ("saturation", "poisson_0.5", "poisson_0.8", "poisson_0.95")}
    solve = {"seconds": 0.2066, "solves_per_s": 4.841, "converged": True, "iterations": 286, "ms_per_iteration": 0.722,
             "ev_report": 5.836668999714588e-09}
    head = {"metric": "smoother GLUP/s", "value": 436.14, "unit": "GLUP/s", "n_gpus": 1, "steps": 20, "warmup": 5,
            "ms_per_step": 3.8467, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64",
            "data": "synthetic", "config": {"workload": "w" * 150, "n": 4096},
            "roofline": {"bound": "hbm", "achieved": 4551.6, "peak": 8000.0, "unit": "GB/s", "kernel": "k" * 60},
            "cpu_baseline": {"value": 0.2996, "unit": "GLUP/s", "sample": "s" * 150}}
    record = dict(head, variants={f"v{q}": {"glups": 457.8, "ms_per_100_sweeps": 3.66, "e_after_sweeps": 0.9960621489751867}
                                  for q in range(9)},
                  solve={"workload": "w" * 150, "f64": solve, "f32_refined": solve},
                  smoother_variants_solve={"workload": "w" * 150, "runs": {f"r{q}": dict(solve, options={"nu1": 8})
                                                                           for q in range(12)}},
                  serve={"workload": "w" * 300, "f64": mode, "f32_refined": mode}, config3=None, fp64_floor=None)
    assert len(json.dumps(record)) > 8192
    line = b.headline(record)
    assert len(json.dumps(line)) < 8192
    assert {k: line[k] for k in head} == head and set(line) == set(record)
    assert line["serve"]["f64"]["saturation"]["solves_per_s"] == 9.6095 and "by_size" not in json.dumps(line)
    assert line["solve"]["f32_refined"]["iterations"] == 286 and line["variants"]["v0"] == {"glups": 457.8}
