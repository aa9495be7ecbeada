"""The benchmark's JSON line: one line that a caller who keeps the last 8 KB of
the output can still parse, whatever the legs measured."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

CONTRACT = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
            "vs_baseline", "dtype", "data", "config")


def full_result(kernels):
    """A result with every leg; `kernels` entries of the fine kernels in each."""
    x = 1234.5678
    fine = [{"kernel": "k" * 90, "achieved": x, "frac": x, "avg_launch_us": x, "traffic": 10 ** 10}] * kernels
    prec = {"levels": 7, "cycles": 11, "time_to_tol_ms": x, "ms_per_cycle": x, "vcycle_mpts_per_s": x, "rel_res": x,
            "cycle_GBps": x, "cycle_frac": x, "total_cycles": 77, "ms_per_sequence": x, "ms": x, "GBps": x,
            "times_ms": [x] * 5, "forward_ms": x, "forward_backward_ms": x, "fine_kernels": fine}
    both = {"mixed": prec, "fp64": prec, "fp32": prec}
    out = {k: k for k in CONTRACT}
    out.update(value=57634.1, ms_per_step=22.415, roofline={"kernel": "k" * 90, "other_fine_kernels": fine[:4]},
               fp64={k: v for k, v in prec.items() if k != "fine_kernels"},
               sweep={str(n): both for n in (32, 64, 128, 256, 512, 1024)}, b512=both,
               moving_mesh={**both, "gradient": both, "ablation": {str(k): prec for k in range(5)}},
               predictors={str(k): prec for k in range(5)}, accel={str(k): prec for k in range(4)},
               cpu_baseline={"sample": "s" * 250, "value": 11.6})
    return out


def test_line_is_short_and_complete():
    for kernels in (0, 4, 40):
        full = full_result(kernels)
        text = json.dumps(bench.headline(full))
        assert len(text) <= bench.LINE_MAX < 8000 and "\n" not in text
        line = json.loads(text)
        for k in CONTRACT + ("roofline",):
            assert line[k] == full[k]
    legs = bench.headline(full_result(0))["legs"]
    assert legs["b512"]["mixed"]["ms_per_cycle"] == 1234.5678
    assert legs["sweep"]["1024"]["fp64"]["cycles"] == 11


def test_skipped_legs_are_left_out():
    full = {**full_result(0), "sweep": {}, "b512": None, "moving_mesh": None, "predictors": None, "accel": None}
    assert bench.headline(full)["legs"] == {}
