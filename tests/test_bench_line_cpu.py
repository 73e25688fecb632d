"""The line bench.py prints stays short enough to be read back whole, however
much a run measures, and holds every field of the result contract."""
import json

import bench

KERNELS = ("zero", "spread", "fft_x", "fft_y", "fft_z", "interp", "direct", "finalize", "transpose", "prephase")


def _report():
    err = {"synthesis": 2.2045719482498062e-11, "analysis": 2.459205903619527e-11,
           "synthesis_max_rel_err": 6.204666932155533e-11, "analysis_max_rel_err": 1.0246818305012691e-10, "rows": 4096}
    roof = {"bound": "alu", "achieved": 93.71234567890123, "peak": 157.3, "unit": "TFLOP/s", "frac": 0.5957555359656149,
            "traffic": 123456789.0, "ops_per_term": 30.0,
            "issue_bound": {"term_rows_per_s": 3.88e12, "achieved_term_rows_per_s": 3.1e12, "frac": 0.8,
                            "valu_instr_per_term_row": 10.125}}
    kernels = {k: {"ms": 123.456, "launches": 1234, "GB_s": 2345.6} for k in KERNELS}
    q = {"median": 204.71234567, "p10": 204.51234567, "p90": 204.91234567}
    dirs = {"runs": 20, "synthesis_ms": q, "analysis_ms": q, "step_ms": q}
    mode = {"ms_per_step": 2407.512345678, "value": 828123.12345678, "ntrans": 1, "workload": "dense-dcos-30km-340578-vis",
            "dtype": "f32", "n_pairs_nufft": 13440, "n_pairs_direct": 0, "kernels": kernels,
            "rooflines": {k: roof for k in KERNELS}, "rel_l2_vs_oracle": err}
    return {
        "metric": bench.METRIC, "value": 4468123.123456789, "unit": "(vis+pix)/s", "n_gpus": 1, "steps": 20, "warmup": 5,
        "ms_per_step": 446.512345678901, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic", "config": {"workload": "ska-like 995000 vis x 1000000 pix (200 antennas, 50 hour angles, "
                                        "10-deg Fibonacci cap), synthesis+analysis", "eps": 1e-4, "n_vis": 995000,
                                        "n_pix": 1000000, "ntrans": 1},
        "roofline": roof, "roofline_kernel": "direct",
        "f64": {"value": 1676123.123456, "ms_per_step": 1190.312345, "steps": 4, "eps": 1e-9, "roofline": roof,
                "roofline_kernel": "direct"},
        "f32_over_f64": 2.6658123456, "plan_seconds": {"f32": 0.4123456, "f64": 0.2123456},
        "plan": {d: {k: 123456 for k in "abcdefghij"} for d in ("f32", "f64")},
        "kernels": {"f32": kernels, "f64": kernels}, "mode": {"direct_threshold": -1.0},
        "directions": {"f32": dirs, "f64": dirs}, "source_hash": "0123456789abcdef",
        "nufft_rooflines": {k: roof for k in KERNELS}, "modes": {f"another_mode_{i}_forced_nufft": mode for i in range(13)},
        "serving": {"p50_latency_s": 0.012345678901, "p99_latency_s": 0.112345678901, "slots": 8, "planners": 8,
                    "requests": 64, "alone_vs_mix_max_rel_diff": {"max": 1e-6, "median": 1e-7},
                    "vs_oracle": {"rows_per_request": 1024, "rel_l2_max": 3.05e-7, "all_within_eps": True,
                                  "per_request": [{"rid": i, "direction": "synthesis", "n_vis": 571186, "n_pix": 22542,
                                                   "rel_l2": 2.7255218664191474e-07,
                                                   "max_rel_err": 2.630655613098946e-07} for i in range(64)]}},
        "cpu_baseline": {"value": 3012.123456, "unit": "(vis+pix)/s", "cores": 16, "kind": "oracle",
                         "host_cpu": "AMD EPYC 9575F 64-Core Processor", "host_cpu_count": 256,
                         "sample": "4096 sampled visibility rows (9.1s) and 4096 sampled pixel rows (9.3s) of the full "
                                   "sums, extrapolated linearly to 995000+1000000 rows"},
        "rel_l2_vs_oracle": {"f32": err, "f64": err},
    }


def test_result_line_is_short_and_complete():
    out = _report()
    line = bench.result_line(out)
    assert len(line) < bench.RESULT_LINE_MAX <= 4000 and "\n" not in line
    d = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config", "roofline_kernel"):
        assert d[k] == out[k]
    for k in ("bound", "achieved", "peak", "unit", "frac", "traffic"):
        assert k in d["roofline"]
    assert d["f64"]["ms_per_step"] and d["rel_l2_vs_oracle"]["f32"] and d["serving"]["p99_latency_s"]
    assert len(d["modes_ms_per_step"]) == 13 and d["cpu_baseline"]["value"] > 0


def test_result_line_of_the_step_alone():
    """--no-modes --skip-f64 --no-cpu-baseline: only the step's own fields."""
    out = {k: v for k, v in _report().items() if k not in ("modes", "serving", "cpu_baseline", "rel_l2_vs_oracle",
                                                           "nufft_rooflines")}
    out.update(f64=None, f32_over_f64=None, directions=None)
    d = json.loads(bench.result_line(out))
    assert d["value"] == out["value"] and "f64" not in d and "modes_ms_per_step" not in d


def test_a_report_without_room_keeps_the_contract():
    out = _report()
    out["modes"] = {f"mode_{i:04d}": next(iter(out["modes"].values())) for i in range(2000)}
    line = bench.result_line(out)
    assert len(line) < bench.RESULT_LINE_MAX and json.loads(line)["value"] == out["value"]
