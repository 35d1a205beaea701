"""The benchmark's line (no GPU): one short line with what is measured of the headline
workload, whatever else was measured beside it."""
import json

import bench

RUN = {"value": 1234567890.123456, "ms_per_step": 0.1234567890123456, "drift": {"all": {"slope": 1.25e-7}},
       "kernels": {k: {"ms_per_step": 0.1, "ms_per_launch": 0.1} for k in ("near", "far", "nlist", "energy")}}
SERVED = {"step_ms_p50": 1.719451904296875, "step_ms_p99": 2.0420188903808594, "wall_s": 0.2139,
          "requests_per_s": 1196.62795664037, "particle_steps_per_s": 1208615738.1153696}


def everything():
    part = {"rel_rms": 3.646718338778331e-14, "max_particle": 1.7146939169531502e-13}
    force = {g: {"total": part, "near": part, "far": part} for g in ("gamma_0.1", "gamma_100")}
    return {
        "metric": bench.METRIC, "value": 712345678.1234567, "unit": "particle-steps/s", "n_gpus": 1, "steps": 200,
        "warmup": 20, "ms_per_step": 1.4038123456789012, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "ocp_n1000000_k0.1_rc5_p500_g0.1+g100", "N": 1000000, "kappa": 0.1,
                   "gamma": [0.1, 100.0], "r_c": 5.0, "P": 500, "eps": 1e-4, "dt": 0.01, "nve_steps_per_run": 200,
                   "force_rel_rms": force},
        "mixed": dict(RUN, speedup_vs_fp64=1.5, dtype="f32 pair and phase arithmetic", force_rel_rms=force),
        "runs": {f"gamma_{g}": {"fp64": RUN, "mixed": RUN} for g in (0.1, 100)},
        "roofline": {"kernel": "near+rho_partial", "bound": "alu", "achieved": 48.56901312380008, "peak": 78.6,
                     "unit": "TFLOP/s", "frac": 0.6179263756208663, "traffic": 63941365.08167116,
                     "ms_per_launch": 0.0471, "basis": "words " * 40, "valu_counters": {"valu_busy": 0.79}},
        "kernel_rooflines": {k: dict(RUN) for k in ("near", "far", "nlist")},
        "elementary_prices_fma_slots": {"exp": 20.1},
        "cpu_baseline": {"value": 1253083.896357407, "unit": "particle-steps/s", "cores": 16, "kind": "oracle",
                         "sample": "words " * 30, "cpu_model": "words " * 10},
        "extra": {"ocp_n1000_k1_g1": RUN, "ocp_n100000_k0.5_g10": {"fp64": RUN, "mixed": RUN, "force_rel_rms": force},
                  "mixture_n200000": {"fp64": RUN, "mixed": RUN}, "variance_ocp_n1000_p20": {"rows": [RUN] * 10},
                  "served": {"saturated": SERVED, "poisson": {r: SERVED for r in ("0.5", "0.8", "1.2")}}},
    }


def test_line():
    out = everything()
    line = bench.headline(out)
    text = json.dumps(line)
    assert len(text) < 2000 and "\n" not in text
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data"):
        assert line[key] == out[key]
    assert line["config"]["workload"] == out["config"]["workload"]
    assert line["config"]["force_rel_rms"]["gamma_100"]["rel_rms"] == 3.6467e-14
    assert line["extra"]["served"]["step_ms_p99"] == 2.042
    assert line["roofline"]["kernel"] == "near+rho_partial" and line["cpu_baseline"]["kind"] == "oracle"


def test_line_of_the_headline_alone():
    out = everything()
    del out["extra"]
    out["roofline"] = out["cpu_baseline"] = None
    out["config"]["force_rel_rms"] = {"gamma_0.1": None, "gamma_100": None}   # not checked
    line = bench.headline(out)
    assert line["roofline"] is None and line["cpu_baseline"] is None and "extra" not in line
