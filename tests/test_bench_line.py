"""The benchmark's JSON line (CPU): short enough to be kept whole, with every field of its contract."""
import json
import random

import bench

CONTRACT = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
            "vs_baseline", "dtype", "data", "config")


def record(full=True):
    rng = random.Random(4)
    f = lambda: rng.random() * 10.0 ** rng.randint(-9, 4)      # 17 digits, like any measured figure
    fields = {k: f() for k in ("X", "rho", "u", "p", "T")}
    kern = {k: f() for k in ("k_state_species", "k_gfield", "k_collide_fg")}
    mode = lambda: {"MLUPS": f(), "ms_per_step": f(), "launch": {"variant": 0}, "kernels_avg_ms": kern,
                    "speedup_vs_weak_fp32": f(), "rel_linf_vs_weak_fp32_after_1000_steps": fields,
                    "worst_field_error": f(), "meets_1e-3": False}
    hop = lambda t0: {"t0": t0, "K": 100, "accepted": False, **{k: f() for k in (
        "X_linf", "X_linf_persistence", "X_rms", "state_residual", "state_change", "ms_lattice", "ms_advance", "ms_forward")}}
    out = {"metric": "D3Q27 mixture MLUPS & % HBM roofline; FP16-store and surrogate vs FP32 plain", "value": f(),
           "unit": "MLUPS", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": f(),
           "timing": {"method": "20 timed steps in 5 segments, median step time",
                      "segment_ms_per_step": [f() for _ in range(5)], "timed_region_s": f()},
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32-store/f64-collide",
           "data": "synthetic",
           "config": {"workload": "binary Kelvin-Helmholtz shear layer 256^3 periodic, D3Q27, 2 species + momentum + "
                                  "energy lattices, strong coupling", "nodes": 16777216, "species": 2,
                      "precision": "fp32", "parallelism": "single GPU", "recipe_departures": bench.RECIPE_DEPARTURES},
           "roofline": {"bound": "hbm", "kernel": "k_collide_fg", "achieved": f(), "peak": 8000.0, "unit": "GB/s",
                        "frac": f(), "traffic": {"hbm_bytes": f()}, "basis": "x" * 160, "frac_of_best_copy": f()},
           "method_min_frac": f(), "kernels": {k: {"avg_ms": v, "launches": 20} for k, v in kern.items()},
           "block_shapes": {str(k): {"shape": k, "MLUPS": f()} for k in range(6)},
           "step_effective_GBs": {"GBs": f()}, "variants": {}, "sixteen_bit_at_1e-3": None, "weak_coupling": None,
           "weak_fp16": None, "weak_i16": None, "cv_of_T": None, "weak_cv_of_T": None, "open_x": None,
           "ensemble": None, "surrogate": None, "cpu_baseline": None}
    if full:
        out["variants"] = {k: mode() for k in ("fp32_fp32", "fp16", "bf16", "i16")}
        out["sixteen_bit_at_1e-3"] = {"storage": "i16", "MLUPS": f(), "speedup_vs_fp32": f(), "worst_field_error": f()}
        for k in ("weak_coupling", "weak_fp16", "weak_i16", "cv_of_T", "weak_cv_of_T", "open_x"):
            out[k] = mode()
        out["ensemble"] = {"workload": "512 ternary tubes L~U{32..256}x16x16 with walls, FP32 storage, one context",
                           "autotune_report": ["0 0 0 0 0 0 0 4.621779"] * 53, "autotuned": {"MLUPS": f()},
                           "speedup_batched_vs_sequential": f(), "finite": True}
        out["surrogate"] = {"train_tubes_left_out": [2110], "workload": "train: 4095 ternary tubes" + "x" * 150,
                            "train": {"iters": 72000, "ms_per_step": f(), "TFLOPs_per_step_approx": f(), "loss_last100": f()},
                            "gate_calibration": {"hops": [hop(k) for k in range(24)], "change_tol": f()},
                            "eval": [hop(t) for t in (0, 1000, 3000, 4000, 6000, 8000)],
                            "speedup_forward_vs_lattice": f(), "roofline_conv_forward": {"achieved": f()}}
        out["cpu_baseline"] = {"value": f(), "unit": "MLUPS", "cores": 16, "cpu_model": "x" * 40}
    return out


def test_the_line_is_short_and_complete():
    for full in (True, False):
        rec = record(full)
        text = json.dumps(bench.line_of(rec))
        line = json.loads(text)
        assert len(text) <= bench.LINE_LIMIT, len(text)
        for k in CONTRACT:
            assert k in line, k
            want = rec[k]
            assert line[k] == (float(f"{want:.6g}") if isinstance(want, float) else want), k
        if full:
            assert len(json.dumps(rec)) > 2 * bench.LINE_LIMIT
            assert line["variants"]["i16"]["MLUPS"] and len(line["surrogate"]["hops"]) == 6


def test_two_read_step_bytes():
    """Binary FP32 step: three lattices of 108 bytes read by the state pass and two again by the collision,
    each written once; ten record fields written, seven read again; G and C_p of a neighbour, Phi and omega once."""
    ab = bench.algorithmic_bytes(2, 4, 4)
    assert ab["k_state_species"] == 3 * 108 + 108 + 40
    assert ab["k_gfield"] == 16 + 12
    assert ab["k_collide_fg"] == 216 + 28 + 16 + 216
    assert ab["step"] == ab["k_state_species"] + ab["k_gfield"] + ab["k_collide_fg"] == 976
    assert ab["method_min"] == 2 * 3 * 108
