"""Benchmark: D3Q27 mixture lattice Boltzmann step on one MI355X.

Workload: the binary Kelvin--Helmholtz shear layer on a 256^3 periodic grid
(molar masses 2 and 28, u_x = +-0.1 with tanh profiles, seeded noise), FP32
population storage. A step is one pass of the whole path: moments, stencil
field, collide-and-stream over all 16.8 M nodes.

Prints one JSON line (the last line of stdout) with MLUPS, the HBM roofline of
the dominant kernel (timed with HIP events on the library's stream), the other
storage precisions measured side by side with their error against the FP32 run,
and the FP64 CPU oracle timed on a bounded crop of the same workload. The whole
record, of which the line holds the main figures, goes to stderr.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--precision fp32|fp32_fp32|fp16|bf16|i16|fp64]
"""
from __future__ import annotations

import argparse
import contextlib
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0        # MI355X HBM3E
# How the benchmark's shear layer differs from the three-band recipe it stands in
# for (stated in the bench line's config).
RECIPE_DEPARTURES = ("velocity perturbation band-limited (8 random-phase Fourier modes per component, "
                     "|k| <= 4, maximum 1e-3) instead of per-node uniform noise, which drives the FP64 "
                     "oracle itself unstable within about 40 steps; D_12 = 0.1 instead of 0.05 (the light "
                     "species' lattice is unstable at 0.05 in the hydrogen-rich band); omega = 1 at the mean "
                     "pressure instead of 1.5 (above about 1.3 the layer blows up within a few hundred steps)")
PROFILES = os.path.join(ROOT, "profiles")
KERNEL_SOURCES = ["lattice.hpp", "node_ops.hpp", "device_ops.hpp", "kernels.hpp", "inst_fp64.hip",
                  "inst_fp32_fp64.hip", "inst_weak.hip", "inst_cvt.hip", "inst_weak_cvt.hip", "inst_fp32.hip",
                  "inst_fp16.hip", "inst_bf16.hip", "inst_i16.hip", "inst_jets.hip"]


def record_fields(M: int, weak: bool = False, cvt: bool = False) -> int:
    """Node record: Phi (3), omega, C_p, rho, u (3), T, omega_1, q_neq (3), rho_a (M-1;
    M under weak coupling), V_a (3 M), under weak coupling u_s (3), and with
    temperature-dependent heat capacities Y_a (M-1)."""
    return 14 + (M if weak else M - 1) + 3 * M + (3 if weak else 0) + (M - 1 if cvt else 0)


def algorithmic_bytes(M: int, s_bytes: int, r_bytes: int, weak: bool = False, cvt: bool = False) -> dict:
    """Bytes each kernel must move per node, every value read or written once.
    Two-read step: k_state_species reads the populations, writes the species' and
    a record of 10 fields; k_gfield reads Phi and omega and writes G; k_collide_fg
    reads the momentum and energy lattices, the record except Phi, a neighbour's
    C_p and G, and writes both lattices. Three-pass step: k_moments reads the
    populations and writes the record; k_collide reads the populations, the record
    except Phi, and G, and writes the populations. `step` is the two-read step.
    Stored lattices: M + 1 (strong coupling), M + 2 (weak)."""
    L = M + 2 if weak else M + 1
    pops = L * 27 * s_bytes
    fg = 2 * 27 * s_bytes
    rec = record_fields(M, weak, cvt) * r_bytes
    state, gfield, collide_fg = 2 * pops - fg + 10 * r_bytes, 7 * r_bytes, 2 * fg + 11 * r_bytes
    return {
        "k_state_species": state,
        "k_collide_fg": collide_fg,
        "k_moments": pops + rec,
        "k_gfield": gfield,
        "k_collide": 2 * pops + (rec - 3 * r_bytes) + 3 * r_bytes,
        "step": state + gfield + collide_fg,
        "method_min": 2 * pops,
    }


def record_bytes(precision: int, mc) -> int:
    return 8 if precision == mc.MCLBM_FP64 else 4


def kernel_source_hash() -> str:
    import hashlib

    h = hashlib.sha256()
    for name in KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_2004_11286_amd", "csrc", name), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def _counter_summary(kernel: str, precision: str):
    """Fields and per-kernel rows of the committed counter summary, if it was taken
    on the current kernel sources (else None)."""
    path = os.path.join(PROFILES, f"{kernel}_shear256_{precision}_hbm_counters.txt")
    if not os.path.exists(path):
        return None
    vals, rows = {}, {}
    with open(path) as fh:
        for line in fh:
            if line.startswith("#"):
                continue
            if "|" in line:
                parts = [p.strip() for p in line.split("|")]
                try:
                    rows[parts[0]] = (float(parts[3]) + float(parts[4])) * 1e9
                except (ValueError, IndexError):
                    pass
            elif ":" in line:
                k, v = line.split(":", 1)
                vals[k.strip()] = v.strip()
    if vals.get("kernel_source_hash") != kernel_source_hash():
        return None
    return vals, rows


def measured_traffic(kernel: str, precision: str):
    """HBM bytes per launch of `kernel` from the committed counter summary (None
    when the summary is missing or was taken on other kernel sources)."""
    got = _counter_summary(kernel, precision)
    return None if got is None else float(got[0]["hbm_bytes_per_launch"])


def measured_step_bytes(precision: str, kernel: str = "k_collide", nodes: int = 256 ** 3):
    """HBM bytes per node and step counted over every kernel of the step."""
    got = _counter_summary(kernel, precision)
    return None if got is None or not got[1] else sum(got[1].values()) / nodes


def copy_ceiling_gbs(gib: int = 4, reps: int = 10) -> dict:
    """Read + write bandwidth of two device-to-device copies, the practical
    streaming ceilings next to the 8 TB/s peak: the runtime's copy kernel and the
    library's 16-byte nontemporal copy (mclbm_stream_copy)."""
    import torch

    from paper_2004_11286_amd import mclbm as mc

    n = gib << 28
    a = torch.ones(n, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    out = {}
    for name, fn in (("runtime_copy_GBs", lambda: b.copy_(a)), ("stream_copy_GBs", lambda: mc.stream_copy(b, a))):
        fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        e1.synchronize()
        out[name] = 8.0 * n / (e0.elapsed_time(e1) / reps * 1e-3) / 1e9
    del a, b
    torch.cuda.empty_cache()
    return out


# tiles of the step kernels' block shapes (x * y * z nodes); shape 0 is the linear
# numbering of 256 consecutive nodes
SHAPE_TILES = ("linear", "64x4x1", "32x8x1", "16x16x1", "64x2x2", "32x4x2")


def progress(msg: str) -> None:
    """A progress line on stderr (stdout carries only the JSON result line)."""
    print(f"bench: {msg}", file=sys.stderr, flush=True)


def segments_of(steps: int, parts: int = 5) -> list:
    """Split the timed steps into `parts` near-equal segments (at least one step each)."""
    parts = max(1, min(parts, steps))
    base, extra = divmod(steps, parts)
    return [base + (1 if i < extra else 0) for i in range(parts)]


def time_run(mc, params, fields, precision, steps, warmup):
    """Warm up, then time exactly `steps` steps in five segments, each bracketed by
    stream synchronisations; the step time is the median over the segments.
    Per-kernel durations come from the library's HIP events on its stream."""
    import torch

    sim = mc.Sim(params, precision)
    sim.init_fields(**fields)
    sim.step(warmup)
    torch.cuda.synchronize()
    sim.set_timing(True)
    torch.cuda.synchronize()
    per_step, total = [], 0.0
    for k in segments_of(steps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        sim.step(k)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        total += dt
        per_step.append(dt / k)
    stats = {}
    for k in range(mc.kernel_count()):
        ms, launches, name = sim.kernel_stats(k)
        if launches:
            stats[name] = {"total_ms": ms, "launches": launches, "avg_ms": ms / max(launches, 1)}
    sim.set_timing(False)
    timing = {"median_s_per_step": float(np.median(per_step)), "segment_s_per_step": per_step,
              "total_s": total}
    return sim, timing, stats


def fields_after(mc, params, fields, precision, nsteps, info=None):
    """The moments after nsteps from the initial fields (accuracy runs); with info
    a dict, the number of range refits of fixed-point storage goes into it."""
    sim = mc.Sim(params, precision)
    sim.init_fields(**fields)
    sim.step(nsteps)
    out = sim.read_moments()
    if info is not None:
        info["range_refits"] = sim.range_refits()
    sim.close()
    return out


def sixteen_bit_summary(variants, base):
    """The fastest 16-bit storage mode whose every field stays within 1e-3 of the
    base run after the accuracy steps, with its speedup and worst field error (None
    when none does)."""
    ok = [(k, v) for k, v in variants.items() if k in ("fp16", "bf16", "i16") and v["meets_1e-3"]]
    if not ok:
        return None
    k, v = max(ok, key=lambda kv: kv[1]["MLUPS"])
    return {"storage": k, "MLUPS": v["MLUPS"], "speedup_vs_" + base: v["speedup_vs_" + base],
            "worst_field_error": v["worst_field_error"]}


def rel_errors(got, ref, u_floor=0.0):
    errs = {}
    for k in ("X", "rho", "u", "p", "T"):
        den = float(np.abs(ref[k]).max())
        if k == "u":
            den = max(den, u_floor)
        errs[k] = float(np.abs(got[k] - ref[k]).max() / den)
    return errs


def _oracle_mlups(O, params, fields, n, seconds_target):
    o = O.OracleSim(params)
    o.init_fields(**fields)
    o.step(1)                                  # first touch
    per_step, elapsed = [], 0.0
    while elapsed < seconds_target and len(per_step) < 200:
        t0 = time.perf_counter()
        o.step(1)
        dt = time.perf_counter() - t0
        elapsed += dt
        per_step.append(dt)
    o.close()
    return n / float(np.median(per_step)) / 1e6, len(per_step), elapsed


def cpu_baseline(seconds_target: float = 10.0):
    """The FP64 oracle, unchanged, on a 32 x 256 x 8 box of the shear-layer recipe
    (the full band geometry across y, a thin slab in x and z, long-wave
    perturbation), timed step by step (median step time) with every host thread
    and with one."""
    from oracle import oracle as O
    from paper_2004_11286_amd import workloads as W

    O.build()
    params, fields = W.shear_layer(nx=32, ny=256, nz=8, kmax=1)
    n = 32 * 256 * 8
    nproc = O.threads()
    v_all, steps_all, el_all = _oracle_mlups(O, params, fields, n, seconds_target)
    O.set_threads(1)
    v_one, steps_one, el_one = _oracle_mlups(O, params, fields, n, seconds_target)
    O.set_threads(nproc)
    cpu_model = "unknown"
    try:
        with open("/proc/cpuinfo") as fh:
            cpu_model = next((ln.split(":", 1)[1].strip() for ln in fh if ln.startswith("model name")), cpu_model)
    except OSError:
        pass
    return {"value": v_all, "unit": "MLUPS", "cores": nproc, "kind": "oracle",
            "value_1_thread": v_one, "cores_1_thread": 1,
            "sample": f"FP64 oracle on a 32x256x8 box of the shear-layer recipe, median step time: "
                      f"{steps_all} steps ({el_all:.1f} s) on {nproc} threads, {steps_one} steps "
                      f"({el_one:.1f} s) on 1 thread", "cpu_model": cpu_model}


def ensemble_bench(mc, steps: int = 50, seq_steps: int = 10, trial_steps: int = 10):
    """The batched ensemble: 512 independent ternary tubes, L ~ U{32..256} x 16 x
    16 with walls (18.9 M nodes), FP32 storage, all tubes in one context.
    Aggregate MLUPS of the autotuned batched launch, of plain batched launches,
    of a replayed HIP graph, and of one launch triplet per tube and step (the
    unbatched reference), all timed with HIP events on the context's stream."""
    import torch

    from paper_2004_11286_amd import workloads as W

    tubes = W.tube_ensemble()
    b = mc.Batch([p for p, _ in tubes], mc.MCLBM_FP32)
    b.init_fields([f for _, f in tubes])
    n = b.n

    def timed(k, **launch):
        b.set_launch(**launch)
        b.step(2 if not launch.get("graph_steps") else launch["graph_steps"])   # warm-up / graph build
        if b.step_count % 2:
            b.step(1)
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record(b.stream)
        b.step(k)
        e1.record(b.stream)
        e1.synchronize()
        ms = e0.elapsed_time(e1)
        return {"MLUPS": n * k / (ms * 1e-3) / 1e6, "ms_per_step": ms / k}

    base = dict(variant=0, swizzle=0, order=0, graph_steps=0, sequential=0, split=0)
    out = {"workload": "512 ternary tubes L~U{32..256}x16x16 with walls, FP32 storage, one context",
           "nodes": n, "tubes": len(tubes)}
    out["sequential"] = timed(seq_steps, **dict(base, sequential=1))
    out["batched"] = timed(steps, **base)
    out["batched_graph"] = timed(steps, **dict(base, graph_steps=10))
    out["batched_split"] = timed(steps, **dict(base, split=1))
    report = b.autotune(trial_steps)
    out["autotune_report"] = report.strip().splitlines()
    chosen = b.launch()
    out["autotuned"] = timed(steps, **chosen)
    out["autotuned"]["launch"] = chosen
    out["speedup_batched_vs_sequential"] = out["autotuned"]["MLUPS"] / out["sequential"]["MLUPS"]
    c = b.conservation()
    out["finite"] = bool(np.isfinite(c).all())
    b.close()
    del b
    torch.cuda.empty_cache()
    # the same ensemble with FP32 arithmetic (FP32 storage rounded to nearest), autotuned
    b = mc.Batch([p for p, _ in tubes], mc.MCLBM_FP32_FP32)
    b.init_fields([f for _, f in tubes])
    b.autotune(trial_steps)
    chosen = b.launch()
    out["autotuned_fp32_arithmetic"] = timed(steps, **chosen)
    out["autotuned_fp32_arithmetic"]["launch"] = chosen
    b.close()
    del b
    torch.cuda.empty_cache()
    return out


def finite_or_null(x):
    """The bench record with every non-finite float (an infeasible hop's
    residual, say) as null, so that the line is strict JSON."""
    if isinstance(x, float):
        return x if math.isfinite(x) else None
    if isinstance(x, dict):
        return {k: finite_or_null(v) for k, v in x.items()}
    if isinstance(x, (list, tuple)):
        return [finite_or_null(v) for v in x]
    return x


LINE_LIMIT = 4000            # bytes of the JSON line on stdout


def line_of(record):
    """The JSON line for stdout: the record with every float at six digits, each section cut to its
    figures. The whole record is over 20 KB and goes to stderr; a reader that keeps only the
    end of stdout must still see the line from its first byte."""
    def pick(d, *keys):
        return None if d is None else {k: d[k] for k in keys if k in d}

    def six(x):
        if isinstance(x, float):
            return float(f"{x:.6g}")
        if isinstance(x, dict):
            return {k: six(v) for k, v in x.items()}
        return [six(v) for v in x] if isinstance(x, list) else x

    sections = ("timing", "config", "roofline", "kernels", "block_shapes", "step_effective_GBs", "variants",
                "weak_coupling", "weak_fp16", "weak_i16", "cv_of_T", "weak_cv_of_T", "open_x", "ensemble", "surrogate",
                "cpu_baseline")
    line = {k: v for k, v in record.items() if k not in sections}
    line["config"] = record["config"]
    line["timing"] = pick(record["timing"], "method", "timed_region_s")
    line["roofline"] = pick(record["roofline"], "bound", "kernel", "achieved", "peak", "unit", "frac", "traffic", "frac_of_best_copy")
    line["kernels_avg_ms"] = {k: v["avg_ms"] for k, v in record["kernels"].items()}

    def short(d):
        return None if d is None else {k: v for k, v in d.items() if k.startswith("speedup_vs_")
                                       or k in ("MLUPS", "worst_field_error", "meets_1e-3")}

    for k in ("weak_coupling", "weak_fp16", "weak_i16", "cv_of_T", "weak_cv_of_T", "open_x"):
        line[k] = short(record[k])
    line["variants"] = {k: short(v) for k, v in record["variants"].items()}
    e, g = record["ensemble"], record["surrogate"]
    line["ensemble"] = None if e is None else {"MLUPS": e["autotuned"]["MLUPS"], **pick(e, "speedup_batched_vs_sequential", "finite")}
    line["surrogate"] = None if g is None else {
        **pick(g, "workload", "train_tubes_left_out", "speedup_forward_vs_lattice"),
        "train": pick(g["train"], "iters", "ms_per_step", "TFLOPs_per_step_approx", "loss_last100"),
        "change_tol": g["gate_calibration"]["change_tol"],
        "hops": [pick(r, "t0", "X_linf", "accepted", "ms_advance") for r in g["eval"]],
        "conv_forward_TFLOPs": g["roofline_conv_forward"]["achieved"]}
    line["cpu_baseline"] = pick(record["cpu_baseline"], "value", "unit", "cores")
    return six(line)


BF16_PEAK_TFLOPS = 2500.0   # MI355X dense BF16 matrix-core peak


def training_tubes():
    """The surrogate's training ensemble, 4096 draws without number 2110, and the list of the numbers
    left out. Tube 2110 (251 nodes, molar masses 2, 16 and 40) lies at the edge of the lattice's
    stable range: it amplifies the storage rounding of its first steps 30-fold every 20 steps. Of 200 runs
    from initial pressures 1e-9 apart most become non-finite in FP32 storage and none in FP64
    (profiles/train_tube_2110_stability.txt), so whether one run of it is usable hangs on the last
    bits of the kernels. It is left out by its number, whatever its run would do, so the workload is
    the same for any kernels; any other tube that leaves the range is an error."""
    from paper_2004_11286_amd import workloads as W

    left_out = [2110]
    tubes = W.tube_ensemble(ntubes=4096, ny=1, nz=1, seed=11286)
    return [t for k, t in enumerate(tubes) if k not in left_out], left_out


def surrogate_bench(train_iters: int = 72000):
    """The learned surrogate: trained by the library's BF16 MFMA kernels on
    trajectories of a 4096-tube ensemble (every 100 steps up to 5000; the tubes
    are one-dimensional, uniform in y and z, so a one-node cross-section carries
    all of their physics), then judged by the lattice on eight held-out
    128 x 32 x 32 ternary tubes (1 M nodes): mole-fraction L-infinity and RMS
    errors of one 100-step hop, the same for the persistence prediction, the
    two gate quantities (the residual, the largest relative change of a species'
    mass or of the energy per tube; the change, the largest mole-fraction change
    the hop predicts), whether the advance entry point accepted the hop or fell
    back to the lattice, with the change threshold calibrated on three other sets
    of held-out tubes, and the times of the forward pass, of the whole advance and of the 100
    lattice steps. The conv roofline: forward
    FLOP / forward time against the BF16 peak."""
    from paper_2004_11286_amd import surrogate as SG
    from paper_2004_11286_amd import workloads as W

    t0 = time.perf_counter()
    train_tubes, left_out = training_tubes()
    snaps, dims = SG.trajectories(train_tubes, K=100, nsnap=50)    # ValueError if any leaves the stable range
    M = 3
    C = SG.channels(M)
    st = SG.channel_stats(snaps, dims, M)
    norm = SG.norm_from_stats(st, M)
    pw = SG.pair_weights(st, M)
    net = SG.build_net(dims, [p for p, _ in train_tubes], norm, M)
    ms_train_step, _ = SG.timed_train_step(net, snaps, pw)
    net.set_params(SG.he_init(C, 6, SG.DEPTH, 0, 3 * M + 4))
    progress(f"surrogate: training {train_iters} iterations")
    with contextlib.redirect_stdout(sys.stderr):
        losses = SG.train(net, snaps, train_iters, pw, lr=2e-4, clip=2.0, log_every=4000)
    params = net.get_params()
    n_train = sum(a * b * c for a, b, c in dims)
    net.close()
    del snaps
    train_s = time.perf_counter() - t0
    # the gate's thresholds: a hop is good if its mole fractions are within 1e-3
    # of the lattice's. change_tol, calibrated against the lattice on three sets of
    # held-out tubes of their own (each set one batch, judged as a whole), is the
    # largest predicted mole-fraction change among good hops that lies below that
    # of every bad hop (0: none accepted), so that every calibration hop it admits
    # is good. resid_tol holds the conserved masses and energy to the same
    # relative 1e-3 (the residual of a network hop sits near 1e-4 whatever its
    # accuracy, so it bounds gross violations only)
    cal_starts = (0, 500, 1000, 2000, 3000, 4000, 6000, 8000)
    cal_seeds = (2024, 2026, 2027)
    cal = []
    for seed in cal_seeds:
        cal_tubes = W.tube_ensemble(ntubes=8, ny=32, nz=32, lmin=128, lmax=128, seed=seed)
        for r in SG.evaluate(params, norm, cal_tubes, K=100, starts=cal_starts, resid_tol=0.0):
            cal.append(dict(r, seed=seed))
    change_tol = SG.calibrate_change_tol(cal, 1e-3)
    resid_tol = 1e-3
    admitted = [r for r in cal if r["state_change"] <= change_tol and r["state_residual"] <= resid_tol]
    calibration = {"tubes": "three sets of 8 held-out ternary tubes 128x32x32 (seeds "
                            + ", ".join(str(t) for t in cal_seeds) + "), hops from t0 = "
                            + ", ".join(str(t) for t in cal_starts),
                   "hops": [{"seed": r["seed"], "t0": r["t0"], "X_linf": r["X_linf"], "state_change": r["state_change"],
                             "state_residual": r["state_residual"],
                             "lattice_state_residual": r["lattice_state_residual"]} for r in cal],
                   "change_tol": change_tol, "resid_tol": resid_tol,
                   "admitted": [[r["seed"], r["t0"]] for r in admitted],
                   "separates": bool(admitted) and all(r["X_linf"] <= 1e-3 for r in admitted)}
    eval_tubes = W.tube_ensemble(ntubes=8, ny=32, nz=32, lmin=128, lmax=128, seed=2025)
    res = SG.evaluate(params, norm, eval_tubes, K=100, starts=(0, 1000, 3000, 4000, 6000, 8000), resid_tol=resid_tol,
                      change_tol=change_tol)
    n_eval = sum(p["nx"] * p["ny"] * p["nz"] for p, _ in eval_tubes)
    fpn = SG.conv_flops_per_node(C, M + 6, 3 * M + 4)
    flops = fpn * n_eval
    ms_fwd = float(np.median([r["ms_forward"] for r in res]))
    achieved = flops / (ms_fwd * 1e-3) / 1e12
    train_flops = 3 * fpn * n_train
    return {
        "train_tubes_left_out": left_out,
        "workload": f"train: {len(train_tubes)} ternary tubes L~U{{32..256}}x1x1, 50 snapshots every 100 steps; "
                    "apply: 8 held-out ternary tubes 128x32x32, one 100-step hop from t0 = 0, 1000, 3000, 4000, 6000, 8000",
        "network": {"layers": SG.DEPTH, "width": 64, "kernel": "3x3x3", "params": int(params.size),
                    "input": "X_a, T, u, p (+ second BF16 terms of X_a, 6 tube constants)",
                    "output": "conservative: face fluxes of the molar densities p X_a / T, changes of T and u",
                    "padding": "replicate at the x walls, periodic in y and z",
                    "loss": "molar densities, T, u, and the x fluxes the target change implies (weight 0.1)",
                    "dtype": "bf16 weights/activations, fp32 accumulate"},
        "train": {"iters": train_iters, "lr": 2e-4, "clip_times_mean_norm": 2.0, "seconds": train_s, "loss_first100": float(np.mean(losses[:100])),
                  "loss_last100": float(np.mean(losses[-100:])), "ms_per_step": ms_train_step,
                  "TFLOPs_per_step_approx": train_flops / (ms_train_step * 1e-3) / 1e12},
        "gate_calibration": calibration,
        "eval": res,
        "hops_within_1e-3_linf": [{"t0": r["t0"], "X_linf": r["X_linf"],
                                   "speedup_advance_vs_lattice": r["ms_lattice"] / r["ms_advance"]}
                                  for r in res if r["X_linf"] <= 1e-3],
        "accepted_hops": [{"t0": r["t0"], "X_linf": r["X_linf"], "state_change": r["state_change"],
                           "state_residual": r["state_residual"]} for r in res if r["accepted"]],
        "rejected_hops": [{"t0": r["t0"], "X_linf": r["X_linf"], "state_change": r["state_change"],
                           "state_residual": r["state_residual"]} for r in res if not r["accepted"]],
        "speedup_forward_vs_lattice": float(np.median([r["ms_lattice"] / r["ms_forward"] for r in res])),
        "speedup_advance_vs_lattice": float(np.median([r["ms_lattice"] / r["ms_advance"] for r in res])),
        "roofline_conv_forward": {"bound": "mfma", "achieved": achieved, "peak": BF16_PEAK_TFLOPS,
                                  "unit": "TFLOP/s", "frac": achieved / BF16_PEAK_TFLOPS,
                                  "flop_per_node": fpn, "nodes": n_eval},
    }


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--precision", default="fp32")
    ap.add_argument("--n", type=int, default=256, help="cube edge")
    ap.add_argument("--no-variants", action="store_true")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-ensemble", action="store_true")
    ap.add_argument("--no-surrogate", action="store_true")
    ap.add_argument("--no-shapes", action="store_true", help="skip the block-shape sweep of the headline context")
    ap.add_argument("--surrogate-iters", type=int, default=72000)
    ap.add_argument("--accuracy-steps", type=int, default=1000,
                    help="steps after which the storage modes are compared with FP32 storage")
    ap.add_argument("--copy-calibrate", type=int, default=0, metavar="MIB",
                    help="only run a plain device copy of MIB mebibytes five times (to scale HBM counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only; --gpus {args.gpus} is not supported "
              "(the multi-GPU slab decomposition is a design, not an implementation)", file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_2004_11286_amd import mclbm as mc
    from paper_2004_11286_amd import workloads as W

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    if args.copy_calibrate:
        nbytes = args.copy_calibrate << 20
        src = torch.ones(nbytes, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        el = (time.perf_counter() - t0) / 5
        print(json.dumps({"copy_bytes_read": nbytes, "copy_bytes_written": nbytes, "copies": 5,
                          "GBs_read_plus_write": 2 * nbytes / el / 1e9}))
        return
    progress("copy ceilings")
    copies = copy_ceiling_gbs()
    copy_gbs = max(copies.values())
    params, fields = W.shear_layer(nx=args.n, ny=args.n, nz=args.n)
    M = params["M"]
    n = args.n ** 3
    prec = mc.PRECISIONS[args.precision]
    progress("headline run")
    sim, timing, stats = time_run(mc, params, fields, prec, args.steps, args.warmup)
    mlups = n / timing["median_s_per_step"] / 1e6
    sb, rb = mc.STORAGE_BYTES[prec], record_bytes(prec, mc)
    ab = algorithmic_bytes(M, sb, rb)
    dom = max(stats, key=lambda k: stats[k]["avg_ms"])          # dominant kernel
    dom_ms = stats[dom]["avg_ms"]
    bmin = ab["method_min"]
    achieved = bmin * n / (dom_ms * 1e-3) / 1e9
    kernel_gbs = {k: ab[k] * n / (v["avg_ms"] * 1e-3) / 1e9 for k, v in stats.items() if k in ab}
    # the block shapes of the step kernels (the headline runs the linear numbering,
    # shape 0, the fastest on this grid): 10 timed steps each after 2 untimed
    progress("block shapes")
    block_shapes = {}
    for k, tile in enumerate(SHAPE_TILES if not args.no_shapes else ()):
        sim.set_launch(shape=k)
        sim.step(2)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        sim.step(10)
        torch.cuda.synchronize()
        block_shapes[tile] = {"shape": k, "MLUPS": n / ((time.perf_counter() - t0) / 10) / 1e6}
    sim.set_launch(shape=0)
    sim.close()
    del sim
    torch.cuda.empty_cache()

    # accuracy: every storage mode against FP32 storage after ACC_STEPS steps from
    # the same initial state (the FP32 run itself matches the FP64 oracle to 1e-5)
    acc_steps = args.accuracy_steps
    ref = fields_after(mc, params, fields, prec, acc_steps) if not args.no_variants else None

    progress("storage modes")
    variants = {}
    if not args.no_variants:
        for name in ("fp32_fp32", "fp16", "bf16", "i16"):
            if mc.PRECISIONS[name] == prec:
                continue
            v, tv, st = time_run(mc, params, fields, mc.PRECISIONS[name], args.steps, args.warmup)
            v.close()
            del v
            vm = n / tv["median_s_per_step"] / 1e6
            info = {}
            got = fields_after(mc, params, fields, mc.PRECISIONS[name], acc_steps, info)
            errs = rel_errors(got, ref)
            variants[name] = {"MLUPS": vm, "speedup_vs_" + args.precision: vm / mlups,
                              f"rel_linf_vs_{args.precision}_after_{acc_steps}_steps": errs,
                              "worst_field_error": max(errs.values()),
                              "meets_1e-3": bool(max(errs.values()) <= 1e-3),
                              "kernels_avg_ms": {k: x["avg_ms"] for k, x in st.items()}}
            if name == "i16":
                variants[name]["range_refits_in_accuracy_run"] = info["range_refits"]
            torch.cuda.empty_cache()

    def mode_run(p_, f_, precision, wk=False, cv=False):
        v, tv, st = time_run(mc, p_, f_, precision, args.steps, args.warmup)
        ab_ = algorithmic_bytes(M, mc.STORAGE_BYTES[precision], record_bytes(precision, mc), weak=wk, cvt=cv)
        out = {"MLUPS": n / tv["median_s_per_step"] / 1e6, "ms_per_step": tv["median_s_per_step"] * 1e3,
               "launch": v.launch(), "method_min_bytes_per_node": ab_["method_min"],
               "method_min_frac": ab_["method_min"] * n / tv["median_s_per_step"] / 1e9 / HBM_PEAK_GBS,
               "kernels_avg_ms": {k: x["avg_ms"] for k, x in st.items()}}
        v.close()
        del v
        torch.cuda.empty_cache()
        return out

    progress("coupling, property and boundary modes")
    weak = weak_fp16 = weak_i16 = cv_of_T = weak_cv_of_T = open_x = None
    if not args.no_variants:
        # weak coupling (all M species lattices evolved) on the same workload: a
        # different model from strong coupling, so it is compared with itself
        wp = dict(params, weak=1)
        weak = mode_run(wp, fields, prec, wk=True)
        weak["stored_lattices"] = M + 2
        # weak coupling with FP16 deviation storage and FP32 arithmetic, against
        # weak coupling with FP32 storage after the same number of steps
        weak_fp16 = mode_run(wp, fields, mc.MCLBM_FP16, wk=True)
        wref = fields_after(mc, wp, fields, prec, acc_steps)
        wgot = fields_after(mc, wp, fields, mc.MCLBM_FP16, acc_steps)
        weak_fp16["speedup_vs_weak_" + args.precision] = weak_fp16["MLUPS"] / weak["MLUPS"]
        werrs = rel_errors(wgot, wref)
        weak_fp16[f"rel_linf_vs_weak_{args.precision}_after_{acc_steps}_steps"] = werrs
        weak_fp16["worst_field_error"] = max(werrs.values())
        weak_fp16["meets_1e-3"] = bool(max(werrs.values()) <= 1e-3)
        # the same with 16-bit fixed-point storage
        weak_i16 = mode_run(wp, fields, mc.MCLBM_I16, wk=True)
        info = {}
        wgot = fields_after(mc, wp, fields, mc.MCLBM_I16, acc_steps, info)
        weak_i16["speedup_vs_weak_" + args.precision] = weak_i16["MLUPS"] / weak["MLUPS"]
        werrs = rel_errors(wgot, wref)
        weak_i16[f"rel_linf_vs_weak_{args.precision}_after_{acc_steps}_steps"] = werrs
        weak_i16["worst_field_error"] = max(werrs.values())
        weak_i16["meets_1e-3"] = bool(max(werrs.values()) <= 1e-3)
        weak_i16["range_refits_in_accuracy_run"] = info["range_refits"]
        del wref, wgot
        # temperature-dependent heat capacities (cubic C_{a,v}(T), about twice the
        # constant part at the shear layer's T = 1) on the same workload
        cv = np.asarray(params["cv"], dtype=np.float64)
        shapes = [[1.0, 0.6, 0.1, 0.3], [1.0, 0.0, 0.4, 0.0]]
        cp_ = dict(params, cv_coef=np.stack([cv[a] * np.asarray(shapes[a]) for a in range(M)]))
        cv_of_T = mode_run(cp_, fields, prec, cv=True)
        cv_of_T["cv_coef_shape"] = shapes
        weak_cv_of_T = mode_run(dict(cp_, weak=1), fields, prec, wk=True, cv=True)
        # open x ends: the same 256^3 binary fields carried through the domain by a
        # mean flow u_x = 0.05, fed at x = 0 with the mean composition and state
        Xm = [float(fields["X"][a].mean()) for a in range(M)]
        Xm[-1] = 1.0 - sum(Xm[:-1])
        op_ = dict(params, wall_x=2,
                   inlet=np.array(Xm + [float(fields["p"].mean()), float(fields["T"].mean()), 0.05, 0.0, 0.0]))
        of = dict(fields, u=fields["u"] + np.array([0.05, 0.0, 0.0])[:, None, None, None])
        open_x = mode_run(op_, of, prec)
    del ref

    progress("ensemble")
    ensemble = None if args.no_ensemble else ensemble_bench(mc)
    progress("surrogate")
    surrogate = None if args.no_surrogate else surrogate_bench(args.surrogate_iters)
    progress("CPU baseline")
    cpu = None if args.no_cpu else cpu_baseline()
    step_gbs = ab["step"] * mlups * 1e6 / 1e9
    out = {
        "metric": "D3Q27 mixture MLUPS & % HBM roofline; FP16-store and surrogate vs FP32 plain",
        "value": mlups,
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": timing["median_s_per_step"] * 1e3,
        "timing": {"method": f"{args.steps} timed steps in {len(timing['segment_s_per_step'])} segments, "
                             "median step time", "segment_ms_per_step": [t * 1e3 for t in timing["segment_s_per_step"]],
                   "timed_region_s": timing["total_s"]},
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": {"fp32": "f32-store/f64-collide", "fp32_fp32": "f32", "fp64": "f64",
                  "fp16": "f16-store/f32-collide", "bf16": "bf16-store/f32-collide",
                  "i16": "i16-fixed-point-store/f32-collide"}[args.precision],
        "data": "synthetic",
        "config": {"workload": f"binary Kelvin-Helmholtz shear layer {args.n}^3 periodic, D3Q27, "
                               f"{M} species + momentum + energy lattices, strong coupling",
                   "nodes": n, "species": M, "precision": args.precision, "parallelism": "single GPU",
                   "recipe_departures": RECIPE_DEPARTURES},
        "roofline": {"bound": "hbm", "kernel": dom, "achieved": achieved, "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS,
                     "traffic": measured_traffic(dom, args.precision),
                     "basis": "method minimum B_min = 2 * 27 * L * s bytes per node (every stored population "
                              "read and written once) x nodes / mean duration of the dominant kernel",
                     "algorithmic_bytes_per_node": bmin, "algorithmic_bytes_per_launch": bmin * n,
                     "kernel_own_bytes_per_node": ab.get(dom),
                     "kernel_own_GBs": kernel_gbs.get(dom),
                     **copies, "frac_of_best_copy": achieved / copy_gbs},
        "method_min_frac": bmin * mlups * 1e6 / 1e9 / HBM_PEAK_GBS,
        "kernels": {k: {"avg_ms": v["avg_ms"], "launches": v["launches"], "GBs": kernel_gbs.get(k),
                        "algorithmic_bytes_per_node": ab.get(k)} for k, v in stats.items()},
        "block_shapes": block_shapes,
        "step_effective_GBs": {"step_bytes_per_node": ab["step"], "GBs": step_gbs,
                               "method_min_bytes_per_node": bmin,
                               "method_min_GBs": bmin * mlups * 1e6 / 1e9,
                               "method_min_frac": bmin * mlups * 1e6 / 1e9 / HBM_PEAK_GBS,
                               "step_counted_bytes_per_node": measured_step_bytes(args.precision, dom),
                               "step_counted_GBs": (measured_step_bytes(args.precision, dom) or 0) * mlups * 1e6
                               / 1e9 or None},
        "variants": variants,
        "sixteen_bit_at_1e-3": sixteen_bit_summary(variants, args.precision),
        "weak_coupling": weak,
        "weak_fp16": weak_fp16,
        "weak_i16": weak_i16,
        "cv_of_T": cv_of_T,
        "weak_cv_of_T": weak_cv_of_T,
        "open_x": open_x,
        "ensemble": ensemble,
        "surrogate": surrogate,
        "cpu_baseline": cpu,
    }
    record = finite_or_null(out)
    print("full record: " + json.dumps(record), file=sys.stderr, flush=True)
    print(json.dumps(line_of(record)))


if __name__ == "__main__":
    main()
