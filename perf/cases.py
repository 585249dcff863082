"""Performance cases: what a user of this framework has it do, through its public calls.

Seven kinds of work, each with a listed case or more and a range that ``draw``
samples:

- ``box``      a short run of the shear layer from given fields: mclbm_init_fields
               on device fields, some steps, the FP32 fields read back on the device;
- ``tube``     one diffusion tube carried on from where it stands: steps, then the fields;
- ``tubes``    the same for a batch of independent ternary tubes of uneven length;
- ``jets``     the opposed jets of Sec. 4.3, carried on;
- ``forward``  the surrogate network's forward pass over a set of tubes;
- ``train``    iterations of the surrogate's training loop on snapshots of
               one-dimensional tubes, then the weights read out;
- ``hop``      mclbm_nn_advance: a batch moved on by the network, then the fields.

``exact`` holds a plain FP64 torch form of the model step, of the network and of
its training iteration, written from the equations with no call into the package.
"""
from __future__ import annotations

import math

import numpy as np
import torch

# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest run: binary interdiffusion 64 x 8 x 8 in FP64 (launches and latency)
        {"name": "tube-binary-64x8x8-fp64", "kind": "tube", "M": 2, "nx": 64, "ny": 8, "nz": 8, "prec": "fp64",
         "steps": 100},
        # the ternary Loschmidt tube, 256 x 4 x 4 between walls, FP32 storage
        {"name": "tube-ternary-256x4x4-fp32", "kind": "tube", "M": 3, "nx": 256, "ny": 4, "nz": 4, "prec": "fp32",
         "steps": 100},
        # the paper's opposed jets at the paper's size: four species, 200 x 400 x 1
        {"name": "jets-200x400-fp32", "kind": "jets", "nx": 200, "ny": 400, "prec": "fp32", "steps": 50},
        # the flagship shear layer, 256^3, FP32 storage with FP64 arithmetic
        {"name": "box-256-fp32", "kind": "box", "nx": 256, "ny": 256, "nz": 256, "prec": "fp32", "weak": 0, "props": 0,
         "open": 0, "steps": 16},
        # 16-bit fixed-point storage, an ordinary ragged size
        {"name": "box-190x164x156-i16", "kind": "box", "nx": 190, "ny": 164, "nz": 156, "prec": "i16", "weak": 0,
         "props": 0, "open": 0, "steps": 48},
        # FP16 storage, odd in every direction
        {"name": "box-131x97x89-fp16", "kind": "box", "nx": 131, "ny": 97, "nz": 89, "prec": "fp16", "weak": 0,
         "props": 0, "open": 0, "steps": 32},
        # weak coupling: every species with its own lattice
        {"name": "box-128x120x100-weak-fp32", "kind": "box", "nx": 128, "ny": 120, "nz": 100, "prec": "fp32", "weak": 1,
         "props": 0, "open": 0, "steps": 24},
        # temperature-dependent heat capacities and transport
        {"name": "box-150x110x90-props-fp32", "kind": "box", "nx": 150, "ny": 110, "nz": 90, "prec": "fp32", "weak": 0,
         "props": 1, "open": 0, "steps": 24},
        # the ensemble: 512 independent ternary tubes, L ~ U{32..256} x 16 x 16, one context
        {"name": "tubes-512x16x16-fp32", "kind": "tubes", "ntubes": 512, "lmin": 32, "lmax": 256, "ny": 16, "nz": 16,
         "prec": "fp32", "steps": 8},
        # the surrogate's forward pass over its evaluation geometry
        {"name": "forward-8x128x32x32", "kind": "forward", "ntubes": 8, "nx": 128, "ny": 32, "nz": 32, "depth": 6},
        # the surrogate's training loop on its training geometry
        {"name": "train-4096-tubes", "kind": "train", "ntubes": 4096, "lmin": 32, "lmax": 256, "depth": 6, "iters": 3},
        # one accepted hop of the surrogate over its evaluation geometry
        {"name": "hop-8x128x32x32", "kind": "hop", "ntubes": 8, "nx": 128, "ny": 32, "nz": 32, "depth": 6},
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    """One more case of the same ranges; box, tubes and train weigh a little more than the rest."""
    kind = rng.choice(["box", "box", "box", "tube", "tube", "tubes", "tubes", "jets", "forward", "train", "train", "hop"])
    if kind == "box":
        mode = rng.choice(["fp32", "fp32", "fp32_fp32", "fp16", "i16", "fp64", "weak", "props", "open"])
        prec = mode if mode in ("fp32", "fp32_fp32", "fp16", "i16", "fp64") else "fp32"
        return {"kind": "box", "nx": _logint(rng, 32, 220), "ny": _logint(rng, 40, 200), "nz": _logint(rng, 8, 160),
                "prec": prec, "weak": int(mode == "weak"), "props": int(mode == "props"), "open": int(mode == "open"),
                "steps": rng.randint(12, 40)}
    if kind == "tube":
        M = rng.choice([2, 3])
        return {"kind": "tube", "M": M, "nx": _logint(rng, 32, 512), "ny": _logint(rng, 1, 16), "nz": _logint(rng, 1, 16),
                "prec": rng.choice(["fp64", "fp32", "fp32"]), "steps": rng.randint(40, 120)}
    if kind == "tubes":
        lmin = _logint(rng, 16, 48)
        return {"kind": "tubes", "ntubes": _logint(rng, 4, 500), "lmin": lmin, "lmax": _logint(rng, lmin + 8, 256),
                "ny": _logint(rng, 1, 16), "nz": _logint(rng, 1, 16), "prec": rng.choice(["fp32", "fp32", "fp32_fp32"]),
                "steps": rng.randint(8, 24)}
    if kind == "jets":
        return {"kind": "jets", "nx": _logint(rng, 48, 260), "ny": _logint(rng, 80, 420),
                "prec": rng.choice(["fp32", "fp64"]), "steps": rng.randint(20, 60)}
    if kind == "train":
        lmin = _logint(rng, 24, 64)
        return {"kind": "train", "ntubes": _logint(rng, 64, 3500), "lmin": lmin, "lmax": _logint(rng, lmin + 16, 256),
                "depth": rng.choice([4, 6]), "iters": 3}
    return {"kind": kind, "ntubes": rng.randint(1, 7), "nx": _logint(rng, 40, 160), "ny": _logint(rng, 4, 32),
            "nz": _logint(rng, 4, 32), "depth": 6}


# ------------------------------------------------------------------ inputs, from the seed alone
DEVICE = "cuda:0" if torch.cuda.is_available() else "cpu"
STORAGE_BYTES = {"fp64": 8, "fp32": 4, "fp32_fp32": 4, "fp16": 2, "i16": 2}
HOP = 100     # lattice steps one surrogate hop stands for


def _species(masses, D, mu, gamma=5.0 / 3.0, prandtl=0.71):
    m = np.asarray(masses, dtype=np.float64)
    cv = 1.0 / ((gamma - 1.0) * m)
    mu = np.full(m.shape, float(mu))
    return {"M": len(m), "molar_mass": m, "cv": cv, "D": np.asarray(D, dtype=np.float64), "mu": mu,
            "lambda": mu * gamma * cv / prandtl}


def _sym(off, M):
    """Symmetric diffusivities from the off-diagonal ones; the diagonal is the row's mean."""
    D = np.zeros((M, M))
    for (a, b), v in off.items():
        D[a, b] = D[b, a] = v
    for a in range(M):
        D[a, a] = sum(D[a, b] for b in range(M) if b != a) / (M - 1)
    return D


def _const(v, shape):
    return torch.full(shape, float(v), dtype=torch.float64, device=DEVICE)


def _step_tube(nx, ny, nz, masses, D, xl, xr, T0, wall):
    """Species data and fields of a tube whose halves hold the compositions xl and xr at rest at one pressure."""
    M = len(masses)
    P0 = T0 / (0.5 * (float(np.dot(xl, masses)) + float(np.dot(xr, masses))))
    params = dict(_species(masses, D, 0.5 * P0), nx=nx, ny=ny, nz=nz, wall_x=wall, slaved=M - 1)
    left = torch.arange(nx, device=DEVICE) < nx // 2
    ends = torch.tensor(np.stack([xl, xr]), dtype=torch.float64, device=DEVICE)
    X = torch.where(left, ends[0][:, None], ends[1][:, None])[:, None, None, :].expand(M, nz, ny, nx).contiguous()
    s = (nz, ny, nx)
    return params, {"X": X, "p": _const(P0, s), "T": _const(T0, s), "u": _const(0.0, (3,) + s)}


def _draw_tube(rng):
    """Masses, diffusivities and end compositions of a random ternary tube whose slaved (last) species
    carries at least 0.3 of the mass at both ends."""
    masses = np.sort(rng.choice([2.0, 16.0, 28.0, 40.0], size=3, replace=False))
    d = rng.uniform(0.01, 0.1, size=3)
    while True:
        xl, xr = rng.dirichlet([1.0, 1.0, 1.0]), rng.dirichlet([1.0, 1.0, 1.0])
        low = np.minimum(xl * masses / np.dot(xl, masses), xr * masses / np.dot(xr, masses))
        if low.max() >= 0.3:
            break
    order = np.argsort(low, kind="stable")
    return masses[order], _sym({(0, 1): d[0], (0, 2): d[1], (1, 2): d[2]}, 3), xl[order], xr[order]


def _box(case, rng):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    T0, masses = 1.0, (2.0, 28.0)
    P0 = T0 / 15.0
    params = dict(_species(masses, np.full((2, 2), 0.1), 0.5 * P0), nx=nx, ny=ny, nz=nz, wall_x=0, slaved=1,
                  weak=case["weak"])
    z, y, x = [torch.arange(k, dtype=torch.float64, device=DEVICE) for k in (nz, ny, nx)]
    s = 0.5 * (torch.tanh((y - ny / 4.0) / 4.0) - torch.tanh((y - 0.75 * ny) / 4.0))
    shape = (nz, ny, nx)
    X1 = (0.9 - 0.8 * s)[None, :, None].expand(shape)
    u = torch.zeros((3,) + shape, dtype=torch.float64, device=DEVICE)
    u[0] += (0.1 * (1.0 - 2.0 * s))[None, :, None]
    for c in range(3):
        pert = torch.zeros(shape, dtype=torch.float64, device=DEVICE)
        for _ in range(8):
            k = [int(rng.integers(-w, w + 1)) for w in (min(4, v // 8) for v in (nx, ny, nz))]   # long waves
            amp, ph = rng.uniform(-1.0, 1.0), rng.uniform(0.0, 2.0 * np.pi)
            pert += amp * torch.sin(2.0 * np.pi * ((k[0] / nx) * x[None, None, :] + (k[1] / ny) * y[None, :, None]
                                                   + (k[2] / nz) * z[:, None, None]) + ph)
        u[c] += 1e-3 * pert / float(pert.abs().max().clamp_min(1e-12))
    if case["props"]:
        cv = params["cv"]
        params["cv_coef"] = np.stack([cv[0] * np.array([1.0, 0.6, 0.1, 0.3]), cv[1] * np.array([1.0, 0.0, 0.4, 0.0])])
        params["transport_exp"] = np.array([0.7, 0.8, 0.75, 0.85, 1.75, T0 / 1.2])
    if case["open"]:
        u[0] += 0.05
        xm = float(X1.mean())
        params.update(wall_x=2, inlet=np.array([xm, 1.0 - xm, P0, T0, 0.05, 0.0, 0.0]))
    return params, {"X": torch.stack([X1, 1.0 - X1]).contiguous(), "p": _const(P0, shape), "T": _const(T0, shape), "u": u}


def _jets(case, rng):
    nx, ny = case["nx"], case["ny"]
    m = np.array([2.0, 32.0, 18.0, 28.0])                     # H2, O2, H2O, N2
    d = rng.uniform(-0.01, 0.01)
    xl, xr = np.array([0.1 + d, 0.0, 0.05, 0.85 - d]), np.array([0.0, 0.1 + d, 0.0, 0.9 - d])
    x0 = 0.5 * (xl + xr)
    phys = {(0, 1): 0.81, (0, 2): 0.95, (0, 3): 0.78, (1, 2): 0.26, (1, 3): 0.21, (2, 3): 0.26}
    D = _sym({k: v * 0.05 / 0.95 for k, v in phys.items()}, 4)
    P0, U = 1.0 / float(np.dot(x0, m)), float(rng.uniform(0.035, 0.045))
    ur = U * math.sqrt(float(np.dot(xl, m)) / float(np.dot(xr, m)))
    params = dict(_species(m, D, 0.5 * P0, gamma=1.4), nx=nx, ny=ny, nz=1, wall_x=3, wall_y=2, slaved=3,
                  nozzle=(int(round(0.1 * ny)), int(round(0.9 * ny))),
                  inlet=np.concatenate([xl, [P0, 1.0, U, 0.0, 0.0]]), inlet_right=np.concatenate([xr, [P0, 1.0, -ur, 0.0, 0.0]]))
    s = (1, ny, nx)
    X = torch.as_tensor(x0, device=DEVICE)[:, None, None, None].expand((4,) + s).contiguous()
    return params, {"X": X, "p": _const(P0, s), "T": _const(1.0, s), "u": _const(0.0, (3,) + s)}


def _lengths(case):
    """The tubes' lengths, U{lmin..lmax}: part of the case, not of its inputs."""
    rng = np.random.default_rng(case["ntubes"])
    return [int(v) for v in rng.integers(case["lmin"], case["lmax"] + 1, size=case["ntubes"])]


def _lattice_inputs(case, seed):
    """A list of (params, fields) per tube."""
    rng = np.random.default_rng(seed)
    if case["kind"] == "box":
        return [_box(case, rng)]
    if case["kind"] == "jets":
        return [_jets(case, rng)]
    if case["kind"] == "tubes":
        out = []
        for nx in _lengths(case):
            m, D, xl, xr = _draw_tube(rng)
            out.append(_step_tube(nx, case["ny"], case["nz"], m, D, xl, xr, 1.0 / 3.0, 1))
        return out
    a = float(rng.uniform(0.0, 0.1))
    if case["M"] == 2:          # binary interdiffusion of a step, periodic
        return [_step_tube(case["nx"], case["ny"], case["nz"], (2.0, 40.0), np.full((2, 2), 0.05), (0.75 + a, 0.25 - a),
                           (0.15 + a, 0.85 - a), 1.0 / 3.0, 0)]
    D = _sym({(0, 1): 0.083, (0, 2): 0.068, (1, 2): 0.017}, 3)      # one species absent on the left
    return [_step_tube(case["nx"], case["ny"], case["nz"], (2.0, 16.0, 40.0), D, (0.0, 0.45 + a, 0.55 - a),
                       (0.45 + a, 0.0, 0.55 - a), 1.0 / 3.0, 1)]


def _net_dims(case):
    if case["kind"] == "train":
        return [(nx, 1, 1) for nx in _lengths(case)]
    return [(case["nx"], case["ny"], case["nz"])] * case["ntubes"]


def _net_inputs(case, seed):
    """Tube constants, a pair of trajectory snapshots (fields now and one hop later, [8][n] per tube:
    X_1..X_3, T, u, p), the normalisation and the weights of the network."""
    rng = np.random.default_rng(seed)
    dims = _net_dims(case)
    tubes, snaps = [], ([], [])
    for nx, ny, nz in dims:
        m, D, xl, xr = _draw_tube(rng)
        P0 = (1.0 / 3.0) / (0.5 * float(np.dot(xl, m) + np.dot(xr, m)))
        tubes.append(dict(_species(m, D, 0.5 * P0), nx=nx, ny=ny, nz=nz, wall_x=1, slaved=2))
        width, grow = rng.uniform(2.0, 12.0), rng.uniform(1.02, 1.10)
        xs = (np.arange(nx) - 0.5 * nx + 0.5)[None, None, :]
        ripple = 1.0 + 0.05 * np.cos(2.0 * np.pi * (np.arange(ny)[None, :, None] / ny + np.arange(nz)[:, None, None] / nz))
        amp = rng.uniform(-1e-3, 1e-3, size=5)
        for k in range(2):
            s = 1.0 / (1.0 + np.exp(-xs / (width * grow ** k))) * (ripple if ny * nz > 1 else 1.0)
            bump = np.exp(-(xs / (2.0 * width)) ** 2) * np.ones((nz, ny, 1)) * (1.0 - 0.1 * k)
            f = np.empty((8, nz, ny, nx), dtype=np.float32)
            s = np.minimum(s, 1.0)
            for c in range(3):
                f[c] = xl[c] + (xr[c] - xl[c]) * s
            f[3] = 1.0 / 3.0 + amp[0] * bump
            f[4] = amp[1] * bump
            f[5], f[6] = (amp[2] * bump, amp[3] * bump) if ny * nz > 1 else (0.0, 0.0)
            f[7] = P0 * (1.0 + 1e-3 * amp[4] * bump)
            snaps[k].append(f.reshape(-1))
    now, later = (torch.from_numpy(np.concatenate(v)).to(DEVICE) for v in snaps)
    flux = 1e-4 if case["kind"] != "hop" else 1e-6
    norm = {"in_shift": np.array([0.3, 0.3, 0.4, 1.0 / 3.0, 0.0, 0.0, 0.0, 0.015], dtype=np.float32),
            "in_scale": np.array([4.0, 4.0, 4.0, 1e3, 1e3, 1e3, 1e3, 100.0], dtype=np.float32),
            "out_scale": np.array([flux] * 9 + [1e-4] * 4, dtype=np.float32)}
    shapes = _layer_shapes(case["depth"])
    parts = []
    for k, (o, i) in enumerate(shapes):
        parts += [rng.normal(0.0, math.sqrt(2.0 / (27 * i)) * (0.1 if k == len(shapes) - 1 else 1.0), 27 * o * i),
                  rng.normal(0.0, 0.02, o)]
    params = np.concatenate(parts).astype(np.float32)
    weights = np.array([[1e9] * 3 + [2e7] + [1e7] * 3 + [1e8]], dtype=np.float32)
    return dims, tubes, now, later, norm, params, weights


def _layer_shapes(depth):
    """(out, in) of each layer: 8 fields and 6 tube constants in, 3 x 3 fluxes and 4 changes out."""
    return list(zip([64] * (depth - 1) + [13], [14] + [64] * (depth - 1)))


# ------------------------------------------------------------------ a user's program
def prepare(case, seed):
    from paper_2004_11286_amd import mclbm as mc

    kind = case["kind"]
    if kind in ("forward", "train"):
        from paper_2004_11286_amd import surrogate as S

        dims, tubes, now, later, norm, params, weights = _net_inputs(case, seed)
        net = S.build_net(dims, tubes, norm, 3, case["depth"], params=params)
        return {"case": case, "S": S, "net": net, "now": now, "snaps": torch.stack([now, later]), "weights": weights}
    if kind == "hop":
        from paper_2004_11286_amd import surrogate as S

        dims, tubes, now, _, norm, params, _ = _net_inputs(case, seed)
        net = S.build_net(dims, tubes, norm, 3, case["depth"], params=params)
        fields = _split_fields(now.double(), dims)
        pairs = list(zip(tubes, fields))
        prec = "fp32"
    else:
        pairs, net, prec = _lattice_inputs(case, seed), None, case["prec"]
    single = kind in ("box", "tube", "jets")
    sim = mc.Sim(pairs[0][0], prec) if single else mc.Batch([p for p, _ in pairs], prec)
    M = sim.M
    flat = [torch.cat([f[k].reshape(-1) for _, f in pairs]) if not single else pairs[0][1][k] for k in ("X", "p", "T", "u")]
    out = None if prec == "fp64" else torch.empty((M + 5) * sim.n, dtype=torch.float32, device=DEVICE)
    state = {"case": case, "mc": mc, "sim": sim, "net": net, "fields": flat, "out": out}
    if kind != "box":
        mc.mclbm_init_fields(sim.ctx, *[t.data_ptr() for t in flat], 1)
    return state


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "forward":
        return state["net"].forward(state["now"])
    if kind == "train":
        net = state["net"]
        losses = state["S"].train(net, state["snaps"], case["iters"], state["weights"], lr=2e-5, warmup=1, clip=2.0)
        return {"losses": np.array(losses), "params": net.get_params()}
    mc, sim = state["mc"], state["sim"]
    if kind == "hop":
        used, _, _ = state["net"].advance(sim, HOP, float("inf"), float("inf"))
        mc.mclbm_read_fields_f32(sim.ctx, state["out"].data_ptr(), 1)
        return {"fields": state["out"], "used_fallback": int(used)}
    if kind == "box":
        mc.mclbm_init_fields(sim.ctx, *[t.data_ptr() for t in state["fields"]], 1)
    sim.step(case["steps"])
    if state["out"] is None:
        return sim.read_moments(on_device=True)
    mc.mclbm_read_fields_f32(sim.ctx, state["out"].data_ptr(), 1)
    return state["out"]


# ------------------------------------------------------------------ the least a pass can do
def _nodes(case):
    if case["kind"] in ("tubes", "train"):
        mean = 0.5 * (case["lmin"] + case["lmax"])
        return case["ntubes"] * mean * case.get("ny", 1) * case.get("nz", 1)
    return case.get("ntubes", 1) * case["nx"] * case["ny"] * case.get("nz", 1)


def work(case):
    n, kind = _nodes(case), case["kind"]
    if kind in ("forward", "train", "hop"):
        macs = sum(27 * o * i for o, i in _layer_shapes(case["depth"]))
        weights = 4 * sum(27 * o * i + o for o, i in _layer_shapes(case["depth"]))
        if kind == "forward":      # fields in and out
            return {"bytes": 2 * 8 * 4 * n + weights, "flops": 2.0 * macs * n}
        if kind == "train":        # forward and the two backward products; weights and both moments updated
            return {"bytes": case["iters"] * (2 * 8 * 4 * n + 7 * weights), "flops": case["iters"] * 6.0 * macs * n}
        # hop: the state read, the new one written (4 lattices of 27 values), the fields out
        return {"bytes": (2 * 4 * 27 * 4 + 8 * 4) * n + weights, "flops": 2.0 * macs * n}
    M = {"box": 2, "tube": case.get("M"), "tubes": 3, "jets": 4}[kind]
    L, s = M + 1 + case.get("weak", 0), STORAGE_BYTES[case["prec"]]
    per_step = 2 * 27 * L * s                  # every stored population read and written once
    out = 27 * L * s + ((M + 6) * 8 if case["prec"] == "fp64" else (M + 5) * 4)
    first = (M + 5) * 8 + 27 * L * s if kind == "box" else 0
    return {"bytes": (per_step * case["steps"] + out + first) * n, "flops": 27.0 * L * 30 * case["steps"] * n}


# ------------------------------------------------------------------ the same in 64 bits
C3 = [(i // 9 - 1, (i // 3) % 3 - 1, i % 3 - 1) for i in range(27)]


def _split_fields(flat, dims):
    out, off = [], 0
    for nx, ny, nz in dims:
        f = flat[8 * off:8 * (off + nx * ny * nz)].reshape(8, nz, ny, nx)
        X = f[:3].clamp_min(0.0)
        X = X / X.sum(0)
        out.append({"X": X.contiguous(), "p": f[7].contiguous(), "T": f[3].contiguous(), "u": f[4:7].contiguous()})
        off += nx * ny * nz
    return out


class _Model:
    """The M+2-lattice step in FP64 on [nz, ny, nx] tensors. Several walled tubes of one cross-section
    stand end to end in x, each with its own species data and walls."""

    def __init__(self, pairs):
        p0 = pairs[0][0]
        self.M, self.wall, self.weak = p0["M"], p0.get("wall_x", 0), p0.get("weak", 0)
        self.NS = self.M if self.weak else self.M - 1
        self.sizes = [p["nx"] for p, _ in pairs]
        one = len(pairs) == 1

        def per(get):
            if one:
                return float(get(p0))
            return torch.cat([torch.full((p["nx"],), float(get(p)), dtype=torch.float64, device=DEVICE) for p, _ in pairs])

        R = range(self.M)
        self.m = [per(lambda p, a=a: p["molar_mass"][a]) for a in R]
        self.cv = [per(lambda p, a=a: p["cv"][a]) for a in R]
        self.mu = [per(lambda p, a=a: p["mu"][a]) for a in R]
        self.lam = [per(lambda p, a=a: p["lambda"][a]) for a in R]
        self.D = [[per(lambda p, a=a, b=b: p["D"][a][b]) for b in R] for a in R]
        self.cvc, self.tex = p0.get("cv_coef"), p0.get("transport_exp")
        X, p, T, u = (torch.cat([f[k] for _, f in pairs], dim=-1) for k in ("X", "p", "T", "u"))
        self.shape = p.shape
        nx = self.shape[2]
        self.lo = torch.zeros(nx, dtype=torch.bool, device=DEVICE)
        self.hi = torch.zeros(nx, dtype=torch.bool, device=DEVICE)
        off = 0
        for k in self.sizes:
            self.lo[off] = True
            self.hi[off + k - 1] = True
            off += k
        if self.wall == 3:
            y = torch.arange(self.shape[1], device=DEVICE)
            self.nozzle = ((y >= p0["nozzle"][0]) & (y < p0["nozzle"][1]))[:, None]
        self.pop = self.equilibrium([X[a] for a in R], p, T, u)
        if self.wall >= 2:
            self.inlets = [self._inlet(p0["inlet"])] + ([self._inlet(p0["inlet_right"])] if self.wall == 3 else [])

    def _inlet(self, v):
        t = [torch.full((1, 1, 1), float(x), dtype=torch.float64, device=DEVICE) for x in v]
        M = self.M
        return [q[:, 0, 0, 0] for q in self.equilibrium(t[:M], t[M], t[M + 1], torch.stack(t[M + 2:]))]

    @staticmethod
    def psi(u, zeta):
        """The 1-D triplets of the product form for the three velocity components."""
        out = []
        for k in range(3):
            s = u[k] * u[k] + zeta
            out.append((0.5 * (s - u[k]), 1.0 - s, 0.5 * (s + u[k])))
        return out

    def U(self, a, T):
        if self.cvc is None:
            return self.cv[a] * T
        c = self.cvc[a]
        return T * (c[0] + T * (c[1] / 2 + T * (c[2] / 3 + T * c[3] / 4)))

    def Cv(self, a, T):
        if self.cvc is None:
            return self.cv[a] + 0.0 * T
        c = self.cvc[a]
        return c[0] + T * (c[1] + T * (c[2] + T * c[3]))

    def g_eq(self, i, th, rhoE, rho, u, usq, H, q):
        """Energy-lattice ansatz with flux q at the equilibrium second moment."""
        c = C3[i]
        w = 1.0
        for k in range(3):
            w = w * ((1.0 - th) if c[k] == 0 else 0.5 * th)
        kappa, base = rho * (H + 0.5 * usq + th), rho * th * th
        con = base * (sum(v * v for v in c) - 3.0 * th) + kappa * (_dot(c, u) ** 2 - th * usq)
        g = w * (rhoE + _dot(c, q) / th + con * 0.5 / (th * th))
        zf = (1.0 - 3.0 * th) * 0.5 / th
        n2 = sum(v * v for v in c)
        if n2 == 0:
            g = g + zf * (3.0 * base + kappa * usq)
        if n2 == 1:
            k = [j for j in range(3) if c[j]][0]
            g = g - 0.5 * zf * (base + kappa * u[k] * u[k])
        return g

    def equilibrium(self, X, p, T, u):
        M = self.M
        mm = sum(X[a] * self.m[a] for a in range(M))
        rho, th = p * mm / T, T / mm
        usq = (u * u).sum(0)
        Y = [X[a] * self.m[a] / mm for a in range(M)]
        out = []
        for a in range(self.NS):
            t = self.psi(u, T / self.m[a])
            out.append(torch.stack([rho * Y[a] * t[0][c[0] + 1] * t[1][c[1] + 1] * t[2][c[2] + 1] for c in C3]))
        t = self.psi(u, th)
        out.append(torch.stack([rho * t[0][c[0] + 1] * t[1][c[1] + 1] * t[2][c[2] + 1] for c in C3]))
        Um = sum(Y[a] * self.U(a, T) for a in range(M))
        H = Um + th
        rhoE, q = rho * (Um + 0.5 * usq), (H + 0.5 * usq) * rho * u
        out.append(torch.stack([self.g_eq(i, th, rhoE, rho, u, usq, H, q) for i in range(27)]))
        return out

    def moments(self):
        M, NS = self.M, self.NS
        f, g = self.pop[NS], self.pop[NS + 1]
        rho, rhoE = f.sum(0), g.sum(0)
        j = [_first(f, k) for k in range(3)]
        ra = [self.pop[a].sum(0) for a in range(NS)]
        ja = [[_first(self.pop[a], k) for k in range(3)] for a in range(NS)]
        u = [v / rho for v in j]
        us, rs = u, rho
        if self.weak:
            rs = sum(ra)
            us = [sum(ja[a][k] for a in range(M)) / rs for k in range(3)]
        else:
            ra.append(rho - sum(ra))
            ja.append([j[k] - sum(v[k] for v in ja) for k in range(3)])
        Y = [v / rs for v in ra]
        Rg = sum(Y[a] / self.m[a] for a in range(M))
        X = [Y[a] / (self.m[a] * Rg) for a in range(M)]
        usq = sum(v * v for v in u)
        e = rhoE / rho - 0.5 * usq
        if self.cvc is None:
            T = e / sum(Y[a] * self.cv[a] for a in range(M))
        else:
            T = e / sum(Y[a] * float(self.cvc[a][0]) for a in range(M))
            for _ in range(12):
                T = T - (sum(Y[a] * self.U(a, T) for a in range(M)) - e) / sum(Y[a] * self.Cv(a, T) for a in range(M))
        return rho, rhoE, u, usq, us, rs, ra, ja, Y, X, Rg, T

    # neighbours: value at x + d along an axis, with the boundary's rule (odd: changes sign at a mirror)
    def sh(self, v, axis, d, odd=False):
        r = torch.roll(v, -d, dims=2 - axis)
        if axis == 0 and self.wall:
            edge = self.lo if d < 0 else self.hi
            if odd and self.wall == 1:
                ghost = -v
            elif odd and self.wall == 3:
                ghost = torch.where(self.nozzle, v, -v)
            else:
                ghost = v
            r = torch.where(edge, ghost, r)
        if axis == 1 and self.wall == 3:
            y = 0 if d < 0 else self.shape[1] - 1
            r[:, y] = v[:, y]
        return r

    def grad(self, v, axis, odd=False):
        for k in range(3):
            p, q = self.sh(v, k, 1, odd and k == 0), self.sh(v, k, -1, odd and k == 0)
            v = 0.5 * (p - q) if k == axis else (p + 4.0 * v + q) / 6.0
        return v

    def step(self):
        M, NS = self.M, self.NS
        rho, rhoE, u, usq, us, rs, ra, ja, Y, X, Rg, T = self.moments()
        th, P = Rg * T, rho * Rg * T
        tr = self.tex
        mua = [self.mu[a] * ((T / tr[-1]) ** tr[a] if tr is not None else 1.0) for a in range(M)]
        lama = [self.lam[a] * ((T / tr[-1]) ** tr[M + a] if tr is not None else 1.0) for a in range(M)]
        fD = (T / tr[-1]) ** tr[2 * M] if tr is not None else 1.0
        mu = 0.0
        for a in range(M):
            den = 0.0
            for b in range(M):
                ratio = (mua[a] / mua[b]) * (self.m[b] / self.m[a]) ** 0.5
                den = den + (1.0 + ratio ** 0.5) ** 2 / (8.0 * (1.0 + self.m[a] / self.m[b])) ** 0.5 * X[b]
            mu = mu + mua[a] * X[a] / den
        lam = 0.5 * (sum(X[a] * lama[a] for a in range(M)) + 1.0 / sum(X[a] / lama[a] for a in range(M)))
        Cp = sum(Y[a] * self.Cv(a, T) for a in range(M)) + Rg
        om, om1 = 2.0 * P / (P + 2.0 * mu), 2.0 * P * Cp / (P * Cp + 2.0 * lam)
        Ha = [self.U(a, T) + T / self.m[a] for a in range(M)]
        H = sum(Y[a] * Ha[a] for a in range(M))
        # diffusion velocities (an absent species has none)
        Ps = rs * Rg * T
        here = [ra[a].abs() > 1e-12 * rho for a in range(M)]
        K = [[torch.where(here[a] & here[b], Ps * X[a] * X[b] / (self.D[a][b] * fD), 0.0 * T) for b in range(M)]
             for a in range(M)]
        A = [[-0.5 * K[a][b] if a != b else
              torch.where(here[a], ra[a], 1.0 + 0.0 * T) + 0.5 * sum(K[a][c] for c in range(M) if c != a)
              for b in range(M)] for a in range(M)]
        V = [[torch.where(here[a], ja[a][k] - ra[a] * us[k], 0.0 * T) for k in range(3)] for a in range(M)]
        for c in range(M):
            for r in range(c + 1, M):
                fac = A[r][c] / A[c][c]
                for b in range(c + 1, M):
                    A[r][b] = A[r][b] - fac * A[c][b]
                V[r] = [V[r][k] - fac * V[c][k] for k in range(3)]
        for r in reversed(range(M)):
            V[r] = [(V[r][k] - sum(A[r][c] * V[c][k] for c in range(r + 1, M))) / A[r][r] for k in range(3)]
        # non-local terms: X_a = -d_a G_a, sum_a H_a d Y_a
        f, g = self.pop[NS], self.pop[NS + 1]
        Xc = []
        for k in range(3):
            phi = rho * u[k] * (1.0 - 3.0 * th) - rho * u[k] ** 3
            Xc.append(-self.grad((1.0 / om - 0.5) * self.grad(phi, k, odd=k == 0), k))
        hg = [0.0, 0.0, 0.0]
        for k in range(3):
            for a in range(M):
                hg[k] = hg[k] + Ha[a] * self.grad(Y[a], k)
        dq = []
        hyd = H + 0.5 * usq
        q = [_first(g, k) for k in range(3)]
        qeq = [hyd * rho * u[k] for k in range(3)]
        for k in range(3):
            up = 0.0
            for c in range(3):
                Pck = 0.0
                for i in range(27):
                    if C3[i][c] * C3[i][k]:
                        Pck = Pck + C3[i][c] * C3[i][k] * f[i]
                up = up + u[c] * (Pck - (P if c == k else 0.0) - rho * u[c] * u[k])
            hv = sum(Ha[a] * Y[a] * V[a][k] for a in range(M))
            dq.append((om - om1) * (q[k] - qeq[k] - up) + om1 * rho * hv + 0.5 * (2.0 - om1) * P * hg[k])
        # collisions and streaming, one lattice after the other
        new = []
        pe = [self.psi(us, T / self.m[b]) for b in range(M)]
        ps = [self.psi([us[k] + V[b][k] for k in range(3)], T / self.m[b]) for b in range(M)]
        for a in range(NS):
            it = sum(Y[b] / (self.D[a][b] * fD) / self.m[b] for b in range(M)) * T / (Rg * self.m[a])
            beta = it / (2.0 + it)
            post = torch.empty_like(self.pop[a])
            for i, c in enumerate(C3):
                F = 0.0
                for b in range(M):
                    e, s = pe[b], ps[b]
                    F = F + K[a][b] * (e[0][c[0] + 1] * e[1][c[1] + 1] * e[2][c[2] + 1]
                                       - s[0][c[0] + 1] * s[1][c[1] + 1] * s[2][c[2] + 1])
                fe = ra[a] * pe[a][0][c[0] + 1] * pe[a][1][c[1] + 1] * pe[a][2][c[2] + 1]
                post[i] = self.pop[a][i] + 2.0 * beta * (fe - self.pop[a][i]) + (beta - 1.0) * F
            new.append(self.stream(post, a))
        post = torch.empty_like(f)
        t = self.psi(u, th)
        for i, c in enumerate(C3):
            post[i] = f[i] + om * (rho * t[0][c[0] + 1] * t[1][c[1] + 1] * t[2][c[2] + 1] - f[i])
            if sum(v * v for v in c) == 1:
                post[i] += 0.5 * _dot(c, Xc)
        new.append(self.stream(post, NS))
        post = torch.empty_like(g)
        for i, c in enumerate(C3):
            w = 1.0
            for k in range(3):
                w = w * ((1.0 - th) if c[k] == 0 else 0.5 * th)
            ge = self.g_eq(i, th, rhoE, rho, u, usq, H, qeq)
            post[i] = g[i] + om * (ge - g[i]) + (w * _dot(c, dq) / th if any(c) else 0.0)
        new.append(self.stream(post, NS + 1))
        self.pop = new

    def stream(self, post, lat):
        out = torch.empty_like(post)
        nx, ny = self.shape[2], self.shape[1]
        for i, c in enumerate(C3):
            out[i] = torch.roll(post[i], (c[2], c[1], c[0]), dims=(0, 1, 2))
            if self.wall == 1 and c[0]:
                out[i] = torch.where(self.lo if c[0] > 0 else self.hi, post[26 - i], out[i])
            if self.wall == 2 and c[0] > 0:
                out[i][:, :, 0] = self.inlets[0][lat][i]
            if self.wall == 2 and c[0] < 0:
                out[i][:, :, -1] = torch.roll(post[i], (c[2], c[1]), dims=(0, 1))[:, :, -1]
            if self.wall == 3:
                if c[0]:                            # beside the nozzles: reflected, c_x reversed
                    x = 0 if c[0] > 0 else nx - 1
                    out[i][:, :, x] = torch.roll(post[i - 18 * c[0]], (c[2], c[1]), dims=(0, 1))[:, :, x]
                if c[1]:                            # outlets: the boundary row's own state
                    y = 0 if c[1] > 0 else ny - 1
                    xs = (torch.arange(nx, device=DEVICE) - c[0]).clamp(0, nx - 1)
                    out[i][:, y] = torch.roll(post[i], c[2], dims=0)[:, y][:, xs]
                if c[0]:
                    n = self.nozzle[:, 0]
                    out[i][:, n, 0 if c[0] > 0 else nx - 1] = self.inlets[0 if c[0] > 0 else 1][lat][i]
        return out

    def read(self):
        rho, _, u, _, _, _, _, _, _, X, Rg, T = self.moments()
        return {"X": torch.stack(X), "rho": rho, "u": torch.stack(u), "p": rho * Rg * T, "T": T}

    def packed(self):
        r = self.read()
        f = torch.cat([r["X"], r["T"][None], r["u"], r["p"][None]])
        return torch.cat([v.reshape(-1) for v in f.split(self.sizes, dim=-1)])


def _dot(c, v):
    out = 0.0
    for k in range(3):
        if c[k]:
            out = out + v[k] if c[k] > 0 else out - v[k]
    return out


def _first(f, k):
    out = 0.0
    for i in range(27):
        if C3[i][k]:
            out = out + f[i] if C3[i][k] > 0 else out - f[i]
    return out


class _Net64:
    """The network in FP64: node indices of every tap over the tubes laid end to end."""

    def __init__(self, dims, tubes, norm, params, depth):
        self.dims, self.depth = dims, depth
        self.flat = all(d[1] == 1 and d[2] == 1 for d in dims)
        off, idx, first = 0, [], []
        for nx, ny, nz in dims:
            z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
            rows = []
            for c in ([(0, 0, d) for d in (-1, 0, 1)] if self.flat else [(t // 9 - 1, (t // 3) % 3 - 1, t % 3 - 1) for t in range(27)]):
                rows.append((off + np.clip(x + c[2], 0, nx - 1) + nx * ((y + c[1]) % ny + ny * ((z + c[0]) % nz))).reshape(-1))
            idx.append(np.stack(rows))
            first.append(np.stack([x.reshape(-1), np.full(x.size, nx)]))
            off += x.size
        self.n = off
        self.idx = torch.from_numpy(np.concatenate(idx, axis=1)).to(DEVICE)
        self.x, self.nx = torch.from_numpy(np.concatenate(first, axis=1)).to(DEVICE)
        iu = np.triu_indices(3, 1)
        cond = [np.concatenate([p["molar_mass"] / 40.0, p["D"][iu] / 0.1]).astype(np.float32) for p in tubes]
        sizes = [d[0] * d[1] * d[2] for d in dims]
        self.cond = torch.from_numpy(np.repeat(np.stack(cond), sizes, axis=0).T.astype(np.float64)).to(DEVICE)
        self.norm = {k: torch.from_numpy(v.astype(np.float64)).to(DEVICE)[:, None] for k, v in norm.items()}
        self.p = torch.from_numpy(params.astype(np.float64)).to(DEVICE)

    def fields(self, flat):
        out, off = [], 0
        for nx, ny, nz in self.dims:
            k = nx * ny * nz
            out.append(flat[8 * off:8 * (off + k)].double().reshape(8, k))
            off += k
        return torch.cat(out, dim=1)

    def pack(self, f):
        return torch.cat([v.reshape(-1) for v in f.split([d[0] * d[1] * d[2] for d in self.dims], dim=1)])

    def raw(self, f, p):
        a, k = torch.cat([(f - self.norm["in_shift"]) * self.norm["in_scale"], self.cond]), 0
        for l, (o, i) in enumerate(_layer_shapes(self.depth)):
            W = p[k:k + 27 * o * i].reshape(27, o, i)
            if self.flat:
                W = W.reshape(9, 3, o, i).sum(0)
            y = p[k + 27 * o * i:k + 27 * o * i + o][:, None]
            k += 27 * o * i + o
            for t in range(W.shape[0]):
                y = y + W[t] @ a[:, self.idx[t]]
            a = torch.relu(y) if l + 1 < self.depth else y
        return a * self.norm["out_scale"]

    def predict(self, f, y):
        """(molar densities, T, u) after the hop."""
        n = f[7] * f[:3] / f[3]
        div = 0.0
        # the taps one node back in x, y and z (tubes one node wide: x alone, the other fluxes cancel)
        for tap, a in ([(0, 0)] if self.flat else [(12, 0), (10, 1), (4, 2)]):
            F = y[a:9:3]
            if a == 0:
                F = torch.where(self.x + 1 < self.nx, F, 0.0 * F)
            low = F[:, self.idx[tap]]
            if a == 0:
                low = torch.where(self.x > 0, low, 0.0 * low)
            div = div + F - low
        return n - div, f[3] + y[9], f[4:7] + y[10:13]

    def forward(self, flat):
        f = self.fields(flat)
        n, T, u = self.predict(f, self.raw(f, self.p))
        s = n.sum(0)
        return self.pack(torch.cat([n / s, T[None], u, (T * s)[None]]))


def _exact_net(case, seed):
    dims, tubes, now, later, norm, params, weights = _net_inputs(case, seed)
    net = _Net64(dims, tubes, norm, params, case["depth"])
    if case["kind"] != "train":
        if case["kind"] == "hop":
            # the lattice starts at the equilibrium of the fields and reads them back; the new
            # state is the equilibrium of the prediction
            parts = _split_fields(now.double(), dims)
            now = torch.cat([torch.cat([q["X"], q["T"][None], q["u"], q["p"][None]]).reshape(-1) for q in parts])
        out = net.forward(now)
        if case["kind"] == "hop":
            parts = _split_fields(out, dims)
            out = torch.cat([torch.cat([q["X"], q["T"][None], q["u"], q["p"][None]]).reshape(-1) for q in parts])
            return {"fields": out.cpu(), "used_fallback": None}
        return out.cpu()
    f, t = net.fields(now), net.fields(later)
    w = torch.from_numpy(weights[0].astype(np.float64)).to(DEVICE)[:, None]
    nt = t[7] * t[:3] / t[3]
    dn = nt - f[7] * f[:3] / f[3]
    rows = torch.cat([torch.cumsum(v, dim=1) for v in dn.split([d[0] for d in dims], dim=1)], dim=1)
    p = net.p.clone().requires_grad_(True)
    m1, m2, losses, mean, N = 0.0, 0.0, [], None, net.n
    for it in range(case["iters"]):
        y = net.raw(f, p)
        n, T, u = net.predict(f, y)
        eF = torch.where(net.x + 1 < net.nx, y[0:9:3] + rows, 0.0 * rows)
        loss = ((w[:3] * (n - nt) ** 2).sum() + (w[3] * (T - t[3]) ** 2).sum() + (w[4:7] * (u - t[4:7]) ** 2).sum()
                + (w[7] * eF ** 2).sum()) / N
        (g,) = torch.autograd.grad(loss, p)
        losses.append(float(loss))
        m1, m2 = 0.9 * m1 + 0.1 * g, 0.999 * m2 + 0.001 * g * g
        lr = 2e-5 * 0.5 * (1.0 + math.cos(math.pi * it / case["iters"])) + 0.02 * 2e-5
        with torch.no_grad():
            p -= lr * (m1 / (1.0 - 0.9 ** (it + 1))) / (torch.sqrt(m2 / (1.0 - 0.999 ** (it + 1))) + 1e-8)
    return {"losses": np.array(losses), "params": p.detach().cpu().numpy()}


@torch.no_grad()
def _exact_lattice(case, seed):
    model = _Model(_lattice_inputs(case, seed))
    for _ in range(case["steps"]):
        model.step()
    if case["prec"] == "fp64":
        return {k: v.cpu() for k, v in model.read().items()}
    return model.packed().cpu()


def exact(case, seed):
    if case["kind"] in ("forward", "train", "hop"):
        return _exact_net(case, seed)
    return _exact_lattice(case, seed)
