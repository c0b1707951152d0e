"""Timed cases: the work a program has the library do, through its public entry points.

    line     1D plans (FP64 and FP32, up to the sizes one workgroup steps and beyond)
    plane    2D plans: small latency-bound grids, ragged ones with mixed walls and maps, large FFT grids
    volume   3D plans in FP32, FP64 and split-bf16, optionally with the particle velocities resampled onto
             the pressure nodes after the steps (a snapshot as a program stores it)
    batch    many uneven 2D solves in one batch, paired Neumann / Dirichlet, then combined
    faces    one 2D box with a reflection coefficient per face (16 basic solves and their weighted sum)
    infer    the surrogate's answer to a batch of requests
    train    the surrogate's forward and backward pass, its gradient handed to the caller

A pass of the first three kinds advances the state it was given, as a time loop does.
"""
from __future__ import annotations

import functools
import math
import os

import numpy as np
import torch

from paper_2005_00322_amd import Batch, Plan
from paper_2005_00322_amd.pstd import STAG_TO_NODES, solve_faces_2d
from paper_2005_00322_amd.surrogate import Surrogate, SurrogateConfig, param_shapes

N, D, P, NH, DH = 0, 1, 2, 3, 4          # Neumann, Dirichlet, periodic, and right walls half a step further
DX, RHO0 = 1e-4, 1000.0
LETTER = {"N": N, "D": D, "P": P, "n": NH, "d": DH}
WEIGHTS = os.path.join("paper_2005_00322_amd", "weights", "nop_128x128_c32_m48_l4.npz")


def listed():
    return [
        # one short line in double precision, a few steps: a call whose cost is latency
        {"name": "line_128_fp64", "kind": "line", "n0": 128, "walls": "DD", "prec": "fp64", "map": False, "steps": 20},
        # a long line of a size no FFT takes, in a medium with a sound-speed map
        {"name": "line_1000_fp32_map", "kind": "line", "n0": 1000, "walls": "ND", "prec": "fp32", "map": True, "steps": 50},
        # the standard 2D box of the benchmark: many steps of a grid that fills the chip once
        {"name": "plane_256_fp32", "kind": "plane", "n0": 256, "n1": 256, "walls": "DDNN", "prec": "fp32", "map": False, "steps": 100},
        # ragged 2D grid, periodic across and a half-step wall, heterogeneous medium
        {"name": "plane_331x197_fp32_map", "kind": "plane", "n0": 331, "n1": 197, "walls": "PPNd", "prec": "fp32", "map": True, "steps": 50},
        # the same in double precision: the reference runs that a study checks its FP32 fields against
        {"name": "plane_300x241_fp64", "kind": "plane", "n0": 300, "n1": 241, "walls": "NDDN", "prec": "fp64", "map": False, "steps": 20},
        # a large 2D grid on the FFT path
        {"name": "plane_2049_fp32", "kind": "plane", "n0": 2049, "n1": 2049, "walls": "DDNN", "prec": "fp32", "map": False, "steps": 20},
        # a ragged 3D grid in single precision (the plans' default) with a map
        {"name": "volume_161x200x129_fp32_map", "kind": "volume", "n0": 161, "n1": 200, "n2": 129, "walls": "NNDDND", "prec": "fp32", "map": True, "steps": 5, "snapshot": False},
        # the benchmark's 3D box on the matrix cores, with the velocities of the snapshot on the nodes
        {"name": "volume_384_split_snapshot", "kind": "volume", "n0": 384, "n1": 384, "n2": 384, "walls": "DNDDND", "prec": "split_bf16", "map": False, "steps": 3, "snapshot": True},
        # 128 uneven instances, each solved with both walls and combined
        {"name": "batch_128x2", "kind": "batch", "count": 128, "lo": 96, "hi": 512, "tile": 64, "steps": 5},
        # a reflection coefficient per face: the whole solve with its initial state and weighted sum
        {"name": "faces_256", "kind": "faces", "n0": 256, "n1": 256, "steps": 50},
        # the shipped surrogate on a batch of requests
        {"name": "infer_256", "kind": "infer", "H": 128, "W": 128, "channels": 32, "modes": 48, "layers": 4, "hidden": 128, "batch": 256, "shipped": True},
        # one training batch: forward, loss and gradient
        {"name": "train_64", "kind": "train", "H": 128, "W": 128, "channels": 32, "modes": 48, "layers": 4, "hidden": 128, "batch": 64, "split": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same kinds and ranges: sizes spread over their logarithm, odd ones among them."""
    kind = rng.choice(["line", "plane", "plane", "plane", "volume", "volume", "batch", "faces", "infer", "train"])
    pair = lambda opts: rng.choice(opts)  # noqa: E731
    if kind == "line":
        n = rng.choice([_log(rng, 16, 1365), _log(rng, 16, 1365), 2 ** rng.randint(9, 11) + 1])
        return {"kind": kind, "n0": n, "walls": pair(["DD", "NN", "ND", "DN"]), "prec": rng.choice(["fp64", "fp32"]),
                "map": rng.random() < 0.3, "steps": rng.choice([10, 25, 50])}
    if kind == "plane":
        n0, n1 = _log(rng, 24, 1200), _log(rng, 24, 1200)
        if rng.random() < 0.2:
            n0 = n1 = 2 ** rng.randint(9, 11) + 1
        walls = "".join(pair(["DD", "NN", "ND", "DN", "NN", "DD", "PP", "Nd", "Dn"]) for _ in range(2))
        return {"kind": kind, "n0": n0, "n1": n1, "walls": walls, "prec": rng.choice(["fp32", "fp32", "fp64", "split_bf16"]),
                "map": rng.random() < 0.3, "steps": 20 if n0 * n1 < 300000 else 5}
    if kind == "volume":
        prec = rng.choice(["fp32", "fp32", "fp64", "split_bf16", "split_bf16"])
        n = [_log(rng, 24, {"fp32": 300, "fp64": 200, "split_bf16": 384}[prec]) for _ in range(3)]
        walls = "".join(pair(["DD", "NN", "ND", "DN"]) for _ in range(3))
        return {"kind": kind, "n0": n[0], "n1": n[1], "n2": n[2], "walls": walls, "prec": prec, "map": rng.random() < 0.3,
                "steps": 3 if n[0] * n[1] * n[2] < 1 << 22 else 1, "snapshot": rng.random() < 0.4}
    if kind == "batch":
        lo = _log(rng, 16, 256)
        return {"kind": kind, "count": _log(rng, 2, 64), "lo": lo, "hi": rng.randint(lo, 512), "tile": rng.choice([32, 64]),
                "steps": 5}
    if kind == "faces":
        return {"kind": kind, "n0": _log(rng, 40, 512), "n1": _log(rng, 40, 512), "steps": rng.choice([10, 20])}
    H, W = _log(rng, 24, 128), _log(rng, 24, 128)
    modes = 2 * rng.randint(2, min(H, W, 48) // 2)
    case = {"kind": kind, "H": H, "W": W, "channels": rng.choice([8, 16, 32, 32]), "modes": modes, "layers": rng.randint(1, 4),
            "hidden": rng.choice([32, 64, 128]), "batch": _log(rng, 1, 64 if kind == "infer" else 24)}
    if kind == "infer":
        case["shipped"] = False
    else:
        case["split"] = rng.random() < 0.3
    return case


# ---- inputs ------------------------------------------------------------------------------------------
def _shape(case):
    return tuple(case[k] for k in ("n0", "n1", "n2") if k in case)


def _bcs(case):
    w = [LETTER[c] for c in case["walls"]]
    return tuple((w[2 * a], w[2 * a + 1]) for a in range(len(w) // 2))


def _pulse(r, shape):
    """One to three Gaussian pulses of a few nodes' width, away from the walls (tapered to zero on them)."""
    p = np.zeros(shape)
    for _ in range(int(r.integers(1, 4))):
        amp, s = r.uniform(0.5, 1.0), r.uniform(3.0, 6.0)
        f = 1.0
        for a, n in enumerate(shape):
            c = r.uniform(0.25 * n, 0.75 * n)
            x = np.arange(n)
            g = np.exp(-0.5 * ((x - c) / s) ** 2)
            f = f * g.reshape([-1 if b == a else 1 for b in range(len(shape))])
        p += amp * f
    for a, n in enumerate(shape):
        x = np.minimum(np.arange(n), n - 1 - np.arange(n)) / max(1.0, min(8.0, n / 4))
        p *= np.clip(x, 0.0, 1.0).reshape([-1 if b == a else 1 for b in range(len(shape))])
    return p


def _medium(r, shape):
    """A smooth sound-speed map in [1400, 1600] m/s, as the float32 array a plan takes."""
    m = np.zeros(shape)
    for a, n in enumerate(shape):
        for _ in range(3):
            x = np.cos(np.pi * r.uniform(0.5, 4.0) * np.arange(n) / n + r.uniform(0, 6.28))
            m = m + r.uniform(0.2, 1.0) * x.reshape([-1 if b == a else 1 for b in range(len(shape))])
    m = (m - m.min()) / (m.max() - m.min())
    return (1400.0 + 200.0 * m).astype(np.float32)


def _problem(case, seed):
    """Shape, walls, initial pressure, map, sound speed (its maximum) and time step of a single solve."""
    r = np.random.default_rng([seed, 1])
    shape = _shape(case)
    p0 = _pulse(r, shape)
    cmap = _medium(r, shape) if case["map"] else None
    c0 = float(cmap.max()) if cmap is not None else float(r.uniform(1450.0, 1550.0))
    cfl = 0.2 if len(shape) == 1 else 0.3
    return shape, _bcs(case), p0, cmap, c0, cfl * DX / c0


def _batch_problem(case, seed):
    """Two solves per instance, all Neumann then all Dirichlet: (shape, walls, p0, c0, dt), and the R values."""
    r = np.random.default_rng([seed, 2])
    sizes = np.random.default_rng([case["count"], case["lo"], case["hi"]])   # the sizes belong to the case
    solves, R = [], []
    for _ in range(case["count"]):
        shape = tuple(int(v) for v in sizes.integers(case["lo"], case["hi"] + 1, 2))
        c0 = float(r.uniform(1400.0, 1600.0))
        p0 = _pulse(r, shape)
        for w in (N, D):
            solves.append((shape, ((w, w), (w, w)), p0, c0, 0.3 * DX / c0))
        R.append(float(r.uniform(-1.0, 1.0)))
    return solves, R


def _requests(case, seed):
    """p0 and c0 maps of a batch of surrogate requests, and fields to fit (float32)."""
    r = np.random.default_rng([seed, 3])
    B, H, W = case["batch"], case["H"], case["W"]
    x, y = np.arange(H)[None, :, None], np.arange(W)[None, None, :]
    p0 = np.zeros((B, H, W))
    for _ in range(3):
        cx, cy = r.uniform(0.2 * H, 0.8 * H, (B, 1, 1)), r.uniform(0.2 * W, 0.8 * W, (B, 1, 1))
        s, amp = r.uniform(3.0, 6.0, (B, 1, 1)), r.uniform(0.0, 1.0, (B, 1, 1))
        p0 += amp * np.exp(-0.5 * ((x - cx) ** 2 + (y - cy) ** 2) / s ** 2)
    k, ph = r.uniform(1.0, 5.0, (2, B, 1, 1)), r.uniform(0.0, 6.28, (2, B, 1, 1))
    c0 = 1500.0 + 50.0 * np.cos(k[0] * x / H * np.pi + ph[0]) + 50.0 * np.cos(k[1] * y / W * np.pi + ph[1])
    target = 0.3 * np.cos(k[1] * x / H * 2 * np.pi + ph[0]) * np.cos(k[0] * y / W * 2 * np.pi + ph[1])
    return p0.astype(np.float32), c0.astype(np.float32), target.astype(np.float32)


def _config(case):
    return SurrogateConfig(case["H"], case["W"], case["channels"], case["modes"], case["layers"], case["hidden"])


@functools.lru_cache(maxsize=1)
def _shipped():
    with np.load(WEIGHTS) as z:
        return np.asarray(z["theta"], np.float32)


def _theta(case, seed):
    """The shipped parameters, or random ones at the scale a network starts training from (biases set too)."""
    if case.get("shipped"):
        return _shipped()
    r = np.random.default_rng([seed, 4])
    out = []
    for name, shape, fan in param_shapes(_config(case)):
        g = 0.1 if fan == 0 else fan ** -0.5 * (0.7 if name[0] in "RW" else 1.0)
        out.append((g * r.standard_normal(int(np.prod(shape)), dtype=np.float32)))
    return np.concatenate(out).astype(np.float32)


# ---- the calls ---------------------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind in ("line", "plane", "volume"):
        shape, bcs, p0, cmap, c0, dt = _problem(case, seed)
        plan = Plan(shape, DX, dt, c0, bcs, rho0=RHO0, precision=case["prec"], c0_map=cmap)
        st = plan.init_state(plan.new_state(p0))
        out = None
        if case.get("snapshot"):
            out = [torch.empty(shape, device=plan.device, dtype=plan.dtype) for _ in shape]
        plan.prepare(st, case["steps"])
        return {"case": case, "plan": plan, "st": st, "out": out}
    if kind == "batch":
        solves, R = _batch_problem(case, seed)
        b = Batch([{"shape": s, "bcs": w, "dx": DX, "dt": dt, "c0": c0} for s, w, _, c0, dt in solves], rho0=RHO0)
        b.set_config(tile=case["tile"])
        st = b.new_states([p for _, _, p, _, _ in solves])
        b.init_states(st)
        pairs = [(2 * i + 1, 2 * i) for i in range(case["count"])]
        outs = [torch.empty_like(st[n].p) for _, n in pairs]
        return {"case": case, "batch": b, "st": st, "pairs": pairs, "R": R, "outs": outs}
    if kind == "faces":
        r = np.random.default_rng([seed, 5])
        shape = _shape(case)
        p0 = torch.from_numpy(_pulse(r, shape)).to(device="cuda", dtype=torch.float32)
        R = tuple(tuple(float(v) for v in r.uniform(-1.0, 1.0, 2)) for _ in range(2))
        args = (shape, DX, 0.3 * DX / 1500.0, 1500.0, R, p0)
        _, batch, _ = solve_faces_2d(*args, 1, rho0=RHO0)      # the batch that later solves of this box reuse
        return {"case": case, "args": args, "batch": batch}
    p0, c0, target = (torch.from_numpy(v).to("cuda") for v in _requests(case, seed))
    net = Surrogate(_config(case), max_batch=case["batch"], split=bool(case.get("split")))
    net.set_params(_theta(case, seed))
    return {"case": case, "net": net, "in": (p0, c0, target), "out": torch.empty_like(p0)}


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("line", "plane", "volume"):
        s["plan"].step(s["st"], case["steps"])
        out = {"p": s["st"].p, "u": s["st"].u}
        if s["out"] is not None:
            out["nodes"] = [s["plan"].apply_operator(a, STAG_TO_NODES, s["st"].u[a], out=o) for a, o in enumerate(s["out"])]
        return out
    if kind == "batch":
        s["batch"].step(s["st"], case["steps"])
        s["batch"].combine_R(s["st"], s["pairs"], s["R"], outs=s["outs"])
        # at most 60 of the fields as outputs of their own: the rest of a large batch in one piece each
        fields = [st.p for st in s["st"]] + s["outs"]
        if 3 * len(s["st"]) + len(s["outs"]) <= 60:
            return {"p": [st.p for st in s["st"]], "u": [u for st in s["st"] for u in st.u], "combined": s["outs"]}
        return {"first": [[st.p] + st.u for st in s["st"][:8]], "combined": s["outs"][:32], "last": fields[-8:]}
    if kind == "faces":
        p, _, states = solve_faces_2d(*s["args"], case["steps"], rho0=RHO0, batch=s["batch"])
        return {"p": p, "basic": [st.p for st in states]}
    p0, c0, target = s["in"]
    if kind == "infer":
        return s["net"].infer(p0, c0, out=s["out"])
    out = s["net"].forward(p0, c0, out=s["out"])
    loss = s["net"].backward(target)
    return {"out": out, "loss": loss, "grad": s["net"].get_grads()}


# ---- what a pass cannot do without ------------------------------------------------------------------------
def _step_work(shape, esz):
    """One time step: every field read and written once; per axis two operators, each a forward and an inverse
    fast transform of a symmetric line (5 n log2(2n) flops together)."""
    pts = float(np.prod(shape))
    return {"bytes": 2.0 * esz * pts * (1 + len(shape)), "flops": sum(2 * 5.0 * pts * math.log2(2 * n) for n in shape)}


def work(case):
    kind = case["kind"]
    if kind in ("line", "plane", "volume"):
        shape = _shape(case)
        esz = 8 if case["prec"] == "fp64" else 4
        w = _step_work(shape, esz)
        pts = float(np.prod(shape))
        b, f = w["bytes"] * case["steps"], w["flops"] * case["steps"]
        if kind == "line":
            b = w["bytes"]                 # a line stays on the chip for all its steps
        if case["map"]:
            b += esz * pts * (1 if kind == "line" else case["steps"])
        if case.get("snapshot"):
            b += 2 * esz * pts * len(shape)
            f += sum(5.0 * pts * math.log2(2 * n) for n in shape)
        return {"bytes": b, "flops": f}
    if kind == "batch":
        solves, _ = _batch_problem({**case}, 0)
        b = f = 0.0
        for i, (shape, *_r) in enumerate(solves):
            w = _step_work(shape, 4)
            b += w["bytes"] * case["steps"] + (6.0 * shape[0] * shape[1])
            f += w["flops"] * case["steps"]
        return {"bytes": b, "flops": f}
    if kind == "faces":
        shape = _shape(case)
        w = _step_work(shape, 4)
        return {"bytes": 16 * w["bytes"] * case["steps"] + 17 * 4.0 * shape[0] * shape[1], "flops": 16 * w["flops"] * case["steps"]}
    C, H, W, L, Hp, B, M = (case[k] for k in ("channels", "H", "W", "layers", "hidden", "batch", "modes"))
    pts = float(B * H * W)
    layer = 2 * C * C * pts + 2 * 2 * C * B * (M * H * W + M * M * H) + 2.0 * C * C * M * M * B
    flops = 2 * 4 * C * pts + L * layer + 2 * Hp * (C + 1) * pts
    # in and out, and each layer's field once written and once read (bf16 in inference, FP32 for training)
    if kind == "infer":
        return {"bytes": pts * (12 + 2 * 2 * C * (L + 1)), "flops": flops}
    return {"bytes": pts * (16 + 2 * 4 * C * (2 * L + 1)), "flops": 3 * flops}


# ---- the same in 64 bits ----------------------------------------------------------------------------------
def _dev():
    return torch.device("cuda") if torch.cuda.is_available() else torch.device("cpu")


@functools.lru_cache(maxsize=512)
def _operators(n, left, right):
    """Unscaled d/dx (dx = 1) from the nodes to the staggered points and back, and the half-step resampling of
    a velocity onto the nodes: sampled sine / cosine modes, differentiated, of the box between the walls."""
    dev = _dev()
    f8 = dict(dtype=torch.float64, device=dev)
    if left == P:
        k = 2 * math.pi * torch.fft.rfftfreq(n, **f8)
        eye = torch.fft.rfft(torch.eye(n, **f8), dim=0)
        G = torch.fft.irfft((1j * k * torch.exp(0.5j * k))[:, None] * eye, n=n, dim=0)
        Dm = torch.fft.irfft((1j * k * torch.exp(-0.5j * k))[:, None] * eye, n=n, dim=0)
        return G.contiguous(), Dm.contiguous(), None
    half = right in (NH, DH)
    rd = right in (D, DH)
    L = n - 0.5 if half else n - 1.0
    ns = n if half else n - 1
    xn, xs = torch.arange(n, **f8)[:, None], torch.arange(ns, **f8)[:, None] + 0.5
    wn, ws = torch.ones(n, **f8), torch.ones(ns, **f8)
    wn[0] = 0.5
    if half:
        ws[-1] = 0.5
    else:
        wn[-1] = 0.5
    mixed = (left == D) != rd
    k = math.pi * (torch.arange(ns if mixed else n, **f8) + (0.5 if mixed else 0.0))[None, :] / L

    def modes(cos, x):
        return torch.cos(k * x) if cos else torch.sin(k * x)

    def analyse(B, w):
        norm = (B * B * w[:, None]).sum(0)
        live = norm > 1e-9 * n
        inv = torch.where(live, 1.0 / torch.where(live, norm, torch.ones_like(norm)), torch.zeros_like(norm))
        return inv[:, None] * B.T * w[None, :]

    cos_p = left == N
    Ap, Au = analyse(modes(cos_p, xn), wn), analyse(modes(not cos_p, xs), ws)
    sp, su = (-1.0, 1.0) if cos_p else (1.0, -1.0)
    G = (sp * k * modes(not cos_p, xs)) @ Ap
    Dm = (su * k * modes(cos_p, xn)) @ Au
    return G, Dm, modes(not cos_p, xn) @ Au


def _along(A, x, axis):
    y = x.movedim(axis, 0)
    rest = y.shape[1:]
    y = A @ y.reshape(y.shape[0], -1).contiguous()
    return y.reshape((A.shape[0],) + tuple(rest)).movedim(0, axis).contiguous()


def _solve(shape, bcs, p0, c2, dt, steps):
    """p and u after `steps` leapfrog steps from rest; p0 as the plan holds it, c2 a number or an array."""
    dev = _dev()
    p = torch.as_tensor(p0, dtype=torch.float64).to(dev).clone()
    ops = [_operators(n, l, r) for n, (l, r) in zip(shape, bcs)]
    for a, (l, r) in enumerate(bcs):
        if l == D:
            p.narrow(a, 0, 1).zero_()
        if r == D:
            p.narrow(a, shape[a] - 1, 1).zero_()
    sG = -dt / RHO0 / DX
    u = [-0.5 * sG * _along(ops[a][0], p, a) for a in range(len(shape))]
    sD = -dt * RHO0 / DX * c2
    for _ in range(steps):
        for a in range(len(shape)):
            u[a] += sG * _along(ops[a][0], p, a)
        acc = 0.0
        for a in range(len(shape)):
            acc = acc + _along(ops[a][1], u[a], a)
        p += sD * acc
    return p, u, ops


def _network(case, theta, p0, c0):
    C, H, W, M, L = (case[k] for k in ("channels", "H", "W", "modes", "layers"))
    dev = _dev()
    f8 = dict(dtype=torch.float64, device=dev)
    prm, o = {}, 0
    for name, shape, _ in param_shapes(_config(case)):
        cnt = int(np.prod(shape))
        prm[name] = theta[o:o + cnt].reshape(shape)
        o += cnt

    def dct(n):
        k, j = torch.arange(M, **f8)[:, None], torch.arange(n, **f8)[None, :]
        s = torch.full((M, 1), math.sqrt(2.0 / n), **f8)
        s[0] = math.sqrt(1.0 / n)
        return s * torch.cos(math.pi * k * (2 * j + 1) / (2 * n))

    Ch, Cw = dct(H), dct(W)
    B = p0.shape[0]
    x = torch.linspace(0, 1, H, **f8)[None, :, None].expand(B, H, W)
    y = torch.linspace(0, 1, W, **f8)[None, None, :].expand(B, H, W)
    f = torch.stack([p0, (c0 - 1500.0) / 100.0, x, y], 1)

    def mix(A, v):
        return (A @ v.reshape(B, v.shape[1], H * W)).reshape(B, A.shape[0], H, W)

    v = mix(prm["P"], f) + prm["pb"][None, :, None, None]
    for l in range(L):
        a = Ch @ v @ Cw.T                                                       # B, C, M, M
        R = prm["R%d" % l].repeat_interleave(2, 0).repeat_interleave(2, 1)      # M, M, C, C
        z = (R.reshape(M * M, C, C) @ a.reshape(B, C, M * M).permute(2, 1, 0).contiguous())
        z = z.permute(2, 1, 0).reshape(B, C, M, M)
        v = torch.nn.functional.gelu(mix(prm["W%d" % l], v) + prm["b%d" % l][None, :, None, None] + Ch.T @ z @ Cw)
    q = torch.nn.functional.gelu(mix(prm["Q1"], v) + prm["q1b"][None, :, None, None])
    return (q * prm["Q2"][None, :, None, None]).sum(1) + prm["q2b"]


def exact(case, seed):
    kind = case["kind"]
    dev = _dev()
    if kind in ("line", "plane", "volume"):
        shape, bcs, p0, cmap, c0, dt = _problem(case, seed)
        p0 = p0 if case["prec"] == "fp64" else p0.astype(np.float32)
        c2 = c0 * c0 if cmap is None else torch.from_numpy(cmap).to(dev).double() ** 2
        p, u, ops = _solve(shape, bcs, p0, c2, dt, case["steps"])
        out = {"p": p, "u": u}
        if case.get("snapshot"):
            out["nodes"] = [_along(ops[a][2], u[a], a) for a in range(len(shape))]
        return out
    if kind == "batch":
        solves, R = _batch_problem(case, seed)
        got = [_solve(s, w, p0.astype(np.float32), c0 * c0, dt, case["steps"])[:2] for s, w, p0, c0, dt in solves]
        comb = [0.5 * (1 + r) * got[2 * i][0] + 0.5 * (1 - r) * got[2 * i + 1][0] for i, r in enumerate(R)]
        fields = [p for p, _ in got] + comb
        if 3 * len(got) + len(comb) <= 60:
            return {"p": [p for p, _ in got], "u": [x for _, u in got for x in u], "combined": comb}
        return {"first": [[p] + u for p, u in got[:8]], "combined": comb[:32], "last": fields[-8:]}
    if kind == "faces":
        r = np.random.default_rng([seed, 5])
        shape = _shape(case)
        p0 = _pulse(r, shape).astype(np.float32)
        R = [[float(v) for v in r.uniform(-1.0, 1.0, 2)] for _ in range(2)]
        walls = [(N, N), (N, D), (D, N), (D, D)]

        def axis_weights(rl, rr):   # images off the left wall, the right wall, both and none, per pair of walls
            return [0.25 * (1 + sl * rl + sr * rr + sl * sr * rl * rr) for sl in (1, -1) for sr in (1, -1)]

        wx, wy = axis_weights(*R[0]), axis_weights(*R[1])
        p, basic = 0.0, []
        for i in range(4):
            for j in range(4):
                basic.append(_solve(shape, (walls[i], walls[j]), p0, 1500.0 ** 2, 0.3 * DX / 1500.0, case["steps"])[0])
                p = p + wx[i] * wy[j] * basic[-1]
        return {"p": p, "basic": basic}
    p0, c0, target = (torch.from_numpy(v).to(dev).double() for v in _requests(case, seed))
    theta = torch.from_numpy(_theta(case, seed)).to(dev).double()
    if kind == "infer":
        with torch.no_grad():
            return torch.cat([_network(case, theta, p0[i:i + 32], c0[i:i + 32]) for i in range(0, case["batch"], 32)])
    theta.requires_grad_(True)
    out, loss = [], 0.0
    for i in range(0, case["batch"], 16):
        o = _network(case, theta, p0[i:i + 16], c0[i:i + 16])
        t = target[i:i + 16]
        part = (((o - t) ** 2).sum((1, 2)) / (t * t).sum((1, 2))).sum() / case["batch"]
        part.backward()
        out.append(o.detach())
        loss += float(part.detach())
    return {"out": torch.cat(out), "loss": loss, "grad": theta.grad.float().double()}
