"""Workloads that the speed of this library is judged by.

Every case goes through the public entry points of
paper_2607_05818_amd.reff with inputs drawn from a seed: stacks of random
resistive tiers with TSV columns and bumps, their node lists, load scenarios,
uniform-tier point sets and screening-model parameters.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  the inputs, handles and output buffers of a program
    run(state)           one pass through the entry point; its outputs
    work(case)           bytes and flops one pass cannot do without
    exact(case, seed)    the outputs in float64 by plain torch, or None
"""
from __future__ import annotations

import math

import numpy as np
import torch

DEV = "cuda:0"

# Node-to-supply samples and full maps, plan batches, pair queries and load
# scenarios, the closed-form pairs of uniform tiers, and the screening model.
LISTED = [
    # the smallest call: an early two-tier sketch, latency and launches count
    {"name": "sample-small", "kind": "diag", "nt": 2, "nx": 32, "ny": 32, "tsv": 16, "pitch": 8,
     "nodes": 128, "precision": "fp64", "tol": 0.0},
    # the headline workload: sampled nodes of a one-million-node stack, mixed precision
    {"name": "sample-large-mixed", "kind": "diag", "nt": 4, "nx": 512, "ny": 512, "tsv": 1024,
     "pitch": 32, "nodes": 128, "precision": "mixed", "tol": 1e-3},
    # design-option exploration: sampled nodes of many candidate TSV plans in one call
    {"name": "plans-sample-mixed", "kind": "plans_pcg", "plans": 24, "lo": 64, "hi": 256,
     "nodes": 64, "precision": "mixed", "tol": 0.0},
    # bump-to-load pair resistances of one stack, float64 (the default precision)
    {"name": "pairs", "kind": "pairs", "nt": 4, "nx": 256, "ny": 256, "tsv": 256, "pitch": 32,
     "m": 24, "n": 40, "floating": False},
    # IR drop and bump currents of load scenarios, default precision and tolerance
    {"name": "ir-drop", "kind": "ir_drop", "nt": 3, "nx": 128, "ny": 128, "tsv": 256, "pitch": 8,
     "loads": 256, "scen": 4},
    # every node of a small ragged stack by the sparse-direct path
    {"name": "map-small", "kind": "map", "nt": 3, "nx": 61, "ny": 47, "tsv": 32, "pitch": 8,
     "nodes": 0},
    # every node of the one-million-node stack
    {"name": "map-large", "kind": "map", "nt": 4, "nx": 512, "ny": 512, "tsv": 1024, "pitch": 32,
     "nodes": 0},
    # candidate plans by the sparse-direct path, every node of each, host analysis included
    {"name": "plans-map", "kind": "plans_map", "plans": 24, "lo": 64, "hi": 256, "nodes": 0},
    # closed-form resistances of every pair of points on one uniform tier
    {"name": "grid-pairs", "kind": "grid", "M": 512, "N": 512, "P": 256},
    # bump-to-load pairs of a stack of uniform tiers by the reduced system
    {"name": "reduced-pairs", "kind": "reduced", "nt": 4, "nx": 512, "ny": 512, "p": 512,
     "m": 128, "n": 2048},
    # screening: predicted maps of one batch of plans
    {"name": "screen-predict", "kind": "predict", "nt": 3, "nx": 128, "ny": 128, "ch": 32,
     "plans": 16},
    # training step of the screening model: loss and gradient of one batch
    {"name": "screen-train", "kind": "grad", "nt": 3, "nx": 128, "ny": 128, "ch": 32,
     "plans": 16, "labels": 64},
]


def listed():
    return [dict(c) for c in LISTED]


def _log(rng, lo, hi):
    """An integer whose logarithm is uniform over [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["diag", "diag", "plans_pcg", "pairs", "ir_drop", "map", "map", "plans_map",
                       "grid", "reduced", "predict", "grad"])
    if kind in ("diag", "map", "pairs", "ir_drop"):
        hi = {"diag": 512, "map": 512, "pairs": 200, "ir_drop": 160}[kind]
        c = {"kind": kind, "nt": rng.randint(1, 4), "nx": _log(rng, 24, hi), "ny": _log(rng, 24, hi)}
        c["tsv"] = _log(rng, 8, 512)
        c["tsv"] = min(c["tsv"], c["nx"] * c["ny"] // 2)
        c["pitch"] = rng.choice([8, 16, 32])
        if kind == "diag":
            c["precision"] = rng.choice(["mixed", "fp64"])
            if c["precision"] == "fp64":
                c["nx"], c["ny"] = min(c["nx"], 200), min(c["ny"], 200)
            c["nodes"] = _log(rng, 4, 128)
            c["tol"] = rng.choice([0.0, 1e-3]) if c["precision"] == "mixed" else 0.0
        elif kind == "map":
            c["nodes"] = rng.choice([0, 0, 64])
        elif kind == "pairs":
            c["m"], c["n"] = _log(rng, 2, 32), _log(rng, 2, 32)
            c["floating"] = rng.random() < 0.3
        else:
            c["loads"], c["scen"] = _log(rng, 8, 192), rng.randint(1, 6)
        return c
    if kind in ("plans_pcg", "plans_map"):
        c = {"kind": kind, "plans": _log(rng, 2, 24), "lo": rng.randint(24, 64),
             "hi": rng.randint(96, 240)}
        c["nodes"] = 64 if kind == "plans_pcg" else rng.choice([0, 64])
        if kind == "plans_pcg":
            c["precision"], c["tol"] = "mixed", 0.0
        return c
    if kind == "grid":
        return {"kind": "grid", "M": _log(rng, 32, 512), "N": _log(rng, 32, 512),
                "P": _log(rng, 16, 400)}
    if kind == "reduced":
        c = {"kind": "reduced", "nt": rng.randint(2, 4), "nx": _log(rng, 64, 400),
             "ny": _log(rng, 64, 400), "p": _log(rng, 16, 448)}
        c["m"], c["n"] = _log(rng, 8, 128), _log(rng, 16, 1024)
        return c
    c = {"kind": kind, "nt": rng.randint(2, 4), "nx": 8 * rng.randint(5, 16),
         "ny": 8 * rng.randint(5, 16), "ch": rng.choice([16, 24, 32]), "plans": _log(rng, 1, 16)}
    if kind == "grad":
        c["labels"] = rng.choice([64, 256])
    return c


# ---------------------------------------------------------------- inputs

def _rng(*key):
    return np.random.default_rng([int(k) for k in key])


def _distinct(rng, nx, ny, count):
    flat = rng.choice(nx * ny, size=min(count, nx * ny), replace=False)
    return np.stack([flat % nx, flat // nx], axis=1).astype(np.int32)


def _array(nx, ny, pitch):
    """Bumps centred in the cells of an array of about `pitch` nodes."""
    kx, ky = max(1, nx // pitch), max(1, ny // pitch)
    xs = (2 * np.arange(kx) + 1) * nx // (2 * kx)
    ys = (2 * np.arange(ky) + 1) * ny // (2 * ky)
    X, Y = np.meshgrid(xs, ys)
    return np.stack([X.ravel(), Y.ravel()], axis=1).astype(np.int32)


def _stack(rng, nt, nx, ny, tsv, pitch):
    """Lognormal(0, 0.3) S edges, 5 S TSV segments (half of the columns in
    Gaussian clusters, half uniform), bumps on an array on tier 0."""
    gx = rng.lognormal(0.0, 0.3, size=(nt, ny, nx - 1))
    gy = rng.lognormal(0.0, 0.3, size=(nt, ny - 1, nx))
    centres = rng.uniform(0.0, 1.0, size=(8, 2)) * (nx, ny)
    near = np.rint(centres[rng.integers(0, 8, tsv)] + 0.08 * min(nx, ny) * rng.standard_normal((tsv, 2)))
    near = np.clip(near, 0, (nx - 1, ny - 1)).astype(np.int64)[: tsv // 2]
    uni = _distinct(rng, nx, ny, tsv).astype(np.int64)
    flat = np.concatenate([near[:, 1] * nx + near[:, 0], uni[:, 1] * nx + uni[:, 0]])
    _, first = np.unique(flat, return_index=True)
    flat = flat[np.sort(first)][:tsv]
    xy = np.stack([flat % nx, flat // nx], axis=1).astype(np.int32)
    return {"n_tiers": nt, "nx": nx, "ny": ny, "gx": gx, "gy": gy, "tsv_xy": xy,
            "tsv_g": np.full((len(xy), nt - 1), 5.0), "pad_xy": _array(nx, ny, pitch)}


def _free_nodes(rng, d, count):
    """`count` distinct nodes that are no bumps, in drawn order."""
    n = d["n_tiers"] * d["nx"] * d["ny"]
    pads = set((d["pad_xy"][:, 1].astype(np.int64) * d["nx"] + d["pad_xy"][:, 0]).tolist())
    got = rng.choice(n, size=min(n, count + len(pads)), replace=False)
    return np.asarray([v for v in got.tolist() if v not in pads][:count], dtype=np.int64)


def _plan_size(case, i):
    """Tiers and side of plan i: the sizes of a batch do not hang on the seed."""
    return 2 + i % 3, case["lo"] + (case["hi"] - case["lo"]) * (2 * i + 1) // (2 * case["plans"])


def _plans(case, seed):
    """Candidate plans: 2-4 tiers, square sides lo..hi, 16-512 TSV columns."""
    out = []
    for i in range(case["plans"]):
        rng = _rng(seed, 3, i)
        nt, side = _plan_size(case, i)
        out.append(_stack(rng, nt, side, side, int(rng.integers(16, min(512, side * side // 2) + 1)), 32))
    return out


def _screen_plans(case, seed):
    """Plans of the screening model's geometry: U[0.5, 2] S edges, TSV density
    U[0.5 %, 3 %] (10 S), bump density U[0.2 %, 1 %]."""
    nt, nx, ny = case["nt"], case["nx"], case["ny"]
    out = []
    for i in range(case["plans"]):
        rng = _rng(seed, 4, i)
        tsv = _distinct(rng, nx, ny, max(1, round(rng.uniform(0.005, 0.03) * nx * ny)))
        pad = _distinct(rng, nx, ny, max(1, round(rng.uniform(0.002, 0.01) * nx * ny)))
        out.append({"n_tiers": nt, "nx": nx, "ny": ny, "gx": rng.uniform(0.5, 2.0, (nt, ny, nx - 1)),
                    "gy": rng.uniform(0.5, 2.0, (nt, ny - 1, nx)), "tsv_xy": tsv,
                    "tsv_g": np.full((len(tsv), nt - 1), 10.0), "pad_xy": pad})
    return out


def _layers(case):
    """(inputs, outputs, kernel side, transposed) of the screening network."""
    c, nt = case["ch"], case["nt"]
    conv = lambda i, o: (i, o, 3, False)  # noqa: E731
    up = lambda i, o: (i, o, 1, True)  # noqa: E731
    return [conv(2 * nt + 2, c), conv(c, c), conv(c, 2 * c), conv(2 * c, 2 * c), conv(2 * c, 4 * c),
            conv(4 * c, 4 * c), conv(4 * c, 8 * c), conv(8 * c, 8 * c), up(8 * c, 4 * c),
            conv(8 * c, 4 * c), conv(4 * c, 4 * c), up(4 * c, 2 * c), conv(4 * c, 2 * c),
            conv(2 * c, 2 * c), up(2 * c, c), conv(2 * c, c), conv(c, c), (c, nt, 1, False)]


def _params(case, seed):
    """He-normal weights and small biases, in the documented order."""
    rng, out = _rng(seed, 5), []
    for cin, cout, k, up in _layers(case):
        width = 4 * cout if up else cout
        out.append(rng.standard_normal(k * k * cin * width) * math.sqrt(2.0 / (k * k * cin)))
        out.append(0.05 * rng.standard_normal(width))
    return np.concatenate(out).astype(np.float32)


def _labels(case, plans, seed):
    out = []
    for i, d in enumerate(plans):
        rng = _rng(seed, 6, i)
        nodes = _free_nodes(rng, d, case["labels"])
        out.append((nodes, rng.lognormal(0.0, 0.5, len(nodes))))
    return out


def _inputs(case, seed):
    kind = case["kind"]
    if kind in ("diag", "map", "pairs", "ir_drop"):
        rng = _rng(seed, 1)
        d = _stack(rng, case["nt"], case["nx"], case["ny"], case["tsv"], case["pitch"])
        s = {"desc": d}
        if kind in ("diag", "map"):
            s["nodes"] = _free_nodes(rng, d, case["nodes"]) if case["nodes"] else None
        elif kind == "pairs":
            ends = _free_nodes(rng, d, case["m"] + case["n"])
            s["a"], s["b"] = ends[: case["m"]], ends[case["m"]:]
        else:
            s["loads"] = _free_nodes(rng, d, case["loads"])
            s["amps"] = rng.uniform(0.0, 0.05, (case["scen"], len(s["loads"])))
        return s
    if kind in ("plans_pcg", "plans_map"):
        plans = _plans(case, seed)
        nodes = [_free_nodes(_rng(seed, 2, i), d, case["nodes"]) if case["nodes"] else None
                 for i, d in enumerate(plans)]
        return {"plans": plans, "nodes": nodes}
    if kind == "grid":
        rng = _rng(seed, 7)
        return {"r": rng.uniform(0.5, 2.0), "s": rng.uniform(0.5, 2.0),
                "xy": _distinct(rng, case["M"], case["N"], case["P"])}
    if kind == "reduced":
        rng = _rng(seed, 8)
        nt, nx, ny = case["nt"], case["nx"], case["ny"]
        return {"r": rng.uniform(0.5, 2.0, nt), "s": rng.uniform(0.5, 2.0, nt),
                "tsv": _distinct(rng, nx, ny, case["p"]),
                "tsv_r": rng.uniform(0.05, 1.0, (case["p"], nt - 1)),
                "bumps": _distinct(rng, nx, ny, case["m"]), "loads": _distinct(rng, nx, ny, case["n"])}
    plans = _screen_plans(case, seed)
    s = {"plans": plans, "params": _params(case, seed)}
    if kind == "grad":
        s["labels"] = _labels(case, plans, seed)
    return s


def _size(d):
    return d["n_tiers"] * d["nx"] * d["ny"]


def _empty(*shape):
    return torch.empty(*shape, dtype=torch.float64, device=DEV)


def prepare(case, seed):
    from paper_2607_05818_amd import reff

    s = _inputs(case, seed)
    s["case"], s["reff"], kind = case, reff, case["kind"]
    if kind in ("diag", "map", "pairs", "ir_drop"):
        s["pdn"] = reff.reff_build_pdn(s["desc"], device=0)
        n = _size(s["desc"])
        if kind in ("diag", "map"):
            s["out"] = _empty(n if s["nodes"] is None else len(s["nodes"]))
        elif kind == "pairs":
            s["out"] = _empty(len(s["a"]), len(s["b"]))
        else:
            s["out"] = _empty(case["scen"], n)
    elif kind in ("plans_pcg", "plans_map"):
        s["out"] = [_empty(_size(d) if v is None else len(v)) for d, v in zip(s["plans"], s["nodes"])]
    elif kind == "grid":
        s["out"] = _empty(len(s["xy"]), len(s["xy"]))
    elif kind == "reduced":
        s["out"] = _empty(case["m"], case["n"])
    else:
        s["model"] = reff.reff_surrogate_create(case["nt"], case["nx"], case["ny"], case["ch"], seed=1)
        reff.reff_surrogate_set_params(s["model"], s["params"])
        if kind == "predict":
            s["out"] = [_empty(_size(d)) for d in s["plans"]]
    return s


def run(s):
    reff, case = s["reff"], s["case"]
    kind = case["kind"]
    if kind == "diag":
        mixed = case["precision"] == "mixed"
        reff.reff_solve_diag(s["pdn"], s["nodes"], s["out"], rel_tol=case["tol"],
                             precision=reff.REFF_PREC_MIXED if mixed else reff.REFF_PREC_FP64)
        return s["out"]
    if kind == "map":
        reff.reff_selinv_diag(s["pdn"], s["nodes"], s["out"])
        return s["out"]
    if kind == "pairs":
        mode = reff.REFF_PAIRS_FLOATING if case["floating"] else reff.REFF_PAIRS_GROUNDED
        reff.reff_query_pairs(s["pdn"], s["a"], s["b"], mode, s["out"])
        return s["out"]
    if kind == "ir_drop":
        drop, pads, _ = reff.reff_ir_drop(s["pdn"], s["loads"], s["amps"], None, s["out"])
        return [drop, pads]
    if kind == "plans_pcg":
        reff.reff_batch_plans(s["plans"], s["nodes"], precision=reff.REFF_PREC_MIXED,
                              rel_tol=case["tol"], R_out=s["out"])
        return s["out"]
    if kind == "plans_map":
        reff.reff_selinv_batch(s["plans"], s["nodes"], s["out"])
        return s["out"]
    if kind == "grid":
        return reff.reff_grid_pairs(case["M"], case["N"], s["r"], s["s"], s["xy"], s["out"])
    if kind == "reduced":
        return reff.reff_reduced_pairs(case["nx"], case["ny"], s["r"], s["s"], s["tsv"], s["tsv_r"],
                                       s["bumps"], s["loads"], s["out"])
    if kind == "predict":
        return reff.reff_surrogate_predict(s["model"], s["plans"], s["out"])
    loss, grad = reff.reff_surrogate_loss_grad(s["model"], s["plans"], s["labels"])
    return [loss, grad]


# ---------------------------------------------------------------- work

def _map_flops(nt, nx, ny):
    """float64 operations of a factorisation and a selected inversion of one
    stack by nested dissection in the plane: a box of a x b columns splits at
    a wall of min(a, b) columns (s = nt min(a, b) unknowns) whose front also
    holds the walls around the box (q unknowns): s^3/3 + s^2 q + s q^2 to
    factor and 2/3 ((s + q)^3 - q^3) to invert.  ia and ib count the box's
    sides across a and across b that are walls."""
    total, boxes = 0.0, {(nx, ny, 0, 0): 1}
    while boxes:
        nxt = {}
        for (a, b, ia, ib), count in boxes.items():
            if a < b:
                a, b, ia, ib = b, a, ib, ia
            if b < 1:
                continue
            leaf = a * b <= 16
            s, q = nt * (a * b if leaf else b), nt * (ia * b + ib * a)
            total += count * (s ** 3 / 3 + s * s * q + s * q * q + 2 / 3 * ((s + q) ** 3 - q ** 3))
            if not leaf:
                for part, walls in (((a - 1) // 2, 1 + (ia > 1)), (a - 1 - (a - 1) // 2, 1 + (ia > 0))):
                    key = (part, b, walls, ib)
                    nxt[key] = nxt.get(key, 0) + count
        boxes = nxt
    return total


def _stack_bytes(nt, nx, ny):
    return 8.0 * nt * (2 * nx * ny)  # its edge conductances


def _solve_work(nt, nx, ny, cols, word):
    """One block of 64 solution columns written and read once per 64 solves,
    and the stencil applied once to it."""
    blocks = -(-cols // 64)
    n = nt * nx * ny
    return {"bytes": _stack_bytes(nt, nx, ny) + blocks * 2.0 * 64 * word * n,
            "flops": blocks * 64.0 * 10 * n}


def work(case):
    kind = case["kind"]
    if kind == "diag":
        return _solve_work(case["nt"], case["nx"], case["ny"], case["nodes"],
                           4 if case["precision"] == "mixed" else 8)
    if kind == "pairs":
        return _solve_work(case["nt"], case["nx"], case["ny"], case["m"] + case["n"], 8)
    if kind == "ir_drop":
        w = _solve_work(case["nt"], case["nx"], case["ny"], case["loads"], 8)
        n = case["nt"] * case["nx"] * case["ny"]
        return {"bytes": w["bytes"] + 8.0 * n * case["scen"],
                "flops": w["flops"] + 2.0 * n * case["loads"] * case["scen"]}
    if kind == "map":
        n = case["nt"] * case["nx"] * case["ny"]
        return {"bytes": _stack_bytes(case["nt"], case["nx"], case["ny"]) + 8.0 * n,
                "flops": _map_flops(case["nt"], case["nx"], case["ny"])}
    if kind in ("plans_pcg", "plans_map"):
        tot = {"bytes": 0.0, "flops": 0.0}
        for i in range(case["plans"]):
            nt, side = _plan_size(case, i)
            if kind == "plans_pcg":
                w = _solve_work(nt, side, side, case["nodes"], 4)
            else:
                w = {"bytes": _stack_bytes(nt, side, side) + 8.0 * nt * side * side,
                     "flops": _map_flops(nt, side, side)}
            tot = {k: tot[k] + w[k] for k in tot}
        return tot
    if kind == "grid":
        M, N, P = case["M"], case["N"], case["P"]
        return {"bytes": 8.0 * P * P, "flops": 1.0 * P * P * M * N}
    if kind == "reduced":
        p, d, m, n = case["p"], case["nt"], case["m"], case["n"]
        k = p * (d - 1)
        tables = d * p * p + 2.0 * p * (m + n)  # resistances of TSV-TSV and endpoint-TSV pairs
        return {"bytes": 8.0 * (m * n + tables),
                "flops": tables * case["nx"] * case["ny"] + k ** 3 / 3 + 2.0 * k * k * (m + n) +
                4.0 * m * n * p}
    px, at = case["plans"] * case["nx"] * case["ny"], 0.0
    level = [0, 0, 1, 1, 2, 2, 3, 3, 3, 2, 2, 2, 1, 1, 1, 0, 0, 0]
    params = 0
    for (cin, cout, k, up), lev in zip(_layers(case), level):
        wide = 4 * cout if up else cout
        at += 2.0 * k * k * cin * wide * px / 4 ** lev
        params += k * k * cin * wide + wide
    io = px * (2.0 * (2 * case["nt"] + 2)) + 4.0 * params
    if kind == "predict":
        return {"bytes": io + 8.0 * px * case["nt"], "flops": at}
    return {"bytes": io + 4.0 * params, "flops": 3.0 * at}


# ---------------------------------------------------------------- float64 values

class _Grid:
    """G of a stack on [columns, tier, y, x] tensors: Dirichlet nodes masked."""

    def __init__(self, d, grounded):
        nt, nx, ny = d["n_tiers"], d["nx"], d["ny"]
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)  # noqa: E731
        self.gx, self.gy = t(d["gx"]), t(d["gy"])
        self.gz = torch.zeros(max(nt - 1, 0), ny, nx, dtype=torch.float64, device=DEV)
        x, y = (torch.as_tensor(d["tsv_xy"][:, k].astype(np.int64), device=DEV) for k in (0, 1))
        for k in range(nt - 1):
            self.gz[k, y, x] = t(d["tsv_g"][:, k])
        self.free = torch.ones(nt, ny, nx, dtype=torch.float64, device=DEV)
        self.free.view(-1)[torch.as_tensor(grounded, device=DEV)] = 0.0
        diag = torch.zeros_like(self.free)
        diag[:, :, 1:] += self.gx
        diag[:, :, :-1] += self.gx
        diag[:, 1:] += self.gy
        diag[:, :-1] += self.gy
        diag[1:] += self.gz
        diag[:-1] += self.gz
        self.diag = diag

    def apply(self, v):
        y = self.diag * v
        y[..., 1:] -= self.gx * v[..., :-1]
        y[..., :-1] -= self.gx * v[..., 1:]
        y[..., 1:, :] -= self.gy * v[..., :-1, :]
        y[..., :-1, :] -= self.gy * v[..., 1:, :]
        if self.gz.numel():
            y[:, 1:] -= self.gz * v[:, :-1]
            y[:, :-1] -= self.gz * v[:, 1:]
        return y.mul_(self.free)

    def solve(self, rhs, tol):
        """Conjugate gradients per column with the diagonal as preconditioner."""
        dot = lambda a, b: (a * b).sum(dim=(1, 2, 3), keepdim=True)  # noqa: E731
        r = rhs * self.free
        x, scale = torch.zeros_like(r), self.free / self.diag
        z = r * scale
        p, rz = z.clone(), dot(r, z)
        stop = rz * tol * tol
        for it in range(20000):
            q = self.apply(p)
            alpha = rz / dot(p, q).clamp_min(1e-300)
            x += alpha * p
            r -= alpha * q
            z = r * scale
            new = dot(r, z)
            if it % 16 == 0 and bool((new <= stop).all()):
                break
            p.mul_(new / rz.clamp_min(1e-300)).add_(z)
            rz = new
        return x

    def units(self, nodes, tol):
        """G^-1 e_v for the nodes v, as rows of a [len(nodes), n] tensor."""
        rhs = torch.zeros(len(nodes), *self.free.shape, dtype=torch.float64, device=DEV)
        at = torch.as_tensor(nodes, device=DEV)
        rhs.view(len(nodes), -1)[torch.arange(len(nodes), device=DEV), at] = 1.0
        return self.solve(rhs, tol).reshape(len(nodes), -1)


def _pads(d):
    return np.unique(d["pad_xy"][:, 1].astype(np.int64) * d["nx"] + d["pad_xy"][:, 0])


def _diag_values(d, nodes):
    g, out = _Grid(d, _pads(d)), []
    for i in range(0, len(nodes), 64):
        part = nodes[i: i + 64]
        # e^T x of conjugate gradients has the square of the solution's error
        x = g.units(part, 1e-8)
        out.append(x[torch.arange(len(part), device=DEV), torch.as_tensor(part, device=DEV)])
    return torch.cat(out)


def _map_values(d):
    """diag(G^-1) by block elimination along the longer axis of the plane from
    both ends: with C the blocks' own matrices and b the (diagonal) couplings,
    left_i = (C_i - b b^T o left_{i-1})^-1, right_i likewise, and block i of
    G^-1 is (C_i - b b^T o left_{i-1} - b b^T o right_{i+1})^-1."""
    g = _Grid(d, _pads(d))
    gx, gy, gz, diag, free = g.gx, g.gy, g.gz, g.diag, g.free
    if d["ny"] > d["nx"]:
        gx, gy = gy.transpose(1, 2), gx.transpose(1, 2)
        gz, diag, free = gz.transpose(1, 2), diag.transpose(1, 2), free.transpose(1, 2)
    nt, ny, nx = diag.shape
    idx = torch.arange(nt * ny, device=DEV).reshape(nt, ny)

    def own(x):
        m = torch.zeros(nt * ny, nt * ny, dtype=torch.float64, device=DEV)
        f = free[:, :, x]
        m[idx, idx] = torch.where(f > 0, diag[:, :, x], torch.ones_like(f))
        for a, b, w in ((idx[:, 1:], idx[:, :-1], gy[:, :, x] * f[:, 1:] * f[:, :-1]),
                        (idx[1:], idx[:-1], gz[:, :, x] * f[1:] * f[:-1])):
            m[a, b] = -w
            m[b, a] = -w
        return m

    couple = [(gx[:, :, x] * free[:, :, x] * free[:, :, x + 1]).reshape(-1) for x in range(nx - 1)]
    right = [None] * nx
    for x in range(nx - 1, 0, -1):
        m = own(x)
        if right[x] is not None:
            m -= right[x]
        b = couple[x - 1]
        right[x - 1] = b[:, None] * torch.linalg.inv(m) * b
    out, left = torch.empty(nt, ny, nx, dtype=torch.float64, device=DEV), None
    for x in range(nx):
        m = own(x)
        if left is not None:
            m -= left
        full = m if right[x] is None else m - right[x]
        out[:, :, x] = torch.linalg.inv(full).diagonal().reshape(nt, ny)
        if x + 1 < nx:
            left = couple[x][:, None] * torch.linalg.inv(m) * couple[x]
    out = out * free
    return (out.transpose(1, 2) if d["ny"] > d["nx"] else out).reshape(-1)


def _grid_values(M, N, r, s, xy):
    """Two-point resistances on a uniform grid: the double cosine sum."""
    x = torch.as_tensor(xy[:, 0].astype(np.float64), device=DEV) + 0.5
    y = torch.as_tensor(xy[:, 1].astype(np.float64), device=DEV) + 0.5
    m = torch.arange(1, M, dtype=torch.float64, device=DEV)
    n = torch.arange(1, N, dtype=torch.float64, device=DEV)
    cx, cy = torch.cos(math.pi / M * x[:, None] * m), torch.cos(math.pi / N * y[:, None] * n)
    T = torch.zeros(len(xy), len(xy), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 25) // max(1, len(xy) * (N - 1)))
    for k in range(0, M - 1, step):
        mk = m[k: k + step]
        w = 1.0 / ((1 - torch.cos(math.pi / M * mk))[:, None] / r + (1 - torch.cos(math.pi / N * n)) / s)
        X = (cx[:, k: k + step, None] * cy[:, None, :]).reshape(len(xy), -1)
        T += (X * w.reshape(-1)) @ X.t()
    t = T.diagonal()
    R = r * (x[:, None] - x).abs() / N + s * (y[:, None] - y).abs() / M + \
        2.0 / (M * N) * (t[:, None] + t - 2 * T)
    return R.fill_diagonal_(0.0)


def _reduced_values(case, s):
    """The saddle-point system of the TSV currents and supply differences,
    one dense solve with every endpoint's right-hand side."""
    d, nx, ny, p, m, n = (case[k] for k in ("nt", "nx", "ny", "p", "m", "n"))
    RT, first, last = [], None, None
    for t in range(d):
        pts = [s["tsv"]] + ([s["bumps"]] if t == 0 else []) + ([s["loads"]] if t == d - 1 else [])
        R = _grid_values(nx, ny, s["r"][t], s["s"][t], np.concatenate(pts))
        RT.append(R[:p, :p].clone())
        first = R[p:, :p].clone() if t == 0 else first
        last = R[p:, :p].clone() if t == d - 1 else last
    k = d - 1
    C = torch.zeros((p + 1) * k, (p + 1) * k, dtype=torch.float64, device=DEV)
    seg = torch.as_tensor(s["tsv_r"], device=DEV)
    for a in range(k):
        C[a * p:(a + 1) * p, a * p:(a + 1) * p] = -(RT[a] + RT[a + 1]) / 2 + torch.diag(seg[:, a])
        if a + 1 < k:
            C[a * p:(a + 1) * p, (a + 1) * p:(a + 2) * p] = RT[a + 1] / 2
            C[(a + 1) * p:(a + 2) * p, a * p:(a + 1) * p] = RT[a + 1] / 2
        C[k * p + a, a * p:(a + 1) * p] = 1.0
        C[a * p:(a + 1) * p, k * p + a] = 1.0
    b = torch.zeros((p + 1) * k, m + n, dtype=torch.float64, device=DEV)
    b[:p, :m] -= first.t() / 2
    b[(k - 1) * p:k * p, m:] -= last.t() / 2
    b[k * p:] = 0.5
    x = torch.linalg.solve(C, b)
    g = x.t() @ b
    e = g.diagonal()
    return -(e[:m, None] + e[m:] + g[:m, m:] + g[m:, :m].t())


def _network(case, plans, params):
    """log R [plan, tier, y, x] of the screening network in float64."""
    nt, nx, ny = case["nt"], case["nx"], case["ny"]
    x = torch.zeros(len(plans), 2 * nt + 2, ny, nx, dtype=torch.float64)
    for i, d in enumerate(plans):
        x[i, :nt, :, :-1] = torch.as_tensor(np.log(d["gx"]))
        x[i, nt:2 * nt, :-1] = torch.as_tensor(np.log(d["gy"]))
        mean = d["tsv_g"].mean(axis=1) if nt > 1 else np.zeros(len(d["tsv_g"]))
        x[i, 2 * nt, d["tsv_xy"][:, 1], d["tsv_xy"][:, 0]] = torch.as_tensor(np.log1p(mean))
        x[i, 2 * nt + 1, d["pad_xy"][:, 1], d["pad_xy"][:, 0]] = 1.0
    x, at, layers = x.to(DEV), 0, []
    for cin, cout, k, up in _layers(case):
        wide = 4 * cout if up else cout
        w = params[at: at + k * k * cin * wide].reshape(k * k * cin, wide)
        at += k * k * cin * wide
        layers.append((w, params[at: at + wide], cout, k, up))
        at += wide

    def layer(v, i, relu=True):
        w, b, cout, k, up = layers[i]
        B, c, H, W = v.shape
        if k == 3:
            p = torch.nn.functional.pad(v, (1, 1, 1, 1))
            v = torch.stack([p[:, :, a:a + H, q:q + W] for a in range(3) for q in range(3)], dim=1)
            v = v.reshape(B, 9 * c, H, W)
        y = v.permute(0, 2, 3, 1).reshape(B * H * W, -1) @ w + b
        if up:
            y = y.reshape(B, H, W, 2, 2, cout).permute(0, 5, 1, 3, 2, 4)
            return y.reshape(B, cout, 2 * H, 2 * W)
        y = y.reshape(B, H, W, cout).permute(0, 3, 1, 2)
        return torch.relu(y) if relu else y

    pool = torch.nn.functional.max_pool2d
    skip = []
    for i in (0, 2, 4):
        x = layer(layer(x, i), i + 1)
        skip.append(x)
        x = pool(x, 2)
    x = layer(layer(x, 6), 7)
    for i in (8, 11, 14):
        x = torch.cat([layer(x, i), skip.pop()], dim=1)
        x = layer(layer(x, i + 1), i + 2)
    return layer(x, 17, relu=False)


def exact(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    if kind == "diag":
        return _diag_values(s["desc"], s["nodes"])
    if kind in ("map", "plans_map"):
        plans = [s["desc"]] if kind == "map" else s["plans"]
        asked = [s["nodes"]] if kind == "map" else s["nodes"]
        # elimination takes max(nx, ny) steps on blocks of nt min(nx, ny); the
        # maps that fit about ten seconds have values
        out, spent = [], 0.0
        for d, v in zip(plans, asked):
            spent += max(d["nx"], d["ny"]) * max(d["n_tiers"] * min(d["nx"], d["ny"]), 400) ** 2
            R = _map_values(d) if spent <= 8e8 else None
            out.append(R if R is None or v is None else R[torch.as_tensor(v, device=DEV)])
        return out[0] if kind == "map" else out
    if kind == "plans_pcg":
        return [_diag_values(d, v) for d, v in zip(s["plans"], s["nodes"])]
    if kind == "pairs":
        d, ends = s["desc"], np.concatenate([s["a"], s["b"]])
        g = _Grid(d, _pads(d)[:1] if case["floating"] else _pads(d))
        K, m = g.units(ends, 1e-13)[:, torch.as_tensor(ends, device=DEV)], len(s["a"])
        K = (K + K.t()) / 2
        e = K.diagonal()
        return e[:m, None] + e[m:] - 2 * K[:m, m:]
    if kind == "ir_drop":
        d = s["desc"]
        g = _Grid(d, _pads(d))
        rhs = torch.zeros(case["scen"], _size(d), dtype=torch.float64, device=DEV)
        rhs[:, torch.as_tensor(s["loads"], device=DEV)] = torch.as_tensor(s["amps"], device=DEV)
        v = g.solve(rhs.reshape(-1, *g.free.shape), 1e-14)
        # a bump delivers the currents of its edges
        whole = _Grid(d, np.zeros(0, dtype=np.int64))
        at = torch.as_tensor(d["pad_xy"][:, 1].astype(np.int64) * d["nx"] + d["pad_xy"][:, 0], device=DEV)
        return [v.reshape(case["scen"], -1), -whole.apply(v).reshape(case["scen"], -1)[:, at]]
    if kind == "grid":
        return _grid_values(case["M"], case["N"], s["r"], s["s"], s["xy"])
    if kind == "reduced":
        return _reduced_values(case, s)
    params = torch.as_tensor(s["params"].astype(np.float64), device=DEV)
    params.requires_grad_(kind == "grad")
    logr = _network(case, s["plans"], params)
    if kind == "predict":
        out = []
        for v, d in zip(torch.exp(logr), s["plans"]):
            v = v.reshape(-1).clone()
            v[torch.as_tensor(_pads(d), device=DEV)] = 0.0
            out.append(v)
        return out
    err = []
    for v, (nodes, R) in zip(logr, s["labels"]):
        err.append(v.reshape(-1)[torch.as_tensor(nodes, device=DEV)] - torch.as_tensor(np.log(R), device=DEV))
    loss = torch.cat(err).square().mean()
    loss.backward()
    # the loss comes back as a number, the gradient as an array
    return [float(loss), params.grad.cpu().numpy()]
