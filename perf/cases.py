"""Performance cases of the optimal-transport library, through its public entry points.

Four kinds of call are covered, each over the sizes and options its users take:

* "lse": one two-sided LogSumExp sweep (Context.lse2 or its allocation-free variant): dense
  costs in every stored type and costs recomputed from points, with and without a prediction of
  the row sums, FP32 and FP64 exponentials, square and rectangular, aligned and ragged rows;
* "round": rounding a plan onto the marginals and certifying it (Context.round_certify);
* "solve": one whole solve to a certified gap, or over the fixed annealing schedule;
* "batch": several solves of uneven sizes submitted together to the serving engine.

Inputs are made from a seed alone: pixel grids with the image families of
`paper_2307_08507_amd.workloads`, random costs and 3-D Gaussian-mixture clouds. Potentials for
the sweeps are Sinkhorn iterates, the kind a solver has in hand.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2307_08507_amd import mdot as M
from paper_2307_08507_amd import workloads as W

DTYPES = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2, "sqeuclid": 0, "l1": 0}
# FP64 operations per entry of one sweep: the exponent argument (3), the exponential (taken as
# 1), a row and a column accumulation (3); d more pairs where the entry is recomputed from points
OPS = 7
# Sweeps per annealing stage in the work of a solve: about what the easiest problems take
SWEEPS_PER_STAGE = 16


def listed():
    return [
        # The small grid workload (16 x 16 pixels) of the smoke run: one sweep, all latency.
        {"name": "lse 256 f32", "kind": "lse", "m": 256, "n": 256, "cost": "f32", "d": 0, "prec": "f32",
         "shift": False, "noalloc": False, "gamma": 64.0},
        # Images of two resolutions, odd sizes, the paper's precision throughout.
        {"name": "lse 1000x777 f64", "kind": "lse", "m": 1000, "n": 777, "cost": "f64", "d": 0, "prec": "f64",
         "shift": False, "noalloc": False, "gamma": 300.0},
        # A line-search trial at the benchmark's size: the row sums are predicted, and the caller
        # cannot allocate.
        {"name": "lse 4096 f32 noalloc", "kind": "lse", "m": 4096, "n": 4096, "cost": "f32", "d": 0, "prec": "f32",
         "shift": True, "noalloc": True, "gamma": 1024.0},
        # A half-precision store with rows that no wide load can take (odd length).
        {"name": "lse 8191 bf16", "kind": "lse", "m": 8191, "n": 8191, "cost": "bf16", "d": 0, "prec": "f32",
         "shift": False, "noalloc": False, "gamma": 128.0},
        # The largest benchmark grid (128 x 128 pixels) with a stored cost: 1 GiB, read from HBM.
        {"name": "lse 16384 f32", "kind": "lse", "m": 16384, "n": 16384, "cost": "f32", "d": 0, "prec": "f32",
         "shift": False, "noalloc": False, "gamma": 512.0},
        # The same grid with the cost recomputed from pixel coordinates, and the prediction a
        # solver has.
        {"name": "lse 16384 points", "kind": "lse", "m": 16384, "n": 16384, "cost": "sqeuclid", "d": 2, "prec": "f32",
         "shift": True, "noalloc": False, "gamma": 512.0},
        # Certifying a caller's own potentials at the benchmark's size.
        {"name": "round 4096 f32", "kind": "round", "m": 4096, "n": 4096, "cost": "f32", "d": 0, "gamma": 1024.0},
        # The smoke run: a whole solve of the small grid workload to gap 1e-4.
        {"name": "solve 256 f32", "kind": "solve", "k": 16, "cost": "f32", "metric": "sqeuclid", "family": "smooth",
         "prec": "f32", "gap": 1e-4, "gamma_f": 0.0},
        # The paper's precision and its fixed schedule, on heavy-tailed images with the L1 cost.
        {"name": "solve 1024 f64", "kind": "solve", "k": 32, "cost": "f64", "metric": "l1", "family": "cauchy",
         "prec": "f64", "gap": 1e-4, "gamma_f": 512.0},
        # The benchmark's problem (64 x 64 pixels) to a certified gap of 1e-4.
        {"name": "solve 4096 f32", "kind": "solve", "k": 64, "cost": "f32", "metric": "sqeuclid", "family": "blobs",
         "prec": "f32", "gap": 1e-4, "gamma_f": 0.0},
        # The benchmark's size with the cost recomputed from pixel coordinates, L1 distances.
        {"name": "solve 4096 points", "kind": "solve", "k": 64, "cost": "l1", "metric": "l1", "family": "uniform",
         "prec": "f32", "gap": 1e-4, "gamma_f": 0.0},
        # The serving workload: requests over 3-D clouds of uneven sizes in flight together.
        {"name": "batch 6 clouds", "kind": "batch", "count": 6, "n_lo": 512, "n_hi": 2500, "gap": 1e-4},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["lse", "lse", "lse", "round", "solve", "solve", "batch"])
    if kind == "lse":
        cost = rng.choice(["f32", "f32", "f64", "f16", "bf16", "sqeuclid", "l1"])
        points = cost in ("sqeuclid", "l1")
        m = _log_uniform(rng, 200, 16000)
        n = m if rng.random() < 0.6 else max(64, min(16000, int(m * rng.uniform(0.3, 2.0))))
        if rng.random() < 0.5:  # half of the sizes allow whole vector loads
            n = max(64, n // 4 * 4)
        noalloc = max(m, n) <= 4096 and rng.random() < 0.3
        return {"kind": "lse", "m": m, "n": n, "cost": cost, "d": rng.choice([2, 2, 3, 5]) if points else 0,
                "prec": "f64" if cost == "f64" else rng.choice(["f32", "f32", "f64"]), "shift": rng.random() < 0.5,
                "noalloc": noalloc, "gamma": float(2 ** rng.randint(4, 11))}
    if kind == "round":
        m = _log_uniform(rng, 200, 6000)
        n = m if rng.random() < 0.6 else max(64, min(6000, int(m * rng.uniform(0.5, 1.6))))
        cost = rng.choice(["f32", "f32", "f64", "sqeuclid"])
        return {"kind": "round", "m": m, "n": n, "cost": cost, "d": rng.choice([2, 3]) if cost == "sqeuclid" else 0,
                "gamma": float(2 ** rng.randint(6, 11))}
    if kind == "solve":
        metric = rng.choice(["sqeuclid", "l1"])
        store = rng.choice(["f32", "f32", "f16", "points", "f64"])
        k = max(12, min(60, _log_uniform(rng, 12, 60)))
        fixed = rng.random() < 0.3
        return {"kind": "solve", "k": k, "cost": metric if store == "points" else store, "metric": metric,
                "family": rng.choice(sorted(W.FAMILIES)), "prec": "f64" if store == "f64" else "f32", "gap": 1e-4,
                "gamma_f": 256.0 if fixed else 0.0}
    lo = _log_uniform(rng, 300, 700)
    return {"kind": "batch", "count": rng.randint(2, 8), "n_lo": lo, "n_hi": int(lo * rng.uniform(1.5, 3.5)), "gap": 1e-4}


# ------------------------------------------------------------------ inputs

def _entries(case, cost, rows=slice(None)):
    """Rows of the scaled cost matrix in FP64, from what the library is given."""
    if case["cost"] in ("sqeuclid", "l1"):
        xy, m, d = cost["data"].double(), case["m"], case["d"]
        x, y = xy[: m * d].reshape(m, d)[rows], xy[m * d:].reshape(-1, d)
        raw = torch.zeros(x.shape[0], y.shape[0], dtype=torch.float64, device=x.device)
        for e in range(d):
            t = x[:, e, None] - y[None, :, e]
            raw += t * t if case["cost"] == "sqeuclid" else t.abs()
        return raw * cost["scale"]
    return cost["data"][rows].double() * cost["scale"]


def _blocks(m, n):
    step = max(1, min(m, (1 << 25) // n))
    return [slice(i, min(m, i + step)) for i in range(0, m, step)]


def _row_lse(case, cost, u, v, gamma):
    return torch.cat([torch.logsumexp(v[None, :] - gamma * _entries(case, cost, b), dim=1) for b in
                      _blocks(case["m"], case["n"])]) + u


def _col_lse(case, cost, u, v, gamma):
    parts = [torch.logsumexp(u[b, None] - gamma * _entries(case, cost, b), dim=0) for b in _blocks(case["m"], case["n"])]
    return torch.logsumexp(torch.stack(parts), dim=0) + v


def _cost(case, seed):
    """The cost a program has: points of a cloud, a grid, or a stored matrix."""
    m, n, d = case["m"], case["n"], case["d"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if d:
        xy = torch.randn((m + n) * d, generator=gen, device="cuda", dtype=torch.float32).clamp_(-4.0, 4.0)
        top = 64.0 * d if case["cost"] == "sqeuclid" else 8.0 * d  # the clamp bounds every distance
        return {"data": xy, "scale": 1.0 / top}
    # a smooth part (distances between points on a line) and a rough one, as a stored cost has
    x = torch.rand(m, generator=gen, device="cuda", dtype=torch.float32)
    y = torch.rand(n, generator=gen, device="cuda", dtype=torch.float32)
    C = torch.rand(m, n, generator=gen, device="cuda", dtype=torch.float32)
    C.mul_(0.4).add_((x[:, None] - y[None, :]).abs_().mul_(0.6)).clamp_(0.0, 1.0)
    if case["cost"] == "f64":
        C = C.double().sub_(1e-9).clamp_(0.0, 1.0)
    return {"data": C.to(DTYPES[case["cost"]]), "scale": 1.0}


def _inputs(case, seed):
    """Everything a "lse" or "round" case is given, apart from descriptors and outputs."""
    m, n, gamma = case["m"], case["n"], case["gamma"]
    cost = _cost(case, seed)
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)

    def marginal(k):
        w = torch.rand(k, generator=gen, device="cuda", dtype=torch.float64) + 0.05
        return w / w.sum()

    r, c = marginal(m), marginal(n)
    s = {"cost": cost, "r": r, "c": c}
    u = torch.randn(m, generator=gen, device="cuda", dtype=torch.float64) * 0.3 + r.log()
    zero = torch.zeros(n, device="cuda", dtype=torch.float64)
    if case["kind"] == "lse":
        s["u"], s["v"] = u, c.log() - _col_lse(case, cost, u, zero, gamma)
        if case["shift"]:  # what the last accepted iterate predicts
            lr = _row_lse(case, cost, u, s["v"], gamma)
            s["shift"] = lr + 0.05 * torch.randn(m, generator=gen, device="cuda", dtype=torch.float64)
        return s
    for name, g in (("prev", gamma / 2 ** (1 / 3)), ("", gamma)):  # two annealing stages
        v = zero
        for _ in range(4):
            v = c.log() - _col_lse(case, cost, u, zero, g)
            u = r.log() - _row_lse(case, cost, torch.zeros_like(u), v, g)
        s["u" + name], s["v" + name] = u, v
        s["gamma" + name] = g
    return s


def _descriptor(case, cost):
    if case["d"]:
        return M.point_cost(cost["data"], case["n"], case["d"], case["cost"], scale=cost["scale"], m=case["m"])
    return M.dense_cost(cost["data"], scale=cost["scale"])


def _grid_descriptor(case):
    k = case["k"]
    xy = torch.as_tensor(W.grid_coords(k), device="cuda")
    top = 2.0 * (k - 1) ** 2 if case["metric"] == "sqeuclid" else 2.0 * (k - 1)
    if case["cost"] in ("sqeuclid", "l1"):
        both = torch.cat([xy, xy]).contiguous()
        return M.point_cost(both, k * k, 2, case["metric"], scale=1.0 / top)
    t = xy.double()[:, None, :] - xy.double()[None, :, :]
    C = ((t * t).sum(-1) if case["metric"] == "sqeuclid" else t.abs().sum(-1)) / top
    return M.dense_cost(C.to(DTYPES[case["cost"]]).contiguous())


def _f64(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def prepare(case, seed):
    ctx = M.Context(0)  # a program keeps one for all of its calls
    kind = case["kind"]
    if kind in ("lse", "round"):
        s = _inputs(case, seed)
        s.update(ctx=ctx, kind=kind, desc=_descriptor(case, s["cost"]))
        if kind == "lse":
            s.update(gamma=case["gamma"], prec=case["prec"], noalloc=case["noalloc"], lr=torch.empty_like(s["r"]),
                     lc=torch.empty_like(s["c"]))
        return s
    if kind == "solve":
        k = case["k"]
        r, c = (_f64(W.grid_problem_marginals(k, case["family"], 2 * seed + j)) for j in (0, 1))
        prm = M.default_params(precision=case["prec"], gamma_f=case["gamma_f"])
        return {"ctx": ctx, "kind": kind, "desc": _grid_descriptor(case), "r": r, "c": c, "gap": case["gap"], "prm": prm,
                "u": torch.empty_like(r), "v": torch.empty_like(c)}
    rng = np.random.default_rng(seed)
    reqs = []
    lo, hi = math.log(case["n_lo"]), math.log(case["n_hi"])
    for j in range(case["count"]):
        # sizes evenly spread over the range, the order and the clouds from the seed
        n = int(round(math.exp(lo + (hi - lo) * (j + 0.5) / case["count"])))
        s1 = int(rng.integers(1, 1 << 30))
        xy = np.concatenate([W.gmm_points(n, 3, s1), W.gmm_points(n, 3, s1 + 1)])
        r, c = _f64(W.dirichlet_marginal(n, s1 + 2)), _f64(W.dirichlet_marginal(n, s1 + 3))
        desc = M.point_cost(torch.as_tensor(xy, device="cuda").contiguous(), n, 3, "sqeuclid")
        reqs.append({"desc": desc, "r": r, "c": c, "u": torch.empty_like(r), "v": torch.empty_like(c)})
    return {"ctx": ctx, "kind": kind, "reqs": reqs, "gap": case["gap"], "prm": M.default_params()}


# ------------------------------------------------------------------ one pass

def _report(res, u, v):
    # marg_err_l1 is left out: on an exactly rounded plan it is the rounding error of two sums
    return {"primal_cost": res.primal_cost, "dual_bound": res.dual_bound, "gamma_final": res.gamma_final,
            "status": res.status, "stages": res.stages, "u": u, "v": v}


def run(s):
    ctx = s["ctx"]
    if s["kind"] == "lse":
        call = ctx.lse2_noalloc if s["noalloc"] else ctx.lse2
        rc = call(s["desc"], s["u"], s["v"], s["gamma"], s["lr"], s["lc"], shift=s.get("shift"), precision=s["prec"])
        return {"rc": rc, "lr": s["lr"], "lc": s["lc"]}
    if s["kind"] == "round":
        ub, lb, _ = ctx.round_certify(s["desc"], s["u"], s["v"], s["gamma"], s["r"], s["c"], u_prev=s["uprev"],
                                      v_prev=s["vprev"], gamma_prev=s["gammaprev"])
        return {"ub": ub, "lb": lb}
    if s["kind"] == "solve":
        res = ctx.solve(s["desc"], s["r"], s["c"], s["gap"], s["prm"], s["u"], s["v"])
        return _report(res, s["u"], s["v"])
    tickets = [ctx.submit(q["desc"], q["r"], q["c"], s["gap"], s["prm"], q["u"], q["v"]) for q in s["reqs"]]
    return [_report(ctx.poll(t, wait=True), q["u"], q["v"]) for t, q in zip(tickets, s["reqs"])]


# ------------------------------------------------------------------ work

def _stages(gamma_f):
    return math.ceil(3 * math.log2(max(gamma_f, 32.0) / 16.0)) + 1


def work(case):
    kind = case["kind"]
    if kind in ("lse", "round"):
        m, n = case["m"], case["n"]
        store = m * n * BYTES[case["cost"]] + (m + n) * case["d"] * 4
        ops = m * n * (OPS + 2 * case["d"])
        if kind == "lse":  # the cost, u and v in, both log-sums out, the prediction where there is one
            return {"bytes": store + 16 * (m + n) + (8 * m if case["shift"] else 0), "flops": ops}
        # the second reading of the cost needs every column sum of the first
        return {"bytes": 2 * store + 24 * (m + n), "flops": 2 * (ops + 8 * m * n)}
    if kind == "solve":
        n = case["k"] ** 2
        sweeps = SWEEPS_PER_STAGE * _stages(case["gamma_f"] or 512.0)
        d = 2 if case["cost"] in ("sqeuclid", "l1") else 0
        return {"bytes": sweeps * (n * n * BYTES[case["cost"]] + 32 * n), "flops": sweeps * n * n * (OPS + 2 * d)}
    lo, hi = math.log(case["n_lo"]), math.log(case["n_hi"])
    sizes = [math.exp(lo + (hi - lo) * (j + 0.5) / case["count"]) for j in range(case["count"])]
    sweeps = SWEEPS_PER_STAGE * _stages(512.0)
    return {"bytes": sweeps * sum(32 * n for n in sizes), "flops": sweeps * (OPS + 6) * sum(n * n for n in sizes)}


# ------------------------------------------------------------------ the same in 64 bits

def exact(case, seed):
    """Log-sums and certificates in plain FP64 torch. A solve stops anywhere inside its
    tolerance, so its iterates have no such value."""
    if case["kind"] not in ("lse", "round"):
        return None
    s = _inputs(case, seed)
    cost, u, v, gamma = s["cost"], s["u"], s["v"], case["gamma"]
    if case["kind"] == "lse":
        return {"rc": None, "lr": _row_lse(case, cost, u, v, gamma), "lc": _col_lse(case, cost, u, v, gamma)}
    r, c = s["r"], s["c"]
    blocks = _blocks(case["m"], case["n"])
    dg = gamma - s["gammaprev"]
    f = [u / gamma, (u - s["uprev"]) / dg]
    g = [v / gamma, (v - s["vprev"]) / dg]
    x = torch.clamp(r / torch.exp(_row_lse(case, cost, u, v, gamma)), max=1.0)
    cF = torch.zeros_like(c)
    gp = [torch.full_like(c, math.inf) for _ in f]
    fpp = [torch.empty_like(r) for _ in f]
    for b in blocks:
        C = _entries(case, cost, b)
        cF += (x[b, None] * torch.exp(u[b, None] + v[None, :] - gamma * C)).sum(0)
        for k in (0, 1):
            gp[k] = torch.minimum(gp[k], (C - f[k][b, None]).amin(0))
            fpp[k][b] = (C - g[k][None, :]).amin(1)
    y = torch.clamp(c / cF, max=1.0)
    errc = c - y * cF
    errr, part = torch.empty_like(r), torch.zeros((), dtype=torch.float64, device=r.device)
    Ce, fp, gpp = torch.empty_like(r), [torch.empty_like(r) for _ in f], [torch.full_like(c, math.inf) for _ in f]
    for b in blocks:
        C = _entries(case, cost, b)
        F = x[b, None] * torch.exp(u[b, None] + v[None, :] - gamma * C) * y[None, :]
        errr[b] = r[b] - F.sum(1)
        part += (F * C).sum()
        Ce[b] = (C * errc[None, :]).sum(1)
        for k in (0, 1):
            fp[k][b] = (C - gp[k][None, :]).amin(1)
            gpp[k] = torch.minimum(gpp[k], (C - fpp[k][b, None]).amin(0))
    total = errr.sum()
    ub = part + ((errr * Ce).sum() / total if total > 0 else 0.0)
    lb = max(max(float((c * gp[k]).sum() + (r * fp[k]).sum()), float((r * fpp[k]).sum() + (c * gpp[k]).sum())) for k in (0, 1))
    return {"ub": float(ub), "lb": lb}
