"""Offline tuner of the sweep kernel's launch variants; writes tuning.json beside this file.

The variants compute the same values bit for bit (the tuner checks it on every measurement) and
differ only in speed. What there is to choose is the loads of dense FP32 costs: the second batch of
each wave's cost rows straight into LDS, or into registers after the first batch. (The instances
capped at 2 waves per SIMD differ from the others for clouds of more than 3 coordinates alone, which
take them by default.)
For each size the tuner times a short solve of the paper's schedule (gamma_f = 2^8, FP32 sweeps; the
device time the library reports, best of three after a warm-up) under both, and keeps the faster; it
must beat the default by more than 1 % to replace it. The sizes are past 1024 tiles: below, a solve's
trials run inside one kernel that has no variants, and timing one would say nothing about the sweep.
Each measured size covers the sizes up to the geometric mean with the next one, the first all smaller
ones. The library reads the file when a context is created (include/mdot.h, "Launch-variant tuning").

Run on the GPU:  python -m paper_2307_08507_amd.tune [--out FILE] [--quick]
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
DEFAULT_OUT = os.path.join(HERE, "tuning.json")
STAGE_DEFAULT = 2048  # the library's built-in staging threshold (tiles)
MAX_N = 131072  # MDOT_MAX_N of include/mdot.h
RESIDENT_TILES = 1024  # the most tiles whose trials run inside one kernel


def _problem(n: int, dev):
    """(descriptor, r, c, kept tensors) of a grid workload of size n with a dense FP32 cost."""
    import numpy as np
    import torch

    from . import mdot as M
    from . import workloads as W

    k = int(round(math.sqrt(n)))
    assert k * k == n
    r = torch.tensor(W.grid_problem_marginals(k, "smooth", 11), dtype=torch.float64, device=dev)
    c = torch.tensor(W.grid_problem_marginals(k, "smooth", 12), dtype=torch.float64, device=dev)
    Xd = torch.tensor(W.grid_coords(k).astype(np.float64), device=dev)
    C = torch.empty((n, n), dtype=torch.float32, device=dev)
    for a in range(0, n, 1024):
        d = Xd[a:a + 1024, None, :] - Xd[None, :, :]
        C[a:a + 1024] = ((d * d).sum(-1) / (2.0 * (k - 1) ** 2)).float()
    return M.dense_cost(C), r, c, (C,)


def _time(ctx, desc, r, c, reps: int = 3):
    import torch

    from . import mdot as M

    prm = M.default_params(gamma_f=2.0**8)
    u = torch.empty(r.numel(), dtype=torch.float64, device=r.device)
    v = torch.empty_like(u)
    ctx.solve(desc, r, c, 1e-4, prm, u, v)  # warm-up (graph capture, caches)
    best, ref = math.inf, None
    for _ in range(reps):
        res = ctx.solve(desc, r, c, 1e-4, prm, u, v)
        best = min(best, res.seconds)
        ref = (res.primal_cost, res.dual_bound, res.sweeps, bytes(u.cpu().numpy().tobytes()))
    return best, ref


def tune(sizes, log=print):
    import torch

    from . import mdot as M

    dev = torch.device("cuda", 0)
    ctx = M.Context(0)
    entries = []
    for i, n in enumerate(sizes):
        tiles = ((n + 63) // 64) * ((n + 255) // 256)
        if tiles <= RESIDENT_TILES:
            raise ValueError(f"n={n}: a solve of {tiles} tiles does not run the sweep kernel's variants")
        desc, r, c, keep = _problem(n, dev)
        times, refs = {}, {}
        for val in (0, 1):
            ctx.tune_override(occ=0, stage=val)
            times[f"stage{val}"], refs[f"stage{val}"] = _time(ctx, desc, r, c)
        ctx.tune_override(0, -1)
        if len(set(refs.values())) != 1:
            raise RuntimeError(f"f32 n={n}: launch variants gave different results")
        default = "stage1" if tiles > STAGE_DEFAULT else "stage0"
        best = min(times, key=times.get)
        choice = best if times[best] < 0.99 * times[default] else default
        entries.append({"code": "f32", "n_max": MAX_N if i + 1 == len(sizes) else int(math.sqrt(n * sizes[i + 1])), "occ": 4,
                        "stage_min_tiles": 0 if choice == "stage1" else 0x7FFFFFFF, "measured_at_n": n,
                        "solve_device_s": {k: round(t, 6) for k, t in sorted(times.items())}, "default": default})
        log(f"f32 n={n}: " + ", ".join(f"{k} {t * 1e3:.2f} ms" for k, t in sorted(times.items()))
            + f" -> {choice} (default {default})")
        del keep
    ctx.close()
    return entries


def write(entries, path):
    """One JSON object per line inside a list, in (code, n_max) order: the library reads it line by line."""
    entries = sorted(entries, key=lambda e: (e["code"], e["n_max"]))
    with open(path, "w") as f:
        f.write("[\n")
        for k, e in enumerate(entries):
            f.write("  " + json.dumps(e, sort_keys=False) + ("," if k + 1 < len(entries) else "") + "\n")
        f.write("]\n")


def main() -> int:
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--out", default=DEFAULT_OUT)
    ap.add_argument("--quick", action="store_true", help="fewer sizes (a smoke run of the tuner)")
    args = ap.parse_args()
    entries = tune([5184, 9216] if args.quick else [5184, 7056, 9216, 12544, 16384],
                   log=lambda s: print(s, file=sys.stderr, flush=True))
    write(entries, args.out)
    print(args.out)
    return 0


if __name__ == "__main__":
    sys.exit(main())
