"""The sweep's launch variants compute the same bits where they are what runs: past the sizes of the
resident kernels, and in an engine whose solves in flight are of different cost types."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2307_08507_amd import mdot as M  # noqa: E402
from paper_2307_08507_amd import workloads as W  # noqa: E402


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


def _cloud(n, d, kind):
    XY = torch.randn(2 * n * d, device="cuda", dtype=torch.float32, generator=torch.Generator("cuda").manual_seed(n + d))
    return M.point_cost(XY, n, d, kind)


def _desc(name, n):
    if name == "f32":
        return M.dense_cost(torch.rand(n, n, device="cuda", dtype=torch.float32, generator=torch.Generator("cuda").manual_seed(n)))
    return _cloud(n, int(name[-1]), "l1" if name.startswith("l1") else "sqeuclid")


def _solve(ctx, desc, n, engine=False):
    r, c = dev(W.dirichlet_marginal(n, 1)), dev(W.dirichlet_marginal(n, 2))
    u, v = torch.empty_like(r), torch.empty_like(c)
    out = []
    for prec in ("f32", "f64"):
        prm = M.default_params(gamma_f=64.0, precision=prec)
        if engine:
            res = ctx.poll(ctx.submit(desc, r, c, 1e-3, prm, u, v), wait=True)
        else:
            res = ctx.solve(desc, r, c, 1e-3, prm, u, v)
        out += [res.sweeps, res.primal_cost, res.dual_bound, u.cpu().numpy(), v.cpu().numpy()]
    return out


@pytest.mark.parametrize("name", ["sq2", "sq3", "sq5", "l12", "l13", "l15", "f32"])
def test_variants_past_the_resident_kernels(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 4200  # 66 x 17 tiles
    desc = _desc(name, n)
    u, v = dev(np.random.default_rng(1).standard_normal(n) * 0.3), dev(np.random.default_rng(2).standard_normal(n) * 0.3)
    ctx = M.Context(0)
    try:
        outs = []
        for occ, stage in ((4, 0), (2, 0), (4, 1), (2, 1)):
            ctx.tune_override(occ, stage)
            print(f"variants {name} occ={occ} stage={stage}", flush=True)
            out = _solve(ctx, desc, n)
            for prec in ("f32", "f64"):
                lr, lc = torch.empty_like(u), torch.empty_like(v)
                ctx.lse2(desc, u, v, 40.0, lr, lc, precision=prec)
                out += [lr.cpu().numpy(), lc.cpu().numpy()]
            outs.append(out)
        for o in outs[1:]:
            for a, b in zip(outs[0], o):
                assert np.array_equal(a, b)
    finally:
        ctx.close()


@pytest.mark.parametrize("name", ["sq2", "l13", "sq5", "f32"])
def test_variants_in_a_mixed_engine(name):
    # beside a solve of another cost type the engine's steps are kernels of their own
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 400
    desc, other = _desc(name, n), M.dense_cost(torch.rand(48, 48, device="cuda", dtype=torch.float64))
    r, c = dev(W.dirichlet_marginal(48, 1)), dev(W.dirichlet_marginal(48, 2))
    outs = []
    for occ in (4, 2):
        ctx = M.Context(0)
        try:
            ctx.tune_override(occ, -1)
            print(f"variants in the engine {name} occ={occ}", flush=True)
            u, v = torch.empty_like(r), torch.empty_like(c)
            ctx.submit(other, r, c, 1e-12, M.default_params(precision="f64", gamma_cap=1e9), u, v)
            outs.append(_solve(ctx, desc, n, engine=True))
        finally:
            ctx.close()
    for a, b in zip(outs[0], outs[1]):
        assert np.array_equal(a, b)
