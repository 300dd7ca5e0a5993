"""Solves whose line-search trials run inside one kernel (at most 1024 tiles) against the serving
engine, whose steps are kernels of their own where a solve in flight has another cost type: the same
bits, at the edges of the workgroup layouts. Then the engine with its solves' trials in one kernel."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2307_08507_amd import mdot as M  # noqa: E402
from paper_2307_08507_amd import workloads as W  # noqa: E402


@pytest.fixture(scope="module")
def ctxs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    a, b = M.Context(0), M.Context(0)
    yield a, b, Company(b)
    a.close()
    b.close()


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


COUNTS = ("status", "primal_cost", "dual_bound", "gap", "gamma_final", "marg_err_l1", "grad_norm", "stages",
          "pncg_iters", "ls_trials", "sweeps", "cg_resets", "ls_failures", "fp64_retries", "cert_sweeps",
          "prec_switches")


class Company:
    """Solves of a cost type (5-D clouds) that keeps the engine on one-step kernels."""

    def __init__(self, eng):
        self.eng, self.n, self.tickets = eng, 48, []
        self.xy = dev(np.random.default_rng(3).random(2 * 48 * 5), torch.float32)
        self.r, self.c = dev(W.dirichlet_marginal(48, 1)), dev(W.dirichlet_marginal(48, 2))

    def keep(self):
        self.tickets = [t for t in self.tickets if self.eng.poll(t[0]) is None]
        while len(self.tickets) < 3:
            u, v = torch.empty_like(self.r), torch.empty_like(self.c)
            desc = M.point_cost(self.xy, 48, 5, "sqeuclid")
            self.tickets.append((self.eng.submit(desc, self.r, self.c, 1e-9, M.default_params(precision="f64"), u, v), u, v))


def _same(ctxs, desc, m, n, seed, gap, **kw):
    r, c = dev(W.dirichlet_marginal(m, seed)), dev(W.dirichlet_marginal(n, seed + 1))
    prm = M.default_params(**kw)
    outs, company = [], ctxs[2]
    for solve in (True, False):
        u, v = torch.empty_like(r), torch.empty_like(c)
        if solve:
            res = ctxs[0].solve(desc, r, c, gap, prm, u, v)
        else:
            company.keep()
            t = ctxs[1].submit(desc, r, c, gap, prm, u, v)
            while (res := ctxs[1].poll(t)) is None:
                ctxs[1].run(16)
                company.keep()
        outs.append((res, u.cpu().numpy(), v.cpu().numpy()))
    (a, ua, va), (b, ub, vb) = outs
    for f in COUNTS:
        assert getattr(a, f) == getattr(b, f), f
    assert np.array_equal(ua, ub) and np.array_equal(va, vb)
    assert a.sweeps > 0 and np.isfinite(ua).all()


# 1, 4 .. 256 tiles in one quad per workgroup, 257 .. 512 in two, .. 1024 in four; more finalize
# blocks than tile workgroups; ragged tiles; rows and columns that are not square
SIZES = [(1, 1), (5, 3), (64, 64), (64, 257), (130, 67), (256, 256), (1000, 1000), (70, 4000), (5000, 90), (2048, 2048),
         (2100, 2049), (2880, 3000), (4096, 4096), (8192, 2048)]


@pytest.mark.parametrize("m,n", SIZES)
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_dense_solves_equal_the_engine(ctxs, m, n, prec):
    print(f"resident dense {m}x{n} {prec}", flush=True)
    C = torch.rand(m, n, device="cuda", dtype=torch.float32)
    _same(ctxs, M.dense_cost(C), m, n, m + n, 1e-3, precision=prec, gamma_f=0.0 if n < 2000 else 64.0)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("m,n", [(250, 131), (2100, 2049), (4000, 4090)])
def test_stored_types_equal_the_engine(ctxs, dtype, m, n):
    print(f"resident {dtype} {m}x{n}", flush=True)
    C = torch.rand(m, n, device="cuda", dtype=torch.float64).to(dtype)
    for prec in ("f32", "f64"):
        _same(ctxs, M.dense_cost(C), m, n, 3, 1e-3, precision=prec, gamma_f=64.0)


@pytest.mark.parametrize("kind", ["sqeuclid", "l1"])
@pytest.mark.parametrize("d", [2, 3, 5])
@pytest.mark.parametrize("n", [300, 2200, 4096])
def test_clouds_equal_the_engine(ctxs, kind, d, n):
    print(f"resident cloud {kind} d={d} n={n}", flush=True)
    XY = torch.randn(2 * n * d, device="cuda", dtype=torch.float32, generator=torch.Generator("cuda").manual_seed(n))
    for prec in ("f32", "f64"):
        _same(ctxs, M.point_cost(XY, n, d, kind), n, n, n, 1e-3, precision=prec, gamma_f=0.0 if n < 2000 else 64.0)


def test_budgets_caps_and_late_stages_equal_the_engine(ctxs):
    # decisions that end a run of trials: the sweep budget at every phase, iteration and trial caps,
    # and the late stages that switch to FP64 exponentials
    C, r, c = W.grid_problem(16, "smooth", "sqeuclid", 0)
    desc = M.dense_cost(dev(C, torch.float32))
    for kw in ([dict(max_sweeps=k) for k in (1, 2, 3, 10, 57)] + [dict(max_pncg_iters=3), dict(max_ls_trials=1),
               dict(max_ls_trials=2), dict(warm_start=0), dict(projector=1, max_sweeps=400), dict(precond=1)]):
        print(f"resident {kw}", flush=True)
        _same(ctxs, desc, 256, 256, 1, 1e-3, **kw)
    _same(ctxs, desc, 256, 256, 1, 1e-8)


def test_many_contexts_on_streams_and_threads(ctxs):
    # solves that want the whole GPU at once: whoever cannot start leaves its steps to the one-step
    # kernels, and every result is the same
    import threading

    n = 1500
    C = torch.rand(n, n, device="cuda", dtype=torch.float32)
    r, c = dev(W.dirichlet_marginal(n, 1)), dev(W.dirichlet_marginal(n, 2))
    torch.cuda.synchronize()
    outs = [None] * 4

    def work(k):
        s = torch.cuda.Stream()
        ctx = M.Context(0, stream=s)
        u, v = torch.empty_like(r), torch.empty_like(c)
        for _ in range(3):
            res = ctx.solve(M.dense_cost(C), r, c, 1e-3, M.default_params(gamma_f=128.0), u, v)
        s.synchronize()
        outs[k] = (res.sweeps, res.primal_cost, u.cpu().numpy(), v.cpu().numpy())
        ctx.close()

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for o in outs[1:]:
        assert o[:2] == outs[0][:2]
        assert np.array_equal(o[2], outs[0][2]) and np.array_equal(o[3], outs[0][3])


# Solves in flight together: one, two and four tiles per workgroup, more tiles than fit, a batch that
# fits only when some have finished, and small solves in every slot
BATCHES = {"one": [(1, 1), (64, 257), (300, 300), (130, 67)], "two": [(1000, 1000), (700, 1300), (900, 512)],
           "four": [(584, 584), (761, 761), (991, 991), (1291, 1291), (1682, 1682), (2191, 2191)],
           "past": [(2500, 2500), (2200, 2600), (2400, 2300)], "slots": [(90 + k, 150 - k) for k in range(64)]}


@pytest.mark.parametrize("name", list(BATCHES))
@pytest.mark.parametrize("kind", ["points", "f32", "f64"])
def test_engine_batches_equal_the_solves(ctxs, name, kind):
    print(f"resident batch {name} {kind}", flush=True)
    probs = []
    for k, (m, n) in enumerate(BATCHES[name]):
        r, c = dev(W.dirichlet_marginal(m, 7 + k)), dev(W.dirichlet_marginal(n, 70 + k))
        if kind == "points":
            desc = M.point_cost(dev(np.random.default_rng(k).random((m + n) * 3), torch.float32), n, 3, "sqeuclid", m=m)
        else:
            desc = M.dense_cost(torch.rand(m, n, device="cuda", dtype=torch.float32 if kind == "f32" else torch.float64))
        probs.append((desc, r, c))
    prm = M.default_params(precision="f64" if kind == "f64" else "f32")
    eng = M.Context(0)
    try:
        held = []
        for desc, r, c in probs:
            u, v = torch.empty_like(r), torch.empty_like(c)
            held.append((eng.submit(desc, r, c, 1e-3, prm, u, v), u, v))
        assert all(h[0] is not None for h in held)
        while eng.inflight()[0]:
            eng.run(64)
        for (desc, r, c), (t, u, v) in zip(probs, held):
            u1, v1 = torch.empty_like(r), torch.empty_like(c)
            a, b = ctxs[0].solve(desc, r, c, 1e-3, prm, u1, v1), eng.poll(t)
            for f in COUNTS:
                assert getattr(a, f) == getattr(b, f), f
            assert torch.equal(u, u1) and torch.equal(v, v1)
    finally:
        eng.close()


def test_engine_advances_the_steps_asked_for(ctxs):
    # stages of few steps, so that resident chunks end early: one call of as many steps as the solve
    # takes (and the rest of a chunk) still ends it; the next call reads that chunk back
    n = 200
    desc = M.dense_cost(torch.rand(n, n, device="cuda", dtype=torch.float32))
    r, c = dev(W.dirichlet_marginal(n, 1)), dev(W.dirichlet_marginal(n, 2))
    prm = M.default_params()
    u, v = torch.empty_like(r), torch.empty_like(c)
    a = ctxs[0].solve(desc, r, c, 1e-2, prm, u, v)
    eng = M.Context(0)
    try:
        t = eng.submit(desc, r, c, 1e-2, prm, u, v)
        eng.run(a.sweeps + a.cert_sweeps + 32)
        eng.run(1)
        assert eng.poll(t) is not None
    finally:
        eng.close()
