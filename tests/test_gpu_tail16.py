"""FP16 and BF16 costs that end in the middle of a dword: the two bytes behind the matrix are not the
library's, so nothing may depend on them. Every call gives the same bits and the same counts whatever
they hold."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2307_08507_amd import mdot as M  # noqa: E402
from paper_2307_08507_amd import workloads as W  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = M.Context(0)
    yield c
    c.close()


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


BEHIND = [0.0, float("nan"), float("inf"), float("-inf")]
# m, n, first element: odd counts at an aligned base and even ones that start in the upper half of a
# dword; in one tile, in the last of several, in a row shorter than a tile, and past the resident kernels
ENDS = [(1, 1, 0), (3, 5, 0), (63, 2, 1), (65, 257, 0), (64, 255, 1), (130, 66, 1), (2049, 2101, 0), (4161, 4097, 0)]
COUNTS = ("status", "primal_cost", "dual_bound", "gamma_final", "marg_err_l1", "grad_norm", "stages", "pncg_iters",
          "ls_trials", "sweeps", "fp64_retries", "cert_sweeps", "prec_switches", "proxy_stages")


def _costs(m, n, first, dtype):
    gen = torch.Generator("cuda").manual_seed(m * n)
    C = torch.rand(m * n, device="cuda", dtype=torch.float64, generator=gen).to(dtype)
    for x in BEHIND:
        flat = torch.full((first + m * n + 64,), x, device="cuda", dtype=dtype)
        flat[first: first + m * n] = C
        yield x, M.dense_cost(flat[first: first + m * n].view(m, n)), flat


def _report(res, u, v):
    assert np.isfinite([res.primal_cost, res.dual_bound]).all()
    return [getattr(res, f) for f in COUNTS], u.cpu().numpy(), v.cpu().numpy()


def _same(base, out, where):
    assert base[0] == out[0], where
    for a, b in zip(base[1:], out[1:]):
        assert np.array_equal(a, b), where
        assert np.isfinite(a).all(), where


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("m,n,first", ENDS)
def test_sweeps_and_certificates(ctx, dtype, m, n, first):
    rng = np.random.default_rng(m + n)
    u, v = dev(rng.standard_normal(m) * 0.3 - np.log(n)), dev(rng.standard_normal(n) * 0.3 - np.log(m))
    r, c = dev(W.dirichlet_marginal(m, 1)), dev(W.dirichlet_marginal(n, 2))
    base = {}
    for x, desc, _keep in _costs(m, n, first, dtype):
        for shift in (None, u):
            for prec in ("f32", "f64"):
                print(f"tail16 lse {dtype} {m}x{n}+{first} behind={x} shift={shift is not None} {prec}", flush=True)
                lr, lc = torch.empty_like(u), torch.empty_like(v)
                rc = ctx.lse2(desc, u, v, 8.0, lr, lc, shift=shift, precision=prec)
                out = ([rc], lr.cpu().numpy(), lc.cpu().numpy())
                _same(base.setdefault((shift is None, prec), out), out, (x, shift is None, prec))
        print(f"tail16 round {dtype} {m}x{n}+{first} behind={x}", flush=True)
        ub, lb, me = ctx.round_certify(desc, u, v, 8.0, r, c)
        out = ([], np.array([ub, lb, me]))
        _same(base.setdefault("round", out), out, x)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("m,n,first", [(3, 5, 0), (65, 257, 0), (130, 66, 1), (2049, 2101, 0)])
def test_solves(ctx, dtype, m, n, first):
    r, c = dev(W.dirichlet_marginal(m, 1)), dev(W.dirichlet_marginal(n, 2))
    prm = M.default_params(gamma_f=64.0 if n > 2000 else 0.0, max_sweeps=4000)
    base = None
    for x, desc, _keep in _costs(m, n, first, dtype):
        for engine in (False, True):
            print(f"tail16 solve {dtype} {m}x{n}+{first} behind={x} engine={engine}", flush=True)
            u, v = torch.empty_like(r), torch.empty_like(c)
            if engine:
                res = ctx.poll(ctx.submit(desc, r, c, 1e-2, prm, u, v), wait=True)
            else:
                res = ctx.solve(desc, r, c, 1e-2, prm, u, v)
            out = _report(res, u, v)
            base = base or out
            _same(base, out, (x, engine))
