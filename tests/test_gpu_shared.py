"""Solves, engine solves and sweeps beside a stream that keeps the compute units busy, so that resident
kernels cannot start now and then: the same bits as alone."""
from __future__ import annotations

import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2307_08507_amd import mdot as M  # noqa: E402
from paper_2307_08507_amd import workloads as W  # noqa: E402


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


@pytest.mark.parametrize("n", [1500, 4096])
def test_beside_a_busy_stream(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    C = torch.rand(n, n, device="cuda", dtype=torch.float32, generator=torch.Generator("cuda").manual_seed(n))
    desc = M.dense_cost(C)
    r, c = dev(W.dirichlet_marginal(n, 1)), dev(W.dirichlet_marginal(n, 2))
    prms = [M.default_params(gamma_f=128.0), M.default_params(max_sweeps=300)]
    own, other = torch.cuda.Stream(), torch.cuda.Stream()
    X = torch.rand(4096, 32768, device="cuda")
    Y = torch.empty_like(X)
    torch.cuda.synchronize()
    ctx = M.Context(0, stream=own)

    def passes():
        out = []
        for prm in prms:
            for engine in (False, True):
                u, v = torch.empty_like(r), torch.empty_like(c)
                if engine:
                    res = ctx.poll(ctx.submit(desc, r, c, 1e-4, prm, u, v), wait=True)
                else:
                    res = ctx.solve(desc, r, c, 1e-4, prm, u, v)
                own.synchronize()
                out.append((res.sweeps, res.primal_cost, res.dual_bound, u.cpu().numpy(), v.cpu().numpy()))
        lr, lc = torch.empty_like(r), torch.empty_like(c)
        ctx.lse2(desc, dev(out[0][3]), dev(out[0][4]), 128.0, lr, lc)
        own.synchronize()
        return out + [(lr.cpu().numpy(), lc.cpu().numpy())]

    stop = threading.Event()

    def feed():
        with torch.cuda.stream(other):
            while not stop.is_set():
                for _ in range(4):
                    torch.cumsum(X, 1, out=Y)
                other.synchronize()

    t = threading.Thread(target=feed)
    try:
        print(f"shared n={n} alone", flush=True)
        alone = passes()
        t.start()
        for k in range(3):
            print(f"shared n={n} pass {k}", flush=True)
            for a, b in zip(alone, passes()):
                for x, y in zip(a, b):
                    assert np.array_equal(x, y)
    finally:
        stop.set()
        if t.ident:
            t.join()
        ctx.close()
