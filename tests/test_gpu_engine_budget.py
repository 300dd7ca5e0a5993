"""The exchange memory of the engine's resident chunks and the HBM budget: it is held only where the
budget has room, and given back before a request is refused."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2307_08507_amd import mdot as M  # noqa: E402
from paper_2307_08507_amd import workloads as W  # noqa: E402

EXCHANGE = 7_000_000  # at least


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


def _request(n, seed):
    C = torch.rand(n, n, device="cuda", dtype=torch.float32, generator=torch.Generator("cuda").manual_seed(seed))
    r, c = dev(W.dirichlet_marginal(n, seed)), dev(W.dirichlet_marginal(n, seed + 50))
    return M.dense_cost(C), r, c, torch.empty_like(r), torch.empty_like(c)


def _footprint(n):
    with_one = M.Context(0)
    try:
        q = _request(n, 1)
        with_one.submit(q[0], q[1], q[2], 1e-3, M.default_params(), q[3], q[4])
        return with_one.inflight()[1]
    finally:
        with_one.close()


# the exchange memory never fits, or only beside the first request
@pytest.mark.parametrize("n,room", [(300, 0), (3000, 8_200_000)])
def test_budget_bounds_the_exchange_memory(n, room):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    one = _footprint(n)
    budget = one + room if room else 2 * one
    assert 2 * one <= budget < 2 * one + EXCHANGE
    prm = M.default_params(gamma_f=128.0)
    reqs = [_request(n, k) for k in (1, 2)]
    alone = M.Context(0)
    eng = M.Context(0, hbm_budget_bytes=budget)
    try:
        want = []
        for q in reqs:
            res = alone.solve(q[0], q[1], q[2], 1e-3, prm, q[3], q[4])
            want.append((res.sweeps, res.primal_cost, q[3].cpu().numpy(), q[4].cpu().numpy()))
        print(f"budget n={n} one={one} budget={budget}", flush=True)
        ts = [eng.submit(reqs[0][0], reqs[0][1], reqs[0][2], 1e-3, prm, reqs[0][3], reqs[0][4])]
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        eng.run(16)
        torch.cuda.synchronize()
        grown = free - torch.cuda.mem_get_info()[0]
        print(f"grown by {grown}", flush=True)
        if not room:
            assert grown < EXCHANGE
        ts.append(eng.submit(reqs[1][0], reqs[1][1], reqs[1][2], 1e-3, prm, reqs[1][3], reqs[1][4]))
        assert ts[1] is not None  # two fit the budget
        for t, q, w in zip(ts, reqs, want):
            res = eng.poll(t, wait=True)
            torch.cuda.synchronize()
            assert (res.sweeps, res.primal_cost) == w[:2]
            assert np.array_equal(q[3].cpu().numpy(), w[2]) and np.array_equal(q[4].cpu().numpy(), w[3])
        assert eng.inflight() == (0, 0)
    finally:
        alone.close()
        eng.close()
