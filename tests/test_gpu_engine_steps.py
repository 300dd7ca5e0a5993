"""mdot_run advances resident solves by about the steps asked for: chunks that end early at a stage's
end are made up for, and no more."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2307_08507_amd import mdot as M  # noqa: E402
from paper_2307_08507_amd import workloads as W  # noqa: E402


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


@pytest.mark.parametrize("count", [1, 2, 6])
@pytest.mark.parametrize("steps", [64, 160])
def test_steps_of_a_call_are_bounded(count, steps):
    # A chunk is at most 32 steps, and no chunk is launched for a solve that has its steps (the one in
    # flight taken for 16): what a call reads back of a solve alone is less than `steps` and one chunk.
    # With others in flight, whose stages end at other times, less than twice that.
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    eng = M.Context(0)
    try:
        held, total = [], 0
        for k in range(count):
            n = 200 + 40 * k
            C = torch.rand(n, n, device="cuda", dtype=torch.float32, generator=torch.Generator("cuda").manual_seed(k))
            r, c = dev(W.dirichlet_marginal(n, k)), dev(W.dirichlet_marginal(n, k + 50))
            u, v = torch.empty_like(r), torch.empty_like(c)
            held.append((eng.submit(M.dense_cost(C), r, c, 1e-4, M.default_params(), u, v), C, r, c, u, v))
        calls = 0
        while eng.inflight()[0] and calls < 10000:
            eng.run(steps)
            calls += 1
        for h in held:
            res = eng.poll(h[0])
            total = max(total, res.sweeps + res.fp64_retries + res.cert_sweeps)
        print(f"engine steps: {count} solves, {total} steps in {calls} calls of {steps}", flush=True)
        assert total > 200
        assert total <= (steps + 32 if count == 1 else 2 * steps + 32) * calls + 32
        assert total >= (calls - 3) * steps  # and a call takes the steps asked for (the last ones collect)
    finally:
        eng.close()
