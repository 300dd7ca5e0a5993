"""Sweeps of potentials and shifts that hold a NaN, by each of its bit patterns that the kernels use
themselves: the empty mark of their exchange slots (a quiet NaN, the signalling one it comes from, and
both signs) gives what any other NaN gives, at once."""
from __future__ import annotations

import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2307_08507_amd import mdot as M  # noqa: E402

EMPTY = 0x7FF8DEAD0000BEEF  # kEmpty of mdot_kernels.hip
MARKS = [EMPTY, EMPTY ^ (1 << 51), EMPTY | (1 << 63), (EMPTY ^ (1 << 51)) | (1 << 63)]


@pytest.mark.parametrize("m,n", [(200, 300), (1000, 1100), (3500, 3300)])
@pytest.mark.parametrize("where", ["u", "v", "shift"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_marked_nans_are_nans(m, n, where, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(m)
    C = torch.rand(m, n, device="cuda", dtype=dtype)
    base = {"u": rng.standard_normal(m) * 0.3 - np.log(n), "v": rng.standard_normal(n) * 0.3}
    base["shift"] = base["u"].copy()
    desc = M.dense_cost(C)
    ctx = M.Context(0)
    try:
        for given in (where == "shift", True):
            outs = []
            for bits in [0x7FF8000000000000] + MARKS:
                x = {k: a.copy() for k, a in base.items()}
                x[where].view(np.uint64)[x[where].size // 2] = bits
                d = {k: torch.as_tensor(a).to("cuda") for k, a in x.items()}
                lr = torch.empty(m, dtype=torch.float64, device="cuda")
                lc = torch.empty(n, dtype=torch.float64, device="cuda")
                torch.cuda.synchronize()
                print(f"nan {bits:x} in {where} of {m}x{n} {dtype} shift={given}", flush=True)
                t = time.monotonic()
                rc = ctx.lse2(desc, d["u"], d["v"], 20.0, lr, lc, shift=d["shift"] if given else None,
                              precision="f64" if dtype == torch.float64 else "f32")
                assert time.monotonic() - t < 2.0
                outs.append((rc, lr.cpu().numpy(), lc.cpu().numpy()))
            for o in outs[1:]:
                assert o[0] == outs[0][0]
                assert np.array_equal(o[1], outs[0][1], equal_nan=True)
                assert np.array_equal(o[2], outs[0][2], equal_nan=True)
    finally:
        ctx.close()


@pytest.mark.parametrize("n", [64, 300, 1100])
def test_a_cost_of_marked_nans_is_refused(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = M.Context(0)
    try:
        for bits in MARKS:
            C = torch.as_tensor(np.full((n, n), bits, dtype=np.uint64).view(np.float64)).to("cuda")
            z = torch.zeros(n, dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()
            print(f"nan cost {bits:x} n={n}", flush=True)
            t = time.monotonic()
            with pytest.raises(M.MdotError) as e:
                ctx.lse2(M.dense_cost(C), z, z, 20.0, z.clone(), z.clone(), precision="f64")
            assert e.value.code == -3 and time.monotonic() - t < 2.0
    finally:
        ctx.close()
