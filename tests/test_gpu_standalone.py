"""Standalone sweeps (mdot_lse2): the cost-range check that rides on their passes, and the wide
loads of rows that start on any element."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2307_08507_amd import mdot as M  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = M.Context(0)
    yield c
    c.close()


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


def _lse(ctx, desc, m, n, shift, prec="f32"):
    rng = np.random.default_rng(m + n)
    u, v = rng.standard_normal(m) * 0.3 - np.log(n), rng.standard_normal(n) * 0.3
    lr = torch.full((m,), 7.0, dtype=torch.float64, device="cuda")
    lc = torch.full((n,), 7.0, dtype=torch.float64, device="cuda")
    sh = dev(u) if shift else None
    try:
        rc = ctx.lse2(desc, dev(u), dev(v), 20.0, lr, lc, shift=sh, precision=prec)
    except M.MdotError as e:
        rc = e.code
    return rc, lr.cpu().numpy(), lc.cpu().numpy(), u, v


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("shift", [False, True])
@pytest.mark.parametrize("bad", [1.5, -0.25, float("nan"), float("inf")])
def test_dense_range_is_checked_in_every_entry(ctx, dtype, shift, bad):
    m, n = 130, 261
    C = torch.rand(m, n, device="cuda", dtype=torch.float64).to(dtype)
    for i, j in ((0, 0), (m - 1, n - 1), (77, 259)):
        D = C.clone()
        D[i, j] = bad
        print(f"range {dtype} shift={shift} bad={bad} at {i},{j}", flush=True)
        rc, lr, lc, _, _ = _lse(ctx, M.dense_cost(D), m, n, shift)
        assert rc == -3
        assert (lr == 7.0).all() and (lc == 7.0).all()  # outputs untouched
    rc, lr, lc, _, _ = _lse(ctx, M.dense_cost(C), m, n, shift)
    assert rc == 0 and not (lr == 7.0).any()


@pytest.mark.parametrize("kind", ["sqeuclid", "l1"])
@pytest.mark.parametrize("d", [1, 3, 8])
def test_point_range_with_loose_boxes(ctx, kind, d):
    # Clouds whose boxes do not bound the distance by 1, so that the exact pass decides: accepted
    # at 1 / max, refused just above; and a box that settles it.
    m, n = 100, 70
    rng = np.random.default_rng(d)
    X, Y = rng.standard_normal((m, d)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
    t = X[:, None].astype(np.float64) - Y[None]
    raw = (t * t).sum(-1) if kind == "sqeuclid" else np.abs(t).sum(-1)
    XY = dev(np.concatenate([X.ravel(), Y.ravel()]), torch.float32)
    for shift in (False, True):
        for scale, want in ((1.0 / raw.max(), 0), (1.001 / raw.max(), -3), (0.1 / raw.max(), 0)):
            print(f"points {kind} d={d} shift={shift} scale={scale}", flush=True)
            rc, lr, lc, u, v = _lse(ctx, M.point_cost(XY, n, d, kind, scale=scale, m=m), m, n, shift, "f64")
            assert rc == want
            if want == 0:  # FP64 throughout, the sums in another order: a few ulp of the log-sums
                lr_o, lc_o = O.lse2(raw * scale, u, v, 20.0)
                np.testing.assert_allclose(lr, lr_o, rtol=0, atol=1e-11)
                np.testing.assert_allclose(lc, lc_o, rtol=0, atol=1e-11)
            else:
                assert (lr == 7.0).all() and (lc == 7.0).all()
    bad = XY.clone()
    bad[-1] = float("nan")
    assert _lse(ctx, M.point_cost(bad, n, d, kind, scale=0.01, m=m), m, n, True)[0] == -3


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("m,n", [(1, 1), (3, 5), (64, 256), (65, 257), (130, 131), (67, 514), (200, 1023)])
@pytest.mark.parametrize("offset", [0, 1])
def test_rows_starting_on_any_element(ctx, dtype, m, n, offset):
    # FP32 exponentials of FP64 arguments: |d log-sum| <= 2e-6, as in the parity tests
    flat = torch.rand(m * n + 1, device="cuda", dtype=torch.float64).to(dtype)
    C = flat[offset: offset + m * n].view(m, n)
    print(f"rows {dtype} {m}x{n} offset={offset}", flush=True)
    for shift in (False, True):
        rc, lr, lc, u, v = _lse(ctx, M.dense_cost(C), m, n, shift)
        lr_o, lc_o = O.lse2(C.double().cpu().numpy(), u, v, 20.0)
        assert rc == 0
        np.testing.assert_allclose(lr, lr_o, rtol=0, atol=2e-6)
        np.testing.assert_allclose(lc, lc_o, rtol=0, atol=2e-6)


# one kernel for the whole call up to two tiles per workgroup (more finalize blocks than tile
# workgroups among the sizes), several kernels beyond, against FP64 torch.
# F64: FP64 throughout, sums in another order: |d log-sum| <= 1e-11. F32: 2e-6 as in the parity tests.
@pytest.mark.parametrize("m,n", [(64, 64), (70, 4000), (2048, 2048), (2100, 2049), (2880, 3000), (4096, 4096), (8192, 1000)])
@pytest.mark.parametrize("dtype,prec", [(torch.float64, "f64"), (torch.float32, "f64"), (torch.float32, "f32"),
                                        (torch.float16, "f32")])
@pytest.mark.parametrize("shift", [False, True])
def test_layouts_of_the_resident_sweep(ctx, m, n, dtype, prec, shift):
    print(f"layout {m}x{n} {dtype} {prec} shift={shift}", flush=True)
    C = torch.rand(m, n, device="cuda", dtype=torch.float64).to(dtype)
    rc, lr, lc, u, v = _lse(ctx, M.dense_cost(C), m, n, shift, prec)
    X = dev(u)[:, None] + dev(v)[None, :] - 20.0 * C.double()
    assert rc == 0
    tol = 1e-11 if prec == "f64" else 2e-6
    np.testing.assert_allclose(lr, torch.logsumexp(X, 1).cpu().numpy(), rtol=0, atol=tol)
    np.testing.assert_allclose(lc, torch.logsumexp(X, 0).cpu().numpy(), rtol=0, atol=tol)


@pytest.mark.parametrize("n", [200, 2200, 4000])
def test_fp32_range_is_retried_in_fp64(ctx, n):
    # predictions 60 nats (86 binary orders) below the row sums: the FP32 sums overflow their range
    # and the call runs the sweep again with FP64 exponentials
    C = torch.rand(n, n, device="cuda", dtype=torch.float32)
    rng = np.random.default_rng(n)
    u, v = rng.standard_normal(n) * 0.3 - np.log(n), rng.standard_normal(n) * 0.3
    X = dev(u)[:, None] + dev(v)[None, :] - 20.0 * C.double()
    want = torch.logsumexp(X, 1)
    lr, lc = torch.empty_like(want), torch.empty_like(want)
    print(f"retry n={n}", flush=True)
    assert ctx.lse2(M.dense_cost(C), dev(u), dev(v), 20.0, lr, lc, shift=want - 60.0) == 0
    np.testing.assert_allclose(lr.cpu().numpy(), want.cpu().numpy(), rtol=0, atol=1e-11)
    np.testing.assert_allclose(lc.cpu().numpy(), torch.logsumexp(X, 0).cpu().numpy(), rtol=0, atol=1e-11)


def test_scale_chosen_by_the_library(ctx):
    for n, d in ((300, 2), (2300, 3)):
        rng = np.random.default_rng(d)
        X, Y = rng.standard_normal((n, d)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
        XY = dev(np.concatenate([X.ravel(), Y.ravel()]), torch.float32)
        a, b = dev(X)[:, None], dev(Y)[None]
        raw = ((a - b) ** 2).sum(-1)
        for shift in (False, True):
            print(f"chosen scale n={n} d={d} shift={shift}", flush=True)
            rc, lr, lc, u, v = _lse(ctx, M.point_cost(XY, n, d, "sqeuclid"), n, n, shift, "f64")
            X2 = dev(u)[:, None] + dev(v)[None, :] - 20.0 * raw / raw.max()
            assert rc == 0
            np.testing.assert_allclose(lr, torch.logsumexp(X2, 1).cpu().numpy(), rtol=0, atol=1e-11)
            np.testing.assert_allclose(lc, torch.logsumexp(X2, 0).cpu().numpy(), rtol=0, atol=1e-11)
