"""Token grouping by several workgroups and the wavefront-per-token combine, around the sizes where
they change over: exact integers against numpy, sums against the definition in 64 bits."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_parity import hx, nerr, small_workload  # noqa: F401  (hx is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k,mode", [
    (2048, 8, 1, "rand"), (2049, 8, 1, "rand"), (1025, 64, 2, "zipf"), (3072, 5, 1, "one"), (3073, 256, 1, "rand"),
    (20000, 256, 4, "zipf"), (70001, 7, 1, "rand"), (33000, 33, 3, "zipf"),
])
def test_grouping_by_several_workgroups_is_exact(hx, T, E, k, mode):  # noqa: F811
    H, B = hx
    print(f"grouping: T={T} E={E} k={k} {mode}", flush=True)
    d = 64
    ctx = B.Context(H.config_for(small_workload("bf16", T, d, 64, E, k)))
    g = np.random.default_rng(T + E)
    if mode == "one":
        idx = np.full((T, k), E - 1)
    elif mode == "zipf":
        idx = np.minimum(g.zipf(1.3, size=(T, k)) - 1, E - 1)
    else:
        idx = g.integers(0, E, size=(T, k))
    if mode == "rand":
        idx[T // 2, 0], idx[T - 1, 0] = -3, E + 9   # out of range: clamped and flagged
    x = torch.from_numpy(g.standard_normal((T, d)).astype(np.float32)).cuda().bfloat16()
    x_perm = torch.zeros((T * k, d), dtype=torch.bfloat16, device="cuda")
    row_of = torch.full((T * k,), -1, dtype=torch.int32, device="cuda")
    offs = torch.full((E + 1,), -1, dtype=torch.int32, device="cuda")
    ctx.device_flags()
    ctx.permute(x, torch.from_numpy(idx.astype(np.int32)).cuda(), T, x_perm, row_of, offs)
    torch.cuda.synchronize()
    e = np.clip(idx.ravel(), 0, E - 1)
    want = np.empty(T * k, np.int64)
    want[np.argsort(e, kind="stable")] = np.arange(T * k)
    assert np.array_equal(row_of.cpu().numpy(), want)
    assert np.array_equal(offs.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(e, minlength=E))]))
    assert torch.equal(x_perm[row_of.long()], x.repeat_interleave(k, dim=0))
    assert ctx.device_flags() == (2 if mode == "rand" else 0)
    ctx.close()


@pytest.mark.parametrize("dtype,T,d,k", [
    ("bf16", 1, 64, 1), ("bf16", 5, 512, 3), ("bf16", 1024, 768, 2), ("bf16", 1025, 768, 2), ("bf16", 1027, 2048, 1), ("bf16", 7, 1024, 2),
    ("f32", 3, 4, 2), ("f32", 1026, 260, 1), ("f32", 9, 1024, 2), ("f32", 2, 22, 2),
])
def test_combine_at_tile_edges(hx, dtype, T, d, k):  # noqa: F811
    H, B = hx
    ctx = B.Context(H.config_for(small_workload(dtype, T, d, 64, 8, k)))
    g = np.random.default_rng(T + d + k)
    yp, xr = (g.standard_normal(s).astype(np.float32) for s in ((T * k, d), (T, d)))
    if dtype == "bf16":
        yp, xr = W.round_to_bf16(yp), W.round_to_bf16(xr)
    row_of = g.permutation(T * k).astype(np.int32)
    prob = g.uniform(0.05, 1.0, size=(T, k)).astype(np.float32)
    want = (prob.astype(np.float64)[:, :, None] * yp.astype(np.float64)[row_of].reshape(T, k, d)).sum(1)
    guard = 7.0
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    y, xn = (torch.full((T + 1, d), guard, dtype=tdt, device="cuda") for _ in range(2))
    args = (H.to_device(yp, dtype), torch.from_numpy(row_of).cuda(), torch.from_numpy(prob).cuda(), T)
    ctx.combine(*args, y, H.to_device(xr, dtype), xn)
    torch.cuda.synchronize()
    tol = 2.0 ** -8 if dtype == "bf16" else 1e-6    # one rounding of the result
    assert nerr(H.to_numpy64(y)[:T], want) <= tol and nerr(H.to_numpy64(xn)[:T], xr + want) <= tol
    assert bool((y[T] == guard).all()) and bool((xn[T] == guard).all())
    only = torch.full((T, d), guard, dtype=tdt, device="cuda")
    ctx.combine(*args, only)
    torch.cuda.synchronize()
    assert torch.equal(only, y[:T])
    ctx.close()
