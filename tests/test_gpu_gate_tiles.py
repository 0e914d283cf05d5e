"""The gate for batches of several token tiles per CU gives the bits of the one-tile kernel: the same
tokens in calls small enough to take that one."""
import pytest
import torch

from test_gpu_parity import hx, small_workload  # noqa: F401  (hx is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,k,probs", [(4097, 1024, 128, 2, True), (4112, 256, 8, 3, False), (8193, 512, 64, 1, True),
                                           (9001, 768, 120, 2, False), (12295, 768, 16, 2, True), (16400, 1024, 72, 1, False)])
def test_many_tiles_give_the_bits_of_single_ones(hx, T, d, E, k, probs):  # noqa: F811
    H, B = hx
    print(f"gate tiles: T={T} d={d} E={E} k={k}", flush=True)
    ctx = B.Context(H.config_for(small_workload("bf16", T, d, 64, E, k)))
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn((T, d), generator=g, device="cuda").bfloat16()
    w = (torch.randn((d, E), generator=g, device="cuda") * 0.05).bfloat16()
    b = torch.randn(E, generator=g, device="cuda") * 0.3
    x[T - 1, 3] = float("nan")     # a NaN logit in the last tile: ranks last, raises the flag
    out = []
    for step in (T, 2048):
        idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
        prob = torch.zeros((T, k), dtype=torch.float32, device="cuda")
        full = torch.zeros((T, E), dtype=torch.float32, device="cuda") if probs else None
        for t in range(0, T, step):
            n = min(step, T - t)
            ctx.pregate_topk(x[t: t + n], w, b, n, idx[t: t + n], prob[t: t + n], full[t: t + n] if probs else None)
        torch.cuda.synchronize()
        assert ctx.device_flags() == 1
        out.append((idx, prob, full))
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32))
    assert not probs or torch.equal(out[0][2].view(torch.int32), out[1][2].view(torch.int32))
    ctx.close()
