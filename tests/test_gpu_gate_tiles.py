"""The gate for batches of many token tiles gives the bits of the one-tile kernel: the same
tokens in calls small enough to take that one.  And the choices of every gate kernel where its arg-max and its
grouping can go wrong."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import reference as R
from test_gpu_parity import hx, small_workload, test_stack_step_equals_the_primitive_call_sequence as step_equals_primitives  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,k,probs", [(4097, 1024, 128, 2, True), (4112, 256, 8, 3, False), (8193, 512, 64, 1, True),
                                           (9001, 768, 120, 2, False), (12295, 768, 16, 2, True), (16400, 1024, 72, 1, False),
                                           # pairs of tiles: the second missing, of one token, whole; one pair a workgroup and several
                                           (2049, 1024, 128, 2, True), (2064, 768, 64, 1, True), (2065, 512, 8, 2, True), (2080, 256, 128, 5, False),
                                           (8191, 768, 128, 2, True), (8225, 1024, 128, 2, True),
                                           # the last without pairs; the second of the last pair of one token, whole, missing, almost whole
                                           (3584, 1024, 128, 2, True), (3585, 1024, 128, 2, True), (3600, 768, 64, 1, True), (3601, 512, 8, 2, True), (3615, 256, 128, 5, False)])
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


@pytest.mark.parametrize("dtype,T,d,E,k", [
    ("bf16", 1, 128, 8, 8), ("bf16", 4, 128, 16, 9), ("bf16", 5, 128, 40, 40), ("bf16", 16, 512, 64, 5), ("bf16", 40, 2048, 128, 6),
    ("bf16", 20, 1024, 256, 7), ("bf16", 2081, 256, 128, 4), ("f32", 3, 64, 128, 6), ("f32", 300, 64, 32, 5), ("f32", 9, 64, 12, 12),
    ("f32", 2, 64, 256, 8),
])
def test_choices_among_equal_infinite_and_nan_logits(hx, dtype, T, d, E, k):  # noqa: F811
    """Tokens of zeros, so that the bias is every token's logits: ties, both zeros, the largest float, infinities and NaN."""
    H, B = hx
    print(f"gate choices: {dtype} T={T} d={d} E={E} k={k}", flush=True)
    ctx = B.Context(H.config_for(small_workload(dtype, T, d, 64 if dtype == "bf16" else 8, E, k)))
    x, wg = np.zeros((T, d), np.float32), (np.random.default_rng(E).standard_normal((d, E)) * 0.05).astype(np.float32)
    few = np.full(E, -np.inf, np.float32)            # fewer finite logits than choices: the rest by index
    few[[E // 2, E - 1]] = 1.0, 3.0e38
    mixed = np.tile(np.array([0.0, -0.0, 1.5, -np.inf, np.nan, 1.5, -2.0, -3.4e38], np.float32), E // 8 + 1)[:E]
    for bias in (few, mixed, np.full(E, -0.0, np.float32), np.full(E, -3.4e38, np.float32)):
        idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
        prob = torch.zeros((T, k), dtype=torch.float32, device="cuda")
        probs = torch.zeros((T, E), dtype=torch.float32, device="cuda")
        ctx.pregate_topk(H.to_device(x, dtype), H.to_device(wg, dtype), torch.from_numpy(bias).cuda(), T, idx, prob, probs)
        torch.cuda.synchronize()
        o = R.gate(x[:1], wg, bias, k)
        assert np.array_equal(idx.cpu().numpy(), np.tile(o["idx"], (T, 1)))
        # float32 exponentials and a sum of E of them: E * 2^-24 of relative error at the most
        np.testing.assert_allclose(probs.cpu().numpy(), np.tile(o["p"], (T, 1)), rtol=E * 2.0 ** -24 + 1e-6)
        np.testing.assert_allclose(prob.cpu().numpy(), np.tile(o["prob"], (T, 1)), rtol=E * 2.0 ** -24 + 1e-6)
        assert ctx.device_flags() == (1 if np.isnan(bias).any() else 0)
    ctx.close()


@pytest.mark.parametrize("T,E,k", [(16, 128, 4), (13, 128, 5), (9, 256, 7), (4, 16, 16), (3, 8, 8), (16, 8, 1), (1, 256, 1), (15, 72, 4)])
def test_gates_that_group_at_the_size_of_a_wavefront(hx, T, E, k):  # noqa: F811
    """63, 64 and 65 selections, experts in one to four groups of 64: the grouping inside the gate against the grouping kernel."""
    print(f"gate groups: T={T} E={E} k={k}", flush=True)
    step_equals_primitives(hx, "bf16", T, 128, 256, E, k, 2, False)
