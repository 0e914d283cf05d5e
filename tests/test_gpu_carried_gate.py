"""A pre-gate carried in two halves (by the expert launch and the combine of the block before) gives
the bits of the separate gate launch: whole stack steps against the primitives called one by one, at
the edges of its token tiles, of the planes the reduction is cut into and of what it serves."""
import pytest
import torch

import workloads as W
from launch_count import kernel_launches
from test_gpu_parity import hx, test_stack_step_equals_the_primitive_call_sequence as step_equals_primitives  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,f,E,k,L", [
    (16, 256, 512, 64, 1, 4), (17, 128, 256, 32, 2, 3), (128, 256, 512, 64, 2, 3), (129, 128, 512, 64, 2, 3),
    (5, 768, 3072, 8, 1, 3),       # the decode-sized expert kernel
    (2, 1024, 4096, 24, 1, 3),
    (33, 64, 128, 8, 3, 3),        # fewer k-tiles than planes
    (100, 2048, 256, 16, 1, 3), (8, 128, 256, 128, 1, 3),
    (16, 128, 256, 128, 16, 2), (16, 128, 256, 128, 17, 2),   # as many selections as a gate groups by itself, and one more
    (9, 128, 256, 136, 1, 3), (9, 128, 256, 12, 1, 3),        # more experts than one pass serves; no multiple of eight
])
def test_step_with_a_carried_gate_equals_the_primitives(hx, T, d, f, E, k, L):  # noqa: F811
    print(f"carried gate: T={T} d={d} f={f} E={E} k={k} L={L}", flush=True)
    step_equals_primitives(hx, "bf16", T, d, f, E, k, L, False)


@pytest.mark.parametrize("T,d,f,E,k,L,carried", [
    (1, 768, 3072, 8, 1, 3, True), (3, 1024, 4096, 16, 1, 2, True),        # the smallest gates, whole in the decode-sized expert launch
    (5, 768, 3072, 8, 1, 3, True), (2, 1024, 4096, 24, 1, 3, True),        # in two halves, the first in the decode-sized launch
    (16, 256, 512, 64, 1, 4, True), (17, 128, 256, 32, 2, 3, True), (128, 256, 2048, 64, 2, 3, True),   # in the fused launch, 16-row chunks
    (100, 2048, 512, 16, 1, 3, True), (33, 64, 1024, 8, 3, 3, True),       # d_model at both ends: 64 k-tiles, and fewer than there are planes
    (60, 256, 2048, 8, 1, 3, True), (60, 768, 3072, 8, 1, 2, True), (112, 1024, 1024, 16, 1, 2, True),  # 32-row chunks
    (4, 1024, 4096, 16, 1, 2, False),                                      # a smallest gate, but no decode-sized launch
    (33, 64, 128, 8, 3, 3, False),                                         # no partial sums, so no combine that could finish it
    (129, 128, 2048, 64, 2, 3, False), (9, 128, 256, 136, 1, 3, False), (9, 128, 256, 12, 1, 3, False),  # tokens, experts, odd experts
])
def test_a_carried_gate_costs_no_launch(hx, T, d, f, E, k, L, carried):  # noqa: F811
    """The launches of a captured step say whether the gates were carried; the results are the primitives' either way."""
    H, B = hx
    print(f"carried gate, launches: T={T} d={d} f={f} E={E} k={k} L={L}", flush=True)
    w = W.Workload("carried_count", 81, L, d, f, E, k, T, 1, "bf16", 0.0, False)
    stack = H.Stack(w, H.ExpertStore(w, H.config_for(w), threads=4))
    assert "gemm" not in stack.ctx.ffn_kernel_name(T * k)
    stack.set_input(W.step_input(w, 0))
    stack.step()                                                   # not captured first: the kernels are loaded
    torch.cuda.synchronize()
    groups_itself = E % 8 == 0 and T <= 16 and T * k <= 256        # a gate of one workgroup also groups the tokens
    own_gates = 1 if carried else L                                # block 0's gate is always a launch
    assert kernel_launches(stack.step, stack.compute) == 2 * L + own_gates + (0 if groups_itself else L)
    stack.close()
    step_equals_primitives(hx, "bf16", T, d, f, E, k, L, False)
