"""The one-launch step of one token (batch-1 decode, experts resident) against the primitives called
one by one, bit for bit: numbers of blocks, widths, experts and sub-slabs at the edges of what it
takes, steps one after the other, replayed from a graph, and the steps it leaves to launches."""
import pytest
import torch

import workloads as W
from launch_count import kernel_launches
from test_gpu_parity import hx, test_stack_step_equals_the_primitive_call_sequence as step_equals_primitives  # noqa: F401

pytestmark = pytest.mark.gpu


def stack_of(H, T, d, f, E, k, L, max_tokens=None):
    w = W.Workload("decode_stack", 84, L, d, f, E, k, T, 1, "bf16", 0.0, False)
    stack = H.Stack(w, H.ExpertStore(w, H.config_for(w), threads=4), **({"max_tokens": max_tokens} if max_tokens else {}))
    return w, stack


@pytest.mark.parametrize("T,d,f,E,k,L,one", [
    (1, 768, 3072, 8, 1, 4, True), (1, 768, 3072, 16, 1, 7, True), (1, 1024, 4096, 8, 1, 5, True), (1, 1024, 512, 16, 1, 4, True),
    (1, 768, 320, 8, 1, 16, True),          # ten sub-slabs, the most blocks
    (1, 768, 256, 8, 1, 4, False),          # eight: the combine adds in another order
    (1, 768, 320, 8, 1, 17, False), (1, 768, 3072, 8, 1, 3, False), (2, 768, 3072, 8, 1, 4, False), (1, 768, 3072, 8, 2, 4, False),
    (1, 768, 3072, 32, 1, 4, False), (1, 512, 2048, 8, 1, 4, False),
])
def test_one_token_step(hx, T, d, f, E, k, L, one):  # noqa: F811
    H, B = hx
    print(f"one-launch step: T={T} d={d} f={f} E={E} k={k} L={L}", flush=True)
    w, stack = stack_of(H, T, d, f, E, k, L)
    stack.set_input(W.step_input(w, 0))
    stack.step()
    torch.cuda.synchronize()
    assert (kernel_launches(stack.step, stack.compute) == 1) == one
    stack.close()
    step_equals_primitives(hx, "bf16", T, d, f, E, k, L, False)


def test_one_token_steps_follow_each_other_and_replay(hx):  # noqa: F811
    """Tags and counts go on from step to step: many steps in a row, queued without a wait, then replays with eager
    steps in between, each the same as in a context of its own; no wait has run out."""
    H, B = hx
    w, stack = stack_of(H, 1, 768, 3072, 8, 1, 6)
    other = H.Stack(w, stack.store)
    keep = lambda s: [t.clone() for t in (s.x_states, s.y_blocks, s.topk_idx, s.topk_prob, s.row_of, s.expert_offsets)]  # noqa: E731
    for n in range(40):
        stack.set_input(W.step_input(w, n))
        for _ in range(3):
            stack.step()
    want = {}
    for n in range(4):
        other.set_input(W.step_input(w, n))
        other.step()
        torch.cuda.synchronize()
        want[n] = keep(other)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stack.compute):
        stack.step()
    for n in (0, 1, 2, 3, 1):
        stack.set_input(W.step_input(w, n))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(keep(stack), want[n]):
            assert torch.equal(a, b)
        stack.step()
        torch.cuda.synchronize()
        for a, b in zip(keep(stack), want[n]):
            assert torch.equal(a, b)
    assert stack.ctx.device_flags() == 0 and other.ctx.device_flags() == 0
    stack.close()
    other.close()


def test_one_token_step_in_a_context_for_more(hx):  # noqa: F811
    """max_tokens above one: the same arrays' first token; other batch sizes in between take their launches."""
    H, B = hx
    w, tight = stack_of(H, 1, 768, 3072, 8, 1, 4)
    tight.set_input(W.step_input(w, 0))
    tight.step()
    torch.cuda.synchronize()
    roomy = H.Stack(w, tight.store, max_tokens=8)
    for _ in range(2):
        roomy.x_states.reshape(-1)[:768].copy_(tight.x_states[0].reshape(-1))
        torch.cuda.synchronize()
        roomy.step(T=1)
        torch.cuda.synchronize()
        assert torch.equal(roomy.x_states.reshape(-1)[: 5 * 768], tight.x_states.reshape(-1))
        assert torch.equal(roomy.topk_idx.reshape(-1)[:4], tight.topk_idx.reshape(-1))
        roomy.step(T=3)
        torch.cuda.synchronize()
    roomy.close()
    tight.close()
