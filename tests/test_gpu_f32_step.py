"""Float32 stack steps whose gate launch groups the tokens and whose second expert kernel does the
combine: the bits of the primitives called one by one, at the edges of what those launches take."""
import pytest
import torch

import workloads as W
from launch_count import kernel_launches
from test_gpu_decode_stack import lanes_in_flight, options_hold
from test_gpu_parity import hx, test_stack_step_equals_the_primitive_call_sequence as step_equals_primitives  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,f,E,k,L,offloaded", [
    (1, 64, 256, 8, 1, 2, False), (64, 64, 256, 8, 1, 3, False), (65, 128, 256, 16, 1, 2, False),
    (256, 64, 128, 64, 2, 2, False),                 # as many tokens and selections as a gate groups
    (257, 64, 128, 64, 1, 2, False), (171, 64, 128, 8, 3, 2, False),    # a token, a selection more
    (100, 128, 256, 256, 1, 1, False), (33, 64, 256, 8, 8, 2, False), (20, 64, 256, 12, 1, 2, False),   # every expert; no power of two
    (50, 68, 132, 8, 1, 2, False), (40, 30, 36, 8, 1, 2, False),        # columns past a tile's end; rows that are no multiple of 16 bytes
    (90, 256, 512, 8, 1, 2, False), (200, 512, 512, 8, 1, 1, False),    # 32- and 64-row chunks
    (9, 64, 256, 8, 1, 3, True), (30, 64, 256, 8, 2, 3, True),
])
def test_f32_step_equals_the_primitives(hx, T, d, f, E, k, L, offloaded):  # noqa: F811
    print(f"f32 step: T={T} d={d} f={f} E={E} k={k} L={L} offloaded={offloaded}", flush=True)
    step_equals_primitives(hx, "f32", T, d, f, E, k, L, offloaded)


@pytest.mark.parametrize("T,k,launches", [(32, 1, 5), (32, 2, 7), (300, 1, 8)])
def test_f32_step_replayed_from_a_graph(hx, T, k, launches):  # noqa: F811
    """Replays on new inputs, with eager steps in between: what a gate launch counts has to be zero again behind it."""
    H, B = hx
    w = W.Workload("f32_replay", 83, 2, 64, 256, 8, k, T, 1, "f32", 0.0, False)
    stack = H.Stack(w, H.ExpertStore(w, H.config_for(w), threads=2))
    stack.set_input(W.step_input(w, 0))
    stack.step()
    torch.cuda.synchronize()
    assert kernel_launches(stack.step, stack.compute) == launches
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stack.compute):
        stack.step()
    other = H.Stack(w, stack.store)
    out = lambda s: (s.x_states, s.y_blocks, s.topk_idx, s.topk_prob, s.row_of, s.expert_offsets)  # noqa: E731
    for n in range(4):
        for m, step in ((n, graph.replay), (n + 10, stack.step)):
            for t in out(stack):
                t.zero_()
            stack.set_input(W.step_input(w, m))
            step()
            other.set_input(W.step_input(w, m))
            other.step()
            torch.cuda.synchronize()
            for a, b in zip(out(stack), out(other)):
                assert torch.equal(a, b)
    other.close()
    stack.close()


@pytest.mark.parametrize("E,k,L,contexts", [(8, 1, 3, 1), (8, 2, 2, 1), (64, 1, 1, 1), (8, 1, 2, 3)])
def test_one_token_f32_steps_in_flight_together(hx, E, k, L, contexts):  # noqa: F811
    """Steps on streams of their own, each with its own buffers: no gate takes another's workgroup for its own."""
    H, B = hx
    print(f"f32 steps in flight: E={E} k={k} L={L} contexts={contexts}", flush=True)
    stacks, lanes, alone = lanes_in_flight(H, W.Workload("f32_lanes", 85, L, 64, 256, E, k, 1, 1, "f32", 1.1, False), contexts)
    for s in [*stacks, alone]:
        s.close()


def test_f32_batches_of_changing_size_in_one_context(hx):  # noqa: F811
    """Each batch size's gates count for themselves."""
    H, B = hx
    w = W.Workload("f32_sizes", 86, 2, 64, 256, 8, 1, 256, 1, "f32", 0.0, False)
    roomy = H.Stack(w, H.ExpertStore(w, H.config_for(w), threads=2))
    for T in (256, 1, 33, 256, 2, 33, 1):
        tight = H.Stack(w.replace(tokens=T), roomy.store)
        x0 = W.step_input(w, T)[:T]
        tight.set_input(x0)
        tight.step()
        roomy.x_states.reshape(-1)[: T * 64].copy_(tight.x_states[0].reshape(-1))
        torch.cuda.synchronize()
        for _ in range(2):
            roomy.step(T=T)
            torch.cuda.synchronize()
            assert torch.equal(roomy.x_states.reshape(-1)[: 3 * T * 64], tight.x_states.reshape(-1)), T
            assert torch.equal(roomy.row_of.reshape(-1)[: 2 * T], tight.row_of.reshape(-1)), T
        tight.close()
    roomy.close()


@pytest.mark.parametrize("T,k,E,L", [(32, 1, 8, 3), (9, 2, 16, 2), (1, 1, 8, 2)])
def test_f32_step_with_biases_without_outputs_and_with_nan(hx, T, k, E, L):  # noqa: F811
    """Against the primitives called one by one."""
    H, B = hx
    print(f"f32 options: T={T} k={k} E={E} L={L}", flush=True)

    def primitives(s):
        ctx, nk = s.ctx, T * k
        for i in range(L):
            for g in ([0, 1] if i == 0 else [i + 1]):
                if g < L:
                    ctx.pregate_topk(s.x_states[i], s.gate_w[g], s.gate_b[g], T, s.topk_idx[g], s.topk_prob[g], None, s.compute)
            ctx.permute(s.x_states[i], s.topk_idx[i], T, s.x_perm, s.row_of[i], s.expert_offsets[i], s.compute)
            ctx.expert_ffn(i, s.x_perm, s.expert_offsets[i], nk, s.y_perm, s.workspace, s.compute)
            ctx.combine(s.y_perm, s.row_of[i], s.topk_prob[i], T, s.y_blocks[i], s.x_states[i], s.x_states[i + 1], s.compute)

    options_hold(H, B, W.Workload("f32_options", 88, L, 64, 256, E, k, T, 1, "f32", 1.1, False), primitives)
