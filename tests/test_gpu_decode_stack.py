"""The two-launch step of one token (batch-1 decode, experts resident) against the primitives called
one by one, bit for bit: numbers of blocks, widths, experts and sub-slabs at the edges of what it
takes, steps one after the other, several in flight, replayed from graphs, and the steps it leaves to launches."""
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
    print(f"two-launch step: T={T} d={d} f={f} E={E} k={k} L={L}", flush=True)
    w, stack = stack_of(H, T, d, f, E, k, L)
    stack.set_input(W.step_input(w, 0))
    stack.step()
    torch.cuda.synchronize()
    assert (kernel_launches(stack.step, stack.compute) == 2) == one  # block 0's gate with the clearing, the rest
    stack.close()
    step_equals_primitives(hx, "bf16", T, d, f, E, k, L, False)


def test_one_token_steps_follow_each_other_and_replay(hx):  # noqa: F811
    """Many steps of different inputs in a row, queued without a wait, then replays with eager steps on another input in between, each
    the same as in a context of its own; no wait has run out."""
    H, B = hx
    w, stack = stack_of(H, 1, 768, 3072, 8, 1, 6)
    other = H.Stack(w, stack.store)
    keep = lambda s: [t.clone() for t in (s.x_states, s.y_blocks, s.topk_idx, s.topk_prob, s.row_of, s.expert_offsets)]  # noqa: E731
    row = Lane(stack, 40, 0)
    for n in range(40):
        row.step(n)
    torch.cuda.synchronize()
    check_lanes([row], other)
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
        for m, step in ((n, graph.replay), ((n + 1) % 4, stack.step)):
            for t in (stack.x_states, stack.y_blocks, stack.topk_idx, stack.topk_prob, stack.row_of, stack.expert_offsets):
                t.zero_()
            stack.set_input(W.step_input(w, m))
            step()
            torch.cuda.synchronize()
            for a, b in zip(keep(stack), want[m]):
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


class Lane:
    """A stream of its own and `n` one-token steps with inputs, outputs and (shared by the lane's steps) scratch of their own."""

    def __init__(self, stack, n, first):
        self.stack, self.stream, w, k = stack, torch.cuda.Stream(), stack.w, stack.w.top_k
        new = lambda like, *shape: torch.zeros((n, *shape), dtype=like.dtype, device="cuda")  # noqa: E731
        L, d, E = w.n_blocks, w.d_model, w.n_experts
        self.out = (new(stack.x_states, L + 1, 1, d), new(stack.y_blocks, L, 1, d), new(stack.topk_idx, L, 1, k), new(stack.topk_prob, L, 1, k),
                    new(stack.row_of, L, k), new(stack.expert_offsets, L, E + 1))
        for i in range(n):
            self.out[0][i, 0] = stack_input(w, first + i)
        # what a step finds in its workspace is anybody's: here words that look like tags and counts of block 1; some behind its end
        self.workspace = torch.full((stack.ctx.workspace_bytes // 4 + 256,), 1, dtype=torch.int32, device="cuda")
        perm = torch.zeros((2, k, d), dtype=stack.x_states.dtype, device="cuda")
        self.bufs = [stack.ctx.make_step_buffers(stack.gate_w, stack.gate_b, *(t[i] for t in self.out), perm[0], perm[1], self.workspace) for i in range(n)]
        torch.cuda.synchronize()

    def step(self, i):
        self.stack.ctx.stack_step(self.bufs[i], 1, self.stream, self.stack.copy)

    def clear(self):
        self.out[0][:, 1:].zero_()
        for t in self.out[1:]:
            t.zero_()
        torch.cuda.synchronize()


def stack_input(w, n):
    t = torch.from_numpy(W.step_input(w, n)).cuda()
    return t if w.dtype == "f32" else t.bfloat16()


def check_lanes(lanes, one_by_one):
    """Every step of every lane, bit for bit, against the same step in a context that has nothing else in flight."""
    for a, lane in enumerate(lanes):
        n = len(lane.bufs)
        assert bool((lane.workspace[-256:] == 1).all())
        alone = Lane(one_by_one, n, 0)
        alone.out[0].copy_(lane.out[0])
        alone.clear()
        for i in range(n):
            alone.step(i)
            torch.cuda.synchronize()
        for got, want in zip(lane.out, alone.out):
            for i in range(n):
                assert torch.equal(got[i], want[i]), f"lane {a}, step {i} of {n}"


def lanes_in_flight(H, w, contexts, steps=16, lanes=3):
    """Lanes dealt to `contexts` contexts, all their steps queued in turn without a wait, three times over."""
    store = H.ExpertStore(w, H.config_for(w), threads=4)
    stacks = [H.Stack(w, store) for _ in range(contexts)]
    lanes = [Lane(stacks[a % contexts], steps, 100 * a) for a in range(lanes)]
    alone = H.Stack(w, store)
    alone.ctx.ffn_timing_begin(1)  # keeps the bf16 step to its separate launches
    for _ in range(3):
        for lane in lanes:
            lane.clear()
        for i in range(steps):
            for lane in lanes:
                lane.step(i)
        torch.cuda.synchronize()
        check_lanes(lanes, alone)
    assert all(s.ctx.device_flags() == 0 for s in stacks)
    alone.ctx.ffn_timing_end()
    return stacks, lanes, alone


@pytest.mark.parametrize("contexts", [1, 3])
@pytest.mark.parametrize("d,f,E,L", [(768, 3072, 8, 6), (1024, 512, 16, 4)])
def test_one_token_steps_in_flight_together(hx, d, f, E, L, contexts):  # noqa: F811
    """Steps on streams of their own, of one context or of several, each with its own buffers and input, have nothing in common."""
    H, B = hx
    print(f"steps in flight: d={d} f={f} E={E} L={L} contexts={contexts}", flush=True)
    stacks, lanes, alone = lanes_in_flight(H, W.Workload("decode_lanes", 84, L, d, f, E, 1, 1, 1, "bf16", 1.1, False), contexts)
    assert kernel_launches(lambda: lanes[0].step(0), lanes[0].stream) == 2
    for s in [*stacks, alone]:
        s.close()


def test_captured_one_token_steps_of_one_context_replay_together(hx):  # noqa: F811
    H, B = hx
    w = W.Workload("decode_lanes", 84, 6, 768, 3072, 8, 1, 1, 1, "bf16", 1.1, False)
    stack = H.Stack(w, H.ExpertStore(w, H.config_for(w), threads=4))
    alone = H.Stack(w, stack.store)
    alone.ctx.ffn_timing_begin(1)
    lanes = [Lane(stack, 4, 100 * a) for a in range(3)]
    graphs = []
    for lane in lanes:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=lane.stream):
            for i in range(4):
                lane.step(i)
        graphs.append(graph)
    eager = Lane(stack, 4, 900)
    for n in range(4):
        for a, lane in enumerate([*lanes, eager]):
            for i in range(4):
                lane.out[0][i, 0] = stack_input(w, 1000 * n + 100 * a + i)
            lane.clear()
        for graph, lane in zip(graphs, lanes):
            with torch.cuda.stream(lane.stream):
                graph.replay()
        for i in range(4):
            eager.step(i)
        torch.cuda.synchronize()
        check_lanes([*lanes, eager], alone)
    assert stack.ctx.device_flags() == 0
    alone.ctx.ffn_timing_end()
    stack.close()
    alone.close()


def same(a, b):
    """Equal, with NaN in the same places."""
    return torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(), b.nan_to_num())


def options_hold(H, B, w, reference):
    """A step without y_blocks, one whose gates see a NaN logit and one of a hidden state with a NaN: the values of the same step made by
    `reference(stack)`, another stack on the same experts that goes another way, and the NaN flag."""
    store = H.ExpertStore(w, H.config_for(w), threads=4)
    for bad_bias, bad_x in ((False, False), (True, False), (False, True)):
        gates = [(gw, gb.copy()) for gw, gb in W.gate_tensors(w)]
        assert not any((gates[0][1] == gb).all() for _, gb in gates[1:])  # every block's bias is another
        if bad_bias:
            for n, (_, gb) in enumerate(gates):
                gb[n % w.n_experts] = float("nan")
        x0 = W.step_input(w, 3)
        if bad_x:
            x0[-1, 5] = float("nan")
        got = []
        for other in (False, True):
            stack = H.Stack(w, store, gates=gates)
            x_in = torch.from_numpy(x0).cuda().to(stack.x_states.dtype)
            stack.x_states[0].copy_(x_in)
            torch.cuda.synchronize()
            (reference if other else H.Stack.step)(stack)
            torch.cuda.synchronize()
            got.append([t.clone() for t in (stack.x_states, stack.y_blocks, stack.topk_idx, stack.topk_prob, stack.row_of, stack.expert_offsets)])
            assert stack.ctx.device_flags() == (1 if bad_bias or bad_x else 0)
            if not other:  # again, without the blocks' outputs
                stack.x_states[1:].zero_()
                stack.y_blocks.zero_()
                bufs = stack.ctx.make_step_buffers(stack.gate_w, stack.gate_b, stack.x_states, None, stack.topk_idx, stack.topk_prob, stack.row_of,
                                                   stack.expert_offsets, stack.x_perm, stack.y_perm, stack.workspace)
                torch.cuda.synchronize()
                stack.ctx.stack_step(bufs, w.tokens, stack.compute, stack.copy)
                torch.cuda.synchronize()
                assert same(stack.x_states, got[0][0]) and not stack.y_blocks.any()
            stack.close()
        for a, b in zip(*got):
            assert same(a, b), (bad_bias, bad_x)
        assert bool(got[0][0].isnan().any()) == bad_x


@pytest.mark.parametrize("d,f,E,L", [(768, 320, 8, 5), (1024, 512, 16, 4)])
def test_one_token_step_with_biases_without_outputs_and_with_nan(hx, d, f, E, L):  # noqa: F811
    H, B = hx
    print(f"options: d={d} f={f} E={E} L={L}", flush=True)

    def launches(stack):
        stack.ctx.ffn_timing_begin(1)
        stack.step()

    options_hold(H, B, W.Workload("decode_options", 87, L, d, f, E, 1, 1, 1, "bf16", 1.1, False), launches)
