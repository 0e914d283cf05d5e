"""The float32 expert FFN at the sizes where its tiles can go wrong: every column width and row-tile
count, reductions and column counts that are no multiple of a tile, shapes that cannot be read 16
bytes at a time, experts without rows, and the stack step that reads its rows through the map."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import reference as R
from launch_count import kernel_nodes
from test_gpu_parity import TOL, hx, nerr, run_ffn_case  # noqa: F401  (hx is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f,E,counts", [
    (64, 256, 8, [1, 0, 2, 16, 17, 0, 5, 3]),
    (68, 132, 3, [4, 31, 0]),                       # neither the reduction nor the columns fill their last tile
    (4, 4, 2, [3, 1]),
    (12, 20, 4, [40, 20, 64, 65]),                  # 64-row chunks
    (256, 512, 64, [1 + e % 9 for e in range(64)]),     # four columns per lane
    (512, 384, 40, [18 + e % 7 for e in range(40)]),    # 32-row chunks, two and four columns per lane
    (128, 1024, 20, [30 + 5 * e for e in range(20)]),
    (30, 36, 3, [7, 0, 20]),                        # d_model no multiple of 4: the scalar kernels
    (32, 37, 3, [7, 18, 2]),
])
def test_f32_expert_ffn_at_tile_edges(hx, d, f, E, counts):  # noqa: F811
    H, B = hx
    print(f"f32 tiles: d={d} f={f} E={E} rows={sum(counts)}", flush=True)
    out, ref = run_ffn_case(H, B, "f32", d, f, E, counts, seed=d + f + E)
    offs = np.concatenate([[0], np.cumsum(counts)])
    for e in range(E):
        if counts[e]:
            assert nerr(out[offs[e]: offs[e + 1]], ref[offs[e]: offs[e + 1]]) <= TOL["f32"], f"expert {e} ({counts[e]} rows)"


@pytest.mark.parametrize("T,d,f,E,k,offloaded", [(32, 64, 256, 8, 2, False), (33, 64, 256, 8, 2, True), (9, 20, 36, 5, 3, False), (8, 22, 36, 5, 3, False)])
def test_f32_block_reads_its_rows_in_place(hx, T, d, f, E, k, offloaded):  # noqa: F811
    """A stack step whose expert kernel takes the un-grouped rows: each block against the oracle on the same input."""
    H, B = hx
    w = W.Workload("f32_rows", 79, 2, d, f, E, k, T, 1, "f32", 0.0, offloaded)
    cache = {}

    def get(b, e):
        cache[(b, e)] = W.expert_weights(w, b, e)
        return cache[(b, e)]

    store = H.ExpertStore(w, H.config_for(w), threads=2, get_expert=get)
    gates = W.gate_tensors(w)
    stack = H.Stack(w, store, gates=gates)
    stack.set_input(W.step_input(w, 0))
    stack.step()
    torch.cuda.synchronize()
    xs, ys, idx = H.to_numpy64(stack.x_states), H.to_numpy64(stack.y_blocks), stack.topk_idx.cpu().numpy()
    for i in range(w.n_blocks):
        o = R.gate(xs[R.routing_source(i)], *gates[i], w.top_k)
        ok = o["gaps"].min(axis=1) >= 1e-4
        assert np.array_equal(idx[i][ok], o["idx"][ok])
        y = R.block(xs[i], o["p"], o["idx"], {int(e): cache[(i, int(e))] for e in np.unique(o["idx"])}, w.d_ff)
        assert nerr(ys[i][ok], y[ok]) <= TOL["f32"], f"block {i}"
    stack.close()


@pytest.mark.parametrize("d,f,E,counts", [
    (768, 1024, 8, [12, 16, 9, 1, 17, 12, 12, 17]),     # sixteen wavefronts in the second product, each with its four blocks of 16 k and no more
    (772, 1028, 8, [12, 16, 9, 0, 17, 12, 13, 17]),     # a block of four k past them, columns past a tile's end
    (832, 2064, 12, [8, 9] * 6),                        # a second round of blocks for the first wavefront only
    (64, 4100, 16, [3] * 16),                           # many rounds, the last one short
])
def test_f32_expert_ffn_over_rounds_of_requests(hx, d, f, E, counts):  # noqa: F811
    test_f32_expert_ffn_at_tile_edges(hx, d, f, E, counts)


@pytest.mark.parametrize("d,f,E,counts", [
    (4, 12, 3, [1, 0, 2]), (60, 68, 4, [9, 40, 100, 3]),                        # less than a block for each wavefront
    (500, 512, 2, [20, 30]), (508, 516, 2, [5, 12]), (512, 508, 3, [40, 1, 60]),  # a block short of a full round of eight wavefronts, a full one, one past it
    (252, 256, 32, [40] * 32), (256, 260, 32, [40, 60] * 16),                    # the same of four
])
def test_f32_expert_ffn_at_the_first_full_round(hx, d, f, E, counts):  # noqa: F811
    test_f32_expert_ffn_at_tile_edges(hx, d, f, E, counts)


@pytest.mark.parametrize("d,f,E,rows,alone", [
    (768, 3072, 4, 40, (False, True)),      # the second product: 192 workgroups of 64 rows and 16 columns
    (768, 3072, 1, 40, (True, True)), (512, 2048, 1, 100, (True, True)),
    (256, 512, 2, 1000, (False, False)), (768, 3072, 8, 40, (False, False)),
])
def test_a_float32_launch_with_a_workgroup_per_cu_keeps_them_apart(hx, d, f, E, rows, alone):  # noqa: F811
    """By the LDS it takes beside what its sums need."""
    H, B = hx
    print(f"f32, workgroups per CU: d={d} f={f} E={E} rows={rows}", flush=True)
    n = E * rows
    ctx = B.Context(B.make_config(d, f, E, 1, 1, n, B.F32))
    blobs = torch.zeros((E, 2 * d * f), dtype=torch.float32, device="cuda")
    ctx.register_resident_experts(blobs, 8 * d * f, 8 * d * f * E)
    x, y = (torch.zeros((n, d), dtype=torch.float32, device="cuda") for _ in range(2))
    offs = (torch.arange(E + 1, device="cuda") * rows).to(torch.int32)
    ws, stream = torch.zeros(ctx.workspace_bytes, dtype=torch.uint8, device="cuda"), torch.cuda.Stream()
    ctx.expert_ffn(0, x, offs, n, y, ws, stream)     # not captured first: the kernels are loaded
    nodes = kernel_nodes(lambda: ctx.expert_ffn(0, x, offs, n, y, ws, stream), stream)
    assert tuple(k.lds > 0 for k in nodes) == alone
    ctx.close()
