"""The two tiled GEMMs of the expert FFN at the sizes where their tiling can go wrong: chunks of
every number of 16-row tiles a workgroup body is built for, one row more and one row less, both
column widths, several K slices, many experts, and scratch that does not hold all rows at once."""
import numpy as np
import pytest
import torch

import workloads as W
from launch_count import kernel_launches, kernel_nodes
from test_gpu_parity import TOL, hx, nerr, run_ffn_case  # noqa: F401  (hx is a fixture)

pytestmark = pytest.mark.gpu

EDGES = [1, 16, 17, 64, 65, 128, 129, 192, 193, 255, 256, 257, 288, 289, 304, 305, 320, 321, 0, 640, 641, 700, 500]


@pytest.mark.parametrize("d,f,E,counts", [
    (256, 512, len(EDGES), EDGES),                                   # 128-column blocks in both products
    (128, 256, len(EDGES), EDGES),
    (128, 1024, 2, [1500, 700]),                                     # K slices of the down-projection
    (512, 256, 130, [200 + (e * 37) % 140 if e % 3 else 300 for e in range(130)]),   # three rounds of 64 experts in the lookup
    (512, 2048, 8, [9, 31, 8, 16, 17, 0, 33, 20]),                   # few rows per expert: chosen over the fused kernel
    (2048, 256, 4, [60, 0, 80, 31]),
])
def test_expert_ffn_at_tile_edges(hx, d, f, E, counts):  # noqa: F811
    H, B = hx
    ctx = B.Context(B.make_config(d, f, E, 1, 1, sum(counts), B.BF16, flags=B.FLAG_HOST_ONLY))
    name = ctx.ffn_kernel_name(sum(counts))
    ctx.close()
    print(f"gemm tiles: d={d} f={f} E={E} rows={sum(counts)} {name}", flush=True)
    assert "gemm" in name
    out, ref = run_ffn_case(H, B, "bf16", d, f, E, counts, seed=d + f + E)
    offs = np.concatenate([[0], np.cumsum(counts)])
    for e in range(E):   # an expert at a time, so that a wrong small one cannot hide behind a big one
        if counts[e]:
            assert nerr(out[offs[e]: offs[e + 1]], ref[offs[e]: offs[e + 1]]) <= TOL["bf16"], f"expert {e} ({counts[e]} rows)"


# every number of row tiles a chunk can have (a wavefront's share, what it loads and the ring go by it), the last tile full, short and of one row
EVERY = [16 * t - (0, 15, 6)[t % 3] for t in range(1, 21)]
LARGE = EVERY + [320] * 6 + [t % 7 + 300 for t in EVERY]


@pytest.mark.parametrize("d,f,counts,columns_up,columns_down,slices", [
    (128, 256, LARGE, 128, 128, 1),     # four k-tiles up, eight down; the rings have 4, 8 and 14 stages
    (256, 768, LARGE, 256, 128, 1),
    (512, 2560, LARGE, 256, 128, 1),    # more k-tiles than the deepest ring: the steady loop and the tail
    (768, 256, LARGE, 128, 256, 1),     # wide column blocks in the down-projection, over the rings of up to 2, 8 and 20 row tiles
    (1024, 512, LARGE, 128, 256, 1),
    (256, 768, EVERY, 128, 128, 2), (256, 2048, EVERY, 256, 128, 4),
    (512, 4096, EVERY + [5] * 16, 256, 256, 2), (256, 8192, EVERY + [5] * 16, 256, 256, 4),
    (256, 256, [320], 128, 128, 4),     # two k-tiles a slice, fewer than the four stages of the largest chunks' ring: surplus requests
    (256, 256, [600, 16, 100], 128, 128, 2),    # four, fewer than the eight and fourteen of the smaller ones'
])
def test_every_number_of_row_tiles(hx, d, f, counts, columns_up, columns_down, slices):  # noqa: F811
    H, B = hx
    E, n = len(counts), sum(counts)
    print(f"gemm row tiles: d={d} f={f} E={E} rows={n}", flush=True)
    ctx = B.Context(B.make_config(d, f, E, 1, 1, n, B.BF16))
    assert "gemm" in ctx.ffn_kernel_name(n)
    # the launch is of the kind it is here for: column blocks and K slices out of its grids
    blobs, x, y = torch.zeros((E, 2 * d * f), dtype=torch.bfloat16, device="cuda"), *(torch.zeros((n, d), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    ctx.register_resident_experts(blobs, 4 * d * f, 4 * d * f * E)
    offs = torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).cuda()
    ws, stream = torch.zeros(ctx.workspace_bytes, dtype=torch.uint8, device="cuda"), torch.cuda.Stream()
    torch.cuda.synchronize()
    ctx.expert_ffn(0, x, offs, n, y, ws, stream)     # not captured first: the kernels are loaded
    nodes = kernel_nodes(lambda: ctx.expert_ffn(0, x, offs, n, y, ws, stream), stream)
    ctx.close()
    chunks = E + n // 320
    assert [k.grid[0] for k in nodes[:3]] == [chunks, chunks * f // columns_up, chunks * d // columns_down * slices]
    assert len(nodes) == (4 if slices > 1 else 3)
    out, ref = run_ffn_case(H, B, "bf16", d, f, E, counts, seed=d + f)
    offs = np.concatenate([[0], np.cumsum(counts)])
    for e in range(E):
        assert nerr(out[offs[e]: offs[e + 1]], ref[offs[e]: offs[e + 1]]) <= TOL["bf16"], f"expert {e} ({counts[e]} rows)"


@pytest.mark.parametrize("counts", [[120] * 16, [700, 0, 321, 5, 64, 100, 1, 16, 17, 90, 200, 33, 50, 150, 80, 93]])
def test_static_scratch_takes_several_passes_and_gives_the_same_bits(hx, counts):  # noqa: F811
    """A launch the static buffer admits but whose hidden activation it does not hold at once."""
    H, B = hx
    d, f, E, n = 128, 8192, 16, sum(counts)
    assert (n // 16 + E) * 16 * (d + f) * 2 > B.STATIC_SCRATCH_BYTES
    w = W.Workload("gemm_passes", 78, 1, d, f, E, 1, n, 1, "bf16", 0.0, False)
    cfg = H.config_for(w)
    store = H.ExpertStore(w, cfg, threads=4)
    ctx = B.Context(cfg)
    ctx.register_resident_experts(store.to_hbm(), store.expert_stride, store.block_stride)
    assert "gemm" in ctx.ffn_kernel_name(n)
    x = H.to_device(W.round_to_bf16(np.random.default_rng(5).standard_normal((n, d)).astype(np.float32)), "bf16")
    offs = torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).cuda()
    ys = [torch.full((n, d), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    ws = torch.full((ctx.workspace_bytes,), 0x5A, dtype=torch.uint8, device="cuda")
    ctx.expert_ffn(0, x, offs, n, ys[0], ws)
    ctx.expert_ffn_static(0, x, offs, n, ys[1])
    torch.cuda.synchronize()
    assert torch.equal(ys[0].view(torch.int16), ys[1].view(torch.int16))
    assert float(ys[0].float().abs().max()) not in (0.0, 7.0)
    ctx.close()


@pytest.mark.parametrize("d,f,E,rows,launches", [
    (2048, 1024, 40, 150, 6), (1024, 2304, 16, 150, 7),         # two passes of three launches (and a reduction of two K slices)
    (512, 1792, 24, 190, 2), (768, 1280, 64, 150, 1),           # the fused kernel, in as many d_ff ranges as the GEMMs have K slices
    (768, 4352, 10, 190, 2), (1024, 2816, 8, 190, 2),           # four ranges that are no multiple of the eight-wavefront kernel's sub-slab
    (1024, 2048, 16, 190, 2), (128, 8192, 16, 120, 2),
    (768, 1536, 8, 150, 4), (768, 3072, 64, 40, 3),             # everything at once, with two K slices and with one
])
def test_static_scratch_takes_the_faster_way_and_gives_the_workspace_bits(hx, d, f, E, rows, launches):  # noqa: F811
    H, B = hx
    g = np.random.default_rng(d + f + E)
    counts = np.bincount(g.integers(0, E, size=E * rows), minlength=E)
    counts[0], counts[-1] = counts[0] + counts[-1], 0
    n = int(counts.sum())
    gen = torch.Generator(device="cuda").manual_seed(d + f)
    blobs = torch.empty((1, E, 2 * d * f), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=gen)
    x = torch.empty((n, d), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    offs = torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).cuda()
    ctx = B.Context(B.make_config(d, f, E, 1, 1, n, B.BF16))
    ctx.register_resident_experts(blobs, 4 * d * f, 4 * d * f * E)
    assert "gemm" in ctx.ffn_kernel_name(n)
    print(f"static route: d={d} f={f} E={E} rows={n}", flush=True)
    ys = [torch.full((n, d), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    ws = torch.full((ctx.workspace_bytes,), 0x5A, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    ctx.expert_ffn(0, x, offs, n, ys[0], ws, stream)
    ctx.expert_ffn_static(0, x, offs, n, ys[1], stream)
    torch.cuda.synchronize()
    assert torch.equal(ys[0].view(torch.int16), ys[1].view(torch.int16))
    assert 0.0 < float(ys[0].float().abs().max()) < 7.0
    assert kernel_launches(lambda: ctx.expert_ffn_static(0, x, offs, n, ys[1], stream), stream) == launches
    ctx.close()
