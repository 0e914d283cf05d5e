"""The fused expert kernel's ring of weight tiles: one, two and more sub-slabs of d_ff per workgroup, every chunk size, experts whose
weights end the store."""
import numpy as np
import pytest
import torch

from launch_count import kernel_nodes
from test_gpu_parity import TOL, hx, nerr, run_ffn_case  # noqa: F401  (hx is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f,E,counts", [
    (64, 192, 4, [1, 0, 2, 3]), (64, 640, 4, [3] * 4), (64, 320, 4, [9, 30, 1, 40]),  # the smallest ring
    (128, 512, 16, [5] * 16), (256, 1024, 12, [20] * 12), (256, 320, 12, [40, 24] * 6),
    (512, 2048, 64, [1 + e % 3 for e in range(64)]),                # two sub-slabs a workgroup
    (768, 3072, 16, [1] * 16), (768, 3072, 60, [1 + e % 7 for e in range(60)]),     # one; several
    (512, 384, 16, [9] * 16), (768, 384, 16, [9] * 16), (1024, 384, 16, [9] * 16),  # 32-row chunks
    (512, 384, 16, [24] * 16), (768, 384, 16, [24] * 16), (768, 320, 16, [24] * 16), (1024, 384, 16, [24] * 16),    # 64-row ones, four and eight wavefronts
    (768, 3072, 5, [4] * 5), (1024, 4096, 3, [4] * 3),              # two wavefronts; the second had a ring out of step with its tiles from the second sub-slab on
    (2048, 8192, 8, [2] * 8), (2048, 512, 8, [30] * 8),
])
def test_fused_expert_kernel_over_sub_slabs(hx, d, f, E, counts):  # noqa: F811
    H, B = hx
    print(f"fused ring: d={d} f={f} E={E} rows={sum(counts)}", flush=True)
    out, ref = run_ffn_case(H, B, "bf16", d, f, E, counts, seed=d + f + E)
    offs = np.concatenate([[0], np.cumsum(counts)])
    for e in range(E):
        if counts[e]:
            assert nerr(out[offs[e]: offs[e + 1]], ref[offs[e]: offs[e + 1]]) <= TOL["bf16"], f"expert {e} ({counts[e]} rows)"


@pytest.mark.parametrize("d,f,E,rows,alone", [
    (512, 2048, 128, 30, True), (512, 2048, 256, 30, False),        # 64-row chunks: 256 and 512 workgroups
    (768, 3072, 32, 12, True), (768, 3072, 64, 18, False),          # 32-row chunks: 256 and 384 workgroups
    (1024, 4096, 16, 9, False), (256, 1024, 16, 3, False),          # kernels that do not mind
])
def test_a_launch_with_a_workgroup_per_cu_keeps_them_apart(hx, d, f, E, rows, alone):  # noqa: F811
    """By the LDS it takes: of a CU's 160 KiB more than half, or what it needs."""
    H, B = hx
    print(f"fused, workgroups per CU: d={d} f={f} E={E} rows={rows}", flush=True)
    n = E * rows
    ctx = B.Context(B.make_config(d, f, E, 1, 1, n, B.BF16))
    blobs = torch.zeros((E, 2 * d * f), dtype=torch.bfloat16, device="cuda")
    ctx.register_resident_experts(blobs, 4 * d * f, 4 * d * f * E)
    assert ctx.ffn_kernel_name(n) == "ffn_fused_kernel"
    x, y = (torch.zeros((n, d), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    offs = (torch.arange(E + 1, device="cuda") * rows).to(torch.int32)
    ws, stream = torch.zeros(ctx.workspace_bytes, dtype=torch.uint8, device="cuda"), torch.cuda.Stream()
    ctx.expert_ffn(0, x, offs, n, y, ws, stream)     # not captured first: the kernels are loaded
    nodes = kernel_nodes(lambda: ctx.expert_ffn(0, x, offs, n, y, ws, stream), stream)
    assert (nodes[0].lds > 80 * 1024) == alone, nodes[0].lds
    ctx.close()
