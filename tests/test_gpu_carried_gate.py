"""A pre-gate carried in two halves (by the expert launch and the combine of the block before) gives
the bits of the separate gate launch: whole stack steps against the primitives called one by one, at
the edges of its token tiles, of the planes the reduction is cut into and of what it serves."""
import pytest

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
