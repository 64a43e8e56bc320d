"""Decode steps on the fast path at the edges of its kernels against the oracle: the weight-streaming GEMM (up to 32 rows:
one and two row blocks, tiles of 64 columns that do not divide evenly over the parts of K, fewer parts than waves) and
the attention that takes the projection as it is (the new key on either side of a 64-key chunk, head_dim 64 and 128); 33 to
128 rows: the small tiles with row-major activations, at the edges of their 64 and 128 rows.  Up to 4
rows the GEMMs form the norm of their input (a width too large for that, the widest one; a FFN they decline)."""
import pytest

import vla_inputs as vi
from parity import GpuCase, compare_rollout, oracle_rollout

pytestmark = pytest.mark.gpu


# (environments, prefix, hidden, heads, ffn): FFN 544 and 528 are declined by all fast paths; 2176 = 34 tiles in four parts, 1152 = 18 in two
@pytest.mark.parametrize("B,S,hidden,heads,ffn", [(1, 62, 256, 2, 544), (16, 126, 256, 2, 544), (17, 5, 256, 4, 512), (32, 60, 256, 4, 544),
                                                  (33, 3, 256, 2, 512), (65, 3, 256, 2, 512), (128, 2, 1024, 8, 512), (3, 509, 256, 2, 512), (2, 1, 1024, 8, 1024),
                                                  (1, 7, 4224, 33, 512), (1, 4, 4096, 32, 512), (4, 3, 1024, 8, 1024), (5, 3, 1024, 8, 1024), (2, 4, 256, 2, 528),
                                                  (7, 5, 256, 2, 2176), (24, 5, 512, 4, 2176), (40, 2, 1024, 8, 1152)])
def test_steps(B, S, hidden, heads, ffn):
    shape = vi.ModelShape(n_layers=1, hidden=hidden, n_heads=heads, ffn=ffn, vocab=300, dtype="bf16")
    wl = vi.Workload("steps", shape, batch=B, n_patches=S - 1, n_instr=1, n_action=4)
    print(compare_rollout(GpuCase(wl, 6).rollout(), oracle_rollout(wl, 6, operand_dtype="bf16"), "bf16", autoregressive=True), flush=True)
