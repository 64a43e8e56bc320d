"""fp32 decode steps at the edges of their attention, which takes the projection as it is: a key per thread (256), V in four
parts of 32 positions, eight blocks of eight dims of K loaded ahead (head_dim 64), the new key's position in the first or a
later round."""
import pytest

import vla_inputs as vi
from parity import GpuCase, compare_rollout, oracle_rollout

pytestmark = pytest.mark.gpu


def _shape(hidden, heads, ffn):
    return vi.ModelShape(n_layers=2, hidden=hidden, n_heads=heads, ffn=ffn, vocab=300, dtype="f32")


# head_dim 16, 64, 48, 256, 208, 80, 64 (the sampler's norm for the next step: widths that fill 1024-wide pieces in part)
@pytest.mark.parametrize("B,S,hidden,heads,ffn", [(1, 1, 16, 1, 20), (16, 30, 256, 4, 100), (17, 62, 96, 2, 64), (2, 126, 1024, 4, 72),
                                                  (3, 254, 64, 1, 64), (2, 300, 1040, 5, 44), (65, 2, 80, 1, 36), (2, 3, 2112, 33, 64)])
def test_steps(B, S, hidden, heads, ffn):
    wl = vi.Workload("steps", _shape(hidden, heads, ffn), batch=B, n_patches=S - 1, n_instr=1, n_action=4)
    print(compare_rollout(GpuCase(wl, 6).rollout(), oracle_rollout(wl, 6), "f32", autoregressive=True), flush=True)
