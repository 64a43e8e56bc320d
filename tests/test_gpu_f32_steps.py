"""fp32 decode steps at the edges of their attention, which takes the projection as it is: a key per thread (256), V in four
parts of 32 positions, eight blocks of eight dims of K loaded ahead (head_dim 64), the new key's position in the first or a
later round."""
import ctypes

import pytest

import vla_inputs as vi
from paper_2510_06710_amd import binding as vb
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


def test_a_step_has_a_label_of_its_own():
    """The step's kernel also rotates and writes K and V: its time is not that of the general attention, which the prefill takes."""
    wl = vi.Workload("labels", _shape(64, 4, 64), batch=2, n_patches=7, n_instr=2, n_action=4)
    vb.lib().vla_profile_enable(1)
    try:
        GpuCase(wl, 6).rollout()
        buf = ctypes.create_string_buffer(1 << 14)
        vb.lib().vla_profile_report(buf, len(buf))
    finally:
        vb.lib().vla_profile_enable(0)
    counts = {line.rsplit(" ", 3)[0]: int(line.rsplit(" ", 3)[1]) for line in buf.value.decode().splitlines()}
    layers, steps = wl.shape.n_layers, wl.n_action - 1
    assert counts["attention_step"] == layers * steps and counts["attention_generic"] == layers, counts
