"""fp32 decode steps at the edges of their attention, which takes the projection as it is: a key per thread (256), V in four
parts of 32 positions, eight blocks of eight dims of K loaded ahead (head_dim 64), the new key's position in the first or a
later round."""
import ctypes

import pytest
import torch

import vla_inputs as vi
from paper_2510_06710_amd import binding as vb
from paper_2510_06710_amd.harness import Rollout
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


# keys of the three steps: S + 1 .. S + 3.  Many environments take a wave per (environment, head), few take four.
@pytest.mark.parametrize("S,hidden,heads,many,few", [(1, 16, 1, 71, 7), (30, 512, 32, 33, 1), (62, 1024, 16, 67, 3), (127, 1040, 13, 90, 5),
                                                     (125, 2048, 16, 65, 2), (77, 768, 3, 220, 40), (30, 1024, 4, 67, 5), (508, 256, 16, 257, 31)])
def test_a_step_does_not_depend_on_the_batch(S, hidden, heads, many, few):
    """The four sums of a head's keys and of its values are formed by one wave or by four: the same bits."""
    shape = _shape(hidden, heads, 64)
    wl = vi.Workload("waves", shape, batch=many, n_patches=0, n_instr=S, n_action=4)
    patch, ids = vi.observation(wl, 3, device="cuda:0")
    run = Rollout(vi.SynthModel(shape, 3, device="cuda:0"), many, S + 4)

    def outputs(n):
        h, _ = run.prefill(patch[:n].contiguous(), ids[:n].contiguous())
        return [x[:few].clone() for x in (h, *run.decode(h, S, 4))]

    assert many * heads >= 8 * (S + 3) and few * heads < 8 * (S + 1) and hidden // heads * (S + 3) <= 20480
    for a, b in zip(outputs(many), outputs(few)):
        assert torch.equal(a, b)


# The norms inside the products: rows that fill the large tile of the generic kernel and leave a remainder, widths that are no multiple
# of a wave's share of K (two, six and eight blocks of 16 at a time), a head whose rows exceed the narrow form's 512 workgroups.
@pytest.mark.parametrize("B,S,hidden,heads,ffn", [(5, 221, 528, 11, 1040), (1, 3, 272, 17, 700), (515, 2, 272, 17, 36), (3, 40, 784, 7, 1200)])
def test_norms_in_the_products(B, S, hidden, heads, ffn):
    wl = vi.Workload("norms", _shape(hidden, heads, ffn), batch=B, n_patches=S - 1, n_instr=1, n_action=3)
    print(compare_rollout(GpuCase(wl, 9).rollout(), oracle_rollout(wl, 9), "f32", autoregressive=True), flush=True)

