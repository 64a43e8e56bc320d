"""The action-bin head and sampler at the edges of its tiles (16 rows, K chunks of 256) and on both sides of the row count
where it stops handing partial logits to a second kernel (4096), against the fp64 oracle."""
import pytest
import torch

import vla_inputs as vi
from paper_2510_06710_amd.harness import Rollout
from parity import GpuCase, compare_rollout, oracle_rollout

pytestmark = pytest.mark.gpu


# (storage, hidden, heads, environments, slots): rows = environments x slots; hidden 272 leaves a chunk of 16
@pytest.mark.parametrize("dtype,hidden,heads,B,A", [("f32", 48, 3, 9, 460), ("bf16", 48, 3, 9, 460), ("f32", 272, 17, 1, 17),
                                                    ("bf16", 272, 17, 1, 17), ("bf16", 528, 11, 5, 3), ("bf16", 256, 2, 8, 512),
                                                    ("f32", 16, 1, 1, 1)])
def test_chunk_head(dtype, hidden, heads, B, A):
    shape = vi.ModelShape(n_layers=1, hidden=hidden, n_heads=heads, ffn=64, vocab=300, dtype=dtype)
    wl = vi.Workload("head", shape, batch=B, n_patches=2, n_instr=1, n_action=A, mode=1, temperature=1.6)
    stats = compare_rollout(GpuCase(wl, 3).rollout(), oracle_rollout(wl, 3), dtype, autoregressive=False)
    print(f"\n[parity] head {dtype} H={hidden} rows={B * A}: {stats}", flush=True)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_autoregressive_head(dtype):
    shape = vi.ModelShape(n_layers=1, hidden=272, n_heads=17, ffn=64, vocab=300, dtype=dtype)
    wl = vi.Workload("head", shape, batch=17, n_patches=2, n_instr=1, n_action=3)
    compare_rollout(GpuCase(wl, 4).rollout(), oracle_rollout(wl, 4), dtype, autoregressive=True)


# A decode step's final norm is the head's, gain before the product and 1 / rms behind it, in either form
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hidden,heads", [(48, 3), (272, 17)])
def test_a_decode_row_does_not_depend_on_the_form(dtype, hidden, heads):
    """Widths whose products have one order of sums for any number of rows: the same bits on both sides of 4096."""
    many, few, S, A = 4131, 70, 3, 3
    shape = vi.ModelShape(n_layers=1, hidden=hidden, n_heads=heads, ffn=64, vocab=300, dtype=dtype)
    wl = vi.Workload("head", shape, batch=many, n_patches=2, n_instr=1, n_action=A, temperature=1.6)
    patch, ids = vi.observation(wl, 5, device="cuda:0")
    noise = vi.gumbel_noise(wl, 5, device="cuda:0")
    run = Rollout(vi.SynthModel(shape, 5, device="cuda:0"), many, S + A)

    def outputs(n):
        h, _ = run.prefill(patch[:n].contiguous(), ids[:n].contiguous())
        return [x[:few].clone() for x in (h, *run.decode(h, S, A, 0, None, 1.6, noise[:n].contiguous()))]

    for a, b in zip(outputs(many), outputs(few)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_autoregressive_whole_head(dtype):
    shape = vi.ModelShape(n_layers=1, hidden=48, n_heads=3, ffn=64, vocab=300, dtype=dtype)
    wl = vi.Workload("head", shape, batch=4099, n_patches=1, n_instr=1, n_action=3)
    compare_rollout(GpuCase(wl, 4).rollout(), oracle_rollout(wl, 4), dtype, autoregressive=True)
