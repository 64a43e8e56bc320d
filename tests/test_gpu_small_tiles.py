"""The large GEMM's small-tile kernels (64 x 64, 64 x 128, 128 x 128 outputs, chosen by the number of tiles) sum in the same
order as its 256 x 256 tiles: what a sequence gets must not depend, bit for bit, on how many others share the call, and
must match the oracle at row counts around the tile edges.  Width 1024: the few-row calls take the small tiles, and the
9,000 and more rows of the large batches 256 x 256 ones (36 tile rows x 12, x 4 and x 22 tile columns)."""
import dataclasses

import pytest
import torch

import vla_inputs as vi
from paper_2510_06710_amd.harness import Rollout
from parity import GpuCase, compare_rollout, oracle_rollout

pytestmark = pytest.mark.gpu
SHAPE = vi.ModelShape(n_layers=2, hidden=1024, n_heads=8, ffn=2816, vocab=640, dtype="bf16")


@pytest.mark.parametrize("prepack", [True, False])
@pytest.mark.parametrize("B", [1, 2, 3, 7, 20])
def test_a_row_does_not_depend_on_the_batch(B, prepack):
    big, P, T, A = 70, 115, 14, 33                           # 129 prefix rows, 33 slots
    wl = vi.Workload("tiles", SHAPE, batch=big, n_patches=P, n_instr=T, n_action=A, mode=1)
    patch, ids = vi.observation(wl, 5, device="cuda:0")
    synth = vi.SynthModel(SHAPE, 5, device="cuda:0")
    slot = synth.slot_embed(A)
    run = Rollout(synth, big, P + T + A, prepack=prepack)
    got = []
    for n in (big, B):
        h, _ = run.prefill(patch[:n], ids[:n], want_value=False)
        bins, logp, ent, logits = run.decode(h, P + T, A, 1, slot)
        got.append([x[:B].clone() for x in (logits, logp, ent, bins)])
    torch.cuda.synchronize()
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B,P,A", [(1, 60, 40), (1, 125, 65), (2, 125, 33), (1, 250, 129)])
def test_against_the_oracle(B, P, A):
    """The oracle rounds the stored tensors as the kernels do; what remains are roundings that fall the other way.  One
    layer: 0.0012 RMS in the log-probs at this width, so the bar of 1e-2 is eight of them.  (Two layers: 0.00245, and the
    largest of 129 draws, 0.0116, is over the bar with any tile: the kernels agree bit for bit.)"""
    wl = vi.Workload("tiles", dataclasses.replace(SHAPE, n_layers=1), batch=B, n_patches=P, n_instr=3, n_action=A, mode=1)
    print(compare_rollout(GpuCase(wl, 7).rollout(), oracle_rollout(wl, 7, operand_dtype="bf16"), "bf16", autoregressive=False), flush=True)
