"""Tiles of 96 and 160 rows, which the small-tile kernel takes where they fill a round of one workgroup per CU: a sequence's prefix and
action chunk do not depend, bit for bit, on whether a call's row count selects them.  Width 2048, FFN 5504: 750 rows take 96 x 64 (O, down) and
160 x 128 (QKV), 1,250 160 x 64, 1,375 96 x 128, all with a ragged last tile; 450 rows 96 x 128 and 300 rows 160 x 128 for QKV and gate/up.
FFN 11008: 90 rows 96 x 128 for gate/up, in one tile that reaches past the rows.  The large batch takes 256-row tiles."""
import pytest
import torch

import vla_inputs as vi
from paper_2510_06710_amd.harness import Rollout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prepack", [True, False])
@pytest.mark.parametrize("hidden,ffn,rows,counts", [(2048, 5504, 125, (6, 10, 11)), (2048, 5504, 90, (5,)), (2048, 5504, 100, (3,)), (1024, 11008, 90, (1,))])
def test_a_row_does_not_depend_on_the_tile(hidden, ffn, rows, counts, prepack):
    shape = vi.ModelShape(n_layers=2, hidden=hidden, n_heads=hidden // 128, ffn=ffn, vocab=640, dtype="bf16")
    big, T, A = 127, 14, 33
    wl = vi.Workload("rounds", shape, batch=big, n_patches=rows - T, n_instr=T, n_action=A, mode=1)
    patch, ids = vi.observation(wl, 6, device="cuda:0")
    synth = vi.SynthModel(shape, 6, device="cuda:0")
    slot = synth.slot_embed(A)
    run = Rollout(synth, big, rows + A, prepack=prepack)

    def outputs(n):
        h, value = run.prefill(patch[:n], ids[:n])
        bins, logp, ent, logits = run.decode(h, rows, A, 1, slot)
        return [x[: min(counts)].clone() for x in (h, value, bins, logp, ent, logits)]

    want = outputs(big)
    for n in counts:
        for a, b in zip(want, outputs(n)):
            assert torch.equal(a, b), n
