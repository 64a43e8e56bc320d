"""The large GEMM's tiles of 160, 192, 224 and 256 rows sum in the same order: a sequence's prefix and action chunk do not depend,
bit for bit, on which of them a call's row count selects.  At width 2048 the O and down projections (8 tile columns) take 160
rows up to 5120 rows, 192 up to 6144, 224 up to 7168; 127 sequences take 256.  127 x 129 rows end in a nearly full tile, the others
in ragged ones; at 53 x 128 rows the last tile of 224 rows reads past the activation buffer's last row."""
import pytest
import torch

import vla_inputs as vi
from paper_2510_06710_amd.harness import Rollout

pytestmark = pytest.mark.gpu
WIDE = vi.ModelShape(n_layers=2, hidden=2048, n_heads=16, ffn=2048, vocab=640, dtype="bf16")


@pytest.mark.parametrize("prepack", [True, False])
@pytest.mark.parametrize("rows,counts", [(129, (33, 40, 48, 55)), (128, (40, 53, 56))])
def test_a_row_does_not_depend_on_the_tile_height(rows, counts, prepack):
    big, T, A = 127, 14, 33
    wl = vi.Workload("heights", WIDE, batch=big, n_patches=rows - T, n_instr=T, n_action=A, mode=1)
    patch, ids = vi.observation(wl, 6, device="cuda:0")
    synth = vi.SynthModel(WIDE, 6, device="cuda:0")
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
