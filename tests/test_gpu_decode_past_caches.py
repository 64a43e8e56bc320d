"""The attention of few (environment, head) pairs reads K and V past the caches where those of all layers exceed 256 MB: the same bits as
through them, which the same environments take in a smaller batch.  head_dim 128 and 64, just past the bound."""
import pytest
import torch

import vla_inputs as vi
from paper_2510_06710_amd.harness import Rollout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,ffn,many", [(32, 256, 31), (64, 512, 15)])
def test_same_bits(heads, ffn, many):
    few, S, A = 3, 508, 3
    shape = vi.ModelShape(n_layers=1, hidden=4096, n_heads=heads, ffn=ffn, vocab=640, dtype="bf16")
    wl = vi.Workload("past", shape, batch=many, n_patches=S - 2, n_instr=2, n_action=A)
    patch, ids = vi.observation(wl, 2, device="cuda:0")
    run = Rollout(vi.SynthModel(shape, 2, device="cuda:0"), many, S + A)

    def outputs(n):
        h, _ = run.prefill(patch[:n].contiguous(), ids[:n].contiguous(), want_value=False)
        return [x[:few].clone() for x in (h, *run.decode(h, S, A))]

    for a, b in zip(outputs(many), outputs(few)):
        assert torch.equal(a, b)
