"""Infinite weights in the action-bin head: a logit that is infinite stays infinite (not NaN), the other bins keep theirs."""
import pytest
import torch

import vla_inputs as vi
from paper_2510_06710_amd.harness import Rollout

pytestmark = pytest.mark.gpu


class _Head(vi.SynthModel):
    def lm_head(self):
        w = super().lm_head()
        w[-256 + 5, 3] = float("inf")
        w[-256 + 200, 258] = float("-inf")
        return w


# rows: the partial form and the whole one (above 4096); hidden 272 leaves a chunk of 16
@pytest.mark.parametrize("rows", [3, 4100])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_infinite_head_weights(dtype, rows):
    shape = vi.ModelShape(n_layers=1, hidden=272, n_heads=17, ffn=64, vocab=300, dtype=dtype)
    model = _Head(shape, 4, device="cuda:0")
    run = Rollout(model, rows, 4)
    # halves and quarters: exact in bf16, so that what a split leaves of them is zero
    h = torch.randint(1, 9, (rows, 272), generator=torch.Generator().manual_seed(1)).float().cuda() / 4
    h[1::2, 3] *= -1                                          # bin 5: +inf in even rows, -inf in odd ones; bin 200: -inf
    bins, logp, ent, logits = run.decode(h, 1, 1)
    torch.cuda.synchronize()
    w = model.lm_head()[-256:].double()
    z = h.double() @ torch.where(w.isinf(), 0.0, w).T
    z[0::2, 5], z[1::2, 5], z[:, 200] = float("inf"), float("-inf"), float("-inf")
    got = logits[:, 0].double()
    assert torch.equal(got.isinf(), z.isinf()) and torch.equal(got.sign()[z.isinf()], z.sign()[z.isinf()])
    assert (got - z)[~z.isinf()].abs().max() < 1e-4
    ref = torch.log_softmax(z[1::2], 1)                       # odd rows: two bins of probability 0
    assert torch.equal(bins[1::2, 0].long(), z[1::2].argmax(1))
    assert (logp[1::2, 0].double() - ref.gather(1, bins[1::2].long())[:, 0]).abs().max() < 1e-4
