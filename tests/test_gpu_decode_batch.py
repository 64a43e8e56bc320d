"""A decode step's result for an environment does not depend, bit for bit, on how many others share the step, up to 128 of
them: whichever kernels the row count selects add in one order."""
import functools

import pytest
import torch

import vla_inputs as vi
from paper_2510_06710_amd.harness import Rollout

pytestmark = pytest.mark.gpu
MANY, S, A = 128, 300, 4
SHAPES = {
    # head_dim 64, K in four parts of 8 and 11 tiles
    "h2048": vi.ModelShape(n_layers=2, hidden=2048, n_heads=32, ffn=2816, vocab=640, dtype="bf16"),
    # the 7B width: eight parts, two for the down projection, repacked weights
    "h4096": vi.ModelShape(n_layers=1, hidden=4096, n_heads=32, ffn=1152, vocab=640, dtype="bf16"),
    # a width that the vectorised norm does not take, three parts of four pieces filled
    "h640": vi.ModelShape(n_layers=1, hidden=640, n_heads=5, ffn=1152, vocab=640, dtype="bf16"),
    # FFN no multiple of 64: the generic kernel for these products, at all row counts
    "h256": vi.ModelShape(n_layers=1, hidden=256, n_heads=2, ffn=544, vocab=640, dtype="bf16"),
}


@functools.lru_cache(maxsize=1)
def _rollout(name, prepack=True):
    shape = SHAPES[name]
    wl = vi.Workload("batch", shape, batch=MANY, n_patches=S - 2, n_instr=2, n_action=A)
    run = Rollout(vi.SynthModel(shape, 8, device="cuda:0"), MANY, S + A, prepack=prepack)
    patch, ids = vi.observation(wl, 8, device="cuda:0")
    noise = vi.gumbel_noise(wl, 8, device="cuda:0")

    @functools.lru_cache(maxsize=None)
    def outputs(n):
        h, _ = run.prefill(patch[:n], ids[:n], want_value=False)
        out = run.decode(h, S, A, gumbel=noise[:n].contiguous())
        torch.cuda.synchronize()
        return h, *out
    return outputs


# 4 | 5: where the norm leaves the GEMMs; 31 | 32: 1024 (environment, head) pairs, where the attention's split of the keys
# changes; 16 | 17, 32 | 33, 64 | 65: where the GEMMs' kernels or tiles do
@pytest.mark.parametrize("few,many", [(1, 2), (3, 4), (4, 5), (31, 32), (5, 16), (16, 17), (32, 33), (64, 65), (17, MANY), (1, MANY)])
@pytest.mark.parametrize("name", list(SHAPES))
def test_few_and_many_environments(name, few, many):
    outputs = _rollout(name)
    for x, y in zip(outputs(few), outputs(many)):
        assert torch.equal(x, y[:few])


@pytest.mark.parametrize("n", [3, 16, 24, 100])
def test_with_and_without_repacked_weights(n):
    packed = _rollout("h4096")(n)
    for x, y in zip(packed, _rollout("h4096", prepack=False)(n)):
        assert torch.equal(x, y)
