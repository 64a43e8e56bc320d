"""The gradient pass over more layers than its first pass leaves intermediates of (without the activations kept: the top two where
the top layer works on its read rows and its intermediates fit beside those of the layer below, else the top one), against the fp64
oracle with the bounds of test_gpu_backward.py."""
import numpy as np
import pytest

import vla_inputs as vi
from test_gpu_backward import _assert_logp_bf16, _compare, _oracle, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers", [1, 3, 4])
@pytest.mark.parametrize("hidden,heads,ffn,S,A,mode", [(64, 4, 96, 40, 7, 0),       # two layers' intermediates
                                                       (64, 4, 96, 9, 7, 0),        # the top layer's, all rows
                                                       (32, 2, 48, 300, 100, 0),    # its read rows, whose scores do not fit beside
                                                       (64, 4, 96, 40, 6, 1)])
def test_fp32_layers(layers, hidden, heads, ffn, S, A, mode):
    shape = vi.ModelShape(n_layers=layers, hidden=hidden, n_heads=heads, ffn=ffn, vocab=640, dtype="f32")
    wl = vi.Workload("layers_bw", shape, batch=3, n_patches=S - 2, n_instr=2, n_action=A, mode=mode)
    case, lora, bins, coef, grads, logp = _run(wl, 31, 4, 0.5, max_batch=2)
    ref, ref_logp = _oracle(wl, 31, lora, bins, coef, 3, 0.5)
    assert np.max(np.abs(logp - ref_logp)) < 1e-4
    _compare(grads, ref, 2e-4)


@pytest.mark.parametrize("S,A,batch,max_batch", [(49, 4, 5, 2), (40, 20, 4, 4)])
def test_bf16_layers(S, A, batch, max_batch):
    shape = vi.ModelShape(n_layers=3, hidden=256, n_heads=2, ffn=512, vocab=640, dtype="bf16")
    wl = vi.Workload("layers_bw", shape, batch=batch, n_patches=S - 9, n_instr=9, n_action=A)
    case, lora, bins, coef, grads, logp = _run(wl, 33, 16, 0.25, max_batch=max_batch)
    ref, ref_logp = _oracle(wl, 33, lora, bins, coef, batch, 0.25, operand_dtype="bf16")
    _assert_logp_bf16(logp, ref_logp)
    print(f"\n[parity] backward bf16 three layers S {S} A {A}: {_compare(grads, ref, 2e-2, 1e-2)}", flush=True)
