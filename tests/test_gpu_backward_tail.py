"""The backward's top layer on the read rows alone: both sides of the rule (a quarter of the rows) and at it, both modes,
more micro-batches than one, against the fp64 oracle (fp32 storage: 2e-4 of each gradient's largest entry, 1e-4 in the
log-probs; bf16: the bounds of test_gpu_backward.py)."""
import numpy as np
import pytest

import vla_inputs as vi
from test_gpu_backward import _assert_logp_bf16, _compare, _oracle, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("mode,S,A", [(0, 10, 3), (0, 9, 3), (0, 40, 7), (1, 9, 3), (1, 8, 3), (1, 33, 4)])
def test_tail_rows(mode, S, A, keep):
    wl = vi.scaled(vi.WORKLOADS["cfg1_tiny_fp32"], batch=3, n_patches=S - 2, n_instr=2, n_action=A, mode=mode)
    case, lora, bins, coef, grads, logp = _run(wl, 21, 4, 0.5, max_batch=2, keep=keep)
    ref, ref_logp = _oracle(wl, 21, lora, bins, coef, 3, 0.5)
    assert np.max(np.abs(logp - ref_logp)) < 1e-4
    _compare(grads, ref, 2e-4)


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("mode,S,A,batch,max_batch", [(0, 40, 20, 4, 4), (1, 40, 20, 4, 4),      # every row through the top layer
                                                      (0, 40, 20, 5, 2),                         # ... in passes of 2, 2 and 1
                                                      (0, 49, 4, 5, 2), (1, 49, 4, 5, 2)])       # the read rows alone
def test_bf16_rows(mode, S, A, batch, max_batch, keep):
    shape = vi.ModelShape(n_layers=2, hidden=256, n_heads=2, ffn=512, vocab=640, dtype="bf16")
    wl = vi.Workload("bf16_bw", shape, batch=batch, n_patches=S - 9, n_instr=9, n_action=A, mode=mode)
    case, lora, bins, coef, grads, logp = _run(wl, 23, 16, 0.25, max_batch=max_batch, keep=keep)
    ref, ref_logp = _oracle(wl, 23, lora, bins, coef, batch, 0.25, operand_dtype="bf16")
    _assert_logp_bf16(logp, ref_logp)
    print(f"\n[parity] backward bf16 mode {mode} S {S} A {A}: {_compare(grads, ref, 2e-2, 1e-2)}", flush=True)


@pytest.mark.parametrize("hidden,heads,ffn,S,A,mode", [
    (1040, 5, 330, 12, 5, 0),      # head_dim 208; more columns than one piece of the head's gradient; ffn not a multiple of 4
    (1040, 5, 332, 21, 5, 1),      # ... read rows alone, 10 of them (not a multiple of 4), ffn a multiple of 4 alone
    (32, 2, 48, 508, 4, 0),        # 511 and 513 rows per sequence: both sides of the softmax's register form
    (32, 2, 48, 510, 4, 0),
])
def test_odd_sizes(hidden, heads, ffn, S, A, mode):
    wl = vi.Workload("odd_bw", vi.ModelShape(n_layers=2, hidden=hidden, n_heads=heads, ffn=ffn, vocab=640, dtype="f32"),
                     batch=2, n_patches=S - 2, n_instr=2, n_action=A, mode=mode)
    case, lora, bins, coef, grads, logp = _run(wl, 22, 4, 0.5, max_batch=2, keep=True)
    ref, ref_logp = _oracle(wl, 22, lora, bins, coef, 2, 0.5)
    assert np.max(np.abs(logp - ref_logp)) < 1e-4
    _compare(grads, ref, 2e-4)
