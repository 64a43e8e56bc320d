"""vla_debug_force_generic reaches the gradient pass: each bit sends its step to the kernels that any shape takes, as the labels of
the launches show, and the gradients stay within the bounds of test_gpu_backward.py."""
import ctypes

import pytest
import torch

import vla_inputs as vi
from paper_2510_06710_amd import binding as vb
from test_gpu_backward import _assert_logp_bf16, _compare, _oracle, _run

pytestmark = pytest.mark.gpu
SHAPE = vi.ModelShape(n_layers=2, hidden=256, n_heads=2, ffn=512, vocab=640, dtype="bf16")
WL = vi.Workload("triage", SHAPE, batch=3, n_patches=60, n_instr=9, n_action=5, mode=0)


def forced(mask, wl, seed, rank, **kw):
    """test_gpu_backward._run under the mask, and the labels of its launches."""
    vb.vla_debug_force_generic(mask)
    vb.lib().vla_profile_enable(1)
    try:
        out = _run(wl, seed, rank, 0.5, **kw)
        buf = ctypes.create_string_buffer(1 << 16)
        assert vb.lib().vla_profile_report(buf, len(buf)) > 0
    finally:
        vb.lib().vla_profile_enable(0)
        vb.vla_debug_force_generic(0)
    return out, {line.rsplit(" ", 3)[0] for line in buf.value.decode().splitlines()}


# keep: no label of the recompute's own forward beside those of the gradient pass
@pytest.mark.parametrize("mask,gone,there", [(1, ("lora_products",), ()), (4, ("bw_attention_rows",), ("lora_products", "bw_attention_mfma")),
                                             (16, ("<qkv_rope>", "<swiglu>"), ("lora_products", "bw_attention_rows"))])
def test_a_bit_sends_its_step_to_the_general_kernels(mask, gone, there):
    _, usual = forced(0, WL, 11, 16, keep=True)
    (_, lora, bins, coef, grads, logp), labels = forced(mask, WL, 11, 16, keep=True)
    for part in gone:
        assert any(part in x for x in usual) and not any(part in x for x in labels), (part, usual, labels)
    assert set(there) <= labels
    ref, ref_logp = _oracle(WL, 11, lora, bins, coef, WL.batch, 0.5, operand_dtype="bf16")
    _assert_logp_bf16(logp, ref_logp)
    print(_compare(grads, ref, 2e-2, 1e-2), flush=True)


# (an FFN width that is no multiple of 128: the gate / up product and SwiGLU are separate either way; a multiple of 256: both forms
# take the product from the same tiles)
@pytest.mark.parametrize("n,hidden,ffn,S,A,mode", [(37, 2048, 320, 92, 8, 0), (4, 256, 320, 30, 40, 1),
                                                   (3, 512, 768, 69, 5, 0),          # small tiles, the top layer on its read rows
                                                   (37, 2048, 2304, 92, 8, 0),       # large tiles
                                                   (4, 256, 512, 30, 40, 1)])        # every row through the top layer
def test_epilogues_give_the_bits_of_the_separate_passes(n, hidden, ffn, S, A, mode):
    """Rotation and SwiGLU on the way out of their projections round and evaluate as the kernels that take the shapes those decline:
    which of the two a model's widths select cannot be seen in its gradients."""
    shape = vi.ModelShape(n_layers=2, hidden=hidden, n_heads=hidden // 128, ffn=ffn, vocab=640, dtype="bf16")
    wl = vi.Workload("epilogues", shape, batch=n, n_patches=S - 9, n_instr=9, n_action=A, mode=mode)
    usual, apart = (forced(mask, wl, 13, 8, keep=True)[0] for mask in (0, 16))
    assert torch.equal(torch.from_numpy(usual[5]), torch.from_numpy(apart[5]))
    differ = {(l, p): max(float((x != y).float().mean()) for x, y in zip(a[p], b[p]))
              for l, (a, b) in enumerate(zip(usual[4], apart[4])) for p in a}
    assert not any(differ.values()), differ
