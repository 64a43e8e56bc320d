"""vla_debug_force_generic reaches the gradient pass: each bit sends its step to the kernels that any shape takes, as the labels of
the launches show, and the gradients stay within the bounds of test_gpu_backward.py."""
import ctypes

import pytest

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
