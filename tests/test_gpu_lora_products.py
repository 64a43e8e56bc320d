"""The one-pass LoRA products of bf16 models around their edges: ranks on both sides of a block of 16 factor rows, more than 128
factor rows in a group (the padded GEMM form takes that group), a width whose last 512-column chunk is partial, fewer rows
than a block of 16, rows that end inside a step of 32, two micro-batches.  Against the fp64 oracle with the bounds of
test_gpu_backward.py."""
import pytest

import vla_inputs as vi
from test_gpu_backward import _assert_logp_bf16, _compare, _oracle, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank,batch,max_batch,S,A,hidden,ffn", [
    (1, 1, 1, 9, 3, 256, 512),             # 11 rows
    (15, 2, 2, 13, 5, 256, 640),
    (17, 3, 3, 30, 4, 256, 640),           # 99 rows and 12 read ones
    (32, 3, 2, 33, 4, 384, 1152),
    (33, 2, 2, 40, 20, 256, 512),          # nine blocks in the q | k | v group
    (64, 2, 2, 40, 4, 256, 512),
])
def test_ranks_and_rows(rank, batch, max_batch, S, A, hidden, ffn):
    shape = vi.ModelShape(n_layers=2, hidden=hidden, n_heads=hidden // 128, ffn=ffn, vocab=640, dtype="bf16")
    wl = vi.Workload("lora", shape, batch=batch, n_patches=S - 4, n_instr=4, n_action=A, mode=0)
    case, lora, bins, coef, grads, logp = _run(wl, 31, rank, 0.5, max_batch=max_batch)
    ref, ref_logp = _oracle(wl, 31, lora, bins, coef, batch, 0.5, operand_dtype="bf16")
    _assert_logp_bf16(logp, ref_logp)
    # The relative RMS of a tensor averages over rank x width entries whose errors are independent across the factor rows only
    # (one row of dA is a sum over the same few rounded dY B): with one factor row and three token rows there is no such averaging,
    # and a tensor may be off by twice the bar (0.0149 here, and 0.0149 with the padded GEMM form, equal to six digits).
    print(_compare(grads, ref, 2e-2, 2e-2 if rank == 1 else 1e-2), flush=True)
