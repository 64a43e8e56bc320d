"""The gradient pass's projections finish in their GEMM's epilogue (rotation; SwiGLU with its pre-activations kept), in tiles chosen
by the row count.  A rollout's rows do not depend on the tile, so the gradients of many rollouts at once (large tiles of 160 to 256
rows, ragged last ones) are the sums of those of passes of one or three (small tiles).  The fp32 sums over at most 5000 rows in
another grouping differ by about sqrt(5000) 2^-24 / 4 = 1e-6 of the largest entry; 2e-5 as in the micro-batch test in fp32.  With
the activations kept, or where the top layer's have room beside those of the layer below at either size of a micro-batch (not at one
rollout): the number of layers whose first forward is the log-prob recompute's depends on it, and bf16 rounding then differs (5e-3)."""
import pytest

import vla_inputs as vi
from test_gpu_backward import _run
from oracle import backward_oracle as bo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,few,hidden,ffn,layers,keep", [(50, 1, 2048, 2176, 2, True), (37, 3, 2048, 2176, 2, True), (24, 1, 512, 640, 2, True),
                                                          (37, 3, 2048, 2176, 3, False)])
def test_many_rollouts_are_the_sum_of_few(n, few, hidden, ffn, layers, keep):
    shape = vi.ModelShape(n_layers=layers, hidden=hidden, n_heads=hidden // 128, ffn=ffn, vocab=640, dtype="bf16")
    wl = vi.Workload("rows_bw", shape, batch=n, n_patches=83, n_instr=9, n_action=8)
    many = _run(wl, 7, rank=16, scale=0.5, keep=keep)[4]
    parts = _run(wl, 7, rank=16, scale=0.5, max_batch=few, keep=keep)[4]
    for a, b in zip(many, parts):
        for p in bo.PROJ:
            for x, y in zip(a[p], b[p]):
                assert float((x - y).abs().max()) <= 2e-5 * float(x.abs().max()), p
