"""Input gradients C = A . [W0; W1; ..] on weights as they lie ([K, N] each): the same products on the same matrix operands in the same
order as on a transposed copy, so the same bits, in every tile (40 to 1400 rows: 64 to 160 rows of 64 and 128 columns, 128 x 128 with one and
two workgroups per CU; more: the large ones), with segments of K that end after four pairs of half tiles, the least, and after five."""
import ctypes

import pytest
import torch

from paper_2510_06710_amd import binding as vb

pytestmark = pytest.mark.gpu


class GemmArgs(ctypes.Structure):                   # csrc/vla_internal.h
    _fields_ = [("A", ctypes.c_void_p), ("W", ctypes.c_void_p * 3), ("Wkb", ctypes.c_void_p * 3), ("n_seg", ctypes.c_int), ("segN", ctypes.c_int),
                ("C", ctypes.c_void_p), ("res", ctypes.c_void_p), ("M", ctypes.c_int), ("K", ctypes.c_int), ("epilogue", ctypes.c_int),
                ("rope", ctypes.c_void_p), ("pre", ctypes.c_void_p), ("kblocked", ctypes.c_int), ("a_rows", ctypes.c_int), ("step", ctypes.c_int),
                ("norm_x", ctypes.c_void_p), ("norm_gain", ctypes.c_void_p), ("norm_eps", ctypes.c_float), ("deferred_splits", ctypes.c_void_p),
                ("segK", ctypes.c_int), ("split_scratch", ctypes.c_void_p), ("split_scratch_bytes", ctypes.c_size_t)]


def _gemm(A, W, out, M, N, segK=0, **fields):
    """1 if the kernels took the product."""
    fn = getattr(vb.lib(), "_Z17try_gemm_bf16_dmaRK8GemmArgsP12ihipStream_t")
    fn.argtypes = [ctypes.POINTER(GemmArgs), ctypes.c_void_p]
    g = GemmArgs(n_seg=len(W), segN=N, M=M, K=A.shape[1], a_rows=A.shape[0], segK=segK, A=A.data_ptr(), C=out.data_ptr(), **fields)
    for i, w in enumerate(W):
        g.W[i] = w.data_ptr()
    rc = fn(ctypes.byref(g), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return rc


@pytest.mark.parametrize("M,N,n_seg,segK", [(1, 256, 1, 256), (40, 256, 3, 256), (65, 512, 2, 320), (300, 3584, 1, 1024), (315, 4096, 1, 1024), (400, 4096, 1, 1024), (600, 4096, 2, 512),
                                            (700, 4096, 1, 1024), (288, 12288, 1, 1024), (193, 12288, 3, 512),
                                            (900, 4096, 1, 1088), (1400, 4096, 3, 320), (2304, 4096, 2, 256), (3000, 4096, 2, 320), (3390, 4096, 3, 256),
                                            (4095, 4096, 1, 256), (5000, 1024, 1, 576), (7150, 1280, 3, 320)])
def test_same_bits_as_on_transposed_weights(M, N, n_seg, segK):
    g = torch.Generator(device="cuda:0").manual_seed(M + N)
    A = torch.randn((M + 255) // 256 * 256 + 32, n_seg * segK, device="cuda:0", generator=g).bfloat16()
    W = torch.randn(n_seg * segK, N, device="cuda:0", generator=g).bfloat16()
    got, want = torch.full((2, M + 1, N), 9.0, device="cuda:0")
    assert _gemm(A, [w.clone() for w in W.split(segK)], got, M, N, segK) == 1
    assert _gemm(A, [W.T.contiguous()], want, M, N) == 1
    exact = A[:M].double() @ W.double()
    assert torch.equal(got, want) and (got[M] == 9.0).all()
    assert float((got[:M].double() - exact).norm() / exact.norm()) <= (n_seg * segK) ** 0.5 * 2.0 ** -23


@pytest.mark.parametrize("M,N,K", [(1, 256, 256), (70, 512, 320), (300, 4096, 1024), (700, 4096, 1024), (288, 12288, 1024), (900, 4096, 1088), (1400, 4096, 320),
                                   (2304, 4096, 256), (3000, 4096, 320), (3390, 4096, 256), (4095, 4096, 256)])
def test_swiglu_gradient_in_the_epilogue(M, N, K):
    """d gate | d up of the product and given pre-activations, against 64 bits on the product as it leaves the plain epilogue (the same
    bits): a few fp32 roundings (of 2^-24, and 2 ulp of the exponential) and the rounding to bf16, which at most one element in 2^9 of them
    takes the other way (an error of 2^-18 or less over half the spacing, 2^-9)."""
    g = torch.Generator(device="cuda:0").manual_seed(M + N)
    A = torch.randn((M + 255) // 256 * 256 + 32, K, device="cuda:0", generator=g).bfloat16()
    W = (torch.randn(K, N, device="cuda:0", generator=g) / 8).bfloat16()
    pre = 2.0 * torch.randn(M, 2 * N, device="cuda:0", generator=g)
    d_act, got = torch.empty(M, N, device="cuda:0"), torch.full((M + 1, 2 * N), 9.0, device="cuda:0").bfloat16()
    assert _gemm(A, [W], d_act, M, N, K) == 1
    assert _gemm(A, [W], got, M, N, K, epilogue=6, pre=pre.data_ptr()) == 1
    gate, up, d = pre[:, :N].double(), pre[:, N:].double(), d_act.double()
    s = gate.sigmoid()
    want = torch.cat((d * up * s * (1.0 + gate * (1.0 - s)), d * gate * s), 1)
    # (silu' has a zero, near which the error counts against the terms: those elements are left out of the count)
    counted = torch.cat(((1.0 + gate * (1.0 - s)).abs() > 2.0 ** -4, gate.abs() > 0), 1)
    flips = float((got[:M] != want.bfloat16())[counted].double().mean())
    assert (got[M] == 9.0).all() and flips <= 2.0 ** -9 and float((got[:M].double() - want).norm() / want.norm()) <= 2.0 ** -8, flips
    assert _gemm(A, [W], got, M, N, epilogue=6, pre=pre.data_ptr()) == 0          # on transposed weights: not offered


def test_declined():
    """Columns that are no multiple of 256, segments of no multiple of 64 or below 256 rows, weights off 16 bytes."""
    A = torch.zeros(288, 512, device="cuda:0").bfloat16()
    W, out = torch.zeros(512 * 256 + 8, device="cuda:0").bfloat16(), torch.zeros(32, 512, device="cuda:0")
    assert _gemm(A, [W], out, 8, 128, 512) == 0 and _gemm(A, [W, W], out, 8, 256, 192) == 0 and _gemm(A, [W, W], out, 8, 256, 128) == 0
    assert _gemm(A, [W[4:]], out, 8, 256, 512) == 0 and _gemm(A, [W], out, 8, 256, 256) == 0
