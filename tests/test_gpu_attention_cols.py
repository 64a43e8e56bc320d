"""The contractions over the queries of the gradient pass's attention (d V, d K), with the transposed rotation and the rounding of all three
gradients, by themselves against 64 bits: one wave's 32 keys and its edges, a workgroup's 128, queries in steps of 32, the top layer's few
read rows, rows that see every key, more rows than the by-rows kernels take.

Bounds.  Before the last rounding: head + tail leave out at most 2^-17 of an operand's element, both operands 2^-16 of a product, and the sums
are fp32.  The output is bf16: relative RMS at most 2^-9, and of the elements at most 1 % take the other neighbour than the exact value
does (2^-16 over half the spacing, 2^-9, is 0.8 % at the worst; where terms cancel, a rotation's among them, the error counts against the
terms and not against their sum: elements below 2^-6 of the RMS are left out of the count)."""
import ctypes

import pytest
import torch

from paper_2510_06710_amd import binding as vb
from test_gpu_attention_rows import CAUSAL, D, _inputs, _rel

pytestmark = pytest.mark.gpu


class AttnColsArgs(ctypes.Structure):               # csrc/vla_internal.h
    _fields_ = [(n, ctypes.c_void_p) for n in ("P", "dS", "dO", "dq", "qkv", "table", "out_q", "out_k")] + \
               [(n, ctypes.c_int) for n in ("ld_q", "ld_kv", "q_packed", "R", "Rq", "ldp", "n_heads", "H", "full_from")] + [("scale", ctypes.c_float)]


def _call(n, **fields):
    fn = getattr(vb.lib(), "_Z18try_attention_colsRK12AttnColsArgsiP12ihipStream_t")
    fn.argtypes = [ctypes.POINTER(AttnColsArgs), ctypes.c_int, ctypes.c_void_p]
    args = AttnColsArgs(**{k: v.data_ptr() if torch.is_tensor(v) else v for k, v in fields.items()})
    rc = fn(ctypes.byref(args), n, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return rc


@pytest.mark.parametrize("R,Rq,full_from,heads", [(1, 1, CAUSAL, 1), (31, 31, CAUSAL, 3), (33, 33, 20, 2), (64, 7, CAUSAL, 3), (129, 129, 97, 8), (161, 161, CAUSAL, 2),
                                                  (294, 294, CAUSAL, 9), (294, 7, CAUSAL, 3), (315, 80, 236, 2), (330, 330, CAUSAL, 1)])
def test_kernel(R, Rq, full_from, heads):
    n, H, ldp, scale, first = 2, heads * D, (R + 3) // 4 * 4, D ** -0.5, R - Rq
    g, qkv, q, k, v, mask = _inputs(n, R, Rq, full_from, heads)
    rand = lambda *z: torch.randn(*z, device="cuda:0", generator=g)  # noqa: E731
    dO, dq = rand(n, Rq, heads, D), rand(n, R, 3, heads, D)
    if first:
        dq[:, :first] = torch.nan                    # no queries there: not read
    P = torch.full((n, heads, Rq, ldp), torch.nan, device="cuda:0")
    dS = P.clone()
    P[..., :R] = (q @ k.transpose(2, 3) * scale).masked_fill(~mask, -torch.inf).softmax(-1)
    dS[..., :R] = rand(n, heads, Rq, R) * P[..., :R]
    ang = torch.arange(R, device="cuda:0", dtype=torch.float64)[:, None] * 10000.0 ** (-torch.arange(0, D, 2, device="cuda:0", dtype=torch.float64) / D)
    table = torch.stack((ang.cos(), ang.sin()), -1).float().contiguous()
    out = torch.full((n, R, 3, heads, D), 9.0, device="cuda:0").bfloat16()
    assert _call(n, P=P, dS=dS, dO=dO, dq=dq, qkv=qkv, table=table, out_q=out, out_k=out[:, :, 1:], ld_q=3 * H, ld_kv=3 * H, q_packed=0, R=R, Rq=Rq, ldp=ldp, n_heads=heads, H=H, full_from=full_from, scale=scale) == 1

    def back(x):                                     # [n, R, heads, D], the transposed rotation
        co, si = table[:, None, :, 0].double(), -table[:, None, :, 1].double()
        a, b = x[..., :64], x[..., 64:]
        return torch.cat((a * co - b * si, b * co + a * si), -1)

    want_v = (P[..., :R].double().transpose(2, 3) @ dO.double().transpose(1, 2).contiguous()).transpose(1, 2)
    want_k = back(((dS[..., :R].double().transpose(2, 3) @ q) * scale).transpose(1, 2))
    want_q = back(dq[:, :, 0].double().nan_to_num(0.0))
    for name, got, want in (("dq", out[:, :, 0], want_q), ("dk", out[:, :, 1], want_k), ("dv", out[:, :, 2], want_v)):
        counted = want.abs() > 2.0 ** -6 * want.square().mean().sqrt()
        flips = float((got != want.bfloat16())[counted].double().mean())
        print(f"{name}: {_rel(got, want):.2e}, {100 * flips:.3f} % round the other way", flush=True)
        assert _rel(got, want) <= 2.0 ** -9 and flips <= 0.01
    assert not out[:, :first, 0].any()
    apart, packed = torch.full((n, R, 2, heads, D), 9.0, device="cuda:0").bfloat16(), torch.full((n, Rq, heads, D), 9.0, device="cuda:0").bfloat16()
    assert _call(n, P=P, dS=dS, dO=dO, dq=dq, qkv=qkv, table=table, out_q=packed, out_k=apart, ld_q=H, ld_kv=2 * H, q_packed=1, R=R, Rq=Rq, ldp=ldp, n_heads=heads, H=H,
                 full_from=full_from, scale=scale) == 1
    assert torch.equal(apart, out[:, :, 1:]) and torch.equal(packed, out[:, first:, 0])


def test_declined():
    """head_dim 64, and rows that do not end on 16 bytes."""
    z = torch.zeros(1 << 16, device="cuda:0")
    common = dict(P=z, dS=z, dO=z, dq=z, qkv=z, table=z, out_q=z, out_k=z, ld_q=384, ld_kv=384, q_packed=0, R=6, Rq=6, n_heads=2, full_from=CAUSAL, scale=1.0)
    assert _call(1, **common, ldp=8, H=128) == 0 and _call(1, **common, ldp=6, H=256) == 0 and _call(1, **common, ldp=4, H=256) == 0
