"""Which kernels the calls enqueue (tests/launches.py): routes that a size or an alignment decides, on any machine."""
import pytest

from launches import record


def count(names, part):
    return sum(part in n for n in names)


# the workspace's offset from a multiple of 256 bytes; read rows: 4 of 63 (the top layer works on those alone), 20 of 79
BACKWARD = """
result = []
cfg = vb.make_config(shape(2, 256, 2, 512), 4, 100)
m = model(cfg)
lora = [{p: (t(), t()) for p in vb.LORA_PROJECTIONS} for _ in range(2)]
for off in (0, 4, 8, 16):
    for keep in (0, 1):
        for A in (4, 20):
            size = (vb.vla_backward_keep_workspace_bytes if keep else vb.vla_backward_workspace_bytes)(cfg, 3, 60, A, 8)
            try:
                vb.vla_logprob_backward(m.handle, t(size, off), t(), t(), t(), t(), 3, 57, 3, A, 0, None, 1.0, 8, 0.5, keep, lora, lora, t())
                error = None
            except vb.VlaError as e:
                error = str(e)
            result.append((off, keep, A, error, launches()))
"""


def test_gradient_pass_takes_any_workspace(tmp_path):
    """vla.h asks for no alignment of the workspace: off 16 bytes the attention's gradient goes to the batched products, in the top layer too."""
    for off, keep, A, error, names in record(BACKWARD, tmp_path):
        assert error is None, (off, keep, A, error)
        assert count(names, "attn_cols_kernel") == (2 if off % 16 == 0 else 0), (off, keep, A)
        assert (count(names, "rope_rows_kernel") > 0) == (off % 16 != 0), (off, keep, A)


NARROW = """
cfg = vb.make_config(shape(2, 1024, 8, 64), 8, 100)
m = model(cfg)
lora = [{p: (t(), t()) for p in vb.LORA_PROJECTIONS} for _ in range(2)]
result = []
for keep in (0, 1):
    size = (vb.vla_backward_keep_workspace_bytes if keep else vb.vla_backward_workspace_bytes)(cfg, 8, 60, 15, 8)
    ws, out = t(size), {}
    for part in ("gather_rows", "rmsnorm_bwd"):
        rt.watch(part.encode())
        vb.vla_logprob_backward(m.handle, ws, t(), t(), t(), t(), 8, 57, 3, 15, 0, None, 1.0, 8, 0.5, keep, lora, lora, t())
        out[part] = [[int(a) for a in n.split()[1:]] for n in launches() if part in n]
    result.append(out)
"""


def test_read_rows_of_the_norm_stay_in_their_buffer(tmp_path):
    """FFN 64 of hidden 1024: the top layer's 8 x 15 read rows of the norm are longer than its SwiGLU gradient, behind which d x lies in the
    storage type (the second argument of the norm's gradient)."""
    for out in record(NARROW, tmp_path):
        dxb = {a[1] for a in out["rmsnorm_bwd"]}
        assert len(dxb) == 1 and out["gather_rows"]
        for dst, _ in out["gather_rows"]:
            assert not any(dst < x < dst + 8 * 15 * 1024 * 2 for x in dxb)
