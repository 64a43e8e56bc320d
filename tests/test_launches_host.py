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


# layers, hidden, heads, FFN, environments, keys of the step, repacked weights: what is read past the caches, K and V ("k"), the repacked
# weights ("w").  MB of weights and of K and V behind each.
STEPS = [((4, 1024, 8, 2816, 1, 71, True), ""),          # 103, 1
         ((8, 1024, 8, 2816, 13, 71, True), ""),         # 206, 30
         ((8, 1024, 8, 2816, 64, 71, True), "w"),        # 206, 149
         ((12, 1024, 8, 2816, 1, 71, True), "w"),        # 308, 3
         ((4, 1024, 8, 2816, 64, 290, True), "k"),       # 103, 304
         ((2, 1024, 8, 2816, 256, 61, True), ""),        # 51, 128
         ((4, 4096, 32, 11008, 1, 289, True), "w"),      # 1619, 19 (and so on)
         ((4, 4096, 32, 11008, 13, 289, True), "w"),     # 246
         ((4, 4096, 32, 11008, 16, 289, True), "kw"),    # 303
         ((4, 4096, 32, 11008, 32, 71, True), "w"),      # 149
         ((4, 4096, 32, 11008, 32, 131, True), "kw"),    # 275
         ((4, 4096, 32, 11008, 40, 71, True), "kw"),     # 186, and 495 of O and down, which come through the caches above 32 rows
         ((4, 4096, 32, 11008, 256, 289, True), "tkw"),
         ((4, 4096, 32, 11008, 54, 289, True), "kw"),     # 1023, 256 of one layer without the step's key
         ((4, 4096, 32, 11008, 55, 289, True), "tkw"),
         ((4, 4096, 32, 11008, 4, 289, False), "k"),     # row-major weights come through the caches
         ((1, 4096, 64, 512, 3, 511, False), ""), ((1, 4096, 64, 512, 15, 511, False), "k"),      # (test_gpu_decode_past_caches.py's sizes)
         ((1, 4096, 32, 256, 3, 509, True), ""), ((1, 4096, 32, 256, 31, 509, True), "tk")]
STEP = """
result = []
for L, H, heads, F, B, keys, packed in %r:
    cfg = vb.make_config(shape(L, H, heads, F), B, keys + 1)
    m = model(cfg, packed)
    kv = t(vb.vla_kv_bytes(cfg, B, keys + 1))
    vb.vla_prefill(m.handle, kv, t(vb.vla_workspace_bytes(cfg, 0, B, keys - 1, 0)), t(), t(), B, keys - 2, 1, t(), None)
    before = launches()
    vb.vla_decode_actions(m.handle, kv, t(vb.vla_workspace_bytes(cfg, 1, B, keys - 1, 2)), t(), B, keys - 1, 2, 0, None, 1.0, None, t(), t(), t(), None)
    result.append((before, launches()))
"""


def test_what_a_step_reads_past_the_caches(tmp_path):
    """K and V, and repacked weights, that fit the memory-side cache until the next step reads them again are left to it; the last read row of a
    prefill ("t"), whose K and V the launch before wrote and the first step reads, leaves them there where those of one layer fit."""
    for (case, past), (prefill, step) in zip(STEPS, record(STEP % ([c for c, _ in STEPS],), tmp_path)):
        L, H, heads, F, B, keys, packed = case
        form = f"attn_decode_kernelILi{H // heads}ELi" + ("8ELb1E" if B * heads < 1024 else "4ELb0E")
        assert count(step, form + f"Lb{int('k' in past)}E") == L and count(step, "attn_decode") == L, case
        assert count(prefill, f"attn_decode_kernelILi{H // heads}ELi4ELb0ELb{int('t' in past)}E") == count(prefill, "attn_decode") == 1, case
        if B <= 16:                                  # all four products of a layer are the streaming kernel's: the last argument of its template
            stream = [n for n in step if "gemm_stream" in n]
            assert len(stream) == 4 * L and all(f"ELi{2 if 'w' in past else int(packed)}EEEv" in n for n in stream), case
        elif B <= 128 and packed:                    # QKV or gate/up on the small tiles: the third argument
            small = [n for n in step if "gemm_bf16_small" in n]
            assert small and all(f"ELb0ELi{3 if 'w' in past else 1}E" in n for n in small), case


GENERIC = """
result = []
for dtype, F in (("bf16", 5461), ("bf16", 5460), ("f32", 2731), ("f32", 2732)):
    cfg = vb.make_config(shape(1, 1024, 16, F, dtype), 2, 20)
    m = model(cfg)
    vb.vla_prefill(m.handle, t(vb.vla_kv_bytes(cfg, 2, 20)), t(vb.vla_workspace_bytes(cfg, 0, 2, 12, 0)), t(), t(), 2, 10, 2, t(), None)
    result.append(launches())
"""


def test_blocks_in_flight_of_the_generic_product(tmp_path):
    """A wave of the small tile: its share of K in up to eight blocks where a load brings 16 bytes, else four."""
    for names, blocks in zip(record(GENERIC, tmp_path), ({4}, {4}, {4, 8}, {8})):
        generic = [n for n in names if "gemm_generic" in n]
        assert generic and {b for n in generic for b in (2, 4, 6, 8) if f"ELi1ELi1ELi{b}E" in n} == blocks, names
