// bf16 MFMA GEMM for gfx950 with direct-to-LDS loads: C[M, N] = A[M, K] . W[N, K]^T, fp32 accumulation.
// This is the kernel of the prefill / recompute / parallel-chunk projections (whole tiles), and, with K cut into
// equal ranges whose fp32 partial products go to a scratch buffer, of the QKV and gate/up projections of decode
// forwards of 129..256 rows.
//
// Tiling: 256 x 256 output tiles (or 32 MB x 256, MB = 5 .. 7, see choose_tile), 4 waves (one per SIMD), 128 x 128 per wave as 8 x 8
// blocks of v_mfma_f32_16x16x32_bf16 (256 fp32 accumulators per lane).  The weight rows are the MFMA's row
// operand and the activation rows its column operand: a lane ends up with activation row (lane % 16) of
// a block and four consecutive output columns.
//
// K moves in half tiles of 32 through a ring of five 32 KB LDS stages (all 160 KB).  `buffer_load ... lds` writes
// the operands straight into LDS (no staging registers, no ds_write): a wave instruction fills 1 KB
// linearly, i.e. 16 tile rows of 64 bytes; chunk c (16 bytes) of row r sits at position
// c ^ ((r >> 1) & 3), chosen on the global side by which chunk a lane fetches, so that the fragment
// reads are free of bank conflicts: a ds_read_b128 is served eight lanes (128 bytes) at a time, and the eight
// 64-byte rows of such a group then cover the eight 16-byte slots of 128 bytes (with (r >> 2) & 3, which would
// suit 256 bytes per step, SQ_LDS_BANK_CONFLICT showed every read taking twice as long).
//
// Schedule.  Half tile g is read into fragment buffer g % 2 while half tile g - 1 multiplies from the other buffer.  One
// barrier per pair of half tiles (g even): before it each wave waits for its loads of g and g + 1 (those of g + 2, eight
// instructions, may still be in flight), after it the stages of g - 2 and g - 1 are free for g + 3 and g + 4, whose loads are
// spread evenly over the pair.  With one wave per SIMD whatever the wave issues between two MFMAs beyond 12 cycles leaves the
// matrix pipe idle, so the loop holds no branch but its own and at most one other instruction, or a load with its two
// scalar ones, after an MFMA: the fragment reads after every second MFMA of a half tile's first 32, the loads after every
// eighth; consecutive loads differ in the instruction's own offset, and the cursor's step to the next tile is outside.  At
// 73,728 rows of the 7B shape, against the same tiles with the loads and their branches in clusters between groups of four
// MFMAs: QKV 5.33 -> 4.80 ms (1420 TFLOP/s), O and down 3.46 -> 3.12 on average, gate/up 10.0 -> 8.8 (1515; the vendor
// library's product of the same shape 1509).  A barrier per half tile with a ring of four: 1.5 % slower; a barrier per pair
// with a ring of four, 16 loads in the pair's first half: 6 %; loads after every fourth or sixth MFMA, reads after every third: the same.
//
// The fragment reads, and the MFMAs with them, are inline assembly with explicit waits: the compiler would otherwise wait for
// every outstanding LDS-bound load before any LDS read, and copies the accumulators where two paths meet.
//
// Operand layout.  In the k-blocked layout (KB: [K / 32][rows][32] for the activations and for repacked weights) a half tile
// of 256 rows is one contiguous 16 KB block and every instruction reads 1 KB of whole lines; the SwiGLU output is then written
// k-blocked as well.  Row-major operands are fetched as whole 128-byte lines too, 8 rows an instruction: a stage then holds both
// half tiles of a pair for half of the tile's rows instead of one half tile of all rows.  (As 64-byte pieces of 16 rows, streaming
// alone runs at 46-53 GB/s per CU where lines reach 65-84.  9,408 rows, fp32 output: 940 -> 817 us on average over the
// gradient products of the 7B shape.)
//
// The gradient of a product's input contracts over the weights' rows: its operands need eight of those rows per column.  The weights
// are read as they lie ([K, N]: runs of 256 bytes, of 128 in 64 x 64 tiles) and transposed on the way out of LDS (ds_read_b64_tr_b16, two for
// the eight rows that a row-major operand's one read brings): the same operands in the same order, the same bits as on transposed copies of the
// weights, without the copies.  us with them and so, weights from memory, 2 x 11008 rows onto 4096 columns: 49 rows 152 + 66 and 148, 1,000 266 +
// 66 and 246, 9,408 1368 + 66 and 1412; 4096 onto 11008: 34 + 30 and 35, 97 + 30 and 93, 671 + 30 and 714.
//
// One workgroup per CU walks its tiles in turn (tile i of a workgroup = id + grid * i, which keeps the
// XCD-contiguous tile order); the half-tile stream simply continues into the next tile, so that only the
// first tile pays an empty pipeline.  A tile's last MFMAs run in the next tile's first iteration, whose loads go out as
// usual; the epilogue follows that iteration and uses the LDS stage just read as its staging panel, and the next
// tile's sums start with an MFMA that adds to zero.
#include "vla_internal.h"

#include <type_traits>
#include <utility>

namespace {

constexpr int BM = 256, BN = 256, HK = 32;
constexpr int REGION = 256 * HK * 2;     // 16 KB per operand per stage
constexpr int STAGE = 2 * REGION;        // 32 KB
constexpr int NSTAGES = 5;

typedef __attribute__((address_space(3))) void lds_void;
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x2_t __attribute__((ext_vector_type(2)));

// How the weights lie: rows of K, k-blocked, or (EPI_STORE) as [K, N], for the gradient of a product's input.
// W_KBLOCKED_PAST (decode steps): k-blocked, read past the caches.
enum WeightLayout { W_ROWS = 0, W_KBLOCKED = 1, W_COLUMNS = 2, W_KBLOCKED_PAST = 3 };

struct DmaGemmParams {
    const bf16_t *A;
    const bf16_t *W0, *W1, *W2;
    void *C;
    const float *res;   // EPI_RESIDUAL: what the product is added to
    int M, N, K, segN;
    int tiles_m, tiles_n;
    int a_rows;      // k-blocked layout: rows per 32-column block of A (and of the SwiGLU output)
    int w_rows;      // k-blocked layout: rows per 32-column block of each weight matrix
    int segK;        // W_COLUMNS: rows of K per weight segment
    // EPI_QKV_ROPE, EPI_QKV_ROWS
    bf16_t *q_out, *kc, *vc;
    float *pre;      // EPI_SWIGLU_KEEP, EPI_SWIGLU_GRAD
    const float2 *table;
    int R, pos0, n_heads, pos_stride, H;
    int seg0;        // EPI_QKV_ROPE, EPI_QKV_ROWS: what the first weight segment is (0 = q, k, v follow; 1 = k, v only)
    int group;
    int splits;      // > 1: K is cut into `splits` equal ranges; item = range * tiles + tile, and range r of an
                     // EPI_STORE launch writes its fp32 partial product to C + r * M * N
    int parts;       // small tiles of a decode step: the parts of K whose sums are added in order (gemm_decode_parts)
};

template <int OFF>
__device__ __forceinline__ bf16x8_t lds_read(int addr) {
    i32x4_t v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return __builtin_bit_cast(bf16x8_t, v);
}

// W_COLUMNS: eight rows of K of 16 columns, transposed on the way: of 16 lanes, lane l names four columns 4 (l % 4) .. of row l / 4 and gets
// the four rows of column l, from OFF rows 0 .. 3 of its eight and from OFF + STEP rows 4 .. 7.  The halves become one operand only behind the
// wait, so that no copy of a register still to be written comes in between.
struct ColumnFrag { i32x2_t lo, hi; };
template <int OFF, int STEP>
__device__ __forceinline__ ColumnFrag lds_read_columns(int addr) {
    ColumnFrag f;
    asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4" : "=&v"(f.lo), "=&v"(f.hi) : "v"(addr), "n"(OFF), "n"(OFF + STEP));
    return f;
}
__device__ __forceinline__ bf16x8_t frag_of(const ColumnFrag &f) {
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(f.lo, f.hi, 0, 1, 2, 3));
}
__device__ __forceinline__ bf16x8_t frag_of(const bf16x8_t &f) { return f; }

// One accumulator element, moved out of its accumulation register exactly where the epilogue consumes it
// (left to the compiler all 256 moves are hoisted to the top of the epilogue and spill the fragments that
// are live across it).
__device__ __forceinline__ float acc_read(const f32x4_t &v, int e) {
    float x;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(v[e]));
    return x;
}
__device__ __forceinline__ f32x4_t acc_read4(const f32x4_t &v) {
    f32x4_t o;
#pragma unroll
    for (int e = 0; e < 4; e++) o[e] = acc_read(v, e);
    return o;
}
// The matrix pipe's last results must have landed before the first such move (the assembler text is
// opaque to the compiler's hazard handling).
__device__ __forceinline__ void acc_settle() { asm volatile("s_nop 15\n\ts_nop 15"); }

// Epilogue staging panel of one wave: 16 rows x 128 fp32 = 8 KB, no padding; the 16-byte column block cb
// of row r sits at block cb ^ r, which keeps both the column-wise writes (16 lanes = 16 rows) and the
// row-wise reads free of bank conflicts.
__device__ __forceinline__ float *panel_at(float *panel, int row, int cb) { return panel + row * 128 + ((cb ^ row) << 2); }

// The panel is read and written by assembly: the next tile's loads are on their way into other stages meanwhile, and the
// compiler would wait for every LDS-bound load before each access it knows of.
__device__ __forceinline__ int lds_addr(const void *p) { return (int)(size_t)(lds_void *)p; }
__device__ __forceinline__ f32x4_t panel_get(float *panel, int row, int cb) {
    f32x4_t v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(lds_addr(panel_at(panel, row, cb))) : "memory");
    return v;
}
__device__ __forceinline__ void panel_put(float *panel, int row, int cb, f32x4_t v) {
    asm volatile("ds_write_b128 %0, %1" ::"v"(lds_addr(panel_at(panel, row, cb))), "v"(v) : "memory");
}
__device__ __forceinline__ void panel_put_acc(float *panel, int row, int cb, const f32x4_t &v) {
    asm volatile("ds_write_b128 %0, %1" ::"v"(lds_addr(panel_at(panel, row, cb))), "a"(v) : "memory");
}
__device__ __forceinline__ void panel_written() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// everything read so far has landed; what is read passes through, so that no use moves above the wait
template <int N>
__device__ __forceinline__ void panel_wait(f32x4_t (&v)[N]) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < N; i++) asm volatile("" : "+v"(v[i]));
}

// One 16-row block of a wave's QKV output, from its panel: the wave's 128 columns are one head of q, k or v (head_dim 128).  ROWS: all
// three go to q_out as rows of 3H.
template <bool ROWS>
__device__ __forceinline__ void qkv_block_out(const DmaGemmParams &p, float *panel, int mblock, int n0, int lane) {
    const int seg_in = n0 / p.H, head = (n0 - seg_in * p.H) >> 7, seg = seg_in + p.seg0;
    f32x4_t v[8];
    if (seg == 2) {
#pragma unroll
        for (int it = 0; it < 4; it++) {
            const int row = it * 4 + (lane >> 4), c = lane & 15;
            v[2 * it] = panel_get(panel, row, 2 * c);
            v[2 * it + 1] = panel_get(panel, row, 2 * c + 1);
        }
        panel_wait(v);
#pragma unroll
        for (int it = 0; it < 4; it++) {
            const int row = it * 4 + (lane >> 4), c = lane & 15, m = mblock + row;
            bf16x8_t o;
#pragma unroll
            for (int e = 0; e < 4; e++) { o[e] = (bf16_t)v[2 * it][e]; o[4 + e] = (bf16_t)v[2 * it + 1][e]; }
            if (m < p.M) {
                const int sq = m / p.R, pos = p.pos0 + (m - sq * p.R);
                if (ROWS) *(bf16x8_t *)(p.q_out + (size_t)m * 3 * p.H + 2 * p.H + head * 128 + c * 8) = o;
                else *(bf16x8_t *)(p.vc + (((size_t)sq * p.n_heads + head) * p.pos_stride + pos) * 128 + c * 8) = o;
            }
        }
    } else {
        f32x4_t cs[2][4];
#pragma unroll
        for (int it = 0; it < 2; it++) {
            // q: consecutive lanes take consecutive chunks of a row; k: consecutive positions of a chunk
            const int item = it * 64 + lane;
            const int row = (ROWS || seg == 0) ? (item >> 3) : (item & 15);
            const int c = (ROWS || seg == 0) ? (item & 7) : (item >> 4);
            // (cos, sin) of the chunk's eight dims, two per piece, on their way while the panel is read
            const f32x4_t *tb = (const f32x4_t *)(p.table + (size_t)((mblock + row) % p.R) * 64 + c * 8);
#pragma unroll
            for (int e2 = 0; e2 < 4; e2++) cs[it][e2] = tb[e2];
            v[4 * it] = panel_get(panel, row, 2 * c);
            v[4 * it + 1] = panel_get(panel, row, 2 * c + 1);
            v[4 * it + 2] = panel_get(panel, row, 16 + 2 * c);
            v[4 * it + 3] = panel_get(panel, row, 17 + 2 * c);
        }
        panel_wait(v);
#pragma unroll
        for (int it = 0; it < 2; it++) {
            const int item = it * 64 + lane;
            const int row = (ROWS || seg == 0) ? (item >> 3) : (item & 15);
            const int c = (ROWS || seg == 0) ? (item & 7) : (item >> 4);
            const int m = mblock + row;
            const f32x4_t lo0 = v[4 * it], lo1 = v[4 * it + 1], hi0 = v[4 * it + 2], hi1 = v[4 * it + 3];
            if (m < p.M) {
                const int sq = m / p.R, rr = m - sq * p.R, pos = p.pos0 + rr;
                bf16x8_t olo, ohi;
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const float co = cs[it][e >> 1][2 * (e & 1)], si = cs[it][e >> 1][2 * (e & 1) + 1];
                    const float a = e < 4 ? lo0[e & 3] : lo1[e & 3], b = e < 4 ? hi0[e & 3] : hi1[e & 3];
                    olo[e] = (bf16_t)(ROWS ? vla_rotate_lo(a, b, co, si) : a * co - b * si);      // (ROWS: as rope_rows_kernel rounds)
                    ohi[e] = (bf16_t)(ROWS ? vla_rotate_hi(a, b, co, si) : b * co + a * si);
                }
                if (ROWS || seg == 0) {
                    bf16_t *q = p.q_out + (ROWS ? (size_t)m * 3 * p.H + seg * p.H : (size_t)m * p.H) + head * 128 + c * 8;
                    *(bf16x8_t *)q = olo;
                    *(bf16x8_t *)(q + 64) = ohi;
                } else {
                    const size_t hb = ((size_t)sq * p.n_heads + head) * 16;
                    *(bf16x8_t *)(p.kc + ((hb + c) * p.pos_stride + pos) * 8) = olo;
                    *(bf16x8_t *)(p.kc + ((hb + 8 + c) * p.pos_stride + pos) * 8) = ohi;
                }
            }
        }
    }
}

// One 16-row block of a wave's 64 SwiGLU output columns from c0 = tn * 128 + wn * 64, from its panel: row-major [M, N], or
// k-blocked: column c of row m at ((c / 32) * a_rows + m) * 32 + c % 32.
template <bool KB>
__device__ __forceinline__ void swiglu_block_out(const DmaGemmParams &p, float *panel, int mblock, int c0, int lane) {
    c0 += (lane & 7) * 8;
    bf16_t *out = (bf16_t *)p.C + (KB ? (size_t)(c0 >> 5) * p.a_rows * 32 + (c0 & 31) : (size_t)c0);
    const size_t row_stride = KB ? 32 : (size_t)p.N;
    f32x4_t v[4];
#pragma unroll
    for (int it = 0; it < 2; it++) {
        const int row = it * 8 + (lane >> 3), c2 = lane & 7;
        v[2 * it] = panel_get(panel, row, 2 * c2);
        v[2 * it + 1] = panel_get(panel, row, 2 * c2 + 1);
    }
    panel_wait(v);
#pragma unroll
    for (int it = 0; it < 2; it++) {
        const int m = mblock + it * 8 + (lane >> 3);
        bf16x8_t o;
#pragma unroll
        for (int e = 0; e < 4; e++) { o[e] = (bf16_t)v[2 * it][e]; o[4 + e] = (bf16_t)v[2 * it + 1][e]; }
        if (m < p.M) *(bf16x8_t *)(out + (size_t)m * row_stride) = o;
    }
}

// One 16-row block of raw gate (panel columns 0 .. 63) and up values, output columns from c0: fp32 [M, 2N], gate then up.
__device__ __forceinline__ void pre_block_out(const DmaGemmParams &p, float *panel, int mblock, int c0, int lane) {
    const int cb = lane & 31;
    float *out = p.pre + (cb < 16 ? c0 + cb * 4 : p.N + c0 + (cb - 16) * 4);
    f32x4_t v[8];
#pragma unroll
    for (int it = 0; it < 8; it++) v[it] = panel_get(panel, it * 2 + (lane >> 5), cb);
    panel_wait(v);
#pragma unroll
    for (int it = 0; it < 8; it++) {
        const int m = mblock + it * 2 + (lane >> 5);
        if (m < p.M) *(f32x4_t *)(out + (size_t)m * 2 * p.N) = v[it];
    }
}
// ... and its SwiGLU outputs, bf16 [M, N]
__device__ __forceinline__ void swiglu_of_pre_out(const DmaGemmParams &p, float *panel, int mblock, int c0, int lane) {
    f32x4_t v[8];
#pragma unroll
    for (int it = 0; it < 2; it++) {
        const int row = it * 8 + (lane >> 3), c2 = lane & 7;
#pragma unroll
        for (int u = 0; u < 2; u++) {
            v[4 * it + u] = panel_get(panel, row, 2 * c2 + u);
            v[4 * it + 2 + u] = panel_get(panel, row, 16 + 2 * c2 + u);
        }
    }
    panel_wait(v);
#pragma unroll
    for (int it = 0; it < 2; it++) {
        const int m = mblock + it * 8 + (lane >> 3);
        bf16x8_t o;
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] = (bf16_t)vla_silu_mul_exact(v[4 * it + (e >> 2)][e & 3], v[4 * it + 2 + (e >> 2)][e & 3]);
        if (m < p.M) *(bf16x8_t *)((bf16_t *)p.C + (size_t)m * p.N + c0 + (lane & 7) * 8) = o;
    }
}

// Output of one wave.  Per 16-row activation block i a lane holds row (lane % 16) and, per weight block j
// and register r, column 16 j + 4 (lane / 16) + r.  Each block goes through the panel and leaves as whole
// rows.
template <int EPI, bool KB, int MB>
__device__ __forceinline__ void epilogue(f32x4_t (&acc)[8][MB], const DmaGemmParams &p, int m0, int tn, int wn,
                                         int lane, float *panel, size_t c_off) {
    const int l16 = lane & 15, kq = lane >> 4;
    if (epi_qkv(EPI)) {
        const int n0 = tn * BN + wn * 128;
#pragma unroll
        for (int i = 0; i < MB; i++) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 8; j++) panel_put_acc(panel, l16, j * 4 + kq, acc[j][i]);
            panel_written();
            qkv_block_out<EPI == EPI_QKV_ROWS>(p, panel, m0 + i * 16, n0, lane);
        }
        return;
    }
    if (EPI == EPI_SWIGLU_KEEP) {
#pragma unroll
        for (int i = 0; i < MB; i++) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 8; j++) panel_put_acc(panel, l16, j * 4 + kq, acc[j][i]);
            panel_written();
            pre_block_out(p, panel, m0 + i * 16, tn * 128 + wn * 64, lane);
            swiglu_of_pre_out(p, panel, m0 + i * 16, tn * 128 + wn * 64, lane);
        }
        return;
    }
    if (EPI == EPI_SWIGLU) {
        // weight blocks 0..3 are gate rows, 4..7 the matching up rows: 64 output columns per wave
#pragma unroll
        for (int i = 0; i < MB; i++) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const f32x4_t g = acc_read4(acc[j][i]), u = acc_read4(acc[j + 4][i]);
                f32x4_t v;
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = vla_silu_mul(g[e], u[e]);
                panel_put(panel, l16, j * 4 + kq, v);
            }
            panel_written();
            swiglu_block_out<KB>(p, panel, m0 + i * 16, tn * 128 + wn * 64, lane);
        }
        return;
    }
    if (EPI == EPI_SWIGLU_GRAD) {
        // d act of 16 rows from the panel with their pre-activations, fp32 [M, 2N], to d gate | d up, bf16 [M, 2N].  Rows past M: outside the
        // descriptors.
        const int rows_in = min(16 * MB, p.M - m0), lane_at = (lane >> 5) * 2 * p.N + (lane & 31) * 4;
        const size_t at = (size_t)m0 * 2 * p.N + (size_t)tn * BN + wn * 128;
        const __amdgpu_buffer_rsrc_t gu_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(p.pre + at), (short)0, rows_in > 0 ? rows_in * p.N * 8 : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t d_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((bf16_t *)p.C + at), (short)0, rows_in > 0 ? rows_in * p.N * 4 : 0, 0x00020000);
        i32x4_t gu[2][2][4];
        auto load = [&](i32x4_t (&x)[2][4], int half) {          // eight rows
            int r2 = 4 * p.N * 4;
            asm volatile("" : "+s"(r2));
#pragma unroll
            for (int it = 0; it < 4; it++)
#pragma unroll
                for (int u = 0; u < 2; u++) x[u][it] = __builtin_amdgcn_raw_buffer_load_b128(gu_rsrc, lane_at * 4, (half * 4 + it) * r2 + u * p.N * 4, 0);
        };
        load(gu[0], 0);
#pragma unroll
        for (int i = 0; i < MB; i++) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 8; j++) panel_put_acc(panel, l16, j * 4 + kq, acc[j][i]);
            panel_written();
            f32x4_t v[8];
#pragma unroll
            for (int it = 0; it < 8; it++) v[it] = panel_get(panel, it * 2 + (lane >> 5), lane & 31);
            panel_wait(v);
#pragma unroll
            for (int h = 0; h < 2; h++) {
                if (i * 2 + h + 1 < 2 * MB) load(gu[1 - h], i * 2 + h + 1);
                int r2 = 4 * p.N * 2;
                asm volatile("" : "+s"(r2));
#pragma unroll
                for (int it = 0; it < 4; it++) {
                    const f32x4_t g = __builtin_bit_cast(f32x4_t, gu[h][0][it]), u = __builtin_bit_cast(f32x4_t, gu[h][1][it]);
                    bf16x4_t dg, du;
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        float a, b;
                        vla_swiglu_grad(g[e], u[e], v[h * 4 + it][e], a, b);
                        dg[e] = (bf16_t)a;
                        du[e] = (bf16_t)b;
                    }
                    const int row = ((i * 2 + h) * 4 + it) * r2;
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2_t, dg), d_rsrc, lane_at * 2, row, 0);
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2_t, du), d_rsrc, lane_at * 2, row + p.N * 2, 0);
                }
            }
        }
        return;
    }
    // fp32 store, or read-modify-write of the fp32 residual stream: whole 512-byte rows, two rows per instruction,
    // through a buffer descriptor over this wave's block (rows past M fall outside it: their loads
    // return zero and their stores are dropped, so no clamp and no predicate).  x is read XD 16-row blocks ahead of
    // the block being staged, so that a memory latency is paid once per tile and not once per block.
    const int rows_in = min(16 * MB, p.M - m0);
    float *wave_out = (float *)p.C + c_off + (size_t)m0 * p.N + (size_t)tn * BN + wn * 128;
    __amdgpu_buffer_rsrc_t c_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)wave_out, (short)0, rows_in > 0 ? rows_in * p.N * 4 : 0, 0x00020000);
    __amdgpu_buffer_rsrc_t x_rsrc = c_rsrc;
    if (EPI == EPI_RESIDUAL) x_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(p.res + (size_t)m0 * p.N + (size_t)tn * BN + wn * 128), (short)0, rows_in > 0 ? rows_in * p.N * 4 : 0, 0x00020000);
    const int voff = ((lane >> 5) * p.N + (lane & 31) * 4) * 4;
    const int row2 = 2 * p.N * 4;                      // bytes between the row pairs of consecutive instructions
    constexpr int XD = 2;
    i32x4_t x[XD][8];
    // (the stride passes through an empty assembler statement per block: otherwise all 64 offsets of a tile are
    // computed once, before the main loop, and held in registers across it)
    auto load_x = [&](i32x4_t (&xb)[8], int i) {
        int r2 = row2;
        asm volatile("" : "+s"(r2));
#pragma unroll
        for (int it = 0; it < 8; it++) xb[it] = __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, voff, (i * 8 + it) * r2, 0);
    };
    if (EPI == EPI_RESIDUAL) {
#pragma unroll
        for (int i = 0; i < XD; i++) load_x(x[i], i);
    }
#pragma unroll
    for (int i = 0; i < MB; i++) {
        __builtin_amdgcn_sched_barrier(0);
        int r2 = row2;
        asm volatile("" : "+s"(r2));
#pragma unroll
        for (int j = 0; j < 8; j++) panel_put_acc(panel, l16, j * 4 + kq, acc[j][i]);
        panel_written();
        f32x4_t v[8];
#pragma unroll
        for (int it = 0; it < 8; it++) v[it] = panel_get(panel, it * 2 + (lane >> 5), lane & 31);
        panel_wait(v);
#pragma unroll
        for (int it = 0; it < 8; it++) {
            if (EPI == EPI_RESIDUAL) {
                const f32x4_t xv = __builtin_bit_cast(f32x4_t, x[i % XD][it]);
#pragma unroll
                for (int e = 0; e < 4; e++) v[it][e] += xv[e];
            }
        }
        if (EPI == EPI_RESIDUAL && i + XD < MB) load_x(x[i % XD], i + XD);
#pragma unroll
        for (int it = 0; it < 8; it++)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4_t, v[it]), c_rsrc, voff, (i * 8 + it) * r2, 0);
    }
}

// f(integral_constant<int, i>) for every i of the sequence
template <typename F, int... I>
__device__ __forceinline__ void for_each_index(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

// One MFMA that adds to its sums in place, and one that starts them.
__device__ __forceinline__ void mfma_add(f32x4_t &c, const bf16x8_t &a, const bf16x8_t &b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_start(f32x4_t &c, const bf16x8_t &a, const bf16x8_t &b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(c) : "v"(a), "v"(b));
}
template <int N>
__device__ __forceinline__ void pass_frags(bf16x8_t (&f)[N]) {
#pragma unroll
    for (int i = 0; i < N; i++) asm volatile("" : "+v"(f[i]));
}
template <int N>
__device__ __forceinline__ void pass_frags(ColumnFrag (&f)[N]) {
#pragma unroll
    for (int i = 0; i < N; i++) asm volatile("" : "+v"(f[i].lo), "+v"(f[i].hi));
}

template <int EPI, bool KB, int WL, int MB>
__global__ void __launch_bounds__(256) gemm_bf16_dma_kernel(DmaGemmParams p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    constexpr bool WKB = WL == W_KBLOCKED, WCOL = WL == W_COLUMNS;
    static_assert(!WCOL || ((EPI == EPI_STORE || EPI == EPI_SWIGLU_GRAD) && !KB), "weights as columns");
    constexpr int ROWS = 32 * MB, NA = (MB + 1) / 2, NL = NA + 4;     // tile rows; load instructions per wave and half tile
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int n_tiles = p.tiles_m * p.tiles_n;
    const int n_items = n_tiles * p.splits;
    const int K = p.K;
    const int nh = K / HK / p.splits;            // half tiles per item; even: the host sees to it
    int item = blockIdx.x, grid = (int)gridDim.x;
    asm volatile("" : "+s"(grid));           // (kept in a register: else read from memory again at every tile)
    if (item >= n_items || (nh & 1) || nh < 8) return;      // (the host never launches such a K)

    // ---- load cursor -------------------------------------------------------------------------------------
    // k-blocked: a stage holds one half tile, a wave instruction 16 tile rows of 64 bytes: lane l -> row l / 4, position l % 4
    // of the row, which holds chunk (l % 4) ^ ((row / 2) % 4).  Row-major: a stage holds both half tiles of the tile rows
    // (of either operand) that one half of the waves multiplies, an instruction 8 of them, a whole 128-byte line each: lane l
    // -> row l / 8, position l % 8, which holds chunk (l % 8) ^ (row % 8).  Per stage a wave loads a quarter of the weight rows,
    // four instructions, and 16 NA (8 NA) activation rows, for an odd MB more than the tile has.  SwiGLU tiles interleave 64
    // gate and 64 up rows per half of the weight rows, so a wave's share comes from one of the two matrices.  Mixed (k-blocked
    // weights, row-major activations): the weights' part of a stage is the two half tiles of 128 rows one behind the other, two
    // waves load one of them each.
    const int chunk_off = KB ? ((lane & 3) ^ ((lane >> 3) & 3)) << 4 : ((lane & 7) ^ (lane >> 3)) << 4;
    const int row_bytes = KB ? 64 : K * 2;       // distance of consecutive tile rows
    const int up = KB ? wave & 1 : wave >> 1;    // SwiGLU: which matrix this wave loads from, and which 64 (32) of its rows
    const int a_thread_off = KB ? (wave * 16 * NA + (lane >> 2)) * 64 + chunk_off : (wave * 8 * NA + (lane >> 3)) * row_bytes + chunk_off;
    const int w_part = epi_swiglu(EPI) ? (KB ? wave >> 1 : wave & 1) : wave;
    // W_COLUMNS: a stage holds 64 rows of K of the 128 columns that one half of the waves multiplies, an instruction four of them, 256 bytes
    // each: lane l -> row l / 16, position l % 16; the 32 bytes that a fragment takes of a row, piece b, lie at position b ^ s of the row's
    // eight with s = row % 4 + 4 (row / 8 % 2), so that the reads of four rows, and of eight further ones, meet no bank conflict.
    const int col_bytes = p.N * 2;
    const int w_thread_off = WCOL ? (wave * 16 + (lane >> 4)) * col_bytes + (((lane & 15) ^ ((lane >> 4) << 1)) << 4)
                             : KB ? (w_part * 64 + (lane >> 2)) * 64 + chunk_off
                             : WKB ? ((wave & 1) * 64 + (lane >> 2)) * 64 + (((lane & 3) ^ ((lane >> 3) & 3)) << 4) + (wave >> 1) * p.w_rows * 64
                                   : (w_part * 32 + (lane >> 3)) * row_bytes + chunk_off;
    // distance of what the cursor steps over: one 32-column block of all rows (mixed: two), or 128 bytes along the row
    const unsigned a_step = KB ? (unsigned)p.a_rows * 64u : 128u, w_step = WKB ? (unsigned)p.w_rows * (KB ? 64u : 128u) : WCOL ? (unsigned)col_bytes * 64u : 128u;
    __amdgpu_buffer_rsrc_t a_rsrc, w_rsrc;
    int ld_item;
    unsigned a_soff, w_soff;
    int nx_tm, nx_tn, nx_split;
    // W_COLUMNS: the cursor's pair at which the next segment of K begins, and that segment
    int seg_end = 0, seg = 0;
    auto set_segment = [&](int s) {
        const bf16_t *Wp = s == 0 ? p.W0 : (s == 1 ? p.W1 : p.W2);
        w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(Wp + (size_t)nx_tn * BN), (short)0, (p.segK - 1) * col_bytes + BN * 2, 0x00020000);
        w_soff = 0;
        seg = s;
        seg_end = (s + 1) * (p.segK / 64);
    };
    auto setup_load = [&](int it) {
        int tm, tn;
        const int split = __builtin_amdgcn_readfirstlane(it / n_tiles);
        vla_tile_of_block(it - split * n_tiles, p.tiles_m, p.tiles_n, tm, tn, p.group);
        const bf16_t *Wp;
        int w_row;
        if (WCOL) { Wp = p.W0; w_row = 0; }
        else if (epi_swiglu(EPI)) { Wp = up ? p.W1 : p.W0; w_row = tn * 128; }
        else {
            const int n = tn * BN, seg = __builtin_amdgcn_readfirstlane(n / p.segN);
            Wp = seg == 0 ? p.W0 : (seg == 1 ? p.W1 : p.W2);
            w_row = n - seg * p.segN;
        }
        // (rows behind the activation buffer's last: the range check takes the scalar offset into account, those loads return zero)
        const unsigned w_tile_rows = epi_swiglu(EPI) ? 128u : 256u;
        if (KB) {            // first element of this item's K range: whole 32-column blocks
            const unsigned avail = MB == 8 ? 256u : (unsigned)min(64 * NA, p.a_rows - tm * ROWS);
            a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(p.A + (size_t)tm * ROWS * 32 + (size_t)split * nh * (a_step / 2)), (short)0, (int)((unsigned)(nh - 1) * a_step + avail * 64u), 0x00020000);
        } else {             // ... columns
            const unsigned k0 = (unsigned)split * nh * HK, avail = MB == 8 ? 256u : (unsigned)min(16 * MB + 32 * NA, p.a_rows - tm * ROWS);
            a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(p.A + (size_t)tm * ROWS * K + k0), (short)0, (int)(avail * (unsigned)K * 2u - k0 * 2u), 0x00020000);
            if (WL == W_ROWS) w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(Wp + (size_t)w_row * K + k0), (short)0, (int)(w_tile_rows * (unsigned)K * 2u - k0 * 2u), 0x00020000);
        }
        if (WKB) w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(Wp + (size_t)w_row * 32 + (size_t)split * nh * p.w_rows * 32), (short)0, (int)((unsigned)(nh - 1) * p.w_rows * 64u + w_tile_rows * 64u), 0x00020000);
        ld_item = it;
        a_soff = w_soff = 0;
        nx_tm = tm; nx_tn = tn; nx_split = split;
        if (WCOL) set_segment(0);
    };
    // piece i (below NA: activations, then weights) of the cursor's next stage (row-major: of row half RH) into the stage at byte
    // `st`.  In the k-blocked layout the instruction's own offset moves both the address in memory and the one in LDS.
    auto dma = [&](auto i_c, auto rh_c, int st) {
        constexpr int i = decltype(i_c)::value, q = i < NA ? i : i - NA, RH = decltype(rh_c)::value;
        char *base = lds + st + (i < NA ? wave * (1024 * NA) : wave * 4096 + REGION);
        if (KB) {
            if (i < NA) __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void *)base, 16, a_thread_off, (int)a_soff, q * 1024, 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void *)base, 16, w_thread_off, (int)w_soff, q * 1024, 0);
        } else {
            constexpr int a_row = RH * 16 * MB + q * 8, w_row = RH * (epi_swiglu(EPI) ? 64 : 128) + q * 8;
            if (i < NA) __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void *)(base + q * 1024), 16, a_thread_off, (int)a_soff + a_row * row_bytes, 0, 0);
            else if (WKB) __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void *)base, 16, w_thread_off, (int)w_soff + RH * 128 * 64, q * 1024, 0);
            else if (WCOL) __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void *)(base + q * 1024), 16, q & 2 ? w_thread_off ^ 128 : w_thread_off,
                                                                    (int)w_soff + q * 4 * col_bytes + RH * 256, 0, 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void *)(base + q * 1024), 16, w_thread_off, (int)w_soff + w_row * row_bytes, 0, 0);
        }
        if (i == NL - 1 && (KB || RH == 1)) { a_soff += a_step; w_soff += w_step; }
    };
    // the item's half tiles have all been issued: on to the next item; behind the last one the same half tiles are fetched again
    // (never used)
    auto next_item = [&]() {
        const int nxt = ld_item + grid;
        if (nxt < n_items) setup_load(nxt);
        else a_soff = w_soff = 0;
    };

    // ---- fragments -----------------------------------------------------------------------------------------
    // k-blocked: half tile h of a pair lies in its own stage, blocks of 16 rows 1 KB apart.  Row-major: both lie in the stage of the
    // wave's row half, the chunks of the second 64 bytes behind those of the first, blocks 2 KB apart.
    const int l16 = lane & 15, kq = lane >> 4;
    const int lds0 = (int)(size_t)(lds_void *)lds;
    const int kb_off = l16 * 64 + ((kq ^ ((l16 >> 1) & 3)) << 4), rm_off = l16 * 128 + ((kq ^ (l16 & 7)) << 4);
    const int a_base = lds0 + (KB ? wm * 16 * MB * 64 + kb_off : rm_off), w_base = lds0 + REGION + (KB ? wn * 128 * 64 : 0)
        + (WCOL ? (kq * 8 + (l16 >> 2)) * 256 + (((l16 >> 2) + 4 * (kq & 1)) << 5) + (l16 & 3) * 8 : WKB ? kb_off : rm_off);
    constexpr int A_BLK = KB ? 1024 : 2048, W_BLK = WKB ? 1024 : 2048;
    f32x4_t acc[8][MB];                  // [weight block][activation block]
    bf16x8_t af[2][MB];
    std::conditional_t<WCOL, ColumnFrag, bf16x8_t> wf[2][8];

#define VLA_SB() __builtin_amdgcn_sched_barrier(0)
    // Iteration: reads half tile g, the pair's B-th (stages at bytes a_st, w_st), into fragment buffer B, multiplies half tile g - 1 from
    // the other buffer (MUL 0: nothing to multiply yet, 1: add, 2: start the sums) and issues the cursor's loads into the
    // stage at byte `to` (row-major: row half 1 of the next pair in a first half, row half 0 of the one after it in a second).
    auto iteration = [&](auto b_c, auto mul_c, int a_st, int w_st, int to) {
        constexpr int B = decltype(b_c)::value, MUL = decltype(mul_c)::value;
        constexpr int RSTEP = 2, LSTEP = 8 * MB / NL / 2 * 2;
        static_assert((7 + MB) * RSTEP < 8 * MB && 1 + LSTEP * (NL - 1) < 8 * MB, "reads and loads fit between the MFMAs");
        const int va = (!KB && B == 1 ? a_base ^ 64 : a_base) + a_st, vw = (KB || B == 0 ? w_base : WKB || WCOL ? w_base + 8192 : w_base ^ 64) + w_st;
        for_each_index([&](auto m_c) {
            constexpr int m = decltype(m_c)::value, j = m / MB, i = m % MB;
            if constexpr (MUL == 1) mfma_add(acc[j][i], frag_of(wf[B ^ 1][j]), af[B ^ 1][i]);
            if constexpr (MUL == 2) mfma_start(acc[j][i], frag_of(wf[B ^ 1][j]), af[B ^ 1][i]);
            VLA_SB();
            if constexpr (m % RSTEP == 0 && m / RSTEP < 8 + MB) {        // weight and activation blocks in turn, the weights' rest last
                constexpr int f = m / RSTEP, blk = f < 2 * MB ? f >> 1 : f - MB;
                if constexpr (f < 2 * MB && (f & 1)) af[B][blk] = lds_read<blk * A_BLK>(va);
                else if constexpr (WCOL) wf[B][blk] = lds_read_columns<0, 1024>(vw ^ (blk << 5));
                else wf[B][blk] = lds_read<blk * W_BLK>(vw);
                VLA_SB();
            }
            if constexpr (m % LSTEP == 1 && m / LSTEP < NL) {
                dma(std::integral_constant<int, m / LSTEP>{}, std::integral_constant<int, 1 - B>{}, to);
                VLA_SB();
            }
        }, std::make_integer_sequence<int, 8 * MB>{});
        // this wave's fragment reads have landed; the fragments pass through so that no MFMA moves above the wait
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        pass_frags(af[B]);
        pass_frags(wf[B]);
        VLA_SB();
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    // s0, s1: the stages of the pair being read; s2, s3: of the next one; s4: the first of the one after that
    int s0 = 0, s1 = STAGE, s2 = 2 * STAGE, s3 = 3 * STAGE, s4 = 4 * STAGE;
    // the pair's two half tiles have landed: at most the NL loads of the third stage may still be in flight (vmcnt counts in issue
    // order; right after an epilogue this also waits for its stores)
    auto arrive = [&]() {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        VLA_SB();
    };
    auto first_half = [&](auto mul_c) { iteration(I0{}, mul_c, KB || !wm ? s0 : s1, KB || !wn ? s0 : s1, s3); };
    auto second_half = [&](auto mul_c) {
        iteration(I1{}, mul_c, KB || wm ? s1 : s0, KB || wn ? s1 : s0, s4);
        const int t0 = s0, t1 = s1;
        s0 = s2; s1 = s3; s2 = s4; s3 = t0; s4 = t1;
    };

    setup_load(item);
    int tm = nx_tm, tn = nx_tn, split = nx_split;
    for_each_index([&](auto i_c) { dma(i_c, I0{}, s0); }, std::make_integer_sequence<int, NL>{});
    for_each_index([&](auto i_c) { dma(i_c, I1{}, s1); }, std::make_integer_sequence<int, NL>{});
    for_each_index([&](auto i_c) { dma(i_c, I0{}, s2); }, std::make_integer_sequence<int, NL>{});
    // Half tile h of the workgroup's n-th item is stream element g = n * nh + h; it is read in iteration g and multiplied in
    // iteration g + 1, so an item is complete after the first iteration of the next one (behind the last item: of the half tiles
    // fetched again).  nh is even, so that iteration is always a pair's first.
    const int np = nh / 2;
    arrive();
    first_half(I0{});
    for (;;) {
        second_half(I2{});
        for (int pr = 1; pr < np; pr++) {
            arrive();
            first_half(I1{});
            if (pr == np - 2) next_item();           // the cursor is two pairs ahead in a pair's second half
            else if (WCOL && pr + 2 == seg_end) set_segment(seg + 1);
            second_half(I1{});
        }
        item += grid;
        arrive();
        first_half(I1{});
        // the staging panel: k-blocked, stage s0, which every wave is through with after one more barrier; row-major, where s0 holds
        // the pair's second half tile as well, s4, free since the pair's barrier until its loads go out in the second half
        if (KB) asm volatile("s_barrier" ::: "memory");
        acc_settle();
        epilogue<EPI, KB, MB>(acc, p, tm * ROWS + wm * 16 * MB, tn, wn, lane, (float *)(lds + (KB ? s0 : s4)) + wave * (16 * 128), (size_t)split * p.M * p.N);
        if (!KB) asm volatile("s_barrier" ::: "memory");
        if (item >= n_items) break;
        tm = nx_tm; tn = nx_tn; split = nx_split;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // no load may reach the LDS after the workgroup's end
}


template <int BASE, int STRIDE, int... I>
__device__ __forceinline__ void read_frags(bf16x8_t (&f)[sizeof...(I)], int addr, std::integer_sequence<int, I...>) {
    ((f[I] = lds_read<BASE + I * STRIDE>(addr)), ...);
}
// Small-tile form for products whose 256 x 256 tiles would leave most of the chip idle: BMT (64, 96, 128, 160) x BNT outputs (SwiGLU: half of
// them gate, half up rows), 4 waves of a quarter each, one tile per workgroup, one or two workgroups per CU.  Same
// operands, same v_mfma_f32_16x16x32_bf16 over K in the same order and the same epilogue arithmetic as the 256 x 256
// kernel: results are identical bit for bit, so the choice between them (choose_tile) is one of speed alone.
//
// K moves in units of 64 through a ring of NS stages of (BMT + BNT) x 128 bytes: per unit one wait for this wave's loads,
// one barrier, the load instructions of unit u + NS - 1, then the two halves' fragment reads, each under the other half's
// MFMAs.  Bound by the loads: without any MFMA the kernel takes the same time, 51 GB/s per CU with one workgroup and
// 72 GB/s with two (a CU on its own streams 58 GB/s from HBM however deep its ring), so what counts is the bytes per CU.
// Workgroups of one XCD take neighbouring tile columns with all their tile rows: a weight panel is then fetched into one
// L2 only (the activations, few rows, into all).
//
// STEP (QKV and gate/up of decode steps): instead the sums of gemm_skinny.hip, bit for bit: v_mfma_f32_32x32x16_bf16 on its
// columns (operand j of a unit: 8 j .. + 7 of either half), K in p.parts parts that are added in order.  Repacked weights are read past
// the caches there where the caller says so (64 rows of the 7B width: QKV 26.2 -> 25.7 us, gate/up 39.7 -> 39.2; in the split-K form of the large
// tile it costs 1 to 3 %).
template <int EPI, bool KB, int WL, int BMT, int BNT, int NS, bool STEP>
__global__ void __launch_bounds__(256, 2) gemm_bf16_small_kernel(DmaGemmParams p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    constexpr bool WKB = WL == W_KBLOCKED || WL == W_KBLOCKED_PAST, WCOL = WL == W_COLUMNS;
    static_assert(!WCOL || ((EPI == EPI_STORE || EPI == EPI_SWIGLU_GRAD) && !KB && !STEP), "weights as columns");
    constexpr int MB = BMT / 32, NB = BNT / 32;          // 16-row / 16-column blocks per wave
    constexpr int A_HALF = BMT * 64, W_HALF = BNT * 64, SSTAGE = 2 * (A_HALF + W_HALF);
    constexpr int NA = BMT / 32, NWI = BNT / 32;                // load instructions per wave and unit
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, kq = lane >> 4;
    const int K = p.K, units = K / 64;
    const int total = p.tiles_m * p.tiles_n, per_xcd = (total + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || tile >= total || units < NS) return;
    const int tn = tile / p.tiles_m, tm = tile - tn * p.tiles_m;

    // ---- loads: an instruction covers 16 rows of one half (AH, WH), or 8 rows of both, a whole line each (see the 256 x 256 kernel).
    // Row-major operands are read as whole lines except by 64 x 64 tiles, whose steps are too short for the second half's own
    // addresses: 40 x 256, K = 9536 36.2 us as halves and 39.6 as lines, 113 x 1792, K = 6336 26.2 and 28.6; 64 x 128 tiles 2 % faster as lines
    // (median of 69 sizes), 128 x 128 the same.
    constexpr bool AH = KB || (BMT == 64 && BNT == 64), WH = WKB || (WL == W_ROWS && BMT == 64 && BNT == 64);
    const int kb_chunk = ((lane & 3) ^ ((lane >> 3) & 3)) << 4, rm_chunk = ((lane & 7) ^ (lane >> 3)) << 4;
    const int row_bytes = KB ? 64 : K * 2, w_row_bytes = WKB ? 64 : K * 2;
    const unsigned a_half = KB ? (unsigned)p.a_rows * 64u : 64u, w_half = WKB ? (unsigned)p.w_rows * 64u : 64u;
    const int thread_off = AH ? (lane >> 2) * row_bytes + kb_chunk : (lane >> 3) * row_bytes + rm_chunk;
    // W_COLUMNS: 64 rows of K of BNT columns, an instruction 1 KB of whole rows of 2 BNT bytes; piece b (32 bytes) of a row at position b ^ s,
    // s = row % 4 + 4 (row / 8 % 2) of eight (BNT = 128) or row % 4 ^ (row / 8 % 2) of four
    constexpr int CROW = 2 * BNT, CPR = CROW / 16, CRI = 1024 / CROW;        // bytes and 16-byte chunks of a row, rows of an instruction
    const int col_bytes = p.N * 2;
    const int w_thread_off = WCOL ? (wave * 16 + lane / CPR) * col_bytes + (((lane % CPR) ^ ((lane / CPR & 3) << 1)) << 4)
                             : WH ? (lane >> 2) * w_row_bytes + kb_chunk : (lane >> 3) * w_row_bytes + rm_chunk;
    const bf16_t *Wp;
    int w_row0;
    if (WCOL) {
        Wp = p.W0;
        w_row0 = 0;
    } else if (epi_swiglu(EPI)) {
        Wp = (wave & 1) ? p.W1 : p.W0;                   // instruction blocks 0..3 gate rows, 4..7 up rows
        w_row0 = tn * 64;
    } else {
        const int n = tn * BNT, seg = n / p.segN;
        Wp = seg == 0 ? p.W0 : (seg == 1 ? p.W1 : p.W2);
        w_row0 = n - seg * p.segN + (wave & 1) * (BNT / 2);
    }
    const size_t row_elems = KB ? 32 : (size_t)K, w_row_elems = WKB ? 32 : (size_t)K;
    const unsigned nh1 = (unsigned)(K / HK - 1);
    const int a_avail = min(BMT, p.a_rows - tm * BMT);   // (a tile may reach past the activation buffer's last row: those loads return zero)
    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(p.A + (size_t)tm * BMT * row_elems), (short)0, KB ? (int)(nh1 * a_half + a_avail * 64u) : a_avail * K * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(Wp + (size_t)w_row0 * w_row_elems), (short)0, WKB ? (int)(nh1 * w_half + BNT * 32u) : BNT * K, 0x00020000);   // (half the tile's rows: one wave's share)
    auto load_unit = [&](int u, int stage) {
        char *base = lds + stage * SSTAGE, *w_base = base + 2 * A_HALF;
        const int seg = WCOL ? (u * 64 >= p.segK) + (u * 64 >= 2 * p.segK) : 0;
        const __amdgpu_buffer_rsrc_t c_rsrc = WCOL ? __builtin_amdgcn_make_buffer_rsrc(
            (void *)((seg == 0 ? p.W0 : seg == 1 ? p.W1 : p.W2) + (size_t)tn * BNT), (short)0, (p.segK - 1) * col_bytes + CROW, 0x00020000) : w_rsrc;
#pragma unroll
        for (int i = 0; i < NA; i++) {
            const int q = wave * NA + i, half = q / (BMT / 16), blk = q % (BMT / 16);
            if (AH) __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void *)(base + half * A_HALF + blk * 1024), 16, thread_off,
                                                             (int)((unsigned)(2 * u + half) * a_half) + blk * 16 * row_bytes, 0, 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void *)(base + q * 1024), 16, thread_off, u * 128 + q * 8 * row_bytes, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < NWI; i++) {
            const int half = wave >> 1, blk = (wave & 1) * NWI + i, row = half * (BNT / 4) + i * 8;
            if (WCOL) __builtin_amdgcn_raw_ptr_buffer_load_lds(c_rsrc, (lds_void *)(w_base + (wave * NWI + i) * 1024), 16,
                                                               (i * CRI) & 8 ? w_thread_off ^ (BNT == 128 ? 128 : 32) : w_thread_off,
                                                               (u * 64 - seg * p.segK + i * CRI) * col_bytes, 0, 0);
            else if (WH) __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void *)(w_base + half * W_HALF + blk * 1024), 16, w_thread_off,
                                                             (int)((unsigned)(2 * u + half) * w_half) + i * 16 * w_row_bytes, 0, WL == W_KBLOCKED_PAST ? 2 : 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void *)(w_base + ((wave & 1) * (BNT / 2) + row) * 128), 16, w_thread_off,
                                                          u * 128 + row * w_row_bytes, 0, 0);
        }
    };

    const int lds0 = (int)(size_t)(lds_void *)lds, a_row0 = wm * (BMT / 2), w_row0_lds = wn * (BNT / 2);
    const int kb_off = l16 * 64 + ((kq ^ ((l16 >> 1) & 3)) << 4), rm_off = l16 * 128 + ((kq ^ (l16 & 7)) << 4);
    const int a_base = lds0 + (AH ? a_row0 * 64 + kb_off : a_row0 * 128 + rm_off);
    const int w_swizzle = BNT == 128 ? (l16 >> 2) + 4 * (kq & 1) : (l16 >> 2) ^ (kq & 1);
    const int w_base = lds0 + 2 * A_HALF + (WCOL ? (kq * 8 + (l16 >> 2)) * CROW + ((w_swizzle ^ (wn * NB)) << 5) + (l16 & 3) * 8
                                            : WH ? w_row0_lds * 64 + kb_off : w_row0_lds * 128 + rm_off);
    // STEP: lane l reads row l % 32 of a 32-row block, from half l / 32 of the unit (chunks 4 (l / 32) .. + 3 of a whole line)
    constexpr int MB2 = MB / 2, NB2 = NB / 2;
    const int l32 = lane & 31, hh = lane >> 5, fsw32 = (l32 >> 1) & 3;
    const int a_step = lds0 + (AH ? hh * A_HALF + (a_row0 + l32) * 64 : (a_row0 + l32) * 128);
    const int w_step = lds0 + 2 * A_HALF + (WH ? hh * W_HALF + (w_row0_lds + l32) * 64 : (w_row0_lds + l32) * 128);
    f32x4_t acc[STEP ? 1 : NB][STEP ? 1 : MB];
    f32x16_t acc32[STEP ? NB2 : 1][STEP ? MB2 : 1], sum32[STEP ? NB2 : 1][STEP ? MB2 : 1];
    if constexpr (STEP) {
#pragma unroll
        for (int j = 0; j < NB2; j++)
#pragma unroll
            for (int i = 0; i < MB2; i++)
#pragma unroll
                for (int r = 0; r < 16; r++) acc32[j][i][r] = 0.f;
    } else {
#pragma unroll
        for (int j = 0; j < NB; j++)
#pragma unroll
            for (int i = 0; i < MB; i++) acc[j][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

    bf16x8_t af[2][MB];                                  // (the first multiply, before any second half, adds zeros)
    std::conditional_t<WCOL, ColumnFrag, bf16x8_t> wf[2][NB];
#pragma unroll
    for (int i = 0; i < MB; i++)
#pragma unroll
        for (int e = 0; e < 8; e++) af[1][i][e] = (bf16_t)0.f;
#pragma unroll
    for (int j = 0; j < NB; j++) {
        if constexpr (WCOL) wf[1][j] = ColumnFrag{{0, 0}, {0, 0}};
        else
#pragma unroll
            for (int e = 0; e < 8; e++) wf[1][j][e] = (bf16_t)0.f;
    }
    auto multiply = [&](int h) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (STEP) {
#pragma unroll
            for (int q = 0; q < 2; q++)
#pragma unroll
                for (int j = 0; j < NB2; j++)
#pragma unroll
                    for (int i = 0; i < MB2; i++)
                        acc32[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[h][q * NB2 + j], af[h][q * MB2 + i], acc32[j][i], 0, 0, 0);
        } else {
#pragma unroll
            for (int j = 0; j < NB; j++)
#pragma unroll
                for (int i = 0; i < MB; i++) acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_of(wf[h][j]), af[h][i], acc[j][i], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // the fragments of half h of a unit (STEP: its operands 2 h and 2 h + 1)
    auto read_half = [&](auto h_c, int so) {
        constexpr int h = decltype(h_c)::value;
        if constexpr (STEP) {
#pragma unroll
            for (int q = 0; q < 2; q++) {
                const int ck = ((2 * h + q) ^ fsw32) << 4, cr = ((4 * hh + 2 * h + q) ^ (l32 & 7)) << 4;
#pragma unroll
                for (int j = 0; j < NB2; j++) wf[h][q * NB2 + j] = lds_read<0>(w_step + so + (WH ? ck + j * 2048 : cr + j * 4096));
#pragma unroll
                for (int i = 0; i < MB2; i++) af[h][q * MB2 + i] = lds_read<0>(a_step + so + (AH ? ck + i * 2048 : cr + i * 4096));
            }
        } else {
            if constexpr (WCOL) {
#pragma unroll
                for (int j = 0; j < NB; j++) wf[h][j] = lds_read_columns<h * 32 * CROW, 4 * CROW>((w_base ^ (j << 5)) + so);
            } else read_frags<WH ? h * W_HALF : 0, WH ? 1024 : 2048>(wf[h], (WH || h == 0 ? w_base : w_base ^ 64) + so, std::make_integer_sequence<int, NB>{});
            read_frags<AH ? h * A_HALF : 0, AH ? 1024 : 2048>(af[h], (AH || h == 0 ? a_base : a_base ^ 64) + so, std::make_integer_sequence<int, MB>{});
        }
    };
    // STEP: the sums of a part join those of the parts before
    auto close_part = [&](bool first) {
#pragma unroll
        for (int j = 0; j < NB2; j++)
#pragma unroll
            for (int i = 0; i < MB2; i++)
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    sum32[j][i][r] = first ? acc32[j][i][r] : sum32[j][i][r] + acc32[j][i][r];
                    acc32[j][i][r] = 0.f;
                }
    };
    int part_end = STEP ? units / p.parts : 0, part = 0;         // part y ends before unit (y + 1) units / parts
    // this wave's fragment reads have landed; the fragments pass through, so that no MFMA moves above the wait
    auto wait_frags = [&](int h) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        pass_frags(wf[h]);
        pass_frags(af[h]);
    };

#pragma unroll
    for (int u = 0; u < NS - 1; u++) load_unit(u, u);
    int stage = 0;
    for (int u = 0; u < units; u++) {
        // unit u has landed when at most the NS - 2 units after it are in flight (towards the end: when nothing is)
        if (u + NS - 2 < units) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * (NA + NWI)) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("s_barrier" ::: "memory");         // ... for every wave, and everyone's reads of unit u - 1 are done
        const int prev = stage == 0 ? NS - 1 : stage - 1;
        if (u + NS - 1 < units) load_unit(u + NS - 1, prev);
        const int so = stage * SSTAGE;
        // first half's fragments while the second half of unit u - 1 multiplies, then the other way round
        read_half(std::integral_constant<int, 0>{}, so);
        multiply(1);
        if constexpr (STEP) {
            if (u == part_end) {
                close_part(part == 0);
                part++;
                part_end = (int)((long)(part + 1) * units / p.parts);
            }
        }
        wait_frags(0);
        read_half(std::integral_constant<int, 1>{}, so);
        multiply(0);
        wait_frags(1);
        stage = stage == NS - 1 ? 0 : stage + 1;
    }
    multiply(1);
    if constexpr (STEP) close_part(part == 0);
    // ---- output: the whole tile as fp32 through LDS, then each wave takes 16-row blocks
    asm volatile("s_barrier" ::: "memory");
    float *panel = (float *)lds;
    if constexpr (STEP) {                                // lane l: row l % 32 of a block, columns 8 g + 4 hh .. + 3 in registers 4 g .. + 3
#pragma unroll
        for (int j = 0; j < NB2; j++)
#pragma unroll
            for (int i = 0; i < MB2; i++)
#pragma unroll
                for (int g = 0; g < 4; g++)
                    *(f32x4_t *)panel_at(panel + (wm * MB + 2 * i + (l32 >> 4)) * 16 * 128, l16, wn * (NB * 4) + j * 8 + 2 * g + hh) =
                        f32x4_t{sum32[j][i][4 * g], sum32[j][i][4 * g + 1], sum32[j][i][4 * g + 2], sum32[j][i][4 * g + 3]};
    } else {
#pragma unroll
        for (int j = 0; j < NB; j++)
#pragma unroll
            for (int i = 0; i < MB; i++)
                *(f32x4_t *)panel_at(panel + (wm * MB + i) * 16 * 128, l16, wn * (NB * 4) + j * 4 + kq) = acc[j][i];
    }
    __syncthreads();
    const int m0 = tm * BMT;
#pragma unroll
    for (int b = wave; b < BMT / 16; b += 4) {
        float *pb = panel + b * 16 * 128;
        const int mblock = m0 + b * 16;
        if (mblock >= p.M) break;
        if (epi_qkv(EPI)) {
            qkv_block_out<EPI == EPI_QKV_ROWS>(p, pb, mblock, tn * 128, lane);
        } else if (EPI == EPI_SWIGLU_KEEP) {
            pre_block_out(p, pb, mblock, tn * 64, lane);
            swiglu_of_pre_out(p, pb, mblock, tn * 64, lane);
        } else if (EPI == EPI_SWIGLU) {
#pragma unroll
            for (int it = 0; it < 2; it++) {
                const int row = it * 8 + (lane >> 3), c2 = lane & 7;
#pragma unroll
                for (int u = 0; u < 2; u++) {            // a lane's own eight columns, in place
                    float *gp = panel_at(pb, row, 2 * c2 + u);
                    f32x4_t g = *(const f32x4_t *)gp;
                    const f32x4_t up = *(const f32x4_t *)panel_at(pb, row, 16 + 2 * c2 + u);
#pragma unroll
                    for (int e = 0; e < 4; e++) g[e] = vla_silu_mul(g[e], up[e]);
                    *(f32x4_t *)gp = g;
                }
            }
            panel_written();
            swiglu_block_out<KB>(p, pb, mblock, tn * 64, lane);
        } else {
            constexpr int LPR = BNT / 4, RPI = 64 / LPR;      // lanes per row, rows per instruction
            const size_t out0 = (size_t)mblock * p.N + (size_t)tn * BNT + (lane % LPR) * 4;
            float *out = (float *)p.C + out0;
#pragma unroll
            for (int it = 0; it < 16 / RPI; it++) {
                const int row = it * RPI + lane / LPR;
                f32x4_t v = *(const f32x4_t *)panel_at(pb, row, lane % LPR);
                if (EPI == EPI_SWIGLU_GRAD) {
                    if (mblock + row < p.M) {
                        const size_t at = (size_t)(mblock + row) * 2 * p.N + (size_t)tn * BNT + (lane % LPR) * 4;
                        const f32x4_t g = *(const f32x4_t *)(p.pre + at), u = *(const f32x4_t *)(p.pre + at + p.N);
                        bf16x4_t dg, du;
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            float a, b;
                            vla_swiglu_grad(g[e], u[e], v[e], a, b);
                            dg[e] = (bf16_t)a;
                            du[e] = (bf16_t)b;
                        }
                        *(bf16x4_t *)((bf16_t *)p.C + at) = dg;
                        *(bf16x4_t *)((bf16_t *)p.C + at + p.N) = du;
                    }
                } else if (mblock + row < p.M) {
                    f32x4_t *dst = (f32x4_t *)(out + (size_t)row * p.N);
                    if (EPI == EPI_RESIDUAL) {
                        const f32x4_t x = *(const f32x4_t *)(p.res + out0 + (size_t)row * p.N);
#pragma unroll
                        for (int e = 0; e < 4; e++) v[e] += x[e];
                    }
                    *dst = v;
                }
            }
        }
    }
}

template <int EPI, bool KB, int WL = KB, int MB = 8>
int launch_plain(const DmaGemmParams &p, hipStream_t st) {
    static bool attr_set = false;
    static int n_cu = 0;
    const size_t lds = NSTAGES * (size_t)STAGE;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)gemm_bf16_dma_kernel<EPI, KB, WL, MB>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) {
            vla_set_error("hipFuncSetAttribute(gemm_bf16_dma) failed: %s", hipGetErrorString(e));
            return VLA_EHIP;
        }
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1) {
            vla_set_error("gemm_bf16_dma: cannot read the compute-unit count");
            return VLA_EHIP;
        }
        attr_set = true;
    }
    // one workgroup per CU (160 KB of LDS, 512 registers per lane); blockIdx % 8 is the XCD, and a stride of a
    // multiple of 8 keeps every workgroup's items on its own XCD's share of the tile order
    const int n_items = p.tiles_m * p.tiles_n * p.splits;
    int grid = n_items;
    if (n_cu % 8 == 0 && n_items > n_cu) grid = n_cu;
    gemm_bf16_dma_kernel<EPI, KB, WL, MB><<<grid, 256, lds, st>>>(p);
    int rc = vla_check_launch("gemm_bf16_dma");
    return rc ? rc : 1;
}

// mb (5 .. 8): 16-row blocks per wave, i.e. tiles of 32 mb rows
template <int EPI, bool KB, int WL = KB>
int launch(DmaGemmParams p, int mb, hipStream_t st) {
    const double flops = 2.0 * p.M * p.K * (epi_swiglu(EPI) ? 2.0 * p.N : (double)p.N);
    ProfScope ps(epi_swiglu(EPI) ? "gemm_bf16_dma<swiglu>" : EPI == EPI_RESIDUAL ? "gemm_bf16_dma<residual>"
                 : epi_qkv(EPI) ? "gemm_bf16_dma<qkv_rope>" : EPI == EPI_SWIGLU_GRAD ? "gemm_bf16_dma<swiglu_grad>" : "gemm_bf16_dma<store>", flops, st);
    p.tiles_m = (p.M + 32 * mb - 1) / (32 * mb);
    switch (mb) {
        case 5: return launch_plain<EPI, KB, WL, 5>(p, st);
        case 6: return launch_plain<EPI, KB, WL, 6>(p, st);
        case 7: return launch_plain<EPI, KB, WL, 7>(p, st);
        default: return launch_plain<EPI, KB, WL>(p, st);
    }
}

template <int EPI, bool KB, int WL, int BMT, int BNT, int NS, bool STEP>
int launch_small(DmaGemmParams p, hipStream_t st) {
    static bool attr_set = false;
    const size_t lds = (size_t)NS * 2 * (BMT * 64 + BNT * 64);
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)gemm_bf16_small_kernel<EPI, KB, WL, BMT, BNT, NS, STEP>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) {
            vla_set_error("hipFuncSetAttribute(gemm_bf16_small) failed: %s", hipGetErrorString(e));
            return VLA_EHIP;
        }
        attr_set = true;
    }
    p.tiles_m = (p.M + BMT - 1) / BMT;
    p.tiles_n = epi_swiglu(EPI) ? p.N / (BNT / 2) : p.N / BNT;
    const int per_xcd = (p.tiles_m * p.tiles_n + 7) / 8;
    gemm_bf16_small_kernel<EPI, KB, WL, BMT, BNT, NS, STEP><<<8 * per_xcd, 256, lds, st>>>(p);
    int rc = vla_check_launch("gemm_bf16_small");
    return rc ? rc : 1;
}

// Which kernel takes a product of M rows, N columns (tile columns are 128 weight rows; SwiGLU counts gate and up) and K:
// the large one with tiles of 32 mb x 256, or a small tile.  All give the same bits; the rule compares estimates in ns, fitted to
// what the four projections of the 7B shape took at 64 .. 18432 rows (per unit of K = 64 and launch):
//   32 mb x 256     a round of 256 tiles 333 + 107 mb per unit (mb = 8: 1190) + 8000 (prologue and epilogue)
//   64 x 64         310 up to 150 tiles, 345 up to 256, then 120 + 1.25 per tile (plain and residual outputs only)
//   128 x 64        445 where one workgroup per CU takes all tiles (plain and residual outputs, more than 128 rows, see below)
//   64 x 128        470 up to 276 tiles, then 1.7 per tile (SwiGLU, two weight panels per tile: 620, at least 1000)
//   128 x 128       640 with one workgroup per CU (3 stages of LDS; SwiGLU 735), 950 for every 512 with two (2 stages)
//   96 x 64 394, 160 x 64 525 (as 128 x 64), 96 x 128 570, 160 x 128 765 (SwiGLU 680, 790): one workgroup per CU, K from 1024
// The heights of 96 and 160 rows fill a round where 64 and 128 leave a second one nearly empty or pad the rows: what a CU loads decides, 59 GB/s
// with one workgroup.  Weights from memory, before and with them, us: 288 rows, O 28.7 and 25.2, down 73.1 and 62.1, QKV 59 and 51.5, k and v 50.3 and
// 36.9; 160 rows, QKV 52.4 and 38.6, gate/up 77.6 and 47.9; 72 rows, gate/up 45.3 and 41.7; 700 rows, O 50.0 and 36.9, down 131.9 and 91.4.
// (288 x 128, three stages: no better than the large tile of 160 rows or 128 x 128 with two workgroups, but for gate/up at 200 rows, 77 and 72.5.)
// E.g. 288 rows, K = 4096: QKV 86 -> 55 us (64 x 128), O and down (K = 11008) on average 133 -> 58 (64 x 64 and 64 x 128) -> 52
// (128 x 64); gate/up 76 with 160 x 256, 86 with 256 x 256, 100 with 64 x 128.
// Tiles lower than 256 rows where the rounds of 256 tiles come out fuller: 2,304 rows, O and down on average 154 -> 133 us (160 rows
// per tile); 4,608 rows 301 -> 250 (160); 3,384 rows, QKV 258 -> 243 (224); 7,150 rows 514 -> 484 and 339 -> 326 (224).  Their
// rounds cost more per row, as each loads all of the tile's weights: below 160 rows the small tiles are faster.
// Where the estimates alone would take a slower tile than there was before: 128 x 64
// moves as many bytes as 64 x 128 and wins only where most of them are weights (not more rows than columns) and the steps are many (K
// from 1024): 7,639 x 256, K = 768 8.2 us with 64 x 128, 10.6 with 128 x 64; 829 x 1792, K = 8768 63 and 56.  64 x 64 tiles of at most
// 288 keep a CU each, all but a few: 315 x 3584, K = 896 6.3 us, 7.3 with 128 x 64.  Low large tiles that do not fill a round stream
// at a lower rate than a single round of 128 x 128: 1,421 x 4096, K = 11008 152 us, 198 with 160 x 256 (whole calls, up to 448 such tiles:
// gradient pass of three layers, 1,415 rows 5.12 ms, 5.30 with low tiles; prefill of 1,132 rows 1.87 and 2.01; at 512, 1,981 rows, 6.00 and
// 5.84); not so where the columns are few (7,208 x 1024: 160 x 256 28 % faster).
enum SmallTile { TILE_LARGE = 0, TILE_64x64, TILE_128x64, TILE_64x128, TILE_128x128_1, TILE_128x128_2, TILE_96x64, TILE_160x64, TILE_96x128, TILE_160x128 };
struct TileChoice { SmallTile small; int mb; };
template <int EPI>
TileChoice choose_tile(const DmaGemmParams &p, int mb_low, bool step = false) {          // large tiles of 32 mb_low .. 256 rows; step: those of decode steps
    const long units = p.K / 64, cols = epi_swiglu(EPI) ? 2L * p.N : p.N;
    const long t64 = (p.M + 63L) / 64 * (cols / 128), t128 = (p.M + 127L) / 128 * (cols / 128);
    TileChoice best{TILE_LARGE, 8};
    long best_ns = -1;
    auto offer = [&](TileChoice tile, long ns) {
        if (best_ns < 0 || ns < best_ns) { best = tile; best_ns = ns; }
    };
    if (t128 <= 448 && p.M <= cols) mb_low = 8;
    for (int mb = 8; mb >= mb_low; mb--) {
        const long tiles = (p.M + 32L * mb - 1) / (32L * mb) * (cols / 256);
        offer({TILE_LARGE, mb}, (tiles + 255) / 256 * (units * (333 + 107 * mb) + 8000));
    }
    if (epi_plain(EPI)) offer({TILE_64x64, 0}, units * (2 * t64 <= 150 ? 310 : 2 * t64 <= 256 && !step ? 345 : 120 + 5 * (2 * t64) / 4));
    if (epi_plain(EPI) && p.M > 128 && p.M <= cols && units >= 16 && 2 * t64 > 288 && 2 * t128 <= 256)
        offer({TILE_128x64, 0}, units * 445);
    if (epi_swiglu(EPI)) offer({TILE_64x128, 0}, units * (t64 <= 276 ? 620 : t64 <= 588 ? 1000 : 17 * t64 / 10));
    else offer({TILE_64x128, 0}, units * (t64 <= 276 ? 470 : 17 * t64 / 10));
    if (t128 <= 256) offer({TILE_128x128_1, 0}, units * (epi_swiglu(EPI) && !step ? 735 : 640));
    if (!step && units >= 16) {
        const long t96 = (p.M + 95L) / 96 * (cols / 128), t160 = (p.M + 159L) / 160 * (cols / 128);
        if (epi_plain(EPI) && p.M > 128 && p.M <= cols && 2 * t64 > 288) {
            if (2 * t96 <= 256) offer({TILE_96x64, 0}, units * 394);
            if (2 * t160 <= 256) offer({TILE_160x64, 0}, units * 525);
        }
        if (t96 <= 256) offer({TILE_96x128, 0}, units * (epi_swiglu(EPI) ? 680 : 570));
        if (t160 <= 256) offer({TILE_160x128, 0}, units * (epi_swiglu(EPI) ? 790 : 765));
    }
    offer({TILE_128x128_2, 0}, units * 950 * ((t128 + 511) / 512));
    return best;
}

template <int EPI, bool KB, int WL = KB, bool STEP = false>
int launch_tile(const DmaGemmParams &p, SmallTile tile, hipStream_t st) {
    const double flops = 2.0 * p.M * p.K * (epi_swiglu(EPI) ? 2.0 * p.N : (double)p.N);
    ProfScope ps(epi_swiglu(EPI) ? "gemm_small<swiglu>" : EPI == EPI_RESIDUAL ? "gemm_small<residual>"
                 : epi_qkv(EPI) ? "gemm_small<qkv_rope>" : EPI == EPI_SWIGLU_GRAD ? "gemm_small<swiglu_grad>" : "gemm_small<store>", flops, st);
    if constexpr (epi_plain(EPI)) {
        if (tile == TILE_64x64) return launch_small<EPI, KB, WL, 64, 64, 4, STEP>(p, st);
        if constexpr (!STEP) {
            if (tile == TILE_128x64) return launch_small<EPI, KB, WL, 128, 64, 4, STEP>(p, st);
        }
    }
    if constexpr (!STEP) {
        if constexpr (epi_plain(EPI)) {
            if (tile == TILE_96x64) return launch_small<EPI, KB, WL, 96, 64, 5, STEP>(p, st);
            if (tile == TILE_160x64) return launch_small<EPI, KB, WL, 160, 64, 4, STEP>(p, st);
        }
        if (tile == TILE_96x128) return launch_small<EPI, KB, WL, 96, 128, 4, STEP>(p, st);
        if (tile == TILE_160x128) return launch_small<EPI, KB, WL, 160, 128, 4, STEP>(p, st);
    }
    if (tile == TILE_64x128) return launch_small<EPI, KB, WL, 64, 128, 3, STEP>(p, st);
    if (tile == TILE_128x128_1) return launch_small<EPI, KB, WL, 128, 128, 3, STEP>(p, st);
    return launch_small<EPI, KB, WL, 128, 128, 2, STEP>(p, st);
}

template <int EPI>
int launch_kb(const DmaGemmParams &p, bool kb, hipStream_t st) {
    const TileChoice t = choose_tile<EPI>(p, 5);
    if constexpr (EPI == EPI_SWIGLU_GRAD) {
        return t.small != TILE_LARGE ? launch_tile<EPI, false, W_COLUMNS>(p, t.small, st) : launch<EPI, false, W_COLUMNS>(p, t.mb, st);
    } else if constexpr (EPI == EPI_QKV_ROWS || EPI == EPI_SWIGLU_KEEP || EPI == EPI_STORE) {          // row-major operands only
        if (kb) return 0;
        if constexpr (EPI == EPI_STORE) {
            if (p.segK) return t.small != TILE_LARGE ? launch_tile<EPI, false, W_COLUMNS>(p, t.small, st) : launch<EPI, false, W_COLUMNS>(p, t.mb, st);
        }
        return t.small != TILE_LARGE ? launch_tile<EPI, false>(p, t.small, st) : launch<EPI, false>(p, t.mb, st);
    } else {
        if (t.small != TILE_LARGE) return kb ? launch_tile<EPI, true>(p, t.small, st) : launch_tile<EPI, false>(p, t.small, st);
        return kb ? launch<EPI, true>(p, t.mb, st) : launch<EPI, false>(p, t.mb, st);
    }
}

}  // namespace

// Handles bf16 problems with K a multiple of 64 and at least 256 (the cursor must never be more than one item
// ahead of the multiply side), N tiles that do not straddle weight segments, and an activation buffer that
// covers whole 256-row tiles.  With g.kblocked the activations (a_rows rows per 32-column block), the weights
// (segN + pad rows per block, each segment repacked on its own) and a SwiGLU output are in the k-blocked layout.
// Returns 1 if handled, 0 if declined, < 0 on a launch error.
int try_gemm_bf16_dma(const GemmArgs &g, hipStream_t st) {
    if (g.M < 1 || g.K % 64 != 0 || g.K < 256 || g.a_rows < (g.M + BM - 1) / BM * BM) return 0;
    const bool kb = g.kblocked != 0;
    if (kb && ((size_t)g.a_rows * g.K * 2 >= ((size_t)1 << 31) || (size_t)(g.segN + VLA_KB_PAD_ROWS) * g.K * 2 >= ((size_t)1 << 31))) return 0;
    DmaGemmParams p{};
    p.A = (const bf16_t *)g.A;
    p.W0 = (const bf16_t *)g.W[0]; p.W1 = (const bf16_t *)g.W[1]; p.W2 = (const bf16_t *)g.W[2];
    p.C = g.C; p.res = g.res ? g.res : (const float *)g.C; p.M = g.M; p.K = g.K; p.segN = g.segN;
    p.a_rows = g.a_rows; p.w_rows = g.segN + VLA_KB_PAD_ROWS;
    p.splits = 1;
    {
        // tile rows per column panel of the walk: 4, except for the QKV projection (1.9 % faster with 2 at
        // M = 73728: 5.73 against 5.84 ms; the other projections within 0.5 % either way)
        p.group = epi_qkv(g.epilogue) ? 2 : 4;
    }
    p.tiles_m = (g.M + BM - 1) / BM;
    if (g.epilogue == EPI_SWIGLU) {
        if (g.segN % 128 != 0) return 0;
        p.N = g.segN;
        p.tiles_n = g.segN / 128;
        return launch_kb<EPI_SWIGLU>(p, kb, st);
    }
    if (g.epilogue == EPI_SWIGLU_KEEP) {
        if (g.segN % 128 != 0) return 0;
        p.N = g.segN;
        p.tiles_n = g.segN / 128;
        p.pre = g.pre;
        return launch_kb<EPI_SWIGLU_KEEP>(p, kb, st);
    }
    if (g.segN % BN != 0) return 0;
    if (g.segK) {
        const bool grad = g.epilogue == EPI_SWIGLU_GRAD;
        if (kb || !(grad || g.epilogue == EPI_STORE) || g.segK % 64 != 0 || g.segK < 256 || g.K != g.n_seg * g.segK || (size_t)g.segK * g.segN * 2 >= ((size_t)1 << 31)) return 0;
        for (int i = 0; i < g.n_seg; i++)
            if ((size_t)g.W[i] % 16 != 0) return 0;
        p.segK = g.segK;
        p.N = g.segN;
        p.tiles_n = p.N / BN;
        p.pre = g.pre;
        return grad ? launch_kb<EPI_SWIGLU_GRAD>(p, false, st) : launch_kb<EPI_STORE>(p, false, st);
    }
    if (g.epilogue == EPI_SWIGLU_GRAD) return 0;
    if (g.epilogue == EPI_QKV_ROWS) {
        const QkvRopeArgs *ra = g.rope;
        if (!ra || ra->kv->d != 128 || (g.n_seg != 3 && g.n_seg != 2) || g.segN != ra->kv->n_heads * 128) return 0;
        p.seg0 = 3 - g.n_seg;
        p.q_out = (bf16_t *)ra->q_out;
        p.table = ra->table;
        p.R = ra->rows->R; p.H = g.segN;
        p.N = g.n_seg * g.segN;
        p.tiles_n = p.N / BN;
        return launch_kb<EPI_QKV_ROWS>(p, kb, st);
    }
    if (g.epilogue == EPI_QKV_ROPE) {
        const QkvRopeArgs *ra = g.rope;
        if (!ra || ra->kv->d != 128 || (g.n_seg != 3 && g.n_seg != 2) || g.segN != ra->kv->n_heads * 128) return 0;
        if (g.n_seg == 3 && !ra->q_out) return 0;
        p.seg0 = 3 - g.n_seg;                   // two segments: the k and v projections alone
        p.q_out = (bf16_t *)ra->q_out;
        p.kc = (bf16_t *)ra->kv->k + (size_t)ra->layer * ra->kv->layer_elems;
        p.vc = (bf16_t *)ra->kv->v + (size_t)ra->layer * ra->kv->layer_elems;
        p.table = ra->table;
        p.R = ra->rows->R; p.pos0 = ra->rows->pos0; p.n_heads = ra->kv->n_heads;
        p.pos_stride = ra->kv->pos_stride; p.H = g.segN;
        p.N = g.n_seg * g.segN;
        p.tiles_n = p.N / BN;
        return launch_kb<EPI_QKV_ROPE>(p, kb, st);
    }
    p.N = g.n_seg * g.segN;
    p.tiles_n = p.N / BN;
    return g.epilogue == EPI_RESIDUAL ? launch_kb<EPI_RESIDUAL>(p, kb, st) : launch_kb<EPI_STORE>(p, kb, st);
}

// QKV and gate/up projections of decode steps of 17 .. 128 rows on the small tiles: row-major activations, the repacked
// weights where the model has them, no partial sums in memory, the sums of the split-K form.  64 rows of the 7B shape against
// that form and its reductions: QKV 31 + 12 -> 28 + 7 us (with rotation and KV write), gate/up 57 + 10 -> 41; 128 rows 41 + 14
// -> 37 + 8 and 75 + 16 -> 53.  (On the instruction and order of the 256 x 256 tiles QKV takes 27 and 35 us, gate/up 40 and 49.)
// The O and down projections have too few tiles (64 rows: 38 us and a norm of 6, split-K 25 and 7) and stay there.  Above 128
// rows the split-K form of the large tiles is faster: at 129 rows QKV 43 + 11 us against 55 + 8 here and gate/up 66 + 7 against 83,
// at 256 rows 45 + 15 against 51 + 10 and 70 + 10 against 81.  Returns 1 if handled, 0 if declined, < 0 on a launch error.
int try_gemm_bf16_dma_step(const GemmArgs &g, hipStream_t st) {
    if (g.epilogue != EPI_STORE && g.epilogue != EPI_SWIGLU) return 0;
    if (g.kblocked || g.M < 1 || g.M > 128 || g.K % 64 != 0 || g.K < 256 || g.a_rows < 256) return 0;
    if (g.epilogue == EPI_SWIGLU ? g.segN % 128 != 0 : g.segN % BN != 0) return 0;
    const int n_seg = g.epilogue == EPI_SWIGLU ? 2 : g.n_seg;
    bool wkb = (size_t)(g.segN + VLA_KB_PAD_ROWS) * g.K * 2 < ((size_t)1 << 31);
    for (int i = 0; i < n_seg; i++) wkb = wkb && g.Wkb[i];
    const void *const *W = wkb ? g.Wkb : g.W;
    DmaGemmParams p{};
    p.A = (const bf16_t *)g.A;
    p.W0 = (const bf16_t *)W[0]; p.W1 = (const bf16_t *)W[1]; p.W2 = (const bf16_t *)W[2];
    p.C = g.C; p.M = g.M; p.K = g.K; p.segN = g.segN; p.a_rows = g.a_rows; p.w_rows = g.segN + VLA_KB_PAD_ROWS;
    p.N = g.epilogue == EPI_SWIGLU ? g.segN : n_seg * g.segN;
    p.parts = gemm_decode_parts(p.N, p.K);
    auto go = [&](auto epi) {
        constexpr int EPI = decltype(epi)::value;
        const SmallTile tile = choose_tile<EPI>(p, 8, true).small;
        if (tile == TILE_LARGE) return 0;
        if (!wkb) return launch_tile<EPI, false, W_ROWS, true>(p, tile, st);
        return g.past_caches ? launch_tile<EPI, false, W_KBLOCKED_PAST, true>(p, tile, st) : launch_tile<EPI, false, W_KBLOCKED, true>(p, tile, st);
    };
    return g.epilogue == EPI_SWIGLU ? go(std::integral_constant<int, EPI_SWIGLU>{}) : go(std::integral_constant<int, EPI_STORE>{});
}

// Split-K form for forwards of at most 256 rows (one tile row): the K range is cut into 2, 4 or 8 equal parts so
// that tiles x parts workgroups are busy, each part's fp32 product goes to `scratch` ([parts][M][N], for SwiGLU
// N = gate columns then up columns) and launch_splitk_reduce adds the parts in order and applies the epilogue.
// Takes the QKV projection (fp32 output) and the gate/up projection; declines everything else, and problems
// where no such split leaves at least a fifth of the CUs more busy than without it.  Row-major operands.
int try_gemm_bf16_dma_splitk(const GemmArgs &g, void *scratch, size_t scratch_bytes, hipStream_t st) {
    if (g.kblocked || g.M < 1 || g.M > BM || g.a_rows < BM || g.K % 64 != 0 || !scratch) return 0;
    if (g.epilogue != EPI_STORE && g.epilogue != EPI_SWIGLU) return 0;
    if (g.segN % BN != 0) return 0;
    static int n_cu = 0;
    if (!n_cu) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1) {
            vla_set_error("gemm_bf16_dma: cannot read the compute-unit count");
            return VLA_EHIP;
        }
    }
    const int n_seg = g.epilogue == EPI_SWIGLU ? 2 : g.n_seg;
    const int N = n_seg * g.segN, tiles = N / BN, nh = g.K / HK;
    int splits = 1;
    while (splits < 8 && tiles * splits * 2 <= n_cu && (nh / (splits * 2)) % 2 == 0 && nh / (splits * 2) >= 8 &&
           nh % (splits * 2) == 0 && (size_t)(splits * 2) * g.M * N * sizeof(float) <= scratch_bytes)
        splits *= 2;
    if (splits < 2 || tiles * splits * 5 < n_cu * 3) return 0;
    DmaGemmParams p{};
    p.A = (const bf16_t *)g.A;
    p.W0 = (const bf16_t *)g.W[0]; p.W1 = (const bf16_t *)g.W[1]; p.W2 = (const bf16_t *)g.W[2];
    p.C = scratch; p.M = g.M; p.K = g.K; p.segN = g.segN;
    p.a_rows = g.a_rows; p.w_rows = 0; p.group = 4; p.splits = splits;
    p.tiles_m = 1; p.N = N; p.tiles_n = tiles;
    // repacked copies of the weights, where the caller has them and the 32-bit offsets of the loads cover a segment: the gate/up
    // projection of 256 rows 61 us with them, 66 without
    bool wkb = g.Wkb[0] && (size_t)(g.segN + VLA_KB_PAD_ROWS) * g.K * 2 < ((size_t)1 << 31);
    for (int i = 1; i < n_seg; i++) wkb = wkb && g.Wkb[i];
    if (wkb) {
        p.W0 = (const bf16_t *)g.Wkb[0]; p.W1 = (const bf16_t *)g.Wkb[1]; p.W2 = (const bf16_t *)g.Wkb[2];
        p.w_rows = g.segN + VLA_KB_PAD_ROWS;
    }
    int rc;
    {
        ProfScope ps(g.epilogue == EPI_SWIGLU ? "gemm_dma_splitk<swiglu>" : "gemm_dma_splitk<store>", 2.0 * g.M * g.K * (double)N, st);
        rc = wkb ? launch_plain<EPI_STORE, false, true>(p, st) : launch_plain<EPI_STORE, false>(p, st);
        if (rc != 1) return rc;
    }
    if (g.deferred_splits && g.epilogue == EPI_STORE) *g.deferred_splits = splits;
    else if ((rc = launch_splitk_reduce(g.epilogue, g.C, (const float *)scratch, splits, g.M, g.epilogue == EPI_SWIGLU ? g.segN : N, st))) return rc;
    return 1;
}

// Split-K form for multi-row problems with few output tiles (the LoRA-gradient products: 256 output columns, or a
// contraction over all rows of a micro-batch): the K range is cut into `parts` equal ranges so that tiles x parts
// items keep the CUs busy, each range's fp32 product goes to `scratch` ([parts][M][N]) and launch_splitk_reduce adds
// them in order.  Row-major operands, fp32 output only.  `parts` minimises a cost estimate (below); declines (0) when
// that leaves one part or the scratch is too small.
int try_gemm_bf16_dma_splitk_rows(const GemmArgs &g, void *scratch, size_t scratch_bytes, hipStream_t st) {
    if (g.kblocked || g.epilogue != EPI_STORE || g.M < 1 || g.K % 64 != 0 || g.K < 256 || !scratch) return 0;
    if (g.segN % BN != 0 || g.a_rows < (g.M + BM - 1) / BM * BM) return 0;
    static int n_cu = 0;
    if (!n_cu) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1) {
            vla_set_error("gemm_bf16_dma: cannot read the compute-unit count");
            return VLA_EHIP;
        }
    }
    const int N = g.n_seg * g.segN, tiles_m = (g.M + BM - 1) / BM, tiles = tiles_m * (N / BN), nh = g.K / HK;
    // cost in half-tile times (about 0.8 us): rounds of items x (half tiles per item + about 8 for an item's prologue
    // and fp32 epilogue), plus the reduction's traffic (0.5 MB written and read per tile and part, about 0.16)
    auto cost_of = [&](int parts) {
        const long rounds = (tiles * parts + n_cu - 1) / n_cu;
        return rounds * (nh / parts + 8) * 100 + (parts > 1 ? 16L * parts * tiles : 0);
    };
    int best = 1;
    long best_cost = cost_of(1);
    for (int parts = 2; parts <= 32; parts++) {
        const int per = nh / parts;
        if (nh % parts != 0 || (per & 1) || per < 8) continue;
        if ((size_t)parts * g.M * N * sizeof(float) > scratch_bytes) break;
        const long cost = cost_of(parts);
        if (cost < best_cost) { best_cost = cost; best = parts; }
    }
    if (best < 2) return 0;
    DmaGemmParams p{};
    p.A = (const bf16_t *)g.A;
    p.W0 = (const bf16_t *)g.W[0]; p.W1 = (const bf16_t *)g.W[1]; p.W2 = (const bf16_t *)g.W[2];
    p.C = scratch; p.M = g.M; p.K = g.K; p.segN = g.segN;
    p.a_rows = g.a_rows; p.w_rows = 0; p.group = 4; p.splits = best;
    p.tiles_m = tiles_m; p.N = N; p.tiles_n = N / BN;
    {
        ProfScope ps("gemm_dma_splitk_rows<store>", 2.0 * g.M * g.K * (double)N, st);
        const int rc = launch_plain<EPI_STORE, false>(p, st);
        if (rc != 1) return rc;
    }
    const int rc = launch_splitk_reduce(EPI_STORE, g.C, (const float *)scratch, best, g.M, N, st);
    return rc ? rc : 1;
}

namespace {

// Repack of one weight matrix [N, K] into [K / 32][N + pad][32]: a thread moves one 16-byte piece (the pad rows
// are never read).
__global__ void __launch_bounds__(256) weight_kblock_kernel(bf16_t *dst, const bf16_t *src, int N, int K) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;       // (n, 8-column piece)
    const int pieces = K / 8;
    if (idx >= (size_t)N * pieces) return;
    const int n = (int)(idx / pieces), pc = (int)(idx - (size_t)n * pieces);
    const bf16x8_t v = *(const bf16x8_t *)(src + (size_t)n * K + pc * 8);
    *(bf16x8_t *)(dst + ((size_t)(pc >> 2) * (N + VLA_KB_PAD_ROWS) + n) * 32 + (pc & 3) * 8) = v;
}

}  // namespace

int launch_weight_kblock(bf16_t *dst, const bf16_t *src, int N, int K, hipStream_t st) {
    if (K % 32 != 0) { vla_set_error("weight repack: K = %d is not a multiple of 32", K); return VLA_ESHAPE; }
    const size_t total = (size_t)N * (K / 8);
    if (total == 0) return 0;
    weight_kblock_kernel<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(dst, src, N, K);
    return vla_check_launch("weight_kblock");
}
