// Internal declarations shared by the translation units of libvla (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "../../include/vla.h"

typedef __bf16 bf16_t;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef int i32x4_v __attribute__((ext_vector_type(4)));

#define VLA_WAVE 64

// ------------------------------------------------------------------------------------------
// KV buffer view.  One layer of K is [n_seq][n_heads][d/8][pos_stride][8] (eight consecutive
// head dims of one position are contiguous: the 16-byte unit both the streaming decode kernel
// and the MFMA operand loads want); one layer of V is [n_seq][n_heads][pos_stride][d].
// ------------------------------------------------------------------------------------------
struct KvView {
    void *k, *v;            // base of layer 0
    size_t layer_elems;     // elements per layer (same for K and V)
    int n_seq, n_heads, d, pos_stride;
};

struct RowsArgs {           // one forward over n_seq sequences x R new rows each
    int n_seq, R, pos0;     // row r of a sequence sits at absolute position pos0 + r
    int full_from;          // rows at positions >= full_from attend to all pos0 + R keys,
                            // rows below attend causally (keys 0..position)
};

// EPI_QKV_ROWS and EPI_SWIGLU_KEEP are those of the gradient pass (row-major operands, direct-to-LDS kernels only): rotated q | k | v
// as rows of 3H instead of the KV layout, and SwiGLU with its pre-activations.  EPI_SWIGLU_GRAD is the input gradient of the down projection (segK)
// with SwiGLU's own behind it: from the product d act and the pre-activations, d gate | d up.
enum GemmEpilogue { EPI_STORE = 0, EPI_RESIDUAL = 1, EPI_SWIGLU = 2, EPI_QKV_ROPE = 3, EPI_QKV_ROWS = 4, EPI_SWIGLU_KEEP = 5, EPI_SWIGLU_GRAD = 6 };
constexpr bool epi_plain(int e) { return e == EPI_STORE || e == EPI_RESIDUAL || e == EPI_SWIGLU_GRAD; }
constexpr bool epi_swiglu(int e) { return e == EPI_SWIGLU || e == EPI_SWIGLU_KEEP; }
constexpr bool epi_qkv(int e) { return e == EPI_QKV_ROPE || e == EPI_QKV_ROWS; }

// Extra arguments of EPI_QKV_ROPE: the QKV projection whose epilogue rotates q and k and writes q to
// q_out [M, H] and k, v straight into layer `layer` of the KV buffer (head_dim 128 only).
struct QkvRopeArgs {
    void *q_out;            // may be NULL when the projection has no q segment (n_seg = 2: k and v only)
    const float2 *table;    // [R][d/2] (cos, sin)
    const KvView *kv;
    int layer;
    const RowsArgs *rows;
};

// k-blocked layouts ([K / 32][rows][32]) pad the row count of a block by this much, so that the 32-column blocks
// of one row panel do not sit an exact power-of-two distance apart.  (A precaution only: the L2's fetch traffic of
// the k-blocked GEMM, 2.3 times that of the row-major one, was the same with and without the pad, and also with a
// pad chosen to spread consecutive blocks over distinct sets of a modulo-indexed 4 MB cache.)
constexpr int VLA_KB_PAD_ROWS = 32;

struct GemmArgs {
    const void *A;          // [M, K] row-major (lda = K), storage dtype (or fp32 for fp32 models)
    const void *W[3];       // up to three weight segments, each [segN, K] row-major
    const void *Wkb[3];     // the same segments repacked k-blocked ([K / 32][segN + pad][32]) or NULL: kernels that stream
                            // the weights from HBM with row-major activations (decode forwards) prefer these
    int n_seg, segN;        // N = n_seg * segN (EPI_SWIGLU: W[0] = gate, W[1] = up, N = segN)
    void *C;                // EPI_STORE: fp32 [M, N]; EPI_SWIGLU: storage dtype [M, N], EPI_SWIGLU_GRAD: [M, 2N]; EPI_RESIDUAL: fp32 [M, N]
    const float *res;       // EPI_RESIDUAL: what the product is added to, fp32 [M, N]; NULL: C (multi-row kernels alone: any other array)
    int M, K;
    int epilogue;
    const QkvRopeArgs *rope;   // EPI_QKV_ROPE, EPI_QKV_ROWS (q_out [M, 3H]; of kv only n_heads and d; two segments: k and v, q's third stays)
    float *pre;             // EPI_SWIGLU_KEEP (out), EPI_SWIGLU_GRAD (in): gate | up pre-activations, fp32 [M, 2N]
    int kblocked;           // A (a_rows rows per 32-column block), the weights (segN rows per block, each segment
                            // on its own) and a SwiGLU output are stored [K / 32][rows][32]: direct-to-LDS kernel only
    int a_rows;             // rows of A that may be read (>= M; contents past M arbitrary): the MFMA kernel
                            // loads whole 256-row tiles and declines if the buffer does not cover them
    int step;               // a decode step (one row per sequence): the weight-streaming kernel of few rows may take it
    int past_caches;        // ... whose weights, where they are repacked, are read past the caches
    const float *norm_x, *norm_gain;   // not NULL (steps for which gemm_stream_norms; fp32 models, K a multiple of 4): A is
    float norm_eps;                    // RMSNorm(norm_x) norm_gain, formed by the kernel from the fp32 rows [M, K]
    int *deferred_splits;   // not NULL (EPI_STORE and EPI_RESIDUAL of the split-K kernels): the kernel leaves its n
                            // partial products [n][M][N] at the start of the scratch buffer, puts n here and does not
                            // reduce them (the caller's next kernel adds them in order); 0 here: C is complete
    int segK;               // not 0 (EPI_STORE or EPI_SWIGLU_GRAD, bf16): an input gradient, C[M, segN] = A[M, n_seg segK] . [W[0]; W[1]; ..] with segments
                            // [segK, segN] as the forward has them; K = n_seg segK
    void *split_scratch;    // not NULL (EPI_STORE, row-major bf16): device scratch of split_scratch_bytes through which a
    size_t split_scratch_bytes;   // multi-row problem with few output tiles may cut its K range into parts
};

// ---- generic (any shape, fp32 or bf16 storage) kernels: kernels_generic.hip -----------------
template <typename T>
int launch_embed_prefix(float *X, const T *patch, const int32_t *ids, const T *embed, int n_seq, int P,
                        int T_, int row_stride_rows, int H, int vocab, hipStream_t st);
template <typename T>
int launch_embed_tokens(float *X, const int32_t *bins, int bins_stride, int n_tok, const T *embed,
                        int n_seq, int rows_per_seq, int row0, int H, int vocab, hipStream_t st);
template <typename T>
int launch_embed_slots(float *X, const T *slot_embed, int n_seq, int A, int rows_per_seq, int row0,
                       int H, hipStream_t st);
template <typename T>
int launch_rmsnorm(T *out, const float *X, const float *gain, int M, int H, float eps, hipStream_t st);
int launch_final_norm_rows(float *out, const float *X, const float *gain, int n_seq, int rows_per_seq,
                           int row0, int n_rows, int H, float eps, hipStream_t st);
template <typename T>
int launch_gemm_generic(const GemmArgs &g, hipStream_t st);
int launch_rope_table(float2 *table, int R, int pos0, int d, float theta, hipStream_t st);
// qkv is the fp32 [M, 3H] output of the QKV projection (never rounded before the rotation); the
// rotated q goes to q_out [M, H] in the storage dtype, k and v to the KV layout.
template <typename T>
int launch_rope_kv_write(T *q_out, const float *qkv, const float2 *table, const KvView &kv, int layer,
                         const RowsArgs &ra, int H, hipStream_t st);
template <typename T>
int launch_attention_generic(T *out, const T *q, const KvView &kv, int layer, const RowsArgs &ra,
                             int H, hipStream_t st);
// fp32 decode step (one row per sequence): the same straight from the QKV projection [n_seq, 3H], with rotation and KV write
int launch_attention_step_qkv(float *out, const float *qkv, const float2 *table, const KvView &kv, int layer, const RowsArgs &ra, int H,
                              hipStream_t st);
// rows first .. first + count - 1 of each of n_seq sequences of R rows, packed
int launch_gather_rows(float *Xt, const float *X, int n_seq, int R, int first, int count, int H, hipStream_t st);
// rotary on q alone: qf fp32 [n_seq * count, H]; packed row m sits at table row first + m % count
template <typename T>
int launch_rope_q(T *q_out, const float *qf, const float2 *table, int n_seq, int count, int first, int n_heads, int d, int H,
                  hipStream_t st);
// Row i of h produces output index o = i * out_stride + out_off: bins_out[o], logp[o], ent[o],
// logits[o * 256 ..]; it reads gumbel[o * 256 ..] (if any) and given_bins[o] (if any: then the
// log-prob is that of the given bin and nothing is sampled).  If X_next is not NULL the embedding
// of token vocab - 256 + bin is written to X_next[i * H ..] as fp32.
// next (with X_next, up to VLA_HEAD_PARTIAL_ROWS rows): what the next decode step needs besides its residual rows, its first
// norm (gain NULL: not wanted) and its row of the rotation table
struct NextStep { void *nrm; const float *gain; float eps; float2 *table; int pos, d; float theta; };
// norm: h is the residual stream and its final norm the head's to form; squares (up to VLA_HEAD_PARTIAL_ROWS rows): [head_chunks(H)][n_rows]
struct HeadNorm { const float *gain; float eps; float *squares; };
template <typename T>
int launch_head_sample(const float *h, const T *lm_head_bins, int n_rows, int H, float temperature,
                       const float *gumbel, const int32_t *given_bins, int32_t *bins_out, float *logp,
                       float *ent, float *logits, int out_stride, int out_off, float *X_next,
                       const T *embed, int vocab, float *scratch, hipStream_t st, const NextStep *next = nullptr, const HeadNorm *norm = nullptr);
// Partial logits h . W^T of n_rows rows, P[head_chunks(H)][n_rows][256] to be added in chunk order.
int head_chunks(int H);
template <typename T>
int launch_head_logits(const float *h, const T *lm_head_bins, float *P, int n_rows, int H, hipStream_t st);
// scratch of launch_head_sample for n_rows rows (device, fp32 partial logits; none above VLA_HEAD_PARTIAL_ROWS rows)
constexpr int VLA_HEAD_PARTIAL_ROWS = 4096;
size_t head_scratch_bytes(int n_rows, int H);
int launch_value_head(float *value, const float *h, const float *w, float b, const float *bias, int vd, int n,
                      int H, int h_stride, hipStream_t st);

// Sums and maxima over lanes by lane moves of the vector ALU instead of through LDS, a latency of 60 cycles and more a step; the order of
// additions is that of __shfl_xor over the same distances.  One step with lane ^ O (O = 8, 16 or 32; f is symmetric):
template <int CTRL> __device__ __forceinline__ float vla_dpp(float v) {
    const int i = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false));
}
// The values of the two lanes that differ in O (32 or 16), the lower lane's first.
struct VlaPair { float a, b; };
template <int O> __device__ __forceinline__ VlaPair vla_pair(float v) {
    static_assert(O == 16 || O == 32, "distance");
    const unsigned u = __builtin_bit_cast(unsigned, v);
    if constexpr (O == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        return {__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])};
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        return {__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])};
    }
}
template <int O, typename F> __device__ __forceinline__ float vla_fold_step(float v, F f) {
    if constexpr (O == 8) return f(v, vla_dpp<0x128>(v));          // row_ror:8
    else {
        const VlaPair p = vla_pair<O>(v);
        return f(p.a, p.b);
    }
}
// Over the 16 lanes of a row, distances 8, 4, 2, 1 (lane ^ 12 has what lane ^ 4 has once lanes ^ 8 agree: a rotation will do), and over all 64.
template <typename F> __device__ __forceinline__ float vla_row_fold(float v, F f) {
    v = vla_fold_step<8>(v, f);
    v = f(v, vla_dpp<0x124>(v));        // row_ror:4
    v = f(v, vla_dpp<0x4e>(v));         // quad_perm 2 3 0 1
    return f(v, vla_dpp<0xb1>(v));      // quad_perm 1 0 3 2
}
template <typename F> __device__ __forceinline__ float vla_wave_fold(float v, F f) { return vla_row_fold(vla_fold_step<16>(vla_fold_step<32>(v, f), f), f); }
struct VlaAdd { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct VlaMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
__device__ __forceinline__ float vla_wave_sum(float v) { return vla_wave_fold(v, VlaAdd{}); }
__device__ __forceinline__ float vla_wave_max(float v) { return vla_wave_fold(v, VlaMax{}); }

// One pair (a, b) rotated by (cos, sin), rounded once after one fused multiply-add each: written out where two kernels must
// agree bit for bit (the compiler fuses either product of a sum of two).
__device__ __forceinline__ float vla_rotate_lo(float a, float b, float co, float si) { return __builtin_fmaf(a, co, -(b * si)); }
__device__ __forceinline__ float vla_rotate_hi(float a, float b, float co, float si) { return __builtin_fmaf(b, co, a * si); }

// (cos, sin) of pair i at a position, evaluated in fp64
__device__ __forceinline__ float2 vla_rope_entry(int pos, int i, int d, float theta) {
    const double inv = pow((double)theta, -2.0 * (double)i / (double)d), phi = (double)pos * inv;
    return make_float2((float)cos(phi), (float)sin(phi));
}

// RMSNorm of a row held by 256 threads: piece j of thread t is elements 4 (256 j + t) .. + 3 (those below H), g the gain's.
// red: 4 floats of LDS.  The one order of sums of all norms by 256 threads.
template <typename T>
__device__ __forceinline__ void vla_norm_held(T *o, const f32x4_t (&v)[8], const f32x4_t (&g)[8], int H, float eps, float *red) {
    typedef T t4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
    const int t = threadIdx.x;
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < 8; j++)
        if ((j * 256 + t) * 4 < H) {
#pragma unroll
            for (int e = 0; e < 4; e++) ss += v[j][e] * v[j][e];
        }
    ss = vla_wave_sum(ss);
    __syncthreads();
    if ((t & 63) == 0) red[t >> 6] = ss;
    __syncthreads();
    ss = red[0] + red[1] + red[2] + red[3];
    const float r = 1.0f / sqrtf(ss / (float)H + eps);
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int i = (j * 256 + t) * 4;
        if (i < H) {
            t4 w;
#pragma unroll
            for (int e = 0; e < 4; e++) w[e] = (T)(v[j][e] * r * g[j][e]);
            *(t4 *)(o + i) = w;
        }
    }
}

// silu(gate) * up of the bf16 fast paths: hardware exponential and reciprocal (1 ulp each, far below
// the bf16 rounding that follows); one formula for the prefill and the decode GEMMs so that both
// round the same way.
__device__ __forceinline__ float vla_silu_mul(float gate, float up) {
    return gate * __builtin_amdgcn_rcpf(1.0f + __expf(-gate)) * up;
}
// ... and that of the gradient pass, whose backward differentiates it at the kept pre-activations: the library's exponential
// and a division.
__device__ __forceinline__ float vla_silu_mul_exact(float gate, float up) { return gate / (1.0f + expf(-gate)) * up; }
// ... which is d gate = d act up silu'(gate), d up = d act silu(gate); silu'(t) = s (1 + t (1 - s)), s = sigmoid(t).
__device__ __forceinline__ void vla_swiglu_grad(float gate, float up, float d_act, float &d_gate, float &d_up) {
    const float s = 1.0f / (1.0f + expf(-gate));
    d_gate = d_act * up * s * (1.0f + gate * (1.0f - s));
    d_up = d_act * gate * s;
}

// Maps a linear work-item id of the large-tile GEMMs to an output tile.  Workgroups are dealt round-robin to
// the eight XCDs, each with its own L2.  The ids of XCD y, taken in order, walk the tile rows y, y + 8, y + 16, ...
// in column panels of `GROUP` of those rows, so that the ~32 tiles resident on an XCD (4 x 8) share activation and
// weight rows in its L2 -- and all eight XCDs start at tile column 0 and move through the columns together, so
// that a weight panel that one XCD pulls from memory is found in the memory-side cache by the other seven
// (contiguous ranges of rows per XCD do the same only when the tile count per XCD is a whole number of panels).
// The row sets differ by one row at most while the ids are dealt evenly: an XCD that is through with its own rows
// takes, at the end, the tiles that the other XCDs' shares of ids do not reach.
// The arithmetic is the same in every lane; the results go back to scalar registers so that everything derived
// from them (tile base addresses) stays scalar.
__device__ __forceinline__ void vla_tile_of_block(int pid, int tiles_m, int tiles_n, int &tm, int &tn, int GROUP = 4) {
    const int total = tiles_m * tiles_n;
    const int q = total >> 3, r = total & 7;                 // XCDs below r are dealt q + 1 ids, the others q
    const int rows_lo = tiles_m >> 3, extra = tiles_m & 7;   // XCDs below `extra` own rows_lo + 1 tile rows
    auto ids_of = [&](int z) { return q + (z < r ? 1 : 0); };
    auto tiles_of = [&](int z) { return (rows_lo + (z < extra ? 1 : 0)) * tiles_n; };
    const int xcd = pid & 7, local = pid >> 3;
    int y = xcd, l = local;                                  // tile l of XCD y's own rows
    if (local >= tiles_of(xcd)) {
        int e = local - tiles_of(xcd);                       // index into the tiles left over, pooled in XCD order
        for (int z = 0; z < 8; z++)
            if (z < xcd) e += max(ids_of(z) - tiles_of(z), 0);
        for (int z = 0; z < 8; z++) {
            const int left = tiles_of(z) - ids_of(z);
            if (left > 0) {
                if (e < left) { y = z; l = ids_of(z) + e; break; }
                e -= left;
            }
        }
    }
    const int rows_y = rows_lo + (y < extra ? 1 : 0);
    // GROUP = 4: measured best of 1, 2, 4, 6, 8, 16, 32 on the 7B shapes (the QKV projection passes 2)
    const int panel = l / (GROUP * tiles_n);
    const int first = panel * GROUP;
    const int rows = min(GROUP, rows_y - first);
    const int in_panel = l - panel * GROUP * tiles_n;
    tm = __builtin_amdgcn_readfirstlane(y + 8 * (first + in_panel % rows));
    tn = __builtin_amdgcn_readfirstlane(in_panel / rows);
}

// ---- gfx950 fast paths (bf16, aligned shapes); each returns 1 if it handled the call, 0 if the
// shape is outside what it supports (caller then uses the generic kernel), <0 on launch error ----
int try_gemm_bf16_dma(const GemmArgs &g, hipStream_t st);
int try_gemm_bf16_dma_step(const GemmArgs &g, hipStream_t st);
int try_gemm_bf16_dma_splitk(const GemmArgs &g, void *scratch, size_t scratch_bytes, hipStream_t st);
int try_gemm_bf16_dma_splitk_rows(const GemmArgs &g, void *scratch, size_t scratch_bytes, hipStream_t st);
int launch_weight_kblock(bf16_t *dst, const bf16_t *src, int N, int K, hipStream_t st);
// qkv: `splits` partial copies of the fp32 [M, 3H] projection, `split_stride` floats apart, added in order
int launch_rope_kv_write_bf16(bf16_t *q_out, const float *qkv, int splits, size_t split_stride, const float2 *table,
                              const KvView &kv, int layer, const RowsArgs &ra, int H, hipStream_t st);
// x[m] += sum of the `splits` partial rows P[k][m] (in order); then, if gain != NULL, out[m] = RMSNorm(x[m]) * gain as
// bf16, row-major.  Returns 1 if handled (H a multiple of 1024, at most 8192), 0 otherwise.
int try_reduce_residual_rmsnorm_bf16(bf16_t *out, float *X, const float *P, int splits, int M, int H, const float *gain,
                                     float eps, hipStream_t st);
// kb_rows = 0: row-major output [M, H]; else k-blocked [H / 32][kb_rows][32]
int try_rmsnorm_bf16(bf16_t *out, const float *X, const float *gain, int M, int H, float eps, int kb_rows, hipStream_t st);
int gemm_decode_parts(int N, int K);       // (N: output columns, gate columns alone for SwiGLU)
bool gemm_stream_norms(int M, int K, int segN);
int try_gemm_bf16_stream(const GemmArgs &g, hipStream_t st);
int try_gemm_bf16_skinny(const GemmArgs &g, void *scratch, hipStream_t st);
int try_gemm_bf16_mid(const GemmArgs &g, void *scratch, size_t scratch_bytes, hipStream_t st);
int launch_splitk_reduce(int epilogue, void *C, const float *P, int splits, int M, int N, hipStream_t st);
size_t gemm_skinny_scratch_bytes(int M, int max_n);
// out_kb_rows = 0: row-major output [M, H]; else k-blocked [H / 32][out_kb_rows][32]
int try_attention_prefill_bf16(bf16_t *out, const bf16_t *q, const KvView &kv, int layer,
                               const RowsArgs &ra, int H, void *vt_scratch, int out_kb_rows, hipStream_t st);
// one new row per sequence; past_caches: K and V are read past the caches
int try_attention_decode_bf16(bf16_t *out, const bf16_t *q, const KvView &kv, int layer,
                              const RowsArgs &ra, int H, bool past_caches, hipStream_t st);
bool attention_decode_fuses_qkv(const KvView &kv, const RowsArgs &ra);
int launch_attention_decode_qkv(bf16_t *out, const float *qkv, const float2 *table, const KvView &kv, int layer, const RowsArgs &ra,
                                int H, bool past_caches, hipStream_t st);
size_t attention_prefill_scratch_bytes(int n_seq, int n_heads, int d, int n_keys);

// Attention of the gradient pass with its [rows x keys] matrices kept (attn_rows.hip).  qkv: rotated q | k | v, bf16 [n_seq * R, 3H];
// the queries are the last Rq rows of every sequence; P, S: [n_seq * n_heads][Rq][ldp] fp32.
//   forward: rows = qkv, S = the probabilities (out), out = bf16 [n_seq * Rq, H];  scale: of the scores
//   backward: rows = d out, fp32 [n_seq * Rq, H], P the probabilities, S = the scores' gradients (out), out = d q, fp32 [n_seq * R, 3H], the
//   queries' rows;  scale: of d q
// Return 1 if handled, 0 if declined, < 0 on a launch error.
struct AttnRowsArgs { const void *rows; const bf16_t *qkv; float *S; const float *P; void *out; int R, Rq, ldp, n_heads, H, full_from; float scale; };
int try_attention_rows_forward(const AttnRowsArgs &a, int n_seq, hipStream_t st);
int try_attention_rows_backward(const AttnRowsArgs &a, int n_seq, hipStream_t st);
// The contractions over the queries that follow, the transposed rotation and the rounding: bf16 d k | d v in rows of ld_kv, d v H columns
// behind d k, and d q in rows of ld_q, all n_seq * R of them (zeros where there is no query) or q_packed: the n_seq * Rq that have one; from
// P, dS ([n_seq * n_heads][Rq][ldp] fp32, zero outside the mask), dO (fp32 [n_seq * Rq, H]), dq (fp32 [n_seq * R, 3H], the queries' rows of its
// first third) and q of qkv.  scale: of d k.  Same return values; attention_cols_takes: whether it does, before anything is launched.
struct AttnColsArgs { const float *P, *dS, *dO, *dq; const bf16_t *qkv; const float2 *table; bf16_t *out_q, *out_k; int ld_q, ld_kv, q_packed, R, Rq, ldp, n_heads, H, full_from; float scale; };
bool attention_cols_takes(const AttnColsArgs &a);
int try_attention_cols(const AttnColsArgs &a, int n_seq, hipStream_t st);

// LoRA gradients of n_p projections that share their input (factors a[p] [rank, in], b[p] [out, rank] in the storage type,
// gradients da[p], db[p] fp32 of the same shapes): lora_grad.hip
struct LoraProducts { const void *a[3], *b[3]; float *da[3], *db[3]; int n_p, in, out, rank; };
int try_lora_products_bf16(const LoraProducts &g, const void *X, const void *dY, int M, float scale, bool accumulate, void *scratch,
                           size_t bytes, hipStream_t st, const void *packed);
size_t lora_packed_bytes(const LoraProducts &g);           // 0: a group that try_lora_products_bf16 declines
int launch_lora_pack(const LoraProducts *g, int n, void *packed, hipStream_t st);

int vla_force_generic();                                   // the mask of vla_debug_force_generic
int vla_check_launch(const char *what);
int vla_allow_lds(const void *kernel, size_t bytes);       // dynamic LDS of a kernel beyond the default limit; 0 or VLA_EHIP
void vla_set_error(const char *fmt, ...);

// The host-side model object behind the opaque handle of the C ABI.
struct vla_model {
    vla_config cfg;
    vla_weights w;
    std::vector<vla_layer_weights> layers;
    std::vector<vla_layer_weights> packed;   // k-blocked copies of the seven projection matrices (vla_prepack), or empty
};
int vla_check_config(const vla_config *c);                                   // VLA_OK or the error code, message set
int vla_check_rows_per_pass(const vla_config &c, long n_seq, long rows_per_seq);
// C = A . W^T of a multi-row forward (row-major operands): the MFMA kernels where the shape allows, else the generic one
int vla_gemm_dispatch(const vla_config &c, const GemmArgs &g, hipStream_t st);
// The same with one of the gradient pass's epilogues: 1 if handled, 0 if declined, < 0 on a launch error
int vla_gemm_fused(const vla_config &c, const GemmArgs &g, hipStream_t st);
// The embedded rows of n rollouts' teacher-forced forward and its first n_layers layers (the kernels vla_logprob_recompute runs;
// n_layers 0: the rows alone): the fp32 residual stream at the input of layer l is left in keep + l * n * R * H ([n * R, H] each, n_layers
// + 1 of them; the layers read and write it there).  fw_ws: device scratch of vla_forward_streams_bytes(c, n_max, R) bytes with n <= n_max.
size_t vla_forward_streams_bytes(const vla_config &c, int n_max, int R);
int vla_forward_streams(vla_model *m, void *fw_ws, int n_max, const void *patch, const int32_t *ids, const int32_t *bins, int n,
                        int P, int T, int A, int mode, const void *slot_embed, int n_layers, float *keep, hipStream_t st);

// Profiling scope: when profiling is enabled, records an event pair around the launches issued
// during its lifetime, tagged with `label` (a string literal) and the algorithmic work.
struct ProfScope {
    ProfScope(const char *label, double work, hipStream_t st);
    ~ProfScope();
    int slot;
    hipStream_t st;
};
