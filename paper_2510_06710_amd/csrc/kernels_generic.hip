// Shape-generic kernels of libvla: every step of the rollout / recompute path for any supported
// dimensions, with fp32 or bf16 storage (fp32 arithmetic throughout).  The tiny fp32 workload
// runs entirely on these; the bf16 7B-shape workloads replace the GEMMs and the attention by the
// MFMA / streaming kernels of the other translation units and keep the rest.
#include "vla_internal.h"

#include <type_traits>

namespace {

typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));   // caller-owned fp32 arrays: element alignment

__device__ __forceinline__ float to_f(float v) { return v; }
__device__ __forceinline__ float to_f(bf16_t v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f(float v);
template <> __device__ __forceinline__ float from_f<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f<bf16_t>(float v) { return (bf16_t)v; }

// Sum over a 256-thread block; `red` is 4 floats of LDS.  Every thread gets the total.
__device__ __forceinline__ float block_sum_256(float v, float *red) {
    v = vla_wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

// ---------------------------------------------------------------------------------- embedding
// One row in fp32, four elements per thread and step (H is a multiple of 16; the source has element alignment).  Element by
// element the 73,728 x 4096 prefix rows of 256 environments took 523 us, now 295.
template <typename T>
__device__ __forceinline__ void widen_row(float *dst, const T *src, int H) {
    typedef T t4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
#pragma unroll 4
    for (int i = threadIdx.x * 4; i < H; i += blockDim.x * 4) {
        const t4 v = *(const t4 *)(src + i);
        *(f32x4_t *)(dst + i) = f32x4_t{to_f((T)v[0]), to_f((T)v[1]), to_f((T)v[2]), to_f((T)v[3])};
    }
}

// Prefix assembly: x_p = patch[p] (p < P), x_{P+t} = embed[ids[t]].
template <typename T>
__global__ void embed_prefix_kernel(float *X, const T *patch, const int32_t *ids, const T *embed, int P,
                                    int T_, int rows_per_seq, int H, int vocab) {
    int S = P + T_;
    int s = blockIdx.x / S, p = blockIdx.x % S;
    const T *src;
    if (p < P) {
        src = patch + ((size_t)s * P + p) * H;
    } else {
        int id = ids[(size_t)s * T_ + (p - P)];
        id = min(max(id, 0), vocab - 1);
        src = embed + (size_t)id * H;
    }
    float *dst = X + ((size_t)s * rows_per_seq + p) * H;
    widen_row(dst, src, H);
}

// Stored action tokens (teacher forcing): row row0 + j of sequence s is embed[vocab-256+bins[s][j]].
template <typename T>
__global__ void embed_tokens_kernel(float *X, const int32_t *bins, int bins_stride, int n_tok,
                                    const T *embed, int rows_per_seq, int row0, int H, int vocab) {
    int s = blockIdx.x / n_tok, j = blockIdx.x % n_tok;
    int b = bins[(size_t)s * bins_stride + j];
    b = min(max(b, 0), VLA_N_BINS - 1);
    const T *src = embed + (size_t)(vocab - VLA_N_BINS + b) * H;
    float *dst = X + ((size_t)s * rows_per_seq + row0 + j) * H;
    widen_row(dst, src, H);
}

template <typename T>
__global__ void embed_slots_kernel(float *X, const T *slot_embed, int A, int rows_per_seq, int row0, int H) {
    int s = blockIdx.x / A, a = blockIdx.x % A;
    const T *src = slot_embed + (size_t)a * H;
    float *dst = X + ((size_t)s * rows_per_seq + row0 + a) * H;
    widen_row(dst, src, H);
}

// ---------------------------------------------------------------------------------- RMSNorm
// n_i = x_i / sqrt(mean(x^2) + eps) * g_i; one 256-thread block per row, which stays in registers between the sum and
// the scaling (H is a multiple of 16 and at most 8192: up to eight 16-byte pieces per thread).  All loads are in flight
// at once: with one element per thread and step the final norm of one row of 4096 took 9.2 us, a chain of sixteen
// memory latencies, now 5 us.
template <typename T>
__device__ __forceinline__ void norm_row(T *o, const float *x, const float *gain, int H, float eps, float *red) {
    f32x4_t v[8], g[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int i = (j * 256 + threadIdx.x) * 4;
        if (i < H) {
            v[j] = *(const f32x4_t *)(x + i);
            g[j] = *(const f32x4_u *)(gain + i);
        }
    }
    vla_norm_held<T>(o, v, g, H, eps, red);
}
template <typename T>
__global__ void __launch_bounds__(256) rmsnorm_kernel(T *out, const float *X, const float *gain, int H, float eps) {
    __shared__ float red[4];
    norm_row<T>(out + (size_t)blockIdx.x * H, X + (size_t)blockIdx.x * H, gain, H, eps, red);
}

// Final norm of selected rows: out row (s * n_rows + j) = norm(X[s * rows_per_seq + row0 + j]).
__global__ void __launch_bounds__(256) final_norm_rows_kernel(float *out, const float *X, const float *gain, int rows_per_seq,
                                                             int row0, int n_rows, int H, float eps) {
    __shared__ float red[4];
    const int s = blockIdx.x / n_rows, j = blockIdx.x % n_rows;
    norm_row<float>(out + (size_t)blockIdx.x * H, X + ((size_t)s * rows_per_seq + row0 + j) * H, gain, H, eps, red);
}

// ---------------------------------------------------------------------------------- GEMM
// C[M, N] = A[M, K] . W^T with W given as n_seg row blocks [segN, K], any sizes.  EPI_SWIGLU computes
// silu(A.Wg^T) * (A.Wu^T) with both products in one pass.
//
// fp32 MFMA (a lane's four consecutive K elements take turns as v_mfma_f32_16x16x4_f32's one element per lane), operands
// straight from global memory.  A workgroup owns MB x NBK blocks of 16 x 16 outputs; K is dealt to its eight waves in
// blocks of 16 and the waves' sums are added in wave order through LDS, so an output's additions are the same whatever
// the tile.  Few outputs (1 x 1 blocks) are bound by latency: every load of a wave is in flight at once, and a tile of
// 16 x 16 makes enough workgroups.  Many outputs (4 x 2) share the operands.  Measured in fp32 against a 64 x 64 tile
// on the vector ALU that paid one memory latency per 16 columns of K: 8 x 256 x 688 (M x N x K, down projection of the
// tiny decoder) 155 -> 5 us, 8 x 768 x 256 39 -> 3.5 us, 512 x 768 x 256 53 -> 9 us.
template <typename T, bool VEC>
__device__ __forceinline__ f32x4_t load4(const T *p, int k, int K) {
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    if (VEC) {
        if (k < K) {
            typedef T t4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
            const t4 w = *(const t4 *)(p + k);
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = to_f(w[e]);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; e++)
            if (k + e < K) v[e] = to_f(p[k + e]);
    }
    return v;
}

// NORM (fp32): A is the residual stream and the product that of RMSNorm(A) gain: (A gain) . W^T as the loads bring A, each row times
// its 1 / rms at the end, whose squares the same loads bring.
template <typename T, int EPI, bool VEC, int MB, int NBK, int UN, bool NORM>
__global__ void __launch_bounds__(512) gemm_generic_kernel(const T *A, const T *W0, const T *W1, const T *W2, int segN, void *Cv,
                                                           const float *res, int M, int N, int K, const float *gain, float eps) {
    constexpr int NW = 8, NP = (EPI == EPI_SWIGLU) ? 2 : 1;
    constexpr bool WIDE = sizeof(T) == 4 && VEC;
    __shared__ __attribute__((aligned(16))) f32x4_t part[NW][NP * MB * NBK][64];
    __shared__ float squares[NORM ? NW : 1][NORM ? MB * 16 : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
    const int m0 = blockIdx.y * (16 * MB), n0 = blockIdx.x * (16 * NBK);
    const T *a[MB], *w[NP][NBK];
#pragma unroll
    for (int i = 0; i < MB; i++) a[i] = A + (size_t)min(m0 + i * 16 + l16, M - 1) * K;
#pragma unroll
    for (int j = 0; j < NBK; j++) {
        const int n = min(n0 + j * 16 + l16, N - 1);      // (past the end: loaded, not stored)
        if (EPI == EPI_SWIGLU) {
            w[0][j] = W0 + (size_t)n * K;
            w[NP - 1][j] = W1 + (size_t)n * K;
        } else {
            const int seg = n / segN, nn = n % segN;
            w[0][j] = (seg == 0 ? W0 : (seg == 1 ? W1 : W2)) + (size_t)nn * K;
        }
    }
    f32x4_t acc[NP][MB][NBK];
#pragma unroll
    for (int b = 0; b < NP; b++)
#pragma unroll
        for (int i = 0; i < MB; i++)
#pragma unroll
            for (int j = 0; j < NBK; j++) acc[b][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float ss[MB];
#pragma unroll
    for (int i = 0; i < MB; i++) ss[i] = 0.f;
#pragma unroll 1
    for (int g = wave * 16; g < K; g += NW * 16 * UN) {
        f32x4_t av[UN][MB], wv[UN][NP][NBK], gv[UN];
#pragma unroll
        for (int i = 0; i < UN; i++) {
            const int k = g + i * NW * 16 + kq * 4;       // (past K: zeros)
#pragma unroll
            for (int x = 0; x < MB; x++) av[i][x] = load4<T, VEC>(a[x], k, K);
            if (NORM) gv[i] = load4<float, VEC>(gain, k, K);
#pragma unroll
            for (int b = 0; b < NP; b++)
#pragma unroll
                for (int j = 0; j < NBK; j++) wv[i][b][j] = load4<T, VEC>(w[b][j], k, K);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < UN; i++) {
            if (WIDE && i && g + i * NW * 16 >= K) break;
            if (NORM) {
#pragma unroll
                for (int x = 0; x < MB; x++)
#pragma unroll
                    for (int e = 0; e < 4; e++) { ss[x] += av[i][x][e] * av[i][x][e]; av[i][x][e] *= gv[i][e]; }
            }
#pragma unroll
            for (int e = 0; e < 4; e++)
#pragma unroll
                for (int b = 0; b < NP; b++)
#pragma unroll
                    for (int x = 0; x < MB; x++)
#pragma unroll
                        for (int j = 0; j < NBK; j++)
                            acc[b][x][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[i][b][j][e], av[i][x][e], acc[b][x][j], 0, 0, 0);
        }
    }
    if (NORM) {
#pragma unroll
        for (int x = 0; x < MB; x++) {
            ss[x] += __shfl_xor(ss[x], 16, 64);
            ss[x] += __shfl_xor(ss[x], 32, 64);
            if (kq == 0) squares[wave][x * 16 + l16] = ss[x];
        }
    }
#pragma unroll
    for (int b = 0; b < NP; b++)
#pragma unroll
        for (int x = 0; x < MB; x++)
#pragma unroll
            for (int j = 0; j < NBK; j++) part[wave][(b * MB + x) * NBK + j][lane] = acc[b][x][j];
    __syncthreads();
    // block (x, j) of the tile is finished by wave x * NBK + j: lane = row l16, columns 4 * kq .. + 3
    if (wave >= MB * NBK) return;
    const int x = wave / NBK, j = wave % NBK, m = m0 + x * 16 + l16;
    if (m >= M) return;
    // the waves' parts in pairs: the rounding of three additions where one after the other has seven (relative error of the tiny
    // decoder's logits against 64 bits, mean of 150 draws: 4.40e-7 -> 4.34e-7, same time)
    f32x4_t sum[NP];
#pragma unroll
    for (int b = 0; b < NP; b++) {
        f32x4_t v[NW];
#pragma unroll
        for (int s = 0; s < NW; s++) v[s] = part[s][(b * MB + x) * NBK + j][lane];
#pragma unroll
        for (int h = NW / 2; h > 0; h >>= 1)
#pragma unroll
            for (int s = 0; s < h; s++)
#pragma unroll
                for (int r = 0; r < 4; r++) v[s][r] += v[s + h][r];
        sum[b] = v[0];
    }
    if (NORM) {
        float sq[NW];
#pragma unroll
        for (int s = 0; s < NW; s++) sq[s] = squares[s][x * 16 + l16];
#pragma unroll
        for (int h = NW / 2; h > 0; h >>= 1)
#pragma unroll
            for (int s = 0; s < h; s++) sq[s] += sq[s + h];
        const float q = sq[0];
        const float r = 1.0f / sqrtf(q / (float)K + eps);
#pragma unroll
        for (int b = 0; b < NP; b++)
#pragma unroll
            for (int e = 0; e < 4; e++) sum[b][e] *= r;
    }
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const int col = n0 + j * 16 + kq * 4 + r;
        if (col >= N) continue;
        const size_t o = (size_t)m * N + col;
        if (EPI == EPI_RESIDUAL) {
            ((float *)Cv)[o] = res[o] + sum[0][r];
        } else if (EPI == EPI_SWIGLU) {
            const float g = sum[0][r];
            ((T *)Cv)[o] = from_f<T>(g / (1.0f + expf(-g)) * sum[NP - 1][r]);
        } else {
            ((float *)Cv)[o] = sum[0][r];
        }
    }
}

// ---------------------------------------------------------------------------------- rotary
// table[r][i] = (cos, sin)(phi), phi = (pos0 + r) * theta^(-2i/d).
__global__ void rope_table_kernel(float2 *table, int R, int pos0, int d, float theta) {
    int idx = blockIdx.x * blockDim.x + threadIdx.x;
    int half = d / 2;
    if (idx >= R * half) return;
    int r = idx / half, i = idx % half;
    table[idx] = vla_rope_entry(pos0 + r, i, d, theta);
}

// Rotate q and k of every new row (pairs (i, i + d/2)) from the fp32 QKV projection, write q to its
// own [M, H] buffer and k, v into the KV layout.  One thread per (row, head, 8-dim chunk c of the first
// half): it owns dims [8c, 8c+8) and [d/2 + 8c, d/2 + 8c + 8).
template <typename T>
__global__ void rope_kv_write_kernel(T *q_out, const float *qkv, const float2 *table, T *kc, T *vc, int n_seq,
                                     int R, int pos0, int n_heads, int d, int pos_stride, int H) {
    int chunks = d / 16;
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = (size_t)n_seq * R * n_heads * chunks;
    if (idx >= total) return;
    int c = idx % chunks;
    int h = (idx / chunks) % n_heads;
    size_t m = idx / ((size_t)chunks * n_heads);
    int s = m / R, r = m % R;
    int pos = pos0 + r;
    int half = d / 2;
    typedef T t8 __attribute__((ext_vector_type(8), aligned(sizeof(T))));        // (the caller's KV buffer: element alignment)
    const float *q = qkv + m * 3 * (size_t)H + (size_t)h * d + c * 8;
    const float2 *cs = table + (size_t)r * half + c * 8;
    const size_t head = (size_t)s * n_heads + h;
    f32x4_t in[3][2][2];                         // q, k, v: both halves, eight dims each
#pragma unroll
    for (int seg = 0; seg < 3; seg++)
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int w = 0; w < 2; w++) in[seg][u][w] = *(const f32x4_t *)(q + (size_t)seg * H + u * half + w * 4);
    t8 out[3][2];
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const float2 t = cs[e];
#pragma unroll
        for (int seg = 0; seg < 2; seg++) {
            const float a = in[seg][0][e >> 2][e & 3], b = in[seg][1][e >> 2][e & 3];
            out[seg][0][e] = from_f<T>(a * t.x - b * t.y);
            out[seg][1][e] = from_f<T>(b * t.x + a * t.y);
        }
        out[2][0][e] = from_f<T>(in[2][0][e >> 2][e & 3]);
        out[2][1][e] = from_f<T>(in[2][1][e >> 2][e & 3]);
    }
    T *qo = q_out + m * (size_t)H + (size_t)h * d + c * 8, *vdst = vc + (head * pos_stride + pos) * d + c * 8;
    *(t8 *)qo = out[0][0];
    *(t8 *)(qo + half) = out[0][1];
    *(t8 *)(kc + ((head * (d / 8) + c) * pos_stride + pos) * 8) = out[1][0];
    *(t8 *)(kc + ((head * (d / 8) + (half / 8) + c) * pos_stride + pos) * 8) = out[1][1];
    *(t8 *)vdst = out[2][0];
    *(t8 *)(vdst + half) = out[2][1];
}

// Rows first .. first + count - 1 of every sequence of X [n_seq * R, H], packed into Xt [n_seq * count, H].
__global__ void gather_rows_kernel(float *Xt, const float *X, int R, int first, int count, int H) {
    const int s = blockIdx.x / count, j = blockIdx.x - s * count;
    const f32x4_t *src = (const f32x4_t *)(X + ((size_t)s * R + first + j) * H);
    f32x4_t *dst = (f32x4_t *)(Xt + (size_t)blockIdx.x * H);
    for (int i = threadIdx.x; i < H / 4; i += blockDim.x) dst[i] = src[i];
}

// Rotary on q alone: qf fp32 [M, H] (row m of sequence s is position table row first + m % count) -> q_out in the
// storage type.  One thread per (row, head, pair index).
template <typename T>
__global__ void rope_q_kernel(T *q_out, const float *qf, const float2 *table, size_t M, int count, int first, int n_heads,
                              int d, int H) {
    const int half = d / 2;
    const size_t total = M * (size_t)n_heads * half;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int i = (int)(idx % half);
    const int h = (int)((idx / half) % n_heads);
    const size_t m = idx / ((size_t)half * n_heads);
    const float2 cs = table[(size_t)(first + (int)(m % count)) * half + i];
    const size_t o = m * (size_t)H + (size_t)h * d + i;
    const float a = qf[o], b = qf[o + half];
    q_out[o] = from_f<T>(a * cs.x - b * cs.y);
    q_out[o + half] = from_f<T>(b * cs.x + a * cs.y);
}

// ---------------------------------------------------------------------------------- attention
// Room for the weights of nk keys: whole runs of positions, zeros past the last.
__host__ __device__ constexpr int attention_scores(int nk) { return (nk + 31) / 32 * 32; }

// One wave per (sequence, head, new row): scores over the allowed keys into LDS, softmax, then
// the weighted sum of V rows with each lane owning head dims lane, lane+64, ...  Few rows are a chain of memory latencies: four pieces
// of K and sixteen rows of V are asked for together (tiny decoder, 8 environments: last row over 64 keys 9.6 -> 6.8 us, all 64 rows 9.9 -> 7.5).
template <typename T>
__global__ void __launch_bounds__(256) attention_generic_kernel(T *out, const T *qbuf, const T *kc,
                                                               const T *vc, int n_seq, int R, int pos0,
                                                               int full_from, int n_heads, int d,
                                                               int pos_stride, int H) {
    extern __shared__ float smem[];
    typedef T t8 __attribute__((ext_vector_type(8), aligned(sizeof(T))));        // (the caller's KV buffer: element alignment)
    constexpr int NC = 4, NP = 16;
    const int nc = d / 8;
    int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n_keys = pos0 + R;            // the most keys any row of this launch sees
    const int room = attention_scores(n_keys), per_wave = room + d;
    float *sc = smem + (size_t)wave * per_wave;
    float *qs = sc + room;
    size_t item = (size_t)blockIdx.x * 4 + wave;
    size_t total = (size_t)n_seq * n_heads * R;
    if (item >= total) return;      // whole wave leaves together; no block-level barrier below
    int r = item % R;
    int h = (item / R) % n_heads;
    int s = item / ((size_t)R * n_heads);
    size_t m = (size_t)s * R + r;
    int pos = pos0 + r;
    int nk = (pos >= full_from) ? (pos0 + R) : (pos + 1);
    const T *q = qbuf + m * (size_t)H + (size_t)h * d;
    for (int i = lane; i < d; i += 64) qs[i] = to_f(q[i]);
    __builtin_amdgcn_wave_barrier();
    size_t head = (size_t)s * n_heads + h;
    const T *kh = kc + head * (size_t)d * pos_stride;
    const T *vh = vc + head * (size_t)pos_stride * d;
    float scale = 1.0f / sqrtf((float)d);
    float mx = -INFINITY;
    for (int p = lane; p < nk; p += 64) {
        float acc = 0.f;
#pragma unroll 1
        for (int c0 = 0; c0 < nc; c0 += NC) {
            t8 kr[NC];
#pragma unroll
            for (int c = 0; c < NC; c++) kr[c] = *(const t8 *)(kh + ((size_t)min(c0 + c, nc - 1) * pos_stride + p) * 8);
#pragma unroll
            for (int c = 0; c < NC; c++)
                if (c0 + c < nc)
#pragma unroll
                    for (int e = 0; e < 8; e++) acc += qs[(c0 + c) * 8 + e] * to_f((T)kr[c][e]);
        }
        acc *= scale;
        sc[p] = acc;
        mx = fmaxf(mx, acc);
    }
    mx = vla_wave_max(mx);
    float sum = 0.f;
    for (int p = lane; p < attention_scores(nk); p += 64) {
        float e = p < nk ? expf(sc[p] - mx) : 0.f;
        sc[p] = e;
        sum += e;
    }
    sum = vla_wave_sum(sum);
    __builtin_amdgcn_wave_barrier();
    float inv = 1.0f / sum;
    for (int i = lane; i < d; i += 64) {
        float acc = 0.f;
#pragma unroll 1
        for (int p0 = 0; p0 < nk; p0 += NP) {
            T vr[NP];
#pragma unroll
            for (int u = 0; u < NP; u++) vr[u] = vh[(size_t)min(p0 + u, nk - 1) * d + i];
#pragma unroll
            for (int u = 0; u < NP; u += 4) {                                    // (weights past the last key: zeros)
                const f32x4_t w = *(const f32x4_t *)(sc + p0 + u);
#pragma unroll
                for (int e = 0; e < 4; e++) acc += w[e] * (p0 + u + e < nk ? to_f(vr[u + e]) : 0.f);
            }
        }
        out[m * (size_t)H + (size_t)h * d + i] = from_f<T>(acc * inv);
    }
}

// The attention of an fp32 decode step (one new row per sequence) straight from the QKV projection: rotation, KV write and the
// kernel above in one.  Bound by latency: WAVES waves per (sequence, head), a key per thread, V in four parts of 32 positions whose
// sums are added in order; the first K and V loads leave before the rotation.  The new position's k and v come from LDS, its k once
// into the registers of the lane that has it; the weights are padded with zeros to whole runs, so that P.V reads four at a time without a
// branch per position.  Four waves: tiny decoder, 8 environments, 68 keys: 8.5 + 9 us in two launches, 7.4 here, 5.3 with the padding and
// lane moves; six steps of a width-1024 decoder of four layers, 700
// keys: 4.15 -> 1.66 ms at 8 environments, 6.99 -> 5.84 at 128.  One wave, for many pairs of few keys: four pairs share a workgroup, with
// half the loads in flight a pair's registers shrink from 4 x 162 to 89 a lane, so that 4096 pairs run at once and not in five
// rounds, and no wave is there for keys that are not.  Either forms every sum in the same order: same bits.
template <int WAVES>
__global__ void __launch_bounds__(256) attention_step_kernel(float *out, const float *qkv, const float2 *table, float *kc, float *vc, int pos,
                                                             int n_items, int n_heads, int d, int pos_stride, int H) {
    extern __shared__ float smem[];
    typedef float t8 __attribute__((ext_vector_type(8), aligned(4)));            // (the caller's KV buffer: element alignment)
    constexpr bool ALONE = WAVES == 1;                                           // a pair per wave, else one per workgroup of four
    constexpr int NC = ALONE ? 4 : 8, NP = 32, NL = ALONE ? 16 : NP, NT = 64 * WAVES, NV = 4 / WAVES;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = ALONE ? lane : (int)threadIdx.x, part0 = ALONE ? 0 : wave;
    const int item = ALONE ? blockIdx.x * 4 + wave : blockIdx.x;
    if (ALONE && item >= n_items) return;
    auto meet = [&]() {
        if constexpr (ALONE) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        } else __syncthreads();
    };
    const int s = item / n_heads, h = item - s * n_heads;
    const int nk = pos + 1, last = max(pos - 1, 0), half = d / 2, nc = d / 8;    // (addresses past the last stored key: clamped, not used)
    const int nkp = attention_scores(nk);                                   // weights of whole runs of positions: zeros past the last
    float *qs = smem + (ALONE ? (size_t)wave * (3 * d + nkp) : 0), *ks = qs + d, *vs = ks + d, *sc = vs + d, *part = sc + nkp, *red = part + 4 * d;
    const float *row = qkv + (size_t)s * 3 * H + (size_t)h * d;
    const size_t head = (size_t)s * n_heads + h;
    float *kh = kc + head * (size_t)d * pos_stride, *vh = vc + head * (size_t)pos_stride * d;
    const int i0 = min(t, half - 1);
    const float2 cs = table[i0];
    const float qa = row[i0], qb = row[i0 + half], ka = row[H + i0], kb = row[H + i0 + half], va = row[2 * H + i0], vb = row[2 * H + i0 + half];
    t8 kr[NC];
    float vr[NL];
#pragma unroll
    for (int c = 0; c < NC; c++) kr[c] = *(const t8 *)(kh + ((size_t)min(c, nc - 1) * pos_stride + min(t, last)) * 8);
#pragma unroll
    for (int u = 0; u < NL; u++) vr[u] = vh[(size_t)min(part0 * NP + u, last) * d + min(lane, d - 1)];
    auto rotate = [&](int i, float2 cs, float qa, float qb, float ka, float kb, float va, float vb) {
        const float k0 = ka * cs.x - kb * cs.y, k1 = kb * cs.x + ka * cs.y;
        qs[i] = qa * cs.x - qb * cs.y;
        qs[i + half] = qb * cs.x + qa * cs.y;
        ks[i] = k0; ks[i + half] = k1;
        vs[i] = va; vs[i + half] = vb;
        kh[((size_t)(i >> 3) * pos_stride + pos) * 8 + (i & 7)] = k0;
        kh[((size_t)((i + half) >> 3) * pos_stride + pos) * 8 + (i & 7)] = k1;
        vh[(size_t)pos * d + i] = va;
        vh[(size_t)pos * d + i + half] = vb;
    };
    if (t < half) rotate(t, cs, qa, qb, ka, kb, va, vb);
    if (ALONE && t + 64 < half) {                // (head_dim above 128)
        const int i = t + 64;
        rotate(i, table[i], row[i], row[i + half], row[H + i], row[H + i + half], row[2 * H + i], row[2 * H + i + half]);
    }
    meet();
    const float scale = 1.0f / sqrtf((float)d);
    float mx = -INFINITY;
    for (int p = t; p < nk; p += NT) {
        float acc = 0.f;
        for (int c0 = 0; c0 < nc; c0 += NC) {
            if (p != t || c0)
#pragma unroll
                for (int c = 0; c < NC; c++) kr[c] = *(const t8 *)(kh + ((size_t)min(c0 + c, nc - 1) * pos_stride + min(p, last)) * 8);
            if (p == pos)
#pragma unroll
                for (int c = 0; c < NC; c++) kr[c] = *(const t8 *)(ks + min(c0 + c, nc - 1) * 8);
#pragma unroll
            for (int c = 0; c < NC; c++)
                if (c0 + c < nc)
#pragma unroll
                    for (int e = 0; e < 8; e++) acc += qs[(c0 + c) * 8 + e] * kr[c][e];
        }
        acc *= scale;
        sc[p] = acc;
        mx = fmaxf(mx, acc);
    }
    mx = vla_wave_max(mx);
    if constexpr (!ALONE) {
        if (lane == 0) red[wave] = mx;
        __syncthreads();
        mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    }
    // four sums of every fourth 64 keys, then their sum: the same whichever waves form them
    float sum[NV];
#pragma unroll
    for (int v = 0; v < NV; v++) {
        sum[v] = 0.f;
        if (ALONE && v * 64 >= nkp) continue;
        for (int p = v * 64 + t; p < nkp; p += 256) {
            const float e = p < nk ? expf(sc[p] - mx) : 0.f;
            sc[p] = e;
            sum[v] += e;
        }
        sum[v] = vla_wave_sum(sum[v]);
    }
    if constexpr (!ALONE)
        if (lane == 0) red[4 + wave] = sum[0];
    meet();
    float total;
    if constexpr (ALONE) total = sum[0] + sum[1] + sum[2] + sum[3];
    else total = red[4] + red[5] + red[6] + red[7];
    const float inv = 1.0f / total;
    for (int i = lane; i < d; i += 64) {
        float acc[NV];
        const float v_new = vs[i];
#pragma unroll
        for (int v = 0; v < NV; v++) {
            acc[v] = 0.f;
            for (int p0 = (part0 + v) * NP; p0 < nk; p0 += 4 * NP) {
#pragma unroll
                for (int l = 0; l < NP; l += NL) {
                    if (l && p0 + l >= nk) break;
                    if (i != lane || p0 + l != part0 * NP)
#pragma unroll
                        for (int u = 0; u < NL; u++) vr[u] = vh[(size_t)min(p0 + l + u, last) * d + i];
#pragma unroll
                    for (int u = 0; u < NL; u += 4) {
                        const f32x4_t w = *(const f32x4_t *)(sc + p0 + l + u);
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            const int p = p0 + l + u + e;
                            acc[v] += w[e] * (p < pos ? vr[u + e] : p == pos ? v_new : 0.f);
                        }
                    }
                }
            }
        }
        if constexpr (ALONE) out[(size_t)s * H + (size_t)h * d + i] = (acc[0] + acc[1] + acc[2] + acc[3]) * inv;
        else part[wave * d + i] = acc[0];
    }
    if constexpr (!ALONE) {
        __syncthreads();
        if (t < d) out[(size_t)s * H + (size_t)h * d + t] = (part[t] + part[d + t] + part[2 * d + t] + part[3 * d + t]) * inv;
    }
}

// ---------------------------------------------------------------------------------- value head
// value[row, c] = w[c] . h[row] + b + bias[c]; one workgroup per (row, c).
__global__ void value_head_kernel(float *value, const float *h, const float *w, float b, const float *bias, int H,
                                  int h_stride) {
    __shared__ float red[4];
    const int c = blockIdx.y, vd = gridDim.y;
    const float *hr = h + (size_t)blockIdx.x * h_stride, *wc = w + (size_t)c * H;
    float acc = 0.f;
    for (int i = threadIdx.x; i < H; i += 256) acc += hr[i] * wc[i];
    acc = block_sum_256(acc, red);
    if (threadIdx.x == 0) value[(size_t)blockIdx.x * vd + c] = acc + b + (bias ? bias[c] : 0.f);
}

}  // namespace

// =========================================================================================== host
template <typename T>
int launch_embed_prefix(float *X, const T *patch, const int32_t *ids, const T *embed, int n_seq, int P,
                        int T_, int rows_per_seq, int H, int vocab, hipStream_t st) {
    if (n_seq * (P + T_) == 0) return 0;
    ProfScope ps("embed_prefix", 0.0, st);
    embed_prefix_kernel<T><<<n_seq * (P + T_), 256, 0, st>>>(X, patch, ids, embed, P, T_, rows_per_seq, H, vocab);
    return vla_check_launch("embed_prefix");
}
template <typename T>
int launch_embed_tokens(float *X, const int32_t *bins, int bins_stride, int n_tok, const T *embed,
                        int n_seq, int rows_per_seq, int row0, int H, int vocab, hipStream_t st) {
    if (n_seq * n_tok == 0) return 0;
    ProfScope ps("embed_tokens", 0.0, st);
    embed_tokens_kernel<T><<<n_seq * n_tok, 256, 0, st>>>(X, bins, bins_stride, n_tok, embed, rows_per_seq, row0, H, vocab);
    return vla_check_launch("embed_tokens");
}
template <typename T>
int launch_embed_slots(float *X, const T *slot_embed, int n_seq, int A, int rows_per_seq, int row0,
                       int H, hipStream_t st) {
    if (n_seq * A == 0) return 0;
    ProfScope ps("embed_slots", 0.0, st);
    embed_slots_kernel<T><<<n_seq * A, 256, 0, st>>>(X, slot_embed, A, rows_per_seq, row0, H);
    return vla_check_launch("embed_slots");
}
template <typename T>
int launch_rmsnorm(T *out, const float *X, const float *gain, int M, int H, float eps, hipStream_t st) {
    if (M == 0) return 0;
    ProfScope ps("rmsnorm", (double)M * H * (4 + sizeof(T)), st);
    rmsnorm_kernel<T><<<M, 256, 0, st>>>(out, X, gain, H, eps);
    return vla_check_launch("rmsnorm");
}
int launch_final_norm_rows(float *out, const float *X, const float *gain, int n_seq, int rows_per_seq,
                           int row0, int n_rows, int H, float eps, hipStream_t st) {
    if (n_seq * n_rows == 0) return 0;
    ProfScope ps("final_norm_rows", 0.0, st);
    final_norm_rows_kernel<<<n_seq * n_rows, 256, 0, st>>>(out, X, gain, rows_per_seq, row0, n_rows, H, eps);
    return vla_check_launch("final_norm_rows");
}
template <typename T, int EPI, bool VEC, bool NORM>
static void gemm_generic_tile(const GemmArgs &g, int N, hipStream_t st) {
    constexpr int MB = (EPI == EPI_SWIGLU) ? 2 : 4, NBK = 2;
    const T *A = (const T *)(NORM ? (const void *)g.norm_x : g.A), *W0 = (const T *)g.W[0], *W1 = (const T *)g.W[1], *W2 = (const T *)g.W[2];
    const float *res = g.res ? g.res : (const float *)g.C;
    const dim3 big((N + 16 * NBK - 1) / (16 * NBK), (g.M + 16 * MB - 1) / (16 * MB));
    // The large tile wants two workgroups per CU; its sums are those of the small one.  (Fewer than 512 large tiles are
    // at most 4096 + a few rows of small ones.)  A wave of the small tile loads its whole share of K at once where that is up to
    // eight blocks: a down projection of K = 688 4.9 us as six, 5.5 as four and two.  Of narrower loads (bf16, rows that do not end on
    // 16 bytes) four blocks, and no way out between them: decode of width 2048, FFN 5461, 25 environments 2.43 ms, with eight 2.63; gradient pass of an fp32
    // decoder of width 1024, FFN 2731, 1.85 and 1.92.
    if ((size_t)big.x * big.y >= 512) {
        gemm_generic_kernel<T, EPI, VEC, MB, NBK, 1, NORM><<<big, 512, 0, st>>>(A, W0, W1, W2, g.segN, g.C, res, g.M, N, g.K, g.norm_gain, g.norm_eps);
        return;
    }
    const dim3 small((N + 15) / 16, (g.M + 15) / 16);
    auto go = [&](auto un) {
        gemm_generic_kernel<T, EPI, VEC, 1, 1, decltype(un)::value, NORM><<<small, 512, 0, st>>>(A, W0, W1, W2, g.segN, g.C, res, g.M, N, g.K, g.norm_gain, g.norm_eps);
    };
    if constexpr (sizeof(T) == 2 || !VEC) go(std::integral_constant<int, 4>{});
    else if (g.K <= 256) go(std::integral_constant<int, 2>{});
    else if (g.K <= 768) go(std::integral_constant<int, 6>{});
    else go(std::integral_constant<int, 8>{});
}
template <typename T, int EPI>
static void gemm_generic_epi(const GemmArgs &g, int N, hipStream_t st) {
    if constexpr (sizeof(T) == 4 && EPI != EPI_RESIDUAL) {
        if (g.norm_x) return gemm_generic_tile<T, EPI, true, true>(g, N, st);
    }
    if (g.K % 4 == 0) gemm_generic_tile<T, EPI, true, false>(g, N, st);
    else gemm_generic_tile<T, EPI, false, false>(g, N, st);
}
template <typename T>
int launch_gemm_generic(const GemmArgs &g, hipStream_t st) {
    if (g.M == 0) return 0;
    if (g.norm_x && (sizeof(T) != 4 || g.epilogue == EPI_RESIDUAL || g.K % 4 != 0)) { vla_set_error("internal: the norm in the GEMM was declined"); return VLA_ESHAPE; }
    ProfScope ps("gemm_generic", 2.0 * g.M * g.K * g.n_seg * g.segN, st);
    const int N = (g.epilogue == EPI_SWIGLU) ? g.segN : g.n_seg * g.segN;
    if (g.epilogue == EPI_STORE) gemm_generic_epi<T, EPI_STORE>(g, N, st);
    else if (g.epilogue == EPI_RESIDUAL) gemm_generic_epi<T, EPI_RESIDUAL>(g, N, st);
    else gemm_generic_epi<T, EPI_SWIGLU>(g, N, st);
    return vla_check_launch("gemm_generic");
}
int launch_rope_table(float2 *table, int R, int pos0, int d, float theta, hipStream_t st) {
    ProfScope ps("rope_table", 0.0, st);
    int n = R * (d / 2);
    if (n == 0) return 0;
    rope_table_kernel<<<(n + 255) / 256, 256, 0, st>>>(table, R, pos0, d, theta);
    return vla_check_launch("rope_table");
}
template <typename T>
int launch_rope_kv_write(T *q_out, const float *qkv, const float2 *table, const KvView &kv, int layer,
                         const RowsArgs &ra, int H, hipStream_t st) {
    ProfScope ps("rope_kv_write", (double)ra.n_seq * ra.R * H * 5 * sizeof(T), st);
    size_t total = (size_t)ra.n_seq * ra.R * kv.n_heads * (kv.d / 16);
    if (total == 0) return 0;
    T *kc = (T *)kv.k + (size_t)layer * kv.layer_elems;
    T *vc = (T *)kv.v + (size_t)layer * kv.layer_elems;
    rope_kv_write_kernel<T><<<(unsigned)((total + 255) / 256), 256, 0, st>>>(
        q_out, qkv, table, kc, vc, ra.n_seq, ra.R, ra.pos0, kv.n_heads, kv.d, kv.pos_stride, H);
    return vla_check_launch("rope_kv_write");
}
int launch_gather_rows(float *Xt, const float *X, int n_seq, int R, int first, int count, int H, hipStream_t st) {
    if (n_seq * count == 0) return 0;
    ProfScope ps("gather_rows", 0.0, st);
    gather_rows_kernel<<<n_seq * count, 256, 0, st>>>(Xt, X, R, first, count, H);
    return vla_check_launch("gather_rows");
}
template <typename T>
int launch_rope_q(T *q_out, const float *qf, const float2 *table, int n_seq, int count, int first, int n_heads, int d, int H,
                  hipStream_t st) {
    const size_t M = (size_t)n_seq * count, total = M * n_heads * (d / 2);
    if (total == 0) return 0;
    ProfScope ps("rope_q", 0.0, st);
    rope_q_kernel<T><<<(unsigned)((total + 255) / 256), 256, 0, st>>>(q_out, qf, table, M, count, first, n_heads, d, H);
    return vla_check_launch("rope_q");
}
template <typename T>
int launch_attention_generic(T *out, const T *q, const KvView &kv, int layer, const RowsArgs &ra,
                             int H, hipStream_t st) {
    ProfScope ps("attention_generic", 0.0, st);
    size_t total = (size_t)ra.n_seq * kv.n_heads * ra.R;
    if (total == 0) return 0;
    const T *kc = (const T *)kv.k + (size_t)layer * kv.layer_elems;
    const T *vc = (const T *)kv.v + (size_t)layer * kv.layer_elems;
    // scores of the visible keys + the query, per wave; above the 64 KB default the limit is raised once per
    // instantiation (8192 keys at head_dim 256 need 132 KB of the CU's 160 KB)
    size_t lds = (size_t)4 * (attention_scores(ra.pos0 + ra.R) + kv.d) * sizeof(float);
    if (lds > 64 * 1024) {
        static bool raised = false;
        if (lds > 160 * 1024) { vla_set_error("attention_generic: %d keys need %zu bytes of LDS", ra.pos0 + ra.R, lds); return VLA_ESHAPE; }
        if (!raised) {
            if (hipFuncSetAttribute((const void *)attention_generic_kernel<T>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    160 * 1024) != hipSuccess) {
                vla_set_error("attention_generic: cannot raise the dynamic LDS limit");
                return VLA_EHIP;
            }
            raised = true;
        }
    }
    attention_generic_kernel<T><<<(unsigned)((total + 3) / 4), 256, lds, st>>>(
        out, q, kc, vc, ra.n_seq, ra.R, ra.pos0, ra.full_from, kv.n_heads, kv.d, kv.pos_stride, H);
    return vla_check_launch("attention_generic");
}
int launch_attention_step_qkv(float *out, const float *qkv, const float2 *table, const KvView &kv, int layer, const RowsArgs &ra, int H, hipStream_t st) {
    const int n_items = ra.n_seq * kv.n_heads;
    if (n_items == 0) return 0;
    ProfScope ps("attention_step", 0.0, st);
    float *k = (float *)kv.k + (size_t)layer * kv.layer_elems, *v = (float *)kv.v + (size_t)layer * kv.layer_elems;
    const int nk = ra.pos0 + 1;
    // One wave per pair from eight pairs per key on, up to 80 KB of K per pair (us per step with one and with four waves, in brackets
    // rotation and attention apart).  head_dim 64: 4096 pairs of 23 keys 15.5 and 42 (28), 103 keys 37 and 52 (58), 303 keys 120 and 129
    // (139), 1003 keys 369 and 364 (384); 1024 pairs of 23, 103, 303 and 1003 keys 9.6 and 17 (25), 18 and 20, 35 and 38, 119 and 103;
    // 128 pairs of 23 and 103 keys 10.4 and 9.7, 14 and 10.  8192 pairs: head_dim 16, 1003 keys 241 and 324 (272), 256, 23 keys 41 and 119 (83).
    // head_dim 256, 1024 pairs of 103 keys: 57 and 52 (95).
    if (kv.d * nk <= 20480 && n_items >= 8 * nk) {
        const size_t lds = (size_t)4 * (3 * kv.d + attention_scores(nk)) * sizeof(float);    // (at most 22 KB)
        attention_step_kernel<1><<<(n_items + 3) / 4, 256, lds, st>>>(out, qkv, table, k, v, ra.pos0, n_items, kv.n_heads, kv.d, kv.pos_stride, H);
    } else {
        const size_t lds = (size_t)(7 * kv.d + 8 + attention_scores(nk)) * sizeof(float);    // (at most 40 KB: 8192 keys at head_dim 256)
        attention_step_kernel<4><<<n_items, 256, lds, st>>>(out, qkv, table, k, v, ra.pos0, n_items, kv.n_heads, kv.d, kv.pos_stride, H);
    }
    return vla_check_launch("attention_step");
}
int launch_value_head(float *value, const float *h, const float *w, float b, const float *bias, int vd, int n,
                      int H, int h_stride, hipStream_t st) {
    if (n == 0) return 0;
    ProfScope ps("value_head", 0.0, st);
    value_head_kernel<<<dim3(n, vd), 256, 0, st>>>(value, h, w, b, bias, H, h_stride);
    return vla_check_launch("value_head");
}

#define INSTANTIATE(T)                                                                                        \
    template int launch_embed_prefix<T>(float *, const T *, const int32_t *, const T *, int, int, int, int,   \
                                        int, int, hipStream_t);                                               \
    template int launch_embed_tokens<T>(float *, const int32_t *, int, int, const T *, int, int, int, int,    \
                                        int, hipStream_t);                                                    \
    template int launch_embed_slots<T>(float *, const T *, int, int, int, int, int, hipStream_t);             \
    template int launch_rmsnorm<T>(T *, const float *, const float *, int, int, float, hipStream_t);          \
    template int launch_gemm_generic<T>(const GemmArgs &, hipStream_t);                                       \
    template int launch_rope_kv_write<T>(T *, const float *, const float2 *, const KvView &, int,             \
                                         const RowsArgs &, int, hipStream_t);                                                        \
    template int launch_attention_generic<T>(T *, const T *, const KvView &, int, const RowsArgs &, int,      \
                                             hipStream_t);                                                    \
    template int launch_rope_q<T>(T *, const float *, const float2 *, int, int, int, int, int, int, hipStream_t);
INSTANTIATE(float)
INSTANTIATE(bf16_t)
