// Action-bin head and sampler: logits z = h . W^T over the 256 bins (fp32 h, weights in the storage type), then per
// row the softmax statistics, the log-probability and the Gumbel-max choice.
//
// The product is a contraction of 256 columns whose weights (2 MB at H = 4096 in bf16) every row needs, so it runs on
// the matrix cores over tiles of 16 rows and is cut along K into chunks of 256: at one row per call (decode at batch 1)
// 64 workgroups share the 2 MB that one workgroup used to walk alone.  bf16 weights: h enters as three bf16 parts
// (8 + 8 + 8 significant bits, i.e. all 24 of the fp32 value), three v_mfma_f32_16x16x32_bf16 per block, products exact
// in fp32.  (An infinite weight meets the first part alone: a later part of zero would make its product NaN, one of the
// other sign the sum.  A chunk that comes out NaN is formed again that way.)  fp32 weights: v_mfma_f32_16x16x4_f32.  Sums
// run over one chunk at a time and the chunks are added in order, the same for every row count and both forms below, so a
// row's result does not depend on the rows around it.
//   partial form: one workgroup per (16 rows, chunk, 64 bins), fp32 partial logits to scratch, a second kernel samples: its
//   time grows with the rows, for the partial logits of every chunk are written and read;
//   whole form (above VLA_HEAD_PARTIAL_ROWS rows): a workgroup walks all chunks for 32 rows and samples them from LDS, a chain
//   of the same length for any rows that fit the chip at once.
// Where they meet, in bf16: 3072 / 4096 / 5120 rows take 101 / 131 / 161 us in the partial form and 129 / 129 / 130 in the whole
// one at H = 4096, 34 / 42 / 49 and 46 / 47 / 48 at H = 1024.
// Measured at H = 4096 in bf16: 1 .. 256 rows took 131-140 us and 7168 rows 3450 us with one workgroup per row and a bin
// per thread (every row fetched the 2 MB again); now (both kernels) 10 us at 1 row, 17 us at 256 and 133 us at 7168, of which a
// kernel launch is about 3.
#include "vla_internal.h"

namespace {

constexpr int CHUNK = 256;

typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));   // the caller's h may be aligned to 4 bytes only

// x = hi + mid + lo to 24 bits; an infinite head keeps its infinity (the remainders would be NaN)
__device__ __forceinline__ void split3(float x, bf16_t &hi, bf16_t &mid, bf16_t &lo) {
    hi = (bf16_t)x;
    const float hf = (float)hi;
    const float r1 = __builtin_isinf(hf) ? 0.f : x - hf;
    mid = (bf16_t)r1;
    lo = (bf16_t)(r1 - (float)mid);
}

// Products of one chunk [k0, k1) (a multiple of 16 long) for 16 * RB rows and 16 * CB bins from bin0:
// acc[rb][cb][r] = bin bin0 + cb * 16 + 4 * (lane / 16) + r of row rb * 16 + lane % 16.
// UN steps are loaded together ahead of their products (a call of few rows is a chain of memory latencies: one per
// group of steps).  FULL: the chunk is CHUNK long; otherwise the steps past k1 count as zeros.  TAME: infinite weights
// meet the first part of h only.
// NORM: the rows come as the residual stream; each element enters times `gain`, and ss[rb] gains the squares of this lane's.
template <int RB, int CB, bool FULL, int UN, bool NORM, bool TAME = false>
__device__ __forceinline__ void chunk_product(f32x4_t (&acc)[RB][CB], float (&ss)[RB], const float *const (&hrow)[RB], const bf16_t *const (&wrow)[CB],
                                              const float *gain, int k0, int k1, int kq) {
#pragma unroll 1
    for (int g = 0; g < CHUNK / 32; g += UN) {
        bf16x8_t w[UN][CB];
        f32x4_t x[UN][RB][2], gv[UN][2];
#pragma unroll
        for (int i = 0; i < UN; i++) {
            const int kk = k0 + (g + i) * 32 + kq * 8;
            const bool in = FULL || kk < k1;
            const int ks = in ? kk : k0;
#pragma unroll
            for (int cb = 0; cb < CB; cb++) w[i][cb] = *(const bf16x8_t *)(wrow[cb] + ks);
#pragma unroll
            for (int rb = 0; rb < RB; rb++)
#pragma unroll
                for (int u = 0; u < 2; u++) {
                    x[i][rb][u] = *(const f32x4_u *)(hrow[rb] + ks + 4 * u);
                    if (!in) x[i][rb][u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                }
            if (NORM)
#pragma unroll
                for (int u = 0; u < 2; u++) gv[i][u] = *(const f32x4_u *)(gain + ks + 4 * u);
            if (!in)
#pragma unroll
                for (int cb = 0; cb < CB; cb++)
#pragma unroll
                    for (int e = 0; e < 8; e++) w[i][cb][e] = (bf16_t)0.f;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < UN; i++) {
            bf16x8_t wt[CB];
#pragma unroll
            for (int cb = 0; cb < CB; cb++) {
                wt[cb] = w[i][cb];
                if (TAME)
#pragma unroll
                    for (int e = 0; e < 8; e++)
                        if (__builtin_isinf((float)wt[cb][e])) wt[cb][e] = (bf16_t)0.f;
            }
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                bf16x8_t hi, mid, lo;
                if (NORM) {
#pragma unroll
                    for (int e = 0; e < 8; e++) {
                        ss[rb] += x[i][rb][e >> 2][e & 3] * x[i][rb][e >> 2][e & 3];
                        x[i][rb][e >> 2][e & 3] *= gv[i][e >> 2][e & 3];
                    }
                }
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    bf16_t a, b, c;
                    split3(x[i][rb][e >> 2][e & 3], a, b, c);
                    hi[e] = a; mid[e] = b; lo[e] = c;
                }
#pragma unroll
                for (int cb = 0; cb < CB; cb++) acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[cb], lo, acc[rb][cb], 0, 0, 0);
#pragma unroll
                for (int cb = 0; cb < CB; cb++) acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[cb], mid, acc[rb][cb], 0, 0, 0);
#pragma unroll
                for (int cb = 0; cb < CB; cb++) acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i][cb], hi, acc[rb][cb], 0, 0, 0);
            }
        }
    }
}
template <int RB, int CB, bool FULL, int UN, bool NORM>
__device__ __forceinline__ void chunk_product(f32x4_t (&acc)[RB][CB], float (&ss)[RB], const float *const (&hrow)[RB], const float *const (&wrow)[CB],
                                              const float *gain, int k0, int k1, int kq) {
    // a lane's four consecutive K elements take turns as the instruction's one element per lane
#pragma unroll 1
    for (int g = 0; g < CHUNK / 16; g += 2 * UN) {
        f32x4_t w[2 * UN][CB], x[2 * UN][RB], gv[2 * UN];
#pragma unroll
        for (int i = 0; i < 2 * UN; i++) {
            const int kk = k0 + (g + i) * 16 + kq * 4;
            const bool in = FULL || kk < k1;
            const int ks = in ? kk : k0;
#pragma unroll
            for (int cb = 0; cb < CB; cb++) {
                w[i][cb] = *(const f32x4_u *)(wrow[cb] + ks);
                if (!in) w[i][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                x[i][rb] = *(const f32x4_u *)(hrow[rb] + ks);
                if (!in) x[i][rb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
            if (NORM) gv[i] = *(const f32x4_u *)(gain + ks);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2 * UN; i++) {
            if (NORM) {
#pragma unroll
                for (int rb = 0; rb < RB; rb++)
#pragma unroll
                    for (int e = 0; e < 4; e++) { ss[rb] += x[i][rb][e] * x[i][rb][e]; x[i][rb][e] *= gv[i][e]; }
            }
#pragma unroll
            for (int e = 0; e < 4; e++)
#pragma unroll
                for (int rb = 0; rb < RB; rb++)
#pragma unroll
                    for (int cb = 0; cb < CB; cb++)
                        acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i][cb][e], x[i][rb][e], acc[rb][cb], 0, 0, 0);
        }
    }
}

struct SampleArgs {
    float temperature;
    const float *gumbel;
    const int32_t *given;
    int32_t *bins_out;
    float *logp, *ent, *logits;
    int out_stride, out_off;
};

// One wave, one row: z holds the row's 256 logits in LDS.  Softmax statistics, log-probability, entropy and the
// Gumbel-max choice with four bins per lane (bins lane, lane + 64, + 128, + 192).  Returns the bin.
// `g`: the row's noise at those bins (the caller loads it ahead of the logits; 0 when there is none).
__device__ __forceinline__ void load_noise(float (&g)[4], const SampleArgs &a, int row, int lane) {
    const size_t o = (size_t)row * a.out_stride + a.out_off;
#pragma unroll
    for (int j = 0; j < 4; j++) g[j] = a.gumbel ? a.gumbel[o * VLA_N_BINS + lane + 64 * j] : 0.f;
}
__device__ __forceinline__ int sample_row(const float *z, const float (&g)[4], const SampleArgs &a, int row, int lane) {
    const size_t o = (size_t)row * a.out_stride + a.out_off;
    float y[4], t[4];
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int k = lane + 64 * j;
        if (a.logits) a.logits[o * VLA_N_BINS + k] = z[k];
        y[j] = z[k] / a.temperature;
        t[j] = a.gumbel ? y[j] + g[j] : y[j];
        mx = fmaxf(mx, y[j]);
    }
    mx = vla_wave_max(mx);
    float se = 0.f, sy = 0.f;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const float e = expf(y[j] - mx);
        se += e;
        sy += e * y[j];
    }
    se = vla_wave_sum(se);
    sy = vla_wave_sum(sy);
    const float lse = mx + logf(se);
    // argmax of t, lowest bin index on ties
    float bt = t[0];
    int bk = lane;
#pragma unroll
    for (int j = 1; j < 4; j++)
        if (t[j] > bt) { bt = t[j]; bk = lane + 64 * j; }
    auto meet = [&](float ot, float okf) {
        const int ok = __builtin_bit_cast(int, okf);
        if (ot > bt || (ot == bt && ok < bk)) { bt = ot; bk = ok; }
    };
    auto as_f = [&] { return __builtin_bit_cast(float, bk); };
    {
        const VlaPair t32 = vla_pair<32>(bt), k32 = vla_pair<32>(as_f());
        bt = t32.a; bk = __builtin_bit_cast(int, k32.a);
        meet(t32.b, k32.b);
        const VlaPair t16 = vla_pair<16>(bt), k16 = vla_pair<16>(as_f());
        bt = t16.a; bk = __builtin_bit_cast(int, k16.a);
        meet(t16.b, k16.b);
    }
    meet(vla_dpp<0x128>(bt), vla_dpp<0x128>(as_f()));                                        // lane ^ 8
    meet(vla_dpp<0x1b>(vla_dpp<0x141>(bt)), vla_dpp<0x1b>(vla_dpp<0x141>(as_f())));          // lane ^ 4: reversed in eights, then in fours
    meet(vla_dpp<0x4e>(bt), vla_dpp<0x4e>(as_f()));
    meet(vla_dpp<0xb1>(bt), vla_dpp<0xb1>(as_f()));
    int bin = __builtin_amdgcn_readfirstlane(bk);
    if (a.given) bin = min(max(a.given[o], 0), VLA_N_BINS - 1);
    if (lane == 0) {
        if (a.bins_out) a.bins_out[o] = bin;
        a.logp[o] = z[bin] / a.temperature - lse;
        a.ent[o] = lse - sy / se;
    }
    return bin;
}

// The embedding of the sampled bin as the next token's residual row; `n` threads, 4 elements each per step.
template <typename T>
__device__ __forceinline__ void next_embedding(float *dst, const T *embed, int vocab, int bin, int H, int i0, int n) {
    typedef T t4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));   // the caller's embedding: element alignment
    const T *src = embed + (size_t)(vocab - VLA_N_BINS + bin) * H;
    for (int i = i0 * 4; i < H; i += n * 4) {                               // H is a multiple of 16
        const t4 v = *(const t4 *)(src + i);
        f32x4_t x;
#pragma unroll
        for (int e = 0; e < 4; e++) x[e] = (float)v[e];
        *(f32x4_t *)(dst + i) = x;
    }
}

// Products of 16 * RB rows and 16 * CB bins from bin0 over the chunks [c0, c1), added in chunk order.  NORM: squares[rb] is the sum of
// the squares of row rb * 16 + lane % 16, a chunk's sum at a time like the products.
template <typename T, int RB, int CB, int UN, bool NORM>
__device__ __forceinline__ void tile_logits(f32x4_t (&total)[RB][CB], float (&squares)[RB], const float *h, const float *gain, const T *Wb, int M, int H,
                                            int m0, int bin0, int c0, int c1) {
    const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
    const T *wrow[CB];
#pragma unroll
    for (int cb = 0; cb < CB; cb++) wrow[cb] = Wb + (size_t)(bin0 + cb * 16 + l16) * H;
    const float *hrow[RB];
#pragma unroll
    for (int rb = 0; rb < RB; rb++) hrow[rb] = h + (size_t)min(m0 + rb * 16 + l16, M - 1) * H;
    for (int c = c0; c < c1; c++) {
        f32x4_t acc[RB][CB];
        auto clear = [&]() {
#pragma unroll
            for (int rb = 0; rb < RB; rb++)
#pragma unroll
                for (int cb = 0; cb < CB; cb++) acc[rb][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        };
        clear();
        float ss[RB];
#pragma unroll
        for (int rb = 0; rb < RB; rb++) ss[rb] = 0.f;
        const int k0 = c * CHUNK, k1 = min(H, k0 + CHUNK);
        if (k1 - k0 == CHUNK) chunk_product<RB, CB, true, UN, NORM>(acc, ss, hrow, wrow, gain, k0, k1, kq);
        else chunk_product<RB, CB, false, 1, NORM>(acc, ss, hrow, wrow, gain, k0, k1, kq);
        if constexpr (sizeof(T) == 2) {
            bool nan = false;
#pragma unroll
            for (int rb = 0; rb < RB; rb++)
#pragma unroll
                for (int cb = 0; cb < CB; cb++)
#pragma unroll
                    for (int r = 0; r < 4; r++) nan = nan || __builtin_isnan(acc[rb][cb][r]);
            if (__any(nan)) {
                clear();
                float again[RB];
                for (int rb = 0; rb < RB; rb++) again[rb] = 0.f;
                chunk_product<RB, CB, false, 1, NORM, true>(acc, again, hrow, wrow, gain, k0, k1, kq);
            }
        }
        if (NORM) {
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                ss[rb] += __shfl_xor(ss[rb], 16, 64);
                ss[rb] += __shfl_xor(ss[rb], 32, 64);
                squares[rb] = c == c0 ? ss[rb] : squares[rb] + ss[rb];
            }
        }
#pragma unroll
        for (int rb = 0; rb < RB; rb++)
#pragma unroll
            for (int cb = 0; cb < CB; cb++)
#pragma unroll
                for (int r = 0; r < 4; r++) total[rb][cb][r] = c == c0 ? acc[rb][cb][r] : total[rb][cb][r] + acc[rb][cb][r];
    }
}

// Partial form: grid (n_chunks, 16-row tiles, parts of the bins), two waves of 16 CB bins each, P[chunk][M][256].  CB = 2; fp32, whose
// instruction takes 128 steps of 32 cycles for a chunk of 32 bins, 1 while that leaves a CU no more than two workgroups: tiny decoder,
// 8 rows, 5.4 -> 4.2 us (with the norm 5.6 -> 5.5).
// NORM: h is the residual stream, whose norm's gain enters here and whose squares' sum per chunk goes to squares[chunk][M]; 1 / rms
// is the sampler's to apply.
template <typename T, int CB, bool NORM>
__global__ void __launch_bounds__(128) head_partial_kernel(const float *h, const float *gain, const T *Wb, float *P, float *squares, int M, int H) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m0 = blockIdx.y * 16, m = m0 + (lane & 15);
    const int bin0 = (blockIdx.z * 2 + wave) * (16 * CB);
    f32x4_t total[1][CB];
    float ss[1];
    tile_logits<T, 1, CB, 8, NORM>(total, ss, h, gain, Wb, M, H, m0, bin0, blockIdx.x, blockIdx.x + 1);
    if (NORM && bin0 == 0 && lane < 16 && m < M) squares[(size_t)blockIdx.x * M + m] = ss[0];
    if (m >= M) return;
    float *out = P + ((size_t)blockIdx.x * M + m) * VLA_N_BINS + bin0 + (lane >> 4) * 4;
#pragma unroll
    for (int cb = 0; cb < CB; cb++) *(f32x4_t *)(out + cb * 16) = total[0][cb];
}

// Second kernel of the partial form, one workgroup per row: thread k adds the partial logits of bin k in chunk order.
// In a decode loop it also readies the next step: the row's first norm while its embedding is in registers, and, by a workgroup
// more, the step's row of the rotation table.  Both were launches of 2 to 5 us that nothing overlaps: tiny decoder, 8 environments,
// rollout of 7 tokens 548 -> 529 us; 7B width, 8 layers, 1 environment 6.50 -> 6.48 ms; 13 environments 6.67 -> 6.63.
template <typename T>
__global__ void __launch_bounds__(256) sample_kernel(const float *P, int n_part, int M, SampleArgs a, float *X_next, const T *embed,
                                                    int vocab, int H, NextStep next, const float *squares, float eps) {
    typedef T t4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));   // the caller's embedding: element alignment
    typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ float z[VLA_N_BINS];
    __shared__ int chosen;
    const int row = blockIdx.x, lane = threadIdx.x & 63;
    if (row == M) {                              // (the last workgroup of a decode step that is followed by another)
        for (int i = threadIdx.x; i < next.d / 2; i += 256) next.table[i] = vla_rope_entry(next.pos, i, next.d, next.theta);
        return;
    }
    f32x4_t v[8], gain[8];
    if (next.gain) {
#pragma unroll
        for (int j = 0; j < 8; j++)
            if ((j * 256 + (int)threadIdx.x) * 4 < H) gain[j] = *(const f32x4_u *)(next.gain + (j * 256 + threadIdx.x) * 4);
    }
    const float *src = P + (size_t)row * VLA_N_BINS + threadIdx.x;
    float g[4];
    load_noise(g, a, row, lane);
    float s = src[0];
    if (squares) {                               // the rows came without their norm's 1 / rms
        float q = squares[row];
#pragma unroll 15
        for (int c = 1; c < n_part; c++) { s += src[(size_t)c * M * VLA_N_BINS]; q += squares[(size_t)c * M + row]; }
        s *= 1.0f / sqrtf(q / (float)H + eps);
    } else {
#pragma unroll 15
        for (int c = 1; c < n_part; c++) s += src[(size_t)c * M * VLA_N_BINS];
    }
    z[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x < 64) {
        const int bin = sample_row(z, g, a, row, lane);
        if (lane == 0) chosen = bin;
    }
    if (X_next) {
        __syncthreads();
        const T *e = embed + (size_t)(vocab - VLA_N_BINS + chosen) * H;
        t4 w[8];
#pragma unroll
        for (int j = 0; j < 8; j++)
            if ((j * 256 + (int)threadIdx.x) * 4 < H) w[j] = *(const t4 *)(e + (j * 256 + threadIdx.x) * 4);
#pragma unroll
        for (int j = 0; j < 8; j++)
            if ((j * 256 + (int)threadIdx.x) * 4 < H) {
#pragma unroll
                for (int u = 0; u < 4; u++) v[j][u] = (float)w[j][u];
                *(f32x4_t *)(X_next + (size_t)row * H + (j * 256 + threadIdx.x) * 4) = v[j];
            }
        if (next.gain) vla_norm_held<T>((T *)next.nrm + (size_t)row * H, v, gain, H, next.eps, z);
    }
}

// Whole form: 32 rows per workgroup over all chunks, then each wave samples a quarter of the rows.  NORM: as in the partial form, every
// wave with the squares of its own.
template <typename T, bool NORM>
__global__ void __launch_bounds__(256) head_whole_kernel(const float *h, const float *gain, float eps, const T *Wb, SampleArgs a, float *X_next, const T *embed,
                                                        int vocab, int M, int H) {
    constexpr int RB = 2, CB = 4, LD = VLA_N_BINS + 4;
    __shared__ __attribute__((aligned(16))) float z[16 * RB * LD];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m0 = blockIdx.x * (16 * RB);
    f32x4_t total[RB][CB];
    float ss[RB];
    tile_logits<T, RB, CB, 2, NORM>(total, ss, h, gain, Wb, M, H, m0, wave * 64, 0, (H + CHUNK - 1) / CHUNK);
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
        const float inv = NORM ? 1.0f / sqrtf(ss[rb] / (float)H + eps) : 1.0f;
#pragma unroll
        for (int cb = 0; cb < CB; cb++) {
            if (NORM)
#pragma unroll
                for (int r = 0; r < 4; r++) total[rb][cb][r] *= inv;
            *(f32x4_t *)(z + (rb * 16 + (lane & 15)) * LD + wave * 64 + cb * 16 + (lane >> 4) * 4) = total[rb][cb];
        }
    }
    __syncthreads();
    for (int r = wave; r < 16 * RB && m0 + r < M; r += 4) {
        float g[4];
        load_noise(g, a, m0 + r, lane);
        const int bin = sample_row(z + r * LD, g, a, m0 + r, lane);
        if (X_next) next_embedding(X_next + (size_t)(m0 + r) * H, embed, vocab, bin, H, lane, 64);
    }
}

}  // namespace

static int chunks_of(int H) { return (H + CHUNK - 1) / CHUNK; }
size_t head_scratch_bytes(int n_rows, int H) {
    return n_rows > VLA_HEAD_PARTIAL_ROWS ? 0 : (size_t)chunks_of(H) * n_rows * VLA_N_BINS * sizeof(float);
}

int head_chunks(int H) { return chunks_of(H); }

template <typename T, bool NORM>
static int launch_head_partial(const float *h, const float *gain, const T *Wb, float *P, float *squares, int n_rows, int H, hipStream_t st) {
    const int tiles = (n_rows + 15) / 16, chunks = chunks_of(H);
    if (sizeof(T) == 4 && (long)tiles * chunks * 8 <= 512) head_partial_kernel<T, 1, NORM><<<dim3(chunks, tiles, 8), 128, 0, st>>>(h, gain, Wb, P, squares, n_rows, H);
    else head_partial_kernel<T, 2, NORM><<<dim3(chunks, tiles, 4), 128, 0, st>>>(h, gain, Wb, P, squares, n_rows, H);
    return vla_check_launch("head_logits");
}

// Partial logits alone: P[chunk][n_rows][256], to be added in chunk order.
template <typename T>
int launch_head_logits(const float *h, const T *lm_head_bins, float *P, int n_rows, int H, hipStream_t st) {
    if (n_rows == 0) return 0;
    return launch_head_partial<T, false>(h, nullptr, lm_head_bins, P, nullptr, n_rows, H, st);
}

template <typename T>
int launch_head_sample(const float *h, const T *lm_head_bins, int n_rows, int H, float temperature,
                       const float *gumbel, const int32_t *given_bins, int32_t *bins_out, float *logp,
                       float *ent, float *logits, int out_stride, int out_off, float *X_next,
                       const T *embed, int vocab, float *scratch, hipStream_t st, const NextStep *next, const HeadNorm *norm) {
    if (n_rows == 0) return 0;
    ProfScope ps("head_sample", 2.0 * n_rows * H * VLA_N_BINS, st);
    const SampleArgs a{temperature, gumbel, given_bins, bins_out, logp, ent, logits, out_stride, out_off};
    if (n_rows > VLA_HEAD_PARTIAL_ROWS) {
        const int grid = (n_rows + 31) / 32;
        if (norm) head_whole_kernel<T, true><<<grid, 256, 0, st>>>(h, norm->gain, norm->eps, lm_head_bins, a, X_next, embed, vocab, n_rows, H);
        else head_whole_kernel<T, false><<<grid, 256, 0, st>>>(h, nullptr, 0.f, lm_head_bins, a, X_next, embed, vocab, n_rows, H);
        return vla_check_launch("head_sample");
    }
    if (int rc = norm ? launch_head_partial<T, true>(h, norm->gain, lm_head_bins, scratch, norm->squares, n_rows, H, st)
                      : launch_head_logits<T>(h, lm_head_bins, scratch, n_rows, H, st)) return rc;
    sample_kernel<T><<<n_rows + (next ? 1 : 0), 256, 0, st>>>(scratch, head_chunks(H), n_rows, a, X_next, embed, vocab, H, next ? *next : NextStep{},
                                                              norm ? norm->squares : nullptr, norm ? norm->eps : 0.f);
    return vla_check_launch("head_sample");
}

#define INSTANTIATE(T)                                                                                        \
    template int launch_head_logits<T>(const float *, const T *, float *, int, int, hipStream_t);             \
    template int launch_head_sample<T>(const float *, const T *, int, int, float, const float *,              \
                                       const int32_t *, int32_t *, float *, float *, float *, int, int,       \
                                       float *, const T *, int, float *, hipStream_t, const NextStep *, const HeadNorm *);
INSTANTIATE(float)
INSTANTIATE(bf16_t)
