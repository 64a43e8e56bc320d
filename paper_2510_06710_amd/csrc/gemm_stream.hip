// bf16 GEMM for decode steps of at most 32 environments: C[M, N] = A[M, K] . W[N, K]^T, bound by the weight bytes from HBM.
//
// One workgroup of eight waves per 16 output columns (SwiGLU: 16 gate and the matching up rows of the weights) and the whole
// of K: each wave takes one of the parts into which a decode step cuts K (gemm_decode_parts; with fewer parts a workgroup may
// have more columns) and walks it alone, without barriers; the parts are added in order through LDS at the end.  So no partial sums
// travel through memory, the epilogue is the final one and no reduction kernel follows.
//
// The sums are those of gemm_skinny.hip bit for bit: v_mfma_f32_32x32x16_bf16 on the same columns (8 j .. + 7 of either half
// of a 64-column tile) in the same order.  That operand is a 16-byte piece of every 64: a lane that loaded it alone would
// leave the rest of the line to three more instructions.  Two loads fetch the whole lines of 16 rows instead and the pieces
// change places between lane rows afterwards (v_permlane16_swap).  Of k-blocked weights each load brings 1 KB by itself (WHOLE),
// past the caches where they are more than these keep until the next step.  With 16 activation rows half of the instruction's columns
// are idle, with 16 weight rows half of its rows: the matrix cores have the time.
//
// What counts is the number of waves with loads in flight, not the loads per wave: with one tile each in flight, about 64
// registers, three or four workgroups share a CU.  Measured on the 7B shape with repacked weights (time between events around
// the launch, at 1 / 16 rows): QKV 24 / 26 us, O and down 16 / 20 (mean; 23 at 32 rows), gate/up 35 / 38 (30 / 32 in the kernel since WHOLE); two or three tiles in
// flight cost gate/up 0 / 2 us more.  The split-K form takes 25 / 26, 22 / 23 (23) and 45 / 47 us and leaves 26 to 33 us of
// reductions a layer that this one does not need.
//
// NORM rows (1, or up to 4): the activations are RMSNorm(x) g of fp32 rows x of at most 4096 columns, which every workgroup
// forms for itself in LDS, with the sums of the norm kernels, while its first weights are on the way: 0 to 2 us more in the
// kernel for a launch of 6 us less.  The rows that a thread holds end the rule at four.
#include "vla_internal.h"

#include <type_traits>

namespace {

constexpr int NW = 8;                  // waves of a workgroup

// Row-major weights half a line per load; k-blocked ones whole kilobytes (WHOLE), past the caches or through them.
enum WeightRead { READ_ROWS = 0, READ_WHOLE = 1, READ_PAST = 2 };

struct StreamParams {
    const bf16_t *A;
    const bf16_t *W0, *W1, *W2;
    void *C;
    const float *x, *gain;     // NORM: the fp32 rows and the norm's gain, instead of A
    float eps;
    int M, N, K, segN;
    int parts;                 // K parts of the sums (1, 2, 4 or 8), one wave each
    int groups;                // blocks of columns per workgroup, at most NW / parts (waves beyond them only help with the norm)
    size_t w_row, w_step;      // elements between weight rows and between 32-column steps of one row
    int read;                  // how they are loaded
};

// A 64-column tile of 16 * B rows as it was loaded (x[c][b]: lane l holds columns 32 (l / 32) + 16 c + 8 (l / 16 % 2) .. + 7 of row
// l % 16 of block b, so that both loads of a block use the same whole cache lines) -> the operands of four 32 x 32 x 16
// instructions: op[j], lane l = columns 32 (l / 32) + 8 j .. + 7 of row l % 32 (B = 1: of row l % 16).
template <int B>
__device__ __forceinline__ void operands(bf16x8_t (&op)[4], const bf16x8_t (&x)[2][B]) {
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int c = 0; c < 2; c++) {
        const u4 v0 = __builtin_bit_cast(u4, x[c][0]), v1 = __builtin_bit_cast(u4, x[c][B - 1]);
        u4 o0, o1;
#pragma unroll
        for (int d = 0; d < 4; d++) {                   // lane rows of 16: second 8 columns of block 0 <-> first 8 of block 1
            const auto r = __builtin_amdgcn_permlane16_swap(v0[d], v1[d], false, false);
            o0[d] = r[0]; o1[d] = r[1];
        }
        op[2 * c] = __builtin_bit_cast(bf16x8_t, o0);
        op[2 * c + 1] = __builtin_bit_cast(bf16x8_t, o1);
    }
}

// x[c][b]: lane l holds columns 32 c + 8 (l / 16) .. + 7 of row l % 16 -> as above (lane 32 + l of x[0] against lane l of x[1])
template <int B>
__device__ __forceinline__ void change_halves(bf16x8_t (&x)[2][B]) {
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int b = 0; b < B; b++) {
        u4 v0 = __builtin_bit_cast(u4, x[0][b]), v1 = __builtin_bit_cast(u4, x[1][b]);
#pragma unroll
        for (int d = 0; d < 4; d++) {
            const auto r = __builtin_amdgcn_permlane32_swap(v0[d], v1[d], false, false);
            v0[d] = r[0]; v1[d] = r[1];
        }
        x[0][b] = __builtin_bit_cast(bf16x8_t, v0);
        x[1][b] = __builtin_bit_cast(bf16x8_t, v1);
    }
}

// A wave multiplies 32 weight rows (SwiGLU: 16 gate and the matching up rows; NB = 1: 16 rows, twice) by 16 * MB activation
// rows.  UN: tiles of 64 columns in flight, NORM: activation rows that the kernel norms itself (0: none).
// WHOLE (k-blocked weights): a load brings 1 KB, 16 rows' whole 64 bytes of one 32-column step, and the steps change places between
// the halves of the wave afterwards; as all of a line is used at once, it may leave the caches at once (READ_PAST, the caller's to choose), and the K
// and V of the step's environments (4.7 MB an environment of 289 keys and layer) find more of them there.  7B width, 1 environment: gate/up 32.7 -> 30.0 us, attention
// 9.3 -> 7.1; 13: 35.1 -> 31.6 and 14.3 -> 10.6.  (Whole pieces without the hint: as before; the hint on halves of pieces: gate/up 36.8.)
template <int EPI, int NB, int MB, int UN, int NORM, int READ>
__global__ void __launch_bounds__(64 * NW) gemm_stream_kernel(StreamParams p) {
    constexpr bool SW = EPI == EPI_SWIGLU, WHOLE = READ != READ_ROWS;
    constexpr int COLS = SW ? 16 : 16 * NB, LDW = 16 * NB + 4;          // output columns, floats of a row of sums
    __shared__ float squares[NORM ? NORM : 1][4], chain[NORM ? NORM : 1][256];
    extern __shared__ __attribute__((aligned(16))) char lds[];
    float *part = (float *)lds;                                         // [wave][M][LDW]
    bf16_t *xs = (bf16_t *)(lds + (size_t)NW * p.M * LDW * 4);          // NORM: [M][K + 32], a 16-bank shift per row
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, l32 = lane & 31, hh = lane >> 5, c1 = (lane >> 4) & 1;
    const int K = p.K, blocks = p.N / COLS, group = wave / p.parts, y = wave - group * p.parts;
    const int block = group < p.groups ? blockIdx.x * p.groups + group : blocks, n0 = min(block, blocks - 1) * COLS;
    const bf16_t *a[MB], *w[NB];
#pragma unroll
    for (int i = 0; i < MB; i++) a[i] = p.A + (size_t)min(i * 16 + l16, p.M - 1) * K + hh * 32 + c1 * 8;
    const bf16_t *xrow = xs + min(l32, p.M - 1) * (K + 32) + hh * 32;
    const size_t w_off = (WHOLE ? (size_t)(lane >> 4) * 8 : hh * p.w_step + c1 * 8) + (size_t)l16 * p.w_row;
    if (SW) {
        w[0] = p.W0 + (size_t)n0 * p.w_row + w_off;
        w[NB - 1] = p.W1 + (size_t)n0 * p.w_row + w_off;
    } else {
        const int seg = n0 / p.segN;                     // (segN is a multiple of 128)
        const bf16_t *W = (seg == 0 ? p.W0 : (seg == 1 ? p.W1 : p.W2)) + (size_t)(n0 - seg * p.segN) * p.w_row + w_off;
#pragma unroll
        for (int r = 0; r < NB; r++) w[r] = W + (size_t)(r * 16) * p.w_row;
    }
    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0.f;
    bf16x8_t wf[UN][2][NB], af[UN][2][MB];
    auto load = [&](int u, int kt) {
        const size_t wo = (size_t)(2 * kt) * p.w_step, ao = (size_t)kt * 64;
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int r = 0; r < NB; r++) {
                if (READ == READ_PAST) wf[u][c][r] = __builtin_bit_cast(bf16x8_t, __builtin_nontemporal_load((const i32x4_v *)(w[r] + wo + c * p.w_step)));
                else if (WHOLE) wf[u][c][r] = *(const bf16x8_t *)(w[r] + wo + c * p.w_step);
                else wf[u][c][r] = *(const bf16x8_t *)(w[r] + wo + c * 16);
            }
        if (!NORM)
#pragma unroll
            for (int c = 0; c < 2; c++)
#pragma unroll
                for (int i = 0; i < MB; i++) af[u][c][i] = *(const bf16x8_t *)(a[i] + ao + c * 16);
    };
    auto multiply = [&](int u, int kt) {
        bf16x8_t ao[4], wo[4];
        if (NORM) {
#pragma unroll
            for (int j = 0; j < 4; j++) ao[j] = *(const bf16x8_t *)(xrow + kt * 64 + j * 8);
        } else {
            operands<MB>(ao, af[u]);
        }
        if (WHOLE) change_halves<NB>(wf[u]);
        operands<NB>(wo, wf[u]);
#pragma unroll
        for (int j = 0; j < 4; j++) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wo[j], ao[j], acc, 0, 0, 0);
    };
    // This wave's tiles: part y of the K range, one after the other.  UN are in flight, each slot reloaded as soon as it is used.
    const int tiles = K / 64, kt0 = (int)((long)y * tiles / p.parts), mine = block < blocks ? (int)((long)(y + 1) * tiles / p.parts) - kt0 : 0;
    // NORM: this thread's two pieces of every row, asked for ahead of the weights (loads return in order).  The sums are those
    // of the norm kernels' 256 threads, of which thread t adds the pieces of columns 4 (256 j + t) .. + 3 for j = 0, 1, ..: here
    // thread t has the first two, thread 256 + t goes on with the other two.
    typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
    const int t256 = threadIdx.x & 255, half = threadIdx.x >> 8;
    f32x4_t xv[NORM ? NORM : 1][2], gv[2];
    if (NORM) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int k = min(((2 * half + h) * 256 + t256) * 4, K - 4);
            gv[h] = *(const f4u *)(p.gain + k);
#pragma unroll
            for (int m = 0; m < NORM; m++) xv[m][h] = *(const f32x4_t *)(p.x + (size_t)min(m, p.M - 1) * K + k);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < UN; u++)
        if (u < mine) load(u, kt0 + u);
    if (NORM) {
        __builtin_amdgcn_sched_barrier(0);
        float ss[NORM ? NORM : 1];
        auto add = [&](int m) {
#pragma unroll
            for (int h = 0; h < 2; h++)
                if (((2 * half + h) * 256 + t256) * 4 < K) {
#pragma unroll
                    for (int e = 0; e < 4; e++) ss[m] += xv[m][h][e] * xv[m][h][e];
                }
        };
        if (half == 0) {
#pragma unroll
            for (int m = 0; m < NORM; m++) { ss[m] = 0.f; add(m); chain[m][t256] = ss[m]; }
        }
        __syncthreads();
        if (half == 1) {
#pragma unroll
            for (int m = 0; m < NORM; m++) {
                ss[m] = chain[m][t256];
                add(m);
                ss[m] = vla_wave_sum(ss[m]);
                if (lane == 0) squares[m][wave & 3] = ss[m];
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < NORM; m++) {
            const float *sq = squares[m];
            const float r_rms = 1.0f / sqrtf((sq[0] + sq[1] + sq[2] + sq[3]) / (float)K + p.eps);
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int k = ((2 * half + h) * 256 + t256) * 4;
                bf16x4_t v;
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = (bf16_t)(xv[m][h][e] * r_rms * gv[h][e]);
                if (m < p.M && k < K) *(bf16x4_t *)(xs + m * (K + 32) + k) = v;
            }
        }
        __syncthreads();
    }
    int i0 = 0;
    for (; i0 + 2 * UN <= mine; i0 += UN) {
#pragma unroll
        for (int u = 0; u < UN; u++) {
            multiply(u, kt0 + i0 + u);
            load(u, kt0 + i0 + UN + u);
        }
    }
    // the last one or two groups: at most 2 UN - 1 tiles
#pragma unroll
    for (int u = 0; u < UN; u++) {
        if (i0 + u < mine) {
            multiply(u, kt0 + i0 + u);
            if (i0 + UN + u < mine) load(u, kt0 + i0 + UN + u);
        }
    }
#pragma unroll
    for (int u = 0; u < UN; u++)
        if (i0 + UN + u < mine) multiply(u, kt0 + i0 + UN + u);
    // lane l holds activation row l % 32, weight rows 8 g + 4 (l / 32) .. + 3 in registers 4 g .. + 3
    if (l32 < p.M && (MB > 1 || l32 < 16)) {
#pragma unroll
        for (int g = 0; g < 2 * NB; g++)
            *(f32x4_t *)(part + (wave * p.M + l32) * LDW + 8 * g + 4 * hh) = f32x4_t{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    }
    __syncthreads();
    // the parts of a block are added in K order: four columns of one row per thread
    constexpr int QUADS = COLS / 4;
    for (int item = threadIdx.x; item < p.groups * p.M * QUADS; item += 64 * NW) {
        const int q = item % QUADS, gm = item / QUADS, gr = gm / p.M, m = gm - gr * p.M;
        const int blk = blockIdx.x * p.groups + gr;
        if (blk >= blocks) break;
        const float *src = part + (gr * p.parts * p.M + m) * LDW + q * 4;
        auto sum_of = [&](int off) {
            f32x4_t sum = *(const f32x4_t *)(src + off);
            for (int k = 1; k < p.parts; k++) {
                const f32x4_t v = *(const f32x4_t *)(src + off + k * p.M * LDW);
#pragma unroll
                for (int e = 0; e < 4; e++) sum[e] += v[e];
            }
            return sum;
        };
        f32x4_t sum = sum_of(0);
        const size_t o = (size_t)m * p.N + blk * COLS + q * 4;
        if (SW) {
            const f32x4_t up = sum_of(16);
            bf16x4_t v;
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = (bf16_t)vla_silu_mul(sum[e], up[e]);
            *(bf16x4_t *)((bf16_t *)p.C + o) = v;
        } else {
            f32x4_t *dst = (f32x4_t *)((float *)p.C + o);
            if (EPI == EPI_RESIDUAL) {
                const f32x4_t x = *dst;
#pragma unroll
                for (int e = 0; e < 4; e++) sum[e] += x[e];
            }
            *dst = sum;
        }
    }
}

template <int EPI, int NB, int MB, int NORM>
int launch(StreamParams p, hipStream_t st) {
    // (at most 21 KB of sums, or 5 KB and 34 KB of normed rows)
    const size_t lds = (size_t)NW * p.M * (16 * NB + 4) * 4 + (NORM ? (size_t)p.M * (p.K + 32) * sizeof(bf16_t) : 0);
    const int blocks = p.N / (EPI == EPI_SWIGLU ? 16 : 16 * NB);
    // One block per workgroup until every CU has one, then as many as there are waves for: width 1024, FFN 2816 (two parts) at
    // 1 row 44 -> 37 us a layer.  One workgroup per CU has the registers for a second tile in flight: 37 -> 34 (above 16 rows
    // each tile brings twice the activations, and one is better: 7B shape, O and down at 32 rows 23 us against 25).
    p.groups = (blocks + 255) / 256 < NW / p.parts ? (blocks + 255) / 256 : NW / p.parts;
    const int grid = (blocks + p.groups - 1) / p.groups;
    auto go = [&](auto read) {
        constexpr int READ = decltype(read)::value;
        if (MB == 1 && grid <= 256) gemm_stream_kernel<EPI, NB, MB, MB == 1 ? 2 : 1, NORM, READ><<<grid, 64 * NW, lds, st>>>(p);
        else gemm_stream_kernel<EPI, NB, MB, 1, NORM, READ><<<grid, 64 * NW, lds, st>>>(p);
    };
    if (p.read == READ_PAST) go(std::integral_constant<int, READ_PAST>{});
    else if (p.read == READ_WHOLE) go(std::integral_constant<int, READ_WHOLE>{});
    else go(std::integral_constant<int, READ_ROWS>{});
    return vla_check_launch("gemm_stream");
}

template <int EPI>
int launch_rows(const StreamParams &p, hipStream_t st) {
    constexpr int NB = EPI == EPI_SWIGLU ? 2 : 1;
    if constexpr (EPI != EPI_RESIDUAL) {
        if (p.x && p.M == 1) return launch<EPI, NB, 1, 1>(p, st);
        if (p.x) return launch<EPI, NB, 1, 4>(p, st);
    }
    if (p.M <= 16) return launch<EPI, NB, 1, 0>(p, st);
    return launch<EPI, NB, 2, 0>(p, st);
}

}  // namespace

// Whether a step's GEMM of these sizes forms its activations' norm itself: a row in one pass of the workgroup's threads.
bool gemm_stream_norms(int M, int K, int segN) {
    return M >= 1 && M <= 4 && K % 64 == 0 && segN % 128 == 0 && K <= 4096;
}

// Takes up to 32 rows (QKV and gate/up of more than 8192 columns: 16) of the shapes that the split-K form takes (K a multiple of
// 64, segments of 128 rows), so that either both can form a product or neither; prefers the repacked weights.  Above those rows
// the activations' traffic, which grows with the columns, costs more than it saves.  7B shape: QKV and gate/up take 26 + 38 us at
// 16 rows, 28 + 39 at 17 and 33 + 46 at 32, on the small tiles 27 + 40 at all of these (row-major weights: 30 + 42, 31 + 45,
// 36 + 53 against 29 + 45); O and down 23 at 32 rows, in the split-K form 23 and a reduction.  Whole decode of 6 steps x 4
// layers at 24 / 32 rows, here against the small tiles: width 1024 1.06 / 1.09 against 1.13 / 1.16 ms, width 2048 with FFN 5504
// 1.58 / 1.70 against 1.78 / 1.84 and with FFN 8192 1.89 / 2.15 against 2.06 / 2.21, width 5120 5.37 / 5.89 against 4.55 / 4.80.
// Returns 1 if handled, 0 if declined, < 0 on a launch error.
int try_gemm_bf16_stream(const GemmArgs &g, hipStream_t st) {
    const bool narrow = g.epilogue == EPI_RESIDUAL || (g.epilogue == EPI_SWIGLU ? 1 : g.n_seg) * (long)g.segN <= 8192;
    if (g.kblocked || g.M < 1 || g.M > (narrow ? 32 : 16) || g.K % 64 != 0 || g.segN % 128 != 0) return 0;
    if (g.epilogue != EPI_STORE && g.epilogue != EPI_RESIDUAL && g.epilogue != EPI_SWIGLU) return 0;
    if (g.norm_x && (g.epilogue == EPI_RESIDUAL || !gemm_stream_norms(g.M, g.K, g.segN))) return 0;
    const int n_seg = g.epilogue == EPI_SWIGLU ? 2 : g.n_seg;
    StreamParams p{};
    p.x = g.norm_x; p.gain = g.norm_gain; p.eps = g.norm_eps;
    p.A = (const bf16_t *)g.A;
    bool kb = true;
    for (int i = 0; i < n_seg; i++) kb = kb && g.Wkb[i];
    const void *const *W = kb ? g.Wkb : g.W;
    p.W0 = (const bf16_t *)W[0]; p.W1 = (const bf16_t *)W[1]; p.W2 = (const bf16_t *)W[2];
    p.read = !kb ? READ_ROWS : g.past_caches ? READ_PAST : READ_WHOLE;
    p.w_row = kb ? 32 : (size_t)g.K;
    p.w_step = kb ? (size_t)(g.segN + VLA_KB_PAD_ROWS) * 32 : 32;
    p.C = g.C; p.M = g.M; p.K = g.K; p.segN = g.segN;
    p.N = g.epilogue == EPI_SWIGLU ? g.segN : g.n_seg * g.segN;
    p.parts = gemm_decode_parts(p.N, p.K);
    const double wbytes = 2.0 * g.K * (double)n_seg * g.segN;
    ProfScope ps(g.epilogue == EPI_SWIGLU ? "gemm_stream<swiglu>" : g.epilogue == EPI_RESIDUAL ? "gemm_stream<residual>"
                                                                                              : "gemm_stream<store>", wbytes, st);
    const int rc = g.epilogue == EPI_SWIGLU ? launch_rows<EPI_SWIGLU>(p, st)
                   : g.epilogue == EPI_RESIDUAL ? launch_rows<EPI_RESIDUAL>(p, st) : launch_rows<EPI_STORE>(p, st);
    return rc ? rc : 1;
}
