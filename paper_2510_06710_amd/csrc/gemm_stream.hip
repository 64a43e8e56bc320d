// bf16 GEMM for forwards of at most 32 rows (decode steps of up to 32 environments, few tail rows):
// C[M, N] = A[M, K] . W[N, K]^T, bound by the weight bytes from HBM.
//
// One workgroup of eight waves per 16 * R weight rows (SwiGLU: 16 * R gate and the matching up rows) and the whole of K:
// the waves take the 32-wide K steps in turn, each on its own, without barriers, with UN steps of loads in flight, and their
// sums are added in wave order through LDS at the end.  So no partial sums travel through memory, the epilogue is the
// final one and no reduction kernel follows.  Weights go from memory straight into MFMA operand registers: in the
// repacked layout ([K / 32][rows][32]) a fragment of 16 rows x 32 columns is 1 KB in a row, one load instruction; row-major
// weights take the same instruction with 64-byte pieces.  Activations (L2) come the same way, shared by the R row blocks.
// One (O, down) to three workgroups share a CU; a CU streams up to 58 GB/s, 256 of them 6 TB/s together.
// Measured at one row on the 7B shape against the split-K form (gemm_skinny.hip) and the reductions that follow it: QKV 23.4
// -> 18.7 us, O and down 27.8 + 5.3 -> 13.6 + 3.9 (mean, with the norm), gate/up 43.1 + 4.6 -> 32.6 us (5.5 TB/s).  The
// activations' L2 traffic (every workgroup reads all of them) grows with the rows: 16 rows 27 / 19 / 39 us, 32 rows 33 /
// 24 / 47 us, where both forms cost the same per layer; 64 rows 49 / 40 / 69 against 32 / 25 / 57 us, so the rule ends at 32.
//
// NORM rows (1, or up to 4): the activations are RMSNorm(x) g of fp32 rows x of at most 4096 columns (eight per thread),
// which every workgroup forms for itself in LDS while its first weights are on the way.  At one row the two norms of a layer
// took 9.4 us in launches of their own; the GEMMs with them take 31.7 us for gate/up (32.7 without: fewer registers, two
// workgroups per CU) and 19.1 for QKV (18.0).  With four rows, norm included, 37 and 26 against 34 + 6 and 21 + 6; the rows
// that a thread holds end the rule there.
#include "vla_internal.h"

namespace {

struct StreamParams {
    const bf16_t *A;
    const bf16_t *W0, *W1, *W2;
    void *C;
    const float *x, *gain;     // NORM: the fp32 rows and the norm's gain, instead of A
    float eps;
    int M, N, K, segN;
    size_t w_row, w_step;      // elements between weight rows and between 32-column steps of one row
};

template <int EPI, int MBK, int R, int UN, int NORM>
__global__ void __launch_bounds__(512) gemm_stream_kernel(StreamParams p) {
    constexpr int NW = 8, NP = (EPI == EPI_SWIGLU) ? 2 : 1;
    __shared__ __attribute__((aligned(16))) f32x4_t part[NW][NP * R * MBK][64];
    __shared__ float squares[NORM ? NORM : 1][NW];
    extern __shared__ __attribute__((aligned(16))) bf16_t xs[];         // NORM: [M][K + 32], a 16-bank shift per row
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kq = lane >> 4;
    const int K = p.K, steps = K / 32, n0 = blockIdx.x * (16 * R);
    const bf16_t *a[MBK], *w[NP][R];
#pragma unroll
    for (int i = 0; i < MBK; i++) a[i] = (NORM ? xs + min(l16, p.M - 1) * (K + 32) : p.A + (size_t)min(i * 16 + l16, p.M - 1) * K) + kq * 8;
    if (EPI == EPI_SWIGLU) {
#pragma unroll
        for (int r = 0; r < R; r++) {
            w[0][r] = p.W0 + (size_t)(n0 + r * 16 + l16) * p.w_row + kq * 8;
            w[NP - 1][r] = p.W1 + (size_t)(n0 + r * 16 + l16) * p.w_row + kq * 8;
        }
    } else {
        const int seg = n0 / p.segN;                     // (segN is a multiple of 16 * R)
        const bf16_t *W = (seg == 0 ? p.W0 : (seg == 1 ? p.W1 : p.W2)) + (size_t)(n0 - seg * p.segN + l16) * p.w_row + kq * 8;
#pragma unroll
        for (int r = 0; r < R; r++) w[0][r] = W + (size_t)(r * 16) * p.w_row;
    }
    f32x4_t acc[NP][R][MBK];
#pragma unroll
    for (int b = 0; b < NP; b++)
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int i = 0; i < MBK; i++) acc[b][r][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    bf16x8_t wf[UN][NP][R], af[UN][MBK];
    auto load = [&](int u, int s) {
        const size_t wo = (size_t)s * p.w_step, ao = (size_t)s * 32;
#pragma unroll
        for (int b = 0; b < NP; b++)
#pragma unroll
            for (int r = 0; r < R; r++) wf[u][b][r] = *(const bf16x8_t *)(w[b][r] + wo);
#pragma unroll
        for (int i = 0; i < MBK; i++)
            if (!NORM) af[u][i] = *(const bf16x8_t *)(a[i] + ao);
    };
    auto multiply = [&](int u, int s) {
        if (NORM) af[u][0] = *(const bf16x8_t *)(a[0] + s * 32);
#pragma unroll
        for (int b = 0; b < NP; b++)
#pragma unroll
            for (int r = 0; r < R; r++)
#pragma unroll
                for (int i = 0; i < MBK; i++)
                    acc[b][r][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[u][b][r], af[u][i], acc[b][r][i], 0, 0, 0);
    };
    // The waves take pairs of steps in turn (a pair is one 128-byte line of a row-major row): step i of this wave is
    // step_of(i), `mine` of them.  UN are in flight, each slot reloaded as soon as it is used.
    auto step_of = [&](int i) { return ((i >> 1) * NW + wave) * 2 + (i & 1); };
    const int pairs = steps >> 1, mine = 2 * ((pairs - wave + NW - 1) / NW) + ((steps & 1) && pairs % NW == wave ? 1 : 0);
    // NORM: this thread's eight columns of every row, asked for ahead of the weights (loads return in order)
    typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
    f32x4_t xv[NORM ? NORM : 1][2], gv[2];
    if (NORM) {
        const int k = min((int)threadIdx.x * 8, K - 8);
#pragma unroll
        for (int h = 0; h < 2; h++) {
            gv[h] = *(const f4u *)(p.gain + k + h * 4);
#pragma unroll
            for (int m = 0; m < NORM; m++) xv[m][h] = *(const f32x4_t *)(p.x + (size_t)min(m, p.M - 1) * K + k + h * 4);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < UN; u++)
        if (u < mine) load(u, step_of(u));
    if (NORM) {
        __builtin_amdgcn_sched_barrier(0);
        const int k = threadIdx.x * 8;
#pragma unroll
        for (int m = 0; m < NORM; m++) {
            float ss = 0.f;
            if (k < K)
#pragma unroll
                for (int e = 0; e < 8; e++) ss += xv[m][e >> 2][e & 3] * xv[m][e >> 2][e & 3];
#pragma unroll
            for (int o = 32; o; o >>= 1) ss += __shfl_xor(ss, o, 64);
            if (lane == 0) squares[m][wave] = ss;
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < NORM; m++) {
            float sq = 0.f;
#pragma unroll
            for (int i = 0; i < NW; i++) sq += squares[m][i];
            const float r_rms = 1.0f / sqrtf(sq / (float)K + p.eps);
            bf16x8_t v;
#pragma unroll
            for (int e = 0; e < 8; e++) v[e] = (bf16_t)(xv[m][e >> 2][e & 3] * r_rms * gv[e >> 2][e & 3]);
            if (m < p.M && k < K) *(bf16x8_t *)(xs + m * (K + 32) + k) = v;
        }
        __syncthreads();
    }
    int i0 = 0;
    for (; i0 + 2 * UN <= mine; i0 += UN) {
#pragma unroll
        for (int u = 0; u < UN; u++) {
            multiply(u, step_of(i0 + u));
            load(u, step_of(i0 + UN + u));
        }
    }
    // the last one or two groups: at most 2 UN - 1 steps
#pragma unroll
    for (int u = 0; u < UN; u++) {
        if (i0 + u < mine) {
            multiply(u, step_of(i0 + u));
            if (i0 + UN + u < mine) load(u, step_of(i0 + UN + u));
        }
    }
#pragma unroll
    for (int u = 0; u < UN; u++)
        if (i0 + UN + u < mine) multiply(u, step_of(i0 + UN + u));
#pragma unroll
    for (int b = 0; b < NP; b++)
#pragma unroll
        for (int r = 0; r < R; r++)
#pragma unroll
            for (int i = 0; i < MBK; i++) part[wave][(b * R + r) * MBK + i][lane] = acc[b][r][i];
    __syncthreads();
    // block (r, i): lane holds row i * 16 + l16, columns n0 + r * 16 + 4 kq .. + 3
    for (int blk = wave; blk < R * MBK; blk += NW) {
        const int r = blk / MBK, i = blk - r * MBK, m = i * 16 + l16;
        if (m >= p.M) continue;
        f32x4_t sum[NP];
#pragma unroll
        for (int b = 0; b < NP; b++) {
            sum[b] = part[0][(b * R + r) * MBK + i][lane];
#pragma unroll
            for (int k = 1; k < NW; k++) {
                const f32x4_t v = part[k][(b * R + r) * MBK + i][lane];
#pragma unroll
                for (int e = 0; e < 4; e++) sum[b][e] += v[e];
            }
        }
        const size_t o = (size_t)m * p.N + n0 + r * 16 + kq * 4;
        if (EPI == EPI_SWIGLU) {
            bf16x4_t v;
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = (bf16_t)vla_silu_mul(sum[0][e], sum[NP - 1][e]);
            *(bf16x4_t *)((bf16_t *)p.C + o) = v;
        } else {
            f32x4_t *dst = (f32x4_t *)((float *)p.C + o);
            if (EPI == EPI_RESIDUAL) {
                const f32x4_t x = *dst;
#pragma unroll
                for (int e = 0; e < 4; e++) sum[0][e] += x[e];
            }
            *dst = sum[0];
        }
    }
}

template <int EPI>
void launch_rows(const StreamParams &p, hipStream_t st) {
    // Steps in flight: as many as leave at most 128 registers, two workgroups per CU (gate/up at 13 rows: 6 steps, 140 registers
    // 37.5 us, 5 steps 34.5; 3 or 4 steps the same)
    constexpr int UN = EPI == EPI_SWIGLU ? 5 : 8, UN_NORM = EPI == EPI_SWIGLU ? 6 : 8;
    if constexpr (EPI != EPI_RESIDUAL) {
        const size_t lds = (size_t)p.M * (p.K + 32) * sizeof(bf16_t);
        if (p.x && p.M == 1) { gemm_stream_kernel<EPI, 1, 1, UN_NORM, 1><<<p.N / 16, 512, lds, st>>>(p); return; }
        if (p.x) { gemm_stream_kernel<EPI, 1, 1, UN_NORM, 4><<<p.N / 16, 512, lds, st>>>(p); return; }
    }
    if (p.M <= 16) gemm_stream_kernel<EPI, 1, 1, UN, 0><<<p.N / 16, 512, 0, st>>>(p);
    else if (EPI == EPI_RESIDUAL) gemm_stream_kernel<EPI, 2, 1, 4, 0><<<p.N / 16, 512, 0, st>>>(p);
    else gemm_stream_kernel<EPI, 2, 2, 4, 0><<<p.N / 32, 512, 0, st>>>(p);     // wide outputs: two row blocks share the activations
}

}  // namespace

// Whether a step's GEMM of these sizes forms its activations' norm itself: a row in one pass of the workgroup's threads.
bool gemm_stream_norms(int M, int K, int segN) {
    return M >= 1 && M <= 4 && K % 32 == 0 && segN % 32 == 0 && K <= 4096;
}

// Takes up to 32 rows (above that the activations' L2 traffic costs more than it saves), K a multiple of 32, segments a multiple of 16 rows; prefers the repacked weights.  Returns 1 if
// handled, 0 if declined, < 0 on a launch error.
int try_gemm_bf16_stream(const GemmArgs &g, hipStream_t st) {
    if (g.kblocked || g.M < 1 || g.M > 32 || g.K % 32 != 0 || g.segN % 32 != 0) return 0;
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
    p.w_row = kb ? 32 : (size_t)g.K;
    p.w_step = kb ? (size_t)(g.segN + VLA_KB_PAD_ROWS) * 32 : 32;
    p.C = g.C; p.M = g.M; p.K = g.K; p.segN = g.segN;
    p.N = g.epilogue == EPI_SWIGLU ? g.segN : g.n_seg * g.segN;
    const double wbytes = 2.0 * g.K * (double)n_seg * g.segN;
    ProfScope ps(g.epilogue == EPI_SWIGLU ? "gemm_stream<swiglu>" : g.epilogue == EPI_RESIDUAL ? "gemm_stream<residual>"
                                                                                              : "gemm_stream<store>", wbytes, st);
    if (g.epilogue == EPI_SWIGLU) launch_rows<EPI_SWIGLU>(p, st);
    else if (g.epilogue == EPI_RESIDUAL) launch_rows<EPI_RESIDUAL>(p, st);
    else launch_rows<EPI_STORE>(p, st);
    const int rc = vla_check_launch("gemm_stream");
    return rc ? rc : 1;
}
