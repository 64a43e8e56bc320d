// LoRA gradients of a group of projections that share their input, for bf16 storage: with X [M, in] the input and
// dY [M, n_p * out] the output gradients side by side,
//   U_p = X A_p^T, V_p = dY_p B_p                            [M, rank], rounded to the storage type like every GEMM operand
//   dB_p = scale dY_p^T U_p [out, rank],  dA_p = scale V_p^T X [rank, in]     fp32, contractions over the rows.
// The factors are so narrow (rank 4 .. 32 columns against thousands) that each product is one pass over X or dY: both kernels
// below are bound by those reads.  They read X and dY as they lie, row-major: no transposed copies, and no columns beyond
// the rank rounded up to 16.  Sums are fp32 in a fixed order (parts of the contraction per wave and workgroup, added in
// order), so results are reproducible bit for bit.
//
// 9,408 rows of the 7B shape, rank 32, a layer's four groups: 1.83 -> 0.79 ms (tile GEMMs on factors padded to 256 columns, with
// transposed copies of X and dY, before).  The passes over dY of gate/up (414 MB): 120 us for V, 87 us for dB (4.8 TB/s).  1,981
// rows, rank 8: 48 us a group.
#include <type_traits>
#include <utility>

#include "vla_internal.h"

namespace {

typedef __attribute__((address_space(3))) void lds_void;

// The factors as the MFMA's row operands, 16 factor rows x 32 columns of a contraction in 1 KB: lane (l16, kq) holds the eight
// columns from 8 kq of row l16.  Wu: blocks of [A_0; A_1; ..] per 32 columns of the input, nj per projection; Wv: per projection
// blocks of B_p^T per 32 of its outputs.  Rows from the rank on are zeros.
struct LoraPack { LoraProducts g[5]; bf16_t *Wu[5], *Wv[5]; int nj; };           // (blockIdx.y: which of a layer's groups)
__global__ void __launch_bounds__(256) lora_pack_kernel(LoraPack pk) {
    const LoraProducts &g = pk.g[blockIdx.y];
    bf16_t *Wu = pk.Wu[blockIdx.y], *Wv = pk.Wv[blockIdx.y];
    const int nj = pk.nj, nb = g.n_p * nj, nu = (g.in / 32) * nb * 64, nv = (g.out / 32) * nj * 64;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < nu + g.n_p * nv; i += gridDim.x * 256) {
        const bool u = i < nu;
        const int p_v = u ? 0 : (i - nu) / nv, e = u ? i : (i - nu) - p_v * nv;
        const int lane = e & 63, blocks = u ? nb : nj, blk = (e >> 6) % blocks, k = (e >> 6) / blocks * 32 + (lane >> 4) * 8;
        const int p = u ? blk / nj : p_v, j = (u ? blk % nj : blk) * 16 + (lane & 15);
        bf16x8_t v;
#pragma unroll
        for (int t = 0; t < 8; t++) v[t] = (bf16_t)0.f;
        if (j < g.rank) {
            if (u) v = *(const bf16x8_t *)((const bf16_t *)g.a[p] + (size_t)j * g.in + k);
            else
#pragma unroll
                for (int t = 0; t < 8; t++) v[t] = ((const bf16_t *)g.b[p])[(size_t)(k + t) * g.rank + j];
        }
        *(bf16x8_t *)((u ? Wu : Wv + (size_t)p_v * nv * 8) + (size_t)e * 8) = v;
    }
}

struct ThinArgs {
    const bf16_t *X;         // [M, ldx]
    const bf16_t *W;         // packed factors: [K / 32][blocks][64][8], one such set per group
    bf16_t *out;             // [groups][blocks * 16][kp]: the products transposed; zeros for the rows M .. kp - 1
    int M, K, ldx, kp;
    int xstep;               // columns of X from one group (blockIdx.y) to the next
};

// out[b * 16 + j][m] = sum_k X[m][k] W_b[j][k] for 16 RB rows of X and NB blocks of 16 factor rows per workgroup.  X goes through
// LDS, 512 columns at a time, three such chunks in turn: a load instruction takes 1 KB of one row (as MFMA operands straight from
// memory, 16 rows x 64 bytes that lie a row's length apart, X arrived at 1.2 TB/s), rows 16 bytes further apart in LDS so
// that the operand reads meet no bank conflict.  Wave w multiplies columns 64 w .. + 63 of a chunk with factors on their way
// since the chunk before (through a buffer descriptor: their addresses stay scalar.  As vector registers those took registers of
// factors still on their way, and every other step waited for all but its own loads; X A^T of q | k | v at 9,408 rows, rank 32, takes
// 41.7 us either way); the waves' sums meet in LDS.
// The first n_u of the grid's columns are group 0 of u, the others the groups of v.
template <int RB, int NB>
__global__ void __launch_bounds__(512) lora_thin_kernel(ThinArgs u, ThinArgs v, int n_u) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const bool of_u = (int)blockIdx.y < n_u;
    const ThinArgs a = of_u ? u : v;
    constexpr int ROWS = 16 * RB, ROW = 1024 + 16, STG = ROWS * ROW, NX = ROWS / 8, NW = 2 * NB;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
    const int m0 = blockIdx.x * ROWS, gr = of_u ? 0 : (int)blockIdx.y - n_u, slices = a.K / 64, chunks = (slices + 7) / 8;
    if (m0 >= a.M) {             // (16-row form: kp ends in a block of padding)
        for (int e = threadIdx.x; e < NB * 16 * 16; e += 512) a.out[((size_t)gr * NB * 16 + (e >> 4)) * a.kp + m0 + (e & 15)] = (bf16_t)0.f;
        return;
    }
    // this workgroup's rows: a buffer of its own, so that a 32-bit offset reaches them; reads past its end return zero
    const int rows_in = min(ROWS, a.M - m0);
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void *)(a.X + (size_t)m0 * a.ldx + (size_t)gr * a.xstep), (short)0,
                                                                       (int)(((unsigned)(rows_in - 1) * a.ldx + a.K) * 2u), 0x00020000);
    auto load_x = [&](int c, int stage) {
#pragma unroll
        for (int i = 0; i < NX; i++) {
            const int row = wave * NX + i;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void *)(lds + stage * STG + row * ROW), 16, lane * 16,
                                                     min(row, rows_in - 1) * a.ldx * 2 + c * 1024, 0, 0);
        }
    };
    const int w_bytes = a.K / 32 * NB * 1024;
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)a.W + (size_t)gr * w_bytes), (short)0, w_bytes, 0x00020000);
    bf16x8_t wf[2][NW];
    auto load_w = [&](int s, int c) {
        const int at = min(c * 8 + wave, slices - 1) * NW * 1024;
#pragma unroll
        for (int q = 0; q < NW; q++) wf[s][q] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(wr, lane * 16, at + q * 1024, 0));
    };
    f32x4_t acc[NB][RB];
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
        for (int i = 0; i < RB; i++) acc[b][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int read0 = (int)(size_t)(lds_void *)lds + l16 * ROW + wave * 128 + kq * 16;
    load_x(0, 0);
    asm volatile("" ::: "memory");               // (the first wait below counts what is issued after chunk 0)
    load_x(min(1, chunks - 1), 1);
    load_w(0, 0);
    int stage = 0;
    auto step = [&](auto s_c, int c) {
        constexpr int s = decltype(s_c)::value;
        // chunk c has landed when at most the loads after its own are in flight: those of chunk c + 1 and the factors of c
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NX + NW) : "memory");
        asm volatile("s_barrier" ::: "memory");
        load_x(min(c + 2, chunks - 1), stage == 0 ? 2 : stage - 1);
        load_w(s ^ 1, min(c + 1, chunks - 1));
        if (c * 8 + wave < slices) {
            bf16x8_t x[2][RB];
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int i = 0; i < RB; i++) {
                    i32x4_v v;
                    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(read0 + stage * STG + i * 16 * ROW + h * 64) : "memory");
                    x[h][i] = __builtin_bit_cast(bf16x8_t, v);
                }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int i = 0; i < RB; i++) asm volatile("" : "+v"(x[h][i]));
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int b = 0; b < NB; b++)
#pragma unroll
                    for (int i = 0; i < RB; i++) acc[b][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s][h * NB + b], x[h][i], acc[b][i], 0, 0, 0);
        }
        stage = stage == 2 ? 0 : stage + 1;
    };
    for (int c = 0; c < chunks; c += 2) {
        step(std::integral_constant<int, 0>{}, c);
        if (c + 1 < chunks) step(std::integral_constant<int, 1>{}, c + 1);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // (the last chunk is fetched again, into stages that become the sums')
    __syncthreads();
    // waves 4 .. 7 hand their sums to the others, and so on down to the first
    f32x4_t *part = (f32x4_t *)lds;
#pragma unroll
    for (int half = 4; half >= 1; half /= 2) {
        if (wave >= half && wave < 2 * half)
#pragma unroll
            for (int b = 0; b < NB; b++)
#pragma unroll
                for (int i = 0; i < RB; i++) part[((wave - half) * NB * RB + b * RB + i) * 64 + lane] = acc[b][i];
        __syncthreads();
        if (wave < half)
#pragma unroll
            for (int b = 0; b < NB; b++)
#pragma unroll
                for (int i = 0; i < RB; i++) acc[b][i] += part[(wave * NB * RB + b * RB + i) * 64 + lane];
        __syncthreads();
    }
    if (wave) return;
    // lane: row l16 of a block of X, factor rows 4 kq .. 4 kq + 3
    bf16_t *out = a.out + (size_t)gr * NB * 16 * a.kp;
#pragma unroll
    for (int i = 0; i < RB; i++) {
        const int m = m0 + i * 16 + l16;
        if (m >= a.kp) continue;
#pragma unroll
        for (int b = 0; b < NB; b++)
#pragma unroll
            for (int r = 0; r < 4; r++) out[(size_t)(b * 16 + 4 * kq + r) * a.kp + m] = m < a.M ? (bf16_t)acc[b][i][r] : (bf16_t)0.f;
    }
}

struct RowsArgsT {
    const bf16_t *Y;         // [M, w] row-major
    const bf16_t *Ut;        // [..][kp]: blocks of 16 columns of U, transposed
    float *part;             // [parts][w][NB * 16]
    int M, w, kp;
    int out;                 // columns of Y that share their blocks of U: column c takes blocks (c / out) * NB .. + NB - 1
    int parts;
};

// part[s][c][j] = sum over the rows m of part s of Y[m][c] U[m][j], for 16 IW columns of Y and NB blocks of 16 columns of U per
// workgroup.  A lane reads IW neighbouring columns of eight rows, whole lines among 16 lanes, and turns them in its registers
// into IW operands of eight rows each; operand e holds the columns IW l + e (l = 0 .. 15).
constexpr int lora_columns(int nb) { return nb <= 4 ? 8 : 4; }         // IW for NB blocks
template <int IW, int NB>
__device__ __forceinline__ void lora_rows(const RowsArgsT &a, int item, f32x4_t (*sums)[64]) {
    typedef int piece_t __attribute__((ext_vector_type(IW / 2)));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kq = lane >> 4;
    const int blocks = a.w / (16 * IW), by = item / blocks;
    const int c0 = (item - by * blocks) * 16 * IW, steps = (a.M + 31) / 32, stride = 4 * a.parts;
    const bf16_t *y = a.Y + c0 + IW * l16 + (size_t)(8 * kq) * a.w;
    const bf16_t *u = a.Ut + ((size_t)(c0 / a.out) * NB * 16 + l16) * a.kp + 8 * kq;
    f32x4_t acc[NB][IW];
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
        for (int e = 0; e < IW; e++) acc[b][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    piece_t yp[2][8];
    bf16x8_t uf[2][NB];
    auto load = [&](int s, int st) {
        const int m0 = st * 32;
#pragma unroll
        for (int t = 0; t < 8; t++) {
            if (m0 + 32 <= a.M || m0 + 8 * kq + t < a.M) yp[s][t] = *(const piece_t *)(y + (size_t)(m0 + t) * a.w);
            else
#pragma unroll
                for (int d = 0; d < IW / 2; d++) yp[s][t][d] = 0;
        }
#pragma unroll
        for (int b = 0; b < NB; b++) uf[s][b] = *(const bf16x8_t *)(u + (size_t)b * 16 * a.kp + m0);
    };
    auto multiply = [&](int s) {
#pragma unroll
        for (int e = 0; e < IW; e++) {
            i32x4_v f;
#pragma unroll
            for (int q = 0; q < 4; q++)
                f[q] = (int)__builtin_amdgcn_perm((unsigned)yp[s][2 * q + 1][e / 2], (unsigned)yp[s][2 * q][e / 2], e & 1 ? 0x07060302u : 0x05040100u);
#pragma unroll
            for (int b = 0; b < NB; b++) acc[b][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(uf[s][b], __builtin_bit_cast(bf16x8_t, f), acc[b][e], 0, 0, 0);
        }
    };
    int st = by * 4 + wave;
    if (st < steps) {
        load(0, st);
        for (; st < steps; st += 2 * stride) {
            const bool second = st + stride < steps;
            if (second) load(1, st + stride);
            multiply(0);
            if (st + 2 * stride < steps) load(0, st + 2 * stride);
            if (second) multiply(1);
        }
    }
#pragma unroll
    for (int half = 2; half >= 1; half /= 2) {
        if (wave >= half && wave < 2 * half)
#pragma unroll
            for (int b = 0; b < NB; b++)
#pragma unroll
                for (int e = 0; e < IW; e++) sums[((wave - half) * NB + b) * IW + e][lane] = acc[b][e];
        __syncthreads();
        if (wave < half)
#pragma unroll
            for (int b = 0; b < NB; b++)
#pragma unroll
                for (int e = 0; e < IW; e++) acc[b][e] += sums[(wave * NB + b) * IW + e][lane];
        __syncthreads();
    }
    if (wave) return;
    // lane: column IW l16 + e, columns 4 kq .. 4 kq + 3 of a block of U
    float *out = a.part + ((size_t)by * a.w + c0 + IW * l16) * (NB * 16) + 4 * kq;
#pragma unroll
    for (int e = 0; e < IW; e++)
#pragma unroll
        for (int b = 0; b < NB; b++) *(f32x4_t *)(out + (size_t)e * (NB * 16) + b * 16) = acc[b][e];
}
// dB's products and dA's in one launch: blocks below n_b are those of `b` (NJ blocks of U each), the others those of `a` (all NJ NP of V).
template <int NJ, int NP>
__global__ void __launch_bounds__(256) lora_rows_kernel(RowsArgsT b, RowsArgsT a, int n_b) {
    constexpr int NB = NJ * NP, IB = lora_columns(NJ), IA = lora_columns(NB), SB = 2 * NJ * IB, SA = 2 * NB * IA;
    __shared__ f32x4_t sums[SB > SA ? SB : SA][64];
    if ((int)blockIdx.x < n_b) lora_rows<IB, NJ>(b, blockIdx.x, sums);
    else lora_rows<IA, NB>(a, blockIdx.x - n_b, sums);
}

// dB_p[o][j] (+)= scale * sum_s Cb[s][p * out + o][j]
__device__ __forceinline__ void lora_finish_b(const LoraProducts &g, const float *Cb, int parts, int jp, float scale, int accumulate, int p, int block) {
    const int i = block * 256 + threadIdx.x;
    if (i >= g.out * g.rank) return;
    const int o = i / g.rank, j = i - o * g.rank, w = g.n_p * g.out;
    float v = 0.f;
    for (int s = 0; s < parts; s++) v += Cb[((size_t)s * w + p * g.out + o) * jp + j];
    v *= scale;
    g.db[p][i] = accumulate ? g.db[p][i] + v : v;
}
// dA_p[j][i] (+)= scale * sum_s Ca[s][i][p * jp + j]: 16 columns i per workgroup, turned in LDS
__device__ __forceinline__ void lora_finish_a(const LoraProducts &g, const float *Ca, int parts, int jp, float scale, int accumulate, int block, float (*tile)[129]) {
    const int i0 = block * 16, n = g.n_p * jp, n4 = n / 4;
    for (int e = threadIdx.x; e < 16 * n4; e += 256) {
        const int i = e / n4, j = (e - i * n4) * 4;
        const float *src = Ca + (size_t)(i0 + i) * n + j;
        f32x4_t v = *(const f32x4_t *)src;
#pragma unroll 4
        for (int s = 1; s < parts; s++) v += *(const f32x4_t *)(src + (size_t)s * g.in * n);
#pragma unroll
        for (int t = 0; t < 4; t++) tile[i][j + t] = v[t] * scale;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < g.n_p * g.rank * 16; e += 256) {
        const int i = e & 15, row = e >> 4, p = row / g.rank, j = row - p * g.rank;
        float *d = g.da[p] + (size_t)j * g.in + i0 + i;
        const float v = tile[i][p * jp + j];
        *d = accumulate ? *d + v : v;
    }
}
// Blocks below n_b (per projection) finish dB, the others dA.
__global__ void __launch_bounds__(256) lora_finish_kernel(LoraProducts g, const float *Cb, int pb, const float *Ca, int pa, int jp, float scale, int accumulate, int n_b) {
    __shared__ float tile[16][129];
    const int b = blockIdx.x;
    if (b < n_b * g.n_p) lora_finish_b(g, Cb, pb, jp, scale, accumulate, b / n_b, b % n_b);
    else lora_finish_a(g, Ca, pa, jp, scale, accumulate, b - n_b * g.n_p, tile);
}

template <int RB, int NB>
int launch_thin(const ThinArgs &u, int n_u, const ThinArgs &v, int n_v, hipStream_t st) {
    const size_t ring = (size_t)3 * 16 * RB * (1024 + 16), sums = (size_t)4 * NB * RB * 1024, lds = ring > sums ? ring : sums;
    if (int rc = vla_allow_lds((const void *)lora_thin_kernel<RB, NB>, lds)) return rc;
    lora_thin_kernel<RB, NB><<<dim3(v.kp / (16 * RB), n_u + n_v), 512, lds, st>>>(u, v, n_u);
    return vla_check_launch("lora_thin");
}
// f(integral_constant) of the block count nb, 1 .. 8
template <int N = 1, typename F>
int with_blocks(int nb, F f) {
    if constexpr (N < 8) {
        if (nb > N) return with_blocks<N + 1>(nb, f);
    }
    return f(std::integral_constant<int, N>{});
}
// nb blocks of factor rows for n_u x u and n_v groups of v (the same rows); 32 rows of X per workgroup, 16 where that leaves CUs idle
int thin(const ThinArgs &u, int n_u, const ThinArgs &v, int n_v, int nb, hipStream_t st) {
    return with_blocks(nb, [&](auto n) {
        constexpr int NB = decltype(n)::value;
        return (v.M + 31) / 32 * (n_u + n_v) >= 192 ? launch_thin<2, NB>(u, n_u, v, n_v, st) : launch_thin<1, NB>(u, n_u, v, n_v, st);
    });
}
int parts_of(int w, int iw, int M, size_t row_bytes, size_t bytes) {
    const int blocks = w / (16 * iw), steps = (M + 31) / 32;
    int s = (1024 + blocks - 1) / blocks;                    // four workgroups of four waves per CU
    if (s > (steps + 7) / 8) s = (steps + 7) / 8;            // ... of at least two steps a wave
    if (s > 16) s = 16;
    while (s > 1 && (size_t)s * w * row_bytes > bytes) s--;
    return s < 1 ? 1 : s;
}
int rows_products(const RowsArgsT &b, const RowsArgsT &a, int nj, int n_p, hipStream_t st) {
    return with_blocks(nj, [&](auto n) {
        constexpr int NJ = decltype(n)::value;
        const int n_b = b.w / (16 * lora_columns(NJ)) * b.parts, n_a = a.w / (16 * lora_columns(NJ * n_p)) * a.parts;
        if (n_p == 1) lora_rows_kernel<NJ, 1><<<n_b + n_a, 256, 0, st>>>(b, a, n_b);
        if constexpr (NJ <= 4)
            if (n_p == 2) lora_rows_kernel<NJ, 2><<<n_b + n_a, 256, 0, st>>>(b, a, n_b);
        if constexpr (NJ <= 2)
            if (n_p == 3) lora_rows_kernel<NJ, 3><<<n_b + n_a, 256, 0, st>>>(b, a, n_b);
        return vla_check_launch("lora_rows");
    });
}

size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }
size_t packed_u(const LoraProducts &g) { return up256((size_t)g.n_p * ((g.rank + 15) / 16) * 16 * g.in * 2); }
size_t packed_v(const LoraProducts &g) { return up256((size_t)g.n_p * ((g.rank + 15) / 16) * 16 * g.out * 2); }
bool takes(const LoraProducts &g) {
    if (g.rank < 1 || g.n_p < 1 || g.n_p > 3 || g.n_p * ((g.rank + 15) / 16) > 8 || g.in % 128 != 0 || g.out % 128 != 0) return false;
    for (int p = 0; p < g.n_p; p++)
        if ((size_t)g.a[p] % 16 != 0) return false;
    return true;
}
int pack(const LoraProducts *g, int n, char *base, hipStream_t st) {
    LoraPack pk{};
    int pieces = 0;
    pk.nj = (g[0].rank + 15) / 16;
    for (int i = 0; i < n; i++) {
        pk.g[i] = g[i];
        pk.Wu[i] = (bf16_t *)base;
        pk.Wv[i] = (bf16_t *)(base + packed_u(g[i]));
        base += packed_u(g[i]) + packed_v(g[i]);
        const int here = g[i].n_p * pk.nj * 2 * (g[i].in + g[i].out);
        if (here > pieces) pieces = here;
    }
    lora_pack_kernel<<<dim3((pieces + 255) / 256, n), 256, 0, st>>>(pk);             // (a piece of eight columns per thread)
    return vla_check_launch("lora_pack");
}

}  // namespace

size_t lora_packed_bytes(const LoraProducts &g) { return takes(g) ? packed_u(g) + packed_v(g) : 0; }
// The packed factors of up to five groups of one rank, one behind the other (lora_packed_bytes of each) from `packed`, for
// try_lora_products_bf16.
int launch_lora_pack(const LoraProducts *g, int n, void *packed, hipStream_t st) { return pack(g, n, (char *)packed, st); }

// packed: the group's factors by launch_lora_pack, or NULL (packed here).  Returns 1 if handled, 0 if declined (more than 128 factor rows, widths that are no multiple of 128, unaligned operands), < 0 on
// a launch error.  scratch: 16-byte aligned, `bytes` of it; declines if that does not hold one part of each product.
int try_lora_products_bf16(const LoraProducts &g, const void *X, const void *dY, int M, float scale, bool accumulate, void *scratch, size_t bytes, hipStream_t st, const void *packed) {
    const int nj = (g.rank + 15) / 16, jp = nj * 16, wout = g.n_p * g.out, nb = g.n_p * nj, kp = (M + 31) / 32 * 32;
    if (M < 1 || !takes(g) || ((size_t)X | (size_t)dY | (size_t)scratch | (size_t)packed) % 16 != 0) return 0;
    const size_t wu_bytes = packed_u(g), w_bytes = wu_bytes + packed_v(g), t_bytes = up256((size_t)nb * 16 * kp * 2);
    const size_t used = w_bytes + 2 * t_bytes, row_b = (size_t)jp * 4, row_a = (size_t)nb * 64;
    if (bytes < used || bytes - used < wout * row_b + g.in * row_a) return 0;
    char *base = (char *)scratch;
    const bf16_t *Wu = packed ? (const bf16_t *)packed : (const bf16_t *)base, *Wv = (const bf16_t *)((const char *)Wu + wu_bytes);
    bf16_t *Ut = (bf16_t *)(base + w_bytes), *Vt = (bf16_t *)((char *)Ut + t_bytes);
    const size_t left = bytes - used;
    ProfScope ps("lora_products", 8.0 * M * g.rank * ((double)g.n_p * g.in + wout), st);
    int rc;
    if (!packed && (rc = pack(&g, 1, base, st))) return rc;
    const ThinArgs u{(const bf16_t *)X, Wu, Ut, M, g.in, g.in, kp, 0}, v{(const bf16_t *)dY, Wv, Vt, M, g.out, wout, kp, g.out};
    if (g.n_p == 1) rc = thin(u, 1, v, 1, nb, st);               // (as many blocks of factors in both: one launch)
    else if ((rc = thin(u, 1, u, 0, nb, st)) == 0) rc = thin(v, 0, v, g.n_p, nj, st);
    if (rc) return rc;
    // the partial products of dB and of dA, one behind the other
    const int pb = parts_of(wout, lora_columns(nj), M, row_b, left - g.in * row_a);
    const size_t b_bytes = (size_t)pb * wout * row_b;
    const int pa = parts_of(g.in, lora_columns(nb), M, row_a, left - b_bytes);
    float *part_b = (float *)(base + used), *part_a = (float *)((char *)part_b + b_bytes);
    if ((rc = rows_products(RowsArgsT{(const bf16_t *)dY, Ut, part_b, M, wout, kp, g.out, pb}, RowsArgsT{(const bf16_t *)X, Vt, part_a, M, g.in, kp, g.in, pa}, nj, g.n_p, st))) return rc;
    const int n_b = (g.out * g.rank + 255) / 256;
    lora_finish_kernel<<<n_b * g.n_p + g.in / 16, 256, 0, st>>>(g, part_b, pb, part_a, pa, jp, scale, accumulate, n_b);
    rc = vla_check_launch("lora_finish");
    return rc ? rc : 1;
}
