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
__global__ void __launch_bounds__(256) lora_pack_kernel(bf16_t *Wu, bf16_t *Wv, LoraProducts g, int nj) {
    const int nb = g.n_p * nj, nu = (g.in / 32) * nb * 64, nv = (g.out / 32) * nj * 64;
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
template <int RB, int NB>
__global__ void __launch_bounds__(512) lora_thin_kernel(ThinArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    constexpr int ROWS = 16 * RB, ROW = 1024 + 16, STG = ROWS * ROW, NX = ROWS / 8, NW = 2 * NB;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
    const int m0 = blockIdx.x * ROWS, gr = blockIdx.y, slices = a.K / 64, chunks = (slices + 7) / 8;
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
    float *part;             // [gridDim.y][w][NB * 16]
    int M, w, kp;
    int out;                 // columns of Y that share their blocks of U: column c takes blocks (c / out) * NB .. + NB - 1
};

// part[s][c][j] = sum over the rows m of part s of Y[m][c] U[m][j], for 16 IW columns of Y and NB blocks of 16 columns of U per
// workgroup.  A lane reads IW neighbouring columns of eight rows, whole lines among 16 lanes, and turns them in its registers
// into IW operands of eight rows each; operand e holds the columns IW l + e (l = 0 .. 15).
template <int IW, int NB>
__global__ void __launch_bounds__(256) lora_rows_kernel(RowsArgsT a) {
    typedef int piece_t __attribute__((ext_vector_type(IW / 2)));
    __shared__ f32x4_t sums[2][NB * IW][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kq = lane >> 4;
    const int c0 = blockIdx.x * 16 * IW, steps = (a.M + 31) / 32, stride = 4 * gridDim.y;
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
    int st = blockIdx.y * 4 + wave;
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
                for (int e = 0; e < IW; e++) sums[wave - half][b * IW + e][lane] = acc[b][e];
        __syncthreads();
        if (wave < half)
#pragma unroll
            for (int b = 0; b < NB; b++)
#pragma unroll
                for (int e = 0; e < IW; e++) acc[b][e] += sums[wave][b * IW + e][lane];
        __syncthreads();
    }
    if (wave) return;
    // lane: column IW l16 + e, columns 4 kq .. 4 kq + 3 of a block of U
    float *out = a.part + ((size_t)blockIdx.y * a.w + c0 + IW * l16) * (NB * 16) + 4 * kq;
#pragma unroll
    for (int e = 0; e < IW; e++)
#pragma unroll
        for (int b = 0; b < NB; b++) *(f32x4_t *)(out + (size_t)e * (NB * 16) + b * 16) = acc[b][e];
}

// dB_p[o][j] (+)= scale * sum_s Cb[s][p * out + o][j]
__global__ void __launch_bounds__(256) lora_finish_b_kernel(LoraProducts g, const float *Cb, int parts, int jp, float scale, int accumulate) {
    const int p = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
    if (i >= g.out * g.rank) return;
    const int o = i / g.rank, j = i - o * g.rank, w = g.n_p * g.out;
    float v = 0.f;
    for (int s = 0; s < parts; s++) v += Cb[((size_t)s * w + p * g.out + o) * jp + j];
    v *= scale;
    g.db[p][i] = accumulate ? g.db[p][i] + v : v;
}
// dA_p[j][i] (+)= scale * sum_s Ca[s][i][p * jp + j]: 16 columns i per workgroup, turned in LDS
__global__ void __launch_bounds__(256) lora_finish_a_kernel(LoraProducts g, const float *Ca, int parts, int jp, float scale, int accumulate) {
    __shared__ float tile[16][129];
    const int i0 = blockIdx.x * 16, n = g.n_p * jp, n4 = n / 4;
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

template <int RB, int NB>
int launch_thin(const ThinArgs &a, int groups, hipStream_t st) {
    const size_t ring = (size_t)3 * 16 * RB * (1024 + 16), sums = (size_t)4 * NB * RB * 1024, lds = ring > sums ? ring : sums;
    if (int rc = vla_allow_lds((const void *)lora_thin_kernel<RB, NB>, lds)) return rc;
    lora_thin_kernel<RB, NB><<<dim3(a.kp / (16 * RB), groups), 512, lds, st>>>(a);
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
// 32 rows of X per workgroup, 16 where that leaves CUs idle
int thin(const ThinArgs &a, int nb, int groups, hipStream_t st) {
    return with_blocks(nb, [&](auto n) {
        constexpr int NB = decltype(n)::value;
        return (a.M + 31) / 32 * groups >= 192 ? launch_thin<2, NB>(a, groups, st) : launch_thin<1, NB>(a, groups, st);
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
int rows_product(const RowsArgsT &a, int nb, int parts, hipStream_t st) {
    return with_blocks(nb, [&](auto n) {
        constexpr int NB = decltype(n)::value, IW = NB <= 4 ? 8 : 4;
        lora_rows_kernel<IW, NB><<<dim3(a.w / (16 * IW), parts), 256, 0, st>>>(a);
        return vla_check_launch("lora_rows");
    });
}

}  // namespace

// Returns 1 if handled, 0 if declined (more than 128 factor rows, widths that are no multiple of 128, unaligned operands), < 0 on
// a launch error.  scratch: 16-byte aligned, `bytes` of it; declines if that does not hold one part of each product.
int try_lora_products_bf16(const LoraProducts &g, const void *X, const void *dY, int M, float scale, bool accumulate, void *scratch, size_t bytes, hipStream_t st) {
    const int nj = (g.rank + 15) / 16, jp = nj * 16, wout = g.n_p * g.out, nb = g.n_p * nj, kp = (M + 31) / 32 * 32;
    if (M < 1 || g.rank < 1 || nb > 8 || g.in % 128 != 0 || g.out % 128 != 0 || ((size_t)X | (size_t)dY | (size_t)scratch) % 16 != 0) return 0;
    for (int p = 0; p < g.n_p; p++)
        if ((size_t)g.a[p] % 16 != 0) return 0;
    auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const size_t wu_bytes = up((size_t)nb * 16 * g.in * 2), wv_bytes = up((size_t)g.n_p * jp * g.out * 2), t_bytes = up((size_t)nb * 16 * kp * 2);
    const size_t used = wu_bytes + wv_bytes + 2 * t_bytes, row_b = (size_t)jp * 4, row_a = (size_t)nb * 64;
    if (bytes < used || bytes - used < wout * row_b || bytes - used < g.in * row_a) return 0;
    char *base = (char *)scratch;
    bf16_t *Wu = (bf16_t *)base, *Wv = (bf16_t *)(base + wu_bytes), *Ut = (bf16_t *)(base + wu_bytes + wv_bytes), *Vt = (bf16_t *)((char *)Ut + t_bytes);
    float *part = (float *)(base + used);
    const size_t left = bytes - used;
    ProfScope ps("lora_products", 8.0 * M * g.rank * ((double)g.n_p * g.in + wout), st);
    int rc;
    lora_pack_kernel<<<(nb * 2 * (g.in + g.out) + 255) / 256, 256, 0, st>>>(Wu, Wv, g, nj);          // (a piece of eight columns per thread)
    if ((rc = vla_check_launch("lora_pack"))) return rc;
    if ((rc = thin(ThinArgs{(const bf16_t *)X, Wu, Ut, M, g.in, g.in, kp, 0}, nb, 1, st))) return rc;
    if ((rc = thin(ThinArgs{(const bf16_t *)dY, Wv, Vt, M, g.out, wout, kp, g.out}, nj, g.n_p, st))) return rc;
    const int pb = parts_of(wout, nj <= 4 ? 8 : 4, M, row_b, left), pa = parts_of(g.in, nb <= 4 ? 8 : 4, M, row_a, left);
    if ((rc = rows_product(RowsArgsT{(const bf16_t *)dY, Ut, part, M, wout, kp, g.out}, nj, pb, st))) return rc;
    lora_finish_b_kernel<<<dim3((g.out * g.rank + 255) / 256, g.n_p), 256, 0, st>>>(g, part, pb, jp, scale, accumulate);
    if ((rc = vla_check_launch("lora_finish_b"))) return rc;
    if ((rc = rows_product(RowsArgsT{(const bf16_t *)X, Vt, part, M, g.in, kp, g.in}, nb, pa, st))) return rc;
    lora_finish_a_kernel<<<g.in / 16, 256, 0, st>>>(g, part, pa, jp, scale, accumulate);
    rc = vla_check_launch("lora_finish_a");
    return rc ? rc : 1;
}
