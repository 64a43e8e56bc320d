// Attention of the gradient pass, whose probabilities and score gradients stay in memory for the products that contract over the
// queries (dV = P^T dO, dK = dS^T q).  One kernel per direction takes 64 query rows of a (sequence, head), all their keys:
//   forward   S = q k^T / sqrt(d), P = softmax(S) under the mask (written), out = P v
//   backward  dP = dO v^T, dS = P (dP - rowsum(P dP)) (written), dq = dS k / sqrt(d)
// The score rows live in LDS between the three steps, so of the [rows x keys] fp32 matrices only P (forward: one write; backward:
// one read, and one write of dS) touches memory; as batched products with a pass in between they were moved four and six times.
// What bounds it is the chain of a workgroup's three steps with two workgroups (of four waves) on a CU.  294 rows, 32 x 32 heads of 128:
// forward 404 -> 239 us (0.6 GB: 120 us), backward 480 -> 299 (1.1 GB: 220); 283 rows, 7 x 32 heads: 98 -> 61 and 110 -> 73.  A wave per 16
// rows over all keys in the last step took 258 and 326.  An fp32 operand enters the matrix cores as bf16 head + tail, as in bgemm_mfma_kernel; sums are fp32 in a
// fixed order.
#include "vla_internal.h"

namespace {

constexpr int HD = 128, BQ = 64, NV = 5;         // head_dim; query rows per workgroup; 64-key pieces of a row

__device__ __forceinline__ void split_bf16(const f32x4_t &a, const f32x4_t &b, bf16x8_t &hi, bf16x8_t &lo) {
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const float v = e < 4 ? a[e & 3] : b[e & 3];
        hi[e] = (bf16_t)v;
        lo[e] = (bf16_t)(v - (float)hi[e]);
    }
}
// Sum or maximum over the 16 lanes that share a row.
template <bool MAX>
__device__ __forceinline__ float reduce16(float v) {
    if constexpr (MAX) return vla_row_fold(v, VlaMax{});
    else return vla_row_fold(v, VlaAdd{});
}

__device__ __forceinline__ f32x4_t pick(bool c, f32x4_t a, f32x4_t b) {
    f32x4_t v;
#pragma unroll
    for (int e = 0; e < 4; e++) v[e] = c ? a[e] : b[e];
    return v;
}

template <bool BWD>
__global__ void __launch_bounds__(256, 2) attn_rows_kernel(AttnRowsArgs a, int n_heads_total, int tiles, int ld) {
    extern __shared__ __attribute__((aligned(16))) float S[];       // [BQ][ld]; ld / 4 odd: rows 16 bytes apart in the banks
    // the tiles of a (sequence, head) share its keys: on one XCD, the one with the most visible keys first
    const int group = blockIdx.x / (8 * tiles), in_group = blockIdx.x - group * 8 * tiles;
    const int head_id = group * 8 + (in_group & 7), tile = tiles - 1 - (in_group >> 3);
    if (head_id >= n_heads_total) return;
    const int s = head_id / a.n_heads, h = head_id - s * a.n_heads, H3 = 3 * a.H;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
    const int R = a.R, Rq = a.Rq, q0 = tile * BQ, first = R - Rq;       // row r of the queries sits at position first + r
    const bf16_t *kv = a.qkv + (size_t)s * R * H3 + h * HD;
    auto keys_of = [&](int row) { const int i = first + min(row, Rq - 1); return i >= a.full_from ? R : i + 1; };

    // ---- the rows' products with k (forward) or v (backward): wave w takes the key blocks w, w + 4, ..
    {
        const int nb = (min(BQ, Rq - q0) + 15) / 16, key_blocks = (keys_of(q0 + BQ - 1) + 15) / 16;
        bf16x8_t qh[4][4], ql[4][4];
#pragma unroll
        for (int b = 0; b < 4; b++) {
            const int row = min(q0 + b * 16 + l16, Rq - 1);
#pragma unroll
            for (int c = 0; c < 4; c++) {
                if (BWD) {
                    const float *p = (const float *)a.rows + ((size_t)s * Rq + row) * a.H + h * HD + c * 32 + kq * 8;
                    split_bf16(*(const f32x4_t *)p, *(const f32x4_t *)(p + 4), qh[b][c], ql[b][c]);
                } else qh[b][c] = *(const bf16x8_t *)((const bf16_t *)a.rows + ((size_t)s * R + first + row) * H3 + h * HD + c * 32 + kq * 8);
            }
        }
        const bf16_t *src = kv + (BWD ? 2 : 1) * a.H + kq * 8;
        bf16x8_t kf[2][4];
        auto load = [&](int st, int kb) {
            const bf16_t *p = src + (size_t)min(kb * 16 + l16, R - 1) * H3;
#pragma unroll
            for (int c = 0; c < 4; c++) kf[st][c] = *(const bf16x8_t *)(p + c * 32);
        };
        auto multiply = [&](int st, int kb) {
            f32x4_t acc[4];
#pragma unroll
            for (int b = 0; b < 4; b++) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 4; c++)
#pragma unroll
                for (int b = 0; b < 4; b++)
                    if (b < nb) {
                        if (BWD) acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[st][c], ql[b][c], acc[b], 0, 0, 0);
                        acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[st][c], qh[b][c], acc[b], 0, 0, 0);
                    }
            // a lane: keys 4 kq .. + 3 of the block, query l16
            const int col = kb * 16 + 4 * kq;
            if (col < ld)
#pragma unroll
                for (int b = 0; b < 4; b++)
                    if (b < nb) *(f32x4_t *)(S + (b * 16 + l16) * ld + col) = BWD ? acc[b] : acc[b] * a.scale;
        };
        if (wave < key_blocks) load(0, wave);
        for (int kb = wave; kb < key_blocks; kb += 8) {
            if (kb + 4 < key_blocks) load(1, kb + 4);
            multiply(0, kb);
            if (kb + 8 < key_blocks) load(0, kb + 8);
            if (kb + 4 < key_blocks) multiply(1, kb + 4);
        }
    }
    __syncthreads();

    // ---- the last step's first v (k) rows leave ahead of the softmax.  There a wave sums 32 rows over every other 32 keys: a quarter of
    // the loads and register turns that 16 rows over all keys would take per workgroup, in half as many steps one after the other
    const int pair = wave >> 1, odd = wave & 1, w0 = q0 + wave * 16;
    const int steps = q0 + pair * 32 < Rq ? (keys_of(q0 + pair * 32 + 31) + 31) / 32 : 0, wave_keys = keys_of(w0 + 15);
    const bf16_t *src = kv + (BWD ? 1 : 2) * a.H + 8 * l16;
    i32x4_v y[2][8];
    auto load = [&](int st, int step) {
#pragma unroll
        for (int t = 0; t < 8; t++) {
            const int key = step * 32 + 8 * kq + t;
            y[st][t] = key < R ? *(const i32x4_v *)(src + (size_t)key * H3) : i32x4_v{0, 0, 0, 0};
        }
    };
    if (odd < steps) load(0, odd);

    // ---- softmax, or its backward: 16 lanes per row, four rows at a time
    f32x4_t pr[2][NV];
    auto load_p = [&](int st, int it) {
        if (BWD) {
            const int row = min(w0 + it * 4 + kq, Rq - 1), nk = keys_of(row);
            const float *p = a.P + ((size_t)head_id * Rq + row) * a.ldp;
#pragma unroll
            for (int u = 0; u < NV; u++) {
                const int c = u * 64 + l16 * 4;
                pr[st][u] = c < nk ? *(const f32x4_t *)(p + c) : f32x4_t{0.f, 0.f, 0.f, 0.f};       // (rows end on 16 bytes)
            }
        }
    };
    load_p(0, 0);
#pragma unroll
    for (int it = 0; it < 4; it++) {
        if (w0 >= Rq) break;
        if (it < 3) load_p((it + 1) & 1, it + 1);
        const int row = w0 + it * 4 + kq, nk = keys_of(row);
        float *sr = S + (size_t)(wave * 16 + it * 4 + kq) * ld;
        f32x4_t v[NV];
        float m = -INFINITY, sum = 0.f;
#pragma unroll
        for (int u = 0; u < NV; u++) {
            const int c = u * 64 + l16 * 4;
            v[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (u * 64 >= wave_keys) continue;           // (the vector unit's time counts: half of a causal matrix is masked)
            if (c < ld) v[u] = *(const f32x4_t *)(sr + c);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                if (BWD) sum += c + e < nk ? pr[it & 1][u][e] * v[u][e] : 0.f;
                else m = fmaxf(m, c + e < nk ? v[u][e] : -INFINITY);
            }
        }
        if (!BWD) {
            m = reduce16<true>(m);
#pragma unroll
            for (int u = 0; u < NV; u++) {
                if (u * 64 >= wave_keys) continue;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    v[u][e] = u * 64 + l16 * 4 + e < nk ? expf(v[u][e] - m) : 0.f;
                    sum += v[u][e];
                }
            }
        }
        sum = reduce16<false>(sum);
        const float inv = BWD ? 0.f : 1.0f / sum;
        float *out = a.S + ((size_t)head_id * Rq + row) * a.ldp;
#pragma unroll
        for (int u = 0; u < NV; u++) {
            const int c = u * 64 + l16 * 4;
            f32x4_t o = v[u];                            // (zeros past the wave's keys)
            if (u * 64 < wave_keys)
#pragma unroll
                for (int e = 0; e < 4; e++) o[e] = BWD ? (c + e < nk ? pr[it & 1][u][e] * (v[u][e] - sum) : 0.f) : v[u][e] * inv;
            if (c < ld) *(f32x4_t *)(sr + c) = o;
            if (c < a.ldp && row < Rq) *(f32x4_t *)(out + c) = o;
        }
    }

    // ---- the rows' sums over v (k): a lane reads eight neighbouring dims of eight keys, whole 256-byte rows among 16 lanes, and
    // turns them in its registers into eight operands of eight keys; operand e holds the dims 8 l + e (l = 0 .. 15)
    __syncthreads();
    f32x4_t acc[2][8];
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
        for (int e = 0; e < 8; e++) acc[b][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const float *pr_row = S + (size_t)(pair * 32 + l16) * ld;
    auto multiply = [&](int st, int step) {
        const int c = step * 32 + 8 * kq;
        bf16x8_t hi[2], lo[2];
#pragma unroll
        for (int b = 0; b < 2; b++) {
            f32x4_t p0 = f32x4_t{0.f, 0.f, 0.f, 0.f}, p1 = p0;
            if (c < ld) p0 = *(const f32x4_t *)(pr_row + b * 16 * ld + c);
            if (c + 4 < ld) p1 = *(const f32x4_t *)(pr_row + b * 16 * ld + c + 4);
            split_bf16(p0, p1, hi[b], lo[b]);
        }
#pragma unroll
        for (int e = 0; e < 8; e++) {
            i32x4_v f;
#pragma unroll
            for (int q = 0; q < 4; q++)
                f[q] = (int)__builtin_amdgcn_perm((unsigned)y[st][2 * q + 1][e / 2], (unsigned)y[st][2 * q][e / 2], e & 1 ? 0x07060302u : 0x05040100u);
#pragma unroll
            for (int b = 0; b < 2; b++) {
                acc[b][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f), lo[b], acc[b][e], 0, 0, 0);
                acc[b][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f), hi[b], acc[b][e], 0, 0, 0);
            }
        }
    };
    for (int step = odd; step < steps; step += 4) {
        if (step + 2 < steps) load(1, step + 2);
        multiply(0, step);
        if (step + 4 < steps) load(0, step + 4);
        if (step + 2 < steps) multiply(1, step + 2);
    }
    // the pair's waves exchange a block of 16 rows each
    __syncthreads();
    f32x4_t *part = (f32x4_t *)S + lane;
#pragma unroll
    for (int e = 0; e < 8; e++) part[(wave * 8 + e) * 64] = pick(odd, acc[0][e], acc[1][e]);
    __syncthreads();
    f32x4_t sum8[8];
#pragma unroll
    for (int e = 0; e < 8; e++) sum8[e] = pick(odd, acc[1][e], acc[0][e]) + part[((wave ^ 1) * 8 + e) * 64];
    // a lane: row l16, dims 8 (4 kq + r) + e
    const int row = w0 + l16;
    if (row >= Rq) return;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const int d0 = 8 * (4 * kq + r);
        if (BWD) {
            float *o = (float *)a.out + ((size_t)s * R + first + row) * H3 + h * HD + d0;
            f32x4_t lo, hi;
#pragma unroll
            for (int e = 0; e < 4; e++) { lo[e] = sum8[e][r] * a.scale; hi[e] = sum8[4 + e][r] * a.scale; }
            *(f32x4_t *)o = lo;
            *(f32x4_t *)(o + 4) = hi;
        } else {
            bf16x8_t v;
#pragma unroll
            for (int e = 0; e < 8; e++) v[e] = (bf16_t)sum8[e][r];
            *(bf16x8_t *)((bf16_t *)a.out + ((size_t)s * Rq + row) * a.H + h * HD + d0) = v;
        }
    }
}

// dV = P^T dO and dK = dS^T q / sqrt(d), the contractions over the queries, and the transposed rotation with the rounding of all three
// gradients: bf16 d q | d k | d v rows from P, d S, d O and the fp32 d q.  A wave takes 32 keys of a (sequence, head) and either d V or,
// with the 32 rows of d q, d K; it walks the queries that see its keys, 32 at a time.  A lane loads eight queries x two keys of P (d S) and
// eight queries x four neighbouring dims of d O (q), twice: the eight values of a key or a dim are then an operand's eight elements
// as they lie in the registers (q's 16-bit values after one byte permutation a pair).  Dims i and i + 64 of a pair end in one lane.
// Splits as everywhere here: P, d S, d O as bf16 head + tail, their products but tail x tail.
// Bound by memory (P and d S once, at 294 rows little more than their lower halves): as two batched products with fp32 outputs and a pass
// over all of q | k | v for the rotation, 294 rows of 32 x 32 heads took 607 us, now 319; 283 rows of 7 x 32 heads 153, now 65; the top layer's seven queries of 294 204 -> 97.
template <bool KEY>
__device__ __forceinline__ void attn_cols(const AttnColsArgs &a, int s, int h, int kw0) {
    const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
    const int R = a.R, Rq = a.Rq, first = R - Rq, head_id = s * a.n_heads + h, H3 = 3 * a.H;
    const int key = kw0 + 2 * l16;                                        // this lane's keys: key, key + 1
    const float *P = (KEY ? a.dS : a.P) + (size_t)head_id * Rq * a.ldp + key;
    const float *d_o = a.dO + (size_t)s * Rq * a.H + h * HD + 4 * l16;
    const bf16_t *q = a.qkv + ((size_t)s * R + first) * H3 + h * HD + 4 * l16;
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef int i32x2_t __attribute__((ext_vector_type(2)));
    f32x2_t p[8];
    f32x4_t dv[KEY ? 1 : 2][8];
    i32x2_t qv[KEY ? 2 : 1][8];
    auto load_p = [&](int q0) {
#pragma unroll
        for (int t = 0; t < 8; t++) {
            const int row = q0 + 8 * kq + t;
            p[t] = f32x2_t{0.f, 0.f};
            if (row < Rq && key < a.ldp) p[t] = *(const f32x2_t *)(P + (size_t)row * a.ldp);
        }
    };
    auto load_d = [&](int half, int q0) {                // (rows past the last: that one's, their P is zero)
#pragma unroll
        for (int t = 0; t < 8; t++) {
            const size_t row = min(q0 + 8 * kq + t, Rq - 1);
            if (KEY) qv[KEY ? half : 0][t] = *(const i32x2_t *)(q + row * H3 + 64 * half);
            else dv[KEY ? 0 : half][t] = *(const f32x4_t *)(d_o + row * a.H + 64 * half);
        }
    };
    f32x4_t acc[2][8];
#pragma unroll
    for (int e = 0; e < 2; e++)
#pragma unroll
        for (int f = 0; f < 8; f++) acc[e][f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    bf16x8_t ph[2], pl[2];
    auto multiply = [&](int half) {
#pragma unroll
        for (int f = 0; f < 4; f++) {
            bf16x8_t hi, lo;
            if (KEY) {
                i32x4_v w;
#pragma unroll
                for (int u = 0; u < 4; u++)
                    w[u] = (int)__builtin_amdgcn_perm((unsigned)qv[KEY ? half : 0][2 * u + 1][f / 2], (unsigned)qv[KEY ? half : 0][2 * u][f / 2], f & 1 ? 0x07060302u : 0x05040100u);
                hi = __builtin_bit_cast(bf16x8_t, w);
            } else {
#pragma unroll
                for (int t = 0; t < 8; t++) {
                    const float v = dv[KEY ? 0 : half][t][f];
                    hi[t] = (bf16_t)v;
                    lo[t] = (bf16_t)(v - (float)hi[t]);
                }
            }
#pragma unroll
            for (int e = 0; e < 2; e++) {
                f32x4_t &c = acc[e][4 * half + f];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, pl[e], c, 0, 0, 0);
                if (!KEY) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, ph[e], c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, ph[e], c, 0, 0, 0);
            }
        }
    };
    const int q_begin = max(0, min(kw0, a.full_from) - first);           // the first query that sees one of the wave's keys
    load_p(q_begin);
    load_d(0, q_begin);
    for (int q0 = q_begin; q0 < Rq; q0 += 32) {
        load_d(1, q0);
#pragma unroll
        for (int e = 0; e < 2; e++)
#pragma unroll
            for (int t = 0; t < 8; t++) {
                ph[e][t] = (bf16_t)p[t][e];
                pl[e][t] = (bf16_t)(p[t][e] - (float)ph[e][t]);
            }
        load_p(q0 + 32);
        multiply(0);
        load_d(0, q0 + 32);
        multiply(1);
    }
    // ---- a lane: keys key + e, dims 16 kq + 4 r + f and those + 64
#pragma unroll
    for (int e = 0; e < 2; e++) {
        if (key + e >= R) break;
        bf16x8_t lo[2], hi[2];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            f32x4_t cs[2] = {};
            if (KEY) {
                const f32x4_t *tb = (const f32x4_t *)(a.table + (size_t)(key + e) * (HD / 2) + 16 * kq + 4 * r);
                cs[0] = tb[0];
                cs[1] = tb[1];
            }
#pragma unroll
            for (int f = 0; f < 4; f++) {
                const float x = acc[e][f][r], y = acc[e][4 + f][r], co = cs[f >> 1][2 * (f & 1)], si = -cs[f >> 1][2 * (f & 1) + 1];
                lo[r >> 1][4 * (r & 1) + f] = (bf16_t)(KEY ? vla_rotate_lo(x * a.scale, y * a.scale, co, si) : x);
                hi[r >> 1][4 * (r & 1) + f] = (bf16_t)(KEY ? vla_rotate_hi(x * a.scale, y * a.scale, co, si) : y);
            }
        }
        bf16_t *o = a.out_k + ((size_t)s * R + key + e) * a.ld_kv + (KEY ? 0 : a.H) + h * HD + 16 * kq;
        *(bf16x8_t *)o = lo[0];
        *(bf16x8_t *)(o + 8) = lo[1];
        *(bf16x8_t *)(o + 64) = hi[0];
        *(bf16x8_t *)(o + 72) = hi[1];
    }
    if (!KEY) return;
    // ---- the same rows of d q (none below the first query: nothing is read there, and zeros written unless d q is packed)
#pragma unroll
    for (int it = 0; it < 8; it++) {
        const int row = kw0 + it * 4 + kq;
        if (row >= R) break;
        if (a.q_packed && row < first) continue;
        bf16x4_t lo, hi;
        if (row >= first) {
            const float *x = a.dq + ((size_t)s * R + row) * H3 + h * HD + 4 * l16;
            const f32x4_t x0 = *(const f32x4_t *)x, x1 = *(const f32x4_t *)(x + 64);
            const f32x4_t *tb = (const f32x4_t *)(a.table + (size_t)row * (HD / 2) + 4 * l16);
            const f32x4_t cs[2] = {tb[0], tb[1]};
#pragma unroll
            for (int f = 0; f < 4; f++) {
                const float co = cs[f >> 1][2 * (f & 1)], si = -cs[f >> 1][2 * (f & 1) + 1];
                lo[f] = (bf16_t)vla_rotate_lo(x0[f], x1[f], co, si);
                hi[f] = (bf16_t)vla_rotate_hi(x0[f], x1[f], co, si);
            }
        } else {
#pragma unroll
            for (int f = 0; f < 4; f++) lo[f] = hi[f] = (bf16_t)0.f;
        }
        bf16_t *o = a.out_q + (a.q_packed ? (size_t)s * Rq + row - first : (size_t)s * R + row) * a.ld_q + h * HD + 4 * l16;
        *(bf16x4_t *)o = lo;
        *(bf16x4_t *)(o + 64) = hi;
    }
}
__global__ void __launch_bounds__(256, 2) attn_cols_kernel(AttnColsArgs a, int n_heads_total, int tiles) {
    // both products of all tiles of a (sequence, head) on one XCD, the tiles with the most queries first
    const int items = 2 * tiles, group = blockIdx.x / (8 * items), in_group = blockIdx.x - group * 8 * items;
    const int head_id = group * 8 + (in_group & 7), item = in_group >> 3;
    const int kw0 = (item >> 1) * 128 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 32;
    if (head_id >= n_heads_total || kw0 >= a.R) return;
    const int s = head_id / a.n_heads, h = head_id - s * a.n_heads;
    if (item & 1) attn_cols<true>(a, s, h, kw0);
    else attn_cols<false>(a, s, h, kw0);
}

}  // namespace

// head_dim 128; any number of rows; arrays on 16 bytes.
bool attention_cols_takes(const AttnColsArgs &a) {
    if (a.H != a.n_heads * HD || a.ldp % 4 != 0 || a.ldp < a.R) return false;
    if (((size_t)a.P | (size_t)a.dS | (size_t)a.dO | (size_t)a.dq | (size_t)a.qkv | (size_t)a.table | (size_t)a.out_q | (size_t)a.out_k) % 16 != 0) return false;
    return a.ld_q % 8 == 0 && a.ld_kv % 8 == 0;
}

// Returns 1 if handled, 0 if declined, < 0 on a launch error.
int try_attention_cols(const AttnColsArgs &a, int n_seq, hipStream_t st) {
    if (!attention_cols_takes(a)) return 0;
    const int heads = n_seq * a.n_heads, tiles = (a.R + 127) / 128;
    ProfScope ps("bw_attention_cols", 4.0 * heads * a.Rq * (double)a.R * HD * (a.Rq == a.R ? 0.5 : 1.0), st);
    attn_cols_kernel<<<(heads + 7) / 8 * 8 * 2 * tiles, 256, 0, st>>>(a, heads, tiles);
    const int rc = vla_check_launch("attn_cols");
    return rc ? rc : 1;
}

// Returns 1 if handled, 0 if declined, < 0 on a launch error.  head_dim 128 and up to 316 keys: then two workgroups of 64 rows share
// a CU's LDS.
template <bool BWD>
static int try_rows(const AttnRowsArgs &a, int n_seq, hipStream_t st) {
    int ld = (a.R + 3) & ~3;
    if (ld % 8 == 0) ld += 4;
    const size_t rows = (size_t)BQ * ld * sizeof(float), sums = (size_t)BQ * HD * sizeof(float), lds = rows > sums ? rows : sums;
    if (a.H != a.n_heads * HD || ld > 64 * NV || 2 * lds > 160 * 1024 || a.ldp % 4 != 0 || a.ldp < a.R) return 0;
    if (((size_t)a.rows | (size_t)a.qkv | (size_t)a.S | (size_t)a.P | (size_t)a.out) % 16 != 0) return 0;
    const int heads = n_seq * a.n_heads, tiles = (a.Rq + BQ - 1) / BQ;
    ProfScope ps("bw_attention_rows", 8.0 * heads * a.Rq * (double)a.R * HD * (a.Rq == a.R ? 0.5 : 1.0), st);
    if (int rc = vla_allow_lds((const void *)attn_rows_kernel<BWD>, lds)) return rc;
    attn_rows_kernel<BWD><<<(heads + 7) / 8 * 8 * tiles, 256, lds, st>>>(a, heads, tiles, ld);
    const int rc = vla_check_launch("attn_rows");
    return rc ? rc : 1;
}
int try_attention_rows_forward(const AttnRowsArgs &a, int n_seq, hipStream_t st) { return try_rows<false>(a, n_seq, st); }
int try_attention_rows_backward(const AttnRowsArgs &a, int n_seq, hipStream_t st) { return try_rows<true>(a, n_seq, st); }
