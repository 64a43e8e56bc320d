// Single-query attention for the autoregressive decode steps (bf16 KV cache, head_dim 64 or 128).
//
// The step is pure HBM streaming: every (environment, head) pair reads its own K and V tiles once
// (multi-head attention, no query sharing).  One workgroup of four waves owns one pair (the keys are
// split over the waves so that small batches still put enough loads in flight):
//   1. scores: a lane owns one key position per 64-key chunk; K is stored [d/8][position][8], so one load
//      instruction of the wave reads 64 consecutive positions x 16 bytes = 1 KB contiguous and no
//      cross-lane reduction is needed for q.k (q is broadcast from LDS, pre-scaled by 1/sqrt(d));
//   2. softmax over all keys with two wave reductions (scores stay in registers: <= 512 keys);
//   3. P.V: V is stored [position][d]; 8 (d = 64) or 16 (d = 128) lanes cover one V row with 16-byte
//      loads, the wave covers 8 / 4 rows per instruction (1 KB contiguous), probabilities come from
//      LDS, and the row groups are summed by lane-xor steps and a four-way add through LDS.
// Of few pairs each gets eight waves (see FEW_PAIRS), half the V columns per lane.
// NT: K and V, whole lines per instruction and used once a step, carry the non-temporal hint: 2048 pairs of 290 keys of 4 layers 64.8 -> 54.6 us
// (5.6 TB/s), 8192 pairs 224 -> 206 (5.9).  The caller's to choose: K and V that fit the memory-side cache are better left to it.
#include "vla_internal.h"

#include <type_traits>

namespace {

constexpr int MAXCH = 8;   // key chunks of 64 held in registers => at most 512 keys

// What the projection left for this step (FUSE): the fp32 [n_seq, 3H] QKV rows.
struct FusedQkv {
    const float *qkv;
    const float2 *table;       // (cos, sin) of this position
};

// One workgroup of NWV waves (4 or 8) per (sequence, head) pair; the waves split the keys.  FUSE: the workgroup also
// rotates its head's q and k and writes k and v to the cache (the rounding of rope_kv_write_bf16_kernel); the new
// position's k and v are then taken from LDS.
// All forms give the same bits, so that a sequence's result does not depend on how many share the step: a score is one
// chain over the dims; the softmax's sum adds key chunks w and w + 4 lane by lane, then the lanes, then w = 0..3; P.V has
// one chain for every 4 * (512 / D) th position (eight waves hold the same chains with half the columns per lane) and a
// fixed tree over the chains.
template <int D, int NWV, bool FUSE, bool NT>
__global__ void __launch_bounds__(64 * NWV) attn_decode_kernel(bf16_t *out, const bf16_t *qbuf, bf16_t *kc, bf16_t *vc, FusedQkv f,
                                                              int n_heads, int nk, int pos_stride, int H) {
    static_assert(NWV == 4 || (NWV == 8 && MAXCH == 8), "the order of the sums");
    constexpr int DC = D / 8;        // 16-byte chunks per head vector
    constexpr int VPL = 32 / NWV;    // V columns per lane
    constexpr int LPR = D / VPL;     // lanes per V row
    constexpr int RPI = 64 / LPR;    // V rows per wave load instruction
    typedef bf16_t bf16v __attribute__((ext_vector_type(VPL)));
    constexpr int CPW = MAXCH / NWV; // key chunks of 64 per wave (chunk index = NWV * it + wave)
    __shared__ __attribute__((aligned(16))) float qs[D];
    __shared__ __attribute__((aligned(16))) bf16_t knew[D], vnew[D];
    __shared__ float ps[MAXCH * 64];
    __shared__ float red[2 * NWV];
    __shared__ __attribute__((aligned(16))) float part[NWV][D];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int item = blockIdx.x;
    const int s = item / n_heads, h = item - s * n_heads;
    const float scale = 1.0f / sqrtf((float)D);
    bf16_t *kh = kc + (size_t)item * D * pos_stride;
    bf16_t *vh = vc + (size_t)item * pos_stride * D;
    const int n_old = FUSE ? nk - 1 : nk;                   // positions read from the cache
    if (FUSE) {
        float *raw = &part[0][0];                           // q, k of the head before the rotation (D floats each)
        float v = 0.f;
        if (t < D) {
            const float *src = f.qkv + (size_t)s * 3 * H + (size_t)h * D + t;
            raw[t] = src[0]; raw[D + t] = src[H];
            v = src[2 * (size_t)H];
        }
        __syncthreads();
        if (t < D) {
            const int half = D / 2, i = t & (half - 1);
            const float2 cs = f.table[i];
            const float qa = raw[i], qb = raw[i + half], ka = raw[D + i], kb = raw[D + i + half];
            const bf16_t qr = (bf16_t)(t < half ? vla_rotate_lo(qa, qb, cs.x, cs.y) : vla_rotate_hi(qa, qb, cs.x, cs.y));
            const bf16_t kr = (bf16_t)(t < half ? vla_rotate_lo(ka, kb, cs.x, cs.y) : vla_rotate_hi(ka, kb, cs.x, cs.y));
            qs[t] = (float)qr * scale;
            knew[t] = kr; vnew[t] = (bf16_t)v;
            kh[((size_t)(t >> 3) * pos_stride + nk - 1) * 8 + (t & 7)] = kr;
            vh[(size_t)(nk - 1) * D + t] = (bf16_t)v;
        }
    } else if (t < D) {
        qs[t] = (float)qbuf[(size_t)s * H + (size_t)h * D + t] * scale;
    }
    __syncthreads();

    // ---- 1. scores: wave w owns key chunks w, w + NWV, ...; lane p one position of each --------------
    float sc[CPW];
    float mx = -INFINITY;
#pragma unroll
    for (int it = 0; it < CPW; it++) {
        sc[it] = -INFINITY;
        const int p = (it * NWV + wave) * 64 + lane;
        if (p < nk) {
            bf16x8_t kv[DC];
            if (!FUSE || p < n_old) {
#pragma unroll
                for (int c = 0; c < DC; c++) {
                    const i32x4_v *src = (const i32x4_v *)(kh + ((size_t)c * pos_stride + p) * 8);
                    kv[c] = __builtin_bit_cast(bf16x8_t, NT ? __builtin_nontemporal_load(src) : *src);
                }
            } else {
#pragma unroll
                for (int c = 0; c < DC; c++) kv[c] = *(const bf16x8_t *)&knew[c * 8];
            }
            float a = 0.f;
#pragma unroll
            for (int c = 0; c < DC; c++) {
                f32x4_t q0 = *(const f32x4_t *)&qs[c * 8];
                f32x4_t q1 = *(const f32x4_t *)&qs[c * 8 + 4];
#pragma unroll
                for (int e = 0; e < 4; e++) a += q0[e] * (float)kv[c][e];
#pragma unroll
                for (int e = 0; e < 4; e++) a += q1[e] * (float)kv[c][4 + e];
            }
            sc[it] = a;
            mx = fmaxf(mx, a);
        }
    }
    // ---- 2. softmax over all keys of the workgroup ---------------------------------------------------
    mx = vla_wave_max(mx);
    if (lane == 0) red[wave] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NWV; w++) mx = fmaxf(mx, red[w]);          // key 0 exists, so this is finite
    float sum = 0.f;
#pragma unroll
    for (int it = 0; it < CPW; it++) {
        const float e = __expf(sc[it] - mx);                       // exp(-inf) = 0 for positions >= nk
        sc[it] = e;
        sum += e;
        if (NWV == 8) ps[(it * NWV + wave) * 64 + lane] = e;
    }
    if (NWV == 8) {
        __syncthreads();
        sum = ps[(wave & 3) * 64 + lane] + ps[((wave & 3) + 4) * 64 + lane];
    }
    sum = vla_wave_sum(sum);
    if (lane == 0) red[NWV + wave] = sum;                          // (of eight waves, 4..7 repeat 0..3)
    __syncthreads();
    float tot = red[NWV];
#pragma unroll
    for (int w = 1; w < 4; w++) tot += red[NWV + w];
    const float inv = 1.0f / tot;
    if (NWV == 4) {
#pragma unroll
        for (int it = 0; it < CPW; it++) {
            const int p = (it * NWV + wave) * 64 + lane;
            if (p < nk) ps[p] = sc[it] * inv;
        }
        __syncthreads();
    }

    // ---- 3. P.V: the workgroup covers NWV * RPI rows per step, wave w rows w * RPI + g ------------------
    const int c = lane % LPR, g = lane / LPR, slot = wave * RPI + g;
    auto probability = [&](int pos) { return NWV == 4 ? ps[pos] : ps[pos] * inv; };
    float acc[VPL] = {};
#pragma unroll 4
    for (int pos = slot; pos < n_old; pos += NWV * RPI) {
        const bf16v *src = (const bf16v *)(vh + (size_t)pos * D + c * VPL);
        const bf16v v = NT ? __builtin_nontemporal_load(src) : *src;
        const float pr = probability(pos);
#pragma unroll
        for (int e = 0; e < VPL; e++) acc[e] += pr * (float)v[e];
    }
    if (FUSE && n_old % (NWV * RPI) == slot) {
        const bf16v v = *(const bf16v *)&vnew[c * VPL];
        const float pr = probability(n_old);
#pragma unroll
        for (int e = 0; e < VPL; e++) acc[e] += pr * (float)v[e];
    }
#pragma unroll
    for (int e = 0; e < VPL; e++) {
        if constexpr (LPR <= 8) acc[e] = vla_fold_step<8>(acc[e], VlaAdd{});
        if constexpr (LPR <= 16) acc[e] = vla_fold_step<16>(acc[e], VlaAdd{});
        acc[e] = vla_fold_step<32>(acc[e], VlaAdd{});
    }
    if (lane < LPR) {
#pragma unroll
        for (int e = 0; e < VPL; e++) part[wave][c * VPL + e] = acc[e];
    }
    __syncthreads();
    if (t < DC) {
        bf16x8_t o;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int i = t * 8 + e;
            float v[NWV];
#pragma unroll
            for (int w = 0; w < NWV; w++) v[w] = part[w][i];
#pragma unroll
            for (int st = 1; st < NWV; st *= 2)
#pragma unroll
                for (int w = 0; w + st < NWV; w += 2 * st) v[w] += v[w + st];
            o[e] = (bf16_t)v[0];
        }
        *(bf16x8_t *)(out + (size_t)s * H + (size_t)h * D + t * 8) = o;
    }
}

// Few pairs: eight waves each, with the projection's sum, rotation and KV write on board.  The step of one environment (32
// pairs, 290 keys) is a chain of launches and memory latencies: 14.5 us with four waves and 9.5 in the kernel before, 8.6 us
// now; 13 environments 17.4 + 9.5 -> 18 us.  From FEW_PAIRS on the chip is full with four waves, and the extra
// latency ahead of the first key costs more than the launch (2048 pairs 62 + 5 against 74 us, 8192 225 + 13 against 271).
constexpr int FEW_PAIRS = 1024;

// f(integral_constant head_dim, bool_constant NT)
template <typename F>
void with_form(int d, bool past_caches, F f) {
    auto width = [&](auto nt) {
        if (d == 128) f(std::integral_constant<int, 128>{}, nt);
        else f(std::integral_constant<int, 64>{}, nt);
    };
    if (past_caches) width(std::true_type{});
    else width(std::false_type{});
}

}  // namespace

static bool decode_shape_ok(const KvView &kv, const RowsArgs &ra) {
    return ra.R == 1 && ra.pos0 + 1 <= MAXCH * 64 && (kv.d == 64 || kv.d == 128);
}

int try_attention_decode_bf16(bf16_t *out, const bf16_t *q, const KvView &kv, int layer, const RowsArgs &ra,
                              int H, bool past_caches, hipStream_t st) {
    if (!decode_shape_ok(kv, ra)) return 0;
    const int nk = ra.pos0 + 1, n_items = ra.n_seq * kv.n_heads;
    if (n_items == 0) return 1;
    bf16_t *kc = (bf16_t *)kv.k + (size_t)layer * kv.layer_elems, *vc = (bf16_t *)kv.v + (size_t)layer * kv.layer_elems;
    // algorithmic bytes: K and V tiles of every (sequence, head) pair, read once
    ProfScope ps("attn_decode", 2.0 * n_items * (double)nk * kv.d * 2.0, st);
    with_form(kv.d, past_caches, [&](auto dim, auto nt) {
        attn_decode_kernel<decltype(dim)::value, 4, false, decltype(nt)::value><<<n_items, 256, 0, st>>>(out, q, kc, vc, FusedQkv{}, kv.n_heads, nk, kv.pos_stride, H);
    });
    int rc = vla_check_launch("attn_decode");
    return rc ? rc : 1;
}

bool attention_decode_fuses_qkv(const KvView &kv, const RowsArgs &ra) {
    return decode_shape_ok(kv, ra) && ra.n_seq * kv.n_heads < FEW_PAIRS;
}

// The decode step's attention straight from the QKV projection, fp32 [n_seq, 3H] rows.  Only where
// attention_decode_fuses_qkv().
int launch_attention_decode_qkv(bf16_t *out, const float *qkv, const float2 *table, const KvView &kv, int layer, const RowsArgs &ra,
                                int H, bool past_caches, hipStream_t st) {
    const int nk = ra.pos0 + 1, n_items = ra.n_seq * kv.n_heads;
    if (n_items == 0) return 0;
    bf16_t *kc = (bf16_t *)kv.k + (size_t)layer * kv.layer_elems, *vc = (bf16_t *)kv.v + (size_t)layer * kv.layer_elems;
    ProfScope ps("attn_decode", 2.0 * n_items * (double)nk * kv.d * 2.0, st);
    const FusedQkv f{qkv, table};
    with_form(kv.d, past_caches, [&](auto dim, auto nt) {
        attn_decode_kernel<decltype(dim)::value, 8, true, decltype(nt)::value><<<n_items, 512, 0, st>>>(out, nullptr, kc, vc, f, kv.n_heads, nk, kv.pos_stride, H);
    });
    return vla_check_launch("attn_decode_qkv");
}
