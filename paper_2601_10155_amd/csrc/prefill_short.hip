// Causal scoring of a short block of queries against coded keys (paper Sec. 3.5, "Lookup and Sum", applied to every
// query position), the same scores as prefill.hip and prefill_dense.hip:
//     scores[b,h,t,l] = sum_i q_t^(i) . C_i[codes[b,h,l,i]]   for l <= t + (L - T),  else -inf.
//
// As in prefill_dense.hip the sum over subspaces is taken as a dense contraction of the queries with the keys' centroids
// on the matrix cores.  With few queries there is nothing to hide the fetch of the centroids behind: every key needs
// 2 d_k bytes of centroids whatever the number of queries, in pieces of 2 d_sub bytes, and fetched from L2 these random
// pieces are the whole time (41 us for 4 x 32 heads x 4096 keys at d_k = 128, m = 16).  So here a head's codebook moves
// into LDS first, once per workgroup, already scaled and split into two fp16 terms (d_k KB in all), and the keys gather
// their matrix operands from there, 16 bytes per read, ready to use.
//
// Shape of the computation
//   * one workgroup of 16 wavefronts per compute unit (two at d_k = 64) looks after one head: its share of the head's
//     (batch entry, 32-key block) list, NG groups of 16 queries at a time.  A wavefront's share is contiguous; the queries
//     of a batch entry are its stationary operand, reloaded when the batch entry changes;
//   * A = keys, B = queries on v_mfma_f32_16x16x32_f16: lane (n, kg) holds 8 coordinates of key n (one 16-byte gather for each
//     of the two terms; two 8-byte ones at d_sub = 4) and the same coordinates of query n of every group.  The result has
//     four consecutive keys of one query in a lane: 16-byte stores, 64 contiguous bytes of a score row;
//   * blocks that no query of the tile may see are filled with -inf without a gather.
// Arithmetic as in prefill_dense.hip where one power of two serves all centroids of the head (largest entry near 2^13):
// hi + lo 2^-11 carries 22 bits of every entry down to 2^-27 of the largest and 16 down to 2^-33; fp32 queries are scaled
// and split per query row, the product of the two small terms is dropped; fp32 accumulation over all d_k coordinates.
// Codebooks whose entries lie further apart (or are not finite: a filler for centroids that shall never be chosen, an outlier):
// the power of two is the one that serves most of them; the four coordinates around an entry that it does not serve are
// stored as NaN, and 32 keys of which one meets such a NaN (or an infinite query) are scored again from the fp32 codebook in
// plain fp32, on the fp32 matrix instruction, which takes operands and results in the same lanes.
// What bounds it: LDS.  Per 64 keys 4 d_k / 16 reads of 1 KB at random 16-byte addresses (about 12 clocks each), then the set-up
// of a workgroup (d_k KB of fp32 codebook through one compute unit, about 3 us).  The codebook is requested 50 instructions after the start, from
// preloaded arguments (470, two 64-bit divisions and four round trips to the argument block before: 4 x 32 heads x 8 queries x 4096 keys, d_k = 128,
// m = 16 13.5 / 12.9 us, 1 x 8 x 2 x 600 7.6 / 6.7).  Figures: see short_block.
#include <type_traits>

#include "common.h"

namespace lookat {

typedef _Float16 ps_v8h __attribute__((ext_vector_type(8)));
typedef _Float16 ps_v4h __attribute__((ext_vector_type(4)));
typedef float ps_v4f __attribute__((ext_vector_type(4)));
typedef unsigned int ps_v2u __attribute__((ext_vector_type(2)));
typedef unsigned int ps_v4u __attribute__((ext_vector_type(4)));

constexpr int kPsThreads = 1024;
constexpr int kPsWaves = kPsThreads / kWave;
constexpr float kPsLoScale = 2048.f;

// What is needed before the codebook and the first codes can be requested comes first, as scalars (14 dwords are delivered in registers at
// wave launch; everything else is a round trip to memory away), and the shares are counted on the host.
#define LOOKAT_PS_PARAMS                                                                                                  \
    const float *__restrict__ p_codebooks /* [H, m, 256, d_sub] */,                                                       \
        const uint8_t *__restrict__ p_codes /* (bh, l, i) at bh*code_stride + l*m + i */, int64_t p_code_stride, int64_t p_L, \
        int p_H, uint32_t p_per_head /* workgroups */, uint32_t p_shares /* per (head, query tile) */,                    \
        uint32_t p_blocks /* of a wavefront */, uint32_t p_rest /* the first so many have one more */,                    \
        uint32_t p_blocks_per_bh /* 32-key blocks */, const PrefillShortLate late
struct PrefillShortLate {
    const void *q;            // [BH, T, d_k] fp16 or fp32
    float *scores;            // [BH, T, L]
    int T;
    int vec4;                 // L % 4 == 0 and scores 16-byte aligned
};
struct PrefillShortArgs {
    const void *q;
    const float *codebooks;
    const uint8_t *codes;
    float *scores;
    int64_t code_stride;
    int64_t L;
    int T;
    int H;
    int vec4;
    uint32_t per_head, shares, blocks, rest, blocks_per_bh;
};

// A power of two that brings magnitudes of this (biased) exponent near 2^13, and its inverse.
__device__ __forceinline__ void ps_scale(int exponent, float &scale, float &inverse)
{
    int se = 13 - (exponent - 127);
    se = se > 100 ? 100 : (se < -100 ? -100 : se);
    scale = __uint_as_float((uint32_t)(se + 127) << 23);
    inverse = __uint_as_float((uint32_t)(127 - se) << 23);
}
constexpr int kPsSpan = 34;                          // exponents that one scale serves
constexpr int kPsLowest = 40, kPsHighest = 240;      // exponents that ps_scale does not clamp

// Largest value of each of the two halves over the wavefront.
typedef unsigned short ps_v2s __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t ps_max2(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ps_v2s, a), __builtin_bit_cast(ps_v2s, b)));
}
__device__ __forceinline__ uint32_t ps_wave_max2(uint32_t v)
{
    auto with = [&](float other) { v = ps_max2(v, __float_as_uint(other)); };
    with(dpp_mov<0xB1>(__uint_as_float(v), __uint_as_float(v)));
    with(dpp_mov<0x4E>(__uint_as_float(v), __uint_as_float(v)));
    with(dpp_mov<0x141>(__uint_as_float(v), __uint_as_float(v)));
    with(dpp_mov<0x140>(__uint_as_float(v), __uint_as_float(v)));
    float a, b;
    lanes_xor16(__uint_as_float(v), a, b);
    v = ps_max2(__float_as_uint(a), __float_as_uint(b));
    lanes_xor32(__uint_as_float(v), a, b);
    return ps_max2(__float_as_uint(a), __float_as_uint(b));
}

// Scores of 16 keys against 16 queries in plain fp32, in the lanes of the other path: lane (n, kg) brings coordinates
// 32 s + 8 kg .. + 7 of key n (codes at cp) and of query n (q: its row, from coordinate 8 kg on); any order of the coordinates
// serves as contraction index as long as both sides use the same one.
template <typename QT, int DK, int M>
__device__ __forceinline__ ps_v4f ps_plain(const float *cb_h, const uint8_t *cp, const QT *q, int kg)
{
    constexpr int DSUB = DK / M;
    ps_v4f acc = {0.f, 0.f, 0.f, 0.f};
    constexpr int kUnroll = DK == 128 ? 2 : 1;      // (registers)
#pragma unroll kUnroll
    for (int s = 0; s < DK / 32; ++s) {
        float x[8], y[8];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int d = 32 * s + 8 * kg + 4 * u, i = d / DSUB;
            const ps_v4f v = *reinterpret_cast<const ps_v4f *>(cb_h + ((int64_t)i * kCentroids + cp[i]) * DSUB + d % DSUB);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[4 * u + e] = v[e];
                y[4 * u + e] = (float)q[32 * s + 4 * u + e];
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], acc, 0, 0, 0);
    }
    return acc;
}

template <typename QT, int DK, int M, int NG>
__global__ __launch_bounds__(kPsThreads, 4) void score_prefill_short_kernel(LOOKAT_PS_PARAMS)
{
    constexpr bool Q32 = std::is_same<QT, float>::value;
    constexpr int DSUB = DK / M;
    constexpr int KW = 32;                            // coordinates per instruction
    constexpr int KS = DK / KW;                       // instructions per term and group
    constexpr uint32_t kTerm = DK * kCentroids * 2;   // bytes of one term's table
    static_assert(DSUB % 4 == 0, "an operand's coordinates come from one or two subspaces");
    extern __shared__ __align__(16) unsigned char smem[];   // [hi, lo][M][256][DSUB] fp16
    __shared__ uint32_t range_s[kPsWaves];

    // all workgroups of a head on one die, whose L2 then holds its codebook, codes and queries
    const uint32_t xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int h = (int)(slot / p_per_head * 8 + xcd);
    if (h >= p_H)
        return;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // the codebook (into LDS below) is what the workgroup waits for: requested before anything else is worked out
    constexpr int NV = DK * kCentroids / 4 / kPsThreads;
    const ps_v4f *cb = reinterpret_cast<const ps_v4f *>(p_codebooks + (int64_t)h * M * kCentroids * DSUB);
    ps_v4f cv[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k)
        cv[k] = cb[tid + k * kPsThreads];
    __builtin_amdgcn_sched_barrier(0);
    PrefillShortArgs a;
    a.q = late.q;
    a.codebooks = p_codebooks;
    a.codes = p_codes;
    a.scores = late.scores;
    a.code_stride = p_code_stride;
    a.L = p_L;
    a.T = late.T;
    a.H = p_H;
    a.vec4 = late.vec4;
    const uint32_t within = slot % p_per_head, share = within % p_shares;
    const int tile = (int)(within / p_shares);
    const int n = lane & 15, kg = lane >> 4;

    // ---- this wavefront's blocks, and the codes of the next one (key n of each half, in every lane group) ----
    // Wavefront by wavefront over the workgroups of a head, so that the blocks that do not come out, which go to the first parts, are as many in every
    // workgroup and one more in the first: a compute unit's wavefronts take turns at its LDS, and a workgroup of those with one more is what the
    // launch waits for (workgroup by workgroup: 1 x 16 heads x 18 queries x 2085 keys, d_k = 128, m = 16 13.4 / 15.2 us).
    const uint32_t part = (uint32_t)wave * p_shares + share;
    const int blk0 = (int)(part * p_blocks + (part < p_rest ? part : p_rest)), blk1 = blk0 + (int)(p_blocks + (part < p_rest ? 1u : 0u));
    int b = (int)((uint32_t)blk0 / p_blocks_per_bh), lb = blk0 - b * (int)p_blocks_per_bh;       // the block's batch entry and number within it
    constexpr int kCodeWords = (M + 3) / 4;
    uint32_t ahead[2][kCodeWords];
    auto load_codes = [&](int b_, int lb_) {
        const uint8_t *base = a.codes + ((int64_t)b_ * a.H + h) * a.code_stride;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int64_t l = (int64_t)lb_ * 32 + 16 * half + n;
            const uint8_t *cp = base + (l < a.L ? l : a.L - 1) * M;         // past the end: a repeat, not stored
            if constexpr (M == 2) {
                ahead[half][0] = *reinterpret_cast<const uint16_t *>(cp);
            } else if constexpr (M == 4) {
                ahead[half][0] = *reinterpret_cast<const uint32_t *>(cp);
            } else if constexpr (M == 8) {
                const ps_v2u t = *reinterpret_cast<const ps_v2u *>(cp);
                ahead[half][0] = t.x;
                ahead[half][1] = t.y;
            } else {
                const ps_v4u t = *reinterpret_cast<const ps_v4u *>(cp);
                ahead[half][0] = t.x;
                ahead[half][1] = t.y;
                ahead[half][2] = t.z;
                ahead[half][3] = t.w;
            }
        }
    };
    if (blk0 < blk1)
        load_codes(b, lb);

    // ---- codebook: registers -> largest magnitude -> LDS, scaled and split ----
    // largest magnitude, and twice the bits of the smallest that is not zero (less one: zero wraps to the top)
    float top = 0.f;
    uint32_t low = ~0u;
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            top = fmaxf(top, fabsf(cv[k][e]));
            low = min(low, (__float_as_uint(cv[k][e]) << 1) - 1u);
        }
    // exponents of both, the smallest's counted from the top
    uint32_t range = ps_wave_max2((__float_as_uint(top) >> 23) << 16 | (255u - (low >> 24)));
    if (lane == 0)
        range_s[wave] = range;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kPsWaves; ++w)
        range = ps_max2(range, range_s[w]);
    int exponent = (int)(range >> 16);
    // Are there entries that one scale does not serve?  (Uniform over the workgroup.  NaN entries need no search, they stay NaN.)
    const bool wide = exponent > kPsHighest || (exponent && exponent < kPsLowest) || exponent - (255 - (int)(range & 0xffffu)) >= kPsSpan;
    if (wide) {
        // the kPsSpan exponents that hold the largest entry of most 16-byte pieces (an eighth of them is looked at, from all
        // subspaces), their top end as low as possible
        uint32_t *count = reinterpret_cast<uint32_t *>(smem) + kPsSpan;   // per exponent, zeros in front; [256]: (pieces, 255 - top of the span)
        if (tid <= 256 + kPsSpan)
            count[tid - kPsSpan] = 0u;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NV; ++k)
            if (k == wave % NV) {
                const float x = fmaxf(fmaxf(fabsf(cv[k][0]), fabsf(cv[k][1])), fmaxf(fabsf(cv[k][2]), fabsf(cv[k][3])));
                if (x > 0.f && x < INFINITY)
                    atomicAdd(&count[__float_as_uint(x) >> 23], 1u);
            }
        __syncthreads();
        if (tid < 255) {
            uint32_t pieces = 0u;
#pragma unroll
            for (int x = 0; x < kPsSpan; ++x)
                pieces += count[tid - x];
            atomicMax(&count[256], pieces << 8 | (uint32_t)(255 - tid));
        }
        __syncthreads();
        exponent = 255 - (int)(count[256] & 255u);
        __syncthreads();                                           // (the operands overwrite the counts)
    }
    float scale, inv;
    ps_scale(exponent, scale, inv);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        ps_v4h hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float w = scale * cv[k][e];                          // exact (a power of two) where the scale serves
            hi[e] = (_Float16)w;
            lo[e] = (_Float16)((w - (float)hi[e]) * kPsLoScale);       // exact difference and scaling, one rounding
        }
        *reinterpret_cast<ps_v4h *>(smem + (uint32_t)(tid + k * kPsThreads) * 8u) = hi;
        *reinterpret_cast<ps_v4h *>(smem + kTerm + (uint32_t)(tid + k * kPsThreads) * 8u) = lo;
    }
    if (wide) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            bool served = true;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float w = fabsf(scale * cv[k][e]);
                served = served && w <= 65504.f && (w >= 0x1p-20f || cv[k][e] == 0.f);
            }
            if (!served)
                *reinterpret_cast<ps_v4h *>(smem + (uint32_t)(tid + k * kPsThreads) * 8u) =
                    ps_v4h{(_Float16)NAN, (_Float16)NAN, (_Float16)NAN, (_Float16)NAN};
        }
    }
    __syncthreads();

    const int64_t off = a.L - a.T;
    const int t0 = tile * 16 * NG;
    const int64_t seen = (t0 + 16 * NG < a.T ? t0 + 16 * NG : a.T) + off;    // keys from here on: -inf for every query of the tile
    ps_v8h qh[NG][KS], ql[Q32 ? NG : 1][Q32 ? KS : 1];     // the batch entry's queries: operand B
    float qinv[NG];
    float *row[NG];                                          // this lane's query of every group (past the end: a repeat, not stored)
    int b_loaded = -1;
    for (int blk = blk0; blk < blk1; ++blk) {
        if (b != b_loaded) {
            b_loaded = b;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int t = t0 + 16 * g + n < a.T ? t0 + 16 * g + n : a.T - 1;
                const int64_t qrow = ((int64_t)b * a.H + h) * a.T + t;
                const QT *q = static_cast<const QT *>(a.q) + qrow * DK + 8 * kg;
                row[g] = a.scores + qrow * a.L;
                qinv[g] = inv;
                if constexpr (!Q32) {
#pragma unroll
                    for (int s = 0; s < KS; ++s)
                        qh[g][s] = *reinterpret_cast<const ps_v8h *>(q + KW * s);
                } else {
                    ps_v4f v[KS][2];
                    float qmax = 0.f, qs, qi, x, y;
#pragma unroll
                    for (int s = 0; s < KS; ++s)
#pragma unroll
                        for (int p = 0; p < 2; ++p)
                            v[s][p] = *reinterpret_cast<const ps_v4f *>(q + KW * s + 4 * p);
#pragma unroll
                    for (int s = 0; s < KS; ++s)
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            qmax = fmaxf(qmax, fabsf(v[s][e / 4][e % 4]));
                    lanes_xor16(qmax, x, y);
                    qmax = fmaxf(x, y);
                    lanes_xor32(qmax, x, y);
                    ps_scale((int)(__float_as_uint(fmaxf(x, y)) >> 23), qs, qi);
                    qinv[g] *= qi;
#pragma unroll
                    for (int s = 0; s < KS; ++s)
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float w = qs * v[s][e / 4][e % 4];
                            qh[g][s][e] = (_Float16)w;
                            ql[g][s][e] = (_Float16)((w - (float)qh[g][s][e]) * kPsLoScale);
                        }
                }
            }
        }
        const int64_t l0 = (int64_t)lb * 32;
        uint32_t now[2][kCodeWords];
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int w = 0; w < kCodeWords; ++w)
                now[half][w] = ahead[half][w];
        if (++lb == (int)p_blocks_per_bh) {
            lb = 0;
            ++b;
        }
        if (blk + 1 < blk1)
            load_codes(b, lb);                               // the next block's codes arrive while this one is scored
        // result register r of lane (n, kg): key lh + 4 kg + r of query n of the group
        // (both halves before the check, so that the second one's gathers do not wait behind it, except where that
        // costs more registers than there are: 128, or 64 for two workgroups per compute unit at d_k = 64)
        constexpr int HJ = NG == 1 && DK == 128 ? 2 : 1;
        ps_v4f sc[2][NG];
#pragma unroll
        for (int half0 = 0; half0 < 2; half0 += HJ) {
            bool redo = false;
#pragma unroll
            for (int half = half0; half < half0 + HJ; ++half) {
                const int64_t lh = l0 + 16 * half;
                const uint32_t(&cw)[kCodeWords] = now[half];
                ps_v4f acc_h[NG], acc_l[NG];
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    acc_h[g] = ps_v4f{0.f, 0.f, 0.f, 0.f};
                    acc_l[g] = ps_v4f{0.f, 0.f, 0.f, 0.f};
                }
                if (lh < seen) {
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        // coordinates 32 s + 8 kg .. + 7 of the key
                        ps_v8h kh, kl;
                        if constexpr (DSUB >= 8) {
                            uint32_t code, base;
                            if constexpr (DSUB >= KW) {                        // one subspace for all lanes
                                constexpr int per = DSUB / KW;
                                const int i = s / per;
                                code = (cw[i / 4] >> (8 * (i % 4))) & 0xffu;
                                base = (uint32_t)(i * kCentroids * DSUB + (s % per) * KW + 8 * kg) * 2u;
                            } else {                                           // lane groups in 2 or 4 consecutive subspaces
                                constexpr int IPS = KW / DSUB;
                                const int isub = kg / (DSUB / 8);
                                code = (cw[(s * IPS) / 4] >> (8 * ((s * IPS) % 4 + isub))) & 0xffu;
                                base = (uint32_t)((s * IPS + isub) * kCentroids * DSUB + (8 * kg) % DSUB) * 2u;
                            }
                            const unsigned char *p = smem + base + code * (DSUB * 2);
                            kh = *reinterpret_cast<const ps_v8h *>(p);
                            kl = *reinterpret_cast<const ps_v8h *>(p + kTerm);
                        } else {                                               // d_sub = 4: two subspaces per lane
                            const int i0 = s * 8 + 2 * kg;
                            const uint32_t word_lo = cw[2 * s], word_hi = cw[2 * s + 1];
                            const uint32_t two = ((kg >= 2 ? word_hi : word_lo) >> (16 * (kg & 1))) & 0xffffu;
                            const unsigned char *p0 = smem + (uint32_t)(i0 * kCentroids + (two & 0xffu)) * 8u;
                            const unsigned char *p1 = smem + (uint32_t)((i0 + 1) * kCentroids + (two >> 8)) * 8u;
                            const ps_v4h h0 = *reinterpret_cast<const ps_v4h *>(p0), h1 = *reinterpret_cast<const ps_v4h *>(p1);
                            const ps_v4h g0 = *reinterpret_cast<const ps_v4h *>(p0 + kTerm), g1 = *reinterpret_cast<const ps_v4h *>(p1 + kTerm);
                            kh = __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7);
                            kl = __builtin_shufflevector(g0, g1, 0, 1, 2, 3, 4, 5, 6, 7);
                        }
#pragma unroll
                        for (int g = 0; g < NG; ++g) {
                            acc_h[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kh, qh[g][s], acc_h[g], 0, 0, 0);
                            acc_l[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kl, qh[g][s], acc_l[g], 0, 0, 0);
                            if constexpr (Q32)
                                acc_l[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kh, ql[g][s], acc_l[g], 0, 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int g = 0; g < NG; ++g) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        sc[half][g][e] = fmaf(acc_l[g][e], 1.f / kPsLoScale, acc_h[g][e]) * qinv[g];
                    redo |= !(fabsf((sc[half][g][0] + sc[half][g][1]) + (sc[half][g][2] + sc[half][g][3])) < INFINITY);
                }
            }
            if (__ballot(redo)) {   // a NaN that stands for an entry outside the scale's reach, an infinite input, or a score near the end of fp32
                const float *cb_h = a.codebooks + (int64_t)h * M * kCentroids * DSUB;
                const uint8_t *codes_b = a.codes + ((int64_t)b_loaded * a.H + h) * a.code_stride;
#pragma unroll
                for (int half = half0; half < half0 + HJ; ++half) {
                    const int64_t lk = l0 + 16 * half + n < a.L ? l0 + 16 * half + n : a.L - 1;
#pragma unroll
                    for (int g = 0; g < NG; ++g) {
                        const int t = t0 + 16 * g + n < a.T ? t0 + 16 * g + n : a.T - 1;
                        const QT *q = static_cast<const QT *>(a.q) + (((int64_t)b_loaded * a.H + h) * a.T + t) * DK + 8 * kg;
                        sc[half][g] = ps_plain<QT, DK, M>(cb_h, codes_b + lk * M, q, kg);
                    }
                }
            }
#pragma unroll
            for (int half = half0; half < half0 + HJ; ++half) {
                const int64_t l = l0 + 16 * half + 4 * kg;
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const int t = t0 + 16 * g + n;
                    if (t < a.T) {
                        ps_v4f o;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            o[e] = l + e <= t + off ? sc[half][g][e] : -INFINITY;
                        if (a.vec4) {
                            if (l < a.L)
                                *reinterpret_cast<ps_v4f *>(row[g] + l) = o;
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (l + e < a.L)
                                    row[g][l + e] = o[e];
                        }
                    }
                }
            }
        }
    }
}

template <typename QT, int DK, int M, int NG>
static int launch_prefill_short_case(const PrefillShortArgs &a, int64_t wgs, hipStream_t st)
{
    const size_t lds = (size_t)DK * kCentroids * 4;
    auto kern = score_prefill_short_kernel<QT, DK, M, NG>;
    if (lds > 48 * 1024) {   // (64 KB with the static part)
        // allow more than 64 KB of LDS: idempotent, so every call makes it (no flag shared between host threads)
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess)
            return fail(LOOKAT_ERR_HIP, "lookat_score_prefill: cannot reserve %zu bytes of LDS: %s", lds, hipGetErrorString(e));
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(kPsThreads), lds, st, a.codebooks, a.codes, a.code_stride, a.L, a.H, a.per_head, a.shares,
                       a.blocks, a.rest, a.blocks_per_bh, PrefillShortLate{a.q, a.scores, a.T, a.vec4});
    return check_launch("lookat_score_prefill");
}

// How a block is dealt out.
struct PsLayout {
    int ng;                  // groups of 16 queries per workgroup
    int tiles;               // query tiles of 16 ng
    int64_t blocks_per_bh;   // 32-key blocks
    int64_t shares;          // workgroups per (head, tile)
    int64_t wgs;
};
static PsLayout ps_layout(const lookat_shape *s, int T, int64_t L, bool q_fp32)
{
    PsLayout o;
    o.ng = (q_fp32 || T <= 16) ? 1 : 2;          // (two groups of split fp32 queries do not fit 128 registers)
    o.tiles = (T + 16 * o.ng - 1) / (16 * o.ng);
    o.blocks_per_bh = (L + 31) / 32;
    // workgroups per head and tile: one per compute unit (two at d_k = 64, whose codebook takes half the LDS), and at least
    // two blocks for a wavefront
    const int64_t heads = ((int64_t)s->H + 7) / 8 * 8;
    const int64_t most = (s->B * o.blocks_per_bh + 2 * kPsWaves - 1) / (2 * kPsWaves);
    o.shares = (s->d_k == 64 ? 512 : 256) / (heads * o.tiles);
    o.shares = o.shares < most ? o.shares : most;
    o.shares = o.shares < 1 ? 1 : o.shares;
    o.wgs = heads * o.tiles * o.shares;
    return o;
}

// Is there an instance, and does the launch stay under a grid of 2^32 threads?
static bool ps_fits(const lookat_shape *s, const PsLayout &o, bool q_fp32)
{
    return (s->d_k == 128 || (s->d_k == 64 && !q_fp32)) && (s->m == 2 || s->m == 4 || s->m == 8 || s->m == 16) && o.wgs <= 0x3fffff &&
           s->B * o.blocks_per_bh <= 0x7fffffff;
}

// Which blocks come here.  The alternatives are the lookup-and-sum kernel (blocks under 24 queries) and the dense kernel that
// fetches centroids from L2.  Which one is faster depends on how the work falls on the chip: here a head's workgroups share one die
// (few heads leave dies idle, nine to fifteen fill some dies twice) and each pays for the codebook, there every (b,h) is a workgroup or
// more.  So the rule compares predicted times, fitted to 15900 measured pairs (13 to 20% off at nine sizes in ten; d_k 64
// and 128, m 2 to 16, 1 to 1024 (b,h) of 1 to 40 heads, 1 to 64 queries, 64 to 12000 keys).  The blocks that it takes are
// 26% faster on the geometric mean at d_k = 128 under 24 queries (4 x 32 heads x 8 queries x 4096 keys, m = 16: 24.7 / 18.6 us, here
// second); of the measured ones five in a thousand are more than 3% slower.  (A rule on m, T and the number of keys alone took 8% of them
// at a loss of 10% and more: 115 x 2 heads x 8 queries x 7625 keys, m = 8: 41 / 145 us.)
static bool short_block(const lookat_shape *s, int T, int64_t L, bool q_fp32)
{
    const int64_t BH = (int64_t)s->B * s->H;
    const int quads = (T + 3) / 4;
    const PsLayout o = ps_layout(s, T, L, q_fp32);
    if (!ps_fits(s, o, q_fp32))
        return false;
    // Only where it was measured to pay at all.  fp32 queries are split like the centroids: 1.1e-7 off 64 bits against 0.93e-7
    // by lookup, so they do not come here where the lookup kernel is the other one.
    if (T >= 24 ? (s->d_k == 64 || T > (q_fp32 ? 64 : 32))
                : (q_fp32 || s->m * quads < (s->d_k == 128 ? 4 : 16) || (s->d_k == 64 && BH > 128)))
        return false;
    const double MB = 4e-6 * (double)BH * T * (double)L;           // of scores
    const int64_t per_die = (s->H + 7) / 8 * o.tiles * o.shares, at_once = s->d_k == 64 ? 64 : 32;
    const double rounds = (double)((per_die + at_once - 1) / at_once);
    // blocks of a wavefront (of the most loaded one, at d_k = 64, where a compute unit holds two workgroups)
    const double blocks = s->d_k == 64 ? (double)((s->B * o.blocks_per_bh + kPsWaves * o.shares - 1) / (kPsWaves * o.shares))
                                       : (double)(s->B * o.blocks_per_bh) / (double)(kPsWaves * o.shares);
    const double setup = s->d_k == 64 ? 1.8 : (q_fp32 ? 4.7 : (o.ng == 2 ? 4.0 : 3.3));
    const double block = s->d_k == 64 ? (o.ng == 2 ? 3.6 : 2.1) : (o.ng == 2 ? 2.5 : 1.8);
    const double odd = L % 4 ? 1.0 : 0.0;                                         // (rows not 16-byte aligned: four-byte stores)
    const double store = ((s->d_k == 64 ? 0.29 : 0.2) + 0.3 * odd) * (s->H < 4 ? 4.0 / s->H : 1.0);   // (one to three dies do not write faster)
    const double here = setup * (1.0 + rounds) + block * rounds * blocks + store * MB;
    double there;
    if (T >= 24) {
        const double panels = (double)BH * (double)((L + 127) / 128) / 512.0, tiles = (double)((T + 31) / 32);
        there = (q_fp32 ? 7.4 + 3.4 * panels + 2.0 * panels * tiles + 0.15 * MB : 5.9 + 2.9 * panels + 0.75 * panels * tiles + 0.09 * MB) +
                0.2 * odd * MB;
    } else {
        const double turns = (double)((BH + 255) / 256), look = 1e-3 * (double)L * quads;
        if (s->d_k == 64)
            there = -0.6 + 6.1 * turns + (0.04 + 0.078 * s->m) * turns * look + (1.0 + 0.023 * s->m) * 1e-3 * BH * look + (0.9 + 0.046 * s->m) * quads;
        else
            there = -2.4 + 11.4 * turns + (0.02 + 0.077 * s->m) * turns * look + (1.7 - 0.037 * s->m) * 1e-3 * BH * look + (1.35 + 0.036 * s->m) * quads;
        there += (0.04 + odd * (s->m <= 4 ? 0.35 : (s->m == 8 ? 0.15 : 0.0))) * MB;
    }
    return here < (T >= 24 ? 0.92 : (s->d_k == 64 ? 0.97 : 1.0)) * there;
}

bool prefill_short_takes(const lookat_shape *s, int T, int64_t L, bool q_fp32) { return short_block(s, T, L, q_fp32); }

// Launches where the rule says so (`any`: wherever there is an instance), status in *rc, and returns true; otherwise returns false.
bool launch_prefill_short(const lookat_shape *s, int T, int64_t L, const void *q, bool q_fp32, const float *codebooks,
                          const uint8_t *codes, int64_t code_stride_bh, float *scores, hipStream_t st, bool any, int *rc)
{
    const PsLayout o = ps_layout(s, T, L, q_fp32);
    if (any ? !ps_fits(s, o, q_fp32) : !short_block(s, T, L, q_fp32))
        return false;
    const int ng = o.ng;
    PrefillShortArgs a;
    a.q = q;
    a.codebooks = codebooks;
    a.codes = codes;
    a.scores = scores;
    a.code_stride = code_stride_bh;
    a.L = L;
    a.T = T;
    a.H = s->H;
    a.shares = (uint32_t)o.shares;
    a.per_head = (uint32_t)(o.tiles * o.shares);
    a.vec4 = (L % 4 == 0) && aligned16(scores);
    a.blocks_per_bh = (uint32_t)o.blocks_per_bh;
    const int64_t wavefronts = o.shares * kPsWaves;
    a.blocks = (uint32_t)(s->B * o.blocks_per_bh / wavefronts);
    a.rest = (uint32_t)(s->B * o.blocks_per_bh % wavefronts);
#define LOOKAT_PS_CASE(DK_, M_)                                                                              \
    if (s->d_k == DK_ && s->m == M_) {                                                                       \
        if constexpr (DK_ == 128) {                                                                          \
            if (q_fp32) {                                                                                    \
                *rc = launch_prefill_short_case<float, DK_, M_, 1>(a, o.wgs, st);                                   \
                return true;                                                                                 \
            }                                                                                                \
        }                                                                                                    \
        if (ng == 1)                                                                                         \
            *rc = launch_prefill_short_case<__half, DK_, M_, 1>(a, o.wgs, st);                                      \
        else                                                                                                 \
            *rc = launch_prefill_short_case<__half, DK_, M_, 2>(a, o.wgs, st);                                      \
        return true;                                                                                         \
    }
    LOOKAT_PS_CASE(64, 2)
    LOOKAT_PS_CASE(64, 4)
    LOOKAT_PS_CASE(64, 8)
    LOOKAT_PS_CASE(64, 16)
    LOOKAT_PS_CASE(128, 2)
    LOOKAT_PS_CASE(128, 4)
    LOOKAT_PS_CASE(128, 8)
    LOOKAT_PS_CASE(128, 16)
#undef LOOKAT_PS_CASE
    return false;
}

}  // namespace lookat
