// Attention decode over the product-quantised key cache (paper Algorithm 1 after the
// table build): s_l = sum_i LUT_i[code_l[i]] (Sec. 3.5 "Lookup and Sum"), softmax of
// scale*s, weighted sum of the fp16 values.
//
// Shape of the computation on gfx950
//   * the value stream (2*d_k bytes per key) and the code stream (m bytes per key) are
//     each read exactly once with 16-byte-per-lane loads, a wavefront covering 1 KB of
//     contiguous memory per load instruction;
//   * the table of one (b,h) (m KB) is staged in LDS once per workgroup and gathered
//     with one ds_read_b32 per (key, subspace);
//   * every wavefront owns 64-key tiles and keeps its own running max / sum / output
//     (online softmax), so the streaming loop has no workgroup barrier;
//   * the sequence is cut into `splits` ranges per (b,h) (flash-decoding style); the
//     ranges are merged by a second small kernel.
#include <mutex>
#include <type_traits>

#include "decode_common.h"
#include "lookat_probe.h"

namespace lookat {

struct DecodeArgs {
    const float *lut;        // [BH, m, 256]
    const uint8_t *codes;    // (bh, l, i) at bh*code_stride + l*m + i
    const __half *values;    // (bh, l, j) at bh*value_stride + l*d_k + j
    float *part;             // [BH, splits, d_k + 2]   (o[d_k], max, sum), unused when splits == 1
    float *out;              // [BH, d_k]
    float *scores_out;       // [BH, L] or nullptr
    int64_t code_stride;
    int64_t value_stride;
    int64_t L;
    int64_t keys_per_split;  // multiple of kTile
    int BH;
    int splits;
    int d_k;
    int m;
    float scale_log2e;       // scale * log2(e): the softmax runs in base 2
    // fused decode step only (lookat_decode_step): the table is built and the new key encoded in-kernel
    const void *q;           // [BH, d_k]
    const void *k_new;       // [BH, d_k]
    const float *codebooks;  // [H, m, 256, d_sub]
    uint8_t *codes_w;        // same cache as `codes`, writable: row L-1 receives the new key's codes
    int H;
};

// Kernel parameters.  The first 14 dwords of a kernel's arguments are delivered in scalar
// registers at wave launch (kernarg preload, -amdgpu-kernarg-preload-count); anything after
// them costs a round trip to memory before it can be used (about a microsecond on a fresh
// argument block, and a 52 MB decode launch lasts about ten).  So everything a wavefront needs
// before it can request its first tile travels in those 14 dwords, as scalars, and the rest
// follows in a struct that is read while the tile is in flight.
struct DecodeLate {
    float *part;
    float *out;
    float *scores_out;
    const void *q;
    const void *k_new;
    uint8_t *codes_w;
    int d_k;
    int m;
};
#define LOOKAT_DECODE_HEAD_PARAMS                                                                              \
    int p_BH, int p_splits, int p_H, const void *p_table, const uint8_t *p_codes, const __half *p_values,     \
        uint32_t p_code_stride, uint32_t p_value_stride, uint32_t p_L, uint32_t p_kps, float p_scale_log2e
#define LOOKAT_DECODE_HEAD_ARGS(a, fused)                                                                      \
    (a).BH, (a).splits, ((fused) ? (a).H : ((a).d_k | (a).m << 16)), ((fused) ? static_cast<const void *>((a).codebooks) : static_cast<const void *>((a).lut)), \
        (a).codes, (a).values, (uint32_t)(a).code_stride, (uint32_t)(a).value_stride, (uint32_t)(a).L,        \
        (uint32_t)(a).keys_per_split, (a).scale_log2e
static DecodeLate late_of(const DecodeArgs &a)
{
    return DecodeLate{a.part, a.out, a.scores_out, a.q, a.k_new, a.codes_w, a.d_k, a.m};
}
__device__ __forceinline__ DecodeArgs rebuild_args(LOOKAT_DECODE_HEAD_PARAMS, const DecodeLate &late, bool fused)
{
    DecodeArgs a;
    a.lut = fused ? nullptr : static_cast<const float *>(p_table);
    a.codebooks = fused ? static_cast<const float *>(p_table) : nullptr;
    a.codes = p_codes;
    a.values = p_values;
    a.part = late.part;
    a.out = late.out;
    a.scores_out = late.scores_out;
    a.code_stride = p_code_stride;
    a.value_stride = p_value_stride;
    a.L = p_L;
    a.keys_per_split = p_kps;
    a.BH = p_BH;
    a.splits = p_splits;
    a.d_k = fused ? late.d_k : (p_H & 0xffff);   // (tables given: no head count is needed, and these are needed early)
    a.m = fused ? late.m : (p_H >> 16);
    a.scale_log2e = p_scale_log2e;
    a.q = late.q;
    a.k_new = late.k_new;
    a.codes_w = late.codes_w;
    a.H = p_H;
    return a;
}

// Workgroup id -> (bh, split).  Consecutive workgroup ids land on different dies, each
// with its own L2; this mapping keeps all splits of one (b,h) on one die so that its
// table is fetched into a single L2.
__device__ __forceinline__ bool map_block_n(const DecodeArgs &a, int count, int &unit, int &split)
{
    const int bid = blockIdx.x;
    const int xcd = bid % kXcds;
    const int slot = bid / kXcds;
    unit = (slot / a.splits) * kXcds + xcd;
    split = slot % a.splits;
    return unit < count;
}
__device__ __forceinline__ bool map_block(const DecodeArgs &a, int &bh, int &split)
{
    return map_block_n(a, a.BH, bh, split);
}

// LDS of the fused step's encoder (see step_candidates): (distance, candidate) [m][4], the new codes [m] bytes.
constexpr int code_words(int m) { return m ? (m + 3) / 4 : 1; }    // words that hold a key's codes
constexpr int kNearest = 4;                           // wavefronts (of 64 centroids) per subspace
__host__ __device__ constexpr size_t step_encoder_bytes(int m) { return ((size_t)m * kNearest * 8 + (size_t)m + 15) / 16 * 16; }
// LDS of one batch entry of the fused step (table, per-wavefront partial results, the encoder's
// candidates), rounded to 16 bytes: the distance between the two entries' blocks of a paired workgroup.
__host__ __device__ constexpr size_t step_pair_lds_bytes(int m, int d_k)
{
    return (((size_t)m * kCentroids + (size_t)(2 * kDecWaves) * (d_k + 2)) * sizeof(float) + 15) / 16 * 16 + step_encoder_bytes(m);
}

// ---- pieces of the fused decode step ---------------------------------------------------
template <typename T>
__device__ __forceinline__ float step_f32(T v);
template <>
__device__ __forceinline__ float step_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float step_f32<__half>(__half v) { return __half2float(v); }

// A dense, 16-byte aligned, read-only array of T addressed uniformly over the wavefront, read
// as 32-bit words through the constant address space: the compiler turns these into scalar
// loads (an s_load needs dword alignment, which a __half pointer would not promise).
typedef const __attribute__((address_space(4))) uint32_t *UniformWords;
template <typename T>
__device__ __forceinline__ float uniform_elem(UniformWords p, int idx);
template <>
__device__ __forceinline__ float uniform_elem<float>(UniformWords p, int idx)
{
    return __uint_as_float(p[idx]);
}
template <>
__device__ __forceinline__ float uniform_elem<__half>(UniformWords p, int idx)
{
    const uint32_t w = p[idx >> 1];
    return __half2float(__ushort_as_half((unsigned short)((idx & 1) ? (w >> 16) : (w & 0xffffu))));
}

// ---- the rule ----
// Squared distance of the encoder (paper Sec. 3.4 "Encoding"), exactly as lookat_encode_keys evaluates it: fp64, ascending coordinates, one
// rounding per subtract, multiply and add.  A row lies over G neighbouring lanes, P coordinates each.  Differences and squares need no order; the
// additions are one chain, which is handed from lane to lane: after G rounds the last lane has added all of it, and every lane of the G gets that.
__device__ __forceinline__ double rule_square(float x, float y)
{
#pragma clang fp contract(off)
    const double diff = (double)x - (double)y;
    return diff * diff;
}
// (Values that only a rarely taken branch uses: without this the compiler widens them ahead of the branch and keeps both in registers.)
__device__ __forceinline__ v4f only_here(v4f v)
{
    asm volatile("" : "+v"(v));
    return v;
}
template <int G, int J>
__device__ __forceinline__ double group_broadcast64(double x)      // as group_broadcast, G up to 16
{
    if constexpr (G == 1)
        return x;
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    float lo = __uint_as_float((uint32_t)u), hi = __uint_as_float((uint32_t)(u >> 32));
    if constexpr (G == 2) {
        constexpr int kOf = J | J << 2 | (2 + J) << 4 | (2 + J) << 6;
        lo = dpp_mov<kOf>(lo, lo);
        hi = dpp_mov<kOf>(hi, hi);
    } else if constexpr (G > 2) {
        lo = group_broadcast<G, J>(lo);
        hi = group_broadcast<G, J>(hi);
    }
    return __longlong_as_double((long long)((uint64_t)__float_as_uint(hi) << 32 | __float_as_uint(lo)));
}
__device__ __forceinline__ void rule_add(double &acc, const v4f &x, const v4f &y)      // four coordinates more
{
#pragma clang fp contract(off)
#pragma unroll
    for (int t = 0; t < 4; ++t)
        acc = acc + rule_square(x[t], y[t]);
}
template <int G, int P>
__device__ __forceinline__ double rule_sum(const double (&sq)[P], int lane)
{
#pragma clang fp contract(off)
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < P; ++j)
        acc = acc + sq[j];
#pragma unroll 1
    for (int n = 1; n < G; ++n) {
        const uint64_t u = (uint64_t)__double_as_longlong(acc);
        const float lo = __uint_as_float((uint32_t)u), hi = __uint_as_float((uint32_t)(u >> 32));
        const uint64_t left = (uint64_t)__float_as_uint(dpp_mov<0x111>(hi, hi)) << 32 | __float_as_uint(dpp_mov<0x111>(lo, lo));   // row_shr:1
        acc = lane % G ? __longlong_as_double((long long)left) : 0.0;
#pragma unroll
        for (int j = 0; j < P; ++j)
            acc = acc + sq[j];
    }
    return group_broadcast64<G, G - 1>(acc);
}

// Encoding the new key, in two steps.  In fp32 a squared distance is off by at most (d_sub + 2) 2^-24 of itself, in whatever order its terms are
// added (each difference is rounded once, each multiply-add and addition once, all terms are positive), so a centroid whose fp32 distance
// exceeds the smallest by more than twice that cannot be the argmin.  A wavefront of 64 centroids with one left has its candidate without the
// fp64 rule, which takes two and a half times the instructions; of those that are not provably beyond the limit (near and exact ties, NaN) the
// repeats of the lowest go, and what is left is evaluated by the rule.  The four candidates of a subspace are compared the same way after the
// barrier by the wavefront that scores the new key, one lane each.
// The largest fp32 distance that a centroid may have to be the argmin when the smallest is `least` (twice the error bound, rounded up; the last
// term for squares below the normal range).  NaN if least is.
template <int DSUB>
__device__ __forceinline__ float step_limit(float least)
{
    return fmaf(least, 1.f + (float)(2 * DSUB + 8) * 0x1p-23f, (float)DSUB * 0x1p-124f);
}
// Minima over the wavefront of N values per lane (a power of two up to 8), NaN left out; uniform results.  A swap of lane halves or rows leaves
// one minimum of two values in each, so N values cost little more than one.
template <int N>
__device__ __forceinline__ void wave_minima(const float (&x)[N], float (&least)[N], int lane)
{
    static_assert(N == 1 || N == 2 || N == 4 || N == 8, "powers of two");
    float v[N], a, b;
    if constexpr (N >= 2) {
#pragma unroll
        for (int e = 0; e < N / 2; ++e) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[e]), __float_as_uint(x[e + N / 2]), false, false);
            v[e] = fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
        }
    } else {
        lanes_xor32(x[0], a, b);
        v[0] = fminf(a, b);
    }
    if constexpr (N >= 4) {
#pragma unroll
        for (int e = 0; e < N / 4; ++e) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[e]), __float_as_uint(v[e + N / 4]), false, false);
            v[e] = fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
        }
    } else {
        lanes_xor16(v[0], a, b);
        v[0] = fminf(a, b);
    }
    if constexpr (N >= 8) {
        const bool odd = lane & 8;
        const float own = odd ? v[1] : v[0], other = odd ? v[0] : v[1];
        v[0] = fminf(own, dpp_mov<0x128>(other, other));
    } else {
        v[0] = fminf(v[0], dpp_mov<0x128>(v[0], v[0]));
    }
    v[0] = fminf(v[0], dpp_mov<0x141>(v[0], v[0]));
    v[0] = fminf(v[0], dpp_mov<0x4E>(v[0], v[0]));
    v[0] = fminf(v[0], dpp_mov<0xB1>(v[0], v[0]));
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const int at = N == 1 ? 0 : (N == 2 ? 32 * e : (N == 4 ? 16 * e : 8 * e));
        least[e] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v[0]), at));
    }
}
// This wavefront's candidates for subspaces i0 .. i0+GS-1: dist[s] is the lane's fp32 distance to centroid c; all four wavefronts of a subspace
// hold ascending ranges of centroids, `quarter` says which.  distinct(s, among) drops lanes of `among` whose row repeats the lowest one's, and
// exact(s, among) gives the rest their distances by the rule, both from the rows in registers: a key that meets ties may meet them in every subspace
// and every step (zeros, say, where unused centroids kept an initial duplicate), and all wavefronts wait for the table.  us, keys that meet no
// tie / nine copies of the nearest centroid over the four wavefronts in every subspace / that with the rows read again, subspace after subspace:
// 32 (b,h) x 600 keys, d_k = 128, m = 16 7.2 / 9.9 / 16.2, m = 2 6.9 / 8.0 / 14.5; 640, d_k = 64, m = 8 13.3 / 17.9 / 26.9; two query heads, 64
// (b,h), d_k = 64, m = 16 8.4 / 10.9 / 18.5.  (The branch is laid out behind the rest: in line it cost groups of 4 and 8, d_k = 128, m = 2 3%.)
template <int DSUB, int GS, typename Distinct, typename Exact>
__device__ __forceinline__ void step_candidates(const float (&dist)[GS], int i0, int c, int quarter, int lane, uint2 *near_s, Distinct distinct,
                                                Exact exact)
{
    float least[GS];
    wave_minima<GS>(dist, least, lane);
    uint64_t among[GS], several = 0;
#pragma unroll
    for (int s = 0; s < GS; ++s) {
        among[s] = __ballot(!(dist[s] > step_limit<DSUB>(least[s])));
        several |= among[s] & (among[s] - 1);
    }
    if (__builtin_expect(several != 0, 0)) {       // the rule, lowest centroid on ties
#pragma unroll
        for (int s = 0; s < GS; ++s)
            if (among[s] & (among[s] - 1)) {
                among[s] = distinct(s, among[s]);
                if (!(among[s] & (among[s] - 1)))
                    continue;
                const bool mine = among[s] >> lane & 1;
                const double by_rule = exact(s, among[s]);
                const double own = mine ? argmin_value(by_rule, c) : (double)INFINITY;
                if (__popcll(among[s]) == 2) {
                    const int a = __builtin_ctzll(among[s]), b = 63 - __builtin_clzll(among[s]);
                    const uint64_t u = (uint64_t)__double_as_longlong(own);
                    auto of = [&](int from) {
                        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, from);
                        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), from);
                        return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
                    };
                    const double da = of(a), db = of(b);
                    const bool first = da < db || (da == db && __builtin_amdgcn_readlane(c, a) < __builtin_amdgcn_readlane(c, b));
                    among[s] = 1ull << (first ? a : b);
                } else {
                    double dv[1] = {own};
                    dmin_wave<1>(dv);
                    const bool holds = mine && own == dv[0];
                    among[s] = __ballot(holds);
                    if (among[s] & (among[s] - 1)) {
                        const float lowest = wave_max(holds ? -(float)c : -INFINITY);
                        among[s] = __ballot(holds && -(float)c == lowest);
                    }
                }
            }
    }
#pragma unroll
    for (int s = 0; s < GS; ++s)
        if (among[s] >> lane & 1)
            near_s[(i0 + s) * kNearest + quarter] = make_uint2(__float_as_uint(dist[s]), (uint32_t)c);
}
// `among` without the lanes whose row repeats that of the lowest of them (a row per lane).
template <int DSUB>
__device__ __forceinline__ uint64_t rows_without_repeats(const float (&row)[DSUB], uint64_t among)
{
    const int lead = __builtin_ctzll(among);
    bool same = true;
#pragma unroll
    for (int j = 0; j < DSUB; ++j)
        same &= __int_as_float(__builtin_amdgcn_readlane(__float_as_int(row[j]), lead)) == row[j];
    return (among & ~__ballot(same)) | 1ull << lead;
}
// The new key's codes (four to a word; uniform) after the barrier, for the wavefront that scores position L-1: lane (i, w) holds the candidate of
// subspace i among centroids 64w .. 64w+63.  They go to the cache and, in the lane that scores that key, in the place of the cached row, which
// may be stale (consume_tile).
template <typename FT, int DSUB, int M>
__device__ __forceinline__ void step_new_codes(uint32_t (&fresh)[code_words(M)], uint2 *near_s, const float *cb_head, const FT *k_row,
                                               uint8_t *code_row, int lane)
{
    const int at = lane < M * kNearest ? lane : 0;
    const uint2 mine = near_s[at];
    const float d = __uint_as_float(mine.x);
    const int c = (int)mine.y;
    float least = fminf(d, dpp_mov<0xB1>(d, d));
    least = fminf(least, dpp_mov<0x4E>(least, least));
    uint64_t left = __ballot(!(d > step_limit<DSUB>(least)));      // the candidates that may be the argmin, four bits a subspace
    constexpr uint64_t kLowest = M == 16 ? 0x1111111111111111ull : (1ull << (M * kNearest % 64)) / 15u;       // bit 0 of every subspace
    constexpr uint64_t kLanes = kLowest * 15u;
    left &= kLanes;
    // (one each: then no subspace has fewer, and all have M together)
    if (__popcll(left) != M) {
        // (a candidate's row lies over 16 / M lanes: one round trip for all of it)
        constexpr int G = kWave / (M * kNearest), P = DSUB / G;
        const int slot = lane / G;
        const FT *x = k_row + slot / kNearest * DSUB + lane % G * P;
        const float *y = cb_head + (slot / kNearest * kCentroids + (int)near_s[slot].y) * DSUB + lane % G * P;
        auto four = [&](int j, v4f &xj, v4f &yj) {
            FT e[4];
            __builtin_memcpy(e, __builtin_assume_aligned(x + j, 8), sizeof(e));
            xj = v4f{step_f32<FT>(e[0]), step_f32<FT>(e[1]), step_f32<FT>(e[2]), step_f32<FT>(e[3])};
            yj = *reinterpret_cast<const v4f *>(y + j);
        };
        double dv = 0.0;
        if constexpr (G == 1) {                  // (80 registers: four coordinates at a time)
            if (left >> lane & 1) {
#pragma unroll 1
                for (int j = 0; j < P; j += 4) {
                    v4f xj, yj;
                    four(j, xj, yj);
                    rule_add(dv, xj, yj);
                }
            }
        } else {
            double sq[P] = {};
            if (left >> slot & 1) {
#pragma unroll
                for (int j = 0; j < P; j += 4) {
                    v4f xj, yj;
                    four(j, xj, yj);
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        sq[j + t] = rule_square(xj[t], yj[t]);
                }
            }
            dv = __shfl(rule_sum<G, P>(sq, lane), lane % (M * kNearest) * G);
        }
        dv = left >> lane & 1 ? argmin_value(dv, c) : (double)INFINITY;
        double dm = dmin_dpp<0xB1>(dv);
        dm = dmin_dpp<0x4E>(dm);
        left &= __ballot(dv == dm);
    }
    if constexpr (M <= 4) {
        fresh[0] = 0;
#pragma unroll
        for (int i = 0; i < M; ++i)            // (candidates ascend: the lowest on ties)
            fresh[0] |= (uint32_t)__builtin_amdgcn_readlane(c, kNearest * i + __builtin_ctz((uint32_t)(left >> (kNearest * i)) & 15u)) << (8 * i);
    } else {
        uint8_t *new_s = reinterpret_cast<uint8_t *>(near_s + M * kNearest);
        if (lane < M * kNearest && (lane & 3) == __builtin_ctz((uint32_t)(left >> (lane & ~3)) & 15u))
            new_s[lane / kNearest] = (uint8_t)c;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint32_t *words = reinterpret_cast<const uint32_t *>(new_s);
#pragma unroll
        for (int w = 0; w < code_words(M); ++w)
            fresh[w] = (uint32_t)__builtin_amdgcn_readfirstlane((int)words[w]);
    }
    if (lane == 0) {
        if constexpr (M == 2) {
            *reinterpret_cast<uint16_t *>(code_row) = (uint16_t)fresh[0];
        } else {
#pragma unroll
            for (int w = 0; w < M / 4; ++w)
                reinterpret_cast<uint32_t *>(code_row)[w] = fresh[w];
        }
    }
}

// ---- the table from whole lines of the codebook ----------------------------------------------------------------
// Four wavefronts take a quarter of a subspace's centroids each.  A wave-wide load fetches a contiguous kilobyte, 16 bytes per lane: LPW = d_sub / 4
// lanes hold a row, and a lane's share of a dot product is four coordinates of the LPW rows that it meets in LPW loads.  Adding across the LPW
// lanes while handing each of them one row's sum takes 3 (LPW - 1) instructions for LPW rows.  (A thread per row, 16 bytes of it per load, keeps the
// compute unit's address pipeline busy for 64 clocks per load at d_sub = 32, 32 at 16, where a contiguous kilobyte takes 16.)
template <int LPW>
__device__ __forceinline__ float sum_rows(float (&p)[LPW], int lane)      // -> the sum of row (lane % LPW) * (64 / LPW) + lane / LPW
{
    if constexpr (LPW == 16) {
        const bool up = lane & 8;
        float r[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float other = up ? p[k] : p[8 + k];
            r[k] = (up ? p[8 + k] : p[k]) + dpp_mov<0x140>(other, other);      // row_mirror: 15 - lane
        }
        return sum_rows<8>(r, lane);
    } else if constexpr (LPW == 8) {
        const bool up = lane & 4;
        float r[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float other = up ? p[k] : p[4 + k];
            r[k] = (up ? p[4 + k] : p[k]) + dpp_mov<0x141>(other, other);      // row_half_mirror: 7 - lane
        }
        return sum_rows<4>(r, lane);
    } else if constexpr (LPW == 4) {
        const bool up = lane & 2;
        float r[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float other = up ? p[k] : p[2 + k];
            r[k] = (up ? p[2 + k] : p[k]) + dpp_mov<0x4E>(other, other);
        }
        return sum_rows<2>(r, lane);
    } else if constexpr (LPW == 2) {
        const bool up = lane & 1;
        const float other = up ? p[0] : p[1];
        return (up ? p[1] : p[0]) + dpp_mov<0xB1>(other, other);
    } else {
        return p[0];
    }
}

// MS subspaces from i0 on, NB batch entries (rows row0 and row0 + H of q and k_new), GS subspaces' rows in registers at a time.
// (Fewer rows at once where the registers decide on a workgroup more per compute unit: paired entries at d_k = 128, and one (b,h) per workgroup with
// 16 subspaces there.)
template <typename FT, int DK, int M, int MS, int NB>
struct StepTable {
    static constexpr int DSUB = DK / M, LPW = DSUB / 4;
    static constexpr int kRegs = DK == 128 && (NB == 2 || (M == 16 && MS == M)) ? 32 : 64;
    static constexpr int GS0 = kRegs / DSUB < 1 ? 1 : (kRegs / DSUB > 8 ? 8 : kRegs / DSUB);
    static constexpr int GS = GS0 < MS ? GS0 : MS;
    static constexpr int kSlice = MS * DSUB;                       // elements of a query, or key, that concern these subspaces
    static constexpr int kWords = 2 * NB * kSlice;                 // [entry][q, k_new][slice], staged as fp32 in LDS
    static constexpr int kPer = kWords / kWave;
    static_assert(kWords % kWave == 0 && MS % GS == 0, "whole loads, whole groups");
    FT word[kPer];
    v4f x[GS][LPW];

    __device__ __forceinline__ void request_words(const FT *q, const FT *k_new, int64_t row0, int H, int i0, int lane)
    {
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int e = r * kWave + lane, which = e / kSlice;
            const FT *from = which & 1 ? k_new : q;
            word[r] = from[(row0 + (which >> 1) * H) * DK + i0 * DSUB + e % kSlice];
        }
    }
    // rows of the centroids 64 quarter .. of subspaces i .. i+GS-1
    __device__ __forceinline__ void request_rows(const float *cb_head, int i, int quarter, int lane)
    {
#pragma unroll
        for (int s = 0; s < GS; ++s) {
            const v4f *from = reinterpret_cast<const v4f *>(cb_head + ((i + s) * kCentroids + quarter * kWave) * DSUB) + lane;
#pragma unroll
            for (int u = 0; u < LPW; ++u)
                x[s][u] = from[u * kWave];
        }
    }
    // stage: kWords floats of LDS for this wavefront alone, 16-byte aligned
    __device__ __forceinline__ void stage_words(float *stage, int lane) const
    {
#pragma unroll
        for (int r = 0; r < kPer; ++r)
            stage[r * kWave + lane] = step_f32<FT>(word[r]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    static constexpr uint64_t kFirst = LPW == 1 ? ~0ull : ~0ull / ((1ull << LPW) - 1);      // lanes that hold a row's first coordinates
    // `among` (a row's bit is that of the lane that has its distance) without the rows that repeat the lowest of them.
    __device__ __forceinline__ uint64_t without_repeats(int s, uint64_t among, int lane) const
    {
        uint64_t keep = 0;
        v4f lowest = {};
#pragma unroll
        for (int u = 0; u < LPW; ++u) {
            const uint64_t rows = among & kFirst << u;
            if (rows) {
                const v4f y = only_here(x[s][u]);
                uint64_t lead = 0;
                if (!keep) {
                    lead = rows & -rows;
                    const int from = 4 * (__builtin_ctzll(rows) / LPW * LPW + lane % LPW);
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        lowest[t] = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(y[t])));
                }
                uint64_t same = __ballot(y.x == lowest.x && y.y == lowest.y && y.z == lowest.z && y.w == lowest.w);
#pragma unroll
                for (int n = LPW / 2; n >= 1; n /= 2)          // (of all of a row's lanes)
                    same &= same >> n;
                keep |= lead | (rows & ~((same & kFirst) << u));
            }
        }
        return keep;
    }
    // Distances by the rule of the rows in `among`, in the lanes that have their bits; k: the lane's four coordinates of the new key.
    __device__ __forceinline__ double exact(const v4f &k, int s, uint64_t among, int lane) const
    {
        double d = 0.0;
#pragma unroll
        for (int u = 0; u < LPW; ++u)
            if (among & kFirst << u) {
                const v4f y = only_here(x[s][u]);
                const double sq[4] = {rule_square(k.x, y.x), rule_square(k.y, y.y), rule_square(k.z, y.z), rule_square(k.w, y.w)};
                const double sum = rule_sum<LPW, 4>(sq, lane);
                d = lane % LPW == u ? sum : d;
            }
        return d;
    }
    // Table entries and, if encode, candidates of the group of subspaces i .. i+GS-1 (g0 = i - i0) for batch entry nb.
    __device__ __forceinline__ void group(const float *stage, int nb, int g0, int i, int quarter, int lane, float *lut_s, uint2 *near_s,
                                          bool encode) const
    {
        const int c = quarter * kWave + lane % LPW * (kWave / LPW) + lane / LPW;
        const float *mine = stage + 2 * nb * kSlice + g0 * DSUB + 4 * (lane % LPW);
#pragma unroll
        for (int s = 0; s < GS; ++s) {
            const v4f q = *reinterpret_cast<const v4f *>(mine + s * DSUB);
            float p[LPW];
#pragma unroll
            for (int u = 0; u < LPW; ++u)
                p[u] = fmaf(q.w, x[s][u].w, fmaf(q.z, x[s][u].z, fmaf(q.y, x[s][u].y, q.x * x[s][u].x)));
            lut_s[(i + s) * kCentroids + c] = sum_rows<LPW>(p, lane);
        }
        if (encode) {
            float dist[GS];
#pragma unroll
            for (int s = 0; s < GS; ++s) {
                const v4f k = *reinterpret_cast<const v4f *>(mine + kSlice + s * DSUB);
                float p[LPW];
#pragma unroll
                for (int u = 0; u < LPW; ++u) {
                    const v4f d = {k.x - x[s][u].x, k.y - x[s][u].y, k.z - x[s][u].z, k.w - x[s][u].w};
                    p[u] = fmaf(d.w, d.w, fmaf(d.z, d.z, fmaf(d.y, d.y, d.x * d.x)));
                }
                dist[s] = sum_rows<LPW>(p, lane);
            }
            step_candidates<DSUB, GS>(
                dist, i, c, quarter, lane, near_s, [&](int s, uint64_t among) { return without_repeats(s, among, lane); },
                [&](int s, uint64_t among) {
                    return exact(only_here(*reinterpret_cast<const v4f *>(mine + kSlice + s * DSUB)), s, among, lane);
                });
        }
    }
};

// One 64-key tile of a wavefront: its codes (kc) and first CH value-row groups (v) are in
// registers or in flight.  Scores one key per lane (key = kb + kofs), updates the running
// max / sum, and accumulates the weighted value rows.
//
// MM (grouped queries, d_k = 128, G >= 4): the weighted value sum of the tile is a dense contraction
// [G query heads x 64 keys] . [64 keys x 128 coordinates] and runs on the matrix cores
// (v_mfma_f32_16x16x16_f16, fp32 accumulate) instead of G x 128 multiply-adds per key on the vector ALU:
//   * A operand = value rows, as loaded: lane (rowin, sub) holds 8 coordinates of the rows 4j + rowin of a
//     16-key step, j = 0..3.  With the instruction's contraction index k = 4*rowin + j standing for key
//     4j + rowin, the four halves a lane must supply for coordinate 8*sub + e are element e of its four
//     loads: two byte permutes per instruction, no data crosses lanes.  Instruction e of a step handles the
//     coordinates {8*s + e}: row s of its 16 x 16 result is coordinate 8*s + e;
//   * B operand = weights: column n < G is the weight of query head n rounded to fp16, column G + n the
//     remainder (p - fp16(p)) * 2^11 rounded to fp16, so that hi + lo * 2^-11 carries 22 bits of p; the
//     weights go from the scoring lanes (one key per lane, all heads) to the operand layout (one column per
//     lane, four keys) through 2 KB of LDS per wavefront, rows XOR-swizzled so that neither side conflicts;
//   * the accumulators (8 instructions x 4 registers) are rescaled only in tiles where the reference
//     moves; hi and lo columns are combined once, after the last tile.
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
constexpr float kLag = 8.f;          // log2 units: weights stay below 2^8, inside fp16 and far from fp32's limits
constexpr float kLoScale = 2048.f;   // 2^11: lifts the remainder of a weight into fp16's normal range

template <int M>
struct CodesOfM {
    typedef KeyCodes<M> type;
};
template <>
struct CodesOfM<0> {
    typedef KeyCodesAny type;
};
template <>
struct CodesOfM<1> {
    typedef KeyCodesBytes<1> type;
};
template <>
struct CodesOfM<32> {
    typedef KeyCodesBytes<32> type;
};
template <int M>
using CodesOf = typename CodesOfM<M>::type;

// `patch(codes, kb, key)` puts the new key's codes in the place of the cached row (fused step).
struct NothingNew {
    template <typename Codes>
    __device__ __forceinline__ void operator()(Codes &, uint32_t, uint32_t) const {}
};
// `ahead(n)` is called when the registers of value rows n .. n+7 are free (whole tiles only).
struct NothingAhead {
    __device__ __forceinline__ void operator()(int) const {}
};
template <int DK, int M, int CH, int G, bool MM, bool PAD, bool FIRST = false, typename Patch, typename Ahead = NothingAhead>
__device__ __forceinline__ void consume_tile(const DecodeArgs &a, SoftmaxState<G> &st, const CodesOf<M> &kc_in,
                                             v4u (&v)[CH], const float *lut_s, __amdgpu_buffer_rsrc_t rc,
                                             __amdgpu_buffer_rsrc_t rv, int bh, uint32_t kb, uint32_t k1,
                                             uint32_t kofs, int lane, int m, Patch patch,
                                             v4f (&accm)[MM ? 8 : 1], uint32_t pstage, uint32_t lane_off,
                                             uint32_t row_bytes, Ahead ahead = Ahead())
{
    constexpr int LPR = DK / 8;
    constexpr int NLD = LPR;
    const uint32_t key = kb + kofs;
    CodesOf<M> kc = kc_in;
    patch(kc, kb, key);
    // one score per query head of the group: the same codes index that head's tables
    float sc[G], p[G];
    bool above = false;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        float raw;
        if constexpr (M != 0)
            raw = kc.score(lut_s + g * (M * kCentroids));
        else
            raw = kc.score(lut_s + g * (m * kCentroids), m);
        sc[g] = -INFINITY;
        if (key < k1) {
            if (a.scores_out)
                a.scores_out[((int64_t)bh * G + g) * a.L + key] = raw;
            sc[g] = raw * a.scale_log2e;
        }
        if constexpr (FIRST)
            st.m_run[g] = wave_max(sc[g]);
        else
            above |= sc[g] > st.m_run[g] + kLag;
    }
    // The weights' reference need not be the running maximum, only near it: it moves (and the sums are rescaled) when a score
    // exceeds it by more than kLag, so most tiles do without the reduction over the wavefront.  A wavefront's first tile (FIRST)
    // sets it and has no sums to rescale: contexts of one tile per wavefront would otherwise pay for the test as well (group 4, up
    // to 512 keys, d_k = 128: 7.5 us a launch before there was a test, 7.9 with it in every tile, 7.5 now).
    if (!FIRST && __builtin_amdgcn_ballot_w64(above)) {
        float corr_n = 1.f;      // MM: the correction of the query head whose column this lane accumulates
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float m_new = fmaxf(st.m_run[g], wave_max(sc[g]));
            const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
            const float corr = fast_exp2(st.m_run[g] - m_use);
            st.z[g] *= corr;
            if constexpr (MM) {
                corr_n = ((lane & (G - 1)) == g) ? corr : corr_n;
            } else {
#pragma unroll
                for (int d = 0; d < 8; ++d)
                    st.acc[g][d] *= corr;
            }
            st.m_run[g] = m_new;
        }
        if constexpr (MM) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                accm[e] *= corr_n;
        }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        // (all scores so far -inf: weights 0)
        p[g] = fast_exp2(sc[g] - ((st.m_run[g] == -INFINITY) ? 0.f : st.m_run[g]));
        st.z[g] += p[g];
    }
    if constexpr (MM) {
        static_assert(DK == 128 && CH % 4 == 0 && G >= 4 && G <= 8, "matrix-core value sum: d_k = 128, 4 or 8 query heads");
        // weights to the staging rows: this lane scored key 16*(sub/4) + 4*(sub%4) + rowin of the tile
        const uint32_t sub_ = (uint32_t)lane & 15u, rowin_ = (uint32_t)lane >> 4;
        const uint32_t r_w = (sub_ & ~3u) + rowin_;                 // staging row (step, rowin)
        const uint32_t w_base = pstage + r_w * 128u + 2u * (sub_ & 3u);
        const uint32_t w_swz = (r_w >> 1) * 8u;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const _Float16 hi = (_Float16)p[g];
            const _Float16 lo = (_Float16)((p[g] - (float)hi) * kLoScale);
            *reinterpret_cast<__attribute__((address_space(3))) _Float16 *>(w_base + (((uint32_t)g * 8u) ^ w_swz)) = hi;
            *reinterpret_cast<__attribute__((address_space(3))) _Float16 *>(w_base + (((uint32_t)(G + g) * 8u) ^ w_swz)) = lo;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint32_t n_ = sub_, kg_ = rowin_;                    // operand column, contraction group
#pragma unroll
        for (int c0 = 0; c0 < NLD; c0 += CH) {
#pragma unroll
            for (int tt = 0; tt < CH / 4; ++tt) {
                const uint32_t r_r = (uint32_t)(c0 / 4 + tt) * 4u + kg_;
                const v4h bw = *reinterpret_cast<const __attribute__((address_space(3))) v4h *>(
                    pstage + r_r * 128u + ((n_ * 8u) ^ ((r_r >> 1) * 8u)));
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
                    v2u aw;
                    aw.x = __builtin_amdgcn_perm(v[4 * tt + 1][e >> 1], v[4 * tt + 0][e >> 1], sel);
                    aw.y = __builtin_amdgcn_perm(v[4 * tt + 3][e >> 1], v[4 * tt + 2][e >> 1], sel);
                    accm[e] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(v4h, aw), bw, accm[e], 0, 0, 0);
                }
            }
            if (c0 + CH < NLD)
                load_rows<DK, CH>(v, rv, kb, c0 + CH, lane);   // next row groups of this tile
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();   // the next tile's weights overwrite the staging rows
        return;
    }
    if constexpr (!std::is_same<Ahead, NothingAhead>::value) {
        static_assert(G == 1 && CH == NLD && CH % 8 == 0, "whole tiles, eight rows at a time");
#pragma unroll
        for (int c0 = 0; c0 < NLD; c0 += 8) {
            fma_rows<LPR, 8>(st.acc[0], p[0], reinterpret_cast<const v4u(&)[8]>(v[c0]), c0);
            __builtin_amdgcn_sched_barrier(0);
            ahead(c0);
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }
#pragma unroll
    for (int c0 = 0; c0 < NLD; c0 += CH) {
#pragma unroll
        for (int g = 0; g < G; ++g)   // the value rows are read once and weighted G times
            fma_rows<LPR, CH>(st.acc[g], p[g], v, c0);
        if (c0 + CH < NLD) {   // next row groups of this tile
            if constexpr (PAD)
                load_rows_padded<DK, CH>(v, rv, kb, c0 + CH, lane_off, row_bytes);
            else
                load_rows<DK, CH>(v, rv, kb, c0 + CH, lane);
        }
    }
}

// DK in {32, 64, 128, 256}; M in {1, 2, 4, 8, 16, 32} or 0 (= runtime m, padded head sizes; 0, 1 and 32 load a byte at a time);
// WAVES wavefronts per workgroup, OCC = wavefronts per SIMD the register budget must allow.
// Codebook rows of centroid `tid` for the GS subspaces i0 .. i0+GS-1 of one head.
template <int DSUB, int GS>
__device__ __forceinline__ void load_centroid_rows(float (&row)[GS][DSUB], const float *__restrict__ cb_head_c, int i0)
{
#pragma unroll
    for (int g = 0; g < GS; ++g) {
        const float *src = cb_head_c + (int64_t)(i0 + g) * kCentroids * DSUB;
        if constexpr (DSUB % 4 == 0) {
#pragma unroll
            for (int j4 = 0; j4 < DSUB / 4; ++j4) {
                const float4 t4 = reinterpret_cast<const float4 *>(src)[j4];
                row[g][4 * j4] = t4.x;
                row[g][4 * j4 + 1] = t4.y;
                row[g][4 * j4 + 2] = t4.z;
                row[g][4 * j4 + 3] = t4.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < DSUB; ++j)
                row[g][j] = src[j];
        }
    }
}

// Fused step, table-building wavefronts (256 threads): from one pass over the head's codebook rows they compute
//   the table entries  LUT_i[c] = q^(i) . C_i[c]           (Sec. 3.5, fp32)
//   the distances      || k_new^(i) - C_i[c] ||^2          (Sec. 3.4; see step_candidates)
// (us for two steps, a thread per row and fp64 distances / now: 40 x 16 (b,h) x 600 keys, d_k = 64, m = 16 36.6 / 22.8; 60 x 32 x 150, d_k = 128,
// m = 4 97 / 60; 24 x 12 x 1024, d_k = 64, m = 4 18.4 / 17.9; 112 launches of more than 256 (b,h) 0.85 of the time on the geometric mean)
// and leave the table and per (subspace, wavefront) the candidate for the new key's code in LDS.
// `encode`: this workgroup's range holds position L-1 (with several ranges per (b,h) only the last one scores the new key and appends its
// codes; the others build the table alone).
// NB = 2 (two batch entries of one head per workgroup, each with its own 256 table builders): the builders of entry `part` fetch the
// codebook rows of subspaces part*M/2 .. part*M/2 + M/2 - 1 only and from each row compute the table entries and distances of BOTH entries (bh
// and bh + H; their LDS blocks lie lds_stride bytes apart), so that the pair reads the head's codebook once instead of twice.
// The staged words of q and k_new occupy the (not yet used) partial results of the wavefronts.
template <typename FT, int DK, int M, int NB>
__device__ __forceinline__ void step_prologue(const DecodeArgs &a, int bh, int part, int lane, int wave, float *lut_s, float *red_s,
                                              uint2 *near_s, int lds_stride, bool encode)
{
    static_assert(NB == 1 || (NB == 2 && M % 2 == 0), "paired batch entries: even m");
    constexpr int MS = M / NB;            // subspaces this builder group covers
    typedef StepTable<FT, DK, M, MS, NB> Table;
    static_assert(Table::kWords * kDecWaves <= 2 * kDecWaves * (DK + 2), "the staged words fit the partial results of the wavefronts");
    const float *cb_head = a.codebooks + (int64_t)(bh % a.H) * kCentroids * DK;
    const FT *k_new = static_cast<const FT *>(a.k_new);
    const int ibase = part * MS;
    float *stage = reinterpret_cast<float *>(reinterpret_cast<char *>(red_s) + part * lds_stride) + wave * Table::kWords;
    Table table;
    table.request_words(static_cast<const FT *>(a.q), k_new, bh, a.H, ibase, lane);
    table.request_rows(cb_head, ibase, wave, lane);
    table.stage_words(stage, lane);
#pragma unroll
    for (int g0 = 0; g0 < MS; g0 += Table::GS) {
        if (g0 > 0)
            table.request_rows(cb_head, ibase + g0, wave, lane);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            table.group(stage, nb, g0, ibase + g0, wave, lane, reinterpret_cast<float *>(reinterpret_cast<char *>(lut_s) + nb * lds_stride),
                        reinterpret_cast<uint2 *>(reinterpret_cast<char *>(near_s) + nb * lds_stride), encode);
    }
}

// Grouped queries: bh is the key/value head; the G query heads bh*G .. bh*G+G-1 each get their table (lut_s[g][i][c]) from one pass over the
// key/value head's codebook, thread c = centroid c.  Four heads at a time run on the matrix cores in fp32 (v_mfma_f32_4x4x1: A = the heads'
// coordinate, lane % 4 picks the head, B = that coordinate of the lane's centroid, ascending; lane c ends with the four heads' entries of
// centroid c): 8 clocks for what the vector ALU takes 16, and the queries come from LDS, four coordinates a read, where scalar loads had to be
// waited for in the middle of the arithmetic.  Every wavefront stages its own copy of the group's queries and the new key, in the
// (not yet used) partial results; the rows of the copy are four words longer than a query, so that four heads' words lie in different banks.
template <typename FT, int DK, int M, int G>
__device__ __forceinline__ void step_prologue_grouped(const DecodeArgs &a, int bh, int tid, int lane, int wave, float *lut_s, float *red_s,
                                                      uint2 *near_s, bool encode)
{
    constexpr int DSUB = DK / M;
    constexpr int kRegs = G >= 4 ? 128 : 64;
    constexpr int GS0 = kRegs / DSUB > 8 ? 8 : kRegs / DSUB, GS = GS0 < M ? GS0 : M;
    constexpr int HQ = G < 4 ? G : 4;                          // heads of an instruction
    constexpr int kRow = DK + 4;
    static_assert(kDecWaves * (G + 1) * kRow <= 2 * kDecWaves * G * (DK + 2), "the staged words fit the partial results of the wavefronts");
    const float *cb_head = a.codebooks + (int64_t)(bh % a.H) * kCentroids * DK;
    const FT *k_row = static_cast<const FT *>(a.k_new) + (int64_t)bh * DK;
    const FT *q_rows = static_cast<const FT *>(a.q) + (int64_t)bh * G * DK;
    float *stage = red_s + wave * (G + 1) * kRow;             // [G] queries, the new key

    constexpr int kVec = 16 / (int)sizeof(FT);                 // elements of a 16-byte load
    constexpr int kLoads = (G * DK / kVec + kWave - 1) / kWave;
    v4u qv[kLoads], kv = {};
#pragma unroll
    for (int r = 0; r < kLoads; ++r)
        if ((r + 1) * kWave * kVec <= G * DK || r * kWave + lane < G * DK / kVec)
            qv[r] = reinterpret_cast<const v4u *>(q_rows)[r * kWave + lane];
    if (lane < DK / kVec)
        kv = reinterpret_cast<const v4u *>(k_row)[lane];
    float frow[GS][DSUB];
    load_centroid_rows<DSUB, GS>(frow, cb_head + tid * DSUB, 0);
    auto put = [&](float *row, int at, const v4u &v) {
        FT e[kVec];
        __builtin_memcpy(e, &v, sizeof(e));
#pragma unroll
        for (int n = 0; n < kVec; n += 4)
            *reinterpret_cast<v4f *>(row + at + n) = v4f{step_f32<FT>(e[n]), step_f32<FT>(e[n + 1]), step_f32<FT>(e[n + 2]), step_f32<FT>(e[n + 3])};
    };
#pragma unroll
    for (int r = 0; r < kLoads; ++r) {
        const int e = (r * kWave + lane) * kVec;
        if ((r + 1) * kWave * kVec <= G * DK || e < G * DK)
            put(stage + e / DK * kRow, e % DK, qv[r]);
    }
    if (lane < DK / kVec)
        put(stage + G * kRow, lane * kVec, kv);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i0 = 0; i0 < M; i0 += GS) {
        if (i0 > 0)
            load_centroid_rows<DSUB, GS>(frow, cb_head + tid * DSUB, i0);
#pragma unroll
        for (int g = 0; g < GS; ++g) {
            v4f e[G / HQ];
#pragma unroll
            for (int n = 0; n < G / HQ; ++n)
                e[n] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < DSUB; j += 4) {
                v4f x[G / HQ];
#pragma unroll
                for (int n = 0; n < G / HQ; ++n)
                    x[n] = *reinterpret_cast<const v4f *>(stage + (n * HQ + lane % HQ) * kRow + (i0 + g) * DSUB + j);
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int n = 0; n < G / HQ; ++n)
                        e[n] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[n][t], frow[g][j + t], e[n], 0, 0, 0);
            }
#pragma unroll
            for (int n = 0; n < G / HQ; ++n)
#pragma unroll
                for (int hq = 0; hq < HQ; ++hq)
                    lut_s[((n * HQ + hq) * M + i0 + g) * kCentroids + tid] = e[n][hq];
        }
        if (encode) {
            float dist[GS];
#pragma unroll
            for (int g = 0; g < GS; ++g) {
                dist[g] = 0.f;
#pragma unroll
                for (int j = 0; j < DSUB; j += 4) {
                    const v4f k = *reinterpret_cast<const v4f *>(stage + G * kRow + (i0 + g) * DSUB + j);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float diff = k[t] - frow[g][j + t];
                        dist[g] = fmaf(diff, diff, dist[g]);
                    }
                }
            }
            step_candidates<DSUB, GS>(dist, i0, tid, wave, lane, near_s, [&](int g, uint64_t among) { return rows_without_repeats(frow[g], among); },
                                      [&](int g, uint64_t) {
                double d = 0.0;
#pragma unroll
                for (int j = 0; j < DSUB; j += 4) {
                    const v4f k = *reinterpret_cast<const v4f *>(stage + G * kRow + (i0 + g) * DSUB + j);
                    rule_add(d, only_here(k), only_here(v4f{frow[g][j], frow[g][j + 1], frow[g][j + 2], frow[g][j + 3]}));
                }
                return d;
            });
        }
    }
}

// The same on the vector ALU, a multiply-add chain per head: q and k_new are addressed uniformly over the wavefront and become scalar loads
// through the constant address space, which stay out of the in-order vector-memory queue.  Taken for two heads, where the matrix instruction
// has no advantage and two workgroups share a compute unit's memory pipe (8 x 4 key/value heads x 4000 keys, d_k = 128, m = 4: 29.9 us two
// layers, 31.4 with staged queries).  Four and eight heads are ahead on the matrix cores: 340 shapes of four heads of fp16 queries at d_k = 128
// with 16 or 32 coordinates 0.96 of the time on the geometric mean, long contexts of more than 256 workgroups up to 1.01.
template <typename FT, int DK, int M, int G>
__device__ __forceinline__ void step_prologue_heads(const DecodeArgs &a, int bh, int tid, int lane, int wave, float *lut_s, uint2 *near_s,
                                                    bool encode)
{
    constexpr int DSUB = DK / M;
    constexpr int GS0 = 64 / DSUB > 8 ? 8 : 64 / DSUB, GS = GS0 < M ? GS0 : M;
    float frow[GS][DSUB];
    const float *cb_head = a.codebooks + (int64_t)(bh % a.H) * kCentroids * DK;
    const FT *k_row = static_cast<const FT *>(a.k_new) + (int64_t)bh * DK;
    const UniformWords qg = (UniformWords)(reinterpret_cast<uintptr_t>(a.q) + (uintptr_t)bh * G * DK * sizeof(FT));
    const UniformWords kg = (UniformWords)(reinterpret_cast<uintptr_t>(k_row));
#pragma unroll
    for (int i0 = 0; i0 < M; i0 += GS) {
        load_centroid_rows<DSUB, GS>(frow, cb_head + tid * DSUB, i0);
        float dist[GS];
#pragma unroll
        for (int g = 0; g < GS; ++g) {
#pragma unroll
            for (int hq = 0; hq < G; ++hq) {
                float e = 0.f;
#pragma unroll
                for (int j = 0; j < DSUB; ++j)
                    e = fmaf(uniform_elem<FT>(qg, hq * DK + (i0 + g) * DSUB + j), frow[g][j], e);
                lut_s[(hq * M + i0 + g) * kCentroids + tid] = e;
            }
            dist[g] = 0.f;
            if (encode) {
#pragma unroll
                for (int j = 0; j < DSUB; ++j) {
                    const float diff = uniform_elem<FT>(kg, (i0 + g) * DSUB + j) - frow[g][j];
                    dist[g] = fmaf(diff, diff, dist[g]);
                }
            }
        }
        if (encode)
            step_candidates<DSUB, GS>(dist, i0, tid, wave, lane, near_s, [&](int g, uint64_t among) { return rows_without_repeats(frow[g], among); },
                                      [&](int g, uint64_t) {
                UniformWords key = kg;
                asm volatile("" : "+s"(key));        // (as only_here: the key is fetched again)
                double d = 0.0;
#pragma unroll
                for (int j = 0; j < DSUB; j += 4) {
                    v4f k;
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        k[t] = uniform_elem<FT>(key, (i0 + g) * DSUB + j + t);
                    rule_add(d, only_here(k), only_here(v4f{frow[g][j], frow[g][j + 1], frow[g][j + 2], frow[g][j + 3]}));
                }
                return d;
            });
    }
}

// Sums over the rows of a wavefront's partial output (lanes that share lane % LPR, eight coordinates each), written to mine[DK].  A swap of
// lane halves leaves one sum of two coordinates in each half, so each step halves the number of values instead of adding all eight in
// every lane (d_k = 64: 15 instructions, 72 before).
template <int LPR>
__device__ __forceinline__ void fold_rows(float (&acc)[8], float *mine, int lane)
{
    if constexpr (LPR >= 8 && LPR <= 32) {
        float s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[e]), __float_as_uint(acc[e + 4]), false, false);
            s[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
        float *to = mine + 8 * (lane % LPR) + ((lane & 32) ? 4 : 0);
        if constexpr (LPR == 32) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                to[e] = s[e];
            return;
        }
        float t[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(s[e]), __float_as_uint(s[e + 2]), false, false);
            t[e] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
        to += (lane & 16) ? 2 : 0;
        if constexpr (LPR == 16) {
            to[0] = t[0];
            to[1] = t[1];
        } else {
            const bool odd = lane & 8;
            const float own = odd ? t[1] : t[0], other = odd ? t[0] : t[1];
            to[odd ? 1 : 0] = own + dpp_mov<0x128>(other, other);      // row_ror:8 -- lane ^ 8
        }
    } else {
#pragma unroll
        for (int d = 0; d < 8; ++d)
            acc[d] = sum_over_lane_classes<LPR>(acc[d]);
        if (lane < LPR) {
#pragma unroll
            for (int d = 0; d < 8; ++d)
                mine[lane * 8 + d] = acc[d];
        }
    }
}

// Merge of the workgroup's partial results of[WAVES], `stride` words apart (coordinates, reference, sum of weights; DK + 2 words each), by a thread
// per coordinate.  write(sum, reference, sum of weights)
template <int DK, int WAVES, typename Write>
__device__ __forceinline__ void merge_coordinate(const float *of, int stride, int j, Write write)
{
    float mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < WAVES; ++w)
        mx = fmaxf(mx, of[w * stride + DK]);
    const float m_use = (mx == -INFINITY) ? 0.f : mx;
    float o = 0.f, zz = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const float wgt = fast_exp2(of[w * stride + DK] - m_use);
        o = fmaf(wgt, of[w * stride + j], o);
        zz = fmaf(wgt, of[w * stride + DK + 1], zz);
    }
    write(o, mx, zz);
}
// The same for the fused steps of 64 coordinates, whose kernels give the same bits: eight neighbouring lanes take one wavefront's share each and add
// across lanes, one LDS round trip and a dozen lane moves.  12 steps of 12 heads x 1024 keys, m = 2 0.994 of the time; of more than 256 (b,h)
// 1.01.  (Everywhere else the lane moves cost more than the reads: fused steps of 128 coordinates 1.02 of the time, tables given 1.02 to 1.03, at
// d_k = 256 and short contexts 1.05.)
__device__ __forceinline__ float sum_octet(float v)
{
    v += dpp_mov<0xB1>(v, v);
    v += dpp_mov<0x4E>(v, v);
    return v + dpp_mov<0x141>(v, v);
}
template <typename Write>
__device__ __forceinline__ void merge_octets(const float *red_s, int tid, Write write)
{
    constexpr int kRow = 64 + 2;
    const float *of = red_s + tid % 8 * kRow;
    const float mw = of[64], zw = of[65], o = of[tid / 8];
    float mx = fmaxf(mw, dpp_mov<0xB1>(mw, mw));
    mx = fmaxf(mx, dpp_mov<0x4E>(mx, mx));
    mx = fmaxf(mx, dpp_mov<0x141>(mx, mx));
    const float wgt = fast_exp2(mw - ((mx == -INFINITY) ? 0.f : mx));
    const float zz = sum_octet(wgt * zw), sum = sum_octet(wgt * o);
    if (tid % 8 == 0)
        write(sum, mx, zz);
}

// FT = void: the table comes from memory (lookat_attend_decode).  FT = __half / float: fused
// decode step (lookat_decode_step): q and the new key have type FT, the table is computed and
// the new key encoded by the workgroup itself (WAVES = 8; see the roles below).
// G > 1: grouped-query attention: the workgroup's (b,h) is a KEY/VALUE head shared by G query heads,
// whose tables (contiguous in memory) are all staged in LDS; codes and values are streamed once.
// PF: tiles of a wavefront requested before anything else is done (1, or more for the fused step,
// whose table build and key encoding would otherwise leave the memory pipe idle for microseconds).
// NB = 2 (fused step only): the workgroup has 2 x WAVES wavefronts and serves TWO batch entries of one head,
// (b, h) and (b + 1, h).  Each half is a complete copy of the roles above with its own LDS block; the only
// thing shared is the codebook, of which each half's table builders fetch half the subspaces and compute
// both entries' table rows and distances.  The head's codebook then crosses from L2 to the compute units
// once per pair instead of once per (b,h).  Both halves execute the same barriers (same L, same ranges).
// PAD (tables given, ungrouped): the head size is a.d_k < DK, a multiple of 8; lanes past the end of a row repeat its last
// 16 bytes and their sums are not written.
template <int DK, int M, int WAVES, int OCC, typename FT = void, int G = 1, int PF = 1, int NB = 1, bool PAD = false>
__global__ __launch_bounds__(WAVES *NB *kWave, OCC) void decode_split_kernel(LOOKAT_DECODE_HEAD_PARAMS,
                                                                             const DecodeLate late)
{
    const DecodeArgs a = rebuild_args(p_BH, p_splits, p_H, p_table, p_codes, p_values, p_code_stride, p_value_stride,
                                      p_L, p_kps, p_scale_log2e, late, !std::is_void<FT>::value);
    constexpr bool FUSED = !std::is_void<FT>::value;
    static_assert(!FUSED || (WAVES == 2 * kDecWaves && M != 0), "fused step: 512 threads, compile-time m");
    static_assert(NB == 1 || (NB == 2 && FUSED && G == 1), "paired batch entries: ungrouped fused step only");
    // Fused step: the eight wavefronts take two roles until the table exists.  The first four
    // (256 threads, thread c = centroid c) fetch the codebook rows, build the table and encode the
    // new key (step_prologue) and request no tile before that is done; the other four request
    // their tiles at once and wait.  A wavefront issues in order, and under a saturated memory
    // pipe a tile request is accepted only as fast as data leaves the pipe: a wavefront that has
    // tile requests queued ahead of its table arithmetic starts that arithmetic microseconds late.
    static_assert(G == 1 || M != 0, "grouped queries: compile-time m");
    static_assert(!PAD || (!FUSED && G == 1), "padded head sizes: tables given, ungrouped");
    const int dk = PAD ? a.d_k : DK;
    constexpr int LPR = DK / 8;            // lanes per value row (16 bytes per lane)
    constexpr int RPL = kWave / LPR;       // value rows covered by one wave-wide load
    constexpr int NLD = kTile / RPL;       // wave-wide loads per tile (= LPR)
    constexpr bool MM = (G >= 4 && DK == 128 && M != 0);   // weighted value sum on the matrix cores
    // loads kept in flight together: 8 KB of a tile; the whole 16 KB tile where the matrix cores take the value sum
    // (its accumulators are half the size, and a second request round in the middle of a tile is a second
    // exposed round trip at two wavefronts per SIMD)
    constexpr int CH = MM ? NLD : (NLD < 8 ? NLD : 8);
    constexpr int NT = WAVES * kWave;

    extern __shared__ __align__(16) float smem_all[];
    // which of the workgroup's NB batch entries this wavefront belongs to (scalar), and its LDS block
    const int hf = (NB == 1) ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / (WAVES * kWave));
    constexpr int kHalfBytes = (NB == 1) ? 0 : (int)step_pair_lds_bytes(M, DK);
    float *smem = reinterpret_cast<float *>(reinterpret_cast<char *>(smem_all) + hf * kHalfBytes);
    float *lut_s = smem;                                   // [G][m][256]
    float *red_s = smem + G * (M ? M : a.m) * kCentroids;  // [WAVES][G][DK + 2]
    uint2 *near_s = reinterpret_cast<uint2 *>(red_s + WAVES * G * (DK + 2));   // fused step: see step_candidates

    int bh, split;
    if constexpr (NB == 1) {
        if (!map_block(a, bh, split))
            return;
    } else {
        // a.BH / 2 pairs are dealt to the workgroups as (b,h) pairs are otherwise: pair p = head p % H of the
        // batch entries 2*(p / H) and 2*(p / H) + 1
        int pair;
        if (!map_block_n(a, a.BH / 2, pair, split))
            return;
        bh = 2 * (pair / a.H) * a.H + pair % a.H + hf * a.H;
    }
    const int m = M ? M : a.m;
    const int tid = (NB == 1) ? (int)threadIdx.x : (int)threadIdx.x - hf * (WAVES * kWave);   // within the half
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);   // in a scalar register: role branches are scalar branches
    const bool builds_table = FUSED && wave < kDecWaves;

    const uint32_t k0 = (uint32_t)split * (uint32_t)a.keys_per_split;
    const uint32_t k1 = (k0 + a.keys_per_split < a.L) ? (uint32_t)(k0 + a.keys_per_split) : (uint32_t)a.L;
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(a.values + (int64_t)bh * a.value_stride, k1 * (uint32_t)(dk * 2));
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(a.codes + (int64_t)bh * a.code_stride, k1 * (uint32_t)m);

    // Everything the first tile needs is requested before anything is waited for, in the
    // order it is needed (loads return in order, so each wait below covers only what precedes):
    // 1) this thread's slice of the table (staged through registers: the wait before the
    //    barrier then covers the table alone, not the value rows behind it);
    const float4 *lut_g = reinterpret_cast<const float4 *>(a.lut + (int64_t)bh * G * m * kCentroids);
    constexpr int kLutRegs = M ? (G * M * (kCentroids / 4) + NT - 1) / NT : 1;
    // (tables of more than one 16-byte piece per thread are copied up front instead: a staging
    // array of several registers ends up in scratch memory)
    constexpr bool STAGED = (M != 0 && !FUSED && kLutRegs == 1);
    float4 lut_r[STAGED ? kLutRegs : 1];
    if constexpr (M != 0 && !FUSED && !STAGED) {
        float4 *s4 = reinterpret_cast<float4 *>(lut_s);
        for (int x = tid; x < G * M * (kCentroids / 4); x += NT)
            s4[x] = lut_g[x];
    }
    if constexpr (STAGED) {
#pragma unroll
        for (int x = 0; x < kLutRegs; ++x)
            if ((x + 1) * NT <= G * M * (kCentroids / 4) || tid + x * NT < G * M * (kCentroids / 4))
                lut_r[x] = lut_g[tid + x * NT];
            else
                lut_r[x] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // 2) the codes of the wave's first tile;  3) its value rows.
    // Lane (rowin, sub) holds the value rows RPL*j + rowin, j = 0..NLD-1, of a tile.  It scores
    // the key RPL*sub + rowin, so the NLD weights a lane needs sit in its own group of LPR
    // consecutive lanes and are fetched with DPP moves instead of LDS shuffles.
    const int sub = lane % LPR;      // which 8-coordinate slice of the value row
    const int rowin = lane / LPR;    // which row of a wave-wide load
    const uint32_t kofs = (uint32_t)(RPL * sub + rowin);
    const uint32_t row_bytes = (uint32_t)dk * 2;
    const uint32_t lane_off = PAD ? (uint32_t)rowin * row_bytes + (uint32_t)(sub < dk / 8 ? sub : dk / 8 - 1) * 16 : (uint32_t)lane * 16;
    uint32_t kb = k0 + (uint32_t)wave * kTile;
    CodesOf<M> kcs[PF];
    v4u vs[PF][CH];
    // Unconditional within its role: requests past the range return zero (descriptor bounds).  Behind a
    // per-tile branch the compiler could no longer count how many requests follow a given one, and every
    // wait would become a wait for all of them.  (A macro: a lambda that captures the register arrays
    // sends them through scratch memory.)
#define LOOKAT_REQUEST_FIRST_TILES()                                                                   \
    _Pragma("unroll") for (int t = 0; t < PF; ++t)                                                     \
    {                                                                                                  \
        const uint32_t kbt = kb + (uint32_t)t * NT;                                                    \
        if constexpr (M != 0)                                                                          \
            kcs[t].load(rc, (kbt + kofs) * M);                                                         \
        else                                                                                           \
            kcs[t].load(rc, (kbt + kofs) * m, m);                                                      \
        __builtin_amdgcn_sched_barrier(0); /* keep the request order: codes before value rows */       \
        if constexpr (PAD)                                                                             \
            load_rows_padded<DK, CH>(vs[t], rv, kbt, 0, lane_off, row_bytes);                          \
        else                                                                                           \
            load_rows<DK, CH>(vs[t], rv, kbt, 0, lane);                                                \
    }
    if constexpr (FUSED) {
        // one branch per role: the table builders' codebook rows and the streamers' tiles then never
        // hold registers at the same time
        if (builds_table) {
            // issue ahead of the streamers that share the SIMD: the codebook requests must enter the
            // compute unit's memory queue before the tile requests fill it
            __builtin_amdgcn_s_setprio(3);
            if constexpr (G == 1) {
                // (paired entries: the LDS blocks and the (b,h) index are handed over as entry 0's)
                auto first = [&](auto *p) { return reinterpret_cast<decltype(p)>(reinterpret_cast<char *>(p) - hf * kHalfBytes); };
                step_prologue<FT, DK, M, NB>(a, bh - hf * a.H, hf, lane, wave, first(lut_s), first(red_s), first(near_s), kHalfBytes,
                                             k1 == (uint32_t)a.L);
            } else if constexpr (G == 2) {
                step_prologue_heads<FT, DK, M, G>(a, bh, tid, lane, wave, lut_s, near_s, k1 == (uint32_t)a.L);
            } else {
                step_prologue_grouped<FT, DK, M, G>(a, bh, tid, lane, wave, lut_s, red_s, near_s, k1 == (uint32_t)a.L);
            }
            __builtin_amdgcn_s_setprio(0);
        } else {
            LOOKAT_REQUEST_FIRST_TILES()
        }
    } else {
        LOOKAT_REQUEST_FIRST_TILES()
    }
    CodesOf<M> &kc = kcs[0];
    v4u(&v)[CH] = vs[0];
    if constexpr (!FUSED) {
        float4 *s4 = reinterpret_cast<float4 *>(lut_s);
        if constexpr (STAGED) {
#pragma unroll
            for (int x = 0; x < kLutRegs; ++x)
                if ((x + 1) * NT <= G * M * (kCentroids / 4) || tid + x * NT < G * M * (kCentroids / 4))
                    s4[tid + x * NT] = lut_r[x];
        } else if constexpr (M == 0) {
            for (int x = tid; x < m * (kCentroids / 4); x += NT)
                s4[x] = lut_g[x];
        }
    }
    __syncthreads();   // table (and, fused, the per-wave argmins) complete in LDS; value rows stay in flight
    if constexpr (FUSED) {
        if (builds_table) {
            LOOKAT_REQUEST_FIRST_TILES()
        }
    }
#undef LOOKAT_REQUEST_FIRST_TILES

    // The newest key (row L-1) was encoded by this workgroup a moment ago; the cached row may be stale.  Ungrouped: the wavefront that scores it
    // picks its codes when it gets to that tile.  Grouped: before or after its first tile, which keeps the loop free of the rule's loads (8 x 4 key/value
    // heads x 32768 keys, group 8, d_k = 128, m = 8: 50.9 us, 52.3 with the test in it;
    // ungrouped the first tile would wait: 32 x 12 x 1024 keys, m = 4, twelve steps 130.6 us, 128.6 as it is).
    auto new_codes = [&](uint32_t(&fresh)[code_words(M)]) {
        if constexpr (FUSED)
            step_new_codes<FT, DK / M, M>(fresh, near_s, a.codebooks + (int64_t)(bh % a.H) * kCentroids * DK,
                                          static_cast<const FT *>(a.k_new) + (int64_t)bh * DK,
                                          a.codes_w + (int64_t)bh * a.code_stride + (a.L - 1) * M, lane);
    };
    uint32_t fresh_early[code_words(M)] = {};
    const uint32_t first_tile = kb;
    const bool scores_new = FUSED && G > 1 && k1 == (uint32_t)a.L && k0 < k1 && (k1 - 1 - k0) / kTile % WAVES == (uint32_t)wave;
    // (Two heads at d_k = 128 have no registers left for that; four at d_k = 64 would take 132, and 128 are what two workgroups share on a compute
    // unit: 8 x 57 key/value heads x 419 keys, m = 4 13.7 us so, 10.4 with the codes before the first tile.)
    constexpr bool kAfterFirst = G == 8 || (G == 4) == (DK == 128);
    if constexpr (FUSED && G > 1) {
        if (scores_new && (!kAfterFirst || k1 - 1 - kb < (uint32_t)kTile))
            new_codes(fresh_early);
    }
    auto patch = [&](CodesOf<M> &codes, uint32_t tile, uint32_t key) {
        if constexpr (FUSED && G > 1) {
#pragma unroll
            for (int w = 0; w < code_words(M); ++w)
                codes.w[w] = key == (uint32_t)(a.L - 1) ? fresh_early[w] : codes.w[w];
        } else if constexpr (FUSED) {
            if ((uint32_t)(a.L - 1) - tile < (uint32_t)kTile) {
                uint32_t fresh[code_words(M)];
                new_codes(fresh);
#pragma unroll
                for (int w = 0; w < code_words(M); ++w)
                    codes.w[w] = key == (uint32_t)(a.L - 1) ? fresh[w] : codes.w[w];
            }
        }
    };

    // First tile (requested above), then the wave's remaining tiles: request, consume.  Tiles
    // are requested only if they exist (a load past the range would return zero but still
    // occupy the address pipeline), and a tile's registers are dead at the loop back-edge.
    SoftmaxState<G> st;
    // Matrix-core value sum (see consume_tile): accumulators, and the wavefront's weight staging rows, which
    // occupy its own slice of the reduction buffer (unused until the epilogue; 2 KB of its G x (DK + 2) floats).
    v4f accm[MM ? 8 : 1];
#pragma unroll
    for (int e = 0; e < (MM ? 8 : 1); ++e)
        accm[e] = v4f{0.f, 0.f, 0.f, 0.f};
    uint32_t pstage = 0;
    if constexpr (MM) {
        static_assert(G * (DK + 2) * sizeof(float) >= 2048, "the staging rows fit the wavefront's reduction slice");
        pstage = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)(red_s + wave * G * (DK + 2));
        // columns no query head owns (G = 4: 8..15) must read as zero in every tile
        *reinterpret_cast<__attribute__((address_space(3))) v4f *>(pstage + (uint32_t)lane * 32u) = v4f{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<__attribute__((address_space(3))) v4f *>(pstage + (uint32_t)lane * 32u + 16u) = v4f{0.f, 0.f, 0.f, 0.f};
    }
    if (kb < k1) {
        consume_tile<DK, M, CH, G, MM, PAD, true>(a, st, kc, v, lut_s, rc, rv, bh, kb, k1, kofs, lane, m, patch, accm, pstage,
                                             lane_off, row_bytes);
        if constexpr (FUSED && G > 1 && kAfterFirst) {
            if (scores_new && k1 - 1 - first_tile >= (uint32_t)kTile)
                new_codes(fresh_early);
        }
#pragma unroll
        for (int t = 1; t < PF; ++t) {   // the other tiles requested at the start
            kb += NT;
            if (kb < k1)
                consume_tile<DK, M, CH, G, MM, PAD>(a, st, kcs[t], vs[t], lut_s, rc, rv, bh, kb, k1, kofs, lane, m, patch, accm,
                                                      pstage, lane_off, row_bytes);
        }
        for (kb += NT; kb < k1; kb += NT) {
            if constexpr (M != 0)
                kc.load(rc, (kb + kofs) * M);
            else
                kc.load(rc, (kb + kofs) * m, m);
            __builtin_amdgcn_sched_barrier(0);   // request order = need order: codes before value rows
            if constexpr (PAD)
                load_rows_padded<DK, CH>(v, rv, kb, 0, lane_off, row_bytes);
            else
                load_rows<DK, CH>(v, rv, kb, 0, lane);
            consume_tile<DK, M, CH, G, MM, PAD>(a, st, kc, v, lut_s, rc, rv, bh, kb, k1, kofs, lane, m, patch, accm, pstage,
                                             lane_off, row_bytes);
        }
    }

    // ---- fold the rows of the wave, then the waves of the workgroup ----
    if constexpr (MM) {
        // lane (q, n): accm[e][r] = coordinate 8*(4q + r) + e of column n; columns n < G hold the fp16 part of
        // the weights, columns G + n the scaled remainder: combine, and lanes n < G hand over head n's sum
        const int n = lane & 15, q = lane >> 4;
        float *mine_n = red_s + (wave * G + (n & (G - 1))) * (DK + 2);
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float lo = dpp_mov<0x100 + G>(accm[e][r], accm[e][r]);   // row_shl:G -- lane n + G of the row
                const float o = fmaf(lo, 1.f / kLoScale, accm[e][r]);
                if (n < G)
                    mine_n[8 * (4 * q + r) + e] = o;
            }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        float *mine = red_s + (wave * G + g) * (DK + 2);
        if constexpr (!MM)
            fold_rows<LPR>(st.acc[g], mine, lane);
        st.z[g] = wave_sum(st.z[g]);
        if (lane == 0) {
            mine[DK] = st.m_run[g];
            mine[DK + 1] = st.z[g];
        }
    }
    __syncthreads();

    auto write_to = [&](int g, int j) {   // query head of the group, output coordinate
        return [&, g, j](float o, float mx, float zz) {
            if (a.splits == 1) {
                a.out[((int64_t)bh * G + g) * dk + j] = o / zz;
            } else {
                float *dst = a.part + (((int64_t)bh * G + g) * a.splits + split) * (dk + 2);
                dst[j] = o;
                if (j == 0) {
                    dst[dk] = mx;
                    dst[dk + 1] = zz;
                }
            }
        };
    };
    if constexpr (FUSED && G == 1 && DK == 64) {
        merge_octets(red_s, tid, write_to(0, tid / 8));
        return;
    }
    auto finish = [&](int x) {
        const int g = x / DK, j = x % DK;
        if (!PAD || j < dk)
            merge_coordinate<DK, WAVES>(red_s + g * (DK + 2), G * (DK + 2), j, write_to(g, j));
    };
    if constexpr (G * DK <= NT) {
        if (tid < G * DK)
            finish(tid);
    } else {
        for (int x = tid; x < G * DK; x += NT)
            finish(x);
    }
}

// ---- the fused step where every workgroup has a compute unit to itself ----------------------------------------
// Up to 32 workgroups on a die: one sequence or a few, whole or cut into ranges.  A launch is then a chain of latencies, and what a compute unit's
// memory pipe takes (a wave-wide load of a kilobyte every 16 clocks) and when.  Sixteen wavefronts: the first eight build the table, 0-3 the first
// half of the subspaces, 4-7 the second, two on a SIMD so that one's arithmetic fills the other's latencies, and end; the others stream the tiles,
// as in decode_split_kernel, from the start.  The builders are the first wavefronts of the workgroup, which start first, and run at raised
// priority until they end, so that their requests enter the pipe first.  (With eight wavefronts doing both jobs the arithmetic waits
// until the pipe has accepted the wavefront's tiles: table complete at 5000 clocks at d_k = 64, 15500 at 128, of 9200 and 21800.)  What has to
// be known before the first request travels in the preloaded arguments (the (b,h) count, ranges and heads in one word: none exceeds 256).
//   Measured against the roles of decode_split_kernel with a thread per centroid row and fp64 distances (us per launch): 12 (b,h), d_k = 64, m = 2:
// 1 key 5.6 / 4.0, 1024 keys 6.3 / 5.2, 8192 19.8 / 18.3; d_k = 128, m = 8: 8.2 / 5.0, 10.6 / 7.8, 39.6 / 36.2; 32 x 8003 keys in ranges 16.6 / 15.6
// with the merge; 176 calls of 4 to 160 (b,h) x 700 to 32000 keys, cut or not, 0.85 of the time on the geometric mean.  (The builders as the last
// wavefronts, and a candidate's distance and number in two places: up to 11% longer, 1024 keys 5.4 and 8.3.)
struct LoneLate {
    float *part;
    float *out;
    float scale_log2e;
};
constexpr size_t lone_lds_bytes(int m, int d_k)
{
    return ((size_t)m * kCentroids + (size_t)(2 * kDecWaves) * (d_k + 2)) * sizeof(float) + step_encoder_bytes(m);
}

template <typename FT, int DK, int M>
__global__ __launch_bounds__(4 * kDecThreads, 4) void decode_step_lone_kernel(const float *p_codebooks, const FT *p_q, const FT *p_k_new,
                                                                              uint8_t *p_codes, const __half *p_values,
                                                                              uint32_t p_counts, uint32_t p_L,
                                                                              uint32_t p_code_stride, uint32_t p_value_stride,
                                                                              const LoneLate late)
{
    constexpr int WAVES = 2 * kDecWaves, NT = WAVES * kWave;   // that stream
    constexpr int MS = M / 2;                                  // subspaces of a builder
    constexpr int LPR = DK / 8, RPL = kWave / LPR, CH = LPR;   // (see decode_split_kernel; a tile's value rows are requested whole)
    typedef StepTable<FT, DK, M, MS, 1> Table;
    static_assert(Table::GS == MS && Table::kWords == DK, "a builder's rows are held at once");

    extern __shared__ __align__(16) float smem_all[];
    float *lut_s = smem_all;                                       // [M][256]
    float *red_s = lut_s + M * kCentroids;                         // [WAVES][DK + 2]
    uint2 *near_s = reinterpret_cast<uint2 *>(red_s + WAVES * (DK + 2));       // see step_candidates

    DecodeArgs a = {};
    a.BH = (int)(p_counts & 0x1ffu);
    a.splits = (int)(p_counts >> 9 & 0x3fu);
    a.H = (int)(p_counts >> 15);
    int bh, split;
    if (!map_block(a, bh, split))
        return;
    const int lane = (int)threadIdx.x & (kWave - 1);
    const int any_wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    uint32_t k0 = 0, k1 = p_L;
    if (a.splits > 1) {      // ranges of whole tiles
        const uint32_t kps = ((p_L + kTile - 1) / kTile + (uint32_t)a.splits - 1) / (uint32_t)a.splits * kTile;
        k0 = (uint32_t)split * kps;
        k1 = k0 + kps < p_L ? k0 + kps : p_L;
    }

    // bh mod H (both at most 256: the quotient of the rounded division is exact)
    const int h = bh - (int)(((float)bh + 0.5f) * __builtin_amdgcn_rcpf((float)a.H)) * a.H;
    const float *cb_head = p_codebooks + (int64_t)h * kCentroids * DK;

    if (any_wave < WAVES) {  // ---- table and candidates ----
        __builtin_amdgcn_s_setprio(3);
        const int builder = any_wave;
        const int i0 = builder / kDecWaves * MS, quarter = builder & (kDecWaves - 1);
        float *stage = red_s + builder * Table::kWords;      // (the partial results are not in use yet)
        Table table;
        table.request_words(p_q, p_k_new, bh, 0, i0, lane);
        __builtin_amdgcn_sched_barrier(0);
        table.request_rows(cb_head, i0, quarter, lane);
        __builtin_amdgcn_sched_barrier(0);
        table.stage_words(stage, lane);
        table.group(stage, 0, 0, i0, quarter, lane, lut_s, near_s, k1 == p_L);
        __syncthreads();
        return;
    }

    // ---- the wavefront's tiles ----
    const int wave = any_wave - WAVES, tid = (int)threadIdx.x - NT;
    a.L = p_L;
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(p_values + (int64_t)bh * p_value_stride, k1 * (uint32_t)(DK * 2));
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(p_codes + (int64_t)bh * p_code_stride, k1 * (uint32_t)M);
    const int sub = lane % LPR, rowin = lane / LPR;
    const uint32_t kofs = (uint32_t)(RPL * sub + rowin);
    uint32_t kb = k0 + (uint32_t)wave * kTile;
    SoftmaxState<1> st;
    v4f accm[1] = {};
    // The new key's codes (see decode_split_kernel): before the first tile at d_k = 64, where all of a short context's tiles are there by then, with
    // the last tile otherwise (twelve steps of 12 heads x 1024 keys, d_k = 64, m = 2: 66.6 us, 68.5 the other way round; 32 heads x 8003 keys,
    // d_k = 128, m = 8: 15.4, 15.9).
    uint32_t fresh[code_words(M)] = {};
    auto new_codes = [&] {
        step_new_codes<FT, DK / M, M>(fresh, near_s, cb_head, p_k_new + (int64_t)bh * DK,
                                      p_codes + (int64_t)bh * p_code_stride + (int64_t)(p_L - 1) * M, lane);
    };
    auto new_key = [&](CodesOf<M> &codes, uint32_t tile, uint32_t key) {
        if constexpr (DK != 64) {
            if (p_L - 1 - tile < (uint32_t)kTile)
                new_codes();
        }
#pragma unroll
        for (int w = 0; w < code_words(M); ++w)
            codes.w[w] = key == p_L - 1 ? fresh[w] : codes.w[w];
    };
#define LOOKAT_LONE_TILE(PATCH_, FIRST_, KC_, V_, ...)                                                                    \
    consume_tile<DK, M, CH, 1, false, false, FIRST_>(a, st, KC_, V_, lut_s, rc, rv, bh, kb, k1, kofs, lane, M, PATCH_, accm, 0, 0, 0, ##__VA_ARGS__)
    if constexpr (DK == 64) {
        // two tiles requested at once, then always the next one while one is consumed
        CodesOf<M> kcs[2];
        v4u vs[2][CH];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t kbt = kb + (uint32_t)t * NT;
            kcs[t].load(rc, (kbt + kofs) * M);
            __builtin_amdgcn_sched_barrier(0);
            load_rows<DK, CH>(vs[t], rv, kbt, 0, lane);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();   // table and candidates complete in LDS; value rows stay in flight
        a.scale_log2e = late.scale_log2e;
        if (k1 == p_L && k0 < k1 && (k1 - 1 - k0) / kTile % WAVES == (uint32_t)wave)
            new_codes();
        if (kb < k1) {
            LOOKAT_LONE_TILE(new_key, true, kcs[0], vs[0]);
            for (kb += NT; kb < k1; kb += NT) {
                const CodesOf<M> kc = kcs[1];
#pragma unroll
                for (int j = 0; j < CH; ++j)
                    vs[0][j] = vs[1][j];
                if (kb + NT < k1) {
                    kcs[1].load(rc, (kb + NT + kofs) * M);
                    load_rows<DK, CH>(vs[1], rv, kb + NT, 0, lane);
                }
                __builtin_amdgcn_sched_barrier(0);
                LOOKAT_LONE_TILE(new_key, false, kc, vs[0]);
            }
        }
    } else {
        // one tile in registers; each half is requested again for the next tile as soon as it has been used
        CodesOf<M> kc;
        v4u v[CH];
        kc.load(rc, (kb + kofs) * M);
        __builtin_amdgcn_sched_barrier(0);
        load_rows<DK, CH>(v, rv, kb, 0, lane);
        __syncthreads();   // table and candidates complete in LDS; value rows stay in flight
        a.scale_log2e = late.scale_log2e;
        for (; kb + NT < k1; kb += NT) {      // (position L-1 is in a wavefront's last tile)
            CodesOf<M> next;
            LOOKAT_LONE_TILE(NothingNew(), false, kc, v, [&](int n) {
                if (n == 0)
                    next.load(rc, (kb + NT + kofs) * M);
                load_rows<DK, 8>(reinterpret_cast<v4u(&)[8]>(v[n]), rv, kb + NT, n, lane);
            });
            kc = next;
        }
        if (kb < k1)
            LOOKAT_LONE_TILE(new_key, false, kc, v);
    }
#undef LOOKAT_LONE_TILE

    float *mine = red_s + wave * (DK + 2);
    fold_rows<LPR>(st.acc[0], mine, lane);
    st.z[0] = wave_sum(st.z[0]);
    if (lane == 0) {
        mine[DK] = st.m_run[0];
        mine[DK + 1] = st.z[0];
    }
    __syncthreads();
    auto write_to = [&](int j) {
        return [&, j](float o, float mx, float zz) {
            if (a.splits == 1) {
                late.out[(int64_t)bh * DK + j] = o / zz;
            } else {
                float *dst = late.part + ((int64_t)bh * a.splits + split) * (DK + 2);
                dst[j] = o;
                if (j == 0) {
                    dst[DK] = mx;
                    dst[DK + 1] = zz;
                }
            }
        };
    };
    if constexpr (DK == 64)
        merge_octets(red_s, tid, write_to(tid / 8));
    else if (tid < DK)
        merge_coordinate<DK, WAVES>(red_s, DK + 2, tid, write_to(tid));
}

// Merge of the split ranges: M* = max_s M_s, out = sum_s 2^(M_s-M*) o_s / sum_s 2^(M_s-M*) Z_s.
// An empty range carries (M=-inf, Z=0, o=0) and gets weight 0.
// The ranges are taken eight at a time with all of a group's loads issued before the first is used: a loop
// that loads and uses one range per iteration pays one memory round trip per range (8 ranges: 5.2 us for a
// kernel that moves 130 floats per range).  Up to eight ranges the sums are formed exactly as a plain
// ascending loop would; beyond, the running sums are rescaled when a later group raises the maximum.
//   grid = BH, block = 256 (threads >= d_k idle)
__global__ __launch_bounds__(kDecThreads) void decode_combine_kernel(const float *__restrict__ part,
                                                                     float *__restrict__ out, int splits, int d_k)
{
    constexpr int GR = 8;
    const int bh = blockIdx.x;
    const int tid = threadIdx.x;
    if (tid >= d_k)
        return;
    const float *p = part + (int64_t)bh * splits * (d_k + 2);
    float mx = -INFINITY, o = 0.f, z = 0.f;
    for (int s0 = 0; s0 < splits; s0 += GR) {
        float mv[GR], zv[GR], ov[GR];
#pragma unroll
        for (int j = 0; j < GR; ++j) {
            const bool live = s0 + j < splits;
            const float *ps = p + (int64_t)(live ? s0 + j : s0) * (d_k + 2);
            const float m_ = ps[d_k], z_ = ps[d_k + 1], o_ = ps[tid];
            mv[j] = live ? m_ : -INFINITY;
            zv[j] = live ? z_ : 0.f;
            ov[j] = live ? o_ : 0.f;
        }
        float gm = mx;
#pragma unroll
        for (int j = 0; j < GR; ++j)
            gm = fmaxf(gm, mv[j]);
        const float m_use = (gm == -INFINITY) ? 0.f : gm;
        const float keep = fast_exp2(mx - m_use);     // 0 for the first group (mx = -inf), 1 when the maximum stays
        o *= keep;
        z *= keep;
#pragma unroll
        for (int j = 0; j < GR; ++j) {
            const float w = fast_exp2(mv[j] - m_use);
            o = fmaf(w, ov[j], o);
            z = fmaf(w, zv[j], z);
        }
        mx = gm;
    }
    out[(int64_t)bh * d_k + tid] = o / z;
}

static int64_t round_up(int64_t x, int64_t q) { return (x + q - 1) / q * q; }

// Ranges of at least 2048 keys, and no more workgroups than compute units.
static int base_splits(const lookat_shape *s, int64_t L)
{
    int64_t want = 256 / ((int64_t)s->B * s->H);
    const int64_t cap = (L + 2047) / 2048;
    want = want < cap ? want : cap;
    return (int)(want < 1 ? 1 : want);
}
static size_t splits_bytes(const lookat_shape *s, int64_t S)
{
    return S == 1 ? 0 : (size_t)s->B * s->H * S * (s->d_k + 2) * sizeof(float);
}
// Predicted us of a launch with S ranges per (b,h).  All ranges of a (b,h) run on one die (map_block_n), so the die with the
// most (b,h) decides: its n workgroups go evenly to its 32 compute units.  A workgroup streams its range at 54 KB/us while few
// share the memory, 54 - 0.11 w with w workgroups, and no faster than its part of the chip's 7.9 w / (w + 17) MB/us or of a die's
// 965 KB/us; where some compute units hold one workgroup more than the rest, those stream their last range alone.  Each round of
// workgroups costs its table or codebook (about 0.9 us at d_k = 128), and more than one range costs the merge launch.
static double splits_us(const lookat_shape *s, int64_t L, int64_t S)
{
    constexpr double kPeak = 7.92e6, kHalf = 17.0, kOne = 53.8e3, kDie = 965e3, kStart = 7.65, kMerge = 2.1;
    const int64_t BH = (int64_t)s->B * s->H;
    const double range = (double)round_up((L + S - 1) / S, kTile) * (2.0 * s->d_k + s->m);   // bytes
    const int64_t n = (BH + kXcds - 1) / kXcds * S;
    const int64_t rounds = (n + 31) / 32, rest = n - 32 * (rounds - 1);
    const int64_t dies = BH < kXcds ? BH : kXcds, fullest = BH < kXcds ? BH : (BH % kXcds ? BH % kXcds : kXcds);
    auto rate = [&](double w, double on_a_die) {
        double r = kOne - 109.0 * w;
        r = r < kPeak / (w + kHalf) ? r : kPeak / (w + kHalf);
        return r < kDie / on_a_die ? r : kDie / on_a_die;
    };
    return kStart + (double)(rounds - 1) * (range / rate(32.0 * (double)dies, 32.0) + 0.88 * s->d_k / 128.0) +
           range / rate((double)(rest * fullest), (double)rest) + (S > 1 ? kMerge : 0.0);
}
// Ranges per (b,h) when the caller leaves the choice to the library: base_splits, unless another count is predicted to take
// 4% less time (and 1 us less, where that means a second launch), then the count with the least; `workspace`: a caller that
// brings less than that needs gets the best count that it holds, but no less than base_splits.
// Measured at 28 numbers of (b,h) from 1 to 520, 600 to 32768 keys and nine (d_k, m), fused and not: 0.86 of the time of
// base_splits on the geometric mean, 3% off the best of ten counts; two launches in a thousand more than 3% slower than
// base_splits.  us per fused call, base / taken [ranges], d_k = 128, m = 8: 1 x 8192 17.1 / 11.4 [16]; 1 x 32768 18.1 / 14.6 [24];
// 12 x 4096 18.4 / 12.1 [8]; 20 x 32768 46.4 / 33.7 [8]; 32 x 2048 17.4 / 13.5 [4]; 264 x 8192 126 / 106 [6].  A model that dealt the
// workgroups evenly to 256 compute units took 128 ranges for 1 x 32768 (37.4 us), 12 for 20 x 8192 (21.5; 8: 14.7) and one for
// 80 x 4096 at d_k = 64 (15.9; 2: 13.0).
static int auto_splits(const lookat_shape *s, int64_t L, size_t workspace = SIZE_MAX)
{
    const int64_t BH = (int64_t)s->B * s->H;
    if (BH > 128 && BH <= 256)
        return 1;                      // one workgroup per compute unit, and too few for a second round
    static const int counts[] = {2, 3, 4, 6, 8, 12, 16, 24, 32};
    const int base = base_splits(s, L);
    const double base_us = splits_us(s, L, base);
    auto choose = [&](int low, size_t bytes) {
        int best = base;
        double best_us = 0.96 * base_us - (base == 1 ? 1.0 : 0.0);
        for (int S : counts) {
            if (L < (int64_t)S * 256 || BH * S > 4096)
                break;
            if (S < low || splits_bytes(s, S) > bytes)
                continue;
            const double us = splits_us(s, L, S);
            if (us < best_us) {
                best = S;
                best_us = us;
            }
        }
        return best;
    };
    const int S = choose(2, SIZE_MAX);
    return splits_bytes(s, S) <= workspace || S < base ? S : choose(base, workspace);
}
// Grouped queries: from group 4 on one 512-thread workgroup per compute unit (see gqa_waves), at
// group 2 two 256-thread ones.  Measured at 8 x 32 query heads x 32768 keys, d_k = 128, m = 8 (us per
// launch at 128 / 256 / 512 / 1024 workgroups): group 4: 148 / 102 / 111 / 113; group 8: 127 / 75 / 84 / 102;
// group 2: 283 / 187 / 186 / 200.
static int auto_splits_gqa(const lookat_shape *s, int group, int64_t L)
{
    if (group == 1)
        return auto_splits(s, L);
    int64_t want = (group >= 4 ? 256 : 512) / ((int64_t)s->B * s->H);
    // Ranges of at least 1024 keys.  With 512 (us per fused step, ranges of 1024 / 512 keys): group 2, 64 key/value heads x 2048 keys
    // 15.0 / 14.0, but 80 x 2686 14.1 / 15.3, and group 4, 6 x 31374 keys 21.0 / 31.7 (42 workgroups for a die's 32 compute units).
    const int64_t cap = (L + 1023) / 1024;
    want = want < cap ? want : cap;
    return (int)(want < 1 ? 1 : (want > 256 ? 256 : want));
}

static bool tuned_dk(int d_k) { return d_k == 32 || d_k == 64 || d_k == 128 || d_k == 256; }

template <int DK, int WAVES, int OCC, bool PAD = false>
static void launch_tuned(const DecodeArgs &a, dim3 grid, hipStream_t st)
{
    dim3 block(WAVES * kWave);
    const size_t lds = ((size_t)a.m * kCentroids + (size_t)WAVES * (DK + 2)) * sizeof(float);
#define LOOKAT_TUNED_LAUNCH(M_)                                                                                 \
    hipLaunchKernelGGL((decode_split_kernel<DK, M_, WAVES, OCC, void, 1, 1, 1, PAD>), grid, block, lds, st,     \
                       LOOKAT_DECODE_HEAD_ARGS(a, false), late_of(a))
    switch (a.m) {
    case 2:
        LOOKAT_TUNED_LAUNCH(2);
        break;
    case 4:
        LOOKAT_TUNED_LAUNCH(4);
        break;
    case 8:
        LOOKAT_TUNED_LAUNCH(8);
        break;
    default:
        if constexpr (WAVES == kDecWaves) {   // (pick_waves: the large workgroup is taken with m = 2, 4 or 8)
            // (32, 64, 128 and 256 coordinates have no other divisors up to 32)
            if (a.m == 16)
                LOOKAT_TUNED_LAUNCH(16);
            else if constexpr (PAD)
                LOOKAT_TUNED_LAUNCH(0);
            else if (a.m == 1)
                LOOKAT_TUNED_LAUNCH(1);
            else
                LOOKAT_TUNED_LAUNCH(32);
        }
        break;
    }
#undef LOOKAT_TUNED_LAUNCH
}

// Wavefronts per workgroup: 16 for long ranges (at least 32 tiles), else 4 (measured on
// MI355X: the small workgroup wins at context 1024, the large one from 16K keys on).
static int pick_waves(int d_k, int m, int64_t keys_per_split)
{
    if ((d_k != 64 && d_k != 128) || (m != 2 && m != 4 && m != 8))
        return 4;   // the 16-wave variant must fit 64 registers; only these shapes do
    return keys_per_split >= 32 * kTile ? 16 : 4;
}

// Fused decode step: one workgroup of 512 threads per (b,h), one range: four wavefronts build the
// table and encode the new key, four request their first kStepPrefetch tiles at once; after the
// barrier the table builders request theirs and all eight stream.  Measured at B=32, H=12,
// L=1024, m=4 (us per launch): 256 threads, every wavefront doing both 13.8 (one tile ahead 14.0,
// four 15.9); 512 threads with the two roles 13.4; the same with the table builders at raised
// wave priority 11.8 (their codebook requests enter the compute unit's memory queue ahead of
// the streamers' tile requests instead of interleaved with them).
constexpr int kStepPrefetch = 2;
constexpr int kStepWaves = 2 * kDecWaves;   // four wavefronts build the table, four start streaming at once
// Where every workgroup has a compute unit to itself, which takes at most 32 on a die (all ranges of a (b,h) run on one).
static bool step_is_lone(const DecodeArgs &a)
{
    return ((int64_t)a.BH + kXcds - 1) / kXcds * a.splits <= 32;
}
template <int DK, typename FT>
static bool launch_step_lone(const DecodeArgs &a, dim3 grid, hipStream_t st)
{
    const uint32_t counts = (uint32_t)a.BH | (uint32_t)a.splits << 9 | (uint32_t)a.H << 15;
#define LOOKAT_LONE_CASE(M_)                                                                                              \
    case M_:                                                                                                              \
        hipLaunchKernelGGL((decode_step_lone_kernel<FT, DK, M_>), grid, dim3(4 * kDecThreads), lone_lds_bytes(M_, DK), st,  \
                           a.codebooks, static_cast<const FT *>(a.q), static_cast<const FT *>(a.k_new), a.codes_w, a.values, \
                           counts, (uint32_t)a.L, (uint32_t)a.code_stride, (uint32_t)a.value_stride,                      \
                           LoneLate{a.part, a.out, a.scale_log2e});                                                       \
        return true;
    switch (a.m) {
        LOOKAT_LONE_CASE(2)
        LOOKAT_LONE_CASE(4)
        LOOKAT_LONE_CASE(8)
        LOOKAT_LONE_CASE(16)
    default:
        return false;
    }
#undef LOOKAT_LONE_CASE
}
template <int DK, typename FT>
static bool launch_step(const DecodeArgs &a, dim3 grid, hipStream_t st)
{
    dim3 block(kStepWaves * kWave);
    const size_t lds = ((size_t)a.m * kCentroids + (size_t)kStepWaves * (DK + 2)) * sizeof(float) + step_encoder_bytes(a.m);
    if (step_is_lone(a))
        return launch_step_lone<DK, FT>(a, grid, st);
    // (16 subspaces: registers for a third workgroup on a compute unit; 640 (b,h) x 600 keys, d_k = 128, two steps 41.3 us, 49 with two.)
#define LOOKAT_STEP_CASE(M_)                                                                                              \
    case M_:                                                                                                              \
        hipLaunchKernelGGL((decode_split_kernel<DK, M_, kStepWaves, M_ == 16 ? 6 : 4, FT, 1, M_ == 16 ? 1 : kStepPrefetch>), grid, block,  \
                           lds, st, LOOKAT_DECODE_HEAD_ARGS(a, true), late_of(a));                                        \
        return true;
    switch (a.m) {
        LOOKAT_STEP_CASE(2)
        LOOKAT_STEP_CASE(4)
        LOOKAT_STEP_CASE(8)
        LOOKAT_STEP_CASE(16)
    default:
        return false;
    }
#undef LOOKAT_STEP_CASE
}

// Two batch entries of one head per workgroup (1024 threads): see decode_split_kernel, NB = 2.
// When the library takes it.  A compute unit holds two 512-thread workgroups of the fused step or one paired
// one, and a launch is as slow as its most loaded compute unit.  Up to 256 (b,h) every workgroup has a
// compute unit to itself and pairing only halves the parallelism (1.2 to 1.7 times the time); from 257 to 512 (b,h) some compute
// units carry two (b,h) either way and the pairs halve the codebook traffic; beyond 512 the pairs need a second round of
// workgroups where single entries still fit two to a compute unit (528: 1.2 to 1.5 times).  us per launch, single / paired, fp16 queries, up to
// twelve layers in rotation: d_k = 64, m = 4: 264 (b,h) x 768 keys 9.8 / 9.6, 264 x 1024 11.1 / 10.5, 320 x 1024 11.6 / 11.1, 384 x 1024 12.06 /
// 12.02, 504 x 1024 14.2 / 14.0, 448 x 1024 12.9 / 13.6, 264 x 4096 33.1 / 29.3, 504 x 4096 43.5 / 43.3; at 512 keys 0.99 to 1.01 of the time.
// m = 8 and 16 are not taken there: 264 x 1024 0.95 and 1.05, 448 x 1024 1.02 and 1.07.  d_k = 128, m = 4: 264 x 512 13.0 / 13.0, 512 x 512 16.4 / 18.1,
// 264 x 768 16.4 / 15.7, 504 x 768 21.3 / 22.0, 264 x 1024 20.0 / 17.7, 384 x 1024 21.4 / 20.9, 504 x 1024 26.5 / 25.7, 320 x 2048 0.85, 504 x 4096 0.99
// of the time; m = 8: 264 x 2048 36.6 / 30.2, 384 x 2048 38.6 / 36.4, 504 x 2048 48.3 / 45.4.  (Eight heads of 1024 keys at d_k = 128, where the
// entries of a pair lie 2 MB apart: 20 to 26% slower from 352 (b,h) on.)
// m = 2 (one codebook row = 64 registers) has no paired instance at d_k = 128: it would spill.
static bool step_pairs_entries(const lookat_shape *s, int group, int64_t L, int S)
{
    const int64_t BH = (int64_t)s->B * s->H;
    if (group != 1 || S != 1 || (s->B & 1) || BH <= 256 || BH > 512)
        return false;
    if (s->d_k == 64)
        return (s->m == 2 || s->m == 4) && L >= 768;
    if (s->d_k == 128)
        return (s->m == 4 && L >= 512) || (s->m == 8 && L >= 2048);
    return false;
}

// Ranges of the fused step when the caller leaves the choice to the library: as the unfused call, except where one range would be
// served by paired batch entries.  Cutting them gives that up and pays only for long contexts of up to 320 (b,h).  us per call,
// paired / cut: d_k = 128, m = 4: 264 (b,h) x 2048 keys 29.1 / 33.5, 320 x 5000 71 / 67, 264 x 12000 149 / 130, 384 x 8192 124 / 135;
// m = 8: 288 x 2048 31 / 34, 264 x 2600 37 / 36, 264 x 5000 67 / 61, 384 x 12000 181 / 186; d_k = 64, m = 2: 288 x 3500 26.0 / 25.1, 320 x 5000 37 / 36,
// 264 x 12000 79 / 66; m = 4: 264 x 3500 26.0 / 24.3, 264 x 8192 53 / 47, 384 x 32768 252 / 244.  (The lines are those of a step that built its table
// more slowly in every range; where they leave a pair whole that a cut would serve, it costs 3 to 7%.)
// Up to 1024 keys, two tiles per wavefront, a cut gains less than the merge's launch costs, or little: one range / four, d_k = 64, m = 8: 12 (b,h)
// 5.0 / 6.4, 64 6.3 / 7.2; d_k = 128, m = 8: 1 (b,h) 6.3 / 6.4, 12 7.7 / 7.1, 32 8.0 / 7.9, 100 9.0 / 11.5.  (At 1536 keys: 12 9.4 / 7.6.)
static int step_auto_splits(const lookat_shape *s, int64_t L, int unfused)
{
    const int64_t pays = s->d_k == 128 ? (s->m == 4 ? 10000 : 2500) : (s->m == 2 ? 10000 : 5000);
    if (L <= 2 * kStepWaves * kTile)
        return 1;
    return step_pairs_entries(s, 1, L, 1) && ((int64_t)s->B * s->H > 320 || L < pays) ? 1 : unfused;
}

template <int DK, typename FT>
static bool launch_step_pair(const DecodeArgs &a, dim3 grid, hipStream_t st)
{
    dim3 block(2 * kStepWaves * kWave);
    const size_t lds = 2 * step_pair_lds_bytes(a.m, DK);
    switch (a.m) {
    case 2:
        if constexpr (DK == 64) {
            hipLaunchKernelGGL((decode_split_kernel<DK, 2, kStepWaves, 4, FT, 1, kStepPrefetch, 2>), grid, block, lds, st,
                               LOOKAT_DECODE_HEAD_ARGS(a, true), late_of(a));
            return true;
        }
        return false;
    case 4:
        hipLaunchKernelGGL((decode_split_kernel<DK, 4, kStepWaves, 4, FT, 1, kStepPrefetch, 2>), grid, block, lds, st,
                           LOOKAT_DECODE_HEAD_ARGS(a, true), late_of(a));
        return true;
    case 8:
        hipLaunchKernelGGL((decode_split_kernel<DK, 8, kStepWaves, 4, FT, 1, kStepPrefetch, 2>), grid, block, lds, st,
                           LOOKAT_DECODE_HEAD_ARGS(a, true), late_of(a));
        return true;
    case 16:
        hipLaunchKernelGGL((decode_split_kernel<DK, 16, kStepWaves, 4, FT, 1, 1, 2>), grid, block, lds, st,
                           LOOKAT_DECODE_HEAD_ARGS(a, true), late_of(a));
        return true;
    default:
        return false;
    }
}

// Grouped queries: 256-thread workgroups; four wavefronts per SIMD up to G = 4 (G accumulator sets
// per lane fit 128 registers), two for G = 8.
// LDS of a grouped-query workgroup: the group's tables and the per-wavefront partial results.
static size_t gqa_lds_bytes(int group, int m, int d_k, int waves)
{
    return ((size_t)group * m * kCentroids + (size_t)waves * group * (d_k + 2)) * sizeof(float);
}
// From group 4 on a workgroup has eight wavefronts where LDS allows: two wavefronts per SIMD share one
// copy of the group's tables (group x m KB) instead of two four-wavefront workgroups holding a copy
// each.  B=8, 32 query heads, 32768 keys, d_k=128, m=8: group 8: 81 us against 97 us; group 4: 102
// against 115 us.
static int gqa_waves(int group, int m, int d_k)
{
    return (group >= 4 && gqa_lds_bytes(group, m, d_k, 2 * kDecWaves) <= 160 * 1024) ? 2 * kDecWaves : kDecWaves;
}

template <int DK, int G, int GW = kDecWaves>
static int launch_gqa(const DecodeArgs &a, dim3 grid, hipStream_t st)
{
    dim3 block(GW * kWave);
    const size_t lds = gqa_lds_bytes(G, a.m, DK, GW);
#define LOOKAT_GQA_CASE(M_)                                                                                    \
    case M_: {                                                                                                 \
        auto kern = decode_split_kernel<DK, M_, GW, ((DK == 128 && G >= 4) ? 2 : (G <= 4 ? 4 : (GW == kDecWaves ? 3 : 2))), void, G>; \
        if (lds > 64 * 1024) {                                                                                 \
            /* allow more than 64 KB of dynamic LDS: idempotent, so every call makes it (no shared flag) */   \
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                          \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);         \
            if (e != hipSuccess)                                                                               \
                return fail(LOOKAT_ERR_HIP, "lookat_attend_decode_gqa: cannot reserve %zu bytes of LDS: %s", lds, \
                            hipGetErrorString(e));                                                             \
        }                                                                                                      \
        hipLaunchKernelGGL(kern, grid, block, lds, st, LOOKAT_DECODE_HEAD_ARGS(a, false), late_of(a));         \
        return LOOKAT_OK;                                                                                      \
    }
    switch (a.m) {
        LOOKAT_GQA_CASE(2)
        LOOKAT_GQA_CASE(4)
        LOOKAT_GQA_CASE(8)
        LOOKAT_GQA_CASE(16)
    default:
        return fail(LOOKAT_ERR_UNSUPPORTED, "lookat_attend_decode_gqa handles m in {2,4,8,16}; got m=%d", a.m);
    }
#undef LOOKAT_GQA_CASE
}

// Fused step with grouped queries: the roles of the ungrouped fused step; the table builders produce the
// tables of all G query heads from one pass over the key/value head's codebook.  Two workgroups per
// compute unit at group 2, one from group 4 on (as the unfused grouped kernel).
static size_t step_gqa_lds_bytes(int group, int m, int d_k)
{
    return gqa_lds_bytes(group, m, d_k, kStepWaves) + step_encoder_bytes(m);
}
template <int DK, typename FT, int G>
static int launch_step_gqa(const DecodeArgs &a, dim3 grid, hipStream_t st)
{
    dim3 block(kStepWaves * kWave);
    const size_t lds = step_gqa_lds_bytes(G, a.m, DK);
#define LOOKAT_STEP_GQA_CASE(M_)                                                                               \
    case M_: {                                                                                                 \
        auto kern = decode_split_kernel<DK, M_, kStepWaves, ((G == 2 && DK / M_ < 64) ? 4 : 2), FT, G, kStepPrefetch>; \
        if (lds > 64 * 1024) {                                                                                 \
            /* allow more than 64 KB of dynamic LDS: idempotent, so every call makes it (no shared flag) */   \
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                          \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);         \
            if (e != hipSuccess)                                                                               \
                return fail(LOOKAT_ERR_HIP, "lookat_decode_step_gqa: cannot reserve %zu bytes of LDS: %s", lds, \
                            hipGetErrorString(e));                                                             \
        }                                                                                                      \
        hipLaunchKernelGGL(kern, grid, block, lds, st, LOOKAT_DECODE_HEAD_ARGS(a, true), late_of(a));          \
        return LOOKAT_OK;                                                                                      \
    }
    switch (a.m) {
        LOOKAT_STEP_GQA_CASE(2)
        LOOKAT_STEP_GQA_CASE(4)
        LOOKAT_STEP_GQA_CASE(8)
        LOOKAT_STEP_GQA_CASE(16)
    default:
        return fail(LOOKAT_ERR_UNSUPPORTED, "lookat_decode_step_gqa handles m in {2,4,8,16}; got m=%d", a.m);
    }
#undef LOOKAT_STEP_GQA_CASE
}

template <int DK, typename FT>
static int launch_step_gqa_group(int group, const DecodeArgs &a, dim3 grid, hipStream_t st)
{
    switch (group) {
    case 2:
        return launch_step_gqa<DK, FT, 2>(a, grid, st);
    case 4:
        return launch_step_gqa<DK, FT, 4>(a, grid, st);
    case 8:
        return launch_step_gqa<DK, FT, 8>(a, grid, st);
    default:
        return fail(LOOKAT_ERR_UNSUPPORTED, "lookat_decode_step_gqa handles group in {1,2,4,8}; got %d", group);
    }
}

template <int DK>
static int launch_gqa_dk(int group, const DecodeArgs &a, dim3 grid, hipStream_t st)
{
    switch (group) {
    case 2:
        return launch_gqa<DK, 2>(a, grid, st);
    case 4:
        return gqa_waves(4, a.m, DK) == kDecWaves ? launch_gqa<DK, 4>(a, grid, st)
                                                  : launch_gqa<DK, 4, 2 * kDecWaves>(a, grid, st);
    case 8:
        return gqa_waves(8, a.m, DK) == kDecWaves ? launch_gqa<DK, 8>(a, grid, st)
                                                  : launch_gqa<DK, 8, 2 * kDecWaves>(a, grid, st);
    default:
        return fail(LOOKAT_ERR_UNSUPPORTED, "lookat_attend_decode_gqa handles group in {1,2,4,8}; got %d", group);
    }
}

}  // namespace lookat

namespace lookat {
// Fused step, S ranges per (b,h) (S = 1: no workspace, results written directly).
// group > 1: shape->H counts key/value heads, q and out have group times as many heads.
static int decode_step_impl(const char *who, const lookat_shape *shape, int group, int64_t L, const void *q,
                            const void *k_new, int qk_dtype, const float *codebooks, uint8_t *codes,
                            int64_t code_stride_bh, const void *values, int64_t value_stride_bh, float scale, int S,
                            void *workspace, size_t workspace_bytes, float *out, void *stream, int force_entries = 0)
{
    // force_entries: 0 = the library's choice of batch entries per workgroup, 1 or 2 = that many (measurement aid).
    // (At d_k = 128 with m = 2 a codebook row alone is 64 registers: two entries' state does not fit the 128
    // registers of a 1024-thread workgroup, so there is no paired instance.)
    if (force_entries == 2 && (group != 1 || (shape->B & 1) || (shape->d_k != 64 && (shape->d_k != 128 || shape->m == 2))))
        return fail(LOOKAT_ERR_UNSUPPORTED,
                    "paired batch entries need an even batch, ungrouped queries and d_k = 64 or d_k = 128 with m > 2; "
                    "got B=%d group=%d d_k=%d m=%d", shape->B, group, shape->d_k, shape->m);
    const bool paired = force_entries == 2 || (force_entries == 0 && step_pairs_entries(shape, group, L, S));
    if (L <= 0)
        return fail(LOOKAT_ERR_SHAPE, "L=%lld must be positive", (long long)L);
    if (qk_dtype != LOOKAT_F16 && qk_dtype != LOOKAT_F32)
        return fail(LOOKAT_ERR_DTYPE, "qk_dtype=%d is neither LOOKAT_F16 nor LOOKAT_F32", qk_dtype);
    if (!q || !k_new || !codebooks || !codes || !values || !out)
        return fail(LOOKAT_ERR_NULL, "q, k_new, codebooks, codes, values and out must be non-NULL");
    if (code_stride_bh < L * shape->m || value_stride_bh < L * shape->d_k)
        return fail(LOOKAT_ERR_SHAPE, "code_stride_bh=%lld / value_stride_bh=%lld smaller than one (b,h) slab",
                    (long long)code_stride_bh, (long long)value_stride_bh);
    if (!aligned16(q) || !aligned16(k_new) || !aligned16(codebooks) || !aligned16(values) || !aligned16(out) ||
        ((value_stride_bh * 2) % 16))
        return fail(LOOKAT_ERR_ALIGN, "q, k_new, codebooks, values, out and value_stride_bh must be 16-byte aligned");
    const bool m_ok = shape->m == 2 || shape->m == 4 || shape->m == 8 || shape->m == 16;
    if (!m_ok || (shape->d_k != 64 && shape->d_k != 128))
        return fail(LOOKAT_ERR_UNSUPPORTED,
                    "%s handles d_k in {64,128} with m in {2,4,8,16}; got d_k=%d m=%d "
                    "(use encode_keys + build_lut + attend_decode)", who, shape->d_k, shape->m);
    if ((reinterpret_cast<uintptr_t>(codes) % shape->m) || (code_stride_bh % shape->m))
        return fail(LOOKAT_ERR_ALIGN, "codes and code_stride_bh must be multiples of m=%d bytes", shape->m);
    if ((L + 2048) * (int64_t)shape->d_k * 2 > 0xffffffffLL)
        return fail(LOOKAT_ERR_UNSUPPORTED, "L=%lld: one (b,h) value slab must stay below 4 GiB", (long long)L);
    if (code_stride_bh > 0xffffffffLL || value_stride_bh > 0xffffffffLL)
        return fail(LOOKAT_ERR_UNSUPPORTED, "(b,h) strides must stay below 2^32 elements");
    if (group > 1 && step_gqa_lds_bytes(group, shape->m, shape->d_k) > 160 * 1024)
        return fail(LOOKAT_ERR_UNSUPPORTED, "group=%d x m=%d tables (%zu bytes with the reduction buffer) exceed the 160 KB of LDS",
                    group, shape->m, step_gqa_lds_bytes(group, shape->m, shape->d_k));
    const int64_t BH = (int64_t)shape->B * shape->H;
    const size_t need = (S == 1) ? 0 : (size_t)BH * group * S * (shape->d_k + 2) * sizeof(float);
    if (need) {
        if (!workspace || workspace_bytes < need)
            return fail(LOOKAT_ERR_WORKSPACE, "workspace of %zu bytes needed for %d splits, got %zu", need, S,
                        workspace_bytes);
        if (!aligned16(workspace))
            return fail(LOOKAT_ERR_ALIGN, "workspace must be 16-byte aligned");
    }
    const int64_t units = paired ? BH / 2 : BH;   // workgroups per range
    const int64_t nblocks = (units + kXcds - 1) / kXcds * kXcds * S;
    if (nblocks > 0x7fffffffLL)
        return fail(LOOKAT_ERR_UNSUPPORTED, "B*H*num_splits=%lld workgroups exceed one launch", (long long)nblocks);

    DecodeArgs a;
    a.lut = nullptr;
    a.codes = codes;
    a.values = static_cast<const __half *>(values);
    a.part = static_cast<float *>(workspace);
    a.out = out;
    a.scores_out = nullptr;
    a.code_stride = code_stride_bh;
    a.value_stride = value_stride_bh;
    a.L = L;
    a.keys_per_split = round_up((L + S - 1) / S, kTile);
    a.BH = (int)BH;
    a.splits = S;
    a.d_k = shape->d_k;
    a.m = shape->m;
    a.scale_log2e = scale * kLog2e;
    a.q = q;
    a.k_new = k_new;
    a.codebooks = codebooks;
    a.codes_w = codes;
    a.H = shape->H;
    hipStream_t st = static_cast<hipStream_t>(stream);
    dim3 grid((unsigned)nblocks);
    if (group == 1) {
        bool ok;
        if (paired) {
            if (shape->d_k == 64)
                ok = (qk_dtype == LOOKAT_F16) ? launch_step_pair<64, __half>(a, grid, st)
                                              : launch_step_pair<64, float>(a, grid, st);
            else
                ok = (qk_dtype == LOOKAT_F16) ? launch_step_pair<128, __half>(a, grid, st)
                                              : launch_step_pair<128, float>(a, grid, st);
        } else if (shape->d_k == 64)
            ok = (qk_dtype == LOOKAT_F16) ? launch_step<64, __half>(a, grid, st) : launch_step<64, float>(a, grid, st);
        else
            ok = (qk_dtype == LOOKAT_F16) ? launch_step<128, __half>(a, grid, st) : launch_step<128, float>(a, grid, st);
        if (!ok)
            return fail(LOOKAT_ERR_UNSUPPORTED, "no fused kernel for this shape");
    } else {
        int rc;
        if (shape->d_k == 64)
            rc = (qk_dtype == LOOKAT_F16) ? launch_step_gqa_group<64, __half>(group, a, grid, st)
                                          : launch_step_gqa_group<64, float>(group, a, grid, st);
        else
            rc = (qk_dtype == LOOKAT_F16) ? launch_step_gqa_group<128, __half>(group, a, grid, st)
                                          : launch_step_gqa_group<128, float>(group, a, grid, st);
        if (rc != LOOKAT_OK)
            return rc;
    }
    if (S > 1)
        hipLaunchKernelGGL(decode_combine_kernel, dim3((unsigned)(BH * group)), dim3(kDecThreads), 0, st,
                           static_cast<const float *>(workspace), out, S, shape->d_k);
    return check_launch(who);
}
}  // namespace lookat

extern "C" int lookat_decode_step(const lookat_shape *shape, int64_t L, const void *q, const void *k_new,
                                  lookat_dtype qk_dtype, const float *codebooks, uint8_t *codes, int64_t code_stride_bh,
                                  const void *values, int64_t value_stride_bh, float scale, float *out, void *stream)
{
    using namespace lookat;
    clear_error();
    if (int rc = check_shape(shape))
        return rc;
    return decode_step_impl("lookat_decode_step", shape, 1, L, q, k_new, qk_dtype, codebooks, codes, code_stride_bh, values,
                            value_stride_bh, scale, 1, nullptr, 0, out, stream);
}

extern "C" int32_t lookat_decode_step_entries_per_workgroup(const lookat_shape *shape, int64_t L)
{
    using namespace lookat;
    clear_error();
    if (check_shape(shape) != LOOKAT_OK || L <= 0)
        return 0;
    const bool m_ok = shape->m == 2 || shape->m == 4 || shape->m == 8 || shape->m == 16;
    if (!m_ok || (shape->d_k != 64 && shape->d_k != 128))
        return 0;
    return step_pairs_entries(shape, 1, L, 1) ? 2 : 1;
}

extern "C" int lookat_probe_decode_step_entries(const lookat_shape *shape, int32_t entries_per_workgroup, int64_t L,
                                                const void *q, const void *k_new, lookat_dtype qk_dtype,
                                                const float *codebooks, uint8_t *codes, int64_t code_stride_bh,
                                                const void *values, int64_t value_stride_bh, float scale, float *out,
                                                void *stream)
{
    using namespace lookat;
    clear_error();
    if (int rc = check_shape(shape))
        return rc;
    if (entries_per_workgroup != 1 && entries_per_workgroup != 2)
        return fail(LOOKAT_ERR_SHAPE, "entries_per_workgroup=%d must be 1 or 2", entries_per_workgroup);
    return decode_step_impl("lookat_probe_decode_step_entries", shape, 1, L, q, k_new, qk_dtype, codebooks, codes,
                            code_stride_bh, values, value_stride_bh, scale, 1, nullptr, 0, out, stream,
                            entries_per_workgroup);
}

extern "C" size_t lookat_decode_step_split_workspace_bytes(const lookat_shape *shape, int64_t L, int32_t num_splits)
{
    return lookat_attend_decode_workspace_bytes(shape, L, num_splits);
}

extern "C" int lookat_decode_step_split(const lookat_shape *shape, int64_t L, const void *q, const void *k_new,
                                        lookat_dtype qk_dtype, const float *codebooks, uint8_t *codes, int64_t code_stride_bh,
                                        const void *values, int64_t value_stride_bh, float scale, int32_t num_splits,
                                        void *workspace, size_t workspace_bytes, float *out, void *stream)
{
    using namespace lookat;
    clear_error();
    if (int rc = check_shape(shape))
        return rc;
    if (num_splits < 0 || num_splits > 65535)
        return fail(LOOKAT_ERR_SHAPE, "num_splits=%d out of range [0,65535]", num_splits);
    const int S = num_splits ? num_splits : (L > 0 ? step_auto_splits(shape, L, auto_splits(shape, L, workspace ? workspace_bytes : 0)) : 1);
    return decode_step_impl("lookat_decode_step_split", shape, 1, L, q, k_new, qk_dtype, codebooks, codes, code_stride_bh,
                            values, value_stride_bh, scale, S, workspace, workspace_bytes, out, stream);
}

extern "C" size_t lookat_decode_step_gqa_workspace_bytes(const lookat_shape *shape, int32_t group, int64_t L,
                                                         int32_t num_splits)
{
    return lookat_attend_decode_gqa_workspace_bytes(shape, group, L, num_splits);
}

extern "C" int lookat_decode_step_gqa(const lookat_shape *shape, int32_t group, int64_t L, const void *q,
                                      const void *k_new, lookat_dtype qk_dtype, const float *codebooks, uint8_t *codes,
                                      int64_t code_stride_bh, const void *values, int64_t value_stride_bh, float scale,
                                      int32_t num_splits, void *workspace, size_t workspace_bytes, float *out,
                                      void *stream)
{
    using namespace lookat;
    clear_error();
    if (int rc = check_shape(shape))
        return rc;
    if (group != 1 && group != 2 && group != 4 && group != 8)
        return fail(LOOKAT_ERR_UNSUPPORTED, "lookat_decode_step_gqa handles group in {1,2,4,8}; got %d", group);
    if (num_splits < 0 || num_splits > 65535)
        return fail(LOOKAT_ERR_SHAPE, "num_splits=%d out of range [0,65535]", num_splits);
    const int S = num_splits ? num_splits
                             : (L <= 0 ? 1 : (group == 1 ? step_auto_splits(shape, L, auto_splits(shape, L, workspace ? workspace_bytes : 0)) : auto_splits_gqa(shape, group, L)));
    return decode_step_impl("lookat_decode_step_gqa", shape, group, L, q, k_new, qk_dtype, codebooks, codes,
                            code_stride_bh, values, value_stride_bh, scale, S, workspace, workspace_bytes, out, stream);
}

extern "C" int32_t lookat_attend_decode_auto_splits(const lookat_shape *shape, int64_t L)
{
    using namespace lookat;
    clear_error();
    if (check_shape(shape) != LOOKAT_OK || L <= 0)
        return 0;
    return auto_splits(shape, L);
}

extern "C" int lookat_attend_decode_launch_shape(const lookat_shape *shape, int64_t L, int32_t num_splits,
                                                 int32_t *ranges, int32_t *wavefronts)
{
    using namespace lookat;
    clear_error();
    if (int rc = check_shape(shape))
        return rc;
    if (L <= 0)
        return fail(LOOKAT_ERR_SHAPE, "L=%lld must be positive", (long long)L);
    if (num_splits < 0 || num_splits > 65535)
        return fail(LOOKAT_ERR_SHAPE, "num_splits=%d out of range [0,65535]", num_splits);
    const int S = num_splits ? num_splits : auto_splits(shape, L);
    if (ranges)
        *ranges = S;
    if (wavefronts)
        *wavefronts = tuned_dk(shape->d_k) ? pick_waves(shape->d_k, shape->m, round_up((L + S - 1) / S, kTile)) : kDecWaves;
    return LOOKAT_OK;
}

extern "C" size_t lookat_attend_decode_workspace_bytes(const lookat_shape *shape, int64_t L, int32_t num_splits)
{
    using namespace lookat;
    clear_error();
    if (check_shape(shape) != LOOKAT_OK || L <= 0 || num_splits < 0)
        return 0;
    const int S = num_splits ? num_splits : auto_splits(shape, L);
    if (S == 1)
        return 0;
    return (size_t)shape->B * shape->H * S * (shape->d_k + 2) * sizeof(float);
}

namespace lookat {
static int attend_decode_impl(const lookat_shape *shape, int64_t L, const float *lut, const uint8_t *codes,
                              int64_t code_stride_bh, const void *values, int64_t value_stride_bh, float scale,
                              int32_t num_splits, void *workspace, size_t workspace_bytes, float *out,
                              float *scores_out, void *stream)
{
    if (int rc = check_shape(shape))
        return rc;
    if (L <= 0)
        return fail(LOOKAT_ERR_SHAPE, "L=%lld must be positive", (long long)L);
    if (num_splits < 0 || num_splits > 65535)
        return fail(LOOKAT_ERR_SHAPE, "num_splits=%d out of range [0,65535]", num_splits);
    if (!lut || !codes || !values || !out)
        return fail(LOOKAT_ERR_NULL, "lut, codes, values and out must be non-NULL");
    if (code_stride_bh < L * shape->m || value_stride_bh < L * shape->d_k)
        return fail(LOOKAT_ERR_SHAPE, "code_stride_bh=%lld / value_stride_bh=%lld smaller than one (b,h) slab",
                    (long long)code_stride_bh, (long long)value_stride_bh);
    if (!aligned16(lut) || !aligned16(values) || !aligned16(out) || ((value_stride_bh * 2) % 16))
        return fail(LOOKAT_ERR_ALIGN, "lut, values, out and value_stride_bh must be 16-byte aligned");
    // a key's m codes are fetched with one m-byte load when m is 2, 4, 8 or 16
    const int cvec = (shape->m == 2 || shape->m == 4 || shape->m == 8 || shape->m == 16) ? shape->m : 1;
    if ((reinterpret_cast<uintptr_t>(codes) % cvec) || (code_stride_bh % cvec))
        return fail(LOOKAT_ERR_ALIGN, "codes and code_stride_bh must be multiples of %d bytes for m=%d", cvec,
                    shape->m);
    if (scores_out && (reinterpret_cast<uintptr_t>(scores_out) & 3u))
        return fail(LOOKAT_ERR_ALIGN, "scores_out must be 4-byte aligned");

    if (code_stride_bh > 0xffffffffLL || value_stride_bh > 0xffffffffLL)
        return fail(LOOKAT_ERR_UNSUPPORTED, "(b,h) strides must stay below 2^32 elements");
    // kernels address one (b,h) slab with 32-bit byte offsets (plus one tile of prefetch)
    if ((L + 2048) * (int64_t)shape->d_k * 2 > 0xffffffffLL)
        return fail(LOOKAT_ERR_UNSUPPORTED, "L=%lld: one (b,h) value slab must stay below 4 GiB", (long long)L);
    const int64_t BH = (int64_t)shape->B * shape->H;
    const int S = num_splits ? num_splits : auto_splits(shape, L, workspace ? workspace_bytes : 0);
    const size_t need = (S == 1) ? 0 : (size_t)BH * S * (shape->d_k + 2) * sizeof(float);
    if (need) {
        if (!workspace || workspace_bytes < need)
            return fail(LOOKAT_ERR_WORKSPACE, "workspace of %zu bytes needed for %d splits, got %zu", need, S,
                        workspace_bytes);
        if (!aligned16(workspace))
            return fail(LOOKAT_ERR_ALIGN, "workspace must be 16-byte aligned");
    }
    const int64_t groups = (BH + kXcds - 1) / kXcds;
    const int64_t nblocks = groups * kXcds * S;
    if (nblocks > 0x7fffffffLL)
        return fail(LOOKAT_ERR_UNSUPPORTED, "B*H*num_splits=%lld workgroups exceed one launch", (long long)nblocks);

    DecodeArgs a;
    a.lut = lut;
    a.codes = codes;
    a.values = static_cast<const __half *>(values);
    a.part = static_cast<float *>(workspace);
    a.out = out;
    a.scores_out = scores_out;
    a.code_stride = code_stride_bh;
    a.value_stride = value_stride_bh;
    a.L = L;
    a.keys_per_split = round_up((L + S - 1) / S, kTile);
    a.BH = (int)BH;
    a.splits = S;
    a.d_k = shape->d_k;
    a.m = shape->m;
    a.scale_log2e = scale * kLog2e;
    a.q = nullptr;
    a.k_new = nullptr;
    a.codebooks = nullptr;
    a.codes_w = nullptr;
    a.H = shape->H;

    hipStream_t st = static_cast<hipStream_t>(stream);
    dim3 grid((unsigned)nblocks);
    // A head size between the instances takes the next larger one, padded (PAD).  4 x 16 heads x 2501 keys of 96
    // coordinates, m = 8: 8.8 us against 101 us for a kernel with one output coordinate per thread.
    const int waves = tuned_dk(shape->d_k) ? pick_waves(shape->d_k, shape->m, a.keys_per_split) : kDecWaves;
    switch (shape->d_k) {
    case 32:
        launch_tuned<32, 4, 4>(a, grid, st);
        break;
    case 64:
        if (waves == 16)
            launch_tuned<64, 16, 8>(a, grid, st);
        else
            launch_tuned<64, 4, 4>(a, grid, st);
        break;
    case 128:
        if (waves == 16)
            launch_tuned<128, 16, 8>(a, grid, st);
        else
            launch_tuned<128, 4, 4>(a, grid, st);
        break;
    case 256:
        launch_tuned<256, 4, 4>(a, grid, st);
        break;
    default:
        if (shape->d_k < 32)
            launch_tuned<32, 4, 4, true>(a, grid, st);
        else if (shape->d_k < 64)
            launch_tuned<64, 4, 4, true>(a, grid, st);
        else if (shape->d_k < 128)
            launch_tuned<128, 4, 4, true>(a, grid, st);
        else
            launch_tuned<256, 4, 4, true>(a, grid, st);
        break;
    }
    if (int rc = check_launch("lookat_attend_decode (split kernel)"))
        return rc;
    if (S > 1) {
        hipLaunchKernelGGL(decode_combine_kernel, dim3((unsigned)BH), dim3(kDecThreads), 0, st,
                           static_cast<const float *>(workspace), out, S, shape->d_k);
        return check_launch("lookat_attend_decode (combine kernel)");
    }
    return LOOKAT_OK;
}

// Scratch memory of lookat_attend_decode_noalloc: the per-range partial results, in the library's own
// device image instead of a caller's workspace.  Every GPU the library runs on holds one copy.
static __device__ __align__(256) float scratch[LOOKAT_NOALLOC_SCRATCH_BYTES / sizeof(float)];

// Device address of `scratch` on the current device (in host code the array's name is only a handle
// for this query), looked up once per device and kept.
static int scratch_address(float **ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static float *known[kMaxDevices] = {};
    int device = -1;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess || device < 0 || device >= kMaxDevices)
        return fail(LOOKAT_ERR_HIP, "lookat_attend_decode_noalloc: cannot identify the current device (%s, device %d)",
                    hipGetErrorString(e), device);
    std::lock_guard<std::mutex> hold(lock);
    if (!known[device]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(LOOKAT_ERR_HIP, "lookat_attend_decode_noalloc: hipGetSymbolAddress failed on device %d: %s", device,
                        hipGetErrorString(e));
        known[device] = static_cast<float *>(p);
    }
    *ptr = known[device];
    return LOOKAT_OK;
}
}  // namespace lookat

extern "C" int lookat_attend_decode(const lookat_shape *shape, int64_t L, const float *lut, const uint8_t *codes,
                                    int64_t code_stride_bh, const void *values, int64_t value_stride_bh, float scale,
                                    int32_t num_splits, void *workspace, size_t workspace_bytes, float *out,
                                    float *scores_out, void *stream)
{
    using namespace lookat;
    clear_error();
    return attend_decode_impl(shape, L, lut, codes, code_stride_bh, values, value_stride_bh, scale, num_splits, workspace,
                              workspace_bytes, out, scores_out, stream);
}

extern "C" int lookat_attend_decode_noalloc(const lookat_shape *shape, int64_t L, const float *lut, const uint8_t *codes,
                                            int64_t code_stride_bh, const void *values, int64_t value_stride_bh,
                                            float scale, int32_t num_splits, float *out, float *scores_out, void *stream)
{
    using namespace lookat;
    clear_error();
    if (int rc = check_shape(shape))
        return rc;
    if (L <= 0)
        return fail(LOOKAT_ERR_SHAPE, "L=%lld must be positive", (long long)L);
    if (num_splits < 0 || num_splits > 65535)
        return fail(LOOKAT_ERR_SHAPE, "num_splits=%d out of range [0,65535]", num_splits);
    if (num_splits == 0)   // the library's choice, as far as the scratch memory holds it
        num_splits = auto_splits(shape, L, (size_t)LOOKAT_NOALLOC_SCRATCH_BYTES);
    const size_t need = lookat_attend_decode_workspace_bytes(shape, L, num_splits);
    if (need > (size_t)LOOKAT_NOALLOC_SCRATCH_BYTES)
        return fail(LOOKAT_ERR_WORKSPACE,
                    "lookat_attend_decode_noalloc: B*H*ranges*(d_k+2) floats = %zu bytes exceed the library's %d bytes of "
                    "scratch memory; use lookat_attend_decode with a workspace", need, (int)LOOKAT_NOALLOC_SCRATCH_BYTES);
    float *ws = nullptr;
    if (need) {   // (one range per (b,h): no partial results, nothing to look up)
        if (int rc = scratch_address(&ws))
            return rc;
    }
    return attend_decode_impl(shape, L, lut, codes, code_stride_bh, values, value_stride_bh, scale, num_splits, ws,
                              need ? (size_t)LOOKAT_NOALLOC_SCRATCH_BYTES : 0, out, scores_out, stream);
}

extern "C" size_t lookat_attend_decode_gqa_workspace_bytes(const lookat_shape *shape, int32_t group, int64_t L,
                                                           int32_t num_splits)
{
    using namespace lookat;
    clear_error();
    if (check_shape(shape) != LOOKAT_OK || L <= 0 || num_splits < 0 || group < 1)
        return 0;
    const int S = num_splits ? num_splits : auto_splits_gqa(shape, group, L);
    if (S == 1)
        return 0;
    return (size_t)shape->B * shape->H * group * S * (shape->d_k + 2) * sizeof(float);
}

extern "C" int lookat_attend_decode_gqa(const lookat_shape *shape, int32_t group, int64_t L, const float *lut,
                                        const uint8_t *codes, int64_t code_stride_bh, const void *values,
                                        int64_t value_stride_bh, float scale, int32_t num_splits, void *workspace,
                                        size_t workspace_bytes, float *out, float *scores_out, void *stream)
{
    using namespace lookat;
    if (group == 1)
        return lookat_attend_decode(shape, L, lut, codes, code_stride_bh, values, value_stride_bh, scale, num_splits,
                                    workspace, workspace_bytes, out, scores_out, stream);
    clear_error();
    if (int rc = check_shape(shape))
        return rc;
    if (group != 2 && group != 4 && group != 8)
        return fail(LOOKAT_ERR_UNSUPPORTED, "group=%d: query heads per key/value head must be 1, 2, 4 or 8", group);
    if (L <= 0)
        return fail(LOOKAT_ERR_SHAPE, "L=%lld must be positive", (long long)L);
    if (num_splits < 0 || num_splits > 65535)
        return fail(LOOKAT_ERR_SHAPE, "num_splits=%d out of range [0,65535]", num_splits);
    if (!lut || !codes || !values || !out)
        return fail(LOOKAT_ERR_NULL, "lut, codes, values and out must be non-NULL");
    if (code_stride_bh < L * shape->m || value_stride_bh < L * shape->d_k)
        return fail(LOOKAT_ERR_SHAPE, "code_stride_bh=%lld / value_stride_bh=%lld smaller than one (b,h) slab",
                    (long long)code_stride_bh, (long long)value_stride_bh);
    if (!aligned16(lut) || !aligned16(values) || !aligned16(out) || ((value_stride_bh * 2) % 16))
        return fail(LOOKAT_ERR_ALIGN, "lut, values, out and value_stride_bh must be 16-byte aligned");
    const bool m_ok = shape->m == 2 || shape->m == 4 || shape->m == 8 || shape->m == 16;
    if (!m_ok || (shape->d_k != 64 && shape->d_k != 128))
        return fail(LOOKAT_ERR_UNSUPPORTED,
                    "lookat_attend_decode_gqa handles d_k in {64,128} with m in {2,4,8,16}; got d_k=%d m=%d", shape->d_k,
                    shape->m);
    if ((reinterpret_cast<uintptr_t>(codes) % shape->m) || (code_stride_bh % shape->m))
        return fail(LOOKAT_ERR_ALIGN, "codes and code_stride_bh must be multiples of m=%d bytes", shape->m);
    if (scores_out && (reinterpret_cast<uintptr_t>(scores_out) & 3u))
        return fail(LOOKAT_ERR_ALIGN, "scores_out must be 4-byte aligned");
    if (code_stride_bh > 0xffffffffLL || value_stride_bh > 0xffffffffLL)
        return fail(LOOKAT_ERR_UNSUPPORTED, "(b,h) strides must stay below 2^32 elements");
    if ((L + 2048) * (int64_t)shape->d_k * 2 > 0xffffffffLL)
        return fail(LOOKAT_ERR_UNSUPPORTED, "L=%lld: one (b,h) value slab must stay below 4 GiB", (long long)L);
    const size_t lds = gqa_lds_bytes(group, shape->m, shape->d_k, gqa_waves(group, shape->m, shape->d_k));
    if (lds > 160 * 1024)
        return fail(LOOKAT_ERR_UNSUPPORTED, "group=%d x m=%d tables (%zu bytes with the reduction buffer) exceed the 160 KB of LDS",
                    group, shape->m, lds);
    const int64_t BH = (int64_t)shape->B * shape->H;   // key/value heads
    const int S = num_splits ? num_splits : auto_splits_gqa(shape, group, L);
    const size_t need = (S == 1) ? 0 : (size_t)BH * group * S * (shape->d_k + 2) * sizeof(float);
    if (need) {
        if (!workspace || workspace_bytes < need)
            return fail(LOOKAT_ERR_WORKSPACE, "workspace of %zu bytes needed for %d splits, got %zu", need, S,
                        workspace_bytes);
        if (!aligned16(workspace))
            return fail(LOOKAT_ERR_ALIGN, "workspace must be 16-byte aligned");
    }
    const int64_t nblocks = (BH + kXcds - 1) / kXcds * kXcds * S;
    if (nblocks > 0x7fffffffLL || BH * group > 0x7fffffffLL)
        return fail(LOOKAT_ERR_UNSUPPORTED, "B*H*num_splits=%lld workgroups exceed one launch", (long long)nblocks);

    DecodeArgs a;
    a.lut = lut;
    a.codes = codes;
    a.values = static_cast<const __half *>(values);
    a.part = static_cast<float *>(workspace);
    a.out = out;
    a.scores_out = scores_out;
    a.code_stride = code_stride_bh;
    a.value_stride = value_stride_bh;
    a.L = L;
    a.keys_per_split = round_up((L + S - 1) / S, kTile);
    a.BH = (int)BH;
    a.splits = S;
    a.d_k = shape->d_k;
    a.m = shape->m;
    a.scale_log2e = scale * kLog2e;
    a.q = nullptr;
    a.k_new = nullptr;
    a.codebooks = nullptr;
    a.codes_w = nullptr;
    a.H = shape->H;
    hipStream_t st = static_cast<hipStream_t>(stream);
    dim3 grid((unsigned)nblocks);
    const int rc = (shape->d_k == 64) ? launch_gqa_dk<64>(group, a, grid, st) : launch_gqa_dk<128>(group, a, grid, st);
    if (rc != LOOKAT_OK)
        return rc;
    if (int rc2 = check_launch("lookat_attend_decode_gqa (split kernel)"))
        return rc2;
    if (S > 1) {
        hipLaunchKernelGGL(decode_combine_kernel, dim3((unsigned)(BH * group)), dim3(kDecThreads), 0, st,
                           static_cast<const float *>(workspace), out, S, shape->d_k);
        return check_launch("lookat_attend_decode_gqa (combine kernel)");
    }
    return LOOKAT_OK;
}
