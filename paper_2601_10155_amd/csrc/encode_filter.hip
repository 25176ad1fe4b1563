// Key encoding (paper Sec. 3.4, "Encoding") for many keys per head: a matrix-core filter in
// front of the exact fp64 rule.
//
// The code of a key sub-vector k is argmin_c d(k, C[c]) with d evaluated in fp64, one rounding per
// subtract / multiply / add, coordinates ascending, lowest index on ties.  Evaluating d for all 256
// centroids costs 3 fp64 operations per coordinate and centroid.  Here the 256 candidates are
// first ranked with
//     a_c = |C[c]|^2 - 2 k.C[c]        ( = d_c - |k|^2 up to rounding )
// computed on the matrix cores (rows = 32 centroids, columns = 32 keys, the norm as the
// accumulator's initial value).  If the smallest and the second smallest a_c of a key are further
// apart than twice a bound on |a_c - (exact d_c - |k|^2)|, the smallest one is the unique exact argmin
// and nothing else is evaluated.  Otherwise (near ties, exact ties, NaN or infinite inputs: a few
// sub-vectors in ten thousand on the workloads here) the wavefront evaluates the exact rule for that key
// over all 256 centroids.  Either way the code is the one the exact scan produces, bit for bit.
//
// The product.  Codebook entries are scaled by a power of two s_c (largest entry near 2^13) and split into
// two fp16 terms, -2 s_c C = hi + lo, |error| <= 2^-22 |2 s_c C|; products of fp16 terms are exact in fp32.
//   * fp16 keys enter as they are (s_k = 1);
//   * fp32 keys are scaled by s_k = s_c 2^-6 (a key as large as the largest centroid entry lands near 2^7,
//     which leaves a factor of 256 to fp16's largest value; longer keys go to the exact rule) and split into
//     two truncated fp16 terms, |error| <= 2^-20 |s_k k|.
// v_mfma_f32_32x32x16_f16 contracts sixteen slots at a time: sub-vectors of up to 4 and up to 8 coordinates
// put the terms of one centroid side by side in the slots of one instruction, longer ones take one
// instruction per 16 coordinates and product of terms (hi.hi, lo.hi, and for fp32 keys hi.lo; lo.lo, below
// 2^-20 of the product, is dropped there).  The scores are s_c s_k a_c.  The fp32 matrix
// instruction is not used: it runs at a sixteenth of the rate and shares the vector ALU's datapath.
// Sub-vector lengths of 2 to 64 without an instance of their own are padded with zeros to 4, 8, 16, 32 or 64.
//
// Smallest, second smallest and index.  What bounds the kernel is vector issue: 128 scores per lane and
// block of 32 keys have to be looked at.  Keeping (smallest, second, index) candidate by candidate takes four
// instructions each.  Here a candidate's index is written as digits (row tile t, quarter q, lane half h,
// element e: index = 32 t + 8 q + 4 h + e) and only group minima are formed, over the candidates that share
// (q, e) and over those that share t, three operands at a time (v_minimum3_f32): one instruction per
// candidate for both.  The digit at which a digit's group minima are smallest is that digit of the argmin; and since
// two different candidates differ in at least one digit, the smallest "second smallest group minimum" over
// the digits is exactly the second smallest score.  A NaN anywhere makes the minima NaN (v_minimum3
// propagates it) and sends the key to the exact rule.  Two blocks of 32 keys are finished together, one per
// lane half.
//   Measured (us per call, this kernel / the one that tracked candidate by candidate and ranked fp32 keys with the fp32
//   matrix instruction): 4 x 32 heads x 2048 fp16 keys, 16 subspaces of 8: 88 / 181; 32 x 12 heads x 1024 fp32 keys, 4
//   of 16: 63 / 167; 32 heads x 16384 fp32 keys, 8 of 16: 145 / 425.  Vector and matrix issue add up (counters: 71% and
//   18% of the busy cycles of the first): the matrix instructions do not hide behind the minima, whatever the order.
// A key that the filter cannot decide is only noted (one ballot per 64 keys in LDS); when its keys are through, the
// workgroup's wavefronts share the noted ones out.  Looked at on the spot, one held up its wavefront for microseconds, and
// the unluckiest wavefront the launch (32 of 88 us at the second size above).
//
// Error bound.  a_c is an fp32 sum of n terms (2 d_sub + 1 for fp16 keys, 4 d_sub + 1 for fp32 keys, whose
// split residuals and dropped terms amount to at most 14 2^-23 more) whose magnitudes add up to at most
// S = |k|^2 + 2 max_c |C[c]|^2 (since 2|k.C| <= |k|^2 + |C|^2) times 1 + 2^-9.  With at most 2^-23 relative
// error per accumulation step (round-to-nearest would give 2^-24) and the fp32 rounding of the norms,
// |a_c - exact| <= (2 d_sub + 4) 2^-23 S, respectively (4 d_sub + 16) 2^-23 S.  The threshold used is
// 2.25 times that (twice for the two candidates, the rest for S and for the threshold's own rounding), plus 1e-30 for flushed
// denormals; an infinite or NaN S, a key beyond fp16's range after scaling and a codebook whose scale would
// leave [2^-60, 2^60] go to the exact rule.
//
// This translation unit must be compiled with -ffp-contract=off (the exact rule).
#include <cstdlib>
#include <type_traits>

#include "common.h"

#pragma clang fp contract(off)

namespace lookat {

typedef float ef_v16f __attribute__((ext_vector_type(16)));
typedef float ef_v4f __attribute__((ext_vector_type(4)));
typedef _Float16 ef_v8h __attribute__((ext_vector_type(8)));
typedef _Float16 ef_v4h __attribute__((ext_vector_type(4)));
typedef _Float16 ef_v2h __attribute__((ext_vector_type(2)));
typedef __fp16 ef_v2fp __attribute__((ext_vector_type(2)));

constexpr int kEfThreads = 256;
constexpr int kEfWaves = kEfThreads / kWave;
constexpr int kEfTiles = kCentroids / 32;
constexpr int kEfRounds = 256;         // pairs of key blocks a wavefront may take
static_assert(kEfThreads == kCentroids, "thread c looks after centroid c while the codebook is set up");

template <typename T>
__device__ __forceinline__ float ef_to_f32(T v);
template <>
__device__ __forceinline__ float ef_to_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float ef_to_f32<__half>(__half v) { return __half2float(v); }

__device__ __forceinline__ float ef_min(float a, float b) { return __builtin_elementwise_minimum(a, b); }
__device__ __forceinline__ float ef_min3(float a, float b, float c) { return ef_min(ef_min(a, b), c); }

// Coordinates j0 .. j0+3 of a sub-vector of d_sub coordinates, zero past its end.  FULL: all four exist and the start
// is a multiple of four elements from a 16-byte aligned row.
template <bool FULL, typename T>
__device__ __forceinline__ void ef_load4(const T *sub, int j0, int d_sub, T (&out)[4])
{
    typedef unsigned int chunk_t __attribute__((ext_vector_type(sizeof(T))));   // 4 elements: 8 or 16 bytes
    if (FULL || d_sub % 4 == 0) {
        chunk_t v = {};
        if (FULL || j0 < d_sub)
            v = *reinterpret_cast<const chunk_t *>(sub + j0);
        __builtin_memcpy(out, &v, sizeof(v));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            out[e] = (j0 + e < d_sub) ? sub[j0 + e] : T(0.f);
    }
}

// The exact rule for one key sub-vector (uniform over the wavefront): lane l takes the centroids l, l + 64,
// l + 128, l + 192, one chain per centroid, coordinates ascending; then the smallest distance with the lowest index
// over the wavefront.  Operands are re-read from memory (the matrix fragments are scaled and split).
template <typename KT>
__device__ __forceinline__ int ef_exact_code(const KT *key_sub, const float *cb, int d_sub, int lane)
{
    constexpr int NC = kCentroids / kWave;
    constexpr int JB = 16;               // coordinates per round of loads
    double acc[NC];
#pragma unroll
    for (int u = 0; u < NC; ++u)
        acc[u] = 0.0;
    for (int j0 = 0; j0 < d_sub; j0 += JB) {
        float y[NC][JB];
        KT x[JB];
#pragma unroll
        for (int q = 0; q < JB; q += 4) {
            KT x4[4];
            ef_load4<false, KT>(key_sub, j0 + q, d_sub, x4);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                x[q + e] = x4[e];
#pragma unroll
            for (int u = 0; u < NC; ++u) {
                float y4[4];
                ef_load4<false, float>(cb + (u * kWave + lane) * d_sub, j0 + q, d_sub, y4);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    y[u][q + e] = y4[e];
            }
        }
#pragma unroll
        for (int q = 0; q < JB; ++q)
            if (j0 + q < d_sub) {
                const double xd = (double)ef_to_f32<KT>(x[q]);
#pragma unroll
                for (int u = 0; u < NC; ++u) {
                    const double diff = xd - (double)y[u][q];
                    const double sq = diff * diff;
                    acc[u] = acc[u] + sq;
                }
            }
    }
    // (argmin_value maps a NaN so that the smallest value with the lowest index is the serial scan's choice)
    double best = argmin_value(acc[0], lane);
    int c = lane;
#pragma unroll
    for (int u = 1; u < NC; ++u) {
        const double d = argmin_value(acc[u], u * kWave + lane);
        if (d < best) {
            best = d;
            c = u * kWave + lane;
        }
    }
    double m[1] = {best};
    dmin_wave<1>(m);
    c = (best == m[0]) ? c : kCentroids;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const int c2 = __shfl_xor(c, o);
        c = c2 < c ? c2 : c;
    }
    return c;
}

// Matrix operands of a (head, subspace): slices of 16 slots; lane (col, g) of an operand holds slots 8g .. 8g+7 of its
// row (centroid) or column (key).
//   DP >= 16: slice s carries coordinates 16s .. 16s+15; one operand of hi terms and one of lo terms;
//   DP == 8:  one operand, hi terms in slots 0..7, lo terms in 8..15; the key's terms stand twice;
//   DP == 4:  one operand, slots hi(4) lo(4) hi(4) lo(4); the key's hi terms in slots 0..7, its lo terms (fp32 keys;
//             zero for fp16 keys) in 8..15.
template <typename KT, int DP>
struct EfShape {
    static constexpr bool K32 = std::is_same<KT, float>::value;
    static constexpr int NS = DP >= 16 ? DP / 16 : 1;              // slices
    static constexpr int NA = DP >= 16 ? 2 * NS : 1;               // centroid operands per row tile
    static constexpr int NB = DP == 4 ? 1 : (K32 ? 2 * NS : NS);   // key operands
    static constexpr int NI = DP == 4 ? 1 : (DP == 8 ? NB : (K32 ? 3 : 2) * NS);   // instructions per row tile
    static constexpr int NL = DP == 4 ? 1 : 2 * NS;                // 4-coordinate pieces a lane loads of a key
    static constexpr bool ALDS = DP >= 16;                         // centroid operands in LDS, not in registers
    static constexpr bool NORM_SLOTS = DP == 4;                    // the norm sits in spare slots, else it starts the accumulator
    static constexpr int WAVES = DP <= 16 ? (K32 && DP == 8 ? 3 : 4) : (DP <= 32 ? 3 : 2); // wavefronts per SIMD the registers (and LDS) allow
    // which operands instruction k of a row tile takes: hi.hi and lo.hi of every slice, then hi.lo
    static __device__ __forceinline__ constexpr int a_of(int k) { return DP >= 16 ? (k < NA ? k : 2 * (k - NA)) : 0; }
    static __device__ __forceinline__ constexpr int b_of(int k) { return DP >= 16 ? (k < NA ? k / 2 : NS + (k - NA)) : k; }
};

// grid: one workgroup per (unit of a head's keys, subspace); all subspaces of a unit follow each other on one die,
// whose L2 then serves a key row's cache lines to all of them.
template <typename KT, int DP, bool FULL>
__global__ __launch_bounds__(kEfThreads, (EfShape<KT, DP>::WAVES)) void encode_filter_kernel(const KT *__restrict__ keys,
                                                                      const float *__restrict__ codebooks,
                                                                      uint8_t *__restrict__ codes,
                                                                      int64_t code_stride_bh, int B, int H, int64_t N,
                                                                      int d_k, int m, int d_sub_arg, int blocks_per_bh,
                                                                      int splits)
{
    typedef EfShape<KT, DP> Sh;
    constexpr bool K32 = Sh::K32;
    constexpr int NS = Sh::NS, NA = Sh::NA, NB = Sh::NB, NI = Sh::NI, NL = Sh::NL;
    __shared__ __align__(16) float cn_s[kCentroids];
    __shared__ float red_s[3][kEfWaves];
    __shared__ uint64_t todo_s[kEfWaves][kEfRounds];   // per pair of blocks: the keys that take the exact rule
    __shared__ __align__(16) ef_v8h a_s[Sh::ALDS ? kEfTiles * NA * kWave : 1];

    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int unit = (slot / m) * 8 + xcd;
    if (unit >= H * splits)
        return;
    const int i = slot % m;
    const int h = unit / splits, part = unit % splits;
    const int d_sub = FULL ? DP : d_sub_arg;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int col = lane & 31;   // centroid within a 32-row tile (operand A), key within a block (operand B)
    const int g = lane >> 5;
    const float *cb = codebooks + ((int64_t)h * m + i) * kCentroids * d_sub;

    // ---- the wavefront's key blocks: pairs 2p, 2p + 1 of the head's 32-key blocks, p = first, first + step, ... ----
    const int total_blocks = B * blocks_per_bh;
    const int pairs = (total_blocks + 1) / 2;
    const int step = splits * kEfWaves;
    const int first = part * kEfWaves + wave;
    KT raw[2][NL][4];
    // Where a pair's two blocks start: (b,h) slab, key, and how many of its 32 keys exist.  All of it is uniform over the
    // wavefront (scalar registers); a lane adds its column.
    struct Where {
        int64_t bh, n0;
        int live;
    };
    auto locate = [&](int kb) {
        const int b = kb / blocks_per_bh;
        const int64_t n0 = (int64_t)(kb - b * blocks_per_bh) * 32;
        const int64_t left = N - n0;
        return Where{(int64_t)b * H + h, n0, kb < total_blocks ? (left < 32 ? (int)left : 32) : 0};
    };
    auto fetch_keys = [&](int kb, KT(&dst)[NL][4]) -> Where {
        const Where w = locate(kb);
        // (columns without a key read the block's last key; a block that does not exist reads a key of the first slab)
        const KT *block = w.live ? keys + (w.bh * N + w.n0) * d_k + (int64_t)i * d_sub : keys + (int64_t)h * N * d_k + (int64_t)i * d_sub;
        const int c = col < w.live ? col : (w.live ? w.live - 1 : 0);
        const KT *sub = block + (uint32_t)(c * d_k);
#pragma unroll
        for (int l = 0; l < NL; ++l)
            ef_load4<FULL, KT>(sub, DP >= 16 ? 16 * (l / 2) + 8 * g + 4 * (l % 2) : 4 * l, d_sub, dst[l]);
        return w;
    };
    Where here[2] = {}, ahead[2] = {};
    if (first < pairs) {
        ahead[0] = fetch_keys(2 * first, raw[0]);
        ahead[1] = fetch_keys(2 * first + 1, raw[1]);
    }

    // ---- norms and scales: thread c reads centroid c ----
    float cn = 0.f, cm = 0.f;
    bool bad = false;
#pragma unroll
    for (int j0 = 0; j0 < DP; j0 += 4) {
        float v[4];
        ef_load4<FULL, float>(cb + tid * d_sub, j0, d_sub, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            cn = cn + v[e] * v[e];
            cm = fmaxf(cm, fabsf(v[e]));
            bad |= !(fabsf(v[e]) < INFINITY);
        }
    }
    const uint64_t any_bad = __ballot(bad);
    cm = wave_max(cm);
    const float cw = wave_max(cn);
    if (lane == 0) {
        red_s[0][wave] = cm;
        red_s[1][wave] = cw;
        red_s[2][wave] = any_bad ? 1.f : 0.f;
    }
    __syncthreads();
    float cmax = red_s[0][0], cnmax = red_s[1][0], nbad = red_s[2][0];
#pragma unroll
    for (int w = 1; w < kEfWaves; ++w) {
        cmax = fmaxf(cmax, red_s[0][w]);
        cnmax = fmaxf(cnmax, red_s[1][w]);
        nbad += red_s[2][w];
    }
    int se = 13 - ((int)((__float_as_uint(cmax) >> 23) & 0xffu) - 127);   // 13 - floor(log2(cmax)) for normal numbers
    if (cmax == 0.f)
        se = 13;
    if (se < -60 || se > 60) {
        nbad = 1.f;                    // no key is ever decided by the filter: every one takes the exact rule
        se = se < 0 ? -60 : 60;
    }
    const int ske = K32 ? se - 6 : 0;
    const float sc = __uint_as_float((uint32_t)(se + 127) << 23), sk = __uint_as_float((uint32_t)(ske + 127) << 23);
    const float cns = (sc * cn) * sk;
    cn_s[tid] = cns;
    // Norms as matrix operands: norm = (nh + nm + nl) 2^x, three fp16 terms against 2^x.  x puts the largest near 2^14; where
    // 2^x would leave fp16's normal range and the terms could not hold the norm, the filter decides nothing.
    float xs = 1.f, xinv = 1.f;
    if constexpr (Sh::NORM_SLOTS) {
        const float top = (sc * cnmax) * sk;
        int x = (int)((__float_as_uint(top) >> 23) & 0xffu) - 127 - 14;
        if (top == 0.f)
            x = 0;
        if (x < -28 || x > 15)
            nbad = 1.f;
        x = x < -14 ? -14 : (x > 15 ? 15 : x);
        xs = __uint_as_float((uint32_t)(x + 127) << 23);
        xinv = __uint_as_float((uint32_t)(127 - x) << 23);
    }
    // threshold: tau = t_k |s_k k|^2 + t_c
    const float bound_factor = (float)(K32 ? 4 * DP + 16 : 2 * DP + 4) * 0x1.2p-22f;   // 2.25 (..) 2^-23
    const float t_k = bound_factor * __uint_as_float((uint32_t)(se - ske + 127) << 23);
    const float t_c = nbad != 0.f ? INFINITY : bound_factor * 2.f * ((sc * cnmax) * sk) + 1e-30f;

    // ---- centroid operands ----
    ef_v8h a_r[Sh::ALDS ? 1 : kEfTiles][NA];
    auto split8 = [&](int row, int j0, ef_v8h &hi, ef_v8h &lo) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            float v[4];
            ef_load4<FULL, float>(cb + row * d_sub, j0 + 4 * p, d_sub, v);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float w = -2.f * sc * v[e];                   // exact (powers of two) unless it overflows
                const _Float16 wh = (_Float16)w;
                hi[4 * p + e] = wh;
                lo[4 * p + e] = (_Float16)(w - (float)wh);          // exact difference, then one rounding
            }
        }
    };
    if constexpr (Sh::ALDS) {
#pragma unroll 1
        for (int t = 2 * wave; t < 2 * wave + 2; ++t)
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                ef_v8h hi, lo;
                split8(32 * t + col, 16 * s + 8 * g, hi, lo);
                a_s[(t * NA + 2 * s) * kWave + lane] = hi;
                a_s[(t * NA + 2 * s + 1) * kWave + lane] = lo;
            }
    } else {
#pragma unroll
        for (int t = 0; t < kEfTiles; ++t) {
            ef_v8h hi, lo;
            if constexpr (DP == 4) {
                float v[4];
                ef_load4<FULL, float>(cb + (32 * t + col) * d_sub, 0, d_sub, v);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float w = -2.f * sc * v[e];
                    const _Float16 wh = (_Float16)w;
                    a_r[t][0][e] = wh;
                    a_r[t][0][4 + e] = (_Float16)(w - (float)wh);
                }
            } else if constexpr (DP == 8) {
                split8(32 * t + col, 0, hi, lo);
                a_r[t][0] = g ? lo : hi;
            } else {
                split8(32 * t + col, 8 * g, hi, lo);
                a_r[t][0] = hi;
                a_r[t][1] = lo;
            }
        }
    }
    __syncthreads();   // norms (and operands) are in LDS
    const ef_v4f *cn4 = reinterpret_cast<const ef_v4f *>(cn_s) + g;
    const _Float16 one = (_Float16)xs;
    if constexpr (Sh::NORM_SLOTS) {
#pragma unroll
        for (int t = 0; t < kEfTiles; ++t)
            if (g) {                                  // slots 12..14 (fp16 keys: and nothing in 8..11)
                const float w = cn_s[32 * t + col] * xinv;
                const _Float16 nh = (_Float16)w;
                const float w1 = w - (float)nh;
                const _Float16 nm = (_Float16)w1;
                if constexpr (!K32)
                    a_r[t][0] = ef_v8h{};
                a_r[t][0][4] = nh;
                a_r[t][0][5] = nm;
                a_r[t][0][6] = (_Float16)(w1 - (float)nm);
                a_r[t][0][7] = (_Float16)0.f;
            }
    }

    for (int p = first, round = 0; p < pairs; p += step, ++round) {
        float kpart[2];             // this lane's share of |s_k k|^2 for its column of the two blocks
        float dq[2][4], de[2][4], dt[2][kEfTiles];   // minima over the candidates that share a digit
        // ---- operand B: this lane's part of its keys ----
        ef_v8h kf[2][NB];
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            float ks = 0.f;
            if constexpr (!K32) {
                _Float16 x[NL * 4];
                __builtin_memcpy(x, raw[blk], sizeof(x));
#pragma unroll
                for (int l = 0; l < NL * 2; ++l) {
                    const ef_v2h v = {x[2 * l], x[2 * l + 1]};
                    ks = __builtin_amdgcn_fdot2(v, v, ks, false);
                }
                if constexpr (DP == 4) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        kf[blk][0][e] = g ? (e < 4 ? (_Float16)0.f : (e < 7 ? one : (_Float16)0.f)) : x[e % 4];
                } else {
#pragma unroll
                    for (int s = 0; s < NS; ++s)
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            kf[blk][s][e] = x[8 * s + e];
                }
            } else {
                _Float16 xh[NL * 4], xl[NL * 4];
#pragma unroll
                for (int l = 0; l < NL * 2; ++l) {
                    const float u0 = sk * raw[blk][l / 2][2 * (l % 2)], u1 = sk * raw[blk][l / 2][2 * (l % 2) + 1];
                    ks = __builtin_fmaf(u0, u0, ks);
                    ks = __builtin_fmaf(u1, u1, ks);
                    const ef_v2fp hh = __builtin_amdgcn_cvt_pkrtz(u0, u1);
                    const ef_v2fp ll = __builtin_amdgcn_cvt_pkrtz(u0 - (float)hh[0], u1 - (float)hh[1]);
                    __builtin_memcpy(xh + 2 * l, &hh, 4);
                    __builtin_memcpy(xl + 2 * l, &ll, 4);
                }
                if constexpr (DP == 4) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        kf[blk][0][e] = g ? (e < 4 ? xl[e % 4] : (e < 7 ? one : (_Float16)0.f)) : xh[e % 4];
                } else {
#pragma unroll
                    for (int s = 0; s < NS; ++s)
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            kf[blk][s][e] = xh[8 * s + e];
                            kf[blk][NS + s][e] = xl[8 * s + e];
                        }
                }
            }
            kpart[blk] = ks;
        }
        here[0] = ahead[0];
        here[1] = ahead[1];
        if (p + step < pairs) {   // the next pair's keys arrive while this one is scored
            ahead[0] = fetch_keys(2 * (p + step), raw[0]);
            ahead[1] = fetch_keys(2 * (p + step) + 1, raw[1]);
        }

        float gm[16];               // minima over the row tiles, by accumulator register (4 q + e)
        auto start_tile = [&](int blk, int t, ef_v16f &acc) {
            if constexpr (Sh::NORM_SLOTS) {
                acc = ef_v16f{};
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {   // rows 8q + 4g + (0..3) of the tile start at their norms
                    const ef_v4f c4 = cn4[8 * t + 2 * q];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[4 * q + e] = c4[e];
                }
            }
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                ef_v8h av;
                if constexpr (Sh::ALDS)
                    av = a_s[(t * NA + Sh::a_of(k)) * kWave + lane];
                else
                    av = a_r[t][Sh::a_of(k)];
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, kf[blk][Sh::b_of(k)], acc, 0, 0, 0);
            }
        };
        auto tile_min = [](const ef_v16f &x) {
            const float a = ef_min3(x[0], x[1], x[2]), b = ef_min3(x[3], x[4], x[5]), c = ef_min3(x[6], x[7], x[8]);
            const float d = ef_min3(x[9], x[10], x[11]), e = ef_min3(x[12], x[13], x[14]);
            return ef_min(ef_min3(a, b, c), ef_min3(d, e, x[15]));
        };
        // Row tiles two at a time, first of block 0, then of block 1.  The scheduling barriers keep the accumulators of one
        // step alive at a time: the other wavefronts of the SIMD fill the wait for the matrix instructions (holding the
        // next two tiles in flight as well measured the same at half the wavefronts, and the compiler's own order
        // up to three times the time).
#pragma unroll
        for (int u = 0; u < kEfTiles; ++u) {
            const int blk = u / (kEfTiles / 2), t = 2 * (u % (kEfTiles / 2));
            ef_v16f x0, x1;
            start_tile(blk, t, x0);
            start_tile(blk, t + 1, x1);
            __builtin_amdgcn_sched_barrier(0);
            dt[blk][t] = tile_min(x0);
            dt[blk][t + 1] = tile_min(x1);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                gm[r] = (t == 0) ? ef_min(x0[r], x1[r]) : ef_min3(gm[r], x0[r], x1[r]);
            if (t + 2 == kEfTiles) {
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    dq[blk][x] = ef_min(ef_min3(gm[4 * x], gm[4 * x + 1], gm[4 * x + 2]), gm[4 * x + 3]);
                    de[blk][x] = ef_min(ef_min3(gm[x], gm[4 + x], gm[8 + x]), gm[12 + x]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- lane l now finishes key l % 32 of block l / 32: the two lane halves hold disjoint centroids ----
        auto halves = [](float x0, float x1, float &a, float &b) {   // (block 0, block 1) -> own block's halves 0 and 1
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
            a = __uint_as_float(r[0]);
            b = __uint_as_float(r[1]);
        };
        float best = 0.f, second = INFINITY;
        auto scan = [&](auto &d0, auto &d1, int n) {      // digit of the smallest group minimum; best, second updated
            int digit = 0;
            float s = INFINITY, bst = 0.f;
#pragma unroll
            for (int x = 0; x < n; ++x) {
                float a, b;
                halves(d0[x], d1[x], a, b);
                const float v = ef_min(a, b);
                if (x == 0) {
                    bst = v;
                } else {
                    digit = (v < bst) ? x : digit;
                    s = __builtin_amdgcn_fmed3f(bst, v, s);    // bst <= s: the middle one
                    bst = ef_min(bst, v);
                }
            }
            best = bst;                                        // (every digit's smallest minimum is the smallest score)
            second = fminf(second, s);
            return digit;
        };
        const int iq = scan(dq[0], dq[1], 4);
        const int ie = scan(de[0], de[1], 4);
        const int it = scan(dt[0], dt[1], kEfTiles);
        float half0, half1;
        halves(ef_min(ef_min3(dq[0][0], dq[0][1], dq[0][2]), dq[0][3]), ef_min(ef_min3(dq[1][0], dq[1][1], dq[1][2]), dq[1][3]),
               half0, half1);
        second = fminf(second, fmaxf(half0, half1));
        int code = 32 * it + 8 * iq + 4 * (half1 < half0 ? 1 : 0) + ie;
        float ka, kb2;
        halves(kpart[0], kpart[1], ka, kb2);
        const float kn = (DP >= 16) ? ka + kb2 : ka;           // up to 8 coordinates every lane holds the whole key
        // beyond 2^31 a scaled fp32 key may not fit fp16 (2^15.5 squared); NaN and infinities fail the comparison
        const float tau = (kn < (K32 ? 0x1p31f : INFINITY)) ? t_k * kn + t_c : INFINITY;
        const bool unique = (second - best) > tau;             // false for NaN / inf on either side

        const bool valid = col < (g ? here[1].live : here[0].live);
        const int64_t at0 = here[0].bh * code_stride_bh + here[0].n0 * m, at1 = here[1].bh * code_stride_bh + here[1].n0 * m;
        // keys the filter could not decide: noted, and left for the end
        const uint64_t todo = __ballot(valid && !unique);
        if (lane == 0)
            todo_s[wave][round] = todo;
        if (valid && unique)
            codes[(g ? at1 : at0) + col * m + i] = (uint8_t)code;
    }
    // ---- the exact rule for the noted keys, shared out to the workgroup's wavefronts ----
    __syncthreads();
    int turn = 0;
    for (int w = 0; w < kEfWaves; ++w) {
        const int first_w = part * kEfWaves + w;
        const int rounds = first_w < pairs ? (pairs - first_w + step - 1) / step : 0;
        for (int r0 = 0; r0 < rounds; r0 += kWave) {
            const uint64_t mine = r0 + lane < rounds ? todo_s[w][r0 + lane] : 0ull;
            uint64_t some = __ballot(mine != 0);
            while (some) {
                const int r = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(some));
                some &= some - 1;
                uint64_t todo = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mine >> 32), r) << 32) |
                                (uint32_t)__builtin_amdgcn_readlane((int)mine, r);
                while (todo) {
                    const int l = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(todo));
                    todo &= todo - 1;
                    if ((turn++ & (kEfWaves - 1)) != wave)
                        continue;
                    const Where w2 = locate(2 * (first_w + (r0 + r) * step) + (l >> 5));
                    const int64_t n = w2.n0 + (l & 31);
                    const int exact = ef_exact_code<KT>(keys + (w2.bh * N + n) * d_k + (int64_t)i * d_sub, cb, d_sub, lane);
                    if (lane == 0)
                        codes[w2.bh * code_stride_bh + n * m + i] = (uint8_t)exact;
                }
            }
        }
    }
}

// Workgroups per (head, subspace).  A wavefront pays for the codebook (norms, scale, operands: about as much as kSetup
// pairs of key blocks) before its first key; `resident` workgroups run at once.  The count
// with the least (rounds of workgroups) x (set-up + pairs per wavefront) is taken.
static int64_t ef_splits(int64_t units, int64_t pairs, int64_t resident)
{
    constexpr int64_t kSetup = 4;
    // (a wavefront has room to note the undecided keys of kEfRounds pairs)
    int64_t best = (pairs + kEfWaves * kEfRounds - 1) / (kEfWaves * kEfRounds);
    int64_t best_cost = INT64_MAX;
    for (int64_t s = best; s <= 1024; ++s) {
        const int64_t per_wave = (pairs + s * kEfWaves - 1) / (s * kEfWaves);
        const int64_t rounds = (units * s + resident - 1) / resident;
        const int64_t cost = rounds * (kSetup + per_wave);
        if (cost < best_cost) {
            best_cost = cost;
            best = s;
        }
        if (per_wave == 1)
            break;
    }
    return best;
}

// Launches the filter encoder if the shape has an instance; returns false otherwise.
template <typename KT>
static bool launch_encode_filter_t(const lookat_shape *s, int64_t N, const void *keys, const float *codebooks,
                                   uint8_t *codes, int64_t code_stride_bh, hipStream_t st)
{
    const int d_sub = s->d_k / s->m;
    const int64_t blocks_per_bh = (N + 31) / 32;
    const int64_t total_blocks = (int64_t)s->B * blocks_per_bh;
    // One coordinate: 256 centroids on a line leave a quarter of the keys between two that the bound cannot tell apart, and
    // the exact scan of them all is faster (320 (b,h) x 2787 fp16 keys, 32 subspaces: 1.46 ms; with the filter 13.0 ms).
    if (d_sub < 2 || d_sub > 64 || total_blocks > 0x3fffffff)
        return false;
    const int64_t resident = 256 * (d_sub <= 4    ? EfShape<KT, 4>::WAVES
                                    : d_sub <= 8  ? EfShape<KT, 8>::WAVES
                                    : d_sub <= 16 ? EfShape<KT, 16>::WAVES
                                    : d_sub <= 32 ? EfShape<KT, 32>::WAVES
                                                  : EfShape<KT, 64>::WAVES);
    const int64_t splits = ef_splits((int64_t)s->H * s->m, (total_blocks + 1) / 2, resident);
    const int64_t wgs = ((int64_t)s->H * splits + 7) / 8 * 8 * s->m;
    if (wgs > 0xffffff)   // (a grid of 2^32 threads)
        return false;
    const dim3 grid((unsigned)wgs), block(kEfThreads);
    const KT *k = static_cast<const KT *>(keys);
#define LOOKAT_EF_LAUNCH(D, FULL)                                                                                         \
    hipLaunchKernelGGL((encode_filter_kernel<KT, D, FULL>), grid, block, 0, st, k, codebooks, codes, code_stride_bh,      \
                       s->B, s->H, N, s->d_k, s->m, d_sub, (int)blocks_per_bh, (int)splits)
#define LOOKAT_EF_CASE(D)                                                                                                 \
    if (d_sub == D) {                                                                                                     \
        LOOKAT_EF_LAUNCH(D, true);                                                                                        \
        return true;                                                                                                      \
    }                                                                                                                     \
    if (d_sub < D) {                                                                                                      \
        LOOKAT_EF_LAUNCH(D, false);                                                                                       \
        return true;                                                                                                      \
    }
    LOOKAT_EF_CASE(4)
    LOOKAT_EF_CASE(8)
    LOOKAT_EF_CASE(16)
    LOOKAT_EF_CASE(32)
    LOOKAT_EF_CASE(64)
#undef LOOKAT_EF_CASE
#undef LOOKAT_EF_LAUNCH
    return false;
}

bool launch_encode_filter(const lookat_shape *s, int64_t N, const void *keys, int key_dtype, const float *codebooks,
                          uint8_t *codes, int64_t code_stride_bh, hipStream_t st)
{
    return (key_dtype == LOOKAT_F16)
               ? launch_encode_filter_t<__half>(s, N, keys, codebooks, codes, code_stride_bh, st)
               : launch_encode_filter_t<float>(s, N, keys, codebooks, codes, code_stride_bh, st);
}

}  // namespace lookat
