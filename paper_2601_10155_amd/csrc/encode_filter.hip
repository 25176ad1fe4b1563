// Key encoding (paper Sec. 3.4, "Encoding") for many keys per head: a matrix-core filter in
// front of the exact fp64 rule.
//
// The code of a key sub-vector k is argmin_c d(k, C[c]) with d evaluated in fp64, one rounding per
// subtract / multiply / add, coordinates ascending, lowest index on ties.  Evaluating d for all 256
// centroids costs 3 fp64 operations per coordinate and centroid.  Here the 256 candidates are
// first ranked with
//     a_c = |C'[c]|^2 - 2 k'.C'[c]        ( = |k' - C'[c]|^2 - |k'|^2 up to rounding )
// computed on the matrix cores (rows = 32 centroids, columns = 32 keys, the norm as the accumulator's initial value) from
// operands k', C' that stand for the key and the centroids in fp16.  The candidates whose a_c lies within a bound tau of
// the smallest are the only ones that the exact rule can choose.  If there is one, it is the code; otherwise (near ties,
// exact ties, NaN or infinite inputs: one or two sub-vectors in a hundred on the workloads here) the exact rule is evaluated
// over these candidates, two of 256 as a rule.  Either way the code is the one the exact scan produces, bit for bit.
//
// The operands.  Codebook entries are scaled by a power of two s_c (largest entry near 2^13); fp32 keys by s_k = s_c 2^-6 (a
// key as large as the largest centroid entry lands near 2^7, which leaves a factor of 500 to fp16's largest value; longer keys
// go to the exact rule), fp16 keys enter as they are (s_k = 1).  v_mfma_f32_32x32x16_f16 contracts sixteen slots at a time:
//   * sub-vectors of 16 and more coordinates enter as ONE fp16 term each, keys and centroids, one instruction per 16
//     coordinates; the norms are those of the rounded centroids, so that a_c is a distance between rounded points;
//   * sub-vectors of up to 8 have room for two terms of a centroid, -2 s_c C = hi + lo, |error| <= 2^-22 |2 s_c C|, beside
//     one term of the key;
//   * sub-vectors of up to 4 have room for both terms of both, and for the norm;
//   * launches of few pairs of key blocks per wavefront (FINE) take both terms of everything, in more instructions: there
//     the undecided keys' round trip to memory would be a fifth of the launch.
//
// Error bound.  Let delta be a bound on |k - k'| + max_c |C[c] - C'[c]| (exact differences, squared and summed in fp32, with
// 1.002 for the rounding of the sums).  By the triangle inequality the exact argmin a and the smallest a_b satisfy
//     |k' - C'[a]| <= |k - C[a]| + delta <= |k - C[b]| + delta <= |k' - C'[b]| + 2 delta,
// so with d = |k' - C'[b]| = sqrt(a_b + |k'|^2) no candidate beyond a_b + 4 delta (d + delta) can be the argmin.  To this
// comes the fp32 rounding of a_c: a sum of n terms (d_sub + 1; 2 d_sub + 1 and 4 d_sub + 1 with two terms of the centroids
// and of both, whose dropped terms amount to at most 2, respectively 14, more 2^-23) whose magnitudes add up to at most
// S = |k'|^2 + 2 max_c |C'[c]|^2 (since 2|k.C| <= |k|^2 + |C|^2) times 1 + 2^-9.  With at most 2^-23 relative error per
// accumulation step (round-to-nearest would give 2^-24) and norms summed in fp64 the error is at most E = (n + 3) 2^-23 S (n + 15 with
// fp32 keys in two terms).  tau = 2.25 E + 4.01 delta (d + delta): twice E for the two candidates, the rest for S, for the rounding of
// tau and of the limit and for d (whose square takes tau instead of E); plus 1e-30 for flushed denormals.  An infinite or NaN limit, fp32
// keys beyond fp16's range after scaling and a codebook whose scale would leave [2^-60, 2^60] make every centroid a candidate.
//
// Which candidates.  128 scores per lane and block of 32 keys have to be looked at.  A candidate's index is written as
// digits (row tile t, quarter q, lane half h, element e: index = 32 t + 8 q + 4 h + e) and only group minima are formed, over the
// candidates that share (q, e) and over those that share t, three operands at a time (v_minimum3_f32): one instruction per candidate
// for both.  A digit value whose group minimum exceeds the limit holds no candidate; the remaining values of 2q + h, e and t, as bits of
// a word, give every combination that can be one.  One bit per digit: the key is decided, and the bits are its code.  A NaN anywhere
// makes the minima NaN (v_minimum3 propagates it).  Two blocks of 32 keys are finished together, one per lane half.
// An undecided key is noted with its word in LDS; when the pairs are through, eight lanes share a noted key's combinations.  A key that
// fills a large part of the notes is decided once: with half of the keys zero and a centroid near zero that has a rival (2 codebooks in a
// hundred), 32 x 12 x 1024 fp32 keys, 4 of 16, took 102 us where every copy was worked off, 51 now, and 42 without such keys.
//
// What bounds it: vector issue and power.  A pair of blocks costs 410 to 480 vector instructions, 256 of them a candidate's minima and 48
// those that form the digits; matrix instructions of one wavefront hide behind another's minima, but the chip lowers its clock for them (a
// loop like this one with four wavefronts per SIMD and operands and norms from LDS or registers as they fit takes 823 ns per block and
// SIMD at 1.48 GHz with the three instructions per tile that two terms of both need, 514 at 1.80 with one), and reads of norms from LDS
// count as well (with two wavefronts 478 ns, 421 from registers).  Hence one term, norms (and operands, where they fit) in registers, two
// wavefronts per SIMD, both blocks sharing what is still read; a spilled register in the loop costs far more than it saves, since its reload
// waits for the key requests ahead of it (no instance spills).  Wavefronts take their pairs from a shared counter: the SIMD favours its oldest
// wavefront, and with fixed shares the last one ran alone for a third of the time.
//   Measured (us per call, this kernel / the one with two terms of everything, norms and operands from LDS, 256 centroids exactly for
// every undecided key): 4 x 32 heads x 2048 fp16 keys, 16 subspaces of 8: 74 / 85; 32 x 12 heads x 1024 fp32 keys, 4 of 16: 42 / 62;
// 32 heads x 16384 fp32 keys, 8 of 16: 95 / 135; 8 x 16 x 2048, d_k = 128: fp16 8 of 16 45 / 59, 4 of 32 35 / 54, 2 of 64 33 / 57;
// fp32 4 of 32 41 / 72, 2 of 64 43 / 80; 8 x 16 x 2048 keys, 8 of 6, 12 and 28 coordinates: fp16 46 / 66, 53 / 61, 70 / 102, fp32 60 / 83,
// 57 / 77, 81 / 141.  Small ones: 24 (b,h) x 100 keys, fp16 8 of 16: 6.9 / 7.2 (with one term 8.5).
//
// This translation unit must be compiled with -ffp-contract=off (the exact rule).
#include <cstdlib>
#include <type_traits>

#include "common.h"
#include "encode_grid.h"

#pragma clang fp contract(off)

namespace lookat {

typedef float ef_v16f __attribute__((ext_vector_type(16)));
typedef float ef_v4f __attribute__((ext_vector_type(4)));
typedef _Float16 ef_v8h __attribute__((ext_vector_type(8)));
typedef _Float16 ef_v2h __attribute__((ext_vector_type(2)));
typedef __fp16 ef_v2fp __attribute__((ext_vector_type(2)));

constexpr int kEfTiles = kCentroids / 32;
// Undecided keys a wavefront can note before they are worked off.  (832: up to 16 coordinates the LDS stays below 64 KB and one base
// register reaches all of it; with 1024 the fp32 form of 16 spilled.)
constexpr int kEfList = 832;
constexpr int kEfShared = 48;           // candidates that eight lanes share; for a key with more the whole wavefront takes all centroids
constexpr int kEfMore = 1 << 16;       // flag beside the number of noted keys: the wavefront has pairs left
constexpr uint32_t kEfAll = 0xfffffu;  // every value of every digit: 2q + h in bits 0..7, e in 8..11, t in 12..19

template <typename T>
__device__ __forceinline__ float ef_to_f32(T v);
template <>
__device__ __forceinline__ float ef_to_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float ef_to_f32<__half>(__half v) { return __half2float(v); }

__device__ __forceinline__ float ef_min(float a, float b) { return __builtin_elementwise_minimum(a, b); }
__device__ __forceinline__ float ef_min3(float a, float b, float c) { return ef_min(ef_min(a, b), c); }

// Coordinates j0 .. j0+3 of a sub-vector whose length d_sub is a multiple of four, zero past its end.  FULL: all four exist and the start
// is a multiple of four elements from a 16-byte aligned row.
template <bool FULL, typename T>
__device__ __forceinline__ void ef_load4(const T *sub, int j0, int d_sub, T (&out)[4])
{
    typedef unsigned int chunk_t __attribute__((ext_vector_type(sizeof(T))));   // 4 elements: 8 or 16 bytes
    chunk_t v = {};
    if (FULL || j0 < d_sub)
        v = *reinterpret_cast<const chunk_t *>(sub + j0);
    __builtin_memcpy(out, &v, sizeof(v));
}

// The same for the other lengths and two-byte elements, in two steps, so that nothing is done with a request before it is due (elements
// that are requested one by one are packed in pairs as they arrive, and the pair loop waited for the next pair's keys; us per call, so / now:
// 8 x 16 x 2048 keys, 8 subspaces of 10 78.5 / 57.2, of 14 83.1 / 56.2, of 6 61.7 / 44.0; 32 x 16 x 2116, 32 of 3 705 / 601): the last
// four coordinates of the sub-vector where j0 .. j0+3 reach past its end (of two or three: the first two, then the last one), ..
template <typename T>
__device__ __forceinline__ void ef_load_tail(const T *sub, int j0, int d_sub, T (&out)[4])
{
    static_assert(sizeof(T) == 2, "two-byte elements");
    struct __attribute__((packed, aligned(2))) two_t { uint32_t v; };
    struct __attribute__((packed, aligned(2))) four_t { uint64_t v; };
    uint64_t v;
    if (d_sub < 4)
        v = (uint64_t)reinterpret_cast<const two_t *>(sub)->v | (uint64_t)*reinterpret_cast<const uint16_t *>(sub + d_sub - 1) << 32;
    else
        v = reinterpret_cast<const four_t *>(sub + (j0 < d_sub - 4 ? j0 : d_sub - 4))->v;
    __builtin_memcpy(out, &v, sizeof(v));
}
// .. shifted to where they belong.
template <typename T>
__device__ __forceinline__ void ef_align_tail(T (&x)[4], int j0, int d_sub)
{
    uint64_t v;
    __builtin_memcpy(&v, x, sizeof(v));
    const int past = j0 + 4 - d_sub;
    if (d_sub < 4)
        v = j0 ? 0 : (d_sub == 3 ? v : v & 0xffffffffu);
    else
        v = past >= 4 ? 0 : v >> (past > 0 ? 16 * past : 0);
    __builtin_memcpy(x, &v, sizeof(v));
}

// Coordinates j0 .. j0+N-1 of a sub-vector of d_sub coordinates, and of M rows of the codebook beside it, all requested at once: past the
// end the last ones again, which the callers leave out.  (With a branch around every piece that may not be there the compiler waits for
// each before the next.  us per call, so / now: 32 heads x 8000 keys, 2 subspaces of 40, fp16 48.4 / 38.4, fp32 66.6 / 54.2; 8 x 16 x 2048,
// 4 of 48, fp32 116 / 95; 8 of 12 71 / 63; eight rounds of the exact rule over 40 coordinates 27 / 14.)
template <int N, int M, typename T, typename R>
__device__ __forceinline__ void ef_load_clamped(const T *x_sub, const R *const (&rows)[M], int j0, int d_sub, T (&x)[N], R (&y)[M][N])
{
    if (d_sub % 4 == 0) {
        typedef unsigned int chunk_t __attribute__((ext_vector_type(sizeof(T))));   // 4 elements: 8 or 16 bytes
        typedef unsigned int row_t __attribute__((ext_vector_type(sizeof(R))));
        chunk_t xv[N / 4];
        row_t yv[M][N / 4];
#pragma unroll
        for (int q = 0; q < N / 4; ++q) {
            const int at = j0 + 4 * q < d_sub ? j0 + 4 * q : d_sub - 4;
            xv[q] = *reinterpret_cast<const chunk_t *>(x_sub + at);
#pragma unroll
            for (int u = 0; u < M; ++u)
                yv[u][q] = *reinterpret_cast<const row_t *>(rows[u] + at);
        }
        __builtin_memcpy(x, xv, sizeof(x));
        __builtin_memcpy(y, yv, sizeof(y));
    } else {
        constexpr int kUsed = N == 4 ? 3 : N;      // (lengths of up to four that are not four)
#pragma unroll
        for (int e = 0; e < kUsed; ++e) {
            const int at = j0 + e < d_sub ? j0 + e : d_sub - 1;
            x[e] = x_sub[at];
#pragma unroll
            for (int u = 0; u < M; ++u)
                y[u][e] = rows[u][at];
        }
        if constexpr (kUsed < N) {
            x[kUsed] = x[0];
#pragma unroll
            for (int u = 0; u < M; ++u)
                y[u][kUsed] = y[u][0];
        }
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
    const float *rows[NC];
#pragma unroll
    for (int u = 0; u < NC; ++u)
        rows[u] = cb + (u * kWave + lane) * d_sub;
    for (int j0 = 0; j0 < d_sub; j0 += JB) {
        float y[NC][JB];
        KT x[JB];
        ef_load_clamped(key_sub, rows, j0, d_sub, x, y);
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

// Squared distance by the exact rule: fp64, one rounding per subtract, multiply and add, coordinates ascending.  (32 of them requested at once: with
// 16, fills of 32 and 64 coordinates took 1 to 10% longer, with 64 registers spill.  Lengths of 33 to 63 take 16, as the last round also requests what
// is not there, 64 coordinates for 40 with 32 a round: 250 undecided fp32 keys of 40 18.5 / 13.5 us.  Four lanes to a key with two candidates
// each instead of eight: 5 to 20% slower from 16 coordinates on, the chain of additions counts and not the round trip.)
template <typename KT, int DP, bool FULL>
__device__ __forceinline__ double ef_exact_distance(const KT *key_sub, const float *row, int d_sub)
{
    constexpr int JB = DP < 32 ? DP : (DP == 64 && !FULL ? 16 : 32);
    double acc = 0.0;
    const float *rows[1] = {row};
#pragma unroll 1
    for (int j0 = 0; j0 < d_sub; j0 += JB) {
        KT x[JB];
        float y[1][JB];
        if constexpr (FULL) {
#pragma unroll
            for (int q = 0; q < JB; q += 4) {
                KT x4[4];
                float y4[4];
                ef_load4<true, KT>(key_sub, j0 + q, d_sub, x4);
                ef_load4<true, float>(row, j0 + q, d_sub, y4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[q + e] = x4[e];
                    y[0][q + e] = y4[e];
                }
            }
        } else {
            ef_load_clamped(key_sub, rows, j0, d_sub, x, y);
        }
#pragma unroll
        for (int q = 0; q < JB; ++q)
            if (FULL || j0 + q < d_sub) {
                const double diff = (double)ef_to_f32<KT>(x[q]) - (double)y[0][q];
                const double sq = diff * diff;
                acc = acc + sq;
            }
    }
    return acc;
}

// Whether key sub-vectors x[u] hold the bits of `one`.
template <int DP, bool FULL, int M, typename KT>
__device__ __forceinline__ void ef_same_key(const KT *one, const KT *const (&x)[M], int d_sub, bool (&same)[M])
{
    constexpr int JB = DP < 16 ? DP : 16;
    typedef unsigned int word_t __attribute__((ext_vector_type(JB * sizeof(KT) / 4)));
    uint32_t differ[M] = {};
#pragma unroll 1
    for (int j0 = 0; j0 < d_sub; j0 += JB) {
        KT a[JB], b[M][JB];
        if constexpr (FULL) {
#pragma unroll
            for (int q = 0; q < JB; q += 4) {
                ef_load4<true, KT>(one, j0 + q, d_sub, reinterpret_cast<KT(&)[4]>(a[q]));
#pragma unroll
                for (int u = 0; u < M; ++u)
                    ef_load4<true, KT>(x[u], j0 + q, d_sub, reinterpret_cast<KT(&)[4]>(b[u][q]));
            }
        } else {
            ef_load_clamped(one, x, j0, d_sub, a, b);
        }
        word_t wa, wb;
        __builtin_memcpy(&wa, a, sizeof(a));
#pragma unroll
        for (int u = 0; u < M; ++u) {
            __builtin_memcpy(&wb, b[u], sizeof(a));
#pragma unroll
            for (int k = 0; k < (int)(JB * sizeof(KT) / 4); ++k)
                differ[u] |= wa[k] ^ wb[k];
        }
    }
#pragma unroll
    for (int u = 0; u < M; ++u)
        same[u] = differ[u] == 0;
}

// Index of the n-th set bit (n from 0, below the number of set bits) of an eight-bit word.
__device__ __forceinline__ int ef_nth_bit(uint32_t bits, int n)
{
    int at = 0;
#pragma unroll
    for (int width = 4; width >= 1; width >>= 1) {
        const uint32_t low = bits >> at & ((1u << width) - 1u);
        const int c = __builtin_popcount(low);
        const bool up = n >= c;
        n = up ? n - c : n;
        at = up ? at + width : at;
    }
    return at;
}

// (value, index) of the lane that the DPP control selects, taken where it is the smaller one (lowest index on ties).
template <int CTRL>
__device__ __forceinline__ void ef_argmin_step(double &best, int &code)
{
    const uint64_t u = (uint64_t)__double_as_longlong(best);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)u, (int)(uint32_t)u, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(u >> 32), (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, false);
    const double d = __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    const int c = __builtin_amdgcn_update_dpp(code, code, CTRL, 0xf, 0xf, false);
    if (d < best || (d == best && c < code)) {
        best = d;
        code = c;
    }
}

// Matrix operands of a (head, subspace): slices of 16 slots; lane (col, g) of an operand holds slots 8g .. 8g+7 of its
// row (centroid) or column (key).
//   DP >= 16: slice s carries coordinates 16s .. 16s+15, one fp16 term each; FINE: two terms each, in two operands;
//   DP == 8:  hi terms of the centroids in slots 0..7, lo terms in 8..15; the key's single term stands twice; FINE: its
//             second term in an operand of its own;
//   DP == 4:  slots hi(4) lo(4) hi(4) norm(3); the key's hi terms in slots 0..7, its lo terms (fp32 keys;
//             zero for fp16 keys) in 8..11, 2^x against the norm's three terms.
// FINE leaves no term out, as DP == 4: for launches of few pairs, where the undecided keys' extra round trip to memory is what
// counts and not the matrix instructions.
template <typename KT, int DP, bool FULL, bool FINE>
struct EfShape {
    static constexpr bool K32 = std::is_same<KT, float>::value;
    static constexpr int NS = DP >= 16 ? DP / 16 : 1;              // slices
    static constexpr int NL = DP == 4 ? 1 : 2 * NS;                // 4-coordinate pieces a lane loads of a key
    static constexpr bool SLOTS = DP == 4;                         // the norm sits in spare slots, else it starts the accumulator
    static constexpr bool KLO = K32 && DP >= 8 && !FINE;           // the keys' lo terms are left out and bounded
    static constexpr bool CLO = DP >= 16 && !FINE;                 // the centroids' lo terms are left out and bounded
    static constexpr int NA = DP >= 16 && FINE ? 2 : 1;            // operands per slice: centroids
    static constexpr int NB = K32 && DP >= 8 && FINE ? 2 : 1;      //                     keys
    static constexpr bool AHEAD = !(K32 && DP == 64) && !FINE;     // a tile pair's operands are read from LDS before they are due
    static constexpr int NREG = (DP == 8 || DP == 16) && !FINE ? (K32 && DP == 16 ? (FULL ? 5 : 4) : 6) : 0;   // tiles whose norms stay in registers (16 each)
    static constexpr bool NTWICE = DP == 64 && (K32 || !FULL) && !FINE;   // norms are read for each block: registers that hold them for both spill others
    static constexpr bool AREG = DP <= 8 || (DP == 16 && !K32 && !FINE);   // centroid operands in 32 registers, else read from LDS
};

// grid: one workgroup per (unit of a head's keys, subspace); all subspaces of a unit follow each other on one die,
// whose L2 then serves a key row's cache lines to all of them.
template <typename KT, int DP, bool FULL, int THREADS, bool FINE>
__global__ __launch_bounds__(THREADS, (DP == 4 ? 3 : FINE && DP == 64 ? 1 : 2)) void encode_filter_kernel(const KT *__restrict__ keys,
                                                                      const float *__restrict__ codebooks,
                                                                      uint8_t *__restrict__ codes,
                                                                      int64_t code_stride_bh, int B, int H, int64_t N,
                                                                      int d_k, int m, int d_sub_arg, uint32_t blocks_per_bh,
                                                                      uint32_t per_block /* floor((2^32 - 1) / blocks_per_bh) */,
                                                                      int splits, int pairs_per_wg)
{
    typedef EfShape<KT, DP, FULL, FINE> Sh;
    constexpr bool K32 = Sh::K32;
    constexpr int NS = Sh::NS, NL = Sh::NL, NA = Sh::NA, NB = Sh::NB;
    constexpr int kEfWaves = THREADS / kWave;
    static_assert(THREADS >= kCentroids, "thread c looks after centroid c while the codebook is set up");
    __shared__ __align__(16) float cn_s[kCentroids];
    __shared__ float red_s[4][kCentroids / kWave];
    __shared__ int next_s, repeated_s, count_s[kEfWaves];
    __shared__ uint2 list_s[kEfWaves][kEfList];        // undecided keys: (local pair, lane), candidate digits
    __shared__ __align__(16) ef_v8h a_s[kEfTiles * NS * NA * kWave];

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

    // ---- the workgroup's key blocks: pairs 2p, 2p + 1 of the head's 32-key blocks, p = first .. first + mine - 1 ----
    const uint32_t total_blocks = (uint32_t)B * blocks_per_bh;
    const int pairs = (int)(total_blocks + 1) / 2;
    const int first = part * pairs_per_wg;
    const int mine = pairs - first < pairs_per_wg ? pairs - first : pairs_per_wg;
    if (mine <= 0)
        return;
    KT raw[2][NL][4];
    // Where a block lies: batch entry, number within it, and how many of its 32 keys exist.  A pair's are uniform over the wavefront (scalar
    // registers; a lane adds its column), and all that is worked out for each pair is one product for the quotient, corrected once (below
    // 2^30 the estimate is at most one short), and two for either address: what the scalar unit does the wavefront waits for (a generic
    // division per block and two full 64-bit address sums, 215 scalar instructions a pair; now 154: 32 x 12 x 1024 fp32 keys, 4 of 16, 42.8 / 41.8
    // us, 4 x 32 x 2048 fp16, 16 of 8 77.5 / 76.6, 32 x 16384 fp32, 8 of 16 105 / 101).
    struct Where {
        uint32_t b, lb;
        int live;
    };
    const int tail = (int)(N - (int64_t)(blocks_per_bh - 1) * 32);       // keys of a batch entry's last block
    auto live_of = [&](uint32_t lb) { return lb == blocks_per_bh - 1 ? tail : 32; };
    auto locate = [&](uint32_t kb) {
        uint32_t b = __umulhi(kb, per_block), lb = kb - b * blocks_per_bh;
        if (lb >= blocks_per_bh) {
            ++b;
            lb -= blocks_per_bh;
        }
        return Where{b, lb, live_of(lb)};
    };
    auto after = [&](const Where &w, uint32_t kb) {      // the block behind w, number kb; one that does not exist has no keys and lies where w does
        if (kb >= total_blocks)
            return Where{w.b, w.lb, 0};
        const bool over = w.lb + 1 == blocks_per_bh;
        const uint32_t lb = over ? 0 : w.lb + 1;
        return Where{w.b + (over ? 1u : 0u), lb, live_of(lb)};
    };
    const KT *keys_h = keys + (int64_t)h * N * d_k + (int64_t)i * d_sub;
    uint8_t *codes_h = codes + h * code_stride_bh + i;
    const uint64_t keys_b = (uint64_t)H * (uint64_t)N * (uint32_t)d_k, codes_b = (uint64_t)H * (uint64_t)code_stride_bh;
    auto keys_at = [&](const Where &w) { return keys_h + (w.b * keys_b + (uint64_t)w.lb * (32u * (uint32_t)d_k)); };
    auto codes_at = [&](const Where &w) { return codes_h + (w.b * codes_b + (uint64_t)w.lb * (32u * (uint32_t)m)); };
    const bool whole = FULL || d_sub % 4 == 0;    // pieces of four coordinates: all of one or nothing
    auto piece = [&](int l) { return DP >= 16 ? 16 * (l / 2) + 8 * g + 4 * (l % 2) : 4 * l; };   // its first coordinate
    auto fetch_keys = [&](const Where &w, KT(&dst)[NL][4]) {
        // (columns without a key read the block's last key)
        const int c = col < w.live ? col : (w.live ? w.live - 1 : 0);
        const KT *sub = keys_at(w) + (uint32_t)(c * d_k);
        if (FULL || whole) {
#pragma unroll
            for (int l = 0; l < NL; ++l)
                ef_load4<FULL, KT>(sub, piece(l), d_sub, dst[l]);
        } else if constexpr (K32) {
#pragma unroll
            for (int l = 0; l < NL; ++l)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    dst[l][e] = piece(l) + e < d_sub ? sub[piece(l) + e] : 0.f;
        } else {
#pragma unroll
            for (int l = 0; l < NL; ++l)
                ef_load_tail(sub, piece(l), d_sub, dst[l]);
        }
    };
    // The first pair's keys are requested behind the codebook's rows, which everything waits for and L2 holds.  Padded lengths take the keys first:
    // their rows are more requests than they need (whole pieces past the end, or coordinate by coordinate), which the keys would wait for.  1800
    // drawn fills of nine padded lengths, rows first / keys first against one order for all: geometric means 0.98 / 0.98, at worst 1.14 (640 (head,
    // subspace) pairs x 76 fp32 keys of 6) / 1.04; 40 and 48 coordinates, fp32, 1.04 / 1.00.
    constexpr bool kRowsFirst = FULL;
    Where here[2] = {}, ahead[2] = {};
    auto fetch_pair = [&](int pair) {
        const uint32_t kb = 2u * (uint32_t)(first + pair);
        ahead[0] = locate(kb);
        ahead[1] = after(ahead[0], kb + 1);
        fetch_keys(ahead[0], raw[0]);
        fetch_keys(ahead[1], raw[1]);
    };
    int p = wave, pn = wave + kEfWaves;     // this wavefront's pair, and the next one
    if constexpr (!kRowsFirst) {
        if (p < mine)
            fetch_pair(p);
    }
    if (tid == 0)
        next_s = 2 * kEfWaves;

    // ---- scale, operands, norms: thread c < 256 looks after centroid c ----
    const bool owner = tid < kCentroids;
    float v[DP];
    float cm = 0.f;
    bool bad = false;
    if (owner) {
        const float *row = cb + tid * d_sub;
        if constexpr (FULL) {
#pragma unroll
            for (int j0 = 0; j0 < DP; j0 += 4) {
                float v4[4];
                ef_load4<true, float>(row, j0, d_sub, v4);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[j0 + e] = v4[e];
            }
        } else if (whole) {
            ef_v4f piece4[DP / 4];
#pragma unroll
            for (int q = 0; q < DP / 4; ++q)
                piece4[q] = *reinterpret_cast<const ef_v4f *>(row + (4 * q < d_sub ? 4 * q : d_sub - 4));
#pragma unroll
            for (int j = 0; j < DP; ++j)
                v[j] = j < d_sub ? piece4[j / 4][j % 4] : 0.f;
        } else {
#pragma unroll
            for (int j = 0; j < DP; ++j)
                v[j] = j < d_sub ? row[j] : 0.f;
        }
    }
    // (without a branch, so that the rows can be waited for alone)
    if constexpr (kRowsFirst) {
        __builtin_amdgcn_sched_barrier(0);
        fetch_pair(p < mine ? p : mine - 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (owner) {
#pragma unroll
        for (int j = 0; j < DP; ++j) {
            cm = fmaxf(cm, fabsf(v[j]));
            bad |= !(fabsf(v[j]) < INFINITY);
        }
        const uint64_t any_bad = __ballot(bad);
        cm = wave_max(cm);
        if (lane == 0) {
            red_s[0][wave] = cm;
            red_s[1][wave] = any_bad ? 1.f : 0.f;
        }
    }
    __syncthreads();
    float cmax = red_s[0][0], nbad = red_s[1][0];
#pragma unroll
    for (int w = 1; w < kCentroids / kWave; ++w) {
        cmax = fmaxf(cmax, red_s[0][w]);
        nbad += red_s[1][w];
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
    if (owner) {
        const float unscale = __uint_as_float((uint32_t)(ske - se - 2 + 127) << 23);   // |2 s_c C|^2 -> s_c s_k |C|^2
        ef_v8h row[DP == 4 ? 1 : DP / 8], low[DP == 4 ? 1 : DP / 8];
        double n2 = 0.0;
        float rest = 0.f;
#pragma unroll
        for (int j = 0; j < DP; ++j) {
            const float w = -2.f * sc * v[j];                   // exact (powers of two) unless it overflows
            const _Float16 wh = (_Float16)w;
            const float r = w - (float)wh;                      // exact
            if constexpr (Sh::CLO) {
                row[j / 8][j % 8] = wh;
                rest = __builtin_fmaf(r, r, rest);
                n2 += (double)(float)wh * (double)(float)wh;
            } else {
                n2 += (double)w * (double)w;
                if constexpr (DP >= 8) {
                    row[j / 8][j % 8] = wh;
                    low[j / 8][j % 8] = (_Float16)r;
                } else {
                    row[0][j] = wh;
                    row[0][4 + j] = (_Float16)r;
                }
            }
        }
        const float cns = (float)n2 * unscale;
        cn_s[tid] = cns;
        ef_v8h *at = a_s + tid / 32 * NS * NA * kWave + col;    // (row `col` of tile tid / 32)
        if constexpr (DP >= 16) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                at[s * NA * kWave] = row[2 * s];
                at[s * NA * kWave + 32] = row[2 * s + 1];
                if constexpr (NA == 2) {
                    at[(2 * s + 1) * kWave] = low[2 * s];
                    at[(2 * s + 1) * kWave + 32] = low[2 * s + 1];
                }
            }
        } else {
            at[0] = row[0];
            if constexpr (DP == 8)
                at[32] = low[0];
        }
        const float cw = wave_max(cns), rw = wave_max(rest * unscale);
        if (lane == 0) {
            red_s[2][wave] = cw;
            red_s[3][wave] = rw;
        }
    }
    __syncthreads();
    float cnmax = red_s[2][0], restmax = red_s[3][0];
#pragma unroll
    for (int w = 1; w < kCentroids / kWave; ++w) {
        cnmax = fmaxf(cnmax, red_s[2][w]);
        restmax = fmaxf(restmax, red_s[3][w]);
    }
    // Norms as matrix operands: norm = (nh + nm + nl) 2^x, three fp16 terms against 2^x.  x puts the largest near 2^14; where
    // 2^x would leave fp16's normal range and the terms could not hold the norm, the filter decides nothing.
    float xs = 1.f;
    if constexpr (Sh::SLOTS) {
        int x = (int)((__float_as_uint(cnmax) >> 23) & 0xffu) - 127 - 14;
        if (cnmax == 0.f)
            x = 0;
        if (x < -28 || x > 15)
            nbad = 1.f;
        x = x < -14 ? -14 : (x > 15 ? 15 : x);
        xs = __uint_as_float((uint32_t)(x + 127) << 23);
        if (owner) {
            ef_v8h hi = {};                                  // slots 8..11 (fp16 keys: nothing there), 12..14
            if constexpr (K32) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    hi[e] = (_Float16)(-2.f * sc * v[e]);
            }
            const float w = cn_s[tid] * __uint_as_float((uint32_t)(127 - x) << 23);
            const _Float16 nh = (_Float16)w;
            const float w1 = w - (float)nh;
            const _Float16 nm = (_Float16)w1;
            hi[4] = nh;
            hi[5] = nm;
            hi[6] = (_Float16)(w1 - (float)nm);
            a_s[tid / 32 * kWave + 32 + col] = hi;
        }
        __syncthreads();
    }
    const _Float16 one = (_Float16)xs;
    float minus_one = -1.f;
    asm("" : "+s"(minus_one));   // (kept from the compiler: a mixed-precision multiply-add instead of two instructions)
    // limit: tau = (t_k kn + t_c) + 4 delta (d + delta), kn = |s_k k|^2 (see the header)
    const float ratio = __uint_as_float((uint32_t)(se - ske + 127) << 23);             // s_c / s_k
    constexpr int kTerms = DP == 4 || FINE ? (K32 ? 4 * DP + 16 : 2 * DP + 4) : (DP == 8 ? 2 * DP + 4 : DP + 4);
    constexpr float kBound = (float)kTerms * 0x1.2p-22f;                               // 2.25 (..) 2^-23
    const float t_k = kBound * ratio;
    const float t_c = nbad != 0.f ? INFINITY : kBound * 2.f * cnmax + 1e-30f;
    const float delta_c = Sh::CLO ? 1.002f * __builtin_amdgcn_sqrtf(restmax) : 0.f;
    const float delta_ratio = 1.002f * 1.002f * ratio;

    for (;;) {   // until no pair is left; the list of undecided keys is worked off whenever it is nearly full
        // ---- centroid operands and norms ----
        ef_v8h a_r[Sh::AREG ? kEfTiles : 1];
        ef_v16f n_r[Sh::NREG ? Sh::NREG : 1];
        const ef_v4f *cn4 = reinterpret_cast<const ef_v4f *>(cn_s) + g;
        auto norms = [&](int t, ef_v16f &n) {   // rows 8q + 4g + (0..3) of the tile
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const ef_v4f c4 = cn4[8 * t + 2 * q];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    n[4 * q + e] = c4[e];
            }
        };
        if constexpr (Sh::AREG) {
#pragma unroll
            for (int t = 0; t < kEfTiles; ++t)
                a_r[t] = a_s[t * kWave + lane];
        }
#pragma unroll
        for (int t = 0; t < Sh::NREG; ++t)
            norms(t, n_r[t]);
        auto start = [&](int t, ef_v16f &n) {
            if (t < Sh::NREG)
                n = n_r[t < Sh::NREG ? t : 0];
            else
                norms(t, n);
        };

        int noted = 0;
        while (p < mine) {
            asm volatile("" ::: "memory");   // (operands and norms that are read from LDS are not kept in registers across pairs)
            float kpart[2], klow[2];    // this lane's share of |s_k k|^2, and of what the fp16 terms leave out, for its columns
            float dq[2][4], de[2][4], dt[2][kEfTiles];   // minima over the candidates that share a digit
            // ---- operand B: this lane's part of its keys ----
            ef_v8h kf[2][NS][NB];
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                float ks = Sh::SLOTS ? 0.f : (float)DP * 0x1p-28f, kl = 0.f;   // (room for flushed fp16 subnormals)
                if constexpr (!K32) {
                    _Float16 x[NL * 4];
                    if (!whole) {
#pragma unroll
                        for (int l = 0; l < NL; ++l)
                            ef_align_tail(raw[blk][l], piece(l), d_sub);
                    }
                    __builtin_memcpy(x, raw[blk], sizeof(x));
#pragma unroll
                    for (int l = 0; l < NL * 2; ++l) {
                        const ef_v2h w = {x[2 * l], x[2 * l + 1]};
                        ks = __builtin_amdgcn_fdot2(w, w, ks, false);
                    }
                    if constexpr (DP == 4) {
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            kf[blk][0][0][e] = g ? (e < 4 ? (_Float16)0.f : (e < 7 ? one : (_Float16)0.f)) : x[e % 4];
                    } else {
#pragma unroll
                        for (int s = 0; s < NS; ++s)
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                kf[blk][s][0][e] = x[8 * s + e];
                    }
                } else if constexpr (DP == 4) {
                    _Float16 xh[4], xl[4];
#pragma unroll
                    for (int l = 0; l < 2; ++l) {
                        const float u0 = sk * raw[blk][0][2 * l], u1 = sk * raw[blk][0][2 * l + 1];
                        ks = __builtin_fmaf(u0, u0, ks);
                        ks = __builtin_fmaf(u1, u1, ks);
                        const ef_v2fp hh = __builtin_amdgcn_cvt_pkrtz(u0, u1);
                        const ef_v2fp ll = __builtin_amdgcn_cvt_pkrtz(u0 - (float)hh[0], u1 - (float)hh[1]);
                        __builtin_memcpy(xh + 2 * l, &hh, 4);
                        __builtin_memcpy(xl + 2 * l, &ll, 4);
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        kf[blk][0][0][e] = g ? (e < 4 ? xl[e % 4] : (e < 7 ? one : (_Float16)0.f)) : xh[e % 4];
                } else {
#pragma unroll
                    for (int l = 0; l < NL * 2; ++l) {
                        float u0 = sk * raw[blk][l / 2][2 * (l % 2)], u1 = sk * raw[blk][l / 2][2 * (l % 2) + 1];
                        asm("" : "+v"(u0), "+v"(u1));   // (else the product is formed twice, once to round it)
                        const ef_v2h hh = {(_Float16)u0, (_Float16)u1};
                        if constexpr (FINE) {
                            ks = __builtin_fmaf(u0, u0, ks);
                            ks = __builtin_fmaf(u1, u1, ks);
                        } else {
                            ks = __builtin_amdgcn_fdot2(hh, hh, ks, false);
                        }
                        const float r0 = __builtin_fmaf((float)hh[0], minus_one, u0), r1 = __builtin_fmaf((float)hh[1], minus_one, u1);   // exact
                        kf[blk][l / 4][0][2 * (l % 4)] = hh[0];
                        kf[blk][l / 4][0][2 * (l % 4) + 1] = hh[1];
                        if constexpr (FINE) {
                            kf[blk][l / 4][NB - 1][2 * (l % 4)] = (_Float16)r0;
                            kf[blk][l / 4][NB - 1][2 * (l % 4) + 1] = (_Float16)r1;
                        } else {
                            kl = __builtin_fmaf(r0, r0, kl);
                            kl = __builtin_fmaf(r1, r1, kl);
                        }
                    }
                }
                kpart[blk] = ks;
                klow[blk] = kl;
            }
            here[0] = ahead[0];
            here[1] = ahead[1];
            int taken = 0;
            if (lane == 0)
                taken = atomicAdd(&next_s, 1);
            if (pn < mine)     // the next pair's keys arrive while this one is scored
                fetch_pair(pn);

            auto tile_min = [](const ef_v16f &x) {
                const float a = ef_min3(x[0], x[1], x[2]), b = ef_min3(x[3], x[4], x[5]), c = ef_min3(x[6], x[7], x[8]);
                const float d = ef_min3(x[9], x[10], x[11]), e = ef_min3(x[12], x[13], x[14]);
                return ef_min(ef_min3(a, b, c), ef_min3(d, e, x[15]));
            };
            auto digits = [](const float (&gm)[16], float (&q4)[4], float (&e4)[4]) {
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    q4[x] = ef_min(ef_min3(gm[4 * x], gm[4 * x + 1], gm[4 * x + 2]), gm[4 * x + 3]);
                    e4[x] = ef_min(ef_min3(gm[x], gm[4 + x], gm[8 + x]), gm[12 + x]);
                }
            };
            // Row tiles two at a time.  The scheduling barriers keep the accumulators of one step alive at a time.
            if constexpr (Sh::AREG) {   // first all tiles of block 0, then of block 1
                float gm[16];               // minima over the row tiles, by accumulator register (4 q + e)
#pragma unroll
                for (int u = 0; u < kEfTiles; ++u) {
                    const int blk = u / (kEfTiles / 2), t = 2 * (u % (kEfTiles / 2));
                    ef_v16f x0 = {}, x1 = {};
                    if constexpr (!Sh::SLOTS) {
                        start(t, x0);
                        start(t + 1, x1);
                    }
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        x0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a_r[t], kf[blk][0][b], x0, 0, 0, 0);
                        x1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a_r[t + 1], kf[blk][0][b], x1, 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    dt[blk][t] = tile_min(x0);
                    dt[blk][t + 1] = tile_min(x1);
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        gm[r] = (t == 0) ? ef_min(x0[r], x1[r]) : ef_min3(gm[r], x0[r], x1[r]);
                    if (t + 2 == kEfTiles)
                        digits(gm, dq[blk], de[blk]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {                    // both blocks share what is read of a tile
                float gm[2][16];
                ef_v8h a0[NS * NA], a1[NS * NA];
                auto operands = [&](int t) {
#pragma unroll
                    for (int s = 0; s < NS * NA; ++s) {
                        a0[s] = a_s[(t * NS * NA + s) * kWave + lane];
                        a1[s] = a_s[((t + 1) * NS * NA + s) * kWave + lane];
                    }
                };
                if constexpr (Sh::AHEAD)
                    operands(0);
#pragma unroll
                for (int t = 0; t < kEfTiles; t += 2) {
                    ef_v16f n0, n1;
                    if constexpr (!Sh::NTWICE) {
                        start(t, n0);
                        start(t + 1, n1);
                    }
                    if constexpr (!Sh::AHEAD)
                        operands(t);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int blk = 0; blk < 2; ++blk) {
                        if constexpr (Sh::NTWICE) {
                            start(t, n0);
                            start(t + 1, n1);
                        }
                        ef_v16f x0 = n0, x1 = n1;
#pragma unroll
                        for (int s = 0; s < NS; ++s)
#pragma unroll
                            for (int k = 0; k < NA + NB - 1; ++k) {   // hi.hi, lo.hi, hi.lo
                                const int a = NA * s + (k < NA ? k : 0), b = k < NA ? 0 : 1;
                                x0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0[a], kf[blk][s][b < NB ? b : 0], x0, 0, 0, 0);
                                x1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1[a], kf[blk][s][b < NB ? b : 0], x1, 0, 0, 0);
                            }
                        if (Sh::AHEAD && blk == 1 && t + 2 < kEfTiles)
                            operands(t + 2);      // (arrive behind this block's minima)
                        __builtin_amdgcn_sched_barrier(0);
                        dt[blk][t] = tile_min(x0);
                        dt[blk][t + 1] = tile_min(x1);
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            gm[blk][r] = (t == 0) ? ef_min(x0[r], x1[r]) : ef_min3(gm[blk][r], x0[r], x1[r]);
                        if (t + 2 == kEfTiles)
                            digits(gm[blk], dq[blk], de[blk]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            // ---- lane l now finishes key l % 32 of block l / 32: the two lane halves hold disjoint centroids ----
            auto halves = [](float x0, float x1, float &a, float &b) {   // (block 0, block 1) -> own block's halves 0 and 1
                const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
                a = __uint_as_float(r[0]);
                b = __uint_as_float(r[1]);
            };
            float mx[8], me[4], mt[kEfTiles];        // group minima by 2 q + h, e and t
#pragma unroll
            for (int x = 0; x < 4; ++x)
                halves(dq[0][x], dq[1][x], mx[2 * x], mx[2 * x + 1]);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                float a, b;
                halves(de[0][x], de[1][x], a, b);
                me[x] = ef_min(a, b);
            }
#pragma unroll
            for (int x = 0; x < kEfTiles; ++x) {
                float a, b;
                halves(dt[0][x], dt[1][x], a, b);
                mt[x] = ef_min(a, b);
            }
            float ka, kb2;
            halves(kpart[0], kpart[1], ka, kb2);
            const float kn = (DP >= 16) ? ka + kb2 : ka;           // up to 8 coordinates every lane holds the whole key
            const float best = ef_min(ef_min3(ef_min3(mx[0], mx[1], mx[2]), mx[3], mx[4]), ef_min3(mx[5], mx[6], mx[7]));
            float tau = __builtin_fmaf(t_k, kn, t_c);
            if constexpr (Sh::KLO || Sh::CLO) {
                float delta = delta_c;
                if constexpr (Sh::KLO) {
                    halves(klow[0], klow[1], ka, kb2);
                    delta += __builtin_amdgcn_sqrtf(delta_ratio * ((DP >= 16) ? ka + kb2 : ka));
                }
                // (the rounding of best and kn cannot make the square smaller than it is: tau is twice their bound)
                const float d = __builtin_amdgcn_sqrtf(fmaxf(__builtin_fmaf(ratio, kn, best) + tau, 0.f));
                tau = __builtin_fmaf(4.01f * delta, d + delta, tau);
            }
            const float limit = best + tau;
            // One bit per digit value, set where no candidate with that digit is within the limit.
            uint32_t out = 0;
            auto push = [&](float m) { out = __builtin_amdgcn_alignbit(out, __float_as_uint(limit - m), 31); };
#pragma unroll
            for (int x = kEfTiles - 1; x >= 0; --x)
                push(mt[x]);
#pragma unroll
            for (int x = 3; x >= 0; --x)
                push(me[x]);
#pragma unroll
            for (int x = 7; x >= 0; --x)
                push(mx[x]);
            // NaN or infinite on either side (fp32 keys whose lo terms count: beyond 2^31 the scaled key may not fit
            // fp16, 2^15.5 squared): everything is a candidate
            const bool sound = limit < INFINITY && limit > -INFINITY && (!(K32 && (DP == 4 || FINE)) || kn < 0x1p31f);
            const uint32_t among = sound ? out ^ kEfAll : kEfAll;
            const bool unique = __builtin_popcount(among) == 3;
            const int code = 32 * __builtin_ctz(among >> 12) + 4 * __builtin_ctz(among) + __builtin_ctz(among >> 8);

            const bool valid = col < (g ? here[1].live : here[0].live);
            uint8_t *const at0 = codes_at(here[0]), *const at1 = codes_at(here[1]);
            if (valid && unique)
                (g ? at1 : at0)[(uint32_t)(col * m)] = (uint8_t)code;
            const int done = p;
            p = pn;
            pn = __builtin_amdgcn_readfirstlane(taken);
            // keys the filter could not decide are noted with their candidates, and left for later
            const uint64_t todo = __ballot(valid && !unique);
            if (todo) {
                if (valid && !unique)
                    list_s[wave][noted + (int)__popcll(todo & ((1ull << lane) - 1ull))] = make_uint2((uint32_t)done << 6 | lane, among);
                noted += (int)__popcll(todo);
                if (noted > kEfList - kWave)
                    break;
            }
        }
        if (lane == 0)
            count_s[wave] = noted | (p < mine ? kEfMore : 0);
        __syncthreads();
        // ---- the exact rule for the noted keys: eight lanes share a key's candidates ----
        int until[kEfWaves];      // entries of the lists up to and with the w-th
        int more = 0, count;
        auto lengths = [&] {
#pragma unroll
            for (int w = 0; w < kEfWaves; ++w) {
                more |= count_s[w] & kEfMore;
                until[w] = (w ? until[w - 1] : 0) + (count_s[w] & (kEfMore - 1));
            }
            count = until[kEfWaves - 1];
        };
        auto noted_at = [&](int at) {      // the at-th entry of all lists
            int list = 0, start = 0;
#pragma unroll
            for (int w = 0; w < kEfWaves - 1; ++w)
                if (at >= until[w]) {
                    list = w + 1;
                    start = until[w];
                }
            return list_s[list][at - start];
        };
        auto place = [&](const uint2 &entry) { return locate(2u * ((uint32_t)first + (entry.x >> 6)) + ((entry.x & 63u) >> 5)); };
        auto key_of = [&](const uint2 &entry) { return keys_at(place(entry)) + (entry.x & 31u) * (uint32_t)d_k; };
        auto code_of = [&](const uint2 &entry) { return codes_at(place(entry)) + (entry.x & 31u) * (uint32_t)m; };
        lengths();
        // A long list may hold one key many times over (zeros that fill up a batch of prompts, say, where a centroid near them has a rival).
        // If one of four entries is met 16 times or more among 64 that are spread over the lists, that key is decided once, and every
        // entry that holds its bits takes its code and leaves the lists; then the next such key.  (One wavefront looks, so that all do the
        // same.  Up to eight rounds of the exact rule are not worth the look.)
        for (int passes = 0; count > kEfWaves * 64 && passes < 8; ++passes) {
            if (wave == 0) {
                auto spread = [&](int k) { return (int)((uint32_t)k * (uint32_t)count / 64u); };
                const uint2 own = noted_at(spread(lane));
                int most = 15, which = -1;
#pragma unroll 1
                for (int k = 13; k < kWave; k += 16) {      // (equal keys have equal candidates)
                    const int equal = (int)__popcll(__ballot(own.y == noted_at(spread(k)).y));
                    which = equal > most ? spread(k) : which;
                    most = equal > most ? equal : most;
                }
                if (which >= 0) {
                    const KT *one = key_of(noted_at(which)), *some[1] = {key_of(own)};
                    bool same[1];
                    ef_same_key<DP, FULL>(one, some, d_sub, same);
                    which = __popcll(__ballot(same[0])) >= 16 ? which << 8 | ef_exact_code<KT>(one, cb, d_sub, lane) : -1;
                }
                if (lane == 0)
                    repeated_s = which;
            }
            __syncthreads();
            const int found = repeated_s;      // (entry, code)
            if (found < 0)
                break;
            const KT *one = key_of(noted_at(found >> 8));
            __syncthreads();                   // (the lists are read)
            int kept = 0;
            noted = count_s[wave] & (kEfMore - 1);
            for (int k0 = 0; k0 < noted; k0 += 2 * kWave) {
                uint2 e[2];
                const KT *x[2];
                bool same[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int k = k0 + u * kWave + lane;
                    e[u] = list_s[wave][k < noted ? k : noted - 1];
                    x[u] = key_of(e[u]);
                }
                ef_same_key<DP, FULL>(one, x, d_sub, same);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const bool there = k0 + u * kWave + lane < noted;
                    if (there && same[u])
                        *code_of(e[u]) = (uint8_t)found;
                    const uint64_t others = __ballot(there && !same[u]);
                    if (there && !same[u])
                        list_s[wave][kept + (int)__popcll(others & ((1ull << lane) - 1ull))] = e[u];
                    kept += (int)__popcll(others);
                }
            }
            if (lane == 0)
                count_s[wave] = kept;
            __syncthreads();
            lengths();
        }
        for (int b0 = wave * 8; b0 < count; b0 += kEfWaves * 8) {
            const bool exists = b0 + lane / 8 < count;
            const uint2 entry = noted_at(exists ? b0 + lane / 8 : count - 1);
            const KT *key_sub = key_of(entry);
            uint8_t *dst = code_of(entry);
            const uint32_t mx = entry.y & 255u, me = entry.y >> 8 & 15u, mt = entry.y >> 12;
            const int nx = __builtin_popcount(mx), ne = __builtin_popcount(me), nt = __builtin_popcount(mt);
            const int all = nx * ne * nt;
            auto evaluate = [&](int c) { return argmin_value(ef_exact_distance<KT, DP, FULL>(key_sub, cb + c * d_sub, d_sub), c); };
            // the lowest or the highest value of each digit, by the lane's bits: all combinations where there are no others
            int code = 32 * (lane & 4 ? 31 - __builtin_clz(mt) : __builtin_ctz(mt)) +
                       4 * (lane & 1 ? 31 - __builtin_clz(mx) : __builtin_ctz(mx)) +
                       (lane & 2 ? 31 - __builtin_clz(me) : __builtin_ctz(me));
            double best = evaluate(code);
            const int upto = all <= kEfShared && (nx > 2 || ne > 2 || nt > 2) ? all : 0;
            for (int k = lane % 8; __ballot(k < upto); k += 8)
                if (k < upto) {   // the k-th combination (quotients below 256: floor is exact)
                    const int r1 = (int)(((float)k + 0.5f) * __builtin_amdgcn_rcpf((float)nx));
                    const int r2 = (int)(((float)r1 + 0.5f) * __builtin_amdgcn_rcpf((float)ne));
                    const int c = 32 * ef_nth_bit(mt, r2) + 4 * ef_nth_bit(mx, k - r1 * nx) + ef_nth_bit(me, r1 - r2 * ne);
                    const double d = evaluate(c);
                    if (d < best || (d == best && c < code)) {
                        best = d;
                        code = c;
                    }
                }
            ef_argmin_step<0xB1>(best, code);     // lane ^ 1, lane ^ 2, the other quad of each eight
            ef_argmin_step<0x4E>(best, code);
            ef_argmin_step<0x141>(best, code);
            const bool writes = lane % 8 == 0 && exists;
            if (writes && all <= kEfShared)
                *dst = (uint8_t)code;
            // many candidates: the wavefront takes such a key together, all centroids
            uint64_t whole = __ballot(writes && all > kEfShared);
            while (whole) {
                const int turn = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(whole));
                whole &= whole - 1;
                const uint64_t src = (uint64_t)(uintptr_t)key_sub;
                const KT *one = reinterpret_cast<const KT *>((uintptr_t)(
                    (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(src >> 32), turn) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)src, turn)));
                const float *rows = cb;
                if constexpr (DP > 16)
                    asm volatile("" : "+s"(rows));   // (rows kept in registers from one key to the next would spill)
                const int exact = ef_exact_code<KT>(one, rows, d_sub, lane);
                if (lane == turn)
                    *dst = (uint8_t)exact;
            }
        }
        if (!more)
            break;
        __syncthreads();     // (the lists are read)
        if (p < mine)        // (the keys of the pair at hand were on their way when the list filled up)
            fetch_pair(p);
    }
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
    const int64_t pairs = (total_blocks + 1) / 2;
    const EfGrid chosen = ef_grid(s->H, s->m, pairs, ef_operand(d_sub), sizeof(KT) == 4);
    const int64_t splits = chosen.splits;
    const int64_t wgs = ((int64_t)s->H * splits + 7) / 8 * 8 * s->m;
    if (wgs > 0xffffff)   // (a grid of 2^32 threads)
        return false;
    const dim3 grid((unsigned)wgs), block((unsigned)chosen.threads);
    const KT *k = static_cast<const KT *>(keys);
#define LOOKAT_EF_LAUNCH(D, FULL, THREADS, FINE)                                                                          \
    hipLaunchKernelGGL((encode_filter_kernel<KT, D, FULL, THREADS, FINE>), grid, block, 0, st, k, codebooks, codes,       \
                       code_stride_bh, s->B, s->H, N, s->d_k, s->m, d_sub, (uint32_t)blocks_per_bh,                           \
                       (uint32_t)(0xffffffffu / (uint32_t)blocks_per_bh), (int)splits,                                    \
                       (int)((pairs + splits - 1) / splits))
#define LOOKAT_EF_FORM(D, FULL)                                                                                           \
    do {                                                                                                                  \
        constexpr int kLarge = ef_has_large(D) ? 512 : 256;                                                               \
        constexpr bool kFine = ef_has_fine(D, sizeof(KT) == 4);                                                           \
        if (chosen.threads == 512)                                                                                        \
            LOOKAT_EF_LAUNCH(D, FULL, kLarge, false);                                                                     \
        else if (chosen.fine)                                                                                             \
            LOOKAT_EF_LAUNCH(D, FULL, 256, kFine);                                                                        \
        else                                                                                                              \
            LOOKAT_EF_LAUNCH(D, FULL, 256, false);                                                                        \
        return true;                                                                                                      \
    } while (0)
#define LOOKAT_EF_CASE(D)                                                                                                 \
    if (d_sub == D)                                                                                                       \
        LOOKAT_EF_FORM(D, true);                                                                                          \
    if (d_sub < D)                                                                                                        \
        LOOKAT_EF_FORM(D, false);
    LOOKAT_EF_CASE(4)
    LOOKAT_EF_CASE(8)
    LOOKAT_EF_CASE(16)
    LOOKAT_EF_CASE(32)
    LOOKAT_EF_CASE(64)
#undef LOOKAT_EF_CASE
#undef LOOKAT_EF_FORM
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
