// Key encoding (paper Sec. 3.4, "Encoding"): per key and subspace, the index of the
// nearest centroid.  The distance is evaluated in fp64 with one rounding per subtract,
// multiply and add, coordinates ascending, and a strict '<' scan over ascending
// centroid index, so the code is unique and identical on every IEEE machine.
//
// This translation unit must be compiled with -ffp-contract=off: a fused multiply-add
// in the distance would change near-tie decisions.
#include <cstdlib>

#include "common.h"

#pragma clang fp contract(off)

namespace lookat {

constexpr int kEncThreads = 256;
constexpr int kEncLdsDoubles = 4096;  // centroid chunk staged in LDS: 32 KB of fp64

template <typename T>
__device__ __forceinline__ double widen(T v);
template <>
__device__ __forceinline__ double widen<float>(float v) { return (double)v; }
template <>
__device__ __forceinline__ double widen<__half>(__half v) { return (double)__half2float(v); }

// One block = 256 keys of one head, one subspace.  The key sub-vector lives in
// registers as fp64; the centroids of the subspace are staged in LDS as fp64 and read
// by all lanes at the same address (LDS broadcast, conflict free).
//   grid = (ceil(B*N / 256), m, H)
template <typename KT, int DSUB>
__global__ __launch_bounds__(kEncThreads) void encode_kernel(const KT *__restrict__ keys,
                                                             const float *__restrict__ codebooks,
                                                             uint8_t *__restrict__ codes, int64_t code_stride_bh,
                                                             int B, int H, int64_t N, int d_k, int m)
{
    __shared__ double cb_s[kEncLdsDoubles];
    constexpr int KC = (kEncLdsDoubles / DSUB) < kCentroids ? (kEncLdsDoubles / DSUB) : kCentroids;

    const int i = blockIdx.y;
    const int h = blockIdx.z;
    const int64_t r = (int64_t)blockIdx.x * kEncThreads + threadIdx.x;  // flat (b, n)
    const bool live = r < (int64_t)B * N;
    const int64_t b = live ? r / N : 0;
    const int64_t n = live ? r % N : 0;
    const int64_t bh = b * H + h;

    double x[DSUB];
    {
        const KT *src = keys + (bh * N + n) * d_k + (int64_t)i * DSUB;
#pragma unroll
        for (int j = 0; j < DSUB; ++j)
            x[j] = live ? widen<KT>(src[j]) : 0.0;
    }

    const float *cb = codebooks + ((int64_t)h * m + i) * kCentroids * DSUB;
    double best = 0.0;
    int best_c = 0;
    for (int c0 = 0; c0 < kCentroids; c0 += KC) {
        __syncthreads();
        for (int e = threadIdx.x; e < KC * DSUB; e += kEncThreads)
            cb_s[e] = (double)cb[(int64_t)c0 * DSUB + e];
        __syncthreads();
        for (int c = 0; c < KC; ++c) {
            const double *y = cb_s + c * DSUB;
            double acc = 0.0;
#pragma unroll
            for (int j = 0; j < DSUB; ++j) {
                double diff = x[j] - y[j];
                double sq = diff * diff;
                acc = acc + sq;
            }
            // first centroid initialises the scan; afterwards strict '<' keeps the lowest index
            if ((c0 + c) == 0 || acc < best) {
                best = acc;
                best_c = c0 + c;
            }
        }
    }
    if (live)
        codes[bh * code_stride_bh + n * m + i] = (uint8_t)best_c;
}

// ---- few keys per head (decode-time append) -------------------------------------------
// With a handful of keys per head the thread-per-key kernel above leaves the chip empty and
// each thread walks all 256 centroids serially.  Here the centroids are spread over the
// threads instead: one block = one (head, subspace) and KEYS keys (1, 2, 4 or 8: see few_keys);
// thread c holds centroid c in registers, evaluates its distance to every key of the block
// (same arithmetic, same order) and the block takes the argmin over (distance, index).
// What bounds it: latency -- the codebook's and the keys' way from memory, then KEYS serial chains of fp64 operations and as many
// reductions over the wavefront.  So the centroid's row is requested in 16-byte pieces, sixteen coordinates at once, beside the keys (element
// by element, four in flight, the row of a 12-coordinate sub-vector took three round trips), and no key is evaluated that is not there.
// us per call before / now: 4 x 16 (b,h), d_k = 96, m = 8 4.9 / 3.0; 2 x 8, d_k = 128, m = 2, fp32 12.5 / 5.4; 1 x 8, d_k = 160, m = 16 4.7 / 3.7.
constexpr int kEncFewKeys = 8;

// Flat (b, n) of a head's keys.  (A decode step appends one key per sequence: no division on the way to its address; else a 32-bit
// one where that does.)
__device__ __forceinline__ void split_row(int64_t r, int64_t N, int64_t &b, int64_t &n)
{
    b = r;
    n = 0;
    if (N > 0xffffffffLL || r > 0xffffffffLL) {
        b = r / N;
        n = r % N;
    } else if (N != 1) {
        b = (uint32_t)r / (uint32_t)N;
        n = r - b * N;
    }
}

// Per key the minimum over the wavefront's 64 centroids (cross-lane moves on the vector ALU, the keys' chains
// interleaved), the lowest lane that holds it (the serial scan's choice among exact ties), and the same over the
// block's wavefronts.
template <int KEYS>
__device__ __forceinline__ void encode_few_finish(const double (&dv)[KEYS], double (&dm)[KEYS],
                                                  double (&red_d)[KEYS][kCentroids / kWave],
                                                  int (&red_c)[KEYS][kCentroids / kWave], uint8_t *codes,
                                                  int64_t code_stride_bh, int B, int H, int64_t N, int m, int i, int h,
                                                  int64_t r0, int lane, int wave)
{
    dmin_wave<KEYS>(dm);
#pragma unroll
    for (int k = 0; k < KEYS; ++k) {
        const uint64_t holders = __ballot(dv[k] == dm[k]);
        if (lane == 0) {
            red_d[k][wave] = dm[k];
            red_c[k][wave] = wave * kWave + (int)__builtin_ctzll(holders);
        }
    }
    __syncthreads();
    if (threadIdx.x < KEYS) {
        const int k = threadIdx.x;
        const int64_t r = r0 + k;
        if (r < (int64_t)B * N) {
            // wavefronts hold ascending centroid ranges: strict '<' keeps the lowest index on ties
            double bd = red_d[k][0];
            int best = red_c[k][0];
#pragma unroll
            for (int w = 1; w < kCentroids / kWave; ++w) {
                const double d = red_d[k][w];
                const int cw = red_c[k][w];
                const bool better = d < bd;
                bd = better ? d : bd;
                best = better ? cw : best;
            }
            int64_t b, n;
            split_row(r, N, b, n);
            codes[(b * H + h) * code_stride_bh + n * m + i] = (uint8_t)best;
        }
    }
}

template <typename KT, int DSUB, int KEYS>
__global__ __launch_bounds__(kCentroids) void encode_few_kernel(const KT *__restrict__ keys,
                                                                const float *__restrict__ codebooks,
                                                                uint8_t *__restrict__ codes, int64_t code_stride_bh,
                                                                int B, int H, int64_t N, int d_k, int m)
{
    __shared__ double x_s[KEYS][DSUB];
    __shared__ double red_d[KEYS][kCentroids / kWave];
    __shared__ int red_c[KEYS][kCentroids / kWave];

    const int i = blockIdx.y;
    const int h = blockIdx.z;
    const int c = threadIdx.x;
    const int lane = c & (kWave - 1), wave = c / kWave;
    const int64_t r0 = (int64_t)blockIdx.x * KEYS;   // first flat (b, n) of the block
    const int64_t rows = (int64_t)B * N;

    // (the row is requested ahead of the keys: their addresses take a division, and staging them waits for them)
    float row[DSUB];
    {
        const float *src = codebooks + (((int64_t)h * m + i) * kCentroids + c) * DSUB;
#pragma unroll
        for (int j = 0; j < DSUB; ++j)
            row[j] = src[j];
    }
    for (int e = threadIdx.x; e < KEYS * DSUB; e += kCentroids) {
        const int64_t r = r0 + e / DSUB;
        double v = 0.0;
        if (r < rows) {
            int64_t b, n;
            split_row(r, N, b, n);
            v = widen<KT>(keys[((b * H + h) * N + n) * d_k + (int64_t)i * DSUB + e % DSUB]);
        }
        x_s[e / DSUB][e % DSUB] = v;
    }
    double y[DSUB];
#pragma unroll
    for (int j = 0; j < DSUB; ++j)
        y[j] = (double)row[j];
    __syncthreads();

    // Distances of centroid c to the block's keys.
    double dv[KEYS], dm[KEYS];
#pragma unroll
    for (int k = 0; k < KEYS; ++k) {
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < DSUB; ++j) {
            double diff = x_s[k][j] - y[j];
            double sq = diff * diff;
            acc = acc + sq;
        }
        dv[k] = argmin_value(acc, c);
        dm[k] = dv[k];
    }
    encode_few_finish<KEYS>(dv, dm, red_d, red_c, codes, code_stride_bh, B, H, N, m, i, h, r0, lane, wave);
}

// Any sub-vector length: the same.  A row of 16-byte pieces (from a 16-byte aligned codebook) is taken JB coordinates at a time, the next
// ones requested before the last are used; JB = 0: its elements are read as they are needed (5, 7, 10, 14 ..: 16 single elements
// ahead measured 5 to 15% slower).  The keys' sub-vectors sit in dynamic LDS.  With many workgroups registers count (one kernel for all took
// 100): 40 heads x 34 keys, 16 subspaces of 5, 15.1 / 13.2 us, 8 of 12 11.7 / 11.1; rows of 128 want sixteen ahead (16 heads x 2000 keys,
// 2 of 128, eight ahead / sixteen 248 / 237).
template <typename KT, int KEYS, int JB>
__global__ __launch_bounds__(kCentroids, (KEYS == 8 && JB == 0 ? 8 : 4)) void encode_few_any_kernel(const KT *__restrict__ keys,
                                                                    const float *__restrict__ codebooks,
                                                                    uint8_t *__restrict__ codes, int64_t code_stride_bh,
                                                                    int B, int H, int64_t N, int d_k, int m)
{
    constexpr bool PIECES = JB > 0;
    extern __shared__ __align__(16) double xs[];   // [d_sub][KEYS]
    __shared__ double red_d[KEYS][kCentroids / kWave];
    __shared__ int red_c[KEYS][kCentroids / kWave];
    const int d_sub = d_k / m;
    const int i = blockIdx.y;
    const int h = blockIdx.z;
    const int c = threadIdx.x;
    const int lane = c & (kWave - 1), wave = c / kWave;
    const int64_t rows = (int64_t)B * N;
    const float *src = codebooks + (((int64_t)h * m + i) * kCentroids + c) * d_sub;
    auto fetch = [&](int j0, float (&y)[PIECES ? JB : 1]) {      // coordinates j0 .. j0 + JB - 1 as far as there are any
#pragma unroll
        for (int q = 0; q < JB; q += 4)
            if (j0 + q < d_sub) {
                const float4 v = *reinterpret_cast<const float4 *>(src + j0 + q);
                y[q] = v.x;
                y[q + 1] = v.y;
                y[q + 2] = v.z;
                y[q + 3] = v.w;
            }
    };
    for (int64_t r0 = (int64_t)blockIdx.x * KEYS; r0 < rows; r0 += (int64_t)gridDim.x * KEYS) {
        [[maybe_unused]] float y[PIECES ? JB : 1], ahead[PIECES ? JB : 1];
        if constexpr (PIECES)
            fetch(0, y);
        {                                           // 256 / KEYS threads per key
            constexpr int kPer = kCentroids / KEYS;
            const int k = c / kPer;
            const int64_t r = r0 + k;
            int64_t b = 0, n = 0;
            if (r < rows)
                split_row(r, N, b, n);
            for (int j = c % kPer; j < d_sub; j += kPer)
                xs[j * KEYS + k] = r < rows ? widen<KT>(keys[((b * H + h) * N + n) * d_k + (int64_t)i * d_sub + j]) : 0.0;
        }
        __syncthreads();
        double dv[KEYS], dm[KEYS];
#pragma unroll
        for (int k = 0; k < KEYS; ++k)
            dv[k] = 0.0;
        auto add = [&](int j, double yd) {
#pragma unroll
            for (int k = 0; k < KEYS; ++k) {
                double diff = xs[j * KEYS + k] - yd;
                double sq = diff * diff;
                dv[k] = dv[k] + sq;
            }
        };
        if constexpr (PIECES) {
            for (int j0 = 0; j0 < d_sub; j0 += JB) {
                if (j0 + JB < d_sub)
                    fetch(j0 + JB, ahead);
#pragma unroll
                for (int q = 0; q < JB; q += 4)
                    if (j0 + q < d_sub) {
#pragma unroll
                        for (int e = q; e < q + 4; ++e)
                            add(j0 + e, (double)y[e]);
                    }
#pragma unroll
                for (int q = 0; q < JB; ++q)
                    y[q] = ahead[q];
            }
        } else {
#pragma unroll 4
            for (int j = 0; j < d_sub; ++j)
                add(j, (double)src[j]);
        }
#pragma unroll
        for (int k = 0; k < KEYS; ++k) {
            dv[k] = argmin_value(dv[k], c);
            dm[k] = dv[k];
        }
        encode_few_finish<KEYS>(dv, dm, red_d, red_c, codes, code_stride_bh, B, H, N, m, i, h, r0, lane, wave);
        __syncthreads();   // the next keys overwrite the staged ones
    }
}

// Keys of a workgroup: as few as leave two workgroups on a compute unit, one where rows are longer than 16 coordinates.  Up to there all run at
// once, and a workgroup's time is its chain, which the further keys make longer: their fp64 distances and minima take the vector ALU in turn.
// With more workgroups the rows' fetch counts, which the keys share.  us per call, 1 / 2 / 4 / 8 keys, subspaces x heads x keys a head: 8
// coordinates, 48 x 12 2.4 / 2.7 / 2.9 / 3.6, 256 x 8 4.5 / 3.2 / 3.2 / 3.8; 12, 128 x 4 3.0 / 3.0 / 3.6, 128 x 8 4.3 / 3.4 / 3.5 / 4.7; 16, 256 x 2
// 2.8 / 2.8, 256 x 4 4.7 / 3.3 / 3.3, 128 x 16 5.0 / 5.5 / 4.1 / 4.5; 20, 16 x 16 3.0 / 3.2 / 3.9 / 5.3, 128 x 4 4.4 / 3.3 / 4.1; 32, 16 x 16
// 3.2 / 3.5 / 4.5 / 6.5, 16 x 24 4.0 / 3.6 / 4.6 / 6.6, 128 x 8 8.0 / 6.2 / 4.8 / 6.7, 256 x 60 54 / 31 / 23 / 22.
static int few_keys(const lookat_shape *s, int64_t rows)
{
    const int64_t most = s->d_k / s->m <= 16 ? 512 : 256;
    int keys = 1;
    while (keys < kEncFewKeys && keys < rows && (rows + keys - 1) / keys * s->m * s->H > most)
        keys *= 2;
    return keys;
}

// (also the exact scan of sub-vector lengths without an encode_kernel instance, however many keys)
template <typename KT>
static void launch_encode_few_any(const lookat_shape *s, int64_t N, const void *keys, const float *codebooks,
                                  uint8_t *codes, int64_t code_stride_bh, hipStream_t st)
{
    const int64_t rows = (int64_t)s->B * N;
    const int keys_wg = few_keys(s, rows);
    const int64_t blocks = (rows + keys_wg - 1) / keys_wg;
    const dim3 grid((unsigned)(blocks < 65536 ? blocks : 65536), (unsigned)s->m, (unsigned)s->H);
    const int d_sub = s->d_k / s->m;
#define LOOKAT_ENCA_FORM(KEYS, JB)                                                                                        \
    hipLaunchKernelGGL((encode_few_any_kernel<KT, KEYS, JB>), grid, dim3(kCentroids), (size_t)KEYS * d_sub * sizeof(double), \
                       st, static_cast<const KT *>(keys), codebooks, codes, code_stride_bh, s->B, s->H, N, s->d_k, s->m)
#define LOOKAT_ENCA_LAUNCH(KEYS)                                                                                          \
    do {                                                                                                                  \
        if (d_sub % 4)                                                                                                    \
            LOOKAT_ENCA_FORM(KEYS, 0);                                                                                    \
        else if (d_sub <= 24)                                                                                             \
            LOOKAT_ENCA_FORM(KEYS, (KEYS == 8 ? 8 : 16));                                                                 \
        else                                                                                                              \
            LOOKAT_ENCA_FORM(KEYS, 16);                                                                                   \
    } while (0)
    if (keys_wg == 1)
        LOOKAT_ENCA_LAUNCH(1);
    else if (keys_wg == 2)
        LOOKAT_ENCA_LAUNCH(2);
    else if (keys_wg == 4)
        LOOKAT_ENCA_LAUNCH(4);
    else
        LOOKAT_ENCA_LAUNCH(8);
#undef LOOKAT_ENCA_FORM
#undef LOOKAT_ENCA_LAUNCH
}

template <typename KT>
static bool launch_encode_few(const lookat_shape *s, int64_t N, const void *keys, const float *codebooks,
                              uint8_t *codes, int64_t code_stride_bh, hipStream_t st)
{
    const int d_sub = s->d_k / s->m;
    const int64_t rows = (int64_t)s->B * N;
    const int keys_wg = few_keys(s, rows);
    dim3 grid((unsigned)((rows + keys_wg - 1) / keys_wg), (unsigned)s->m, (unsigned)s->H);
    dim3 block(kCentroids);
    const KT *k = static_cast<const KT *>(keys);
#define LOOKAT_ENCF_LAUNCH(D, KEYS)                                                                             \
    hipLaunchKernelGGL((encode_few_kernel<KT, D, KEYS>), grid, block, 0, st, k, codebooks, codes,               \
                       code_stride_bh, s->B, s->H, N, s->d_k, s->m)
#define LOOKAT_ENCF_CASE(D)                                                                                     \
    case D:                                                                                                     \
        if (keys_wg == 1)                                                                                       \
            LOOKAT_ENCF_LAUNCH(D, 1);                                                                           \
        else if (keys_wg == 2)                                                                                  \
            LOOKAT_ENCF_LAUNCH(D, 2);                                                                           \
        else if (keys_wg == 4)                                                                                  \
            LOOKAT_ENCF_LAUNCH(D, 4);                                                                           \
        else                                                                                                    \
            LOOKAT_ENCF_LAUNCH(D, 8);                                                                           \
        return true;
    switch (d_sub) {
        LOOKAT_ENCF_CASE(1)
        LOOKAT_ENCF_CASE(2)
        LOOKAT_ENCF_CASE(4)
        LOOKAT_ENCF_CASE(8)
        LOOKAT_ENCF_CASE(16)
        LOOKAT_ENCF_CASE(32)
    default:
        launch_encode_few_any<KT>(s, N, keys, codebooks, codes, code_stride_bh, st);
        return true;
    }
#undef LOOKAT_ENCF_CASE
#undef LOOKAT_ENCF_LAUNCH
}

template <typename KT>
static void launch_encode(const lookat_shape *s, int64_t N, const void *keys, const float *codebooks, uint8_t *codes,
                          int64_t code_stride_bh, hipStream_t st)
{
    const int d_sub = s->d_k / s->m;
    const int64_t rows = (int64_t)s->B * N;
    dim3 grid((unsigned)((rows + kEncThreads - 1) / kEncThreads), (unsigned)s->m, (unsigned)s->H);
    dim3 block(kEncThreads);
    const KT *k = static_cast<const KT *>(keys);
#define LOOKAT_ENC_CASE(D)                                                                                      \
    case D:                                                                                                     \
        hipLaunchKernelGGL((encode_kernel<KT, D>), grid, block, 0, st, k, codebooks, codes, code_stride_bh,     \
                           s->B, s->H, N, s->d_k, s->m);                                                        \
        break;
    switch (d_sub) {
        LOOKAT_ENC_CASE(1)
        LOOKAT_ENC_CASE(2)
        LOOKAT_ENC_CASE(4)
        LOOKAT_ENC_CASE(8)
        LOOKAT_ENC_CASE(16)
        LOOKAT_ENC_CASE(32)
        LOOKAT_ENC_CASE(64)
    default:
        launch_encode_few_any<KT>(s, N, keys, codebooks, codes, code_stride_bh, st);
        break;
    }
#undef LOOKAT_ENC_CASE
}

// encode_filter.hip: matrix-core filter in front of the exact rule (d_sub 2 to 64)
bool launch_encode_filter(const lookat_shape *s, int64_t N, const void *keys, int key_dtype, const float *codebooks,
                          uint8_t *codes, int64_t code_stride_bh, hipStream_t st);

}  // namespace lookat

extern "C" int lookat_encode_keys(const lookat_shape *shape, int64_t N, const void *keys, lookat_dtype key_dtype,
                                  const float *codebooks, uint8_t *codes, int64_t code_stride_bh, void *stream)
{
    using namespace lookat;
    clear_error();
    if (int rc = check_shape(shape))
        return rc;
    if (N < 0)
        return fail(LOOKAT_ERR_SHAPE, "N=%lld is negative", (long long)N);
    if (key_dtype != LOOKAT_F16 && key_dtype != LOOKAT_F32)
        return fail(LOOKAT_ERR_DTYPE, "key_dtype=%d is neither LOOKAT_F16 nor LOOKAT_F32", key_dtype);
    if (N == 0)
        return LOOKAT_OK;
    if (!keys || !codebooks || !codes)
        return fail(LOOKAT_ERR_NULL, "keys, codebooks and codes must be non-NULL");
    if (code_stride_bh < N * shape->m)
        return fail(LOOKAT_ERR_SHAPE, "code_stride_bh=%lld is smaller than N*m=%lld", (long long)code_stride_bh,
                    (long long)(N * shape->m));
    if (!aligned16(keys) || !aligned16(codebooks))
        return fail(LOOKAT_ERR_ALIGN, "keys and codebooks must be 16-byte aligned");
    const int64_t rows = (int64_t)shape->B * N;
    if ((rows + kEncThreads - 1) / kEncThreads > 0x7fffffffLL || shape->H > 65535 || shape->m > 65535)
        return fail(LOOKAT_ERR_UNSUPPORTED, "B*N=%lld keys per head exceed one launch", (long long)rows);
    hipStream_t st = static_cast<hipStream_t>(stream);
    // Few keys per head (a decode step appends one per sequence): spread the centroids over
    // the threads.  Many keys (prefill): one thread per key.  The crossover is where the
    // thread-per-key grid reaches a few workgroups per compute unit.
    const int64_t per_key_blocks = (rows + kEncThreads - 1) / kEncThreads * shape->m * shape->H;
    bool done = false;
    // From a few 32-key blocks per head upwards the filter kernel is the fast path; the environment
    // variable LOOKAT_ENCODE_EXACT=1 forces the plain exact kernels (same codes, for comparison runs).
    const char *exact_env = getenv("LOOKAT_ENCODE_EXACT");
    const bool exact_only = exact_env && exact_env[0] == '1';
    if (!exact_only && rows >= 64)
        done = launch_encode_filter(shape, N, keys, key_dtype, codebooks, codes, code_stride_bh, st);
    if (!done && per_key_blocks < 1024 && (rows + kEncFewKeys - 1) / kEncFewKeys <= 0x7fffffffLL) {
        done = (key_dtype == LOOKAT_F16)
                   ? launch_encode_few<__half>(shape, N, keys, codebooks, codes, code_stride_bh, st)
                   : launch_encode_few<float>(shape, N, keys, codebooks, codes, code_stride_bh, st);
    }
    if (!done) {
        if (key_dtype == LOOKAT_F16)
            launch_encode<__half>(shape, N, keys, codebooks, codes, code_stride_bh, st);
        else
            launch_encode<float>(shape, N, keys, codebooks, codes, code_stride_bh, st);
    }
    return check_launch("lookat_encode_keys");
}
