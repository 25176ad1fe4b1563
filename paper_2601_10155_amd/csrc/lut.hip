// Lookup-table construction (paper Sec. 3.5, "Precomputation Lookup Tables";
// Algorithm 1, first loop): lut[b,h,t,i,c] = q[b,h,t]^(i) . C_{h,i}[c], fp32 accumulate.
#include "common.h"

namespace lookat {

constexpr int kLutThreads = kCentroids;  // one thread per centroid

template <typename QT>
__device__ __forceinline__ float to_f32(QT v);
template <>
__device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float to_f32<__half>(__half v) { return __half2float(v); }

// (b, t) of a head's query in flattened order (B*T < 2^31).  A decode step has one query per sequence: no division on the way to
// its address.
__device__ __forceinline__ void split_query(int64_t qi, int T, int64_t &b, int64_t &t)
{
    b = qi;
    t = 0;
    if (T != 1) {
        b = (uint32_t)qi / (uint32_t)T;
        t = qi - b * T;
    }
}

// (subspace, head, part of the queries) of a workgroup, grid = (parts, m, H) or (m, H, parts).
struct RowBlock {
    int i, h;
    uint32_t part;
};
__device__ __forceinline__ RowBlock row_block(bool rows_together)
{
    if (rows_together)
        return {(int)blockIdx.x, (int)blockIdx.y, blockIdx.z};
    return {(int)blockIdx.y, (int)blockIdx.z, blockIdx.x};
}
static dim3 row_grid(const lookat_shape *s, int64_t parts, bool rows_together)
{
    return rows_together ? dim3((unsigned)s->m, (unsigned)s->H, (unsigned)parts) : dim3((unsigned)parts, (unsigned)s->m, (unsigned)s->H);
}

// One block = one head h, one subspace i, QB consecutive queries of the flattened
// (b, t) list.  Thread c keeps centroid c of the subspace in registers and reuses it for
// every query of the block; the query sub-vectors sit in LDS and are read by all lanes
// at the same address (broadcast).  Each query's 256 table entries are written as one
// contiguous 1 KB row.  Rows of 32 and 64 coordinates are requested first, as staging the queries waits for them (4 tables of 32 coordinates
// 2.8 / 2.7 us, 1024 of 64 10.6 / 9.1); shorter ones behind the queries (first: 30720 tables of 8 coordinates 10.8 / 13.8 us).
//   grid = (ceil(B*T / QB), m, H), or (m, H, ceil(B*T / QB)): see lut_rows_together
template <typename QT, int DSUB>
__global__ __launch_bounds__(kLutThreads) void build_lut_kernel(const QT *__restrict__ q,
                                                                const float *__restrict__ codebooks,
                                                                float *__restrict__ lut, int B, int H, int T, int d_k,
                                                                int m, int QB, bool rows_together)
{
    extern __shared__ float q_s[];  // [QB][DSUB]
    const RowBlock block = row_block(rows_together);
    const int i = block.i, h = block.h;
    const int c = threadIdx.x;
    const int64_t nq = (int64_t)B * T;
    const int64_t q0 = (int64_t)block.part * QB;

    float row[DSUB];
    if constexpr (DSUB >= 32) {
        const float *src = codebooks + (((int64_t)h * m + i) * kCentroids + c) * DSUB;
#pragma unroll
        for (int j = 0; j < DSUB; ++j)
            row[j] = src[j];
    }
    for (int e = threadIdx.x; e < QB * DSUB; e += kLutThreads) {
        const int64_t qi = q0 + e / DSUB;
        float v = 0.f;
        if (qi < nq) {
            int64_t b, t;
            split_query(qi, T, b, t);
            v = to_f32<QT>(q[((b * H + h) * T + t) * d_k + (int64_t)i * DSUB + e % DSUB]);
        }
        q_s[e] = v;
    }
    if constexpr (DSUB < 32) {
        const float *src = codebooks + (((int64_t)h * m + i) * kCentroids + c) * DSUB;
#pragma unroll
        for (int j = 0; j < DSUB; ++j)
            row[j] = src[j];
    }
    __syncthreads();

    for (int k = 0; k < QB; ++k) {
        const int64_t qi = q0 + k;
        if (qi >= nq)
            break;
        float acc = 0.f;
#pragma unroll
        for (int j = 0; j < DSUB; ++j)
            acc = fmaf(q_s[k * DSUB + j], row[j], acc);
        int64_t b, t;
        split_query(qi, T, b, t);
        lut[((((b * H + h) * T + t) * m) + i) * kCentroids + c] = acc;
    }
}

// Any d_sub: the same, the centroid's row taken JB coordinates at a time (8 for the shortest rows, else 32; longer rows come from cache
// again for every query).  Latency is what counts in a decode step (one query per sequence): the row is requested at once, in 16-byte
// pieces where it has them, beside the queries.  us per call, element by element as they were needed / now: 32 x 12 (b,h) x 1 query, m = 8,
// d_k = 96 15.0 / 6.5, d_k = 112 20.3 / 9.7; 16 x 12, d_k = 160, m = 4, fp32 32 / 8.9; 8 x 32 x 8 queries, d_k = 96, m = 8 71 / 26.
template <typename QT, int JB>
__global__ __launch_bounds__(kLutThreads) void build_lut_generic_kernel(const QT *__restrict__ q,
                                                                        const float *__restrict__ codebooks,
                                                                        float *__restrict__ lut, int B, int H, int T,
                                                                        int d_k, int m, int QB, bool rows_together)
{
    extern __shared__ float q_s[];  // [QB][d_sub]
    const int d_sub = d_k / m;
    const RowBlock block = row_block(rows_together);
    const int i = block.i, h = block.h;
    const int c = threadIdx.x;
    const int64_t nq = (int64_t)B * T;
    const int64_t q0 = (int64_t)block.part * QB;
    const float *src = codebooks + (((int64_t)h * m + i) * kCentroids + c) * d_sub;
    float row[JB];
    auto fetch = [&](int j0) {                      // coordinates j0 .. j0 + JB - 1 as far as there are any
        if (d_sub % 4 == 0) {                       // (rows of 16-byte pieces, from a 16-byte aligned codebook)
#pragma unroll
            for (int p = 0; p < JB; p += 4)
                if (j0 + p < d_sub) {
                    const float4 v = *reinterpret_cast<const float4 *>(src + j0 + p);
                    row[p] = v.x;
                    row[p + 1] = v.y;
                    row[p + 2] = v.z;
                    row[p + 3] = v.w;
                }
        } else {
#pragma unroll
            for (int p = 0; p < JB; p += 8)
                if (j0 + p < d_sub)                 // (a branch per eight; past the end the last one again, not used)
#pragma unroll
                    for (int e = p; e < p + 8; ++e)
                        row[e] = src[j0 + e < d_sub ? j0 + e : d_sub - 1];
        }
    };
    fetch(0);
    {                                               // 256 / QB threads per query (QB is a power of two, 16 at most)
        const int per = kLutThreads / QB, k = c / per;
        const int64_t qi = q0 + k;
        if (qi < nq) {
            int64_t b, t;
            split_query(qi, T, b, t);
            for (int j = c % per; j < d_sub; j += per)
                q_s[k * d_sub + j] = to_f32<QT>(q[((b * H + h) * T + t) * d_k + (int64_t)i * d_sub + j]);
        }
    }
    __syncthreads();
    for (int k = 0; k < QB; ++k) {
        const int64_t qi = q0 + k;
        if (qi >= nq)
            break;
        float acc = 0.f;
        for (int j0 = 0; j0 < d_sub; j0 += JB) {
            if (d_sub > JB && (j0 > 0 || k > 0))
                fetch(j0);
#pragma unroll
            for (int p = 0; p < JB; ++p)
                if (j0 + p < d_sub)
                    acc = fmaf(q_s[k * d_sub + j0 + p], row[p], acc);
        }
        int64_t b, t;
        split_query(qi, T, b, t);
        lut[((((b * H + h) * T + t) * m) + i) * kCentroids + c] = acc;
    }
}

// ---- many queries per head: the table build is a dense contraction -> matrix cores ------
// Per (head h, subspace i):  LUT[r][c] = sum_j Q[r][j] * C[c][j]  with r over the B*T queries
// of the head, c over the 256 centroids, j over d_sub: an [R x d_sub] . [d_sub x 256] product on
// v_mfma_f32_32x32x2_f32 (fp32 in, fp32 accumulate: same accuracy class as the vector kernel).
// What bounds it: the output stream (d_sub*2 flops per 4 bytes written), and that stream depends on the order in which it
// is written.  One workgroup makes 32 queries x 256 centroids of one subspace, 32 KB, and ends; the subspaces of the same
// queries, then the next queries, are made by the workgroups that follow, so what the chip writes at one time is
// one compact piece of the tables.  A launch that only stores writes 1.07 GB in this order in 155 us, 182-218 us with the
// 256 KB strips of 256 queries of one subspace that a workgroup made before (its codebook slice kept in registers).
// us per call before / now: 4 x 32 x 512 queries, m = 16 (1.07 GB) 194 / 175; 32 x 12 x 128, m = 4 86 / 53; 12 x 1000, m = 4, fp32
// 27.8 / 15.8; 256 x 32 x 1, m = 8 31.2 / 19.6; 3 x 7 x 333, m = 8 30.6 / 16.4.  The LDS holds four workgroups per compute unit;
// three: 176 us, two: 198.
// Sub-vectors of 32 and 64 (vector kernel / this one): 4 x 32 x 512 queries, d_k = 64, m = 2 77 / 56; 2 x 16 x 300, d_k = 128, m = 2
// 33 / 23; 4 x 32 x 300, d_k = 128, m = 4, fp32 87 / 71: the vector ALU's multiply-adds, not the stores, were the bound.
// Each wavefront makes 64 of the 256 centroids: two 32-column blocks of the MFMA, whose results cross LDS so that they leave
// as 1 KB table rows, 16 bytes per lane (stored straight from the accumulators, a store instruction would write 4 bytes
// per lane in two 128-byte pieces).  NTS = 1 writes with non-temporal stores: a table set far larger than
// the last-level cache is read back from HBM by its consumer whatever the stores do, and stores that do not
// allocate cache lines are faster; small table sets keep plain stores so that the consumer finds them in cache.
//   fragment layout of the 32x32x2 MFMA: A[row = lane%32][k = lane/32], B[k = lane/32][col = lane%32],
//   D[row = 8*(r/4) + 4*(lane/32) + r%4][col = lane%32] for accumulator register r = 0..15.
typedef float v16f __attribute__((ext_vector_type(16)));
constexpr int kMfmaWaves = 4;
constexpr int kMfmaRows = 32;            // queries per workgroup

typedef float lut_v4f __attribute__((ext_vector_type(4)));


// DSUB consecutive elements, loaded in pieces of up to 16 bytes (aligned to their size)
template <typename T, int DSUB>
__device__ __forceinline__ void lut_load_row(const T *src, T (&v)[DSUB])
{
    constexpr int kBytes = DSUB * (int)sizeof(T) < 16 ? DSUB * (int)sizeof(T) : 16;
    typedef uint32_t piece_t __attribute__((ext_vector_type(kBytes / 4)));
    constexpr int kPieces = DSUB * (int)sizeof(T) / kBytes;
    piece_t p[kPieces];
#pragma unroll
    for (int k = 0; k < kPieces; ++k)
        p[k] = reinterpret_cast<const piece_t *>(src)[k];
    __builtin_memcpy(v, p, sizeof(p));
}

template <typename QT, int DSUB, int NTS>
__global__ __launch_bounds__(kMfmaWaves *kWave) void build_lut_mfma_kernel(const QT *__restrict__ q,
                                                                           const float *__restrict__ codebooks,
                                                                           float *__restrict__ lut, int B, int H,
                                                                           int T, int d_k, int m, uint32_t run)
{
    constexpr int KS = DSUB / 2;
    constexpr int kBlocks = kCentroids / 32 / kMfmaWaves;     // 32-column blocks per wavefront
    constexpr int kStageStride = kCentroids + 4;              // floats per staged table row (pad: rows 4 apart on distinct banks)
    __shared__ __align__(16) float stage_s[kMfmaRows * kStageStride];
    // subspaces fastest, then `run` query tiles (a batch entry's), then heads, then the next tiles
    const uint32_t w0 = blockIdx.x, w1 = w0 / (uint32_t)m, w2 = w1 / run, w3 = w2 / (uint32_t)H;
    const int i = (int)(w0 - w1 * (uint32_t)m);
    const int h = (int)(w2 - w3 * (uint32_t)H);
    const int64_t nq = (int64_t)B * T;
    const int64_t r0 = ((int64_t)w3 * run + (w1 - w2 * run)) * kMfmaRows;
    if (r0 >= nq)
        return;
    const int b0 = (int)((uint32_t)r0 / (uint32_t)T);         // (B*T < 2^31)
    const int t0 = (int)((uint32_t)r0 - (uint32_t)b0 * (uint32_t)T);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n = lane & 31;
    const int kh = lane >> 5;

    float a[KS], c[kBlocks][KS];
    {
        int b = b0, t = r0 + n < nq ? t0 + n : t0;            // past the end: any query of the tile (not stored)
        if (t >= T) {
            b += t / T;
            t %= T;
        }
        QT qv[DSUB];
        lut_load_row<QT, DSUB>(q + (((int64_t)b * H + h) * T + t) * d_k + (int64_t)i * DSUB, qv);
        const float *cb = codebooks + (((int64_t)h * m + i) * kCentroids + wave * (32 * kBlocks) + n) * DSUB;
        float cv[kBlocks][DSUB];
#pragma unroll
        for (int nb = 0; nb < kBlocks; ++nb)
            lut_load_row<float, DSUB>(cb + nb * 32 * DSUB, cv[nb]);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            a[s] = kh ? to_f32<QT>(qv[2 * s + 1]) : to_f32<QT>(qv[2 * s]);
#pragma unroll
            for (int nb = 0; nb < kBlocks; ++nb)
                c[nb][s] = kh ? cv[nb][2 * s + 1] : cv[nb][2 * s];
        }
    }
#pragma unroll
    for (int nb = 0; nb < kBlocks; ++nb) {
        v16f acc;
#pragma unroll
        for (int rr = 0; rr < 16; ++rr)
            acc[rr] = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], c[nb][s], acc, 0, 0, 0);
#pragma unroll
        for (int rr = 0; rr < 16; ++rr)
            stage_s[(8 * (rr / 4) + 4 * kh + (rr % 4)) * kStageStride + (wave * kBlocks + nb) * 32 + n] = acc[rr];
    }
    __syncthreads();
    // a wavefront stores whole table rows, one per instruction
#pragma unroll
    for (int k = 0; k < kMfmaRows / kMfmaWaves; ++k) {
        const int row = k * kMfmaWaves + wave;
        if (r0 + row >= nq)
            break;
        int b = b0, t = t0 + row;
        if (t >= T) {
            b += t / T;
            t %= T;
        }
        const lut_v4f v = *reinterpret_cast<const lut_v4f *>(stage_s + row * kStageStride + 4 * lane);
        lut_v4f *dst = reinterpret_cast<lut_v4f *>(lut + ((((int64_t)b * H + h) * T + t) * m + i) * kCentroids) + lane;
        if (NTS)
            __builtin_nontemporal_store(v, dst);
        else
            *dst = v;
    }
}

template <typename QT>
static bool launch_build_lut_mfma(const lookat_shape *s, int T, const void *q, const float *codebooks, float *lut,
                                  hipStream_t st)
{
    const int d_sub = s->d_k / s->m;
    const int64_t nq = (int64_t)s->B * T;
    const int64_t ntiles = (nq + kMfmaRows - 1) / kMfmaRows;
    const int64_t run = T >= kMfmaRows ? T / kMfmaRows : 1;
    const int64_t wgs = (ntiles + run - 1) / run * run * s->H * s->m;
    if (wgs > 0xffffffLL)          // (a grid of 2^32 threads; 550 GB of tables)
        return false;
    dim3 grid((unsigned)wgs);
    dim3 block(kMfmaWaves * kWave);
    const QT *qp = static_cast<const QT *>(q);
    // tables that fill the last-level cache (256 MB) bypass it on the way out (us to build / to read once by a
    // reduction, plain and non-temporal stores: 192 MB 49 / 47 and 48 / 67; 256 MB 59 / 77 and 46 / 84)
    const bool nts = (int64_t)nq * s->H * s->m * kCentroids * (int64_t)sizeof(float) >= (int64_t)256 << 20;
#define LOOKAT_LUTM_CASE(D)                                                                                       \
    case D:                                                                                                       \
        if (nts)                                                                                                  \
            hipLaunchKernelGGL((build_lut_mfma_kernel<QT, D, 1>), grid, block, 0, st, qp, codebooks, lut, s->B,   \
                               s->H, T, s->d_k, s->m, (uint32_t)run);                                             \
        else                                                                                                      \
            hipLaunchKernelGGL((build_lut_mfma_kernel<QT, D, 0>), grid, block, 0, st, qp, codebooks, lut, s->B,   \
                               s->H, T, s->d_k, s->m, (uint32_t)run);                                             \
        return true;
    switch (d_sub) {
        LOOKAT_LUTM_CASE(2)
        LOOKAT_LUTM_CASE(4)
        LOOKAT_LUTM_CASE(8)
        LOOKAT_LUTM_CASE(16)
        LOOKAT_LUTM_CASE(32)
        LOOKAT_LUTM_CASE(64)
    default:
        return false;   // other sub-vectors: vector kernel
    }
#undef LOOKAT_LUTM_CASE
}

// Which workgroups follow each other: the queries of one subspace, which go to the eight dies in turn so that every die fetches the subspace's rows
// (d_sub KB), or the subspaces of the same queries: with m*H a multiple of eight a subspace's rows are then fetched by one die and found there by
// the next queries.  With rows below 12 coordinates the tables (a KB a query) are what counts: the first order is up to 4% faster where m*H is no
// multiple, and with many queries the attention that reads the tables is faster behind it (append, tables and attention of 32 x 32 heads, 300 keys,
// 8 subspaces of 8, 21.6 / 22.3 us; of 16 x 25 heads 18.8 / 17.7): there up to 16 queries only.  us per table call, first /
// second: 256 (head, subspace) x 4 queries, d_sub 4 2.5 / 2.5, 8 2.8 / 2.5, 12 4.9 / 3.9, 16 4.7 / 3.0, 20 6.1 / 4.2, 32 7.6 / 5.7; x 32, 4 4.7 / 4.6,
// 8 5.5 / 4.8, 16 7.2 / 5.9, 32 10.7 / 10.0; x 240, 8 18.3 / 17.2, 16 22.8 / 22.3, 32 39.6 / 38.5; 64 x 128, 40 52.5 / 35.8; 100 x 32, 8 3.3 / 3.4,
// 16 5.1 / 4.2.  Few subspaces whose number is no multiple of eight go round the dies in either order, and up to 28 coordinates the first is faster:
// 20 x 40, 16 3.2 / 3.4, 20 x 100 4.3 / 4.6, 2 x 200 2.7 / 2.8.  (The grid's last dimension ends at 65535.)
static bool lut_rows_together(const lookat_shape *s, int64_t nq, int64_t blocks)
{
    const int d_sub = s->d_k / s->m;
    const int64_t tables = (int64_t)s->m * s->H;
    if (blocks > 65535)
        return false;
    return d_sub >= 32 || (tables % 8 == 0 ? d_sub >= 12 || nq <= 16 : d_sub >= 12 && tables >= 96);
}

template <typename QT>
static void launch_build_lut(const lookat_shape *s, int T, const void *q, const float *codebooks, float *lut,
                             hipStream_t st)
{
    const int d_sub = s->d_k / s->m;
    const int64_t nq = (int64_t)s->B * T;
    // queries per block: reuse the centroid registers, but keep >= ~1024 blocks in flight
    int QB = 1;
    while (QB < 16 && (nq / (QB * 2)) * s->m * s->H >= 1024)
        QB *= 2;
    const int64_t blocks = (nq + QB - 1) / QB;
    const bool together = lut_rows_together(s, nq, blocks);
    const dim3 grid = row_grid(s, blocks, together);
    dim3 block(kLutThreads);
    const QT *qp = static_cast<const QT *>(q);
#define LOOKAT_LUT_CASE(D)                                                                                         \
    case D:                                                                                                        \
        hipLaunchKernelGGL((build_lut_kernel<QT, D>), grid, block, (size_t)QB * D * sizeof(float), st, qp,         \
                           codebooks, lut, s->B, s->H, T, s->d_k, s->m, QB, together);                             \
        break;
    switch (d_sub) {
        LOOKAT_LUT_CASE(1)
        LOOKAT_LUT_CASE(2)
        LOOKAT_LUT_CASE(4)
        LOOKAT_LUT_CASE(8)
        LOOKAT_LUT_CASE(16)
        LOOKAT_LUT_CASE(32)
        LOOKAT_LUT_CASE(64)
    default:
        if (d_sub <= 8)
            hipLaunchKernelGGL((build_lut_generic_kernel<QT, 8>), grid, block, (size_t)QB * d_sub * sizeof(float), st, qp,
                               codebooks, lut, s->B, s->H, T, s->d_k, s->m, QB, together);
        else
            hipLaunchKernelGGL((build_lut_generic_kernel<QT, 32>), grid, block, (size_t)QB * d_sub * sizeof(float), st, qp,
                               codebooks, lut, s->B, s->H, T, s->d_k, s->m, QB, together);
        break;
    }
#undef LOOKAT_LUT_CASE
}

}  // namespace lookat

extern "C" int lookat_build_lut(const lookat_shape *shape, int32_t T, const void *q, lookat_dtype q_dtype,
                                const float *codebooks, float *lut, void *stream)
{
    using namespace lookat;
    clear_error();
    if (int rc = check_shape(shape))
        return rc;
    if (T <= 0)
        return fail(LOOKAT_ERR_SHAPE, "T=%d must be positive", T);
    if (q_dtype != LOOKAT_F16 && q_dtype != LOOKAT_F32)
        return fail(LOOKAT_ERR_DTYPE, "q_dtype=%d is neither LOOKAT_F16 nor LOOKAT_F32", q_dtype);
    if (!q || !codebooks || !lut)
        return fail(LOOKAT_ERR_NULL, "q, codebooks and lut must be non-NULL");
    if (!aligned16(q) || !aligned16(codebooks) || !aligned16(lut))
        return fail(LOOKAT_ERR_ALIGN, "q, codebooks and lut must be 16-byte aligned");
    if ((int64_t)shape->B * T > 0x7fffffffLL || shape->H > 65535)
        return fail(LOOKAT_ERR_UNSUPPORTED, "B*T or H too large for one launch");
    hipStream_t st = static_cast<hipStream_t>(stream);
    // From 256 queries per head on, the build is a dense [B*T x d_sub].[d_sub x 256] contraction
    // per (head, subspace) and runs on the matrix cores; below that the 32-row MFMA tiles would be
    // mostly padding and the vector kernel is used.  With 32 and 64 coordinates a tile is a chain of 16 or 32 matrix instructions, and
    // up to three tables per compute unit the vector kernel ends sooner (us, vector / matrix; m = 1 or 2, d_sub 64: 256 tables 3.9 / 7.6, fp32
    // queries 8.1; 512 5.7 / 7.7; 768 7.4 / 7.7, 8.1; 900 9.5 / 7.7, 8.2; d_sub 32: 256 2.9 / 4.7, 5.2; 768 4.7 / 4.8, 5.3; 900 5.7 / 4.8, 5.3).
    // Both kernels add the products in the same order: the tables have the same bits.
    const int64_t queries = (int64_t)shape->B * T;
    bool done = false;
    if (queries >= 256 && (shape->d_k / shape->m < 32 || queries * shape->H * shape->m > 768))
        done = (q_dtype == LOOKAT_F16) ? launch_build_lut_mfma<__half>(shape, T, q, codebooks, lut, st)
                                       : launch_build_lut_mfma<float>(shape, T, q, codebooks, lut, st);
    if (!done) {
        if (q_dtype == LOOKAT_F16)
            launch_build_lut<__half>(shape, T, q, codebooks, lut, st);
        else
            launch_build_lut<float>(shape, T, q, codebooks, lut, st);
    }
    return check_launch("lookat_build_lut");
}
