// Codebook learning (paper Sec. 3.4, "Prototype Learning"): one Lloyd iteration of k-means
// per (head, subspace).  Assignment is the key encoder itself; the update moves every
// centroid to the mean of its members.  The mean is an fp64 sum taken in ascending key
// order by a single thread per (centroid, coordinate), so the result does not depend on
// scheduling and is reproducible bit for bit.
#include "common.h"

namespace lookat {

// Update: one workgroup per (head, subspace, up to kKmPieces pieces of V coordinates).  The keys are taken
// kKmChunk at a time; for a chunk the workgroup turns the assignment column into per-centroid member lists in LDS
// and thread (centroid, piece) adds the members of its centroid to sums it keeps in registers.  The lists hold
// the members in ascending key order, so every sum is taken in the order a scan of all keys would take.
// List building is a stable counting sort by code.  Each of the sixteen (eight) wavefronts owns a contiguous
// share of the chunk and keeps its codes in registers: it histograms them (LDS atomics; counts do not depend on
// order), 256 threads turn these histograms into every (wavefront, code) pair's first slot, and
// each wavefront then walks its share 64 keys at a time in ascending order: the lanes that hold
// equal codes find each other with eight ballots (one per code bit), a lane's slot is the pair's
// running offset plus the number of equal-code lanes below it, and the lowest of them advances
// the offset.  (LDS operations of one wavefront execute in program order.)
// What bounds it: scattered reads.  The sums are serial chains behind reads of V * 4 bytes, 4 d_sub of a row, so a thread
// requests kKmBatch members' pieces before it adds the first, and a sub-vector longer than 16 coordinates is shared by
// several workgroups, each with its own lists (cheap beside the reads).  Half of every 128-byte line belongs to another
// subspace at d_sub = 16: the workgroups of a head run side by side on one die and take the same chunk of keys at about
// the same time, so that its L2 serves the other half.  32 heads x 16384 keys x 128 coordinates, m = 8: 305 us with 256 threads,
// four single floats in flight and every thread taking d_sub chains in turn; 113 us with 1024 threads, 16-byte pieces
// and eight in flight; 86 us with the subspaces of a head on one die and chunks of 4096 keys (2048: 93, 8192: 93, 16384: 103;
// 12 or 16 pieces in flight: no change; the lists alone: 29); 80 us with the next chunk's lists built while members are on their way (AHEAD: for
// sets of more than one chunk; whole steps, without / with: 32 x 16384, d_k = 128, m = 8 184.6 / 178.5 us, 4 x 24000, d_k = 64, m = 4 85 / 70;
// for one chunk there is nothing to overlap, and the second buffer costs a workgroup per compute unit: 40 x 512, d_k = 64, m = 16 19.4 / 22.6).
// Left at 32 x 16384: 333 MB fetched where 268 are needed, the address units busy 56% of the time.  Centroids dealt to the wavefronts by
// size, so that none waits for the largest lists: 84 us; the codes requested a chunk ahead: 84.
//   LDS: first[257] | run[16][256] (512 threads: [8][256]) | list [kKmChunk] uint16; AHEAD: first and list twice
//   grid = (8 heads x m x groups of a sub-vector's pieces, ceil(H / 8)), 512 or 1024 threads; consecutive workgroups go to the
//   eight dies in turn
constexpr int kKmPieces = 4;                         // 1024 threads, one (centroid, piece) each
constexpr int kKmChunk = 4096;
constexpr int kKmBatch = 8;

template <int V, int THREADS, bool AHEAD>
__global__ __launch_bounds__(THREADS) void kmeans_update_kernel(const float *__restrict__ calib,
                                                                   const uint8_t *__restrict__ assign,
                                                                   const float *__restrict__ cb_in,
                                                                   float *__restrict__ cb_out, int64_t Nc, int d_k,
                                                                   int H, int m, int groups, int pieces_per_wg)
{
    constexpr int kKmThreads = THREADS;
    constexpr int kKmWaves = kKmThreads / kWave;
    constexpr int kKmRounds = kKmChunk / kKmThreads;     // 64-key rounds of a wavefront in a full chunk
    typedef float vec_t __attribute__((ext_vector_type(V)));
    __shared__ uint32_t first_s[AHEAD ? 2 : 1][kCentroids + 1];
    __shared__ uint32_t run_s[kKmWaves][kCentroids];
    __shared__ uint16_t list_s[AHEAD ? 2 : 1][kKmChunk];
    __shared__ uint32_t wave_tot[kCentroids / kWave];

    const int d_sub = d_k / m;
    // all workgroups of a head side by side on one die
    const int h = (int)blockIdx.y * 8 + blockIdx.x % 8;
    if (h >= H)
        return;
    const int slot = blockIdx.x / 8;
    const int i = slot / groups;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const int p0 = slot % groups * pieces_per_wg;
    const int np = (d_sub / V - p0) < pieces_per_wg ? (d_sub / V - p0) : pieces_per_wg;
    const bool sums = tid < kCentroids * np;         // this thread owns a (centroid, piece)
    const int c = sums ? tid / np : 0;
    const int piece = p0 + (sums ? tid % np : 0);
    const uint8_t *as = assign + (int64_t)h * Nc * m + i;
    const float *x = calib + (int64_t)h * Nc * d_k + (int64_t)i * d_sub + piece * V;

    double sum[V];
#pragma unroll
    for (int e = 0; e < V; ++e)
        sum[e] = 0.0;
    int64_t members = 0;

    // The members at hand, [at, end) of the lists of one chunk, kKmBatch of them requested.
    uint32_t at = 0, end = 0;
    const uint16_t *list = list_s[0];
    const float *rows = x;
    vec_t v[kKmBatch];
    auto fetch = [&] {
#pragma unroll
        for (int k = 0; k < kKmBatch; ++k)   // past the end: the last member again, not added
            v[k] = *reinterpret_cast<const vec_t *>(rows + (int64_t)list[at + k < end ? at + k : end - 1] * d_k);
    };
    auto take = [&] {
#pragma unroll
        for (int k = 0; k < kKmBatch; ++k)
            if (at + k < end) {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    sum[e] += (double)v[k][e];
            }
        at += kKmBatch;
    };
    auto request = [&] {
        if (at < end)
            fetch();
    };
    auto add = [&] {
        if (at < end)
            take();
    };

    // AHEAD: chunk n0's lists are built while the members of the chunk before it are fetched, each step of the sort starts with a batch requested.
    for (int64_t n0 = 0, buf = 0;; n0 += kKmChunk, buf ^= AHEAD ? 1 : 0) {
        const int len = n0 >= Nc ? 0 : (Nc - n0 < kKmChunk ? (int)(Nc - n0) : kKmChunk);
        // this wavefront's share of the chunk: [q0, q1), a multiple of 64 long except at the end
        const int rounds = (len + kKmThreads - 1) / kKmThreads;
        const int q0 = wave * rounds * kWave < len ? wave * rounds * kWave : len;
        const int q1 = q0 + rounds * kWave < len ? q0 + rounds * kWave : len;
        uint32_t code[kKmRounds];
#pragma unroll
        for (int r = 0; r < kKmRounds; ++r) {
            const int n = q0 + r * kWave + lane;
            code[r] = (r < rounds && n < q1) ? as[(n0 + n) * m] : 0u;
        }
        if constexpr (AHEAD) {
            request();
            if (len == 0)
                break;
        }
        for (int e = tid; e < kKmWaves * kCentroids; e += kKmThreads)
            run_s[e / kCentroids][e % kCentroids] = 0u;
        __syncthreads();
        uint32_t *run_w = run_s[wave];
#pragma unroll
        for (int r = 0; r < kKmRounds; ++r)
            if (r < rounds && q0 + r * kWave + lane < q1)
                atomicAdd(&run_w[code[r]], 1u);
        if constexpr (AHEAD) {
            add();
            request();
        }
        __syncthreads();

        // thread t < 256: members of centroid t per wavefront -> first slot of (wavefront, t); exclusive prefix sum over t
        uint32_t cnt = 0, incl = 0;
        if (tid < kCentroids) {
#pragma unroll
            for (int w = 0; w < kKmWaves; ++w)
                cnt += run_s[w][tid];
            incl = cnt;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint32_t up = __shfl_up(incl, d);
                if (lane >= d)
                    incl += up;
            }
            if (lane == kWave - 1)
                wave_tot[wave] = incl;
        }
        __syncthreads();
        if (tid < kCentroids) {
            uint32_t pos = incl - cnt;
            for (int w = 0; w < wave; ++w)
                pos += wave_tot[w];
            first_s[buf][tid] = pos;
            if (tid == kCentroids - 1)
                first_s[buf][kCentroids] = pos + cnt;
#pragma unroll
            for (int w = 0; w < kKmWaves; ++w) {
                const uint32_t mine = run_s[w][tid];
                run_s[w][tid] = pos;
                pos += mine;
            }
        }
        __syncthreads();

        if constexpr (AHEAD) {
            add();
            request();
        }
#pragma unroll
        for (int r = 0; r < kKmRounds; ++r) {
            if (r < rounds) {   // wave-uniform
                const int n = q0 + r * kWave + lane;
                const bool valid = n < q1;
                uint64_t peers = __ballot(valid);
#pragma unroll
                for (int bit = 0; bit < 8; ++bit) {
                    const uint64_t set = __ballot((code[r] >> bit) & 1u);
                    peers &= ((code[r] >> bit) & 1u) ? set : ~set;
                }
                const uint32_t below = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
                const uint32_t to = run_w[code[r]];
                if (valid)
                    list_s[buf][to + below] = (uint16_t)n;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();   // every lane has read the offset before it moves
                if (valid && below == 0)
                    run_w[code[r]] = to + (uint32_t)__popcll(peers);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
        if constexpr (AHEAD) {
            while (at < end) {
                add();
                request();
            }
        }
        __syncthreads();   // the chunk's lists are there, those of the chunk before it are read
        if (sums) {
            at = first_s[buf][c];
            end = first_s[buf][c + 1];
            members += end - at;
            list = list_s[buf];
            rows = x + n0 * d_k;
        }
        if constexpr (!AHEAD) {
            while (at < end) {
                fetch();
                take();
            }
            if (n0 + kKmChunk >= Nc)
                break;
            __syncthreads();
        }
    }
    if constexpr (AHEAD) {
        while (at < end) {
            add();
            request();
        }
    }
    if (sums) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const int64_t o = (((int64_t)h * m + i) * kCentroids + c) * d_sub + piece * V + e;
            cb_out[o] = members ? (float)(sum[e] / (double)members) : cb_in[o];   // a centroid without members stays
        }
    }
}

}  // namespace lookat

extern "C" int lookat_kmeans_step(const lookat_shape *shape, int64_t Nc, const float *calib,
                                  const float *codebooks_in, float *codebooks_out, uint8_t *assign, void *stream)
{
    using namespace lookat;
    clear_error();
    if (int rc = check_shape(shape))
        return rc;
    if (shape->B != 1)
        return fail(LOOKAT_ERR_SHAPE, "kmeans_step takes one calibration set per head: B must be 1, got %d", shape->B);
    if (Nc <= 0)
        return fail(LOOKAT_ERR_SHAPE, "Nc=%lld must be positive", (long long)Nc);
    if (!calib || !codebooks_in || !codebooks_out || !assign)
        return fail(LOOKAT_ERR_NULL, "calib, codebooks_in, codebooks_out and assign must be non-NULL");
    if (codebooks_in == codebooks_out)
        return fail(LOOKAT_ERR_SHAPE, "codebooks_out must not alias codebooks_in");
    if (int rc = lookat_encode_keys(shape, Nc, calib, LOOKAT_F32, codebooks_in, assign, Nc * shape->m, stream))
        return rc;
    const int d_sub = shape->d_k / shape->m;
    const int V = d_sub % 4 == 0 ? 4 : 1;            // coordinates per load
    const int pieces = d_sub / V;
    // pieces per workgroup: four fill its 1024 threads; fewer where that would leave compute units without a workgroup
    int per = kKmPieces < pieces ? kKmPieces : pieces;
    while (per > 1 && (int64_t)shape->m * shape->H * ((pieces + per - 1) / per) < 256)
        per /= 2;
    const int groups = (pieces + per - 1) / per;      // workgroups per (head, subspace)
    const dim3 grid((unsigned)(8 * shape->m * groups), (unsigned)(((int64_t)shape->H + 7) / 8));
    hipStream_t st = static_cast<hipStream_t>(stream);
    // With one or two pieces per workgroup half of 1024 threads or more would only build lists.  Where there are more workgroups than
    // compute units, two of 512 on one list and add at different times (us per step, 1024 / 512 threads: 40 heads x 2000 keys, d_k = 128,
    // m = 16 67 / 60; 32 x 8000, d_k = 64, m = 16 127 / 113; 25 x 700 23.8 / 20.0), and up to 1024 keys there is little to list (12 x 600,
    // d_k = 64, m = 8 15.0 / 14.3); else the lists are made faster by all (4 x 24000, d_k = 64, m = 2 90.0 / 91.2; with four pieces, whose
    // lists two workgroups would build twice, 32 x 16384, d_k = 128, m = 8 175 / 203).
    const bool half = per <= 2 && ((int64_t)shape->m * shape->H * groups > 256 || Nc <= 1024);
#define LOOKAT_KM_LAUNCH_AHEAD(V, THREADS, AHEAD)                                                                         \
    hipLaunchKernelGGL((kmeans_update_kernel<V, THREADS, AHEAD>), grid, dim3(THREADS), 0, st, calib, assign, codebooks_in, \
                       codebooks_out, Nc, shape->d_k, shape->H, shape->m, groups, per)
#define LOOKAT_KM_LAUNCH(V, THREADS)                                                                                      \
    do {                                                                                                                  \
        if (Nc > kKmChunk)                                                                                                \
            LOOKAT_KM_LAUNCH_AHEAD(V, THREADS, true);                                                                     \
        else                                                                                                              \
            LOOKAT_KM_LAUNCH_AHEAD(V, THREADS, false);                                                                    \
    } while (0)
    if (V == 4 && half)
        LOOKAT_KM_LAUNCH(4, 512);
    else if (V == 4)
        LOOKAT_KM_LAUNCH(4, 1024);
    else if (half)
        LOOKAT_KM_LAUNCH(1, 512);
    else
        LOOKAT_KM_LAUNCH(1, 1024);
#undef LOOKAT_KM_LAUNCH
#undef LOOKAT_KM_LAUNCH_AHEAD
    return check_launch("lookat_kmeans_step (update kernel)");
}
