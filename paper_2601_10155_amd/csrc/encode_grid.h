// How the ranking encoder's work is split over the chip (host arithmetic only).
#pragma once

#include <stdint.h>

namespace lookat {

// Coordinates of a matrix operand that takes sub-vectors of d_sub coordinates (2 to 64).
constexpr int ef_operand(int d_sub) { return d_sub <= 4 ? 4 : (d_sub <= 8 ? 8 : (d_sub <= 16 ? 16 : (d_sub <= 32 ? 32 : 64))); }

// The three forms of a kernel: 512 threads, 256 threads, 256 threads with two terms of everything (fine).  Which there are, and how many
// workgroups of each a compute unit holds (by registers, and with 64 coordinates in two terms by LDS).
constexpr bool ef_has_large(int dp) { return dp > 4; }
constexpr bool ef_has_fine(int dp, bool key32) { return dp > 8 || (dp == 8 && key32); }
constexpr int ef_resident(int dp, int threads, bool fine)
{
    return threads == 512 ? 1 : (fine ? (dp == 8 ? 3 : (dp == 64 ? 1 : 2)) : (dp == 4 ? 3 : 2));
}

// What a launch takes on the fullest compute unit, in 1/32 of the time of a pair of key blocks on a SIMD that two wavefronts share (about 1.05
// us with 8 coordinates, 1.85 with 64 fp16 ones): with n workgroups at once start[n] (scale, operands, norms, the round of undecided keys) and
// pair[n] for a pair on each SIMD.  A workgroup of 512 threads sets up once for two wavefronts per SIMD; two of 256 measured 5 to 15% slower
// at the same work, but their later rounds start while others still run, where 512 threads wait for their slowest.  One wavefront alone on a
// SIMD needs half as long again for a pair.  Two terms of everything save the undecided keys' round and cost more matrix instructions.
// Fitted to 780 fills of 1 to 3000 pairs per (head, subspace), every form and up to 20 split counts timed: the choice is 0.9% from the best
// on average (4% with a choice that knew neither the dies nor that one workgroup of the fine form fills a compute unit).
struct EfForm {
    int threads;
    bool fine;
    uint32_t resident;
    int start[4], pair[4], again;

    EfForm(int dp, bool key32, int threads_, bool fine_)
        : threads(threads_), fine(fine_), resident((uint32_t)ef_resident(dp, threads_, fine_)), start{}, pair{}
    {
        const int setup = dp <= 8 ? 92 : (dp == 16 ? 150 : (dp == 32 ? 200 : 215));
        const int from = setup - (fine ? (dp == 8 ? 40 : 48) : 0), one = fine ? (key32 ? 68 : 64) : 52;
        start[1] = threads == 512 ? setup : from - 18;
        start[2] = dp > 4 ? from + 12 : from + 8;
        start[3] = dp > 4 ? from + 12 : from + 16;
        pair[1] = threads == 512 ? 32 : one;
        pair[2] = fine ? one * 27 / 20 : (dp > 4 ? 70 : 68);
        pair[3] = fine ? one * 2 : 92;
        again = threads == 512 ? setup : -setup * 3 / 8;      // every round but the last
    }
    // c workgroups on one compute unit, `pairs` on the fullest SIMD of each
    int64_t cost(uint32_t c, int64_t pairs) const
    {
        const uint32_t n = c < resident ? c : resident;
        const int64_t alone = threads == 512 && pairs % 2 ? (pairs == 1 ? 20 : 12) : 0, round = pair[n] * pairs + alone;
        if (c <= resident)
            return start[n] + round;
        const uint32_t full = resident == 1 ? c - 1 : (resident == 2 ? (c - 1) / 2 : (c - 1) / 3), last = c - full * resident;
        // (the last round is as fast as its share of a full one)
        return full * (start[n] + again + round) + start[n] + (last == resident ? round : (resident == 2 ? round / 2 : round * last / 3));
    }
};

struct EfGrid {
    int splits;      // workgroups per (head, subspace)
    int threads;
    bool fine;
};

// Workgroups on the fullest compute unit: heads x splits are dealt to the eight dies in turn, with all their subspaces, and a die has 32.
inline uint32_t ef_on_a_cu(uint32_t heads, uint32_t subspaces, uint32_t splits) { return ((heads * splits + 7) / 8 * subspaces + 31) / 32; }

// The form and the number of splits with the least cost for heads (below 2^16) x subspaces (up to 32) with `pairs` pairs of key blocks (below
// 2^30) each.  For a number of workgroups on the fullest compute unit only the largest split count that stays within it is of interest; 24
// such numbers from the smallest are looked at (0.04 to 0.5 us on the host).
inline EfGrid ef_grid(int heads, int subspaces, int64_t pairs, int dp, bool key32)
{
    EfGrid best = {1, 256, false};
    int64_t best_cost = INT64_MAX;
    const uint32_t h = (uint32_t)heads, m = (uint32_t)subspaces, p = (uint32_t)pairs;   // (32-bit divisions)
    const uint32_t first = ef_on_a_cu(h, m, 1);
    for (int f = ef_has_large(dp) ? 0 : 1; f < (ef_has_fine(dp, key32) ? 3 : 2); ++f) {
        const EfForm form(dp, key32, f == 0 ? 512 : 256, f == 2);
        const uint32_t most = f == 0 ? (p + 7) / 8 : (p + 3) / 4;      // a pair per wavefront
        uint32_t before = 0;
        for (uint32_t c = first; c < first + 24 && before != most; ++c) {
            uint32_t s = 8 * (32 * c / m) / h;
            s = s < 1024 ? s : 1024;
            s = s < most ? s : most;
            if (s == before)
                continue;
            before = s;
            const int64_t cost = form.cost(ef_on_a_cu(h, m, s), ((p + s - 1) / s + 3) / 4);
            if (cost < best_cost) {
                best_cost = cost;
                best = EfGrid{(int)s, form.threads, form.fine};
            }
        }
    }
    return best;
}

}  // namespace lookat
