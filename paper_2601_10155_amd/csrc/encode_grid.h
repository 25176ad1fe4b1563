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

// What a launch takes on the fullest compute unit, in 1/64 of the time of a pair of key blocks on every wavefront where eight run (about
// 2.1 us with 8 coordinates, 3.7 with 64 fp16 ones): with n workgroups at once start[n] (scale, operands, norms, the round of undecided
// keys) and pair[n] for a pair of each wavefront's.  A workgroup of 512 threads sets up once for twice as many wavefronts; two of 256
// measured 5 to 15% slower at the same work, and one alone has half the wavefronts but needs more than half as long for a pair.  Two terms
// of everything save the undecided keys' round and cost more matrix instructions.
// Fitted to 162 fills of 1 to 250 pairs per (head, subspace), every form and split timed: the choice is 1% from the best on average
// (23% at worst, where the few undecided keys of an input decide).
struct EfForm {
    int threads;
    bool fine;
    uint32_t resident;
    int start[4], pair[4];

    EfForm(int dp, bool key32, int threads_, bool fine_)
        : threads(threads_), fine(fine_), resident((uint32_t)ef_resident(dp, threads_, fine_)), start{}, pair{}
    {
        const int setup = (dp <= 8 ? 96 : (dp == 16 ? 150 : (dp == 32 ? 200 : 215))) - (fine && dp > 8 ? 52 : 0);
        const int one = fine ? (key32 ? 68 : 62) : 52;
        start[0] = setup * 3 / 8;                         // a later set-up overlaps a little with the end of the round before
        start[1] = threads == 512 ? setup : setup - 20;
        start[2] = dp > 4 || fine ? setup + 12 : setup + 8;
        start[3] = dp > 4 || fine ? setup + 12 : setup + 16;
        pair[1] = threads == 512 ? 64 : one;
        pair[2] = fine ? one * 27 / 20 : (dp > 4 ? 72 : 68);
        pair[3] = fine ? one * 2 : 96;
    }
    // c workgroups with `pairs` pairs per wavefront on one compute unit
    int64_t cost(uint32_t c, int64_t pairs) const
    {
        if (c <= resident)
            return start[c] + pair[c] * pairs;
        const uint32_t full = resident == 1 ? c - 1 : (resident == 2 ? (c - 1) / 2 : (c - 1) / 3), last = c - full * resident;
        const int64_t round = pair[resident] * pairs;     // (the last round is as fast as its share of a full one)
        return full * (start[resident] - start[0] + round) + start[resident] + (last == resident ? round : (resident == 2 ? round / 2 : round * last / 3));
    }
};

struct EfGrid {
    int splits;      // workgroups per (head, subspace)
    int threads;
    bool fine;
};

// The form and the number of splits with the least cost, for `units` (head, subspace) pairs (below 2^22) with `pairs` pairs of key blocks
// (below 2^30) each.  For a number of workgroups on the fullest of the 256 compute units only the largest split count that stays within it is
// of interest; 24 such numbers from the smallest are looked at (0.04 to 0.5 us on the host).
inline EfGrid ef_grid(int64_t units, int64_t pairs, int dp, bool key32)
{
    EfGrid best = {1, 256, false};
    int64_t best_cost = INT64_MAX;
    const uint32_t u = (uint32_t)units, p = (uint32_t)pairs;   // (32-bit divisions)
    const uint32_t first = (u + 255) / 256;
    for (int f = ef_has_large(dp) ? 0 : 1; f < (ef_has_fine(dp, key32) ? 3 : 2); ++f) {
        const EfForm form(dp, key32, f == 0 ? 512 : 256, f == 2);
        const uint32_t waves = f == 0 ? 8 : 4;
        uint32_t before = 0;
        for (uint32_t c = first; c < first + 24; ++c) {
            uint32_t s = 256 * c / u;
            s = s < 1024 ? s : 1024;
            if (s == before)
                continue;
            before = s;
            const uint32_t per_wave = (p + s * waves - 1) / (s * waves);
            const int64_t cost = form.cost((u * s + 255) / 256, per_wave);
            if (cost < best_cost) {
                best_cost = cost;
                // (the fewest splits with as many pairs per wavefront)
                best = EfGrid{(int)((p + per_wave * waves - 1) / (per_wave * waves)), form.threads, form.fine};
            }
            if (per_wave == 1)
                break;
        }
    }
    return best;
}

}  // namespace lookat
