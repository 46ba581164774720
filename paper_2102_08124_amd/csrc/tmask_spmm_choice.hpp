// The tile size that a product of tmask_spmm24 runs with.  Host arithmetic in plain C++: the CPU tests compile this header
// by itself.
#pragma once
#include <cmath>
#include <cstdint>

namespace tmask {

constexpr uint64_t kSpmmThreads = 256;     // of a workgroup of any of the kernels
constexpr int64_t kSpmmStep = 64;          // k per step

// How many rounds (what the compute units do side by side) a launch of `full` tiles per compute unit takes:
enum SpmmRounds {
    kRoundsFraction,     // the smallest tiles: so many workgroups share a compute unit that rounds count in fractions
    kRoundsPairs,        // two workgroups share a compute unit, which then takes 1.6 times as long as for one
    kRoundsWhole
};

// What a product takes with tiles of rows x tokens, in microseconds: fixed + rounds (per_round + per_step cols / 64).
// The coefficients are a fit to 100 products (rows and cols 256 .. 4096, 1 .. 8192 tokens, bf16 results) timed with every
// tile size; the choice they lead to is on average 0.3 % and at most 10 % slower than the fastest tile, and 3.3 times as
// fast (geometric mean) as one kernel with 256 x 128 tiles for all: small tiles win while they fill no more than a few
// rounds, because a compute unit alone moves 50 GB/s whatever its tile (W 4096 x 1024, 16 tokens: 15.8 -> 3.6 us on 16 x 16
// tiles, 19 on 256 x 256; 1024 x 4096, 1003 tokens: 55 -> 16 us on 64 x 64 tiles, 60 on 256 x 256), large ones when there
// are many, because they move less (4096 x 1024, 8192 tokens: 55 us on 256 x 256, 70 on 128 x 128, 163 on 64 x 64).
struct SpmmTile {
    int64_t rows, tokens;
    SpmmRounds rounds_as;
    uint32_t persistent;                   // workgroups per compute unit that a launch has at most (0: one per tile)
    double fixed, per_round, per_step;

    uint64_t tiles(int64_t r, int64_t t) const { return (uint64_t)((r + rows - 1) / rows) * (uint64_t)((t + tokens - 1) / tokens); }

    // Tile numbers have 31 bits, and a launch fewer than 2^32 work-items in a dimension: a workgroup per tile reaches that
    // at 2^24 tiles.
    bool launchable(uint64_t n) const { return n <= 0x7FFFFFFFull && (persistent || n * kSpmmThreads <= 0xFFFFFFFFull); }

    double estimate(uint64_t n, int64_t cols, uint64_t cus) const
    {
        const double full = (double)n / (double)cus;
        double rounds = std::ceil(full);
        if (rounds_as == kRoundsFraction)
            rounds = full > 1.0 ? full : 1.0;
        else if (rounds_as == kRoundsPairs && full > 1.0)
            rounds = 1.6 * (full > 2.0 ? std::ceil(2.0 * full) / 4.0 : 1.0);
        return fixed + rounds * (per_round + per_step * (double)(cols / kSpmmStep));
    }
};

constexpr int kSpmmTiles = 7;
constexpr SpmmTile kSpmmTile[kSpmmTiles] = {
    {16, 16, kRoundsFraction, 0, 2.78, 0.295, 0.033},
    {32, 32, kRoundsWhole, 0, 1.47, 1.55, 0.071},
    {64, 64, kRoundsWhole, 0, 0.83, 3.16, 0.138},
    {128, 64, kRoundsWhole, 0, 0.17, 5.14, 0.197},
    {128, 128, kRoundsPairs, 2, 0.0, 4.2, 0.38},
    {128, 256, kRoundsWhole, 1, 0.0, 5.74, 0.524},
    {256, 256, kRoundsWhole, 1, 0.0, 8.08, 0.782},
};

// The index of the tile size with the least estimated time; -1 if none can be launched.
inline int spmm_choose(int64_t rows, int64_t cols, int64_t tokens, uint64_t cus)
{
    int best = -1;
    double best_us = 0.0;
    for (int v = 0; v < kSpmmTiles; v++) {
        const uint64_t n = kSpmmTile[v].tiles(rows, tokens);
        if (!kSpmmTile[v].launchable(n))
            continue;
        const double us = kSpmmTile[v].estimate(n, cols, cus);
        if (best < 0 || us < best_us) {
            best = v;
            best_us = us;
        }
    }
    return best;
}

}  // namespace tmask
