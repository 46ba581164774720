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
    kRoundsPairs,        // two workgroups share a compute unit, each at half the speed: rounds count in halves
    kRoundsWhole
};

// What a product takes with tiles of rows x tokens, in microseconds:
//     fixed + rounds (per_round + per_store filled results + per_step steps) + shared full steps
// with filled = the share of the tiles' area that lies inside the matrix, results = 1 for bf16, 2 for fp32, steps =
// cols / 64, full = tiles per compute unit: per_step is what a compute unit needs by itself, shared what the whole chip's
// traffic from the caches adds.  The coefficients are a fit to 1448 timed products (rows 4 .. 2^20, cols 64 .. 16384, 1 ..
// 2^20 tokens, both types, every tile size): the choice is on average 0.1 % and at most 13 % slower than the fastest tile.
// Without the share of the area and the type (a fit to rows and cols of 256 .. 4096 and bf16 alone) thin products took small
// tiles: 1048576 x 64, 4 tokens 95 us on 16 x 16 tiles, 31 on 128 x 128; 16 x 64, 1048576 tokens 96 and 36.
// Small tiles win while they fill no more than a few rounds (W 4096 x 1024, 16 tokens: 3.2 us on 16 x 16 tiles, 16 on
// 256 x 256; 1024 x 4096, 1003 tokens: 15 us on 64 x 64 tiles, 58 on 256 x 256), large ones when there are many, because
// they move less (4096 x 1024, 8192 tokens: 51 us on 256 x 256, 64 on 128 x 128, 166 on 64 x 64).
struct SpmmTile {
    int64_t rows, tokens;
    SpmmRounds rounds_as;
    uint32_t persistent;                   // workgroups per compute unit that a launch has at most (0: one per tile)
    double fixed, per_round, per_store, per_step, shared;

    uint64_t tiles(int64_t r, int64_t t) const { return (uint64_t)((r + rows - 1) / rows) * (uint64_t)((t + tokens - 1) / tokens); }

    // Tile numbers have 31 bits, and a launch fewer than 2^32 work-items in a dimension: a workgroup per tile reaches that
    // at 2^24 tiles.
    bool launchable(uint64_t n) const { return n <= 0x7FFFFFFFull && (persistent || n * kSpmmThreads <= 0xFFFFFFFFull); }

    double estimate(uint64_t n, int64_t r, int64_t cols, int64_t t, double results, uint64_t cus) const
    {
        const double full = (double)n / (double)cus;
        double rounds = std::ceil(full);
        if (rounds_as == kRoundsFraction)
            rounds = full > 1.0 ? full : 1.0;
        else if (rounds_as == kRoundsPairs && full > 2.0)
            rounds = std::ceil(2.0 * full) / 2.0;
        const double filled = (double)r * (double)t / ((double)n * (double)(rows * tokens));
        const double steps = (double)(cols / kSpmmStep);
        return fixed + rounds * (per_round + per_store * filled * results + per_step * steps) + shared * full * steps;
    }
};

constexpr int kSpmmTiles = 7;
constexpr SpmmTile kSpmmTile[kSpmmTiles] = {
    {16, 16, kRoundsFraction, 0, 2.07, 0.284, 0.0, 0.037, 0.003},
    {32, 32, kRoundsWhole, 0, 1.587, 1.301, 0.03, 0.043, 0.038},
    {64, 64, kRoundsWhole, 0, 0.811, 2.382, 0.135, 0.114, 0.086},
    {128, 64, kRoundsWhole, 0, 0.937, 3.533, 0.196, 0.186, 0.145},
    {128, 128, kRoundsPairs, 2, 2.979, 0.362, 1.222, 0.239, 0.219},
    {128, 256, kRoundsWhole, 1, 2.874, 1.208, 2.431, 0.399, 0.436},
    {256, 256, kRoundsWhole, 1, 3.544, 1.44, 5.142, 0.561, 0.583},
};

// The index of the tile size with the least estimated time; -1 if none can be launched.
inline int spmm_choose(int64_t rows, int64_t cols, int64_t tokens, bool out_f32, uint64_t cus)
{
    int best = -1;
    double best_us = 0.0;
    for (int v = 0; v < kSpmmTiles; v++) {
        const uint64_t n = kSpmmTile[v].tiles(rows, tokens);
        if (!kSpmmTile[v].launchable(n))
            continue;
        const double us = kSpmmTile[v].estimate(n, rows, cols, tokens, out_f32 ? 2.0 : 1.0, cus);
        if (best < 0 || us < best_us) {
            best = v;
            best_us = us;
        }
    }
    return best;
}

}  // namespace tmask
