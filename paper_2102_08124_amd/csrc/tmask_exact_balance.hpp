// tmask_exact for M = 8 or 16: the start under row prices and the augmenting-path searches of tmask_solvers.hpp.
//
// The start is uniform work, every lane busy, and balances all but a few per cent of the blocks.  What is left is a
// serial chain of searches per block; a workgroup lasts as long as its longest.  So the unbalanced blocks are
// collected (by rank, deterministic), their costs and starts go to LDS, and every wavefront takes 64 / M of them at a
// time, M lanes to a block: a step of a search is then a few dozen instructions instead of the hundreds it takes where a
// lane holds four columns (with those, after a sort of the blocks by their excess, half of the kernel's time was one
// wavefront of each workgroup searching).  4096 x 4096 fp32, whole calls: 4:8 100 -> 49 us, 8:16 196 -> 89 us.  By copies
// that leave them out, the searches took 11 and 25 of that, the price rounds 14 and 37, and the load, the last choice, mask,
// objective and its second stage 24 and 27.  The vector ALU issues 97 % of the time, so instructions count: fewer of them in
// rounds, costs, mask bytes and kept sum took 4:8 from 48 to 44 us, and 8192 x 8192 fp32 4:8 / 8:16 from 138 / 252 to
// 131 / 236 us; searches that pass labels by DPP took 4096 x 4096 from 44 / 83 to 43 / 79 us and, both trees in turn,
// 8192 x 8192 from 135 / 239 to 131 / 231.
#pragma once
#include <type_traits>

#include "tmask_device.hpp"
#include "tmask_networks.hpp"
#include "tmask_solvers.hpp"

namespace tmask {

// Magnitude keys (fp32 bit patterns) of the C values a lane holds of one row: four dwords (fp32, or eight bf16),
// or two dwords (four bf16) where a lane takes half a 16-byte strip.
template <int DT, int C>
__device__ __forceinline__ void unpack_row(const u32x4 &r, uint32_t (&a)[C])
{
    const uint32_t d[4] = {r.x, r.y, r.z, r.w};
    if constexpr (DT == kF32) {
        static_assert(C == 4, "an fp32 lane holds four columns");
#pragma unroll
        for (int c = 0; c < 4; c++)
            a[c] = d[c] & 0x7FFFFFFFu;
    } else {
#pragma unroll
        for (int c = 0; c < C / 2; c++) {
            a[2 * c] = (d[c] << 16) & 0x7FFF0000u;
            a[2 * c + 1] = d[c] & 0x7FFF0000u;
        }
    }
}

// A bf16 lane takes half a strip, four columns, as an fp32 lane does (the host launches twice the workgroups): eight
// columns of a block and the prices' state do not fit a lane's registers.
constexpr bool exact_half_strips(int dt, int M) { return dt == kBF16 && M >= 8; }
// Workgroups per compute unit, which the registers are held to: 96 at M = 8 (no value of a lane in
// scratch memory, at bf16 with bit masks and any N four), 168 at M = 16 (none to two).
constexpr int exact_workgroups_per_cu(int dt, int M) { return M == 16 ? 3 : 5; }

// GENERAL: any N (K = args.K pruned per line); otherwise N = M/2.
template <int DT, int M, int FMT, bool GENERAL = false>
__global__ __launch_bounds__(kThreads, exact_workgroups_per_cu(DT, M)) void exact_balanced_kernel(const BatchArgs args)
{
    const uint32_t K = GENERAL ? args.K : (uint32_t)(M / 2);
    const uint32_t NKEEP = (uint32_t)M - K;
    using Ge = Geo<DT, M>;
    constexpr bool HALF = exact_half_strips(DT, M);
    constexpr int C = 4, G = M / 4;                               // columns per lane, lanes per block
    using Row = std::conditional_t<HALF, u32x2, u32x4>;           // the lane's part of a row as it lies in memory
    constexpr int kWaves = kThreads / 64;
    constexpr uint32_t SLOTS = kWaves * (64 / M);                 // blocks whose searches run at the same time
    __shared__ int slot_cost[SLOTS][M][M + 1];
    __shared__ uint32_t slot_x[SLOTS][M];                         // pruned rows of every column
    __shared__ SearchLds search_lds[kWaves];
    __shared__ uint32_t left[kWaves];                             // unbalanced blocks per wavefront: much to search, and little
    constexpr uint32_t kMuch = M / 4;
    __shared__ double red[kWaves];

    const uint32_t tile = blockIdx.x;
    const MatDev md = args.m[find_matrix(args, tile)];
    const Handover out = objective_of(args, md, tile);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t s = (tile - md.tile0) * kThreads + tid;
    const uint32_t gpos = tid & (G - 1);
    const bool valid = s < md.n_strips * (HALF ? 2u : 1u);      // s counts half strips if HALF

    // first byte of the lane's part of row 0 of its block
    const StripPos pos = strip_pos(md, HALF ? s >> 1 : s);
    const size_t col = (size_t)pos.sc * Ge::C + (HALF ? (s & 1u) * 4u : 0u);
    const char *const base = (const char *)md.w + ((size_t)pos.br * M * md.ld + col) * Ge::ES;
    const size_t row_bytes = (size_t)md.ld * Ge::ES;
    // Magnitudes of the lane's part of the block.  Lanes past the matrix' last strip take a filler block that any start
    // balances (a band of ones: entry (i, j) is 1 iff (i + j) mod M < N).
    auto load_block = [&](uint32_t (&a)[M][C]) {
        Row raw[M];
        if (valid) {
#pragma unroll
            for (int i = 0; i < M; i++)
                raw[i] = *(const Row *)(base + i * row_bytes);       // read again below: may stay in the cache
        }
#pragma unroll
        for (int i = 0; i < M; i++) {
            u32x4 r;
            if constexpr (HALF)
                r = u32x4{raw[i].x, raw[i].y, 0u, 0u};
            else
                r = raw[i];
            unpack_row<DT, C>(r, a[i]);
#pragma unroll
            for (int c = 0; c < C; c++)
                asm volatile("" : "+v"(a[i][c]));                // the raw rows end here
        }
        if (!valid) {                                            // hardly any wavefront: as selects, two instructions a weight
#pragma unroll
            for (int i = 0; i < M; i++)
#pragma unroll
                for (int c = 0; c < C; c++) {
                    a[i][c] = (((uint32_t)i + gpos * 4u + (uint32_t)c) & (M - 1)) < NKEEP ? 0x3F800000u : 0u;
                    asm volatile("" : "+v"(a[i][c]));
                }
        }
    };

    // ---- the start, and the rank of the block among those it leaves unbalanced ----
    uint32_t xcol[C];
    uint32_t e;
    {
        uint32_t a[M][C];
        float cost[M][C];
        load_block(a);
        exact_costs<M, C, G>(a, cost);
        e = exact_priced_start<M, C, G, GENERAL>(cost, gpos, xcol, K);
    }
    __builtin_amdgcn_sched_barrier(0);
    // a bit per unbalanced block, at its first lane; those with much to search come first, since the blocks of a wavefront wait
    // for the slowest (2048^2 fp32 4:8: three levels 65 -> 58 us, 50 % zeros 62 -> 51; random values take as long as before)
    const lanemask_t much = lm(gpos == 0 && e > kMuch), little = lm(gpos == 0 && e != 0u && e <= kMuch);
    if (lane == 0)
        left[wave] = (uint32_t)__builtin_popcountll(much) | (uint32_t)__builtin_popcountll(little) << 16;
    __syncthreads();
    const lanemask_t below = (1ull << (lane - gpos)) - 1ull;
    uint32_t rank = e > kMuch ? (uint32_t)__builtin_popcountll(much & below) : (uint32_t)__builtin_popcountll(little & below);
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w++) {
        before += (uint32_t)w < wave ? left[w] : 0u;
        all += left[w];
    }
    const uint32_t n_much = all & 0xFFFFu, n_open = n_much + (all >> 16);
    rank += e > kMuch ? before & 0xFFFFu : n_much + (before >> 16);

    // ---- searches, SLOTS blocks at a time ----
#pragma unroll 1
    for (uint32_t first = 0; first < n_open; first += SLOTS) {
        const uint32_t slot = rank - first;
        const bool mine = e != 0u && rank >= first && slot < SLOTS;
        if (mine) {
            uint32_t a[M][C];
            int cost[M][C];
            load_block(a);
            exact_costs<M, C, G>(a, cost);
#pragma unroll
            for (int c = 0; c < C; c++) {
#pragma unroll
                for (int i = 0; i < M; i++)
                    slot_cost[slot][i][gpos * C + c] = cost[i][c];
                slot_x[slot][gpos * C + c] = xcol[c];
            }
        }
        __syncthreads();
        const uint32_t q = wave * (64u / M) + lane / M, j = lane % M;
        if (first + wave * (64u / M) < n_open) {                 // this wavefront has a block
            const bool active = first + q < n_open;
            int ccol[M], crow[M];
            uint32_t x = active ? slot_x[q][j] : 0u, xrow = 0;
#pragma unroll
            for (int i = 0; i < M; i++) {
                ccol[i] = active ? slot_cost[q][i][j] : 0;
                crow[i] = active ? slot_cost[q][j][i] : 0;
                xrow |= ((active ? slot_x[q][i] : 0u) >> j & 1u) << i;
            }
            exact_search<M>(ccol, crow, x, xrow, active, K, search_lds[wave]);
            if (active)
                slot_x[q][j] = x;
        }
        __syncthreads();
        if (mine) {
#pragma unroll
            for (int c = 0; c < C; c++)
                xcol[c] = slot_x[slot][gpos * C + c];
        }
        __syncthreads();                                         // the slots may be filled again
    }

    // ---- mask and objective ----
    __builtin_amdgcn_sched_barrier(0);
    float acc = 0.f;
    if (valid) {
        // the kept entries of eight rows in a word, a column to a byte: row i's mask bytes are a shift and an AND (as bits put
        // together one by one and spread again they were ten instructions a row)
        uint32_t kept[M / 8];
        if constexpr (M == 8) {
            kept[0] = ~(xcol[0] | (xcol[1] << 8) | (xcol[2] << 16) | (xcol[3] << 24));
        } else {
            const uint32_t x01 = __builtin_amdgcn_perm(xcol[1], xcol[0], 0x05010400u), x23 = __builtin_amdgcn_perm(xcol[3], xcol[2], 0x05010400u);
            kept[0] = ~__builtin_amdgcn_perm(x23, x01, 0x05040100u);
            kept[1] = ~__builtin_amdgcn_perm(x23, x01, 0x07060302u);
        }
        char *mrow = (char *)md.mask + (size_t)pos.br * M * md.mask_ld + (FMT == kMaskU8 ? col : col >> 3);
#pragma unroll
        for (int i = 0; i < M; i++) {
            const uint32_t bytes = (kept[i / 8] >> (i % 8)) & 0x01010101u;
            if constexpr (FMT == kMaskU8) {
                stream_store(bytes, (uint32_t *)mrow);
            } else {                                             // a nibble, which the even lane of a pair completes
                const uint32_t bits = bytes4_to_bits(bytes), other = quad_xor<1>(bits);
                if ((s & 1u) == 0)
                    *mrow = (char)(bits | (other << 4));
            }
            mrow += md.mask_ld;
        }
        // the magnitudes are read again: they need not occupy registers in between
#pragma unroll
        for (int i = 0; i < M; i++) {
            const Row r = __builtin_nontemporal_load((const Row *)(base + i * row_bytes));
#pragma unroll
            for (int c = 0; c < C; c++) {
                const uint32_t w = DT == kF32 ? r[c] : (c & 1) ? r[c / 2] & 0xFFFF0000u : r[c / 2] << 16;
                const uint32_t pruned = (uint32_t)__builtin_amdgcn_sbfe((int)xcol[c], (uint32_t)i, 1u);     // all ones or none
                acc += __builtin_fabsf(__uint_as_float(w & ~pruned));
            }
        }
    }
    if (out.dst)
        hand_over<kThreads>(out, block_sum_f32(acc, red), red);
}

}  // namespace tmask
