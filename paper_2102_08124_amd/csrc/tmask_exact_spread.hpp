// tmask_exact for M = 8 or 16 in calls that leave the chip idle: a column of a block per lane.
//
// The kernel of tmask_exact_balance.hpp gives a lane four columns of a block, all work of a full chip at the fewest
// instructions a block; a call of a few hundred blocks takes as long with it as one wavefront does: 13 rounds of 540 instructions
// and a search at M = 16, 30 us.  Here M lanes hold a block from the loads to the mask, a quarter of the work each.  Lane j
// holds column j and the price of row j: the prices reach the keys by DPP (an operand of the addition), and a round's columns reach the
// rows' lanes through LDS, sixteen dwords written and four times four read.  A round takes 150 instructions at M = 16.  The lanes are
// already those of the searches: no collecting, no second reading of the weights.
//
// Every sum is taken in the order of that kernel (four columns one after the other, then pairwise), and what a block's start and
// searches do depends on the block alone: both kernels return the same mask, bit for bit, whatever else is in the call.  (Sums over
// lanes that halve the values at each step are 33 instructions for sixteen rows and no LDS, but in another order; in this order, with
// transposes over four lanes, 63.  us, halving / transposes / LDS: fp32 8:16 464 x 128 15.4 / 16.1 / 16.1, 2048^2 30.6 / 33.2 / 30.3, 2048 x
// 2560 36.8 / 39.6 / 35.7; 4:8 128^2 8.8 / 9.2 / 9.2, 1024^2 11.6 / 12.3 / 11.5.)
#pragma once
#include "tmask_column.hpp"
#include "tmask_device.hpp"
#include "tmask_exact_balance.hpp"
#include "tmask_networks.hpp"
#include "tmask_solvers.hpp"

namespace tmask {

// v summed over the M lanes of a block, in every lane (integers below 2^24: in any order).
template <int M>
__device__ __forceinline__ float over_lanes(float v)
{
    v = quad_xor_sum<1>(v);
    v = quad_xor_sum<2>(v);
    v += __uint_as_float(dpp_read<kRowHalfMirror>(__float_as_uint(v)));
    if constexpr (M == 16)
        v += __uint_as_float(dpp_read<kRowRor8>(__float_as_uint(v)));
    return v;
}

// Lane I of the block's M.
template <int M, int I>
__device__ __forceinline__ float of_lane_f(float v) { return __uint_as_float(of_lane<M, I>(__float_as_uint(v))); }

// A block's values in LDS, row by row.  Rows are M + 4 dwords apart, so that sixteen lanes read four dwords of a row each from
// different banks, and blocks so that the lanes of a wavefront write a row of each to different ones (blocks without gaps: 4:8 1024^2
// 11.8 us against 11.5, 8:16 464 x 128 16.8 against 16.1).
template <int M>
struct SpreadBlocks {
    static constexpr int kPitch = M + 4, kBlock = M * kPitch;
    static constexpr int kDwords = M == 16 ? 4 * (kBlock + 16) : 4 * (2 * kBlock + 8);       // of a wavefront
    static constexpr __device__ uint32_t first(uint32_t blk) { return M == 16 ? blk * (kBlock + 16) : blk * kBlock + blk / 2u * 8u; }
};

// LDS accesses of a wavefront happen in program order.
__device__ __forceinline__ void lds_fence()
{
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// x[i] summed over the M lanes of a block; lane j is left with the sum of x[j].  Four columns one after the other, then these
// pairwise: the order of lanes that hold four columns.
template <int M>
__device__ __forceinline__ float row_sums(const float (&x)[M], uint32_t j, uint32_t *block)
{
    constexpr int P = SpreadBlocks<M>::kPitch;
#pragma unroll
    for (int i = 0; i < M; i++)
        block[i * P + j] = __float_as_uint(x[i]);
    lds_fence();
    float z[M / 4];
#pragma unroll
    for (int q = 0; q < M / 4; q++) {
        const u32x4 r = *(const u32x4 *)&block[j * P + 4 * q];
        z[q] = ((__uint_as_float(r.x) + __uint_as_float(r.y)) + __uint_as_float(r.z)) + __uint_as_float(r.w);
    }
    lds_fence();
    if constexpr (M == 16)
        return (z[0] + z[1]) + (z[2] + z[3]);
    else
        return z[0] + z[1];
}

// exact_priced_start for a block in M lanes: cost = the costs of column j, x = its pruned rows, xrow = the pruned columns of row j;
// returns the excess.
template <int M, bool GENERAL>
__device__ __forceinline__ uint32_t exact_spread_start(const float (&cost)[M], uint32_t j, uint32_t &xcol, uint32_t &xrow, uint32_t K,
                                                       uint32_t *block)
{
    constexpr int H = M / 2;
    constexpr int S = exact_cost_bits(M);
    constexpr float kOffset = (float)(1 << S);
    using Sched = PriceSchedule<M>;
    const float own = row_sums<M>(cost, j, block);
    float mean = 0.f, row_dev = 0.f, spread = 0.f;
    each_of<M>([&](auto c) { mean += of_lane_f<M, decltype(c)::value>(own); });
    mean = mean * (1.f / (M * M));
    const float dev = mean - own * (1.f / M);
    each_of<M>([&](auto c) { row_dev += __builtin_fabsf(of_lane_f<M, decltype(c)::value>(dev)); });
    each_of<H>([&](auto c) {
        constexpr int i = decltype(c)::value;
        const float rows = of_lane_f<M, i>(dev) - of_lane_f<M, H + i>(dev);
        const float apart = __builtin_fabsf((cost[i] - cost[H + i]) + rows);
        each_of<4>([&](auto lane) { spread += __uint_as_float(dpp_read<0x55 * decltype(lane)::value>(__float_as_uint(apart))); });
    });
    spread += __uint_as_float(dpp_read<kRowHalfMirror>(__float_as_uint(spread)));
    if constexpr (M == 16)
        spread += __uint_as_float(dpp_read<kRowRor8>(__float_as_uint(spread)));
    const PriceScale<M> scale(mean, spread * (2.f / (M * M)), row_dev);
    float price = kOffset + scale.part * dev, vel = 0.f;
    float slope = scale.slope, step = scale.step;
    float drift = 0.f, dvel = 0.f;
    constexpr float kCarry = Sched::momentum / Sched::step_next;
#pragma unroll 1
    for (int round = 0; round < Sched::rounds; round++) {
        uint32_t k[M];
        each_of<M>([&](auto c) {
            constexpr int i = decltype(c)::value;
            k[i] = __float_as_uint(__uint_as_float(of_lane<M, i>(__float_as_uint(price))) + cost[i]);
        });
        float f[M];
        price_window<M, GENERAL>(k, slope, K, f);
        vel = __builtin_fmaf(kCarry, vel, row_sums<M>(f, j, block));
        price = __builtin_fmaf(step, vel, price);
        dvel = __builtin_fmaf(kCarry, dvel, (float)K);
        drift = __builtin_fmaf(step, dvel, drift);
        slope *= 1.f / Sched::window_next;
        step *= Sched::step_next;
    }

    constexpr int PMIN = 1, PMAX = (1 << S) - 1;
    const float p = price - drift - (kOffset - (float)(1 << (S - 1)));
    const uint32_t prices[2] = {1u << (S - 1), (uint32_t)(int)__builtin_amdgcn_fmed3f(p, (float)PMIN, (float)(PMAX - 64))};
    auto choose = [&](uint32_t own_price, uint32_t &x, uint32_t &xr) -> uint32_t {
        uint32_t k[M];
        each_of<M>([&](auto c) {
            constexpr int i = decltype(c)::value;
            k[i] = (((uint32_t)(int)cost[i] + of_lane<M, i>(own_price)) << 4) | (((uint32_t)i - j) & (uint32_t)(M - 1));
        });
        uint32_t t;
        {
            uint32_t srt[M];
#pragma unroll
            for (int i = 0; i < M; i++)
                srt[i] = k[i];
            if constexpr (GENERAL) {
                sort_asc<M>(srt);
                t = srt[K & (uint32_t)(M - 1)];
            } else {
                uint32_t lo[H], hi[H];
#pragma unroll
                for (int i = 0; i < H; i++) {
                    lo[i] = srt[i];
                    hi[i] = srt[H + i];
                }
                t = upper_half_min<H>(lo, hi);
            }
        }
        x = 0u;
#pragma unroll
        for (int i = M - 1; i >= 0; i--)
            lm_shift_in(x, lm(k[i] < t));
        xr = transposed_bits<M>(x);
        const uint32_t n = (uint32_t)__builtin_popcount(xr);
        return (uint32_t)over_lanes<M>((float)(n > K ? n - K : 0u));
    };
    uint32_t e = choose(prices[1], xcol, xrow);
    if (__any(e > 2u)) {
        uint32_t x, xr;
        const uint32_t plain = choose(prices[0], x, xr);
        const bool better = plain < e && e > 2u;                 // a block's own excess decides, not its neighbours'
        e = better ? plain : e;
        xcol = better ? x : xcol;
        xrow = better ? xr : xrow;
    }
    return e;
}

// GENERAL: any N (K = args.K pruned per line); otherwise N = M/2.
template <int DT, int M, int FMT, bool GENERAL, typename Args, int NT = kThreads>
__global__ __launch_bounds__(NT, NT > kThreads ? 6 : 4) void exact_spread_kernel(const Args args)
{
    using Ge = Geo<DT, M>;
    constexpr int kWaves = NT / 64;
    constexpr int P = SpreadBlocks<M>::kPitch;
    __shared__ __attribute__((aligned(16))) uint32_t blocks[kWaves][SpreadBlocks<M>::kDwords];
    __shared__ SearchLds search_lds[kWaves];
    __shared__ double red[kWaves];
    const uint32_t K = GENERAL ? args.K : (uint32_t)(M / 2);

    const uint32_t tile = blockIdx.x;
    const MatDev md = args.m[find_matrix(args, tile)];
    const Handover out = objective_of(args, md, tile);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, j = lane % M, blk = lane / M;
    const ColumnPos pos = column_pos<Ge::C>(md, (tile - md.tile0) * NT + tid);
    const bool valid = pos.valid;
    const size_t col = pos.col;

    // Lanes past the matrix' last column hold a filler block that any start balances (see exact_balanced_kernel).
    uint32_t a[M][1];
    if (valid) {
        const char *base = (const char *)md.w + ((size_t)pos.br * M * md.ld + col) * Ge::ES;
        const size_t row_bytes = (size_t)md.ld * Ge::ES;
#pragma unroll
        for (int i = 0; i < M; i++) {
            if constexpr (DT == kF32)
                a[i][0] = __builtin_nontemporal_load((const uint32_t *)(base + i * row_bytes)) & 0x7FFFFFFFu;
            else
                a[i][0] = (uint32_t)(__builtin_nontemporal_load((const uint16_t *)(base + i * row_bytes)) & 0x7FFFu) << 16;
        }
    } else {
#pragma unroll
        for (int i = 0; i < M; i++)
            a[i][0] = (((uint32_t)i + j) & (uint32_t)(M - 1)) < (uint32_t)M - K ? 0x3F800000u : 0u;
    }
    uint32_t *const block = &blocks[wave][SpreadBlocks<M>::first(blk)];
    uint32_t xcol, xrow;
    {
        float column[M][1], cost[M];
        exact_costs<M, 1, M>(a, column);
#pragma unroll
        for (int i = 0; i < M; i++)
            cost[i] = column[i][0];
        const uint32_t e = exact_spread_start<M, GENERAL>(cost, j, xcol, xrow, K, block);
        if (__any(e != 0u)) {
            int ccol[M], crow[M];
#pragma unroll
            for (int i = 0; i < M; i++) {
                ccol[i] = (int)cost[i];
                block[i * P + j] = (uint32_t)ccol[i];
            }
            lds_fence();
#pragma unroll
            for (int c = 0; c < M; c++)
                crow[c] = (int)block[j * P + c];
            exact_search<M>(ccol, crow, xcol, xrow, true, K, search_lds[wave]);
        }
    }

    const uint32_t kept = ~xcol;
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < M; i++)
        acc += (kept >> i) & 1u ? __uint_as_float(a[i][0]) : 0.f;
    store_column<M, FMT>(md, pos, kept);
    if (out.dst)
        hand_over<NT>(out, block_sum_f32<kF32, NT>(valid ? acc : 0.f, red), red);
}

}  // namespace tmask
