// tmask_exact for M = 8 or 16 in calls that leave the chip idle: a column of a block per lane.
//
// The kernel of tmask_exact_balance.hpp gives a lane four columns of a block, all work of a full chip at the fewest
// instructions a block; a call of a few hundred blocks takes as long with it as one wavefront does: 13 rounds of 540 instructions
// and a search at M = 16, 30 us.  Here M lanes hold a block from the loads to the mask, a quarter of the work each.  Lane j
// holds column j and the price of row j: the prices reach the keys by DPP (an operand of the addition), and the rows' sums come
// from a sum over lanes that halves the values at each step, so that lane j is left with row j's (33 instructions for
// sixteen sums over sixteen lanes).  A round takes 150 instructions at M = 16.  The lanes are already those of the searches: no
// collecting, no second reading of the weights.
#pragma once
#include "tmask_column.hpp"
#include "tmask_device.hpp"
#include "tmask_exact_balance.hpp"
#include "tmask_networks.hpp"
#include "tmask_solvers.hpp"

namespace tmask {

// v summed over the M lanes of a block, in every lane.
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

// x[0 .. 8) of sixteen lanes, summed over lanes l, l ^ 7 of each eight: banks (four lanes) 0, 2 keep values 0 ... 3, banks 1, 3
// values 4 ... 7.  Two additions for two values, each writing the banks that keep its sum.  (The waits: an operand that was just
// written cannot be read across lanes for two instructions, on either side of the block.)
__device__ __forceinline__ void halve8(const float (&x)[8], float (&y)[4])
{
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %4, %4 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %1, %5, %5 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %2, %6, %6 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %3, %7, %7 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %0, %8, %8 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %1, %9, %9 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %2, %10, %10 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %3, %11, %11 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "s_nop 1"
        : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3])
        : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]));
}

// The same for sixteen values: over lanes l, l ^ 8; lanes 0 ... 7 keep values 0 ... 7, the others 8 ... 15.
__device__ __forceinline__ void halve16(const float (&x)[16], float (&y)[8])
{
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %8, %8 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %9, %9 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %2, %10, %10 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %3, %11, %11 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %4, %12, %12 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %5, %13, %13 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %6, %14, %14 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %7, %15, %15 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %0, %16, %16 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %17, %17 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %18, %18 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %3, %19, %19 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %4, %20, %20 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %5, %21, %21 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %6, %22, %22 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %7, %23, %23 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "s_nop 1"
        : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3]), "=&v"(y[4]), "=&v"(y[5]), "=&v"(y[6]), "=&v"(y[7])
        : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]),
          "v"(x[8]), "v"(x[9]), "v"(x[10]), "v"(x[11]), "v"(x[12]), "v"(x[13]), "v"(x[14]), "v"(x[15]));
}

// x[i] summed over the M lanes of a block; lane j is left with the sum of x[j].
template <int M>
__device__ __forceinline__ float row_sums(const float (&x)[M])
{
    float z[4];
    if constexpr (M == 16) {
        float y[8];
        halve16(x, y);
        halve8(y, z);
    } else {
        halve8(x, z);
    }
    auto read = [](float v, auto ctrl) { return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), decltype(ctrl)::value, 0xF, 0xF, true)); };
    constexpr std::integral_constant<int, 0xB1> pair{};
    constexpr std::integral_constant<int, 0x4E> across{};
    const bool odd = threadIdx.x & 1u, upper = threadIdx.x & 2u;
    const float u0 = (odd ? z[1] : z[0]) + read(odd ? z[0] : z[1], pair);
    const float u1 = (odd ? z[3] : z[2]) + read(odd ? z[2] : z[3], pair);
    return (upper ? u1 : u0) + read(upper ? u0 : u1, across);
}

// exact_priced_start for a block in M lanes: cost = the costs of column j, x = its pruned rows, xrow = the pruned columns of row j;
// returns the excess.  The same rounds, sums in another order.
template <int M, bool GENERAL>
__device__ __forceinline__ uint32_t exact_spread_start(const float (&cost)[M], uint32_t j, uint32_t &xcol, uint32_t &xrow, uint32_t K)
{
    constexpr int H = M / 2;
    constexpr int S = exact_cost_bits(M);
    constexpr float kOffset = (float)(1 << S);
    using Sched = PriceSchedule<M>;
    const float own = row_sums<M>(cost);
    const float mean = over_lanes<M>(own) * (1.f / (M * M));
    const float dev = mean - own * (1.f / M);
    float spread = 0.f;
    {
        float level[M];
        each_of<M>([&](auto c) {
            constexpr int i = decltype(c)::value;
            level[i] = __uint_as_float(of_lane<M, i>(__float_as_uint(dev))) + cost[i];
        });
#pragma unroll
        for (int i = 0; i < H; i++)
            spread += __builtin_fabsf(level[i] - level[H + i]);
    }
    const PriceScale<M> scale(mean, over_lanes<M>(spread) * (2.f / (M * M)), over_lanes<M>(__builtin_fabsf(dev)));
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
        vel = __builtin_fmaf(kCarry, vel, row_sums<M>(f));
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
        const bool better = plain < e;
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
    constexpr int kWaves = NT / 64, NB = 64 / M;
    __shared__ int costs[kWaves][NB][M][M + 1];                   // of a wavefront's blocks, for their rows
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
    uint32_t xcol, xrow;
    {
        float column[M][1], cost[M];
        exact_costs<M, 1, M>(a, column);
#pragma unroll
        for (int i = 0; i < M; i++)
            cost[i] = column[i][0];
        const uint32_t e = exact_spread_start<M, GENERAL>(cost, j, xcol, xrow, K);
        if (__any(e != 0u)) {
            int ccol[M], crow[M];
#pragma unroll
            for (int i = 0; i < M; i++) {
                ccol[i] = (int)cost[i];
                costs[wave][blk][i][j] = ccol[i];
            }
            __builtin_amdgcn_wave_barrier();                     // LDS accesses of a wavefront happen in program order
            asm volatile("" ::: "memory");
#pragma unroll
            for (int c = 0; c < M; c++)
                crow[c] = costs[wave][blk][j][c];
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
