// tmask: streaming kernels (approx / exact / score) and the C ABI.  gfx950 only.
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

#include "../../include/tmask.h"
#include "tmask_device.hpp"
#include "tmask_host.hpp"
#include "tmask_solvers.hpp"
#include "tmask_approx4.hpp"
#include "tmask_approx_sel.hpp"
#include "tmask_approx_spread.hpp"
#include "tmask_pack.hpp"
#include "tmask_pack4.hpp"
#include "tmask_pack8.hpp"
#include "tmask_exact_balance.hpp"
#include "tmask_exact_spread.hpp"
#include "tmask_fused4.hpp"

namespace tmask {

// =================================================================================================
// Kernels
// =================================================================================================

enum { kSolveApprox = 0, kSolveExact = 1, kSolveRow1D = 2 };

// One workgroup = 256 consecutive strips of one matrix: load M rows x 16 B per lane, solve the
// block(s) in registers, write the mask, leave one partial objective per workgroup.
template <int SOLVER, int DT, int M, int FMT>
__global__ __launch_bounds__(kThreads) void mask_kernel(const BatchArgs args)
{
    using Ge = Geo<DT, M>;
    __shared__ double red[kThreads / 64];
    const uint32_t tile = blockIdx.x;
    const MatDev md = args.m[find_matrix(args, tile)];
    const Handover out = objective_of(args, md, tile);
    const uint32_t s = (tile - md.tile0) * kThreads + threadIdx.x;
    const uint32_t gpos = threadIdx.x & (Ge::G - 1);
    float acc = 0.f;
    if (s < md.n_strips) {
        const StripPos pos = strip_pos(md, s);
        uint32_t a[M][Ge::C];
        u32x4 raw[M];
        uint32_t bits[M];
        load_strip<DT, M>(md, pos, a, raw);
        static_assert(SOLVER == kSolveApprox || SOLVER == kSolveRow1D, "the exact solvers have kernels of their own");
        if constexpr (SOLVER == kSolveApprox) {
            approx_keep<DT, M>(a, args.K, gpos, bits);
        } else {
            // structured N:M along rows only: an entry is kept iff at least K entries of its group of M
            // precede it in the (magnitude, position) order
            bool done = false;
            if constexpr (DT == kBF16 && M >= 8) {
                if (2u * args.K == (uint32_t)M) {      // N = M/2: thresholds on unique keys instead of pairwise ranks
                    row_half_keep_bf16<M>(raw, gpos, bits);
                    done = true;
                } else if constexpr (M == 8) {         // any N: the sorted row group read at index K
                    row_half_keep_bf16<M, true>(raw, gpos, bits, args.K);
                    done = true;
                }
            }
            if constexpr (DT == kF32 && M == 16) {
                // N = M/2: thresholds on magnitudes (8192^2 8:16: 89 -> 63 us); a wavefront with a cut among equal
                // values falls through to the ranks.  At M = 8 the ranks already run at the speed of the memory.
                if (2u * args.K == (uint32_t)M)
                    done = !__any(row_half_keep_f32<M>(a, gpos, bits));
            }
            if (!done) {
#pragma unroll
                for (int i = 0; i < M; i++)
                    bits[i] = (1u << Ge::C) - 1u;
                row_rank_keep<M, Ge::C, Ge::G, Ge::B, (M >= 16 && FMT == kMaskBits)>(a, args.K, gpos, bits);
            }
        }
        store_mask<DT, M, FMT>(md, pos, bits);
        acc = kept_sum<M, Ge::C>(a, bits);
    }
    if (out.dst)
        hand_over<kThreads>(out, block_sum_f32<DT>(acc, red), red);
}

// A strip of tmask_approx for 2:4, decisions taken as lane-mask logic; returns what the lane keeps.
template <int DT, int FMT>
__device__ __forceinline__ float approx24_strip(const MatDev &md, uint32_t s)
{
    const StripPos pos = strip_pos(md, s);
    uint32_t a[4][Geo<DT, 4>::C];
    u32x4 raw[4];
    load_strip<DT, 4>(md, pos, a, raw);
    return approx_2of4_strip<DT, FMT>(md, pos, a);
}

// tmask_approx for 2:4: same tiling as mask_kernel.
template <int DT, int FMT, typename Args>
__global__ __launch_bounds__(kThreads) void approx24_kernel(const Args args)
{
    __shared__ double red[kThreads / 64];
    const uint32_t tile = blockIdx.x;
    const MatDev md = args.m[find_matrix(args, tile)];
    const Handover out = objective_of(args, md, tile);
    const uint32_t s = (tile - md.tile0) * kThreads + threadIdx.x;
    float acc = 0.f;
    if (s < md.n_strips)
        acc = approx24_strip<DT, FMT>(md, s);
    if (out.dst)
        hand_over<kThreads>(out, block_sum_f32<DT>(acc, red), red);
}

// tmask_approx for fp32 with N = M/2, M = 8 or 16: thresholds on magnitudes; a wavefront in which some
// line has a tie across its cut redoes its strips with the form that resolves ties by position (uniform branch).
// GENERAL: any N, thresholds read from the sorted line; at M = 8 ties send the wavefront to the rank form, at M = 16 each line settles its own.
template <int M, int FMT, bool GENERAL, typename Args>
__global__ __launch_bounds__(kThreads, (M == 16 && FMT == kMaskBits) ? 4 : 1) void approx_sel_f32_kernel(const Args args)
{
    using Ge = Geo<kF32, M>;
    __shared__ double red[kThreads / 64];
    const uint32_t tile = blockIdx.x;
    const MatDev md = args.m[find_matrix(args, tile)];
    const Handover out = objective_of(args, md, tile);
    const uint32_t s = (tile - md.tile0) * kThreads + threadIdx.x;
    const uint32_t gpos = threadIdx.x & (Ge::G - 1);
    float acc = 0.f;
    if (s < md.n_strips) {
        const StripPos pos = strip_pos(md, s);
        uint32_t a[M][4];
        u32x4 raw[M];
        load_strip<kF32, M>(md, pos, a, raw);
        uint32_t rowbytes[M];
        bool tie = false;
        if constexpr (M == 16 && GENERAL)
            approx16_f32_by_lines(raw, gpos, args.K, rowbytes, acc);
        else
            tie = approx_half_f32<M, GENERAL>(a, gpos, rowbytes, acc, args.K);
        uint32_t bits[M];
        // Some cut among equal values (a matrix full of zeros, say).  M = 8: the form that sorts them out by position
        // (8192^2 with 90 % zeros: 80 -> 60 us).  M = 16 at N = 8: the rank form; the other one takes the kernel from 119 to
        // 154-209 registers whichever way it is attached, which costs the common case more (60 -> 69 us) than it
        // saves here (165 -> 118 us).
        bool stored = false;
        if (__any(tie)) {
            if constexpr (M == 8 && !GENERAL) {
                approx_half_f32_ties<M>(a, gpos, rowbytes, acc);
            } else if constexpr (M == 8 || !GENERAL) {
                approx_keep<kF32, M, (M >= 16 && FMT == kMaskBits)>(a, args.K, gpos, bits);
                acc = kept_sum<M, 4>(a, bits);
                if constexpr (FMT == kMaskU8)
                    store_mask<kF32, M, FMT>(md, pos, bits);
                stored = true;
            }
        }
        if constexpr (FMT == kMaskU8) {
            if (!stored) {
                char *mb = (char *)md.mask + (size_t)pos.br * M * md.mask_ld + (size_t)pos.sc * 4;
#pragma unroll
                for (int i = 0; i < M; i++)
                    stream_store(rowbytes[i], (uint32_t *)(mb + (size_t)i * md.mask_ld));
            }
        } else {
            // bit masks leave through one place (the cross-lane assembly of a row's bytes is long code: twice it cost
            // the M = 16 kernel a wavefront of occupancy)
            if (!stored) {
#pragma unroll
                for (int i = 0; i < M; i++)
                    bits[i] = bytes4_to_bits(rowbytes[i]);
            }
            store_mask<kF32, M, kMaskBits>(md, pos, bits);
        }
    }
    if (out.dst)
        hand_over<kThreads>(out, block_sum_f32(acc, red), red);
}

// A strip of tmask_exact at M = 4: every block by enumeration (NK = 2: all 90 patterns; NK = 1, 3: the 24 permutations,
// kept resp. pruned), the kept sum comes with the optimum.
template <int DT, int FMT, int NK>
__device__ __forceinline__ float exact24_strip(const MatDev &md, uint32_t s)
{
    using Ge = Geo<DT, 4>;
    const StripPos pos = strip_pos(md, s);
    uint32_t a[4][Ge::C];
    u32x4 raw[4];
    uint32_t bits[4] = {0u, 0u, 0u, 0u};
    load_strip<DT, 4>(md, pos, a, raw);
    float sum = 0.f;
#pragma unroll
    for (int b = 0; b < Ge::B; b++) {
        float v[4][4];
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int c = 0; c < 4; c++)
                v[i][c] = __uint_as_float(a[i][b * 4 + c]);
        float best;
        uint32_t m16;
        if constexpr (NK == 2) {
            m16 = exact24_block(v, best);
        } else if constexpr (NK == 1) {
            m16 = best_permutation4<true>(v, best);
        } else {
            m16 = ~best_permutation4<false>(v, best) & 0xFFFFu;
            float all = 0.f;
#pragma unroll
            for (int i = 0; i < 4; i++)
                all += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
            best = all - best;
        }
        sum += best;
#pragma unroll
        for (int i = 0; i < 4; i++)
            bits[i] |= ((m16 >> (4 * i)) & 0xFu) << (4 * b);
    }
    store_mask<DT, 4, FMT>(md, pos, bits);
    return sum;
}

template <int DT, int FMT, int NK, typename Args>
__global__ __launch_bounds__(kThreads) void exact24_kernel(const Args args)
{
    __shared__ double red[kThreads / 64];
    const uint32_t tile = blockIdx.x;
    const MatDev md = args.m[find_matrix(args, tile)];
    const Handover out = objective_of(args, md, tile);
    const uint32_t s = (tile - md.tile0) * kThreads + threadIdx.x;
    float acc = 0.f;
    if (s < md.n_strips)
        acc = exact24_strip<DT, FMT, NK>(md, s);
    if (out.dst)
        hand_over<kThreads>(out, block_sum_f32<DT>(acc, red), red);
}

// A few small matrices with their objectives, 2:4: a workgroup of 1024 threads takes a whole matrix, a strip per thread, and
// writes its objective itself, so that the call is one launch instead of two, and one with 1.8 KB of arguments instead of
// 16.  Such a call is bound by its launches (each 2.3 us of host time, 1.2 more for the large arguments) and by the few
// microseconds that a kernel lasts at least.  Back to back / in a graph, 1 ... 32 matrices of 1024 strips: fp32 8.2 - 9.3 / 4.5 -
// 5.4 -> 4.9 - 5.3 / 3.3 - 3.9 us, bf16 8.2 - 9.2 / 5.2 - 6.2 -> 4.8 - 5.4 / 4.6 - 5.3.  Two strips per thread are as slow as two
// launches in a graph (fp32 5.3 against 4.8 us, bf16 8.4 against 5.3): one compute unit then moves all of it in two goes.
constexpr int kWholeThreads = 1024, kWholeMats = 32;

struct WholeArgs {
    MatDev m[kWholeMats];     // aux: the objective (or null)
};

template <int SOLVER, int DT, int FMT>
__global__ __launch_bounds__(kWholeThreads) void whole24_kernel(const WholeArgs args)
{
    __shared__ double red[kWholeThreads / 64];
    const MatDev md = args.m[blockIdx.x];
    float acc = 0.f;
    if (threadIdx.x < md.n_strips)
        acc = SOLVER == kSolveApprox ? approx24_strip<DT, FMT>(md, threadIdx.x) : exact24_strip<DT, FMT, 2>(md, threadIdx.x);
    const double sum = wave_kept<DT>(acc);
    if ((threadIdx.x & 63u) == 0)
        red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0 && md.aux) {
        double total = red[0];
#pragma unroll
        for (int k = 1; k < kWholeThreads / 64; k++)
            total += red[k];
        *(double *)md.aux = total;
    }
}

// tmask_approx for bf16 with N = M/2, M = 8 or 16: thresholds from min/max networks on unique keys.  GENERAL: any N,
// the threshold read from the sorted line at index K = M - N (8192^2 3:8: 40 us; 63 us in the rank form).
template <int M, int FMT, bool GENERAL, typename Args>
__global__ __launch_bounds__(kThreads) void approx_sel_bf16_kernel(const Args args)
{
    using Ge = Geo<kBF16, M>;
    __shared__ double red[kThreads / 64];
    const uint32_t tile = blockIdx.x;
    const MatDev md = args.m[find_matrix(args, tile)];
    const Handover out = objective_of(args, md, tile);
    const uint32_t s = (tile - md.tile0) * kThreads + threadIdx.x;
    const uint32_t gpos = threadIdx.x & (Ge::G - 1);
    float acc = 0.f;
    if (s < md.n_strips) {
        const StripPos pos = strip_pos(md, s);
        u32x4 raw[M];
        const char *base = (const char *)md.w + ((size_t)pos.br * M * md.ld + (size_t)pos.sc * 8) * 2;
        const size_t row_bytes = (size_t)md.ld * 2;
#pragma unroll
        for (int i = 0; i < M; i++)
            raw[i] = __builtin_nontemporal_load((const u32x4 *)(base + i * row_bytes));
        if constexpr (FMT == kMaskU8) {
            char *mb = (char *)md.mask + (size_t)pos.br * M * md.mask_ld + (size_t)pos.sc * 8;
            const uint32_t mld = md.mask_ld;
            acc = approx_half_bf16<M, GENERAL>(raw, gpos, [&](int i, uint32_t b0, uint32_t b1) {
                u32x2 v;
                v.x = b0;
                v.y = b1;
                stream_store(v, (u32x2 *)(mb + (size_t)i * mld));
            }, args.K);
        } else {
            uint32_t bits[M];
            acc = approx_half_bf16<M, GENERAL>(raw, gpos, [&](int i, uint32_t b0, uint32_t b1) {
                bits[i] = bytes4_to_bits(b0) | (bytes4_to_bits(b1) << 4);
            }, args.K);
            store_mask<kBF16, M, kMaskBits>(md, pos, bits);
        }
    }
    if (out.dst)
        hand_over<kThreads>(out, block_sum_f32(acc, red), red);
}

// tmask_approx_dense / tmask_prune_1d_dense: a mask and the masked copy W (.) S in one pass.  Same tiling as the
// kernels above; the keep flags come from the same routines.  MODE: kDenseApprox = Algorithm 1 for any N (fp32 at M = 16: every line
// in a lane; bf16 at M = 8, 16: thresholds on unique keys; else the rank form), kDenseApproxHalf = Algorithm 1 at N = M/2 (the lane-mask form at M = 4, the threshold networks at M = 8, 16),
// kDenseRow1D = N:M pruning along rows, kDenseRow1DAbsorb = the same with the mean of every row group's pruned
// weights added to its kept ones (Sec. 5; fp32 sums inside the lane in position order, then across the lanes of the
// group pairwise; bf16 results rounded to nearest even).  md.aux = the output matrix, md.pad = its leading dimension
// in elements; the mask is written only if md.mask is not NULL.
// kDenseRow1DHalf / kDenseRow1DHalfAbsorb: the row modes at N = M/2 for bf16 with M = 8, 16, where the row rule is a
// threshold on unique keys (row_half_keep_bf16) and only the raw rows need registers.
enum { kDenseApprox = 0, kDenseApproxHalf = 1, kDenseRow1D = 2, kDenseRow1DAbsorb = 3, kDenseRow1DHalf = 4, kDenseRow1DHalfAbsorb = 5 };

template <int DT, int M, int FMT, int MODE, typename Args>
__global__ __launch_bounds__(kThreads) void approx_dense_kernel(const Args args)
{
    constexpr bool HALFN = MODE == kDenseApproxHalf;
    constexpr bool ROWHALF = MODE == kDenseRow1DHalf || MODE == kDenseRow1DHalfAbsorb;
    constexpr bool ABSORB = MODE == kDenseRow1DAbsorb || MODE == kDenseRow1DHalfAbsorb;
    static_assert(!ROWHALF || (DT == kBF16 && M >= 8), "the threshold form of the row rule exists for bf16, M = 8, 16");
    using Ge = Geo<DT, M>;
    constexpr int C = Ge::C, ES = Ge::ES;
    const uint32_t tile = blockIdx.x;
    const MatDev md = args.m[find_matrix(args, tile)];
    const uint32_t s = (tile - md.tile0) * kThreads + threadIdx.x;
    const uint32_t gpos = threadIdx.x & (Ge::G - 1);
    if (s >= md.n_strips)
        return;
    const StripPos pos = strip_pos(md, s);
    uint32_t bits[M];                  // bit c = column c of the lane's strip kept
    u32x4 raw[M];
    constexpr bool GEN8 = MODE == kDenseApprox && DT == kBF16 && M >= 8;   // any N at bf16 M = 8, 16: threshold form too
    if constexpr ((HALFN || ROWHALF || GEN8) && DT == kBF16 && M >= 8) {
        const char *base = (const char *)md.w + ((size_t)pos.br * M * md.ld + (size_t)pos.sc * 8) * 2;
        const size_t row_bytes = (size_t)md.ld * 2;
#pragma unroll
        for (int i = 0; i < M; i++)
            raw[i] = __builtin_nontemporal_load((const u32x4 *)(base + i * row_bytes));
        if constexpr (HALFN || GEN8) {
            (void)approx_half_bf16<M, GEN8>(raw, gpos, [&](int i, uint32_t b0, uint32_t b1) {
                bits[i] = bytes4_to_bits(b0) | (bytes4_to_bits(b1) << 4);
            }, args.K);
        } else {
            row_half_keep_bf16<M>(raw, gpos, bits);
        }
    } else {
        uint32_t a[M][C];
        load_strip<DT, M>(md, pos, a, raw);
        if constexpr (HALFN && M == 4) {
#pragma unroll
            for (int i = 0; i < 4; i++)
                bits[i] = 0;
#pragma unroll
            for (int b = 0; b < C / 4; b++) {
                uint32_t k[4][4], bytes[4];
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int c = 0; c < 4; c++)
                        k[i][c] = a[i][4 * b + c];
                (void)approx_2of4_block(k, bytes);
#pragma unroll
                for (int i = 0; i < 4; i++)
                    bits[i] |= bytes4_to_bits(bytes[i]) << (4 * b);
            }
        } else if constexpr (MODE == kDenseApprox && DT == kF32 && M == 16) {
            uint32_t rowbytes[M];
            float unused;
            approx16_f32_by_lines(raw, gpos, args.K, rowbytes, unused);
#pragma unroll
            for (int i = 0; i < M; i++) {
                bits[i] = bytes4_to_bits(rowbytes[i]);
                asm volatile("" : "+v"(bits[i]));                // else the masked weights are made here and held through the mask's stores
            }
        } else if constexpr (HALFN && DT == kF32 && M >= 8) {
            uint32_t rowbytes[M];
            float unused = 0.f;
            const bool tie = approx_half_f32<M>(a, gpos, rowbytes, unused);
            if (__any(tie)) {
                if constexpr (M == 8)
                    approx_half_f32_ties<M>(a, gpos, rowbytes, unused);
                else
                    approx_keep<kF32, M, false>(a, (uint32_t)(M / 2), gpos, bits);
            }
            if (M == 8 || !__any(tie)) {
#pragma unroll
                for (int i = 0; i < M; i++)
                    bits[i] = bytes4_to_bits(rowbytes[i]);
            }
        } else if constexpr (MODE == kDenseRow1D || MODE == kDenseRow1DAbsorb) {
            bool done = false;
            if constexpr (DT == kF32 && M == 16) {
                if (2u * args.K == (uint32_t)M)
                    done = !__any(row_half_keep_f32<M>(a, gpos, bits));
            }
            if (!done) {
#pragma unroll
                for (int i = 0; i < M; i++)
                    bits[i] = (1u << C) - 1u;
                row_rank_keep<M, C, Ge::G, Ge::B, false>(a, args.K, gpos, bits);
            }
        } else {
            approx_keep<DT, M, false>(a, args.K, gpos, bits);
        }
    }
    if (md.mask)
        store_mask<DT, M, FMT>(md, pos, bits);
    char *ob = (char *)md.aux + ((size_t)pos.br * M * md.pad + (size_t)pos.sc * C) * ES;
    const size_t out_row_bytes = (size_t)md.pad * ES;
#pragma unroll
    for (int i = 0; i < M; i++) {
        uint32_t d[4] = {raw[i].x, raw[i].y, raw[i].z, raw[i].w};
        if constexpr (ABSORB) {
            constexpr int S = M < C ? M : C;          // entries of one row group inside the lane
            float v[C];
            if constexpr (DT == kF32) {
#pragma unroll
                for (int c = 0; c < 4; c++)
                    v[c] = __uint_as_float(d[c]);
            } else {
#pragma unroll
                for (int c = 0; c < C / 2; c++) {
                    v[2 * c] = __uint_as_float(d[c] << 16);
                    v[2 * c + 1] = __uint_as_float(d[c] & 0xFFFF0000u);
                }
            }
#pragma unroll
            for (int g = 0; g < C / S; g++) {
                float ps = 0.f;
                uint32_t pc = 0;
#pragma unroll
                for (int c = g * S; c < (g + 1) * S; c++) {
                    const bool k = (bits[i] >> c) & 1u;
                    ps += k ? 0.f : v[c];
                    pc += k ? 0u : 1u;
                }
                if constexpr (Ge::G >= 2) {
                    ps += __uint_as_float(quad_xor<1>(__float_as_uint(ps)));
                    pc += quad_xor<1>(pc);
                }
                if constexpr (Ge::G == 4) {
                    ps += __uint_as_float(quad_xor<2>(__float_as_uint(ps)));
                    pc += quad_xor<2>(pc);
                }
                const float mean = (pc != 0u && pc != (uint32_t)M) ? ps / (float)pc : 0.f;
#pragma unroll
                for (int c = g * S; c < (g + 1) * S; c++)
                    v[c] = ((bits[i] >> c) & 1u) ? v[c] + mean : 0.f;
            }
            if constexpr (DT == kF32) {
#pragma unroll
                for (int c = 0; c < 4; c++)
                    d[c] = __float_as_uint(v[c]);
            } else {
                typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                typedef float f32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
                for (int c = 0; c < C / 2; c++) {
                    union { bf16x2 h; uint32_t w; } cv;
                    cv.h = __builtin_convertvector(f32x2{v[2 * c], v[2 * c + 1]}, bf16x2);   // round to nearest even
                    d[c] = cv.w;
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < C * ES / 4; q++) {
                if constexpr (DT == kF32)
                    d[q] &= 0u - ((bits[i] >> q) & 1u);
                else
                    d[q] &= ((0u - ((bits[i] >> (2 * q)) & 1u)) & 0xFFFFu) | ((0u - ((bits[i] >> (2 * q + 1)) & 1u)) << 16);
            }
        }
        if constexpr (DT == kBF16N)
            stream_store(u32x2{d[0], d[1]}, (u32x2 *)(ob + i * out_row_bytes));
        else
            stream_store(u32x4{d[0], d[1], d[2], d[3]}, (u32x4 *)(ob + i * out_row_bytes));
    }
}

struct ReduceArgs {
    double *objective[kMaxBatch];
    uint32_t tile0[kMaxBatch + 1];
    uint32_t n_mats;
    uint32_t partial0;
    const double *partials;
};

// Second stage of the objective: workgroup m adds the partials of matrix m in a fixed order.  1024 threads: one
// matrix can have hundreds of thousands of partials, and the loop is a chain of load latencies.
constexpr int kReduceThreads = 1024;
constexpr int kReduceThreadsSmall = 256;    // when no matrix of the launch has more than 2048 partial results

template <int THREADS>
__global__ __launch_bounds__(THREADS) void objective_reduce_kernel(const ReduceArgs args)
{
    constexpr int kReduceThreads = THREADS;           // shadows the file-scope constant inside this kernel
    __shared__ double red[kReduceThreads / 64];
    const uint32_t m = blockIdx.x;
    double *dst = args.objective[m];
    if (!dst)
        return;
    // several loads of a thread are in flight; the order of additions is fixed: with 256 threads that of hand_over, with 1024
    // four sums side by side
    const uint32_t t0 = args.tile0[m], t1 = args.tile0[m + 1];
    const double *src = args.partials + args.partial0;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    uint32_t t = t0 + threadIdx.x;
    if constexpr (kReduceThreads == kReduceThreadsSmall) {
        // at most eight a thread: all in flight at once, places behind the end count as zero (one after the other 1536 of them took
        // 1.3 us longer)
        double v[8];
#pragma unroll
        for (uint32_t k = 0; k < 8; k++)
            v[k] = t + k * kReduceThreads < t1 ? src[t + k * kReduceThreads] : 0.0;
#pragma unroll
        for (uint32_t k = 0; k < 8; k++)
            a0 += v[k];
    } else {
        for (; t + 7 * kReduceThreads < t1; t += 8 * kReduceThreads) {
            const double v0 = src[t], v1 = src[t + kReduceThreads], v2 = src[t + 2 * kReduceThreads], v3 = src[t + 3 * kReduceThreads];
            const double v4 = src[t + 4 * kReduceThreads], v5 = src[t + 5 * kReduceThreads], v6 = src[t + 6 * kReduceThreads],
                         v7 = src[t + 7 * kReduceThreads];
            a0 += v0; a1 += v1; a2 += v2; a3 += v3;
            a0 += v4; a1 += v5; a2 += v6; a3 += v7;
        }
        for (; t + 3 * kReduceThreads < t1; t += 4 * kReduceThreads) {
            a0 += src[t];
            a1 += src[t + kReduceThreads];
            a2 += src[t + 2 * kReduceThreads];
            a3 += src[t + 3 * kReduceThreads];
        }
        for (; t < t1; t += kReduceThreads)
            a0 += src[t];
    }
    const double w = wave_sum((a0 + a1) + (a2 + a3));
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
        double total = red[0];
#pragma unroll
        for (int k = 1; k < kReduceThreads / 64; k++)
            total += red[k];
        dst[0] = total;
    }
}

// One workgroup per matrix; 256 threads instead of 1024 when every matrix has at most 2048 partial results, as in hand_over, whose
// sums have to be the same bits (tmask_approx_noalloc takes two launches where tmask_approx takes one).
static void enqueue_objective_reduce(const ReduceArgs &rargs, int nb, hipStream_t stream)
{
    uint32_t most = 0;
    for (int k = 0; k < nb; k++)
        most = rargs.tile0[k + 1] - rargs.tile0[k] > most ? rargs.tile0[k + 1] - rargs.tile0[k] : most;
    if (most <= 8 * kReduceThreadsSmall)
        hipLaunchKernelGGL(objective_reduce_kernel<kReduceThreadsSmall>, dim3(nb), dim3(kReduceThreadsSmall), 0, stream, rargs);
    else
        hipLaunchKernelGGL(objective_reduce_kernel<kReduceThreads>, dim3(nb), dim3(kReduceThreads), 0, stream, rargs);
}

// Score of a bf16 strip at M = 4 with byte masks (4 rows x 8 columns = two blocks per lane) in packed arithmetic: the
// mask bytes of a row group are normalised to 0x80 / 0x00 once, column counts are byte-wise sums, row counts popcounts
// packed one per byte, "more than N" / "not N" are byte-wise tests followed by a popcount, and the sums run two
// magnitudes at a time through the bf16 dot-product instruction against (1, 1), pruned entries cleared to +0 first
// (a select, so a pruned Inf or NaN does not reach the sum).  About 5 vector instructions per weight instead of 15,
// which matters because bf16 leaves 18 to 24 per weight at HBM speed.
typedef __bf16 score_bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float dot2_ones(uint32_t pair, float acc)
{
    union { uint32_t u; score_bf16x2 v; } a, o;
    a.u = pair;
    o.u = 0x3F803F80u;
    return __builtin_amdgcn_fdot2_f32_bf16(a.v, o.v, acc, false);
}

__device__ __forceinline__ uint32_t bytes_nonzero(uint32_t v)      // 0x80 in every byte of v that is not zero
{
    return (((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v) & 0x80808080u;
}

__device__ __forceinline__ void score_strip_bf16_m4(const MatDev &md, StripPos pos, uint32_t N, float &retained, float &total,
                                                    uint32_t &kept, uint32_t &rowv, uint32_t &colv, uint32_t &rowne,
                                                    uint32_t &colne)
{
    const char *base = (const char *)md.w + ((size_t)pos.br * 4 * md.ld + (size_t)pos.sc * 8) * 2;
    const size_t row_bytes = (size_t)md.ld * 2;
    const char *mb = (const char *)md.mask + (size_t)pos.br * 4 * md.mask_ld + (size_t)pos.sc * 8;
    u32x4 raw[4];
    u32x2 mk[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        raw[i] = __builtin_nontemporal_load((const u32x4 *)(base + i * row_bytes));
        mk[i] = __builtin_nontemporal_load((const u32x2 *)(mb + (size_t)i * md.mask_ld));
    }
    const uint32_t nrep = N * 0x01010101u;
    float blk[2] = {0.f, 0.f}, tot = 0.f;
    uint32_t colsum[2] = {0u, 0u}, rowpk[2] = {0u, 0u};     // kept per column / per row of a block, one count per byte
#pragma unroll
    for (int i = 0; i < 4; i++) {
#pragma unroll
        for (int b = 0; b < 2; b++) {
            const uint32_t nz = bytes_nonzero(b ? mk[i].y : mk[i].x);
            const uint32_t one = nz >> 7;
            colsum[b] += one;
            rowpk[b] |= (uint32_t)__builtin_popcount(nz) << (8 * i);
            const uint32_t ff = (nz - one) | nz;                                   // 0xFF in every kept byte
            const uint32_t lo = __builtin_amdgcn_perm(ff, ff, 0x01010000u);        // columns 0, 1 as 16-bit masks
            const uint32_t hi = __builtin_amdgcn_perm(ff, ff, 0x03030202u);        // columns 2, 3
            const uint32_t d0 = (b ? raw[i].z : raw[i].x) & 0x7FFF7FFFu;
            const uint32_t d1 = (b ? raw[i].w : raw[i].y) & 0x7FFF7FFFu;
            tot = dot2_ones(d0, tot);
            tot = dot2_ones(d1, tot);
            blk[b] = dot2_ones(d0 & lo, blk[b]);
            blk[b] = dot2_ones(d1 & hi, blk[b]);
        }
    }
    // counts are at most 4 and N at most 3: byte + (0x7F - N) has its top bit set exactly when the count exceeds N
    auto over = [&](uint32_t c) { return (uint32_t)__builtin_popcount((c + (0x7F7F7F7Fu - nrep)) & 0x80808080u); };
    auto differ = [&](uint32_t c) { return (uint32_t)__builtin_popcount(bytes_nonzero(c ^ nrep)); };
#pragma unroll
    for (int b = 0; b < 2; b++) {
        kept += __builtin_amdgcn_sad_u8(colsum[b], 0u, 0u);
        colv += over(colsum[b]);
        colne += differ(colsum[b]);
        rowv += over(rowpk[b]);
        rowne += differ(rowpk[b]);
    }
    if (md.aux) {   // the lane's two per-block sums are neighbours in memory; streamed, not left dirty in the caches
        u32x2 o;
        o.x = __float_as_uint(blk[0]);
        o.y = __float_as_uint(blk[1]);
        float *dst = (float *)md.aux + (size_t)pos.br * (md.spr * 2u) + pos.sc * 2u;
        if (((uintptr_t)dst & 7u) == 0u) {
            stream_store(o, (u32x2 *)dst);
        } else {
            stream_store(o.x, (uint32_t *)dst);
            stream_store(o.y, (uint32_t *)dst + 1);
        }
    }
    retained = blk[0] + blk[1];
    total = tot;
}

template <int DT, int M, int FMT, typename Args>
__global__ __launch_bounds__(kThreads) void score_kernel(const Args args)
{
    using Ge = Geo<DT, M>;
    constexpr int C = Ge::C, CL = Ge::CL;
    __shared__ double redd[kThreads / 64][2];
    __shared__ uint32_t redu[kThreads / 64][5];
    const uint32_t tile = blockIdx.x;
    int which = find_matrix(args, tile);
    const MatDev md = args.m[which];
    Handover out;
    auto where = [&](auto early) {
        return handover<sizeof(ScorePartial), 7, decltype(early)::value>(args.partials, args.tags, args.partial0 + tile, tile - args.m[which].tile0,
                                                                         args.m[which].pad, args.score + which);
    };
    if constexpr (DT != kBF16N)
        out = where(std::true_type{});
    const uint32_t s = (tile - md.tile0) * kThreads + threadIdx.x;
    const uint32_t gpos = threadIdx.x & (Ge::G - 1);
    const uint32_t N = args.N;
    float retained = 0.f, total = 0.f;
    uint32_t kept = 0, rowv = 0, colv = 0, rowne = 0, colne = 0;
    if constexpr (DT == kBF16 && M == 4 && FMT == kMaskU8) {
        if (s < md.n_strips)
            score_strip_bf16_m4(md, strip_pos(md, s), N, retained, total, kept, rowv, colv, rowne, colne);
    } else if (M >= 16 && s < md.n_strips) {
        // M = 16 (one block per lane group, B = 1): a row at a time, so that only the raw rows and the mask bits stay
        // in registers (with every magnitude unpacked up front the bf16 8:16 kernel held 248 registers: two wavefronts
        // per SIMD; now 94, 8192^2 bf16 8:16: 42 -> 39 us).  Same order of additions as below.  At M = 8 the form below is
        // the faster one (it keeps more loads and additions in flight).
        const StripPos pos = strip_pos(md, s);
        u32x4 raw[M];
        uint32_t bits[M];
        const char *base = (const char *)md.w + ((size_t)pos.br * M * md.ld + (size_t)pos.sc * C) * Ge::ES;
        const size_t row_bytes = (size_t)md.ld * Ge::ES;
#pragma unroll
        for (int i = 0; i < M; i++)
            raw[i] = __builtin_nontemporal_load((const u32x4 *)(base + i * row_bytes));
        load_mask<DT, M, FMT>(md, pos, bits);
        // opaque from here on: otherwise every bit test below is rewritten as a test on the intermediate values of the
        // byte-to-bit conversion, all of which then stay in registers
#pragma unroll
        for (int i = 0; i < M; i++)
            asm volatile("" : "+v"(bits[i]));
        float tot = 0.f, blk = 0.f;
        uint32_t colcnt[C];
#pragma unroll
        for (int c = 0; c < C; c++)
            colcnt[c] = 0;
#pragma unroll
        for (int i = 0; i < M; i++) {
            u32x4 r = raw[i];
            asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w));    // unpack here, not ahead of the loop
            const uint32_t d[4] = {r.x, r.y, r.z, r.w};
            float m[C];
            if constexpr (DT == kF32) {
#pragma unroll
                for (int c = 0; c < 4; c++)
                    m[c] = __uint_as_float(d[c] & 0x7FFFFFFFu);
            } else {
#pragma unroll
                for (int c = 0; c < 4; c++) {
                    m[2 * c] = __uint_as_float((d[c] << 16) & 0x7FFF0000u);
                    m[2 * c + 1] = __uint_as_float(d[c] & 0x7FFF0000u);
                }
            }
            uint32_t cnt = __builtin_popcount(bits[i] & ((1u << C) - 1u));
            if constexpr (Ge::G >= 2)
                cnt = quad_xor_sum<1>(cnt);
            if constexpr (Ge::G == 4)
                cnt = quad_xor_sum<2>(cnt);
            if (gpos == 0) {
                rowv += cnt > N ? 1u : 0u;
                rowne += cnt != N ? 1u : 0u;
            }
#pragma unroll
            for (int c = 0; c < C; c++) {
                const bool k = (bits[i] >> c) & 1u;
                tot += m[c];
                blk += k ? m[c] : 0.f;
                colcnt[c] += k ? 1u : 0u;
            }
            // the row's contributions are added here and now (left alone, the additions sink to the end of the kernel
            // and every magnitude stays in a register until then)
            asm volatile("" : "+v"(tot), "+v"(blk), "+v"(rowv), "+v"(rowne));
#pragma unroll
            for (int c = 0; c < C; c++)
                asm volatile("" : "+v"(colcnt[c]));
        }
        total = tot;
        retained = blk;
#pragma unroll
        for (int c = 0; c < C; c++) {
            kept += colcnt[c];
            colv += colcnt[c] > N ? 1u : 0u;
            colne += colcnt[c] != N ? 1u : 0u;
        }
        if constexpr (Ge::G >= 2)
            blk += __uint_as_float(quad_xor<1>(__float_as_uint(blk)));
        if constexpr (Ge::G == 4)
            blk += __uint_as_float(quad_xor<2>(__float_as_uint(blk)));
        if (md.aux && gpos == 0) {
            const uint32_t bpr = md.spr / Ge::G;        // blocks per block-row
            stream_store(blk, (float *)md.aux + (size_t)pos.br * bpr + pos.sc / Ge::G);
        }
    } else if (s < md.n_strips) {
        const StripPos pos = strip_pos(md, s);
        uint32_t a[M][C];
        u32x4 raw[M];
        uint32_t bits[M];
        load_strip<DT, M>(md, pos, a, raw);
        load_mask<DT, M, FMT>(md, pos, bits);
        float tot = 0.f;
#pragma unroll
        for (int i = 0; i < M; i++)
#pragma unroll
            for (int c = 0; c < C; c++)
                tot += __uint_as_float(a[i][c]);
        total = tot;
        // columns: lane-local
#pragma unroll
        for (int c = 0; c < C; c++) {
            uint32_t cnt = 0;
#pragma unroll
            for (int i = 0; i < M; i++)
                cnt += (bits[i] >> c) & 1u;
            kept += cnt;
            colv += cnt > N ? 1u : 0u;
            colne += cnt != N ? 1u : 0u;
        }
        // rows: per block inside the lane, summed over the G lanes of the block, counted once
#pragma unroll
        for (int b = 0; b < Ge::B; b++) {
            float blk = 0.f;
#pragma unroll
            for (int i = 0; i < M; i++) {
                uint32_t cnt = __builtin_popcount((bits[i] >> (b * CL)) & ((1u << CL) - 1u));
                if constexpr (Ge::G >= 2)
                    cnt += quad_xor<1>(cnt);
                if constexpr (Ge::G == 4)
                    cnt += quad_xor<2>(cnt);
                if (gpos == 0) {
                    rowv += cnt > N ? 1u : 0u;
                    rowne += cnt != N ? 1u : 0u;
                }
#pragma unroll
                for (int c = 0; c < CL; c++)
                    blk += ((bits[i] >> (b * CL + c)) & 1u) ? __uint_as_float(a[i][b * CL + c]) : 0.f;
            }
            retained += blk;
            if constexpr (Ge::G >= 2)
                blk += __uint_as_float(quad_xor<1>(__float_as_uint(blk)));
            if constexpr (Ge::G == 4)
                blk += __uint_as_float(quad_xor<2>(__float_as_uint(blk)));
            if (md.aux && gpos == 0) {
                // block index inside the matrix: block-row-major
                const uint32_t bpr = md.spr * Ge::B / Ge::G;
                const uint32_t bc = pos.sc * Ge::B / Ge::G + b;
                stream_store(blk, (float *)md.aux + (size_t)pos.br * bpr + bc);
            }
        }
    }
    // One reduction pass: fp32 / packed 32-bit counts inside a wavefront (a lane contributes at most
    // 128 kept, 16 row events and 8 column events, so 16-bit fields cannot overflow over 64 lanes),
    // then the four wavefronts in fp64 / 64-bit through LDS.
    const double w_ret = wave_kept<DT>(retained), w_tot = wave_kept<DT>(total);
    const uint32_t w_a = wave_sum(kept | (rowv << 16));
    const uint32_t w_b = wave_sum(colv | (colne << 16));
    const uint32_t w_c = wave_sum(rowne);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        redd[wave][0] = w_ret;
        redd[wave][1] = w_tot;
        redu[wave][0] = w_a & 0xFFFFu;
        redu[wave][1] = w_a >> 16;
        redu[wave][2] = w_b & 0xFFFFu;
        redu[wave][3] = w_c;
        redu[wave][4] = w_b >> 16;
    }
    __syncthreads();
    ScoreSums own = {};
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kThreads / 64; k++) {
            own.retained += redd[k][0]; own.total += redd[k][1];
            own.kept += redu[k][0]; own.rowv += redu[k][1]; own.colv += redu[k][2]; own.rowne += redu[k][3]; own.colne += redu[k][4];
        }
    }
    if constexpr (DT == kBF16N) {
        // read here: these lanes have half the work, and what their launches mostly leave to a second one is not worth scalar loads
        // ahead of theirs (8192 x 8196: 47.9 us with them, 47.3 here, 47.2 where no launch adds up its own)
        asm volatile("" : "+s"(which));
        out = where(std::false_type{});
    }
    hand_over_score<kThreads>(out, own);
}

struct ScoreReduceArgs {
    uint32_t tile0[kMaxBatch + 1];
    uint32_t n_mats;
    uint32_t partial0;
    const ScorePartial *partials;
    tmask_score_out *out;   // entry of the first matrix of this launch
};

// 1024 threads, two records in flight per thread: the loop is a chain of load latencies.  A matrix of 16384 x 16384
// leaves 32768 (bf16) or 65536 (fp32) records, which one workgroup still needs 24 / 41 us for, so large matrices are
// reduced in two launches: STAGE 1, workgroup (m, s) adds slice s of matrix m's records and leaves the sum in the
// slice's first record (only this workgroup reads the slice); STAGE 2, workgroup m adds those first records.
// STAGE 0 is the single launch: workgroup m adds all records of matrix m.
constexpr uint32_t kReduceSlices = 32;
constexpr uint32_t kReduceTwoStageFrom = 8192;    // records of the largest matrix of a launch

// THREADS: 1024, or 256 when no matrix of the launch has more than 2048 records: four wavefronts to start, reduce and add up
// instead of sixteen (mask, compression and score, us: 52 matrices of up to 576 records 93.1 -> 90.4, 4096 x 1024 fp32 of 1024
// records 30.2 -> 26.4, 4096 x 2048 of 2048 43.0 -> 40.8).
template <int STAGE, int THREADS = kReduceThreads>
__global__ __launch_bounds__(THREADS) void score_reduce_kernel(const ScoreReduceArgs args)
{
    constexpr uint32_t kReduceThreads = THREADS;      // shadows the file-scope constant inside this kernel
    __shared__ double redd[2][kReduceThreads / 64];
    __shared__ unsigned long long redu[5][kReduceThreads / 64];
    const uint32_t m = blockIdx.x;
    double retained = 0.0, total = 0.0;
    unsigned long long kept = 0, rowv = 0, colv = 0, rowne = 0, colne = 0;
    const uint32_t t0 = args.tile0[m], t1 = args.tile0[m + 1];
    const uint32_t len = (t1 - t0 + kReduceSlices - 1) / kReduceSlices;     // records per slice
    // records base + i * stride, i < count
    uint32_t base = t0, count = t1 - t0, stride = 1;
    if constexpr (STAGE == 1) {
        base = t0 + blockIdx.y * len;
        if (base >= t1)
            return;                                   // the whole workgroup: nothing in this slice
        count = t1 - base < len ? t1 - base : len;
    } else if constexpr (STAGE == 2) {
        stride = len;
        count = len ? (t1 - t0 + len - 1) / len : 0;
    }
    const ScorePartial *src = args.partials + args.partial0 + base;
    uint32_t i = threadIdx.x;
    for (; i + kReduceThreads < count; i += 2 * kReduceThreads) {
        const ScorePartial p = src[(size_t)i * stride];
        const ScorePartial q = src[(size_t)(i + kReduceThreads) * stride];
        retained += p.retained; total += p.total;
        kept += p.kept; rowv += p.rowv; colv += p.colv; rowne += p.rowne; colne += p.colne;
        retained += q.retained; total += q.total;
        kept += q.kept; rowv += q.rowv; colv += q.colv; rowne += q.rowne; colne += q.colne;
    }
    for (; i < count; i += kReduceThreads) {
        const ScorePartial p = src[(size_t)i * stride];
        retained += p.retained; total += p.total;
        kept += p.kept; rowv += p.rowv; colv += p.colv; rowne += p.rowne; colne += p.colne;
    }
    // all seven sums per wavefront first, one barrier, then thread 0 adds the wavefronts in a fixed order
    const double d[2] = {wave_sum(retained), wave_sum(total)};
    const unsigned long long u[5] = {wave_sum(kept), wave_sum(rowv), wave_sum(colv), wave_sum(rowne), wave_sum(colne)};
    if ((threadIdx.x & 63) == 0) {
        const uint32_t w = threadIdx.x >> 6;
#pragma unroll
        for (int k = 0; k < 2; k++)
            redd[k][w] = d[k];
#pragma unroll
        for (int k = 0; k < 5; k++)
            redu[k][w] = u[k];
    }
    __syncthreads();          // every thread's records have arrived by now: STAGE 1 may overwrite the slice's first one
    if (threadIdx.x == 0) {
        double r[2];
        unsigned long long c[5];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            r[k] = redd[k][0];
            for (int w = 1; w < (int)(kReduceThreads / 64); w++)
                r[k] += redd[k][w];
        }
#pragma unroll
        for (int k = 0; k < 5; k++) {
            c[k] = redu[k][0];
            for (int w = 1; w < (int)(kReduceThreads / 64); w++)
                c[k] += redu[k][w];
        }
        if constexpr (STAGE == 1) {
            ScorePartial *o = const_cast<ScorePartial *>(src);
            o->retained = r[0]; o->total = r[1];
            o->kept = c[0]; o->rowv = c[1]; o->colv = c[2]; o->rowne = c[3]; o->colne = c[4];
        } else {
            tmask_score_out *o = args.out + m;
            o->retained_l1 = r[0]; o->total_l1 = r[1];
            o->kept = c[0]; o->row_violations = c[1]; o->col_violations = c[2]; o->row_not_n = c[3]; o->col_not_n = c[4];
        }
    }
}

// =================================================================================================
// Host side
// =================================================================================================

static thread_local char g_err[512] = "";

int fail(int code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

static bool valid_nm(int N, int M) { return (M == 4 || M == 8 || M == 16 || M == 32) && N > 0 && N < M; }

static size_t elem_size(int dt) { return dt == TMASK_F32 ? 4 : 2; }

// s / d == (uint64(s) * mul) >> shift for every s < 2^31 (d >= 1).
static void magic_div(uint32_t d, uint32_t *mul, uint32_t *shift)
{
    uint32_t l = 0;
    while ((1ull << l) < d)
        l++;
    const uint32_t k = 31 + l;
    *mul = (uint32_t)(((1ull << k) / d) + 1);
    *shift = k;
}

struct HostMat {
    const void *w; int64_t rows, cols, ld;
    void *mask; int64_t mask_ld;
    double *objective;
};

// What the matrices of a call let it run on: strips of 16 bytes, the 8-byte strips that exist for bf16 at M = 4, or only
// the column-per-lane kernels (also M = 32).  Narrow strips move half the bytes per instruction, but a matrix whose width
// is an odd multiple of four then runs at the speed of the others: 1000 x 2052 bf16 2:4, mask 20 -> 5 us, score 24 -> 5 us,
// compression 13 -> 8 us (the three calls with their second stages 62.9 -> 32.2 us).
enum Fit { kFitColumns, kFitNarrow, kFitWide };

static Fit fit_at_best(int M) { return M == 32 ? kFitColumns : kFitWide; }

// Lowers *fit to what addresses (or pitches in bytes) allow that are all multiples of the powers of two in `bits`, for
// accesses of `wide` bytes, or `wide` / 2 with narrow strips.
static void lower_fit(Fit *fit, uint64_t bits, uint64_t wide, bool narrow)
{
    if (*fit == kFitWide && bits % wide)
        *fit = narrow ? kFitNarrow : kFitColumns;
    if (*fit == kFitNarrow && bits % (wide / 2))
        *fit = kFitColumns;
}

// Validates one matrix for (dt, N, M, mf).  *fit is lowered (never raised) when the matrix misses what the strip
// kernels read and write with: w 16-byte aligned with ld and cols multiples of 16 bytes, a U8 mask and its pitch
// multiples of the strip width; half of all that for narrow strips.
static int check_mat(const HostMat &h, int idx, int dt, int M, int mf, bool need_mask, Fit *fit)
{
    const size_t es = elem_size(dt);
    const int64_t C = 16 / (int64_t)es;
    const bool narrow = dt == TMASK_BF16 && M == 4;
    if (!h.w || (need_mask && !h.mask))
        return fail(TMASK_ERR_NULL, "matrix %d: w or mask is NULL", idx);
    if (h.rows <= 0 || h.cols <= 0 || h.rows % M || h.cols % M || h.ld < h.cols)
        return fail(TMASK_ERR_SHAPE, "matrix %d: rows=%lld cols=%lld ld=%lld must be positive multiples of M=%d with ld >= cols",
                    idx, (long long)h.rows, (long long)h.cols, (long long)h.ld, M);
    if (h.ld > 0x7FFFFFFFll || h.mask_ld > 0x7FFFFFFFll || (h.rows / M) * ((h.cols + 3) / 4) >= 0x7FFFFFFFll)
        return fail(TMASK_ERR_SHAPE, "matrix %d: too large (ld, mask_ld and strip count must stay below 2^31)", idx);
    if ((uintptr_t)h.w % es)
        return fail(TMASK_ERR_ALIGN, "matrix %d: w must be aligned to its element size", idx);
    lower_fit(fit, (uint64_t)(uintptr_t)h.w | (uint64_t)(h.ld * es) | (uint64_t)(h.cols * es), 16, narrow);
    if (h.mask) {
        if (mf == TMASK_MASK_U8) {
            if (h.mask_ld < h.cols)
                return fail(TMASK_ERR_SHAPE, "matrix %d: mask_ld=%lld < cols", idx, (long long)h.mask_ld);
            lower_fit(fit, (uint64_t)(uintptr_t)h.mask | (uint64_t)h.mask_ld, (uint64_t)C, narrow);
        } else {
            if (h.cols % 8)
                return fail(TMASK_ERR_SHAPE, "matrix %d: BITS masks need cols to be a multiple of 8", idx);
            if (h.mask_ld < h.cols / 8)
                return fail(TMASK_ERR_SHAPE, "matrix %d: mask_ld=%lld < cols/8", idx, (long long)h.mask_ld);
        }
    }
    return TMASK_OK;
}

// sdt: the strip kernels' type (kF32, kBF16, or kBF16N for narrow strips)
static int strip_type(int dt, Fit fit) { return fit == kFitNarrow ? (int)kBF16N : dt; }

static int64_t strip_cols(int sdt) { return sdt == kBF16 ? 8 : 4; }

static uint32_t strips_of(const HostMat &h, int sdt, int M)
{
    const int64_t C = strip_cols(sdt);
    return (uint32_t)((h.rows / M) * (h.cols / C));
}

static uint32_t tiles_of(uint32_t n_strips) { return (n_strips + kThreads - 1) / kThreads; }

static void fill_desc(MatDev &d, const HostMat &h, int sdt, int M, uint32_t tile0)
{
    const int64_t C = strip_cols(sdt);
    d.w = h.w; d.mask = h.mask; d.aux = nullptr;
    d.ld = (uint32_t)h.ld; d.mask_ld = (uint32_t)h.mask_ld;
    d.spr = (uint32_t)(h.cols / C);
    d.n_strips = strips_of(h, sdt, M);
    magic_div(d.spr, &d.div_mul, &d.div_shift);
    d.tile0 = tile0; d.pad = 0;
}

// A kernel with the two sizes of its table; few may be null.
struct BatchKernel {
    void (*many)(const BatchArgs);
    void (*few)(const FewArgs);
};
#define TMASK_BOTH(KERN, ...) BatchKernel{KERN<__VA_ARGS__, BatchArgs>, KERN<__VA_ARGS__, FewArgs>}
#define TMASK_MANY(KERN, ...) BatchKernel{KERN<__VA_ARGS__>, nullptr}

// Calls go(table, kernel) with the table that a launch over n matrices takes, cleared.
template <typename Go>
static int with_table(const BatchKernel &k, int n, Go go)
{
    if (k.few && n <= kFewMats) {
        FewArgs args;
        memset(&args, 0, sizeof args);
        return go(args, k.few);
    }
    BatchArgs args;
    memset(&args, 0, sizeof args);
    return go(args, k.many);
}

template <int SOLVER>
static BatchKernel pick_mask_kernel(int dt, int M, int mf)
{
#define TMASK_PICK(DT, MM, FM) \
    if (dt == DT && M == MM && mf == FM) return TMASK_MANY(mask_kernel, SOLVER, DT, MM, FM);
    TMASK_PICK(kF32, 4, kMaskU8) TMASK_PICK(kBF16, 4, kMaskU8) TMASK_PICK(kBF16N, 4, kMaskU8)
    TMASK_PICK(kF32, 4, kMaskBits) TMASK_PICK(kBF16, 4, kMaskBits) TMASK_PICK(kBF16N, 4, kMaskBits)
    if constexpr (SOLVER == kSolveRow1D) {        // Algorithm 1 at M = 8, 16 has threshold forms for every N
        TMASK_PICK(kF32, 8, kMaskU8) TMASK_PICK(kF32, 16, kMaskU8) TMASK_PICK(kBF16, 8, kMaskU8) TMASK_PICK(kBF16, 16, kMaskU8)
        TMASK_PICK(kF32, 8, kMaskBits) TMASK_PICK(kF32, 16, kMaskBits) TMASK_PICK(kBF16, 8, kMaskBits) TMASK_PICK(kBF16, 16, kMaskBits)
    }
#undef TMASK_PICK
    return BatchKernel{nullptr, nullptr};
}

static BatchKernel pick_score_kernel(int dt, int M, int mf)
{
#define TMASK_PICK(DT, MM, FM) \
    if (dt == DT && M == MM && mf == FM) return TMASK_BOTH(score_kernel, DT, MM, FM);
    TMASK_PICK(kF32, 4, kMaskU8) TMASK_PICK(kF32, 8, kMaskU8) TMASK_PICK(kF32, 16, kMaskU8)
    TMASK_PICK(kBF16, 4, kMaskU8) TMASK_PICK(kBF16, 8, kMaskU8) TMASK_PICK(kBF16, 16, kMaskU8)
    TMASK_PICK(kF32, 4, kMaskBits) TMASK_PICK(kF32, 8, kMaskBits) TMASK_PICK(kF32, 16, kMaskBits)
    TMASK_PICK(kBF16, 4, kMaskBits) TMASK_PICK(kBF16, 8, kMaskBits) TMASK_PICK(kBF16, 16, kMaskBits)
    TMASK_PICK(kBF16N, 4, kMaskU8) TMASK_PICK(kBF16N, 4, kMaskBits)
#undef TMASK_PICK
    return BatchKernel{nullptr, nullptr};
}

// Whether a launch over these matrices has at most `per_cu` tiles of TR x TC for a compute unit, so that tiles of half the
// height, or width, (one or two block-rows per lane instead of two or four) pay.  A launch of a tile or two per compute unit takes
// as long as a tile does, and half the work per lane nearly halves that; with more tiles the shorter runs per column of W^T
// cost more.  Whole tile / half tile in us, graph replays: bf16 4:8 compression 1024^2 10.8 / 7.8, 4096 x 3072 (384 tiles)
// 18.9 / 18.4, 4096^2 (512) 20.3 / 26.0; in one pass 14.4 / 9.8, 4096^2 21.9 / 20.8, 20 x 1024^2 (640) 28.9 / 26.8, 4096 x
// 6144 (768) 31.0 / 35.1.  bf16 2:4 the same lines; fp32 2:4 1024^2 8.3 / 6.3, 6 x 1024^2 (384) 15.1 / 13.4, 4096 x 2048
// (512) 16.7 / 19.0; in one pass 10.0 / 7.0, 512 tiles 14.6 / 13.7, 768 tiles 22.7 / 26.8.  fp32 4:8 (half the width, one block-row to
// a lane) 128^2 8.9 / 6.1, 2048^2 (256) 11.7 / 9.7, 3144 x 3192 (650) 28.7 / 34.0; in one pass 128^2 16.9 / 8.3, 2048^2 15.5 / 12.2, 3072^2
// (576) 24.1 / 20.2, 4096 x 3072 (768) 25.6 / 29.3.
// Quarter tiles of the 2:4 kernels, one block-row to a lane, where there are no more than 0.7 whole tiles (1 in one pass) for a compute unit.  Half
// / quarter, us: fp32 1024 x 512 5.6 / 4.8, 1948 x 1216 (155 tiles) 10.0 / 8.1, 2048^2 (256) 8.1 / 9.1; in one pass 8.0 / 6.9, 11.9 / 9.8, 10.1 / 10.1,
// 2048 x 3072 (384) 12.6 / 14.3; bf16 1024 x 512 6.5 / 5.1, 2048^2 (128) 7.5 / 7.1, 2048 x 3072 (192) 9.3 / 9.5; in one pass 9.8 / 7.5, 10.9 / 9.5, 13.2 / 12.1.
// Narrow strips (tiles of 64 x 128): 1000 x 1028 6.4 / 5.5, 1000 x 2052 (272) 7.5 / 6.6, 2048 x 1540 (416) 7.7 / 7.5, 2048 x 2052 (544) 9.8 / 11.3.
constexpr double kQuarterTilesPack = 0.7, kQuarterTilesFused = 1.0, kQuarterTilesNarrow = 1.75;
// The kernel for any N:M takes workgroups of 1024 threads instead of 256 up to two tiles for a compute unit, which is what one holds of
// them: a unit to a thread instead of four to eight one after the other.  256 / 1024, us: fp32 8:16 464 x 128 5.9 / 4.3, 2048 x 1024 (512
// tiles) 7.0 / 6.2, 2048^2 (1024) 10.5 / 11.9; 7:8 464 x 128 8.2 / 5.3, 2048 x 1024 13.9 / 11.8; bf16 8:16 464 x 128 7.3 / 4.7, 2048^2 (512) 9.8 / 7.9,
// 1712 x 2752 (594) 12.1 / 12.7; 3:8 9.5 / 5.8, 13.0 / 10.1, 15.3 / 14.8.
constexpr double kWideTilesPack = 2.0;
constexpr double kHalfTilesPack = 1.5, kHalfTilesFusedF32 = 2.0, kHalfTilesFusedF32M8 = 2.5, kHalfTilesFusedBf16 = 2.5;

template <typename DESC>
static bool few_tiles(const DESC *descs, int n, int64_t TR, int64_t TC, double per_cu)
{
    uint64_t tiles = 0;
    for (int i = 0; i < n; i++)
        tiles += (uint64_t)((descs[i].rows + TR - 1) / TR) * (uint64_t)((descs[i].cols + TC - 1) / TC);
    return (double)tiles <= per_cu * cu_count();
}

static int check_common(const void *mats, int n_mats, int dt, int N, int M, int mf)
{
    if (!mats)
        return fail(TMASK_ERR_NULL, "descriptor array is NULL");
    if (n_mats <= 0)
        return fail(TMASK_ERR_SHAPE, "n_mats=%d must be positive", n_mats);
    if (dt != TMASK_F32 && dt != TMASK_BF16)
        return fail(TMASK_ERR_DTYPE, "unknown dtype %d", dt);
    if (mf != TMASK_MASK_U8 && mf != TMASK_MASK_BITS)
        return fail(TMASK_ERR_DTYPE, "unknown mask format %d", mf);
    if (!valid_nm(N, M))
        return fail(TMASK_ERR_NM, "unsupported N:M = %d:%d (need M in {4,8,16,32}, 0 < N < M)", N, M);
    return TMASK_OK;
}

static size_t workspace_need(const tmask_mat *mats, int n_mats, int M)
{
    // Upper bound over dtypes: fp32 strips (4 columns) are the narrower ones.
    size_t tiles = 0, pack_tiles = 0;
    for (int i = 0; i < n_mats; i++) {
        if (mats[i].rows <= 0 || mats[i].cols <= 0)
            return 0;
        const size_t strips = (size_t)((mats[i].rows + M - 1) / M) * (size_t)((mats[i].cols + 3) / 4);
        // M = 32 runs on the column-per-lane kernels: one partial result per tile of 32 rows x 64 columns
        tiles += M == 32 ? (size_t)((mats[i].rows + 31) / 32) * (size_t)((mats[i].cols + 63) / 64) : (strips + kThreads - 1) / kThreads;
        // tmask_approx_pack keeps one fp64 partial per tile of its one-pass kernels (64 rows x 256 columns at least)
        pack_tiles += (size_t)((mats[i].rows + 63) / 64) * (size_t)((mats[i].cols + 255) / 256);
    }
    const size_t a = tiles * sizeof(ScorePartial), b = pack_tiles * sizeof(double);
    return (a > b ? a : b) + 256;
}

static int check_workspace(const tmask_mat *mats, int n_mats, int M, void *ws, size_t ws_bytes)
{
    if (!ws || ((uintptr_t)ws & 255))
        return fail(TMASK_ERR_WORKSPACE, "workspace is NULL or not 256-byte aligned");
    const size_t need = workspace_need(mats, n_mats, M);
    if (ws_bytes < need)
        return fail(TMASK_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", ws_bytes, need);
    return TMASK_OK;
}

int hip_fail(hipError_t e, const char *what)
{
    return fail(TMASK_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

// One-shot profiling events (tmask_profile_next): recorded around the main kernel of the next call.
thread_local hipEvent_t g_prof_start = nullptr, g_prof_stop = nullptr;

// The tags of a launch that adds up its own partial results: two numbers that no other launch of this process has beside
// each other, scattered (splitmix64 of a counter that starts anywhere), neither zero, not equal.
Tags draw_tags()
{
    static std::atomic<uint64_t> next{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() ^ (uint64_t)(uintptr_t)&g_prof_start};
    for (;;) {
        uint64_t z = next.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        const Tags t{(uint32_t)z, (uint32_t)(z >> 32)};
        if (t.a && t.b && t.a != t.b)
            return t;
    }
}

// Scratch memory of tmask_approx_noalloc: the per-workgroup partial sums of the objective, which the other entry
// points keep in the caller's workspace.  One copy per GPU, held until the process ends; every call on a GPU shares
// it, so calls that overlap on one GPU race.  Nothing in it has to start at zero: every partial a call reads was
// written by that call.
constexpr size_t kScratchPartials = 65536;      // 512 KiB: one double per workgroup of 256 strips
static __device__ __align__(256) __attribute__((used)) double scratch[kScratchPartials];

constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];        // device address of `scratch` on each GPU (the array's name is only a
static std::mutex g_scratch_lock;               // host-side handle, never a device address)

// Address of the current device's copy of `scratch`, looked up once per device.
static int scratch_of_current_device(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices)
        return fail(TMASK_ERR_HIP, "device ordinal %d is outside the %d this library keeps scratch addresses for", dev, kMaxDevices);
    std::lock_guard<std::mutex> guard(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return TMASK_OK;
}

// Workgroups per compute unit up to which every column of a block has a lane of its own.  tmask_exact: at M = 16 what a compute unit
// holds of that kernel, at M = 8 less, since a block is an eighth of the work there and the start of a kernel weighs more.  One matrix,
// four columns / one column to a lane, us: fp32 8:16 464 x 128 34.7 / 16.1, 2048 x 1024 (two workgroups per unit) 38.1 / 23.4, 2048^2 (4) 37.8 /
// 30.3, 2048 x 2560 (5) 53.6 / 35.7, 3072 x 2048 (6) 46.5 / 40.4, 4096 x 2048 (8) 47.4 / 49.2; 13:16 2048 x 2560 51.4 / 37.2, 4096 x 2048 52.3 / 52.7;
// 4:8 128^2 13.6 / 9.2, 1024 x 512 (1) 15.9 / 11.1, 1024^2 (2) 16.1 / 11.5, 2048 x 1024 (4) 15.5 / 14.4; bf16 4:8 11.7 / 8.1, 14.5 / 10.4, 15.0 / 11.2,
// 2048 x 1024 14.2 / 14.4; 3:8 1024^2 17.7 / 12.5.  (The lines were swept with sums over lanes, 4:8 2048 x 1024 17.4 then; six and four would do now.)
// Algorithm 1 for bf16 at M = 16, eight columns / one: 8:16 1024 x 512 9.0 / 4.8, 1024^2 9.9 / 5.9, 2048^2 (4) 10.7 / 8.0, 3072 x 2048 (6) 10.8 / 10.1, 4096 x
// 2048 (8) 11.4 / 12.5; 5:16 1024^2 12.8 / 6.0, 4096 x 2048 14.0 / 12.1; masked copies 8:16 1024^2 10.1 / 4.8, 4096 x 2048 12.4 / 10.9, 13:16 15.0 / 10.8.
static uint64_t spread_exact(int M) { return M == 16 ? 5u : 2u; }
static uint64_t spread_approx16(bool dense, int N) { return dense || N != 8 ? 8u : 6u; }

// One launch for at most kWholeMats matrices of at most kWholeThreads strips at 2:4 (checked by the caller, like the rest).
template <int SOLVER>
static int run_whole(const tmask_mat *mats, int n_mats, int sdt, int mf, hipStream_t stream)
{
    WholeArgs args;
    for (int k = 0; k < n_mats; k++) {
        const tmask_mat &t = mats[k];
        fill_desc(args.m[k], HostMat{t.w, t.rows, t.cols, t.ld, t.mask, t.mask_ld, t.objective}, sdt, 4, (uint32_t)k);
        args.m[k].aux = t.objective;
    }
    memset(args.m + n_mats, 0, sizeof(MatDev) * (size_t)(kWholeMats - n_mats));
    void (*kern)(const WholeArgs) = nullptr;
#define TMASK_PICK(DT) \
    if (sdt == DT) \
        kern = mf == kMaskU8 ? whole24_kernel<SOLVER, DT, kMaskU8> : whole24_kernel<SOLVER, DT, kMaskBits>;
    TMASK_PICK(kF32) TMASK_PICK(kBF16) TMASK_PICK(kBF16N)
#undef TMASK_PICK
    {
        ProfileScope prof(stream, true);
        hipLaunchKernelGGL(kern, dim3(n_mats), dim3(kWholeThreads), 0, stream, args);
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? TMASK_OK : hip_fail(e, "mask kernel launch");
}

// own_scratch: the partial sums go to the library's static array instead of a caller workspace (ws, ws_bytes unused).
template <int SOLVER>
static int run_mask(const tmask_mat *mats, int n_mats, int dt, int N, int M, int mf, void *ws, size_t ws_bytes,
                    void *stream_, bool own_scratch = false)
{
    int rc = check_common(mats, n_mats, dt, N, M, mf);
    if (rc)
        return rc;
    bool want_obj = false;
    Fit fit = fit_at_best(M);
    for (int i = 0; i < n_mats; i++) {
        const HostMat h{mats[i].w, mats[i].rows, mats[i].cols, mats[i].ld, mats[i].mask, mats[i].mask_ld,
                        mats[i].objective};
        if ((rc = check_mat(h, i, dt, M, mf, true, &fit)))
            return rc;
        want_obj = want_obj || mats[i].objective;
    }
    const int sdt = strip_type(dt, fit);
    if (own_scratch) {
        size_t tiles = 0;
        for (int i = 0; i < n_mats; i++) {
            const HostMat h{mats[i].w, mats[i].rows, mats[i].cols, mats[i].ld, nullptr, 0, nullptr};
            tiles += fit != kFitColumns ? tiles_of(strips_of(h, sdt, M)) : cw_workgroups(h.rows, h.cols, M);
        }
        if (want_obj && tiles > kScratchPartials)
            return fail(TMASK_ERR_WORKSPACE,
                        "this call needs %zu partial sums (one per 256 strips of 16 bytes x M rows); the library's own scratch "
                        "array holds %zu: split the batch, or use the entry point that takes a caller workspace",
                        tiles, kScratchPartials);
        if ((rc = scratch_of_current_device(&ws)))
            return rc;
    } else if (want_obj && (rc = check_workspace(mats, n_mats, M, ws, ws_bytes))) {
        return rc;
    }
    // N != M/2 at M = 16, row pruning: the strip kernels have only their rank form there; the column-per-lane kernels take a
    // threshold from a sorting network
    const bool general_n = 2 * N != M && M == 16 && SOLVER == kSolveRow1D;
    if (fit == kFitColumns || general_n)     // also M = 32, or a matrix that the strips cannot read
        return cw_run_mask(SOLVER == kSolveApprox ? 0 : SOLVER == kSolveExact ? 1 : 2, mats, n_mats, dt, N, M, mf, ws, !own_scratch,
                           (hipStream_t)stream_);
    if constexpr (SOLVER != kSolveRow1D) {       // without objectives the call is one launch anyway
        bool whole = M == 4 && N == 2 && want_obj && n_mats <= kWholeMats;
        for (int i = 0; i < n_mats && whole; i++) {
            const HostMat h{mats[i].w, mats[i].rows, mats[i].cols, mats[i].ld, nullptr, 0, nullptr};
            whole = strips_of(h, sdt, M) <= (uint32_t)kWholeThreads;
        }
        if (whole)
            return run_whole<SOLVER>(mats, n_mats, sdt, mf, (hipStream_t)stream_);
    }
    BatchKernel kern{nullptr, nullptr};
    if constexpr (SOLVER != kSolveExact)      // exact: enumeration at M = 4, the balanced kernel at M = 8, 16 (below)
        kern = pick_mask_kernel<SOLVER>(sdt, M, mf);
    if (SOLVER == kSolveApprox && M == 4 && N == 2) {
        if (sdt == kF32)
            kern = mf == kMaskU8 ? TMASK_BOTH(approx24_kernel, kF32, kMaskU8) : TMASK_BOTH(approx24_kernel, kF32, kMaskBits);
        else if (sdt == kBF16N)
            kern = mf == kMaskU8 ? TMASK_BOTH(approx24_kernel, kBF16N, kMaskU8) : TMASK_BOTH(approx24_kernel, kBF16N, kMaskBits);
        else
            kern = mf == kMaskU8 ? TMASK_BOTH(approx24_kernel, kBF16, kMaskU8) : TMASK_BOTH(approx24_kernel, kBF16, kMaskBits);
    }
    if (SOLVER == kSolveExact && M == 4 && N == 2) {
        if (sdt == kF32)
            kern = mf == kMaskU8 ? TMASK_BOTH(exact24_kernel, kF32, kMaskU8, 2) : TMASK_BOTH(exact24_kernel, kF32, kMaskBits, 2);
        else if (sdt == kBF16N)
            kern = mf == kMaskU8 ? TMASK_BOTH(exact24_kernel, kBF16N, kMaskU8, 2) : TMASK_BOTH(exact24_kernel, kBF16N, kMaskBits, 2);
        else
            kern = mf == kMaskU8 ? TMASK_BOTH(exact24_kernel, kBF16, kMaskU8, 2) : TMASK_BOTH(exact24_kernel, kBF16, kMaskBits, 2);
    }
    if (SOLVER == kSolveExact && M == 4 && N == 1) {
        if (sdt == kF32)
            kern = mf == kMaskU8 ? TMASK_MANY(exact24_kernel, kF32, kMaskU8, 1, BatchArgs) : TMASK_MANY(exact24_kernel, kF32, kMaskBits, 1, BatchArgs);
        else if (sdt == kBF16N)
            kern = mf == kMaskU8 ? TMASK_MANY(exact24_kernel, kBF16N, kMaskU8, 1, BatchArgs) : TMASK_MANY(exact24_kernel, kBF16N, kMaskBits, 1, BatchArgs);
        else
            kern = mf == kMaskU8 ? TMASK_MANY(exact24_kernel, kBF16, kMaskU8, 1, BatchArgs) : TMASK_MANY(exact24_kernel, kBF16, kMaskBits, 1, BatchArgs);
    }
    if (SOLVER == kSolveExact && M == 4 && N == 3) {
        if (sdt == kF32)
            kern = mf == kMaskU8 ? TMASK_MANY(exact24_kernel, kF32, kMaskU8, 3, BatchArgs) : TMASK_MANY(exact24_kernel, kF32, kMaskBits, 3, BatchArgs);
        else if (sdt == kBF16N)
            kern = mf == kMaskU8 ? TMASK_MANY(exact24_kernel, kBF16N, kMaskU8, 3, BatchArgs) : TMASK_MANY(exact24_kernel, kBF16N, kMaskBits, 3, BatchArgs);
        else
            kern = mf == kMaskU8 ? TMASK_MANY(exact24_kernel, kBF16, kMaskU8, 3, BatchArgs) : TMASK_MANY(exact24_kernel, kBF16, kMaskBits, 3, BatchArgs);
    }
    bool spread = false;
    uint32_t threads = kThreads;
    const bool can_spread = SOLVER == kSolveExact ? M == 8 || M == 16 : SOLVER == kSolveApprox && M == 16 && dt == kBF16;
    if (can_spread && n_mats <= kMaxBatch) {
        uint64_t wgs = 0;
        LaunchSums sums;
        for (int i = 0; i < n_mats; i++) {
            const uint64_t own = (uint64_t)(mats[i].rows / M * mats[i].cols + kThreads - 1) / kThreads;
            sums.add((uint32_t)own, mats[i].objective);
            wgs += own;
        }
        // Four of its workgroups take the weights that the workspace reserves 56 bytes for, 64 in records.  Where those do not fit,
        // workgroups of twice the threads leave half of them (8:16 of 1024^2 bf16 8.9 -> 5.9 us against a second launch, 4:8 fp32 14.0 -> 11.8; the
        // optimal masks at M = 16 are faster with one: 20.2, 22.1); several matrices of tmask_exact keep the one launch of the other kernel.
        // By the size that a workspace must have, not by what this one has: the order of the additions is the same with any.
        const bool fits = !want_obj || sums.waiting > kMostWaiting || wgs * 16u <= workspace_need(mats, n_mats, M), exact = SOLVER == kSolveExact;
        spread = (fits || (n_mats <= kFewMats && (n_mats == 1 || !exact))) &&
                 wgs <= (exact ? spread_exact(M) : spread_approx16(false, N)) * (uint64_t)cu_count();
        threads = spread && !fits && !(exact && M == 16) ? 2u * kThreads : kThreads;
    }
    if (spread && SOLVER == kSolveExact) {
#define TMASK_PICK(DT, MM, FM) \
    if (dt == DT && M == MM && mf == FM) \
        kern = 2 * N == M ? TMASK_BOTH(exact_spread_kernel, DT, MM, FM, false) : TMASK_BOTH(exact_spread_kernel, DT, MM, FM, true);
        TMASK_PICK(kF32, 8, kMaskU8) TMASK_PICK(kF32, 16, kMaskU8) TMASK_PICK(kBF16, 8, kMaskU8)
        TMASK_PICK(kBF16, 16, kMaskU8) TMASK_PICK(kF32, 8, kMaskBits) TMASK_PICK(kF32, 16, kMaskBits)
        TMASK_PICK(kBF16, 8, kMaskBits) TMASK_PICK(kBF16, 16, kMaskBits)
#undef TMASK_PICK
#define TMASK_PICK(DT, FM) \
    if (dt == DT && mf == FM && threads > (uint32_t)kThreads) \
        kern.few = 2 * N == M ? exact_spread_kernel<DT, 8, FM, false, FewArgs, 2 * kThreads> : exact_spread_kernel<DT, 8, FM, true, FewArgs, 2 * kThreads>;
        TMASK_PICK(kF32, kMaskU8) TMASK_PICK(kF32, kMaskBits) TMASK_PICK(kBF16, kMaskU8) TMASK_PICK(kBF16, kMaskBits)
#undef TMASK_PICK
    } else if (SOLVER == kSolveExact && (M == 8 || M == 16)) {
#define TMASK_PICK(DT, MM, FM) \
    if (dt == DT && M == MM && mf == FM) \
        kern = 2 * N == M ? TMASK_MANY(exact_balanced_kernel, DT, MM, FM, false) : TMASK_MANY(exact_balanced_kernel, DT, MM, FM, true);
        TMASK_PICK(kF32, 8, kMaskU8) TMASK_PICK(kF32, 16, kMaskU8) TMASK_PICK(kBF16, 8, kMaskU8)
        TMASK_PICK(kBF16, 16, kMaskU8) TMASK_PICK(kF32, 8, kMaskBits) TMASK_PICK(kF32, 16, kMaskBits)
        TMASK_PICK(kBF16, 8, kMaskBits) TMASK_PICK(kBF16, 16, kMaskBits)
#undef TMASK_PICK
    }
    if (SOLVER == kSolveApprox && dt == kF32 && M == 8 && N == 4)
        kern = mf == kMaskU8 ? TMASK_BOTH(approx_sel_f32_kernel, 8, kMaskU8, false) : TMASK_BOTH(approx_sel_f32_kernel, 8, kMaskBits, false);
    if (SOLVER == kSolveApprox && dt == kF32 && M == 16 && N == 8)
        kern = mf == kMaskU8 ? TMASK_BOTH(approx_sel_f32_kernel, 16, kMaskU8, false) : TMASK_BOTH(approx_sel_f32_kernel, 16, kMaskBits, false);
    if (SOLVER == kSolveApprox && dt == kF32 && M == 16 && N != 8)
        kern = mf == kMaskU8 ? TMASK_MANY(approx_sel_f32_kernel, 16, kMaskU8, true, BatchArgs) : TMASK_MANY(approx_sel_f32_kernel, 16, kMaskBits, true, BatchArgs);
    if (SOLVER == kSolveApprox && dt == kBF16 && M == 16 && N != 8)
        kern = mf == kMaskU8 ? TMASK_MANY(approx_sel_bf16_kernel, 16, kMaskU8, true, BatchArgs) : TMASK_MANY(approx_sel_bf16_kernel, 16, kMaskBits, true, BatchArgs);
    if (SOLVER == kSolveApprox && dt == kF32 && M == 8 && N != 4)
        kern = mf == kMaskU8 ? TMASK_MANY(approx_sel_f32_kernel, 8, kMaskU8, true, BatchArgs) : TMASK_MANY(approx_sel_f32_kernel, 8, kMaskBits, true, BatchArgs);
    if (SOLVER == kSolveApprox && dt == kBF16 && M == 8 && N == 4)
        kern = mf == kMaskU8 ? TMASK_BOTH(approx_sel_bf16_kernel, 8, kMaskU8, false) : TMASK_BOTH(approx_sel_bf16_kernel, 8, kMaskBits, false);
    if (SOLVER == kSolveApprox && dt == kBF16 && M == 16 && N == 8)
        kern = mf == kMaskU8 ? TMASK_BOTH(approx_sel_bf16_kernel, 16, kMaskU8, false) : TMASK_BOTH(approx_sel_bf16_kernel, 16, kMaskBits, false);
    if (SOLVER == kSolveApprox && dt == kBF16 && M == 8 && N != 4)
        kern = mf == kMaskU8 ? TMASK_MANY(approx_sel_bf16_kernel, 8, kMaskU8, true, BatchArgs) : TMASK_MANY(approx_sel_bf16_kernel, 8, kMaskBits, true, BatchArgs);
    if (spread && SOLVER == kSolveApprox) {
        kern = mf == kMaskU8 ? TMASK_BOTH(approx_spread16_kernel, kMaskU8, false) : TMASK_BOTH(approx_spread16_kernel, kMaskBits, false);
        if (threads > (uint32_t)kThreads)
            kern.few = mf == kMaskU8 ? approx_spread16_kernel<kMaskU8, false, FewArgs, 2 * kThreads> : approx_spread16_kernel<kMaskBits, false, FewArgs, 2 * kThreads>;
    }
    // the exact kernels give a lane half a strip of bf16 (twice the workgroups) or a column
    const uint32_t unit_split = spread ? (uint32_t)strip_cols(sdt) : (SOLVER == kSolveExact && exact_half_strips(dt, M)) ? 2u : 1u;
    hipStream_t stream = (hipStream_t)stream_;
    uint32_t partial0 = 0;
    for (int first = 0; first < n_mats; first += kMaxBatch) {
        const int nb = n_mats - first < kMaxBatch ? n_mats - first : kMaxBatch;
        ReduceArgs rargs;
        uint32_t tiles = 0;
        LaunchSums sums;
        bool one_launch = false;
        rc = with_table(kern, nb, [&](auto &args, auto kernel) -> int {
            for (int k = 0; k < nb; k++) {
                const tmask_mat &t = mats[first + k];
                const HostMat h{t.w, t.rows, t.cols, t.ld, t.mask, t.mask_ld, t.objective};
                fill_desc(args.m[k], h, sdt, M, tiles);
                rargs.objective[k] = t.objective;
                rargs.tile0[k] = tiles;
                args.m[k].aux = t.objective;
                args.m[k].pad = (args.m[k].n_strips * unit_split + threads - 1) / threads;
                sums.add(args.m[k].pad, t.objective);
                tiles += args.m[k].pad;
            }
            rargs.tile0[nb] = tiles;
            fill_coarse(args.ci, rargs.tile0, nb, tiles);
            args.n_mats = (uint32_t)nb; args.K = (uint32_t)(M - N); args.N = (uint32_t)N;
            args.partial0 = partial0; args.partials = want_obj ? ws : nullptr;
            // the array of tmask_approx_noalloc has room for the sums alone, and calls that overlap share it
            one_launch = want_obj && !own_scratch && adds_up_itself(sums, kThreads, false) &&
                         (size_t)(partial0 + tiles) * 16u <= ws_bytes;
            if (one_launch)
                args.tags = draw_tags();
            {
                ProfileScope prof(stream, first + kMaxBatch >= n_mats);
                launch_kernel(kernel, dim3(tiles), dim3(threads), 0, stream, args);
            }
            const hipError_t e = hipGetLastError();
            return e == hipSuccess ? TMASK_OK : hip_fail(e, "mask kernel launch");
        });
        if (rc)
            return rc;
        if (want_obj && !one_launch) {
            rargs.n_mats = (uint32_t)nb; rargs.partial0 = partial0; rargs.partials = (const double *)ws;
            enqueue_objective_reduce(rargs, nb, stream);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess)
                return hip_fail(e, "objective reduce launch");
        }
        partial0 += tiles;
    }
    return TMASK_OK;
}

// Second-stage reductions for the kernels of other translation units: first0[k] = index (inside this launch) of the
// first partial result of matrix k, first0[nb] = their total number.
int launch_objective_reduce(double *const *objective, const uint32_t *first0, int nb, uint32_t partial0, const void *partials,
                            hipStream_t stream)
{
    ReduceArgs rargs;
    memset(&rargs, 0, sizeof rargs);
    for (int k = 0; k < nb; k++) {
        rargs.objective[k] = objective[k];
        rargs.tile0[k] = first0[k];
    }
    rargs.tile0[nb] = first0[nb];
    rargs.n_mats = (uint32_t)nb; rargs.partial0 = partial0; rargs.partials = (const double *)partials;
    enqueue_objective_reduce(rargs, nb, stream);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? TMASK_OK : hip_fail(e, "objective reduce launch");
}

int launch_score_reduce(const uint32_t *first0, int nb, uint32_t partial0, const void *partials, tmask_score_out *out,
                        hipStream_t stream)
{
    ScoreReduceArgs rargs;
    memset(&rargs, 0, sizeof rargs);
    for (int k = 0; k <= nb; k++)
        rargs.tile0[k] = first0[k];
    rargs.n_mats = (uint32_t)nb; rargs.partial0 = partial0;
    rargs.partials = (const ScorePartial *)partials; rargs.out = out;
    uint32_t most = 0;
    for (int k = 0; k < nb; k++)
        most = first0[k + 1] - first0[k] > most ? first0[k + 1] - first0[k] : most;
    if (most >= kReduceTwoStageFrom) {
        hipLaunchKernelGGL(score_reduce_kernel<1>, dim3(nb, kReduceSlices), dim3(kReduceThreads), 0, stream, rargs);
        hipLaunchKernelGGL(score_reduce_kernel<2>, dim3(nb), dim3(kReduceThreads), 0, stream, rargs);
    } else {
        if (most <= 8 * kReduceThreadsSmall)
            hipLaunchKernelGGL((score_reduce_kernel<0, kReduceThreadsSmall>), dim3(nb), dim3(kReduceThreadsSmall), 0, stream, rargs);
        else
            hipLaunchKernelGGL(score_reduce_kernel<0>, dim3(nb), dim3(kReduceThreads), 0, stream, rargs);
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? TMASK_OK : hip_fail(e, "score reduce launch");
}

// The kernels for any N:M: with workgroups of 256 and the large table, or of 1024 and the small one.
template <int NT, typename Args>
static void (*pick_pack_kernel(int dt, int M, int mf, int N))(const Args)
{
    if (2 * N == M) {   // N known at compile time
#define TMASK_PICK(DT, MM, FM) \
    if (dt == DT && M == MM && mf == FM) return pack_kernel<DT, MM, FM, MM / 2, NT, Args>;
        TMASK_PICK(kF32, 4, kMaskU8) TMASK_PICK(kF32, 8, kMaskU8) TMASK_PICK(kF32, 16, kMaskU8)
        TMASK_PICK(kBF16, 4, kMaskU8) TMASK_PICK(kBF16, 8, kMaskU8) TMASK_PICK(kBF16, 16, kMaskU8)
        TMASK_PICK(kF32, 4, kMaskBits) TMASK_PICK(kF32, 8, kMaskBits) TMASK_PICK(kF32, 16, kMaskBits)
        TMASK_PICK(kBF16, 4, kMaskBits) TMASK_PICK(kBF16, 8, kMaskBits) TMASK_PICK(kBF16, 16, kMaskBits)
        TMASK_PICK(kF32, 32, kMaskU8) TMASK_PICK(kBF16, 32, kMaskU8) TMASK_PICK(kF32, 32, kMaskBits) TMASK_PICK(kBF16, 32, kMaskBits)
#undef TMASK_PICK
    }
#define TMASK_PICK(DT, MM, FM) \
    if (dt == DT && M == MM && mf == FM) return pack_kernel<DT, MM, FM, 0, NT, Args>;
    TMASK_PICK(kF32, 4, kMaskU8) TMASK_PICK(kF32, 8, kMaskU8) TMASK_PICK(kF32, 16, kMaskU8)
    TMASK_PICK(kBF16, 4, kMaskU8) TMASK_PICK(kBF16, 8, kMaskU8) TMASK_PICK(kBF16, 16, kMaskU8)
    TMASK_PICK(kF32, 4, kMaskBits) TMASK_PICK(kF32, 8, kMaskBits) TMASK_PICK(kF32, 16, kMaskBits)
    TMASK_PICK(kBF16, 4, kMaskBits) TMASK_PICK(kBF16, 8, kMaskBits) TMASK_PICK(kBF16, 16, kMaskBits)
#undef TMASK_PICK
    return nullptr;
}

}  // namespace tmask

using namespace tmask;

extern "C" {

int tmask_approx(const tmask_mat *mats, int n_mats, tmask_dtype dt, int N, int M, tmask_mask_fmt mf, void *workspace,
                 size_t workspace_bytes, void *hip_stream)
{
    return run_mask<kSolveApprox>(mats, n_mats, (int)dt, N, M, (int)mf, workspace, workspace_bytes, hip_stream);
}

int tmask_approx_noalloc(const tmask_mat *mats, int n_mats, tmask_dtype dt, int N, int M, tmask_mask_fmt mf,
                         void *hip_stream)
{
    return run_mask<kSolveApprox>(mats, n_mats, (int)dt, N, M, (int)mf, nullptr, 0, hip_stream, true);
}

int tmask_prune_1d(const tmask_mat *mats, int n_mats, tmask_dtype dt, int N, int M, tmask_mask_fmt mf, void *workspace,
                   size_t workspace_bytes, void *hip_stream)
{
    return run_mask<kSolveRow1D>(mats, n_mats, (int)dt, N, M, (int)mf, workspace, workspace_bytes, hip_stream);
}

int tmask_exact(const tmask_mat *mats, int n_mats, tmask_dtype dt, int N, int M, tmask_mask_fmt mf, void *workspace,
                size_t workspace_bytes, void *hip_stream)
{
    return run_mask<kSolveExact>(mats, n_mats, (int)dt, N, M, (int)mf, workspace, workspace_bytes, hip_stream);
}

int tmask_score(const tmask_mat *mats, int n_mats, tmask_dtype dt, int N, int M, tmask_mask_fmt mf,
                tmask_score_out *out, float *per_block_obj, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    int rc = check_common(mats, n_mats, (int)dt, N, M, (int)mf);
    if (rc)
        return rc;
    if (!out)
        return fail(TMASK_ERR_NULL, "out is NULL");
    Fit fit = fit_at_best(M);
    for (int i = 0; i < n_mats; i++) {
        const HostMat h{mats[i].w, mats[i].rows, mats[i].cols, mats[i].ld, mats[i].mask, mats[i].mask_ld, nullptr};
        if ((rc = check_mat(h, i, (int)dt, M, (int)mf, true, &fit)))
            return rc;
    }
    if ((rc = check_workspace(mats, n_mats, M, workspace, workspace_bytes)))
        return rc;
    if (per_block_obj && ((uintptr_t)per_block_obj & 3))
        return fail(TMASK_ERR_ALIGN, "per_block_obj must be 4-byte aligned");
    if (fit == kFitColumns)
        return cw_run_score(mats, n_mats, (int)dt, N, M, (int)mf, out, per_block_obj, workspace, (hipStream_t)hip_stream);
    const int sdt = strip_type((int)dt, fit);
    const BatchKernel kern = pick_score_kernel(sdt, M, (int)mf);
    hipStream_t stream = (hipStream_t)hip_stream;
    uint32_t partial0 = 0;
    size_t block0 = 0;
    for (int first = 0; first < n_mats; first += kMaxBatch) {
        const int nb = n_mats - first < kMaxBatch ? n_mats - first : kMaxBatch;
        uint32_t tile0[kMaxBatch + 1];
        uint32_t tiles = 0;
        LaunchSums sums;
        bool one_launch = false;
        rc = with_table(kern, nb, [&](auto &args, auto kernel) -> int {
            for (int k = 0; k < nb; k++) {
                const tmask_mat &t = mats[first + k];
                const HostMat h{t.w, t.rows, t.cols, t.ld, t.mask, t.mask_ld, nullptr};
                fill_desc(args.m[k], h, sdt, M, tiles);
                args.m[k].aux = per_block_obj ? (void *)(per_block_obj + block0) : nullptr;
                block0 += (size_t)(t.rows / M) * (size_t)(t.cols / M);
                tile0[k] = tiles;
                args.m[k].pad = tiles_of(args.m[k].n_strips);
                sums.add(args.m[k].pad, true);
                tiles += args.m[k].pad;
            }
            tile0[nb] = tiles;
            fill_coarse(args.ci, tile0, nb, tiles);
            args.n_mats = (uint32_t)nb; args.K = (uint32_t)(M - N); args.N = (uint32_t)N;
            args.partial0 = partial0; args.partials = workspace;
            static_assert(sizeof(ScorePartial) == sizeof(tmask_score_out), "the last workgroup of a matrix writes its result");
            args.score = (ScorePartial *)(out + first);
            one_launch = adds_up_itself(sums, kThreads, true);
            if (one_launch)
                args.tags = draw_tags();
            {
                ProfileScope prof(stream, first + kMaxBatch >= n_mats);
                launch_kernel(kernel, dim3(tiles), dim3(kThreads), 0, stream, args);
            }
            const hipError_t e = hipGetLastError();
            return e == hipSuccess ? TMASK_OK : hip_fail(e, "score kernel launch");
        });
        if (rc)
            return rc;
        if (!one_launch && (rc = launch_score_reduce(tile0, nb, partial0, workspace, out + first, stream)))
            return rc;
        partial0 += tiles;
    }
    return TMASK_OK;
}

typedef void (*pack_kernel_t)(const PackArgs);
typedef void (*few_pack_kernel_t)(const FewPackArgs);

int tmask_apply_pack(const tmask_pack_desc *descs, int n, tmask_dtype dt, int N, int M, tmask_mask_fmt mf,
                     void *workspace, size_t workspace_bytes, void *hip_stream)
{
    (void)workspace; (void)workspace_bytes;   // this call needs no scratch memory
    int rc = check_common(descs, n, (int)dt, N, M, (int)mf);
    if (rc)
        return rc;
    // M = 32: the tiled kernel at 16:32 (a tile row's position bits are then whole bytes), the column-per-lane one else
    Fit fit = (M != 32) || (N == 16) ? kFitWide : kFitColumns;
    for (int i = 0; i < n; i++) {
        const tmask_pack_desc &p = descs[i];
        const HostMat h{p.w, p.rows, p.cols, p.ld, const_cast<void *>(p.mask), p.mask_ld, nullptr};
        if ((rc = check_mat(h, i, (int)dt, M, (int)mf, true, &fit)))
            return rc;
        if (!p.vals || !p.idx || !p.valsT || !p.idxT)
            return fail(TMASK_ERR_NULL, "matrix %d: a packed output pointer is NULL", i);
        if (((uintptr_t)p.vals | (uintptr_t)p.valsT) % elem_size((int)dt))
            return fail(TMASK_ERR_ALIGN, "matrix %d: vals and valsT must be aligned to the element size", i);
        if (((uintptr_t)p.vals & 3) || ((uintptr_t)p.valsT & 3))
            fit = kFitColumns;
        if (M == 32 && ((uintptr_t)p.vals & 15))     // its row groups leave as 16-byte stores only
            fit = kFitColumns;
    }
    const bool narrow24 = fit == kFitNarrow && N == 2;           // the only kernel with narrow strips
    if (fit != kFitWide && !narrow24)
        return cw_run_pack(descs, n, (int)dt, N, M, (int)mf, (hipStream_t)hip_stream);
    pack_kernel_t kern = pick_pack_kernel<kThreads, PackArgs>((int)dt, M, (int)mf, N);
    few_pack_kernel_t few = nullptr;      // of kern, where it has one
    uint32_t TC = 256 / (uint32_t)elem_size((int)dt);
    bool fast24 = (M == 4 && N == 2) && !narrow24;
    for (int i = 0; i < n && fast24; i++)
        fast24 = (((uintptr_t)descs[i].vals | (uintptr_t)descs[i].valsT) & 7) == 0;
    uint32_t TR = kPackTR, lds_reserve = 0, threads = kThreads;
    if (n <= kFewMats && few_tiles(descs, n, TR, TC, kWideTilesPack)) {
        few = pick_pack_kernel<kPackThreads, FewPackArgs>((int)dt, M, (int)mf, N);
        threads = kPackThreads;
    }
    if (fast24) {
        // tile widths in strips: measured best per element type (bf16: narrower and taller, so the runs written
        // per column of W^T are 128 bytes long)
        constexpr int SF = 64, SB = 32;
        // four wavefronts working through four block-rows each (eight with two each halves the time a tile stays
        // resident, and measured the same within 1 % at fp32, 8 % slower at bf16)
        constexpr int NW = 4;
        const uint32_t strips = dt == TMASK_F32 ? SF : SB;
        TC = strips * 16 / (uint32_t)elem_size((int)dt);
        TR = 4 * 4 * (64 / strips) * NW;
        const bool small = few_tiles(descs, n, TR, TC, kHalfTilesPack);
#define TMASK_PICK(DT, SS, FM, QN) \
        if ((int)dt == DT && (int)mf == FM && small == (QN == 2)) { kern = pack24_kernel<DT, FM, SS, NW, QN>; few = pack24_kernel<DT, FM, SS, NW, QN, FewPackArgs>; }
        TMASK_PICK(kF32, SF, kMaskU8, 4) TMASK_PICK(kF32, SF, kMaskBits, 4) TMASK_PICK(kBF16, SB, kMaskU8, 4) TMASK_PICK(kBF16, SB, kMaskBits, 4)
        TMASK_PICK(kF32, SF, kMaskU8, 2) TMASK_PICK(kF32, SF, kMaskBits, 2) TMASK_PICK(kBF16, SB, kMaskU8, 2) TMASK_PICK(kBF16, SB, kMaskBits, 2)
#undef TMASK_PICK
        TR = small ? TR / 2 : TR;
        threads = 64 * NW;
        lds_reserve = dt == TMASK_F32 && !small ? kPack4LdsReservePackF32 : 0;
        if (n <= kFewMats && few_tiles(descs, n, 2 * TR, TC, kQuarterTilesPack)) {
#define TMASK_PICK(DT, FM) \
            if ((int)dt == DT && (int)mf == FM) few = pack24_kernel<DT, FM, kPack4Quarter, NW, 1, FewPackArgs>;
            TMASK_PICK(kF32, kMaskU8) TMASK_PICK(kF32, kMaskBits) TMASK_PICK(kBF16, kMaskU8) TMASK_PICK(kBF16, kMaskBits)
#undef TMASK_PICK
            TC = kPack4Quarter * 16 / (uint32_t)elem_size((int)dt);
            TR = Pack4Geo<kF32, kPack4Quarter, NW, 1>::TR;
        }
    }
    if (narrow24) {
        // 8-byte strips, which write 4 bytes per row: tiles of 64 rows x 128 columns, a quarter of the others' bytes, since
        // such matrices are mostly small (1000 x 2052: 272 workgroups)
        kern = mf == TMASK_MASK_U8 ? pack24_kernel<kBF16N, kMaskU8, 32, 4, 2> : pack24_kernel<kBF16N, kMaskBits, 32, 4, 2>;
        few = mf == TMASK_MASK_U8 ? pack24_kernel<kBF16N, kMaskU8, 32, 4, 2, FewPackArgs> : pack24_kernel<kBF16N, kMaskBits, 32, 4, 2, FewPackArgs>;
        using PG = Pack4Geo<kBF16N, 32, 4, 2>;
        TC = PG::TC;
        TR = PG::TR;
        threads = PG::NT;
        if (n <= kFewMats && few_tiles(descs, n, TR, TC, kQuarterTilesNarrow)) {
            few = mf == TMASK_MASK_U8 ? pack24_kernel<kBF16N, kMaskU8, 32, 4, 1, FewPackArgs> : pack24_kernel<kBF16N, kMaskBits, 32, 4, 1, FewPackArgs>;
            TR = Pack4Geo<kBF16N, 32, 4, 1>::TR;
        }
    }
    bool fast48 = (M == 8 && N == 4 && dt == TMASK_BF16);
    for (int i = 0; i < n && fast48; i++)
        fast48 = (((uintptr_t)descs[i].vals | (uintptr_t)descs[i].valsT) & 7) == 0;
    if (fast48) {
        const bool small = few_tiles(descs, n, Pack8Geo<2>::TR, Pack8Geo<2>::TC, kHalfTilesPack);
#define TMASK_PICK(FM, ST) \
        if ((int)mf == FM && small == (ST == 1)) { \
            kern = pack48_bf16_kernel<FM, false, false, PackArgs, ST>; \
            few = pack48_bf16_kernel<FM, false, false, FewPackArgs, ST>; \
        }
        TMASK_PICK(kMaskU8, 1) TMASK_PICK(kMaskU8, 2) TMASK_PICK(kMaskBits, 1) TMASK_PICK(kMaskBits, 2)
#undef TMASK_PICK
        TC = Pack8Geo<2>::TC;
        TR = small ? Pack8Geo<1>::TR : Pack8Geo<2>::TR;
        threads = kThreads;
    }
    bool fast48f = (M == 8 && N == 4 && dt == TMASK_F32);
    for (int i = 0; i < n && fast48f; i++)
        fast48f = (((uintptr_t)descs[i].vals | (uintptr_t)descs[i].valsT) & 7) == 0;
    if (fast48f) {
        constexpr int SW = kPack8F32Strips, SH = kPack8F32Half;
        const bool small = few_tiles(descs, n, Pack8F32Geo<SW>::TR, Pack8F32Geo<SW>::TC, kHalfTilesPack);
#define TMASK_PICK(FM, SS, QN) \
        if ((int)mf == FM && small == (QN == 1)) { \
            kern = pack48_f32_kernel<FM, SS, false, false, PackArgs, QN>; \
            few = pack48_f32_kernel<FM, SS, false, false, FewPackArgs, QN>; \
        }
        TMASK_PICK(kMaskU8, SH, 1) TMASK_PICK(kMaskU8, SW, 2) TMASK_PICK(kMaskBits, SH, 1) TMASK_PICK(kMaskBits, SW, 2)
#undef TMASK_PICK
        TC = small ? Pack8F32Geo<SH, 1>::TC : Pack8F32Geo<SW>::TC;
        TR = small ? Pack8F32Geo<SH, 1>::TR : Pack8F32Geo<SW>::TR;
        threads = kThreads;
    }
    hipStream_t stream = (hipStream_t)hip_stream;
    for (int first = 0; first < n; first += kMaxPackBatch) {
        const int nb = n - first < kMaxPackBatch ? n - first : kMaxPackBatch;
        auto go = [&](auto &args, auto kernel) -> int {
            memset(&args, 0, sizeof args);
            uint32_t tiles = 0;
            for (int k = 0; k < nb; k++) {
                const tmask_pack_desc &p = descs[first + k];
                PackDev &d = args.d[k];
                d.w = p.w; d.mask = p.mask; d.vals = p.vals; d.idx = p.idx; d.valsT = p.valsT; d.idxT = p.idxT;
                d.rows = (uint32_t)p.rows; d.cols = (uint32_t)p.cols; d.ld = (uint32_t)p.ld; d.mask_ld = (uint32_t)p.mask_ld;
                d.tiles_x = (d.cols + TC - 1) / TC;
                d.tile0 = tiles;
                tiles += d.tiles_x * ((d.rows + TR - 1) / TR);
            }
            {
                uint32_t first0[kMaxPackBatch + 1];
                for (int k = 0; k < nb; k++)
                    first0[k] = args.d[k].tile0;
                first0[nb] = tiles;
                fill_coarse(args.ci, first0, nb, tiles);
            }
            args.n = (uint32_t)nb; args.N = (uint32_t)N;
            {
                ProfileScope prof(stream, first + kMaxPackBatch >= n);
                launch_kernel(kernel, dim3(tiles), dim3(threads), lds_reserve, stream, args);
            }
            const hipError_t e = hipGetLastError();
            return e == hipSuccess ? TMASK_OK : hip_fail(e, "pack kernel launch");
        };
        if (few && nb <= kFewMats) {
            FewPackArgs args;
            rc = go(args, few);
        } else {
            PackArgs args;
            rc = go(args, kern);
        }
        if (rc)
            return rc;
    }
    return TMASK_OK;
}

int tmask_approx_pack(const tmask_fused_desc *descs, int n, tmask_dtype dt, int N, int M, tmask_mask_fmt mf,
                      void *workspace, size_t workspace_bytes, void *hip_stream)
{
    int rc = check_common(descs, n, (int)dt, N, M, (int)mf);
    if (rc)
        return rc;
    bool fused24 = (M == 4 && N == 2);                         // both need aligned inputs and 8-byte aligned outputs,
    bool fused48 = (M == 8 && N == 4);                         // else the call runs as two steps
    int with_mask = 0;
    bool want_obj = false;
    Fit fit = fit_at_best(M);
    for (int i = 0; i < n; i++) {
        const tmask_fused_desc &p = descs[i];
        with_mask += p.mask ? 1 : 0;
        want_obj = want_obj || p.objective;
        const HostMat h{p.w, p.rows, p.cols, p.ld, p.mask, p.mask_ld, p.objective};
        if ((rc = check_mat(h, i, (int)dt, M, (int)mf, p.mask != nullptr, &fit)))
            return rc;
        if (!p.vals || !p.idx || !p.valsT || !p.idxT)
            return fail(TMASK_ERR_NULL, "matrix %d: a packed output pointer is NULL", i);
        if (((uintptr_t)p.vals | (uintptr_t)p.valsT) % elem_size((int)dt))
            return fail(TMASK_ERR_ALIGN, "matrix %d: vals and valsT must be aligned to the element size", i);
        const bool out8 = ((((uintptr_t)p.vals | (uintptr_t)p.valsT) & 7) == 0);
        fused24 = fused24 && out8;
        fused48 = fused48 && out8;
    }
    const bool fused = fit == kFitWide && (fused24 || fused48);
    if (with_mask != 0 && with_mask != n)
        return fail(TMASK_ERR_NULL, "mask must be given for all matrices or for none (%d of %d have one)", with_mask, n);
    if (!fused && with_mask == 0)
        return fail(TMASK_ERR_NULL, "this call (N:M = %d:%d, or matrices / outputs that miss the alignment of the one-pass "
                                    "kernels) runs as two steps and needs the mask buffers", N, M);

    if (!fused) {
        std::vector<tmask_mat> mats((size_t)n);
        std::vector<tmask_pack_desc> pds((size_t)n);
        for (int i = 0; i < n; i++) {
            const tmask_fused_desc &p = descs[i];
            mats[i] = tmask_mat{p.w, p.rows, p.cols, p.ld, p.mask, p.mask_ld, p.objective};
            pds[i] = tmask_pack_desc{p.w, p.rows, p.cols, p.ld, p.mask, p.mask_ld, p.vals, p.idx, p.valsT, p.idxT};
        }
        if ((rc = run_mask<kSolveApprox>(mats.data(), n, (int)dt, N, M, (int)mf, workspace, workspace_bytes, hip_stream)))
            return rc;
        return tmask_apply_pack(pds.data(), n, dt, N, M, mf, workspace, workspace_bytes, hip_stream);
    }

    // tile shapes as in tmask_apply_pack
    constexpr int SF = 64, SB = 32;
    const uint32_t strips = dt == TMASK_F32 ? SF : SB;
    using G8F = Pack8F32Geo<kPack8F32Strips>;
    uint32_t TC = fused48 ? (dt == TMASK_F32 ? (uint32_t)G8F::TC : (uint32_t)Pack8Geo<2>::TC)
                                : strips * 16 / (uint32_t)elem_size((int)dt);
    uint32_t kPack4Rows = !fused48 ? 4096 / strips : dt == TMASK_F32 ? (uint32_t)G8F::TR : (uint32_t)Pack8Geo<2>::TR;
    auto partials_bytes = [&](uint32_t tile_rows, uint32_t tile_cols) {
        size_t tiles = 0;
        for (int i = 0; i < n; i++)
            tiles += (size_t)((descs[i].cols + tile_cols - 1) / tile_cols) * (size_t)((descs[i].rows + tile_rows - 1) / tile_rows);
        return tiles * sizeof(double);
    };
    // half tiles leave more partial sums than the workspace was asked to hold: only where it happens to
    const bool f48 = fused48 && dt == TMASK_F32;
    const uint32_t half_rows = f48 ? (uint32_t)Pack8F32Geo<kPack8F32Half, 1>::TR : kPack4Rows / 2, half_cols = f48 ? (uint32_t)Pack8F32Geo<kPack8F32Half, 1>::TC : TC;
    const bool small = few_tiles(descs, n, kPack4Rows, TC, f48 ? kHalfTilesFusedF32M8 : dt == TMASK_F32 ? kHalfTilesFusedF32 : kHalfTilesFusedBf16) &&
                       (!want_obj || workspace_bytes >= partials_bytes(half_rows, half_cols));
    const uint32_t quarter_rows = Pack4Geo<kF32, kPack4Quarter, 4, 1>::TR, quarter_cols = kPack4Quarter * 16 / (uint32_t)elem_size((int)dt);
    const bool quarter = fused24 && small && few_tiles(descs, n, kPack4Rows, TC, kQuarterTilesFused) && (!want_obj || workspace_bytes >= partials_bytes(quarter_rows, quarter_cols));
    if (small) {
        kPack4Rows = quarter ? quarter_rows : half_rows;
        TC = quarter ? quarter_cols : half_cols;
    }
    if (want_obj) {
        if (!workspace || ((uintptr_t)workspace & 255))
            return fail(TMASK_ERR_WORKSPACE, "workspace is NULL or not 256-byte aligned");
        const size_t need = partials_bytes(kPack4Rows, TC);
        if (workspace_bytes < need)
            return fail(TMASK_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes, need);
    }
    typedef void (*fused_kernel_t)(const FusedArgs);
    fused_kernel_t kern = nullptr;
#define TMASK_PICK(DT, FM, SS, QN) \
    if ((int)dt == DT && (int)mf == FM && small == (QN == 2)) \
        kern = with_mask ? approx_pack24_kernel<DT, FM, true, SS, QN> : approx_pack24_kernel<DT, FM, false, SS, QN>;
    TMASK_PICK(kF32, kMaskU8, SF, 4) TMASK_PICK(kF32, kMaskBits, SF, 4) TMASK_PICK(kBF16, kMaskU8, SB, 4) TMASK_PICK(kBF16, kMaskBits, SB, 4)
    TMASK_PICK(kF32, kMaskU8, SF, 2) TMASK_PICK(kF32, kMaskBits, SF, 2) TMASK_PICK(kBF16, kMaskU8, SB, 2) TMASK_PICK(kBF16, kMaskBits, SB, 2)
#undef TMASK_PICK
#define TMASK_PICK(DT, FM) \
    if (quarter && (int)dt == DT && (int)mf == FM) \
        kern = with_mask ? approx_pack24_kernel<DT, FM, true, kPack4Quarter, 1> : approx_pack24_kernel<DT, FM, false, kPack4Quarter, 1>;
    TMASK_PICK(kF32, kMaskU8) TMASK_PICK(kF32, kMaskBits) TMASK_PICK(kBF16, kMaskU8) TMASK_PICK(kBF16, kMaskBits)
#undef TMASK_PICK
    if (f48) {
#define TMASK_PICK(FM, SS, QN) \
        if ((int)mf == FM && small == (QN == 1)) \
            kern = with_mask ? pack48_f32_kernel<FM, SS, true, true, FusedArgs, QN> : pack48_f32_kernel<FM, SS, true, false, FusedArgs, QN>;
        TMASK_PICK(kMaskU8, kPack8F32Half, 1) TMASK_PICK(kMaskU8, kPack8F32Strips, 2)
        TMASK_PICK(kMaskBits, kPack8F32Half, 1) TMASK_PICK(kMaskBits, kPack8F32Strips, 2)
#undef TMASK_PICK
    } else if (fused48) {
#define TMASK_PICK(FM, ST) \
        if ((int)mf == FM && small == (ST == 1)) \
            kern = with_mask ? pack48_bf16_kernel<FM, true, true, FusedArgs, ST> : pack48_bf16_kernel<FM, true, false, FusedArgs, ST>;
        TMASK_PICK(kMaskU8, 1) TMASK_PICK(kMaskU8, 2) TMASK_PICK(kMaskBits, 1) TMASK_PICK(kMaskBits, 2)
#undef TMASK_PICK
    }
    hipStream_t stream = (hipStream_t)hip_stream;
    uint32_t partial0 = 0;
    for (int first = 0; first < n; first += kMaxPackBatch) {
        const int nb = n - first < kMaxPackBatch ? n - first : kMaxPackBatch;
        FusedArgs args;
        ReduceArgs rargs;
        memset(&args, 0, sizeof args);
        memset(&rargs, 0, sizeof rargs);
        uint32_t tiles = 0;
        LaunchSums sums;
        for (int k = 0; k < nb; k++) {
            const tmask_fused_desc &p = descs[first + k];
            PackDev &d = args.d[k];
            d.w = p.w; d.mask = p.mask; d.vals = p.vals; d.idx = p.idx; d.valsT = p.valsT; d.idxT = p.idxT;
            d.rows = (uint32_t)p.rows; d.cols = (uint32_t)p.cols; d.ld = (uint32_t)p.ld; d.mask_ld = (uint32_t)p.mask_ld;
            d.tiles_x = (d.cols + TC - 1) / TC;
            d.tile0 = tiles;
            rargs.objective[k] = p.objective;
            rargs.tile0[k] = tiles;
            if (k < kFewMats)
                args.objective[k] = p.objective;
            const uint32_t own = d.tiles_x * ((d.rows + kPack4Rows - 1) / kPack4Rows);
            sums.add(own, p.objective);
            tiles += own;
        }
        rargs.tile0[nb] = tiles;
        fill_coarse(args.ci, rargs.tile0, nb, tiles);
        args.n = (uint32_t)nb; args.partial0 = partial0; args.partials = want_obj ? workspace : nullptr;
        // a pointer for each of 224 matrices would be 2 KB of arguments more, which calls without objectives pay for too (512^2
        // fp32 2:4 6.18 us with them, 6.04 without)
        const bool one_launch = want_obj && nb <= kFewMats && adds_up_itself(sums, kThreads, false) && workspace_bytes >= 2 * partials_bytes(kPack4Rows, TC);
        if (one_launch)
            args.tags = draw_tags();
        {
            ProfileScope prof(stream, first + kMaxPackBatch >= n);
            hipLaunchKernelGGL(kern, dim3(tiles), dim3(kThreads), (fused24 && dt == TMASK_F32 && !small) ? kPack4LdsReserveFusedF32 : 0, stream,
                               args);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return hip_fail(e, "fused approx+pack kernel launch");
        if (want_obj && !one_launch) {
            rargs.n_mats = (uint32_t)nb; rargs.partial0 = partial0; rargs.partials = (const double *)workspace;
            enqueue_objective_reduce(rargs, nb, stream);
            e = hipGetLastError();
            if (e != hipSuccess)
                return hip_fail(e, "objective reduce launch");
        }
        partial0 += tiles;
    }
    return TMASK_OK;
}

static int run_mask_dense(const tmask_mask_dense_desc *descs, int n, tmask_dtype dt, int N, int M, tmask_mask_fmt mf,
                          int mode, void *hip_stream)
{
    int rc = check_common(descs, n, (int)dt, N, M, (int)mf);
    if (rc)
        return rc;
    const int64_t es = elem_size((int)dt);
    int with_mask = 0;
    Fit fit = fit_at_best(M);
    for (int i = 0; i < n; i++) {
        const tmask_mask_dense_desc &p = descs[i];
        with_mask += p.mask ? 1 : 0;
        const HostMat h{p.w, p.rows, p.cols, p.ld, p.mask, p.mask_ld, nullptr};
        if ((rc = check_mat(h, i, (int)dt, M, (int)mf, p.mask != nullptr, &fit)))
            return rc;
        if (!p.out)
            return fail(TMASK_ERR_NULL, "matrix %d: out is NULL", i);
        if (p.ld_out < p.cols || p.ld_out * es > 0x7FFFFFFFll)
            return fail(TMASK_ERR_SHAPE, "matrix %d: ld_out=%lld must cover a row of %lld columns", i, (long long)p.ld_out,
                        (long long)p.cols);
        if ((uintptr_t)p.out % (uintptr_t)es)
            return fail(TMASK_ERR_ALIGN, "matrix %d: out must be aligned to its element size", i);
        lower_fit(&fit, (uint64_t)(uintptr_t)p.out | (uint64_t)(p.ld_out * es), 16, dt == TMASK_BF16 && M == 4);
    }
    if (with_mask != 0 && with_mask != n)
        return fail(TMASK_ERR_NULL, "mask must be given for all matrices or for none (%d of %d have one)", with_mask, n);
    if (fit == kFitColumns) {
        const bool absorb = mode == kDenseRow1DAbsorb || mode == kDenseRow1DHalfAbsorb;
        const bool rows_only = absorb || mode == kDenseRow1D || mode == kDenseRow1DHalf;
        return cw_run_dense(descs, n, (int)dt, N, M, (int)mf, absorb ? 2 : rows_only ? 1 : 0, (hipStream_t)hip_stream);
    }
    const int sdt = strip_type((int)dt, fit);
    BatchKernel kern{nullptr, nullptr};
#define TMASK_PICK(DT, MM, FM) \
    if (sdt == DT && M == MM && (int)mf == FM) \
        kern = mode == kDenseApprox ? TMASK_MANY(approx_dense_kernel, DT, MM, FM, kDenseApprox, BatchArgs) \
             : mode == kDenseApproxHalf ? TMASK_BOTH(approx_dense_kernel, DT, MM, FM, kDenseApproxHalf) \
             : mode == kDenseRow1D ? TMASK_MANY(approx_dense_kernel, DT, MM, FM, kDenseRow1D, BatchArgs) \
             : mode == kDenseRow1DAbsorb ? TMASK_MANY(approx_dense_kernel, DT, MM, FM, kDenseRow1DAbsorb, BatchArgs) : kern;
    TMASK_PICK(kF32, 4, kMaskU8) TMASK_PICK(kF32, 8, kMaskU8) TMASK_PICK(kF32, 16, kMaskU8)
    TMASK_PICK(kBF16, 4, kMaskU8) TMASK_PICK(kBF16, 8, kMaskU8) TMASK_PICK(kBF16, 16, kMaskU8)
    TMASK_PICK(kF32, 4, kMaskBits) TMASK_PICK(kF32, 8, kMaskBits) TMASK_PICK(kF32, 16, kMaskBits)
    TMASK_PICK(kBF16, 4, kMaskBits) TMASK_PICK(kBF16, 8, kMaskBits) TMASK_PICK(kBF16, 16, kMaskBits)
    TMASK_PICK(kBF16N, 4, kMaskU8) TMASK_PICK(kBF16N, 4, kMaskBits)
#undef TMASK_PICK
#define TMASK_PICK(MM, FM) \
    if ((int)dt == kBF16 && M == MM && (int)mf == FM && mode >= kDenseRow1DHalf) \
        kern = mode == kDenseRow1DHalf ? TMASK_MANY(approx_dense_kernel, kBF16, MM, FM, kDenseRow1DHalf, BatchArgs) \
                                       : TMASK_MANY(approx_dense_kernel, kBF16, MM, FM, kDenseRow1DHalfAbsorb, BatchArgs);
    TMASK_PICK(8, kMaskU8) TMASK_PICK(16, kMaskU8) TMASK_PICK(8, kMaskBits) TMASK_PICK(16, kMaskBits)
#undef TMASK_PICK
    uint32_t unit_split = 1;
    if (M == 16 && dt == TMASK_BF16 && n <= kFewMats && (mode == kDenseApprox || mode == kDenseApproxHalf)) {
        uint64_t wgs = 0;
        for (int i = 0; i < n; i++)
            wgs += (uint64_t)(descs[i].rows / M * descs[i].cols + kThreads - 1) / kThreads;
        if (wgs <= spread_approx16(true, N) * (uint64_t)cu_count()) {
            kern.few = mf == TMASK_MASK_U8 ? approx_spread16_kernel<kMaskU8, true, FewArgs> : approx_spread16_kernel<kMaskBits, true, FewArgs>;
            unit_split = (uint32_t)strip_cols(sdt);
        }
    }
    hipStream_t stream = (hipStream_t)hip_stream;
    for (int first = 0; first < n; first += kMaxBatch) {
        const int nb = n - first < kMaxBatch ? n - first : kMaxBatch;
        rc = with_table(kern, nb, [&](auto &args, auto kernel) -> int {
            uint32_t tiles = 0;
            for (int k = 0; k < nb; k++) {
                const tmask_mask_dense_desc &p = descs[first + k];
                const HostMat h{p.w, p.rows, p.cols, p.ld, p.mask, p.mask_ld, nullptr};
                fill_desc(args.m[k], h, sdt, M, tiles);
                args.m[k].aux = p.out;
                args.m[k].pad = (uint32_t)p.ld_out;
                tiles += tiles_of(args.m[k].n_strips * unit_split);
            }
            {
                uint32_t first0[kMaxBatch + 1];
                for (int k = 0; k < nb; k++)
                    first0[k] = args.m[k].tile0;
                first0[nb] = tiles;
                fill_coarse(args.ci, first0, nb, tiles);
            }
            args.n_mats = (uint32_t)nb; args.K = (uint32_t)(M - N); args.N = (uint32_t)N;
            {
                ProfileScope prof(stream, first + kMaxBatch >= n);
                launch_kernel(kernel, dim3(tiles), dim3(kThreads), 0, stream, args);
            }
            const hipError_t e = hipGetLastError();
            return e == hipSuccess ? TMASK_OK : hip_fail(e, "mask + dense copy kernel launch");
        });
        if (rc)
            return rc;
    }
    return TMASK_OK;
}

int tmask_approx_dense(const tmask_mask_dense_desc *descs, int n, tmask_dtype dt, int N, int M, tmask_mask_fmt mf,
                       void *hip_stream)
{
    return run_mask_dense(descs, n, dt, N, M, mf, 2 * N == M ? kDenseApproxHalf : kDenseApprox, hip_stream);
}

int tmask_prune_1d_dense(const tmask_mask_dense_desc *descs, int n, tmask_dtype dt, int N, int M, int absorb_mean,
                         tmask_mask_fmt mf, void *hip_stream)
{
    const bool half = dt == TMASK_BF16 && M >= 8 && 2 * N == M;
    const int mode = half ? (absorb_mean ? kDenseRow1DHalfAbsorb : kDenseRow1DHalf)
                          : (absorb_mean ? kDenseRow1DAbsorb : kDenseRow1D);
    return run_mask_dense(descs, n, dt, N, M, mf, mode, hip_stream);
}

size_t tmask_workspace_bytes(const tmask_mat *mats, int n_mats, int N, int M)
{
    if (!mats || n_mats <= 0 || !valid_nm(N, M))
        return 0;
    return workspace_need(mats, n_mats, M);
}

int tmask_profile_next(void *start_event, void *stop_event)
{
    g_prof_start = (hipEvent_t)start_event;
    g_prof_stop = (hipEvent_t)stop_event;
    return TMASK_OK;
}

const char *tmask_last_error(void) { return g_err; }

int tmask_version(void) { return 100; }

}  // extern "C"
