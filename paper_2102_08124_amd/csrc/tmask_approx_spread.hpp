// Algorithm 1 for bf16 at M = 16, any N, in calls that leave the chip idle: a column of a block per lane.
//
// The strip kernels hold 16 x 8 entries in a lane and find 16 + 8 thresholds one after the other, 2000 instructions; a call of a few
// hundred blocks lasts that long.  Here a lane finds two, of its column and, through LDS, of a row (91 instructions each).  The rule
// is that of approx_half_bf16: keys |w| << 16 | position, kept iff not among the K smallest of its row or of its column.
#pragma once
#include "tmask_column.hpp"
#include "tmask_device.hpp"
#include "tmask_networks.hpp"

namespace tmask {

// Bit i: entry i of sixteen magnitudes (bf16, in the upper half of a word) is not among the K first of the (magnitude, position) order.
__device__ __forceinline__ uint32_t kept_of_16(const uint32_t (&mag)[16], uint32_t K)
{
    uint32_t k[16], srt[16];
#pragma unroll
    for (int i = 0; i < 16; i++)
        srt[i] = k[i] = mag[i] | (uint32_t)i;
    sort_asc<16>(srt);
    const uint32_t t = srt[K & 15u];                              // K is the same in every lane
    uint32_t w = 0u;
#pragma unroll
    for (int i = 15; i >= 0; i--)
        lm_shift_in(w, lm(k[i] >= t));
    return w;
}

// DENSE: the masked copy to md.aux, of leading dimension md.pad, and a mask if there is one; else the mask, and the kept sum.
template <int FMT, bool DENSE, typename Args, int NT = kThreads>
__global__ __launch_bounds__(NT, NT > kThreads ? 6 : 1) void approx_spread16_kernel(const Args args)
{
    constexpr int M = 16, kWaves = NT / 64;
    using Ge = Geo<kBF16, M>;
    __shared__ uint32_t lds[kWaves][4][M][M + 1];                 // the magnitudes of a wavefront's blocks, for their rows
    __shared__ double red[kWaves];
    const uint32_t tile = blockIdx.x;
    const MatDev md = args.m[find_matrix(args, tile)];
    Handover out = {};
    if constexpr (!DENSE)
        out = objective_of(args, md, tile);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, j = lane % M, blk = lane / M;
    const ColumnPos pos = column_pos<Ge::C>(md, (tile - md.tile0) * NT + tid);
    uint32_t raw[M], mag[M];
    if (pos.valid) {
        const char *base = (const char *)md.w + ((size_t)pos.br * M * md.ld + pos.col) * 2;
#pragma unroll
        for (int i = 0; i < M; i++)
            raw[i] = __builtin_nontemporal_load((const uint16_t *)(base + (size_t)i * md.ld * 2));
    } else {
#pragma unroll
        for (int i = 0; i < M; i++)
            raw[i] = 0u;
    }
    auto &T = lds[tid >> 6][blk];
#pragma unroll
    for (int i = 0; i < M; i++) {
        mag[i] = (raw[i] & 0x7FFFu) << 16;
        T[i][j] = mag[i];
    }
    uint32_t kept = kept_of_16(mag, args.K);
    __builtin_amdgcn_wave_barrier();                              // LDS accesses of a wavefront happen in program order
    asm volatile("" ::: "memory");
    {
        uint32_t row[M];
#pragma unroll
        for (int c = 0; c < M; c++)
            row[c] = T[j][c];
        kept &= transposed_bits<M>(kept_of_16(row, args.K));
    }
    if (!DENSE || md.mask)
        store_column<M, FMT>(md, pos, kept);
    if constexpr (DENSE) {
        if (pos.valid) {
            char *base = (char *)md.aux + ((size_t)pos.br * M * md.pad + pos.col) * 2;
#pragma unroll
            for (int i = 0; i < M; i++)
                *(uint16_t *)(base + (size_t)i * md.pad * 2) = (uint16_t)((kept >> i) & 1u ? raw[i] : 0u);
        }
    } else if (out.dst) {
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < M; i++)
            acc += (kept >> i) & 1u ? __uint_as_float(mag[i]) : 0.f;
        hand_over<NT>(out, block_sum_f32<kF32, NT>(acc, red), red);
    }
}

}  // namespace tmask
