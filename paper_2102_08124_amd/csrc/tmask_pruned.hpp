// Algorithm 1's choice in one line (a row or a column of a block) whose M magnitudes a lane holds.
#pragma once
#include "tmask_device.hpp"
#include "tmask_networks.hpp"

namespace tmask {

// the (K+1)-th smallest of M keys (1 <= K <= M - 1; the keys may repeat).  M = 32: two halves of 16 sorted by network,
// for K = 16 the minimum over i of max(a_i, b_15-i), for any other K a bitonic merge and a register read at an index
// that is the same in every lane.  M <= 16: one sorting network and that register read.
template <int M>
__device__ __forceinline__ uint32_t threshold_of_line(const uint32_t (&k)[M], uint32_t K)
{
    if constexpr (M == 32) {
        uint32_t a[16], b[16];
#pragma unroll
        for (int i = 0; i < 16; i++) {
            a[i] = k[i];
            b[i] = k[16 + i];
        }
        sort_asc<16>(a);
        sort_asc<16>(b);
        uint32_t t;
        if (K == 16u) {
            t = 0xFFFFFFFFu;
#pragma unroll
            for (int i = 0; i < 16; i++) {
                const uint32_t m = a[i] > b[15 - i] ? a[i] : b[15 - i];
                t = m < t ? m : t;
            }
        } else {
            uint32_t s[32];
#pragma unroll
            for (int i = 0; i < 16; i++) {
                s[i] = a[i];
                s[16 + i] = b[15 - i];
            }
            bitonic_merge_asc<32>(s);
            t = s[__builtin_amdgcn_readfirstlane(K) & 31u];
        }
        return t;
    } else {
        uint32_t s[M];
#pragma unroll
        for (int i = 0; i < M; i++)
            s[i] = k[i];
        sort_asc<M>(s);
        return s[__builtin_amdgcn_readfirstlane(K) & (uint32_t)(M - 1)];
    }
}

// M magnitudes held by one lane: bit i of the result is set when entry i is among the first K of the (magnitude,
// position) order, i.e. pruned: the entries below the (K+1)-th smallest key.  bf16 keys carry the position in their low
// bits (15 + 5 bits), so they are distinct.  fp32 magnitudes are compared as they are; if the threshold value occurs
// on both sides of the cut, fewer than K entries lie below it and the missing ones are the entries equal to it at the
// lowest positions (a wavefront-uniform detour).  At M = 32: 350-550 instructions against 1500 for pairwise ranks.
template <int DT, int M>
__device__ __forceinline__ uint32_t pruned_of_line(const uint32_t (&mag)[M], uint32_t K)
{
    uint32_t k[M];
#pragma unroll
    for (int i = 0; i < M; i++)
        k[i] = DT == kF32 ? mag[i] : ((mag[i] >> 11) | (uint32_t)i);
    const uint32_t t = threshold_of_line<M>(k, K);
    uint32_t w = 0;
#pragma unroll
    for (int i = M - 1; i >= 0; i--)
        lm_shift_in(w, lm(k[i] < t));
    if constexpr (DT == kF32) {
        const uint32_t lt = (uint32_t)__builtin_popcount(w);
        if (lm(lt != K) != 0) {
            uint32_t eq = 0;
#pragma unroll
            for (int i = M - 1; i >= 0; i--)
                lm_shift_in(eq, lm(k[i] == t));
            uint32_t q = K - lt;
            while (lm(q != 0u) != 0) {
                const uint32_t low = q != 0u ? (eq & (0u - eq)) : 0u;
                w |= low;
                eq ^= low;
                q -= q != 0u ? 1u : 0u;
            }
        }
    }
    return w;
}

}  // namespace tmask
