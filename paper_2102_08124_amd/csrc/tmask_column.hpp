// Kernels with a column of a block per lane, for calls that leave the chip idle: a workgroup takes 256 or 512 columns (its threads) of
// the block-rows, one after the other, and M neighbouring lanes hold a block.
#pragma once
#include <type_traits>

#include "tmask_device.hpp"

namespace tmask {

struct ColumnPos {
    uint32_t br;      // block-row
    size_t col;
    bool valid;       // inside the matrix; a block's lanes all are, or none
};

// Column number u of the matrix' block-rows, counted in strips of C columns.
template <int C>
__device__ __forceinline__ ColumnPos column_pos(const MatDev &md, uint32_t u)
{
    const uint32_t s = u / C;
    const StripPos p = strip_pos(md, s);
    return ColumnPos{p.br, (size_t)p.sc * C + u % C, s < md.n_strips};
}

// An M x M bit matrix held as one word per lane (lane l, bit i) -> its transpose (lane i, bit l): quarters off the diagonal
// change places at sizes M/2, ..., 1.
template <int M>
__device__ __forceinline__ uint32_t transposed_bits(uint32_t w)
{
    auto step = [&](auto size, uint32_t other) {
        constexpr int S = decltype(size)::value;
        constexpr uint32_t m = S == 8 ? 0x00FFu : S == 4 ? 0x0F0Fu : S == 2 ? 0x3333u : 0x5555u;
        w = (threadIdx.x & (uint32_t)S) ? ((w & ~m) | ((other >> S) & m)) : ((w & m) | ((other << S) & (m << S)));
    };
    if constexpr (M == 16)
        step(std::integral_constant<int, 8>{}, dpp_read<kRowRor8>(w));
    step(std::integral_constant<int, 4>{}, dpp_read<0x1B>(dpp_read<kRowHalfMirror>(w)));      // l ^ 7, then ^ 3
    step(std::integral_constant<int, 2>{}, dpp_read<0x4E>(w));
    step(std::integral_constant<int, 1>{}, dpp_read<0xB1>(w));
    return w;
}

// Writes the keep flags of the lane's column (bit i of kept = row i of its block).  All lanes of the wavefront take part.
template <int M, int FMT>
__device__ __forceinline__ void store_column(const MatDev &md, const ColumnPos &pos, uint32_t kept)
{
    unsigned char *row = (unsigned char *)md.mask + (size_t)pos.br * M * md.mask_ld + (FMT == kMaskU8 ? pos.col : pos.col >> 3);
    if constexpr (FMT == kMaskU8) {
        if (pos.valid) {
#pragma unroll
            for (int i = 0; i < M; i++)
                row[(size_t)i * md.mask_ld] = (unsigned char)((kept >> i) & 1u);
        }
    } else {
        const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
        for (int i = 0; i < M; i++) {
            const lanemask_t flags = lm((kept >> i) & 1u);
            if (pos.valid && (lane & 7u) == 0u)
                row[(size_t)i * md.mask_ld] = (unsigned char)(flags >> lane);
        }
    }
}

}  // namespace tmask
