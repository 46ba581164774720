// tmask_apply_pack: W (.) S and compression of W and W^T into N values + N positions per group of M.
//
// The paper (arXiv 2102.08124, Sec. 1 (Eq. 1) and Sec. 4) only states why both operands are needed: the
// forward product reads W and the backward product reads W^T, and a transposable mask leaves N
// non-zeros in every M contiguous elements of both.  The storage format is this library's own and
// is described in include/tmask.h.
//
// One workgroup, of 256 threads or, in calls of few tiles, of 1024, packs a 64-row x 256-byte tile (64 fp32 or 128 bf16 columns):
//   A  coalesced 16-byte loads of W and of the mask; masked values and 0/1 flags go to LDS
//   E  every thread takes its row-direction units (one row x one group of M columns) and its column-direction units (one group of M
//      rows x one column); each is compacted (kept entries, then lowest unused positions as +0 fillers, in position
//      order) and scattered into LDS staging: values row-major for W, column-major for W^T, index
//      bits OR-ed into per-row bit strings
//   G  staging is streamed out with coalesced stores (runs of 128..256 bytes per output row)
#pragma once
#include "tmask_device.hpp"

namespace tmask {

constexpr int kMaxPackBatch = 224;  // descriptors of 72 bytes, passed by value as kernel argument (16 KiB)
constexpr int kPackTR = 64;
constexpr int kPackThreads = 1024;    // of the kernel for any N:M where a call has few tiles

struct PackDev {
    const void *w;
    const void *mask;
    void *vals, *idx, *valsT, *idxT;
    uint32_t rows, cols, ld, mask_ld;
    uint32_t tiles_x;   // tiles per tile-row
    uint32_t tile0;     // first workgroup of this matrix inside the launch
};

template <int CAP>
struct PackArgsOf {
    PackDev d[CAP];
    CoarseIndex<CAP == kMaxPackBatch ? kCoarse : 16> ci;
    uint32_t n;
    uint32_t N;
};
using PackArgs = PackArgsOf<kMaxPackBatch>;
using FewPackArgs = PackArgsOf<kFewMats>;
static_assert(sizeof(PackArgs) <= 16384 + 2048, "descriptor table is sized to stay a small kernel argument");

// Arguments of the kernels that compute the mask themselves (tmask_approx_pack).
struct FusedArgs {
    PackDev d[kMaxPackBatch];   // mask = output here (may be null when WMASK is false)
    CoarseIndex<kCoarse> ci;
    uint32_t n;
    uint32_t partial0;          // index of this launch's first partial in the workspace
    void *partials;             // a record per workgroup (tags given) or a double, or null
    Tags tags;
    double *objective[kFewMats];        // tags given: of each matrix, in launches of so many at most
};
static_assert(sizeof(FusedArgs) <= 16384 + 2048, "descriptor table is sized to stay a small kernel argument");


// Tile number inside a matrix -> tile coordinates, for the kernels that write W^T in short runs per column.
// Workgroups go to the eight XCDs round-robin, so tile numbers t, t + 8, t + 16, ... run on one XCD one after
// the other.  They walk down a column band of tiles in runs of `run` tiles (4096 rows), band x, 8 + x, ... for
// XCD x, then the next 4096 rows: the pieces that the tiles of a run write into one row of W^T are neighbours
// in memory and arrive close in time, which the memory system rewards (fp32 2:4 pack: 66 -> 73 % of the HBM
// peak at 8192 x 8192; shorter runs lose it again, full-height runs cost the bf16 kernels 5 points).
// Bands beyond the last multiple of eight are walked column by column.
// ADJ > 1: an XCD takes ADJ neighbouring tile columns together, one after the other at each height: for kernels whose
// tiles are narrower than a cache line of the mask or of an index row, so that the tiles sharing such a line meet in
// one L2 instead of each fetching (or partly writing) it.  The generic kernel (256-byte tiles: 64 mask bytes and 16
// index bytes per tile row at fp32 8:16) fetched 1.20x and wrote 1.14x its algorithmic bytes without it; with four
// columns together 8192^2 fp32 8:16 goes from 145 to 121 us, 16384^2 from 715 to 505 us, 3:8 from 192 to 143 us.  The
// kernels with 1 KB tiles lose with it (fp32 2:4: 107 -> 115 us), except the bf16 4:8 pack with two (78 -> 73 us).
constexpr uint32_t kPackRunRows = 4096;


// Which descriptor does workgroup `tile` belong to (PackArgs or FusedArgs): coarse index, then a short binary search.
template <typename Args>
__device__ __forceinline__ int find_pack_desc(const Args &args, uint32_t tile)
{
    const uint32_t e = args.ci.e[tile >> args.ci.shift];
    int lo = (int)(e & 0xFFFFu), hi = (int)(e >> 16);
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (args.d[mid].tile0 <= tile)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// The objective of the one-pass kernels; d: the matrix, number k of the launch, in tiles TR rows high.
template <int TR>
__device__ __forceinline__ Handover objective_of(const FusedArgs &args, const PackDev &d, int k, uint32_t tile)
{
    return handover<8, 2>(args.partials, args.tags, args.partial0 + tile, tile - d.tile0, d.tiles_x * ((d.rows + TR - 1u) / TR),
                          args.objective[k % kFewMats]);
}

template <uint32_t ADJ = 1>
__device__ __forceinline__ void tile_coords(uint32_t tl, uint32_t tiles_x, uint32_t tiles_y, uint32_t run, uint32_t &ty,
                                            uint32_t &tx)
{
    const uint32_t bands8 = tiles_x / (8u * ADJ), full = bands8 * 8u * ADJ * tiles_y;
    if (tl < full) {
        const uint32_t x = tl & 7u, ka = tl >> 3;
        const uint32_t a = ka % ADJ, k = ka / ADJ;
        const uint32_t per_chunk = run * bands8;
        const uint32_t chunk = k / per_chunk, rk = k - chunk * per_chunk;
        const uint32_t rows_here = min(run, tiles_y - chunk * run);       // the last chunk may be shorter
        const uint32_t band = rk / rows_here;
        ty = chunk * run + (rk - band * rows_here);
        tx = (band * 8u + x) * ADJ + a;
    } else {
        const uint32_t r = tl - full;
        const uint32_t c = r / tiles_y;
        ty = r - c * tiles_y;
        tx = bands8 * 8u * ADJ + c;
    }
}

// ---- finished tiles out of LDS ------------------------------------------------------------------------------------------
// Lines of position bits, and of values where N and the matrix' height are odd, start at any byte.  What they cost is lines touched
// per store instruction, so a line leaves in one: neighbouring lanes store its dwords wherever these lie (the memory path takes
// dwords at any byte), and the last one, of a length that is no multiple of four, overlaps the one before.  (By bytes before, each
// with a division by the length: bf16 4:8 of 3576 x 3456 29.9 -> 19.0 us, 2:8 of 4096^2 33.0 -> 28.8.  A lane that stores three dwords of a line in a row touches it
// three times: fp32 3:16 of 4096^2 36.7 -> 39.7.)

// Byte `x` dwords into a line of nb (>= 4) bytes, or four before its end.
__device__ __forceinline__ uint32_t piece_at(uint32_t x, uint32_t nb) { return min(4u * x, nb - 4u); }

__device__ __forceinline__ void store_anywhere(uint32_t v, unsigned char *p) { __builtin_memcpy(p, &v, 4); }

__device__ __forceinline__ void store_three(uint32_t v, unsigned char *p, uint32_t nb)        // the first nb < 4 bytes
{
    if (nb > 0u)
        p[0] = (unsigned char)v;
    if (nb > 1u)
        p[1] = (unsigned char)(v >> 8);
    if (nb > 2u)
        p[2] = (unsigned char)(v >> 16);
}

// Dword x of the first nb bytes of a line of LB in LDS.
template <int LB>
__device__ __forceinline__ void copy_piece(const uint8_t *line, unsigned char *dst, uint32_t x, uint32_t nb)
{
    const uint32_t *const words = (const uint32_t *)line;
    if (nb < 4u) {
        if (x == 0u)
            store_three(words[0], dst, nb);
    } else if (4u * x < nb) {
        const uint32_t at = piece_at(x, nb), w = at / 4u;
        store_anywhere(__builtin_amdgcn_alignbyte(words[min(w + 1u, (uint32_t)LB / 4u - 1u)], words[w], at & 3u), dst + at);
    }
}

// The first nb (<= NB) bytes of `rows` lines of LB in LDS to lines `pitch` bytes apart.
template <int LB, int NT, int NB = LB>
__device__ __forceinline__ void copy_lines(const uint8_t (*src)[LB], unsigned char *dst, size_t pitch, uint32_t rows, uint32_t nb)
{
    static_assert(LB % 4 == 0 && NB <= LB, "lines of whole dwords");
    if (NB % 8 == 0 && LB % 8 == 0 && (((uint32_t)(uintptr_t)dst | (uint32_t)pitch | nb) & 7u) == 0u) {
        constexpr uint32_t P = (NB + 7) / 8;
        for (uint32_t j = threadIdx.x; j < rows * P; j += NT) {
            const uint32_t r = j / P, x = j % P;
            if (8u * x < nb)
                *(u32x2 *)(dst + (size_t)r * pitch + 8 * x) = ((const u32x2 *)&src[r][0])[x];
        }
    } else {
        constexpr uint32_t P = (NB + 3) / 4;
        for (uint32_t j = threadIdx.x; j < rows * P; j += NT) {
            const uint32_t r = j / P;
            copy_piece<LB>(&src[r][0], dst + (size_t)r * pitch, j % P, nb);
        }
    }
}

// The same for lines that are mostly much shorter than LB: their dwords to the next power of two of lanes.
template <int LB, int NT>
__device__ __forceinline__ void copy_short_lines(const uint8_t (*src)[LB], unsigned char *dst, size_t pitch, uint32_t rows, uint32_t nb)
{
    static_assert(LB % 4 == 0, "lines of whole dwords");
    const uint32_t nd = (nb + 3u) / 4u, shift = nd > 1u ? 32u - (uint32_t)__builtin_clz(nd - 1u) : 0u;
    const uint32_t x = threadIdx.x & ((1u << shift) - 1u);
    if (x < nd)
        for (uint32_t r = threadIdx.x >> shift; r < rows; r += (uint32_t)NT >> shift)
            copy_piece<LB>(&src[r][0], dst + (size_t)r * pitch, x, nb);
}

// The same of a tile that lies in LDS as [byte of the line][line]: NB bytes of TC lines.  Lines of eight bytes, or of aligned pieces of eight,
// go as above; the dwords of others to one lane for each line (side by side they meet in one bank of LDS: 4:8 in one pass 17.9 -> 18.6 us;
// two of them do not matter: 3300 x 2468 bf16 2:4 19.0 / 18.6).
template <int NB, int TC, int NT>
__device__ __forceinline__ void copy_columns(const uint8_t (*src)[TC], unsigned char *dst, size_t pitch, uint32_t cols, uint32_t nb)
{
    static_assert(NB % 4 == 0 && NT % TC == 0, "whole dwords; a thread keeps its line");
    auto word = [&](uint32_t at, uint32_t c) {
        return (uint32_t)src[at][c] | ((uint32_t)src[at + 1][c] << 8) | ((uint32_t)src[at + 2][c] << 16) | ((uint32_t)src[at + 3][c] << 24);
    };
    if (NB % 8 == 0 && nb == (uint32_t)NB && (((uint32_t)(uintptr_t)dst | (uint32_t)pitch) & 7u) == 0u) {
        constexpr uint32_t P = (NB + 7) / 8;
        for (uint32_t j = threadIdx.x; j < cols * P; j += NT) {
            const uint32_t c = j / P, x = j % P;
            *(u32x2 *)(dst + (size_t)c * pitch + 8 * x) = u32x2{word(8 * x, c), word(8 * x + 4, c)};
        }
        return;
    }
    if (NB == 8 && nb == 8u) {
        for (uint32_t j = threadIdx.x; j < cols * 2u; j += NT) {
            const uint32_t c = j / 2u, at = 4u * (j % 2u);
            store_anywhere(word(at, c), dst + (size_t)c * pitch + at);
        }
        return;
    }
    const uint32_t c = threadIdx.x % (uint32_t)TC, first = threadIdx.x / (uint32_t)TC;
    if (c >= cols)
        return;
    unsigned char *const line = dst + (size_t)c * pitch;
    if (nb < 4u) {
        if (first == 0u)
            store_three(word(0, c), line, nb);
    } else {
        for (uint32_t x = first; 4u * x < nb; x += NT / TC) {
            const uint32_t at = piece_at(x, nb);
            store_anywhere(word(at, c), line + at);
        }
    }
}

// Four dwords of a column of W^T, `left` (> 0) of them valid, to an address that is a multiple of four bytes: where the columns' runs are
// not whole 16-byte pieces.  Plain stores: with streaming ones the lines that two tiles share are not put together in L2.
__device__ __forceinline__ void store_dwords(u32x4 v, char *p, uint32_t left)
{
    typedef u32x4 dwords __attribute__((aligned(4)));
    if (left >= 4u) {
        *(dwords *)p = v;
    } else {
        ((uint32_t *)p)[0] = v.x;
        if (left > 1u)
            ((uint32_t *)p)[1] = v.y;
        if (left > 2u)
            ((uint32_t *)p)[2] = v.z;
    }
}

template <int M>
struct Log2 {
    static constexpr int v = (M == 4) ? 2 : (M == 8) ? 3 : (M == 16) ? 4 : 5;
};

// Which positions of a group of M fill its N slots.  kbits = keep flags (bit p = position p).
// sel    = kept positions that get a slot: all of them, or the first N if the mask (wrongly) keeps more;
// chosen = sel plus, if fewer than N are kept, the lowest-numbered other positions as +0 fillers.
template <int M>
__device__ __forceinline__ void choose_slots(uint32_t kbits, uint32_t N, uint32_t &sel, uint32_t &chosen)
{
    sel = kbits;
    uint32_t cnt = (uint32_t)__builtin_popcount(sel);
    while (cnt > N) {                                   // caller error, rare: drop the highest kept position
        sel &= ~(0x80000000u >> __builtin_clz(sel));
        cnt--;
    }
    uint32_t z = ~sel & (M == 32 ? 0xFFFFFFFFu : ((1u << (M & 31)) - 1u)), f = 0;
    for (uint32_t need = N - cnt; need > 0; need--) {   // approximate masks: usually zero to two rounds
        const uint32_t low = z & (0u - z);
        f |= low;
        z ^= low;
    }
    chosen = sel | f;
}

// ORs `nbits` (<= 60) bits of `code` into an LDS bit string at bit offset `off`.
__device__ __forceinline__ void lds_or_bits(uint32_t *words, uint32_t off, unsigned long long code)
{
    const uint32_t w = off >> 5, sh = off & 31u;
    const unsigned long long lo = code << sh;                       // bits landing in words w, w+1
    const uint32_t hi = sh ? (uint32_t)(code >> (64 - sh)) : 0u;    // bits landing in word w+2
    if ((uint32_t)lo)
        atomicOr(&words[w], (uint32_t)lo);
    if ((uint32_t)(lo >> 32))
        atomicOr(&words[w + 1], (uint32_t)(lo >> 32));
    if (hi)
        atomicOr(&words[w + 2], hi);
}

// NN = N when it is known at compile time (N = M/2: slot loops unrolled, a row group's values leave as 16-byte
// stores), 0 = any N (args.N).
// The BITS position bits of group number `g` of a line into the line's bit string (cleared beforehand): whole words are
// stored, anything else is ORed in.
template <int BITS>
__device__ __forceinline__ void put_code(uint32_t *words, uint32_t g, unsigned long long code)
{
    if constexpr (BITS % 32 == 0) {
#pragma unroll
        for (int w = 0; w < BITS / 32; w++)
            words[g * (BITS / 32) + w] = (uint32_t)(code >> (32 * w));
    } else {
        lds_or_bits(words, g * BITS, code);
    }
}

template <int DT, int M, int FMT, int NN = 0, int NT = kThreads, typename Args = PackArgs>
__global__ __launch_bounds__(NT) void pack_kernel(const Args args)
{
    using T = typename std::conditional<DT == kF32, uint32_t, uint16_t>::type;
    constexpr int ES = sizeof(T);
    constexpr int C = 16 / ES;                 // elements per 16-byte chunk
    constexpr int TR = kPackTR;
    constexpr int TC = 256 / ES;               // tile columns
    constexpr int IB = Log2<M>::v;
    constexpr int GPT = TC / M;                // groups per tile row
    constexpr int BPT = TR / M;                // block-rows per tile
    constexpr int OTR = NN ? TR * NN / M : TR; // staged W^T values per column: N per block-row (at most M - 1 if N is not known)
    constexpr int OTP = OTR + 4 / ES;          // pitch of the transposed staging (bank-conflict free)
    constexpr int NMAX = NN ? NN : M - 1;      // slots per group the staging must hold
    constexpr int IDXW = (GPT * NMAX * IB + 31) / 32 + 2;
    constexpr int IDXTW = (BPT * NMAX * IB + 31) / 32 + 2 + 1;
    constexpr int RU = TR * GPT, CU = BPT * TC;                 // row-direction and column-direction units
    static_assert(RU % 64 == 0, "a wavefront's units are of one direction");
    // Position codes of a group: NN * IB bits.  Beyond 64 bits (16:32: 80) they are kept as two halves of NN / 2 slots,
    // which go into the bit string as groups number 2g and 2g + 1 of half the width.
    constexpr bool SPLIT = NN * IB > 64;
    constexpr int HS = SPLIT ? NN / 2 : NN;    // slots per code word
    static_assert(M < 32 || NN == 16, "M = 32 comes here at 16:32 only (whole bytes of position bits per tile row)");

    __shared__ __attribute__((aligned(16))) T V[TR][TC];   // masked tile
    __shared__ __attribute__((aligned(16))) uint8_t FN[TR][16];   // keep flags of each 16-byte chunk (C bits), 16 chunks per tile row
    __shared__ T OT[TC][OTP];
    __shared__ uint32_t IDX[TR][IDXW];
    __shared__ uint32_t IDXT[TC][IDXTW];

    // ---- which tile ----
    const uint32_t tile = blockIdx.x;
    const PackDev d = args.d[find_pack_desc(args, tile)];
    const uint32_t N = NN ? (uint32_t)NN : args.N;
    const uint32_t tl = tile - d.tile0;
    uint32_t ty, tx;
    tile_coords<4>(tl, d.tiles_x, (d.rows + TR - 1) / TR, kPackRunRows / TR, ty, tx);
    const uint32_t row0 = ty * TR, col0 = tx * TC;
    const uint32_t tid = threadIdx.x;
    const uint32_t g_valid = min((uint32_t)GPT, (d.cols - col0) / M);   // groups of this tile inside the matrix
    const uint32_t b_valid = min((uint32_t)BPT, (d.rows - row0) / M);
    const uint32_t r_valid = b_valid * M, c_valid = g_valid * M;

    // ---- A: load ----
    for (uint32_t k = tid; k < TR * IDXW; k += NT)
        (&IDX[0][0])[k] = 0;
    for (uint32_t k = tid; k < TC * IDXTW; k += NT)
        (&IDXT[0][0])[k] = 0;
    // all loads of the thread go out before the first is used, none inside a branch (its result would be waited for
    // at the join): chunks outside the matrix read chunk (0, 0) and are dropped
    constexpr int PASSES = TR * 16 / NT;
    u32x4 raws[PASSES];
    uint32_t mlo[PASSES], mhi[PASSES];
#pragma unroll
    for (int pass = 0; pass < PASSES; pass++) {
        const uint32_t r = pass * (NT / 16) + (tid >> 4), ch = tid & 15u;
        const uint32_t row = row0 + r, col = col0 + ch * C;
        const bool ok = row < d.rows && col < d.cols;
        const uint32_t rowc = ok ? row : 0u, colc = ok ? col : 0u;
        raws[pass] = __builtin_nontemporal_load((const u32x4 *)((const char *)d.w + ((size_t)rowc * d.ld + colc) * ES));
        mhi[pass] = 0;
        if constexpr (FMT == kMaskU8) {
            const char *mp = (const char *)d.mask + (size_t)rowc * d.mask_ld + colc;
            if constexpr (C == 4) {
                mlo[pass] = __builtin_nontemporal_load((const uint32_t *)mp);
            } else {
                const u32x2 mv = __builtin_nontemporal_load((const u32x2 *)mp);
                mlo[pass] = mv.x;
                mhi[pass] = mv.y;
            }
        } else {
            mlo[pass] = ((const unsigned char *)d.mask)[(size_t)rowc * d.mask_ld + (colc >> 3)];
        }
    }
#pragma unroll
    for (int pass = 0; pass < PASSES; pass++) {
        const uint32_t r = pass * (NT / 16) + (tid >> 4), ch = tid & 15u;
        const uint32_t row = row0 + r, col = col0 + ch * C;
        const bool ok = row < d.rows && col < d.cols;
        u32x4 raw = raws[pass];
        uint32_t flags;
        if constexpr (FMT == kMaskU8)
            flags = (C == 4) ? bytes4_to_bits(mlo[pass]) : (bytes4_to_bits(mlo[pass]) | (bytes4_to_bits(mhi[pass]) << 4));
        else
            flags = (C == 8) ? mlo[pass] : ((mlo[pass] >> (col & 4u)) & 0xFu);
        flags = ok ? flags : 0u;                 // everything of such a chunk is then masked to zero below
        uint32_t w4[4] = {raw.x, raw.y, raw.z, raw.w};
        if constexpr (DT == kF32) {
#pragma unroll
            for (int c = 0; c < 4; c++)
                w4[c] = ((flags >> c) & 1u) ? w4[c] : 0u;
            FN[r][ch] = (uint8_t)flags;
        } else {
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const uint32_t keep_lo = ((flags >> (2 * c)) & 1u) ? 0x0000FFFFu : 0u;
                const uint32_t keep_hi = ((flags >> (2 * c + 1)) & 1u) ? 0xFFFF0000u : 0u;
                w4[c] &= keep_lo | keep_hi;
            }
            FN[r][ch] = (uint8_t)flags;
        }
        u32x4 mv = {w4[0], w4[1], w4[2], w4[3]};
        *(u32x4 *)&V[r][ch * C] = mv;
    }
    __syncthreads();

    // ---- E: compact.  Row units write W's values straight to memory (consecutive threads own
    // consecutive groups of a row); column units park W^T's values in LDS, column-major. ----
    const size_t pitchW = (size_t)(d.cols / M) * N;               // elements per row of vals
    const bool pair_ok = ES == 2 && ((N | (uint32_t)pitchW) & 1u) == 0;
    constexpr int MD = M * ES / 4;                                // dwords of a group
    // Large N: a slot of every lane to a store touches every line of a row N times, so the tile's rows leave whole at the end, through V, which
    // the column units read until then.  Start / rows whole, us: fp32 13:16 1440^2 17.4 / 13.4, 4096^2 89.9 / 52.5, 8192 x 4096 178 / 121; 7:8
    // 15.4 / 13.6, 69.7 / 52.0; 12:16 of 8192^2 301 / 183; bf16 13:16 4096^2 55.6 / 44.8, 15:16 66.1 / 47.2.  Small N pay more for the barrier and
    // LDS than they save (fp32 3:8 4096^2 39.3 / 40.9, 5:16 1440^2 10.9 / 11.2), even N of bf16 leave by pairs (10:16 38.5 / 41.5), 9:16 and 11:16
    // are even; so do calls for the kernel with 1024 threads (bf16 13:16 464 x 256 6.4 / 7.8).
    constexpr bool WHOLE = NN == 0 && NT == kThreads && (ES == 4 ? M > 6 : M > 13);
    const bool whole = WHOLE && (ES == 4 ? N > 5u : (N & 1u) && N > 12u);
    [[maybe_unused]] uint32_t held[WHOLE ? (RU + NT - 1) / NT : 1][MD] = {};   // values of a row unit
#pragma unroll
    for (int k = 0; k < (RU + CU + NT - 1) / NT; k++) {
        const uint32_t unit = tid + (uint32_t)k * NT;
        if (unit < (uint32_t)RU) {
            const uint32_t r = unit / GPT, g = unit % GPT;
            if (r >= r_valid || g >= g_valid)
                continue;   // outside the matrix: must not leave index bits in a row's padding
            uint32_t kb = 0;
            if constexpr (M >= C) {
#pragma unroll
                for (int q = 0; q < M / C; q++)
                    kb |= (uint32_t)FN[r][g * (M / C) + q] << (C * q);
            } else {
                kb = ((uint32_t)FN[r][g / (C / M)] >> (M * (g % (C / M)))) & ((1u << M) - 1u);
            }
            uint32_t sel, rem;
            choose_slots<M>(kb, N, sel, rem);
            T *dst = (T *)d.vals + (size_t)(row0 + r) * pitchW + (size_t)(col0 / M + g) * N;
            unsigned long long code = 0, code_hi = 0;
            uint32_t pend = 0;
            if constexpr (NN != 0 && (NN * ES) % 16 == 0) {
                if ((((uintptr_t)d.vals | (pitchW * ES)) & 15) == 0) {
                    // the group's NN values as whole 16-byte pieces
                    uint32_t out[NN * ES / 4];
#pragma unroll
                    for (int q = 0; q < NN * ES / 4; q++)
                        out[q] = 0;
#pragma unroll
                    for (int sl = 0; sl < NN; sl++) {
                        const uint32_t p = (uint32_t)__builtin_ctz(rem);
                        rem &= rem - 1u;
                        const uint32_t val = ((sel >> p) & 1u) ? (uint32_t)V[r][g * M + p] : 0u;
                        if constexpr (ES == 4)
                            out[sl] = val;
                        else
                            out[sl / 2] |= val << (16 * (sl & 1));
                        if (sl < HS)
                            code |= (unsigned long long)p << (sl * IB);
                        else
                            code_hi |= (unsigned long long)p << ((sl - HS) * IB);
                    }
#pragma unroll
                    for (int q = 0; q < NN * ES / 16; q++)
                        stream_store(u32x4{out[4 * q], out[4 * q + 1], out[4 * q + 2], out[4 * q + 3]}, (u32x4 *)dst + q);
                    if constexpr (SPLIT) {
                        put_code<HS * IB>(IDX[r], 2u * g, code);
                        put_code<HS * IB>(IDX[r], 2u * g + 1u, code_hi);
                    } else {
                        put_code<NN * IB>(IDX[r], g, code);
                    }
                    continue;
                }
            }
            if constexpr (WHOLE) {
                if (whole) {
#pragma unroll
                    for (int sl = 0; sl < M - 1; sl++) {
                        if ((uint32_t)sl >= N)
                            break;
                        const uint32_t p = (uint32_t)__builtin_ctz(rem);
                        rem &= rem - 1u;
                        const uint32_t val = ((sel >> p) & 1u) ? (uint32_t)V[r][g * M + p] : 0u;
                        held[k][sl * ES / 4] |= ES == 4 ? val : val << (16 * (sl & 1));
                        code |= (unsigned long long)p << (sl * IB);
                    }
                    lds_or_bits(IDX[r], g * N * IB, code);
                    continue;
                }
            }
            if constexpr (M == 32)
                continue;   // not reached: the host sends 16:32 here only with vals aligned to 16 bytes
            for (uint32_t sl = 0; sl < N; sl++) {
                const uint32_t p = (uint32_t)__builtin_ctz(rem);
                rem &= rem - 1u;
                const uint32_t val = ((sel >> p) & 1u) ? (uint32_t)V[r][g * M + p] : 0u;
                if constexpr (ES == 4) {
                    ((uint32_t *)dst)[sl] = val;
                } else if (pair_ok) {
                    if (sl & 1u)
                        *(uint32_t *)(dst + sl - 1) = pend | (val << 16);
                    else
                        pend = val;
                } else {
                    dst[sl] = (T)val;
                }
                code |= (unsigned long long)p << (sl * IB);
            }
            lds_or_bits(IDX[r], g * N * IB, code);
            continue;
        }
        const uint32_t u = unit - (uint32_t)RU, b = u / TC, c = u % TC;
        if (u >= (uint32_t)CU || b >= b_valid || c >= c_valid)
            continue;
        uint32_t kb = 0;
#pragma unroll
        for (int p = 0; p < M; p++)
            kb |= (((uint32_t)FN[b * M + p][c / C] >> (c % C)) & 1u) << p;
        uint32_t sel, rem;
        choose_slots<M>(kb, N, sel, rem);
        unsigned long long code = 0, code_hi = 0;
        if constexpr (NN != 0) {
#pragma unroll
            for (int sl = 0; sl < NN; sl++) {
                const uint32_t p = (uint32_t)__builtin_ctz(rem);
                rem &= rem - 1u;
                OT[c][b * NN + sl] = ((sel >> p) & 1u) ? V[b * M + p][c] : (T)0;
                if (sl < HS)
                    code |= (unsigned long long)p << (sl * IB);
                else
                    code_hi |= (unsigned long long)p << ((sl - HS) * IB);
            }
        } else {
            for (uint32_t sl = 0; sl < N; sl++) {
                const uint32_t p = (uint32_t)__builtin_ctz(rem);
                rem &= rem - 1u;
                OT[c][b * N + sl] = ((sel >> p) & 1u) ? V[b * M + p][c] : (T)0;
                code |= (unsigned long long)p << (sl * IB);
            }
        }
        if constexpr (SPLIT) {
            put_code<HS * IB>(IDXT[c], 2u * b, code);
            put_code<HS * IB>(IDXT[c], 2u * b + 1u, code_hi);
        } else if constexpr (NN != 0) {
            put_code<NN * IB>(IDXT[c], b, code);
        } else {
            lds_or_bits(IDXT[c], b * N * IB, code);
        }
    }
    __syncthreads();
    if (whole) {
        // dword q of a group of row r in place (q + r) mod MD of the group: the lanes of a store are 64 / GPT rows and meet in no bank
#pragma unroll
        for (int k = 0; k < (RU + NT - 1) / NT; k++) {
            const uint32_t unit = tid + (uint32_t)k * NT, r = unit / GPT, g = unit % GPT;
            if (unit < (uint32_t)RU) {
#pragma unroll
                for (int q = 0; q < MD; q++)
                    if ((uint32_t)q * (4 / ES) < N)
                        ((uint32_t *)&V[r][0])[g * MD + (((uint32_t)q + r) & (uint32_t)(MD - 1))] = held[k][q];
            }
        }
    }

    // ---- G: stream the staged W^T values and both index arrays out ----
    {
        // valsT: c_valid rows (columns of W), b_valid*N elements each
        const uint32_t run = b_valid * N;
        const size_t pitch = (size_t)(d.rows / M) * N;
        T *dst = (T *)d.valsT + (size_t)col0 * pitch + (size_t)(row0 / M) * N;
        if (ES == 4 || (((run | (uint32_t)pitch | (uint32_t)((row0 / M) * N)) & 1u) == 0)) {
            // fp32 runs of more than 64 bytes: one to a wavefront's store at M = 16 and 32 (5:16 of 8192 x 4096 84 -> 75 us, two to a store 81;
            // 6:16 87 -> 78), two where they fit at M = 8 (3:8, 96 bytes: 69.8, one to a store 72.1; 8192^2 135, 139)
            const uint32_t rd = run * ES / 4, shift = ES == 4 && M > 8 && rd > 16u ? 6u : rd > 1u ? 32u - (uint32_t)__builtin_clz(rd - 1u) : 0u;
            const uint32_t x = tid & ((1u << shift) - 1u);
            if (x < rd)
                for (uint32_t c = tid >> shift; c < c_valid; c += (uint32_t)NT >> shift)
                    stream_store(((const uint32_t *)&OT[c][0])[x], (uint32_t *)(dst + (size_t)c * pitch) + x);
        } else {
            copy_short_lines<OTP * ES, NT>((const uint8_t (*)[OTP * ES])OT, (unsigned char *)dst, pitch * ES, c_valid, run * ES);
        }
    }
    {
        // per row, the tile's bit string starts on a byte boundary (GPT*N*IB is a multiple of 8)
        const size_t pitch = ((size_t)(d.cols / M) * N * IB + 7) / 8, pitchT = ((size_t)(d.rows / M) * N * IB + 7) / 8;
        unsigned char *const dst = (unsigned char *)d.idx + (size_t)row0 * pitch + ((size_t)(col0 / M) * N * IB) / 8;
        unsigned char *const dstT = (unsigned char *)d.idxT + (size_t)col0 * pitchT + ((size_t)(row0 / M) * N * IB) / 8;
        const uint32_t nb = (g_valid * N * IB + 7) / 8, nbT = (b_valid * N * IB + 7) / 8;
        auto lines = (const uint8_t (*)[IDXW * 4])IDX;
        auto linesT = (const uint8_t (*)[IDXTW * 4])IDXT;
        if constexpr (NN != 0) {
            copy_lines<IDXW * 4, NT, GPT * NN * IB / 8>(lines, dst, pitch, r_valid, nb);
            copy_lines<IDXTW * 4, NT, BPT * NN * IB / 8>(linesT, dstT, pitchT, c_valid, nbT);
        } else {
            copy_short_lines<IDXW * 4, NT>(lines, dst, pitch, r_valid, nb);
            copy_short_lines<IDXTW * 4, NT>(linesT, dstT, pitchT, c_valid, nbT);
        }
    }
    if (whole) {
        __syncthreads();
        const uint32_t n = g_valid * N, inv = 65535u / N + 1u;           // e / N = e * inv >> 16 for e < 256
        T *dst = (T *)d.vals + (size_t)row0 * pitchW + (size_t)(col0 / M) * N;
        auto value = [&](uint32_t r, uint32_t e) {
            const uint32_t g = (e * inv) >> 16, sl = e - g * N;
            const uint32_t w = ((const uint32_t *)&V[r][0])[g * MD + ((sl * ES / 4 + r) & (uint32_t)(MD - 1))];
            return ES == 4 ? w : (w >> (16u * (sl & 1u))) & 0xFFFFu;
        };
        const uint32_t nd = (n * ES + 3u) / 4u, shift = nd > 16u ? 6u : nd > 1u ? 32u - (uint32_t)__builtin_clz(nd - 1u) : 0u;
        const uint32_t x = tid & ((1u << shift) - 1u);
        if (x < nd)
            for (uint32_t r = tid >> shift; r < r_valid; r += (uint32_t)NT >> shift) {
                T *line = dst + (size_t)r * pitchW;
                if constexpr (ES == 4) {
                    line[x] = value(r, x);
                } else {
                    const uint32_t e = min(2u * x, n - 2u);               // n > 12; the last dword may repeat an entry
                    store_anywhere(value(r, e) | (value(r, e + 1u) << 16), (unsigned char *)(line + e));
                }
            }
    }
}

}  // namespace tmask
