// tmask_spmm24: products with the compressed 2:4 operands written by tmask_apply_pack / tmask_approx_pack,
// on the structured-sparse matrix cores of gfx950 (arXiv 2102.08124, Sec. 1, Eq. 1, and Sec. 4: the forward
// product uses W, the backward product W^T, and a transposable mask makes both of them 2:4 sparse).
//
//     y[t][r] = sum_c x[t][c] * Wd[r][c],   Wd = the rows x cols matrix whose compressed form is (vals, idx)
//
// The instructions: D(16x16, fp32) += A(16x64, 2:4 sparse along k, bf16) * B(64x16, bf16), and the same as
// 32x32 += 32x32 * 32x32.  Lane l of the wavefront holds, with m = l % 16 and a = l / 16 (m = l % 32, a = l / 32):
//   A: 8 compressed values of row m: the two values of each of the groups of four g0, g0+1, g0+4, g0+5,
//      g0 = 8 (a % 2) + 2 (a / 2) (g0 = 2 a), i.e. two runs of four consecutive compressed values;
//   index register: bits 2j..2j+1 = position inside its group of the j-th value, j = 0..7 (low 16 bits);
//   B: 16 consecutive k of column n = m: k = 16 a .. 16 a + 15;
//   D: rows 4 a .. 4 a + 3 of column m (rows 8 (i / 4) + 4 a + i % 4, i = 0 .. 15).
// (Layouts established by probes on the hardware; the tests compare whole products with a CPU reference, which fixes
// every part of them.)  One byte of the packed `idx` array holds the positions of two consecutive groups, low nibble
// first, two bits per value in slot order: exactly eight index bits of the instruction, so the packed operands feed
// it unchanged.
//
// Two kernels: one whose wavefronts split the reduction of a small tile, for products with few tokens or few rows, and
// one whose wavefronts share a large tile.  tmask_spmm24 (at the end) chooses between their tile sizes.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "../../include/tmask.h"
#include "tmask_host.hpp"
#include "tmask_spmm_choice.hpp"

namespace tmask {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t su32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t su32x2 __attribute__((ext_vector_type(2)));

constexpr int kSpKS = (int)kSpmmStep;

struct SpmmArgs {
    const void *vals;     // rows x cols/2 bf16
    const void *idx;      // rows x cols/8 bytes
    const void *x;        // tokens x cols bf16, leading dimension ld_x
    void *y;              // tokens x rows, leading dimension ld_y
    uint32_t rows, cols, tokens;
    uint32_t ld_x, ld_y;
    uint32_t tiles_r, tiles_t;
    uint32_t lines;       // the shared tiles write whole lines of y, with streaming stores
};

// y[tok][r .. r+3] (fp32 -> bf16 rounds to nearest even, by the hardware's packed conversion)
template <bool OUT_BF16>
__device__ __forceinline__ void store_quad(const SpmmArgs &p, uint32_t tok, uint32_t r, f32x4 v)
{
    if constexpr (OUT_BF16) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        union { bf16x2 h; uint32_t u; } c0, c1;
        c0.h = __builtin_convertvector(f32x2{v.x, v.y}, bf16x2);
        c1.h = __builtin_convertvector(f32x2{v.z, v.w}, bf16x2);
        *(su32x2 *)((unsigned char *)p.y + ((size_t)tok * p.ld_y + r) * 2u) = su32x2{c0.u, c1.u};
    } else {
        *(f32x4 *)((unsigned char *)p.y + ((size_t)tok * p.ld_y + r) * 4u) = v;
    }
}

// ---------------------------------------------------------------------------------------------------------------------
// Direct global -> LDS copies.  The instruction writes lane l's piece at the (wavefront-uniform) LDS address in m0 plus
// l times the piece size, so a swizzle of the LDS image is a permutation of the addresses the lanes read from.  Inline
// asm, because the compiler would make every LDS read wait for all copies in flight; the waits below count them.  The
// copies have no destination register, and the address registers are read when the instruction issues.
// ---------------------------------------------------------------------------------------------------------------------
__device__ __forceinline__ void copy16(const unsigned char *base, uint32_t lane_off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(lane_off), "s"(base)
                 : "m0");
}

__device__ __forceinline__ void copy4(const unsigned char *base, uint32_t lane_off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(lane_off), "s"(base)
                 : "m0");
}

// at most N of the wavefront's global memory operations are still in flight (they finish in order)
template <int N>
__device__ __forceinline__ void wait_copies()
{
    static_assert(N >= 0 && N < 64, "six bits of counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// the wavefront's LDS reads have arrived in registers (as the builtin, so that the compiler knows and adds no wait of its
// own in front of their first use)
__device__ __forceinline__ void wait_lds_reads()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);                         // lgkmcnt(0)
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)p;
}

// ---------------------------------------------------------------------------------------------------------------------
// Few tokens or few rows: the reduction split over the wavefronts of a workgroup
// ---------------------------------------------------------------------------------------------------------------------
//
// With tens of large tiles most compute units stand idle, so these products take small tiles (16 RT rows x 16 CT
// tokens) and what a workgroup has in excess, wavefronts, shares the reduction: wavefront w takes the units of 256 k
// numbered w, w + W, ... for the whole tile.  Every byte is then needed by one wavefront only, so each keeps a ring of
// D steps (64 k) in its own part of LDS, filled by direct copies and read back as fragments, and no wavefront waits for
// another before the final sum.  (Fragments loaded straight into registers need no LDS, but sixteen consecutive lanes
// then read sixteen different rows and the memory path delivers a quarter of its 64 bytes per clock.)
//
// Which k a position of the instruction stands for is free as long as both operands agree.  Position groups (of four
// k) 4b, 4b+1 stand for the step's groups 2b, 2b+1 and 4b+2, 4b+3 for 8+2b, 9+2b: lane a's compressed values are then
// the 16 bytes at 16 a of the row's 64 with the index bytes 2a, 2a+1 of its eight, its x values the 16 bytes at 16 a and
// at 64 + 16 a of the token's 128.
//
// LDS images are swizzled in 16-byte pieces so that eight consecutive lanes of a fragment read cover all banks: piece c
// of row r of A lies in slot c ^ ((r >> 1) & 3), piece c of token t of B in slot c ^ (t & 7).
constexpr int kSkUnit = 4;           // steps per unit (a row's index bytes of a unit are 32 contiguous bytes)

template <int RT, int CT, int W, int D, bool OUT_BF16>
__global__ __launch_bounds__(64 * W, 1) void spmm24_ksplit_kernel(const SpmmArgs p)
{
    constexpr int TR = RT * 16, TT = CT * 16;
    constexpr int kPitch = TR + 4;                              // floats per token in the exchange buffer
    constexpr uint32_t kStep = RT * 1024u + CT * 2048u;         // bytes of a step: A, then B
    constexpr uint32_t kIdx = RT * 512u;                        // index bytes of a unit
    constexpr uint32_t kWave = D * kStep + 2u * kIdx;
    constexpr uint32_t kPart = TT * kPitch * 4u;
    constexpr int kData = RT + 2 * CT;                          // copy instructions of a step
    constexpr uint32_t kLds = kWave > kPart ? kWave : kPart;
    __shared__ __attribute__((aligned(16))) unsigned char lds[W * kLds];

    // Each XCD takes a contiguous range of tile numbers; 32 consecutive ones form a block of 4 row panels x 8 token
    // panels, so that the workgroups that run on an XCD together share panels in its L2.
    const uint32_t n_tiles = p.tiles_r * p.tiles_t;
    uint32_t id = blockIdx.x;
    const uint32_t per = n_tiles / 8u;
    if (id < per * 8u)
        id = (id & 7u) * per + (id >> 3);
    constexpr uint32_t kGroup = 4;
    const uint32_t in_group = kGroup * p.tiles_t;
    const uint32_t group = id / in_group, rem = id - group * in_group;
    const uint32_t first_r = group * kGroup;
    const uint32_t group_rows = min(p.tiles_r - first_r, kGroup);
    const uint32_t tt = rem / group_rows;
    const uint32_t row0 = (first_r + (rem - tt * group_rows)) * TR, tok0 = tt * TT;

    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t m = lane & 15u, a = lane >> 4;
    const uint32_t steps = p.cols / kSpKS;

    // ---- copies: rows and tokens past the edge re-read the last valid one; their results are not stored ----
    uint32_t off_a[RT], off_i[2 * RT], off_b[2 * CT];
#pragma unroll
    for (int i = 0; i < RT; i++) {                              // 16 rows x 64 bytes
        const uint32_t r = (uint32_t)i * 16u + (lane >> 2);
        off_a[i] = (min(row0 + r, p.rows - 1u) - row0) * p.cols + (((lane & 3u) ^ ((lane >> 3) & 3u)) * 16u);
    }
#pragma unroll
    for (int i = 0; i < 2 * RT; i++)                            // 8 rows x 32 bytes
        off_i[i] = (min(row0 + (uint32_t)i * 8u + (lane >> 3), p.rows - 1u) - row0) * (p.cols >> 3);
#pragma unroll
    for (int j = 0; j < 2 * CT; j++) {                          // 8 tokens x 128 bytes
        const uint32_t t = (uint32_t)j * 8u + (lane >> 3);
        off_b[j] = (min(tok0 + t, p.tokens - 1u) - tok0) * p.ld_x * 2u + (((lane & 7u) ^ ((lane >> 3) & 7u)) * 16u);
    }
    const unsigned char *base_a = (const unsigned char *)p.vals + (size_t)row0 * p.cols;
    const unsigned char *base_b = (const unsigned char *)p.x + (size_t)tok0 * p.ld_x * 2u;
    const unsigned char *base_i = (const unsigned char *)p.idx + (size_t)row0 * (p.cols >> 3);
    unsigned char *const mine = lds + wave * kWave;
    const uint32_t mine_at = __builtin_amdgcn_readfirstlane(lds_address(mine));

    // The wavefront's steps as one stream t = 0 .. n - 1: unit wave + W (t / 4), step t % 4 of it.  Only the last unit of
    // all can be short, and it is the last of its wavefront.
    const uint32_t units = (steps + kSkUnit - 1u) / kSkUnit;
    const uint32_t my_units = wave < units ? (units - wave + W - 1u) / W : 0u;
    uint32_t n = my_units * kSkUnit;
    if (my_units && wave + (my_units - 1u) * W == units - 1u)
        n -= units * kSkUnit - steps;
    auto copy_step = [&](uint32_t t) {
        const uint32_t s = (wave + (t / kSkUnit) * W) * kSkUnit + t % kSkUnit;
        const unsigned char *pa = base_a + (size_t)s * 64u, *pb = base_b + (size_t)s * 128u;
        uint32_t at = mine_at + (t % D) * kStep;
#pragma unroll
        for (int i = 0; i < RT; i++, at += 1024u)
            copy16(pa, off_a[i], at);
#pragma unroll
        for (int j = 0; j < 2 * CT; j++, at += 1024u)
            copy16(pb, off_b[j], at);
    };
    auto copy_idx = [&](uint32_t k) {                           // the wavefront's k-th unit; bytes past the row's end repeat its last
        const uint32_t d = min((wave + k * W) * (2u * kSkUnit) + (lane & 7u), 2u * steps - 1u) * 4u;
        uint32_t at = mine_at + D * kStep + (k & 1u) * kIdx;
#pragma unroll
        for (int i = 0; i < 2 * RT; i++, at += 256u)
            copy4(base_i, off_i[i] + d, at);
    };

    // ---- fragments ----
    struct Frag {
        bf16x8 a[RT];
        bf16x16 b[CT];
        int sel[RT];
    };
    const uint32_t read_a = m * 64u + ((a ^ ((m >> 1) & 3u)) * 16u);
    const uint32_t read_b0 = RT * 1024u + m * 128u + ((a ^ (m & 7u)) * 16u);
    const uint32_t read_b1 = RT * 1024u + m * 128u + (((a + 4u) ^ (m & 7u)) * 16u);
    const uint32_t read_i = D * kStep + m * 32u + a * 2u;
    auto read_step = [&](Frag &f, uint32_t t) {
        const unsigned char *src = mine + (t % D) * kStep;
        const unsigned char *src_i = mine + ((t / kSkUnit) & 1u) * kIdx + (t % kSkUnit) * 8u;
#pragma unroll
        for (int i = 0; i < RT; i++) {
            f.a[i] = *(const bf16x8 *)(src + read_a + i * 1024);
            f.sel[i] = (int)*(const uint16_t *)(src_i + read_i + i * 512);
        }
#pragma unroll
        for (int j = 0; j < CT; j++) {
            union { su32x4 u[2]; bf16x16 v; } cv;
            cv.u[0] = *(const su32x4 *)(src + read_b0 + j * 2048);
            cv.u[1] = *(const su32x4 *)(src + read_b1 + j * 2048);
            f.b[j] = cv.v;
        }
    };
    f32x4 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; i++)
#pragma unroll
        for (int j = 0; j < CT; j++)
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const Frag &f) {
#pragma unroll
        for (int i = 0; i < RT; i++)
#pragma unroll
            for (int j = 0; j < CT; j++)
                acc[i][j] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(f.a[i], f.b[j], acc[i][j], f.sel[i], 0, 0);
    };

    // Step t: its fragments are in registers; those of step t + 1 are read while it is multiplied, and once they have
    // arrived step t + 1 + D may overwrite them.  Copies of steps t + 2 .. t + D are in flight meanwhile.
    if (n) {
        copy_idx(0);
#pragma unroll
        for (int t = 0; t < D; t++)
            if ((uint32_t)t < n)
                copy_step(t);
        if (my_units > 1u)
            copy_idx(1);
        Frag f[2];
        auto arrive = [&](uint32_t t) {                         // step t is in LDS
            if (t + D <= n)                                     // steps t + 1 .. t + D - 1 may be in flight
                wait_copies<(D - 1) * kData>();
            else
                wait_copies<0>();
        };
        arrive(0);
        read_step(f[0], 0);
        wait_lds_reads();
        if (D < n)
            copy_step(D);
        uint32_t t = 0;
        auto step = [&](int cur) {                              // t + 1 < n
            arrive(t + 1u);
            read_step(f[cur ^ 1], t + 1u);
            __builtin_amdgcn_sched_barrier(0);
            multiply(f[cur]);
            __builtin_amdgcn_sched_barrier(0);
            t++;
            wait_lds_reads();
            // the unit that step t ends gives its place to the one after the next
            if (t % kSkUnit == kSkUnit - 1u && t / kSkUnit + 2u < my_units)
                copy_idx(t / kSkUnit + 2u);
            if (t + D < n)
                copy_step(t + D);
        };
        while (t + 2u < n) {
            step(0);
            step(1);
        }
        if (t + 1u < n) {
            step(0);
            multiply(f[1]);
        } else {
            multiply(f[0]);
        }
    }

    // ---- the wavefronts' sums, added in a fixed order; a lane holds rows 4a..4a+3 of token m of each instruction tile ----
    __syncthreads();                                            // the rings are no longer read
    float *const part = (float *)lds;
#pragma unroll
    for (int i = 0; i < RT; i++)
#pragma unroll
        for (int j = 0; j < CT; j++)
            *(f32x4 *)&part[wave * (TT * kPitch) + (j * 16u + m) * kPitch + i * 16u + a * 4u] = acc[i][j];
    __syncthreads();
    constexpr int kQuads = TR * TT / 4;                         // four rows of a token each
    const uint32_t used = min(units, (uint32_t)W);
#pragma unroll
    for (int q0 = 0; q0 < kQuads; q0 += 64 * W) {
        const uint32_t q = q0 + threadIdx.x;
        if (kQuads % (64 * W) != 0 && q >= (uint32_t)kQuads)
            break;
        const uint32_t t = q / (TR / 4), r = (q % (TR / 4)) * 4u;
        f32x4 v = *(const f32x4 *)&part[t * kPitch + r];
        for (uint32_t w = 1; w < used; w++)
            v += *(const f32x4 *)&part[w * (TT * kPitch) + t * kPitch + r];
        const uint32_t tok = tok0 + t, row = row0 + r;
        if (tok < p.tokens && row < p.rows)                     // rows is a multiple of 4: the four entries are in or out together
            store_quad<OUT_BF16>(p, tok, row, v);
    }
}

// ---------------------------------------------------------------------------------------------------------------------
// Many tokens and rows: tiles shared by four wavefronts
// ---------------------------------------------------------------------------------------------------------------------
//
// A workgroup computes 64 RT rows x 64 CT tokens with 2 x 2 wavefronts, each 32 RT x 32 CT on the 32 x 32 x 32
// instruction.  Positions are assigned to k as in the split kernel: lane a's values of a half step (32 k) are the 16 bytes
// at 16 a of the row's 32, its x values the 16 bytes at 16 a and 32 + 16 a of the token's 64.
//
// What bounds a step is the arrival of its tiles: a 256 x 256 one needs 50 KB, which one compute unit by itself has in 0.63 us
// (81 GB/s) and each of 256 at work in 1.08 us (47 GB/s, 12 TB/s over the chip; 128 x 128: 0.31 and 0.43 us, 15 TB/s), while
// its matrix instructions take 0.43.  So the tile is as large as the registers allow: 256 x 256, with 256 accumulator
// registers per lane, moves 50 KB per 2^22 products, a third of what the 256 x 128 tiles of a kernel with eight wavefronts
// moved that staged them through registers.  A tile costs 7 to 8 us besides its steps, with bf16 results: the first copies,
// and the results, which leave while nothing is multiplied (W 4096 x 1024, 8192 tokens: 77 -> 50 us, two rounds of sixteen
// steps).  Steps of 64 k arrive in a ring of three LDS images by direct copies, two steps ahead.  The fragments of a half step are read while the half before it is multiplied.  One barrier per
// step, between its halves: when all wavefronts have read the second half of step g its image is overwritten by step
// g + 3, and step g + 1, whose copies every wavefront has waited for, may be read.  Workgroups are persistent and treat
// the steps of all their tiles as one stream, so the copies of a tile's first steps are in flight while the one before
// is stored.
//
// Swizzle: 32 rows of one piece are read at a time, sixteen lanes per pass over the 64 banks, so piece c of row r of A
// lies in slot c ^ ((r >> 2) & 3) and piece c of token t of B in slot c ^ ((t >> 1) & 7) (bank conflict cycles 14.7e6 ->
// 2.1e6 per product against the split kernel's swizzle).
constexpr int kTileRing = 3;

// acc += A B with the sums in accumulation registers.  As the builtin, with 256 of them, the compiler moves sums between
// the two register files in every step.  What it would do for the builtin is done here by hand: two wait states in case
// an operand was just written by a vector instruction; and whoever reads the sums afterwards waits (sums_ready) and takes
// them through take_sums.  The compiler does not know that sums are in flight between the two: a test reads the assembly
// for anything that touches an accumulation register there.
__device__ __forceinline__ void multiply32(f32x16 &acc, bf16x8 a, bf16x16 b, int sel)
{
    asm volatile("s_nop 1\n\tv_smfmac_f32_32x32x32_bf16 %0, %1, %2, %3" : "+a"(acc) : "v"(a), "v"(b), "v"(sel));
}

// The last matrix instruction's results can be read by vector instructions (16 passes; 18 wait states needed).
__device__ __forceinline__ void sums_ready()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15");
    __builtin_amdgcn_sched_barrier(0);
}

// What reads these sums hangs on this point, which stays behind sums_ready() (no volatile asm passes another) and behind
// the stores before it, so that no more than one tile's results wait in vector registers.
__device__ __forceinline__ void take_sums(f32x16 &acc) { asm volatile("" : "+a"(acc)::"memory"); }

template <int RT, int CT, bool OUT_BF16>
__global__ __launch_bounds__(256, RT * CT <= 4 ? 2 : 1) void spmm24_tile_kernel(const SpmmArgs p)
{
    constexpr int TR = RT * 64, TT = CT * 64;
    constexpr uint32_t kA = TR * 64u, kB = TT * 128u, kI = TR * 8u, kImage = kA + kB + kI;
    constexpr int kCopyA = RT, kCopyB = 2 * CT, kCopyI = RT / 2 > 0 ? RT / 2 : 1;       // copies of a wavefront per step
    constexpr int kCopies = kCopyA + kCopyB + kCopyI;
    constexpr int kStores = RT * CT * (OUT_BF16 ? 2 : 4);                               // of a wavefront per tile
    static_assert(RT % 2 == 0, "index bytes: four wavefronts x 32 rows per copy");
    __shared__ __attribute__((aligned(16))) unsigned char lds[kTileRing * kImage];

    // Tiles b, b + G, b + 2G, ... of the launch, as one stream of steps.  Each XCD takes a contiguous range of tile
    // numbers, and 64 consecutive ones form an 8 x 8 block of the output, so that the workgroups that run on an XCD together
    // share panels in its L2.
    const uint32_t n_tiles = p.tiles_r * p.tiles_t;
    const uint32_t G = gridDim.x, b = blockIdx.x;
    const uint32_t my_tiles = (n_tiles - b + G - 1u) / G;       // b < G <= n_tiles
    const uint32_t steps = p.cols / kSpKS;
    auto locate = [&](uint32_t j, uint32_t &row0, uint32_t &tok0) {
        uint32_t id = b + j * G;
        const uint32_t per = n_tiles / 8u;
        if (id < per * 8u)
            id = (id & 7u) * per + (id >> 3);
        constexpr uint32_t kGroup = 8;
        const uint32_t in_group = kGroup * p.tiles_t;
        const uint32_t group = id / in_group, rem = id - group * in_group;
        const uint32_t first_r = group * kGroup;
        const uint32_t group_rows = min(p.tiles_r - first_r, kGroup);
        const uint32_t tt = rem / group_rows;
        row0 = (first_r + (rem - tt * group_rows)) * TR;
        tok0 = tt * TT;
    };
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lds_at = __builtin_amdgcn_readfirstlane(lds_address(lds));

    // ---- copies (rows and tokens past the edge re-read the last valid one; their results are not stored) ----
    // wavefront w copies rows 16 (w + 4 i) .. + 15 of A, tokens 8 (w + 4 i) .. + 7 of B, index bytes of rows 32 (w + 4 i) .. + 31
    uint32_t off_a[kCopyA], off_b[kCopyB], off_i[kCopyI];
    const unsigned char *base_a, *base_b, *base_i;
    auto set_tile = [&](uint32_t j) {
        uint32_t row0, tok0;
        locate(j, row0, tok0);
        base_a = (const unsigned char *)p.vals + (size_t)row0 * p.cols;
        base_b = (const unsigned char *)p.x + (size_t)tok0 * p.ld_x * 2u;
        base_i = (const unsigned char *)p.idx + (size_t)row0 * (p.cols >> 3);
#pragma unroll
        for (int i = 0; i < kCopyA; i++) {
            const uint32_t r = ((uint32_t)i * 4u + wave) * 16u + (lane >> 2);
            off_a[i] = (min(row0 + r, p.rows - 1u) - row0) * p.cols + (((lane & 3u) ^ (lane >> 4)) * 16u);
        }
#pragma unroll
        for (int i = 0; i < kCopyB; i++) {
            const uint32_t t = ((uint32_t)i * 4u + wave) * 8u + (lane >> 3);
            off_b[i] = (min(tok0 + t, p.tokens - 1u) - tok0) * p.ld_x * 2u + (((lane & 7u) ^ ((wave & 1u) * 4u + (lane >> 4))) * 16u);
        }
#pragma unroll
        for (int i = 0; i < kCopyI; i++) {
            const uint32_t r = ((uint32_t)i * 4u + wave) * 32u + (lane >> 1);
            off_i[i] = (min(row0 + r, p.rows - 1u) - row0) * (p.cols >> 3) + (lane & 1u) * 4u;
        }
    };
    uint32_t fj = 0, fk = 0;                                    // tile ordinal and step of the next copy
    uint32_t slot = 0;                                          // its image
    auto copy_piece = [&](int i) {                              // i < kCopies, a compile-time constant at every call
        const uint32_t at = lds_at + slot * kImage;
        if (i < kCopyA)
            copy16(base_a + (size_t)fk * 64u, off_a[i], at + ((uint32_t)i * 4u + wave) * 1024u);
        else if (i < kCopyA + kCopyB)
            copy16(base_b + (size_t)fk * 128u, off_b[i - kCopyA], at + kA + ((uint32_t)(i - kCopyA) * 4u + wave) * 1024u);
        else
            copy4(base_i + (size_t)fk * 8u, off_i[i - kCopyA - kCopyB],
                  at + kA + kB + ((uint32_t)(i - kCopyA - kCopyB) * 4u + wave) * 256u);
    };
    auto copied = [&]() {                                       // on to the next step
        slot = slot == kTileRing - 1 ? 0 : slot + 1;
        if (++fk == steps) {                                    // past the end of the stream its last tile is copied again
            fk = 0;
            if (fj + 1u < my_tiles)
                set_tile(++fj);
        }
    };

    // ---- fragments ----
    struct Frag {
        bf16x8 a[RT];
        su32x4 b[CT][2];
        int sel[RT];
    };
    const uint32_t wr = wave >> 1, wc = wave & 1u;              // position of this wavefront in the tile
    const uint32_t m = lane & 31u, a = lane >> 5;
    uint32_t read_a[2], read_b[2][2];
#pragma unroll
    for (uint32_t h = 0; h < 2; h++) {
        read_a[h] = (wr * RT * 32u + m) * 64u + (((2u * h + a) ^ ((m >> 2) & 3u)) * 16u);
        read_b[h][0] = kA + (wc * CT * 32u + m) * 128u + (((4u * h + a) ^ ((m >> 1) & 7u)) * 16u);
        read_b[h][1] = kA + (wc * CT * 32u + m) * 128u + (((4u * h + 2u + a) ^ ((m >> 1) & 7u)) * 16u);
    }
    const uint32_t read_i = kA + kB + (wr * RT * 32u + m) * 8u + a * 2u;
    // read i of a half step's fragments, in the order in which the multiplication needs them: x of token tile 0, A and
    // positions of row tile 0, x of the other token tiles, A and positions of the other row tiles
    constexpr int kReads = 2 * CT + RT;
    auto read_piece = [&](Frag &f, uint32_t image, int h, int i) {
        const unsigned char *src = lds + image;
        if (i == 2 || i > 2 * CT) {
            const int rt = i == 2 ? 0 : i - 2 * CT;
            f.a[rt] = *(const bf16x8 *)(src + read_a[h] + rt * 2048);
            f.sel[rt] = (int)*(const uint16_t *)(src + read_i + rt * 256 + h * 4);
        } else {
            const int k = i < 2 ? i : i - 1;
            f.b[k / 2][k % 2] = *(const su32x4 *)(src + read_b[h][k % 2] + (k / 2) * 4096);
        }
    };
    f32x16 acc[RT][CT];
    // Multiplies the fragments of a half step; between its instructions go the reads of the next one's fragments and, with
    // COPY, the copies of a step three ahead: there is one wavefront per SIMD, so the matrix cores would wait for whatever
    // is issued in a run of its own.
    auto half = [&](const Frag &cur, Frag &nxt, uint32_t nxt_image, int nxt_h, auto copy) {
        constexpr bool COPY = decltype(copy)::value;
        constexpr int kMul = RT * CT;
#pragma unroll
        for (int q = 0; q < kMul; q++) {
            union { su32x4 u[2]; bf16x16 v; } bv;
            bv.u[0] = cur.b[q % CT][0];
            bv.u[1] = cur.b[q % CT][1];
            multiply32(acc[q / CT][q % CT], cur.a[q / CT], bv.v, cur.sel[q / CT]);
            // reads all go out in the first three quarters
#pragma unroll
            for (int i = q * kReads * 4 / (3 * kMul); i < (q + 1) * kReads * 4 / (3 * kMul) && i < kReads; i++)
                read_piece(nxt, nxt_image, nxt_h, i);
            if constexpr (COPY) {
#pragma unroll
                for (int i = q * kCopies / kMul; i < (q + 1) * kCopies / kMul; i++)
                    copy_piece(i);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (COPY)
            copied();
        wait_lds_reads();
    };

    // Writes the tile; returns whether all of kStores store instructions were issued.  A store covers 64 contiguous bytes of
    // each of sixteen tokens (32 of 32 tokens as the sums lie in the lanes: twice the requests for the same lines, and products
    // with a short reduction are bound by what they write: fp32 8192 x 64, 8192 tokens 55 -> 50 us on 128 x 128 tiles, 62 ->
    // 53 on 256 x 256; bf16 4096 x 1024, 8192 tokens 52 -> 50).  Instruction tiles that lie outside the matrix are skipped
    // whole (1048576 x 64, 4 tokens: 38 -> 31 us).
    // With p.lines it covers whole lines of 128 bytes of eight tokens, and the stores are streaming ones: as plain stores the
    // results push out of L2 the panels that the next tiles read (8192 tokens, three / four rotating sets of buffers, us: 4096 x
    // 1024 bf16 52 -> 48 / 57.5 -> 50, fp32 64 -> 55 / 68 -> 59; 1024 x 4096 fp32 63 -> 49; 1024 x 256 bf16 10.0 -> 8.1).  What stays in
    // the memory-side cache gains nothing: one set of buffers 4096 x 1024 bf16 50.3 -> 50.5, the same product with
    // new inputs and results for each call 46.9 -> 46.7, fp32 3072 x 64 into the same 100 MB each time 20.1 -> 22.9 (four sets 24.5 -> 23.0).
    // Streaming stores of parts of lines lose (fp32 8192 x 64 54 -> 78), which is where the line lies on the host.
    auto store_tile = [&](uint32_t j) -> bool {
        uint32_t row0, tok0;
        locate(j, row0, tok0);
        const bool whole = row0 + TR <= p.rows && tok0 + TT <= p.tokens;
        row0 += wr * RT * 32u;
        tok0 += wc * CT * 32u;
        constexpr uint32_t kPiece = OUT_BF16 ? 8u : 4u;         // results of a lane's 16 bytes
        auto put = [&](uint32_t tok, uint32_t r, su32x4 v, auto streamed) {
            unsigned char *dst = (unsigned char *)p.y + ((size_t)tok * p.ld_y + r) * (16u / kPiece);
            if (whole || (tok < p.tokens && r + kPiece <= p.rows)) {
                if constexpr (decltype(streamed)::value)
                    __builtin_nontemporal_store(v, (su32x4 *)dst);
                else
                    *(su32x4 *)dst = v;
            } else if (OUT_BF16 && tok < p.tokens && r + 4u <= p.rows) {
                *(su32x2 *)dst = su32x2{v.x, v.y};
            }
        };
        // Lane 16 g + n holds 16 bytes of token tok + n, the four g side by side: v0 of the 64 bytes at r, v1 of the 64 after.
        // Lines: lanes n < 8 keep v0 and take the v0 of token n + 8 for the second store, lanes n >= 8 the same with v1.
        const uint32_t n = lane & 15u, lane_r = kPiece * (2u * ((lane >> 4) & 1u) + a);
        auto put_pair = [&](uint32_t tok, uint32_t r, su32x4 v0, su32x4 v1) {
            constexpr uint32_t kNext = 4u * kPiece;
            if (p.lines) {
                const bool upper = n >= 8u;
                su32x4 s0, s1;
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(upper ? v0[k] : v1[k]), 0x128, 0xF, 0xF, false);   // row_ror:8
                    s0[k] = upper ? got : v0[k];
                    s1[k] = upper ? v1[k] : got;
                }
                const uint32_t t = tok + (n & 7u), rr = r + (upper ? kNext : 0u);
                put(t, rr, s0, std::true_type{});
                put(t + 8u, rr, s1, std::true_type{});
            } else {
                put(tok + n, r, v0, std::false_type{});
                put(tok + n, r + kNext, v1, std::false_type{});
            }
        };
        constexpr int kPair = OUT_BF16 ? 2 : 1;                 // instruction tiles to a line
#pragma unroll
        for (int ct = 0; ct < CT; ct++) {
#pragma unroll
            for (int rt = 0; rt < RT; rt += kPair) {
                if (row0 + (uint32_t)rt * 32u >= p.rows || tok0 + (uint32_t)ct * 32u >= p.tokens)
                    continue;
                const uint32_t r = row0 + (uint32_t)rt * 32u + lane_r, tok = tok0 + (uint32_t)ct * 32u;
                su32x4 v[2][2];                                 // of the line's first and second 64 bytes, tokens n and n + 16
                if constexpr (OUT_BF16) {
#pragma unroll
                    for (int z = 0; z < 2; z++) {
                        take_sums(acc[rt + z][ct]);
                        // lanes l, l + 32 exchange quads so that each holds eight consecutive rows of its token, then l, l + 16
                        // so that the four lanes of a token hold its 32 rows
                        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                        typedef float f32x2 __attribute__((ext_vector_type(2)));
                        uint32_t d[8], e[2][4];
#pragma unroll
                        for (int q = 0; q < 8; q++) {
                            union { bf16x2 h; uint32_t u; } cv;
                            cv.h = __builtin_convertvector(f32x2{acc[rt + z][ct][2 * q], acc[rt + z][ct][2 * q + 1]}, bf16x2);
                            d[q] = cv.u;
                        }
#pragma unroll
                        for (int q = 0; q < 2; q++)
#pragma unroll
                            for (int k = 0; k < 2; k++) {
                                const auto x = __builtin_amdgcn_permlane32_swap(d[4 * q + k], d[4 * q + 2 + k], false, false);
                                e[q][k] = x[0];
                                e[q][2 + k] = x[1];
                            }
#pragma unroll
                        for (int k = 0; k < 4; k++) {
                            const auto x = __builtin_amdgcn_permlane16_swap(e[0][k], e[1][k], false, false);
                            v[z][0][k] = x[0];
                            v[z][1][k] = x[1];
                        }
                    }
                } else {
                    take_sums(acc[rt][ct]);
                    // lanes l, l + 16 exchange quads so that the four lanes of a token hold sixteen of its rows
#pragma unroll
                    for (uint32_t q = 0; q < 2; q++)
#pragma unroll
                        for (int k = 0; k < 4; k++) {
                            const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[rt][ct][8 * q + k]),
                                                                            __float_as_uint(acc[rt][ct][8 * q + 4 + k]), false, false);
                            v[q][0][k] = x[0];
                            v[q][1][k] = x[1];
                        }
                }
                put_pair(tok, r, v[0][0], v[1][0]);
                put_pair(tok + 16u, r, v[0][1], v[1][1]);
            }
        }
        return whole;
    };

    set_tile(0);
#pragma unroll
    for (int g = 0; g < kTileRing; g++) {
#pragma unroll
        for (int i = 0; i < kCopies; i++)
            copy_piece(i);
        copied();
    }
    // The next step is in LDS, for every wavefront.  The copies of the step after it may be in flight (those of the one after
    // that are issued behind the barrier), and so may the stores of a tile if they were issued after the copies of the step.
    uint32_t stored = 0;                                        // arrivals for which the last tile's stores count
    auto arrive = [&]() {
        constexpr int kFlight = (kTileRing - 2) * kCopies;
        if (stored)
            wait_copies<(kFlight + kStores < 63 ? kFlight + kStores : 63)>();
        else
            wait_copies<kFlight>();
        stored -= stored ? 1u : 0u;
        asm volatile("s_barrier" ::: "memory");
    };
    Frag f[2];
    wait_copies<(kTileRing - 1) * kCopies>();
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < kReads; i++)
        read_piece(f[0], 0, 0, i);
    wait_lds_reads();
    uint32_t image = 0;                                         // image being multiplied
    for (uint32_t mj = 0; mj < my_tiles; mj++) {
#pragma unroll
        for (int i = 0; i < RT; i++)
#pragma unroll
            for (int j = 0; j < CT; j++)
                acc[i][j] = (f32x16)(0.f);
        uint32_t k = 0;
        do {                                                    // steps is not zero: no path on which the sums stay as they are
            const uint32_t next = image == (kTileRing - 1) * kImage ? 0 : image + kImage;
            half(f[0], f[1], image, 1, std::false_type{});
            arrive();
            half(f[1], f[0], next, 0, std::true_type{});
            image = next;
        } while (++k < steps);
        sums_ready();
        stored = store_tile(mj) ? kTileRing - 1u : 0u;
    }
    wait_copies<0>();                                           // the last copies land while the workgroup still owns its LDS
}

// The kernels of the tile sizes of kSpmmTile: fp32, bf16 results.
typedef void (*spmm_kernel_t)(const SpmmArgs);
static const spmm_kernel_t kSpmmKernels[kSpmmTiles][2] = {
    {spmm24_ksplit_kernel<1, 1, 4, 4, false>, spmm24_ksplit_kernel<1, 1, 4, 4, true>},
    {spmm24_ksplit_kernel<2, 2, 4, 4, false>, spmm24_ksplit_kernel<2, 2, 4, 4, true>},
    {spmm24_ksplit_kernel<4, 4, 4, 3, false>, spmm24_ksplit_kernel<4, 4, 4, 3, true>},
    {spmm24_ksplit_kernel<8, 4, 4, 2, false>, spmm24_ksplit_kernel<8, 4, 4, 2, true>},
    {spmm24_tile_kernel<2, 2, false>, spmm24_tile_kernel<2, 2, true>},
    {spmm24_tile_kernel<2, 4, false>, spmm24_tile_kernel<2, 4, true>},
    {spmm24_tile_kernel<4, 4, false>, spmm24_tile_kernel<4, 4, true>},
};

}  // namespace tmask

using namespace tmask;

extern "C" int tmask_spmm24(const void *vals, const void *idx, int64_t rows, int64_t cols, const void *x, int64_t ld_x,
                            void *y, int64_t ld_y, int64_t tokens, tmask_dtype out_dt, void *hip_stream)
{
    if (!vals || !idx || !x || !y)
        return fail(TMASK_ERR_NULL, "vals, idx, x or y is NULL");
    if (out_dt != TMASK_F32 && out_dt != TMASK_BF16)
        return fail(TMASK_ERR_DTYPE, "unknown output dtype %d", (int)out_dt);
    if (rows <= 0 || cols <= 0 || tokens <= 0 || rows % 4 || cols % kSpKS || ld_x < cols || ld_y < rows)
        return fail(TMASK_ERR_SHAPE,
                    "rows=%lld (multiple of 4) cols=%lld (multiple of 64) tokens=%lld ld_x=%lld (>= cols) ld_y=%lld (>= rows)",
                    (long long)rows, (long long)cols, (long long)tokens, (long long)ld_x, (long long)ld_y);
    if (rows > 0x7FFFFFFFll || tokens > 0x7FFFFFFFll || ld_y > 0x7FFFFFFFll || cols > (1ll << 22) || ld_x > (1ll << 22))
        return fail(TMASK_ERR_SHAPE, "rows, tokens, ld_y must stay below 2^31, cols and ld_x at or below 2^22");
    const int64_t ysz = out_dt == TMASK_F32 ? 4 : 2;
    if (((uintptr_t)vals & 15) || ((uintptr_t)idx & 7) || ((uintptr_t)x & 15) || (ld_x % 8) || ((uintptr_t)y & 15) ||
        (ld_y * ysz) % 16)
        return fail(TMASK_ERR_ALIGN,
                    "vals, x, y must be 16-byte aligned, idx 8-byte aligned, ld_x a multiple of 8, ld_y*sizeof(y) a multiple of 16");
    SpmmArgs p;
    p.vals = vals; p.idx = idx; p.x = x; p.y = y;
    p.rows = (uint32_t)rows; p.cols = (uint32_t)cols; p.tokens = (uint32_t)tokens;
    p.ld_x = (uint32_t)ld_x; p.ld_y = (uint32_t)ld_y;
    if ((uint64_t)((rows + 255) / 256) * (uint64_t)((tokens + 127) / 128) > 0x7FFFFFFFull)    // 256 x 256 tiles always fit below that
        return fail(TMASK_ERR_SHAPE, "too many tiles");
    const uint64_t cus = (uint64_t)cu_count();
    const int choice = spmm_choose(rows, cols, tokens, out_dt == TMASK_F32, cus);
    if (choice < 0)
        return fail(TMASK_ERR_SHAPE, "too many tiles");
    const SpmmTile &tile = kSpmmTile[choice];
    p.tiles_r = (uint32_t)((rows + tile.rows - 1) / tile.rows);
    p.tiles_t = (uint32_t)((tokens + tile.tokens - 1) / tile.tokens);
    uint32_t grid = p.tiles_r * p.tiles_t;
    if (tile.persistent && grid > tile.persistent * cus)
        grid = (uint32_t)(tile.persistent * cus) & ~7u;         // a multiple of the XCD count, which the tile numbering assumes
    // Whole lines by streaming stores where y and its pitch are multiples of 64 bytes and a token's results fill a line: at other
    // pitches lines are cut, and the streaming stores lose (512 columns, 8192 tokens, plain / streaming us: fp32 1000 rows 15 /
    // 21, 1004 15.0 / 16.5, 1032 18.4 / 23.0, 1040 (64 bytes) 19.0 / 18.0, 1120 (128) 19.8 / 18.0; bf16 1032 16.1 / 16.6,
    // 1040 (32) 16.2 / 16.1, 1056 (64) 16.5 / 15.7, 1088 (128) 17.0 / 15.8; 2052 22.4 / 23.8).
    p.lines = (((uintptr_t)y | (uintptr_t)(ld_y * ysz)) & 63) == 0 && rows * ysz >= 128;
    hipStream_t stream = (hipStream_t)hip_stream;
    {
        ProfileScope prof(stream, true);
        hipLaunchKernelGGL(kSpmmKernels[choice][out_dt == TMASK_BF16 ? 1 : 0], dim3(grid), dim3(kSpmmThreads), 0, stream, p);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_fail(e, "spmm kernel launch");
    return TMASK_OK;
}
