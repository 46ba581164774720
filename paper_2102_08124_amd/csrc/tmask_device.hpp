// Device-side building blocks shared by the tmask kernels (gfx950 only).
//
// Data layout ("strip" layout).  A lane owns a 16-byte-wide column strip of a block-row: C = 4 fp32
// or 8 bf16 consecutive columns, all M rows.  Consecutive lanes own consecutive strips, so every
// global load instruction of a wavefront reads one contiguous 1 KiB run of a matrix row, and mask
// rows are written as contiguous 256 B / 512 B runs.
//   M*sizeof(elem) == 16 : one lane = one block            (fp32 M=4, bf16 M=8)
//   M*sizeof(elem)  > 16 : G = M/C adjacent lanes = one block (fp32 M=8: 2, M=16: 4; bf16 M=16: 2);
//                          column-direction work is lane-local, row-direction work crosses the G
//                          lanes with DPP quad permutes (G lanes are an aligned part of a quad)
//   M*sizeof(elem)  < 16 : one lane = B = 2 adjacent blocks (bf16 M=4)
// Narrow strips (kBF16N): bf16 at M = 4 in strips of 8 bytes, one block per lane, for matrices that are only 8-byte
// aligned (a width that is a multiple of four, not of eight); everything past the load is as at fp32 M = 4.
// Strips of a matrix are numbered block-row-major; a workgroup handles 256 consecutive strips.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tmask {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Store with the non-temporal hint, for data this kernel does not read again.  (Plain stores look up to 10 %
// faster when a benchmark rewrites one output buffer over and over, because part of it then stays in the
// memory-side cache; with fresh output buffers they are 5-20 % slower than these.)
template <typename T>
__device__ __forceinline__ void stream_store(T v, T *p)
{
    __builtin_nontemporal_store(v, p);
}

constexpr int kF32 = 0;
constexpr int kBF16 = 1;
constexpr int kBF16N = 2;            // bf16 in strips of 8 bytes; exists at M = 4
constexpr int kMaskU8 = 0;
constexpr int kMaskBits = 1;
constexpr int kThreads = 256;        // workgroup size of the streaming kernels
constexpr int kMaxBatch = 256;       // matrices per launch (descriptor table travels as kernel argument, 14 KiB)

// One matrix as the kernels see it, 56 bytes.  The table of a launch is passed by value: the kernel-argument
// segment takes tens of KiB (launches with 64 KiB of arguments were checked on the device), workgroups read only the
// entries their binary search touches, with scalar loads, and nothing has to be uploaded or allocated per call.
struct MatDev {
    const void *w;
    void *mask;
    void *aux;           // masks: the objective; score: per-block objective base for this matrix (float*); dense: the output
    uint32_t ld;         // elements
    uint32_t mask_ld;    // bytes
    uint32_t spr;        // strips per block-row = cols / C
    uint32_t n_strips;   // spr * rows / M
    uint32_t div_mul;    // s / spr == (uint64(s) * div_mul) >> div_shift for s < 2^31
    uint32_t div_shift;
    uint32_t tile0;      // first workgroup of this matrix inside the launch
    uint32_t pad;        // masks, score: workgroups of this matrix; dense: leading dimension of the output
};

// Which matrix does workgroup `tile` belong to?  A binary search over the table costs a chain of dependent scalar
// loads before a workgroup can issue its first vector load (eight for 144 matrices: several percent of a workgroup's
// life).  The host therefore adds a coarse index: the workgroups of a launch are cut into at most 256 buckets of
// 2^shift, and entry b packs the matrix of the bucket's first workgroup (low half) with that of the next bucket's
// first workgroup (high half).  One load narrows the search to that range, usually a single matrix.
constexpr int kCoarse = 256;

template <int N>
struct CoarseIndex {
    uint32_t shift;
    uint32_t e[N];
};

// How the workgroups of a launch hand their partial results to the one that adds up those of a matrix: see take_words.
// a = 0: they leave them for a second launch.
struct Tags {
    uint32_t a, b;
};

// CAP matrices.  The arguments of a launch are copied to where the device reads them, 16 KB in about a microsecond, and a small
// call has little else to do; so Algorithm 1, its masked copies and the compressions at N = M/2, the optimal 2:4 and the scores exist
// with a table of eight too.  Back to back, us: masked copy 256^2 .. 1024^2 5.4 -> 4.2, optimal 2:4 of 512^2 5.4 -> 4.6, masks at 4:8
// 5.3 -> 5.0, mask, compression and score of 1000 x 2052 22.7 -> 21.1.  The others have the large table alone: the optimal masks at M =
// 8, 16 would gain 0.2 us of 14 or more; other N, row pruning, the one-pass compression and the column-per-lane kernels are not
// measured with a small one (a mask of 512^2 fp32 without objective takes 3.3 us at 2:4, 4.2 at 1:4).
template <int CAP>
struct BatchArgsOf {
    MatDev m[CAP];
    CoarseIndex<CAP == kMaxBatch ? kCoarse : 16> ci;
    uint32_t n_mats;
    uint32_t K;          // pruned per row/column = M - N
    uint32_t N;
    uint32_t partial0;   // index of this launch's first partial in the workspace
    void *partials;      // workspace
    Tags tags;
    struct ScorePartial *score;   // score: the results, one per matrix of the launch
};
using BatchArgs = BatchArgsOf<kMaxBatch>;

constexpr int kFewMats = 8;
using FewArgs = BatchArgsOf<kFewMats>;

// What a workgroup of the score kernels leaves to be added up; the results of the call have the same layout.
struct ScorePartial {
    double retained, total;
    unsigned long long kept, rowv, colv, rowne, colne;
};

static_assert(sizeof(BatchArgs) <= 16384, "descriptor table is sized to stay a small kernel argument");

template <int DT, int M>
struct Geo {
    static constexpr int ES = (DT == kF32) ? 4 : 2;          // element bytes
    static constexpr int C = DT == kBF16 ? 8 : 4;            // columns per strip
    static constexpr int G = (M > C) ? M / C : 1;            // lanes per block
    static constexpr int B = (M < C) ? C / M : 1;            // blocks per lane
    static constexpr int CL = C / B;                         // columns of one block inside a lane
};

// ---- cross-lane helpers -------------------------------------------------------------------------

// Value of lane (lane ^ X) within the quad, X in {1,2,3}: DPP quad_perm.
template <int X>
__device__ __forceinline__ uint32_t quad_xor(uint32_t v)
{
    constexpr int ctrl = (X == 1) ? 0xB1 : (X == 2) ? 0x4E : 0x1B;   // [1,0,3,2] [2,3,0,1] [3,2,1,0]
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, 0xF, 0xF, false);
}

// v + the value of lane (lane ^ X) within the quad.  The source lane always exists and every lane is enabled, so
// "0 where the source is missing" never applies; written that way the move folds into the add (v_add_u32_dpp).
template <int X>
__device__ __forceinline__ uint32_t quad_xor_sum(uint32_t v)
{
    constexpr int ctrl = (X == 1) ? 0xB1 : (X == 2) ? 0x4E : 0x1B;
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xF, 0xF, true);
}

// max / min of a and the value that lane (lane ^ X) of the quad holds in o, the move folded into the operation the same
// way (v_max_u32_dpp / v_min_u32_dpp: one instruction, and no wait states between a move and its use).
template <int X>
__device__ __forceinline__ uint32_t quad_xor_max(uint32_t a, uint32_t o)
{
    constexpr int ctrl = (X == 1) ? 0xB1 : (X == 2) ? 0x4E : 0x1B;
    const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)o, ctrl, 0xF, 0xF, true);
    return a > y ? a : y;
}

template <int X>
__device__ __forceinline__ uint32_t quad_xor_min(uint32_t a, uint32_t o)
{
    constexpr int ctrl = (X == 1) ? 0xB1 : (X == 2) ? 0x4E : 0x1B;
    const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)o, ctrl, 0xF, 0xF, true);
    return a < y ? a : y;
}

// A wavefront-wide boolean: bit l = the predicate in lane l.  Held in a scalar register pair, so
// logic on it is scalar-ALU work.
typedef unsigned long long lanemask_t;

__device__ __forceinline__ lanemask_t lm(bool pred) { return __builtin_amdgcn_ballot_w64(pred); }
__device__ __forceinline__ bool lm_test(lanemask_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

__device__ __forceinline__ lanemask_t maj3(lanemask_t x, lanemask_t y, lanemask_t z)
{
    return (x & y) | (z & (x | y));
}

// r += 1 in the lanes whose bit is set in m: one add-with-carry-in, the carry being the lane mask.
__device__ __forceinline__ void lm_inc(uint32_t &r, lanemask_t m)
{
    lanemask_t carry_out;
    asm("v_addc_co_u32_e64 %0, %1, 0, %0, %2" : "+v"(r), "=s"(carry_out) : "s"(m));
}

// r = 2 r + (1 in the lanes whose bit is set in m): shifts a flag into a bit word, one add-with-carry-in.
__device__ __forceinline__ void lm_shift_in(uint32_t &r, lanemask_t m)
{
    lanemask_t carry_out;
    asm("v_addc_co_u32_e64 %0, %1, %0, %0, %2" : "+v"(r), "=s"(carry_out) : "s"(m));
}

// Wavefront sums by DPP, in a fixed order (deterministic): quad, then the four quads of a row of 16
// lanes by row rotation, then the four rows through scalar reads.  All 64 lanes must be active.
// The result is uniform.
constexpr int kRowHalfMirror = 0x141, kRowRor8 = 0x128, kRowNewbcast = 0x150;     // lane l of sixteen reads lane l ^ 7, l ^ 8, the one given

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_read(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, false);
}

// go(std::integral_constant<int, I>) for I = 0 ... M - 1: lane numbers within DPP controls are constants of the instruction.
template <int M, int I = 0, typename Go>
__device__ __forceinline__ void each_of(Go &&go)
{
    if constexpr (I < M) {
        go(std::integral_constant<int, I>{});
        each_of<M, I + 1>(go);
    }
}

// What lane I of the M = 8 or 16 lanes of a block (an aligned part of sixteen lanes) holds.
template <int M, int I>
__device__ __forceinline__ uint32_t of_lane(uint32_t v)
{
    static_assert(M == 8 || M == 16, "a row of sixteen lanes or half of one");
    if constexpr (M == 16) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowNewbcast + I, 0xF, 0xF, true);
    } else {
        const int low = __builtin_amdgcn_update_dpp(0, (int)v, kRowNewbcast + I, 0xF, 0x3, true);
        return (uint32_t)__builtin_amdgcn_update_dpp(low, (int)v, kRowNewbcast + 8 + I, 0xF, 0xC, false);
    }
}

__device__ __forceinline__ float wave_sum(float v)
{
    v += __uint_as_float(dpp_read<0xB1>(__float_as_uint(v)));    // quad_perm [1,0,3,2]
    v += __uint_as_float(dpp_read<0x4E>(__float_as_uint(v)));    // quad_perm [2,3,0,1]
    v += __uint_as_float(dpp_read<0x124>(__float_as_uint(v)));   // row_ror:4
    v += __uint_as_float(dpp_read<0x128>(__float_as_uint(v)));   // row_ror:8
    const uint32_t u = __float_as_uint(v);
    return (__uint_as_float(__builtin_amdgcn_readlane(u, 0)) + __uint_as_float(__builtin_amdgcn_readlane(u, 16))) +
           (__uint_as_float(__builtin_amdgcn_readlane(u, 32)) + __uint_as_float(__builtin_amdgcn_readlane(u, 48)));
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
    v += dpp_read<0xB1>(v);
    v += dpp_read<0x4E>(v);
    v += dpp_read<0x124>(v);
    v += dpp_read<0x128>(v);
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
           __builtin_amdgcn_readlane(v, 48);
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off, 64);
    return v;
}

// Sum over the workgroup in a fixed tree order (deterministic); result valid in thread 0.
template <typename T>
__device__ __forceinline__ T block_sum(T v, T *lds /* kThreads/64 entries */)
{
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        lds[wave] = v;
    __syncthreads();
    T r = lds[0];
#pragma unroll
    for (int k = 1; k < kThreads / 64; k++)
        r += lds[k];
    __syncthreads();
    return r;
}

// Sum over a wavefront of what its lanes keep: fp32, in fp64 for narrow strips, whose 1024 values of eight bits no longer
// add up exactly in fp32 (the column-per-lane kernels, which read such matrices otherwise, add 256 at a time: objective
// against 64 bits 2e-11, 6e-10 in fp32).
template <int DT>
__device__ __forceinline__ double wave_kept(float v)
{
    if constexpr (DT == kBF16N)
        return wave_sum((double)v);
    else
        return (double)wave_sum(v);
}

// Workgroup sum of per-thread fp32 values: inside a wavefront as above, fp64 across wavefronts.
template <int DT = kF32, int NT = kThreads>
__device__ __forceinline__ double block_sum_f32(float v, double *lds /* NT/64 entries */)
{
    const double w = wave_kept<DT>(v);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        lds[wave] = w;
    __syncthreads();
    double r = lds[0];
#pragma unroll
    for (int k = 1; k < NT / 64; k++)
        r += lds[k];
    return r;
}

// ---- partial results, added up in the launch that leaves them ----------------------------------------------------------
//
// A second launch that adds a workgroup's partial results costs 3-4 us on the device and 2 on the host, as much as a small
// matrix takes; counting the workgroups that are done needs a counter that is zero when the launch begins, and the
// workspace holds anything.  So a partial result travels as words of 32 bits of it beside 32 bits of tag, which the host
// draws for each launch, and the last workgroup of a matrix reads the words of the others until their tags are right: every
// word proves by itself that it was written by this launch.  It then clears them, so that a captured launch, whose tags are
// the same each time it is replayed, finds none of its own.  (Contents of a workspace pass for a result only if they hold both
// 32-bit tags of a call in the right places, two tags that differ and are drawn anew for each call.)
// The wait ends: so few workgroups wait at a time that every workgroup finds a place that none of them holds (see kMostWaiting),
// and those that are waited for wait for nobody.  Should a result never come, a wavefront gives up after kMostReads reads, 1-3 us
// each, that found something missing, and the sum is NaN.

constexpr uint32_t kMostReads = 1u << 21;     // by a wavefront, of all the records that it takes: 2-6 s

__device__ __forceinline__ void put_word(unsigned long long *at, uint32_t value, uint32_t tag)
{
    __hip_atomic_store(at, ((unsigned long long)tag << 32) | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long get_word(const unsigned long long *at)
{
    return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The words of a record (even ones tagged a, odd ones b), cleared when all of them are there.  The lanes of a wavefront read
// together until each has its record, at most `left` times in vain, a number that they share and that later records have less of;
// false if the record has not come by then.  (A lane that has its record reads it again: keeping it would take registers.)  A
// read goes to memory and takes 2-3 us behind what the chip has in flight; four records at a time took registers, and with them a
// wavefront of occupancy, for no gain.
template <int W>
__device__ __forceinline__ bool take_words(unsigned long long *at, const Tags &tags, uint32_t (&v)[W], uint32_t &left)
{
    bool all;
    for (;;) {
        unsigned long long w[W];
#pragma unroll
        for (int k = 0; k < W; k++)
            w[k] = get_word(at + k);
        uint32_t wrong = 0u;                      // not a chain of &&: its branches took 20 registers with a score's seven words
#pragma unroll
        for (int k = 0; k < W; k++) {
            v[k] = (uint32_t)w[k];
            wrong |= (uint32_t)(w[k] >> 32) ^ ((k & 1) ? tags.b : tags.a);
        }
        all = wrong == 0u;
        if (!__any(!all) || left == 0u)
            break;
        left--;
        __builtin_amdgcn_s_sleep(1);
    }
    if (all) {
#pragma unroll
        for (int k = 0; k < W; k++)
            __hip_atomic_store(at + k, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return all;
}

__device__ __forceinline__ double words_as_double(uint32_t lo, uint32_t hi, bool came)
{
    return came ? __hiloint2double((int)hi, (int)lo) : __hiloint2double(0x7FF80000, 0);
}

// Where a workgroup's part of a sum goes: the workgroup is number `which` of `others` + 1.
struct Handover {
    void *dst;                       // of the whole sum; null: nobody asked for it
    unsigned long long *records;     // of the matrix' workgroups
    uint32_t a, b, which, others;
};

// partials: the workspace or null; index: the workgroup's number among all of the call; which of count: among its matrix'; SIZE
// of a result for a second launch, which is then the whole of the sum; WORDS of a record.
template <int SIZE, int WORDS, bool EARLY = true>
__device__ __forceinline__ Handover handover(void *partials, const Tags &tags, uint32_t index, uint32_t which, uint32_t count, void *dst)
{
    const bool tagged = tags.a != 0u;
    Handover h;
    h.dst = !partials ? nullptr : tagged ? dst : (void *)((char *)partials + (size_t)index * SIZE);
    h.records = (unsigned long long *)partials + (size_t)(index - which) * WORDS;
    h.a = tags.a;
    h.b = tags.b;
    h.which = tagged ? which : 0u;
    h.others = tagged ? count - 1u : 0u;
    // Read now, with the descriptor: at the workgroup's end these would be a chain of scalar loads that nothing overlaps
    // (4096 x 3072 bf16, 16:32: 15.2 / 14.95 us).
    if constexpr (EARLY)
        asm volatile("" : "+s"(h.dst), "+s"(h.records), "+s"(h.a), "+s"(h.b), "+s"(h.which), "+s"(h.others));
    return h;
}

// Leaves t (the same in every thread) in the workgroup's record, or, as the last workgroup of its matrix, adds all of them to
// *dst (not null), in the order of objective_reduce_kernel<256>: result i by thread i mod 256, one after the other, then each
// wavefront, then the four.  red: a double of LDS for each wavefront (THREADS = 64: unused, a lane does the work of four; 512: the
// upper four wavefronts have none to do).
template <int THREADS>
__device__ __forceinline__ void hand_over(const Handover &h, double t, double *red)
{
    const Tags tags{h.a, h.b};
    if (h.which != h.others) {
        if (threadIdx.x == 0) {
            const unsigned long long bits = (unsigned long long)__double_as_longlong(t);
            put_word(h.records + 2u * h.which, (uint32_t)bits, tags.a);
            put_word(h.records + 2u * h.which + 1u, (uint32_t)(bits >> 32), tags.b);
        }
        return;
    }
    if (h.others == 0u) {
        if (threadIdx.x == 0)
            *(double *)h.dst = t;
        return;
    }
    static_assert(THREADS == 64 || THREADS == kThreads || THREADS == 2 * kThreads, "the order above");
    double total = 0.0;
    uint32_t left = kMostReads;
#pragma nounroll
    for (uint32_t q = 0; q < (uint32_t)kThreads; q += THREADS) {
        const uint32_t first = threadIdx.x + q;
        double sum = 0.0;
#pragma nounroll
        for (uint32_t i = THREADS > kThreads && first >= (uint32_t)kThreads ? h.others : first; i < h.others; i += kThreads) {
            uint32_t v[2];
            const bool came = take_words<2>(h.records + 2u * i, tags, v, left);
            sum += words_as_double(v[0], v[1], came);
        }
        if (h.others % kThreads == first)
            sum += t;
        sum = wave_sum(sum);
        total = q == 0 ? sum : total + sum;
    }
    if constexpr (THREADS > 64) {
        __syncthreads();                          // what red held has been read
        if ((threadIdx.x & 63u) == 0)
            red[threadIdx.x >> 6] = total;
        __syncthreads();
        total = ((red[0] + red[1]) + red[2]) + red[3];
    }
    if (threadIdx.x == 0)
        *(double *)h.dst = total;
}

// The objective of the strip kernels.
template <int CAP>
__device__ __forceinline__ Handover objective_of(const BatchArgsOf<CAP> &args, const MatDev &md, uint32_t tile)
{
    return handover<8, 2>(args.partials, args.tags, args.partial0 + tile, tile - md.tile0, md.pad, md.aux);
}

// What a workgroup of the score kernels counts: at most 2^15 entries each (256 lanes x 128), so two counts share a word, and
// those of a matrix' workgroups that hand theirs over add up in 32 bits.
struct ScoreSums {
    double retained, total;
    uint32_t kept, rowv, colv, rowne, colne;
};

// The same for the seven sums of a score.
template <int THREADS>
__device__ __forceinline__ void hand_over_score(const Handover &h, ScoreSums own)
{
    constexpr int W = 7;
    const Tags tags{h.a, h.b};
    if (h.which != h.others) {
        if (threadIdx.x == 0) {
            const unsigned long long r = (unsigned long long)__double_as_longlong(own.retained);
            const unsigned long long t = (unsigned long long)__double_as_longlong(own.total);
            const uint32_t v[W] = {(uint32_t)r, (uint32_t)(r >> 32), (uint32_t)t, (uint32_t)(t >> 32), own.kept | (own.rowv << 16),
                                   own.colv | (own.rowne << 16), own.colne};
#pragma unroll
            for (int k = 0; k < W; k++)
                put_word(h.records + (size_t)W * h.which + k, v[k], (k & 1) ? tags.b : tags.a);
        }
        return;
    }
    ScorePartial *const dst = (ScorePartial *)h.dst;
    if (h.others == 0u) {
        if (threadIdx.x == 0)
            *dst = ScorePartial{own.retained, own.total, own.kept, own.rowv, own.colv, own.rowne, own.colne};
        return;
    }
    if (threadIdx.x != 0)
        own = ScoreSums{};
    uint32_t left = kMostReads;
#pragma nounroll
    for (uint32_t i = threadIdx.x; i < h.others; i += THREADS) {
        uint32_t v[W];
        const bool came = take_words<W>(h.records + (size_t)W * i, tags, v, left);
        own.retained += words_as_double(v[0], v[1], came);
        own.total += words_as_double(v[2], v[3], came);
        own.kept += v[4] & 0xFFFFu; own.rowv += v[4] >> 16;
        own.colv += v[5] & 0xFFFFu; own.rowne += v[5] >> 16;
        own.colne += v[6];
    }
    own = ScoreSums{wave_sum(own.retained), wave_sum(own.total), wave_sum(own.kept), wave_sum(own.rowv), wave_sum(own.colv),
                    wave_sum(own.rowne), wave_sum(own.colne)};
    if constexpr (THREADS > 64) {
        __shared__ ScoreSums sums[THREADS / 64];
        if ((threadIdx.x & 63u) == 0)
            sums[threadIdx.x >> 6] = own;
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 1; k < THREADS / 64; k++) {
                const ScoreSums o = sums[k];
                own.retained += o.retained; own.total += o.total;
                own.kept += o.kept; own.rowv += o.rowv; own.colv += o.colv; own.rowne += o.rowne; own.colne += o.colne;
            }
        }
    }
    if (threadIdx.x == 0)
        *dst = ScorePartial{own.retained, own.total, own.kept, own.rowv, own.colv, own.rowne, own.colne};
}

// ---- tile addressing ----------------------------------------------------------------------------

// Which matrix of the batch does workgroup `tile` belong to (largest m with tile0[m] <= tile).
template <int CAP>
__device__ __forceinline__ int find_matrix(const BatchArgsOf<CAP> &a, uint32_t tile)
{
    const uint32_t e = a.ci.e[tile >> a.ci.shift];
    int lo = (int)(e & 0xFFFFu), hi = (int)(e >> 16);
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (a.m[mid].tile0 <= tile)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

struct StripPos {
    uint32_t br;   // block-row
    uint32_t sc;   // strip column inside the block-row
};

__device__ __forceinline__ StripPos strip_pos(const MatDev &md, uint32_t s)
{
    StripPos p;
    p.br = (uint32_t)(((uint64_t)s * md.div_mul) >> md.div_shift);
    p.sc = s - p.br * md.spr;
    return p;
}

// ---- strip load / store -------------------------------------------------------------------------

// Loads the lane's strip: a[i][c] = |W| as an fp32 bit pattern (bf16 widened by << 16), i.e. the
// magnitude ordering key, and raw[i] = the untouched 16 (kBF16N: 8) bytes of row i.
template <int DT, int M>
__device__ __forceinline__ void load_strip(const MatDev &md, StripPos p, uint32_t (&a)[M][Geo<DT, M>::C],
                                           u32x4 (&raw)[M])
{
    constexpr int C = Geo<DT, M>::C;
    const char *base = (const char *)md.w + ((size_t)p.br * M * md.ld + (size_t)p.sc * C) * Geo<DT, M>::ES;
    const size_t row_bytes = (size_t)md.ld * Geo<DT, M>::ES;
#pragma unroll
    for (int i = 0; i < M; i++) {
        if constexpr (DT == kBF16N) {
            const u32x2 v = __builtin_nontemporal_load((const u32x2 *)(base + i * row_bytes));
            raw[i] = u32x4{v.x, v.y, 0u, 0u};
        } else {
            raw[i] = __builtin_nontemporal_load((const u32x4 *)(base + i * row_bytes));
        }
    }
#pragma unroll
    for (int i = 0; i < M; i++) {
        const uint32_t d[4] = {raw[i].x, raw[i].y, raw[i].z, raw[i].w};
        if constexpr (DT == kF32) {
#pragma unroll
            for (int c = 0; c < 4; c++)
                a[i][c] = d[c] & 0x7FFFFFFFu;
        } else {
#pragma unroll
            for (int c = 0; c < C / 2; c++) {
                a[i][2 * c] = (d[c] << 16) & 0x7FFF0000u;
                a[i][2 * c + 1] = d[c] & 0x7FFF0000u;
            }
        }
    }
}

// Spread the low 4 bits of b into 4 bytes (bit k -> byte k, value 0/1).
__device__ __forceinline__ uint32_t bits_to_bytes4(uint32_t b)
{
    return (b | (b << 7) | (b << 14) | (b << 21)) & 0x01010101u;
}

__device__ __forceinline__ uint32_t bytes4_to_bits(uint32_t v)
{
    // any non-zero byte counts as kept
    uint32_t nz = ((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v;       // bit 7 of each byte = byte != 0
    nz = (nz >> 7) & 0x01010101u;
    return (nz | (nz >> 7) | (nz >> 14) | (nz >> 21)) & 0xFu;
}

// Writes the lane's C keep-bits of each of the M rows (bit c of rowbits[i] = column c kept).
template <int DT, int M, int FMT>
__device__ __forceinline__ void store_mask(const MatDev &md, StripPos p, const uint32_t (&rowbits)[M])
{
    constexpr int C = Geo<DT, M>::C;
    if constexpr (FMT == kMaskU8) {
        char *base = (char *)md.mask + (size_t)p.br * M * md.mask_ld + (size_t)p.sc * C;
#pragma unroll
        for (int i = 0; i < M; i++) {
            if constexpr (C == 4) {
                stream_store(bits_to_bytes4(rowbits[i]), (uint32_t *)(base + (size_t)i * md.mask_ld));
            } else {
                u32x2 v;
                v.x = bits_to_bytes4(rowbits[i] & 0xFu);
                v.y = bits_to_bytes4(rowbits[i] >> 4);
                stream_store(v, (u32x2 *)(base + (size_t)i * md.mask_ld));
            }
        }
    } else {
        // BITS: C bits per lane and row. fp32 (C=4): the even lane of a pair writes one byte built
        // from both lanes; bf16 (C=8): every lane writes its byte.
        char *base = (char *)md.mask + (size_t)p.br * M * md.mask_ld + (((size_t)p.sc * C) >> 3);
#pragma unroll
        for (int i = 0; i < M; i++) {
            if constexpr (C == 8) {
                base[(size_t)i * md.mask_ld] = (char)rowbits[i];
            } else {
                uint32_t other = quad_xor<1>(rowbits[i]);
                if ((threadIdx.x & 1) == 0)
                    base[(size_t)i * md.mask_ld] = (char)(rowbits[i] | (other << 4));
            }
        }
    }
}

// Reads the lane's C mask entries of each row into bit c of rowbits[i].
template <int DT, int M, int FMT>
__device__ __forceinline__ void load_mask(const MatDev &md, StripPos p, uint32_t (&rowbits)[M])
{
    constexpr int C = Geo<DT, M>::C;
    if constexpr (FMT == kMaskU8) {
        const char *base = (const char *)md.mask + (size_t)p.br * M * md.mask_ld + (size_t)p.sc * C;
#pragma unroll
        for (int i = 0; i < M; i++) {
            if constexpr (C == 4) {
                rowbits[i] = bytes4_to_bits(
                    __builtin_nontemporal_load((const uint32_t *)(base + (size_t)i * md.mask_ld)));
            } else {
                u32x2 v = __builtin_nontemporal_load((const u32x2 *)(base + (size_t)i * md.mask_ld));
                rowbits[i] = bytes4_to_bits(v.x) | (bytes4_to_bits(v.y) << 4);
            }
        }
    } else {
        const unsigned char *base =
            (const unsigned char *)md.mask + (size_t)p.br * M * md.mask_ld + (((size_t)p.sc * C) >> 3);
#pragma unroll
        for (int i = 0; i < M; i++) {
            uint32_t v = base[(size_t)i * md.mask_ld];
            if constexpr (C == 8)
                rowbits[i] = v;
            else
                rowbits[i] = (v >> ((p.sc & 1) * 4)) & 0xFu;
        }
    }
}

// Sum of the kept magnitudes of the lane's strip (fp32 within the strip).
template <int M, int C>
__device__ __forceinline__ float kept_sum(const uint32_t (&a)[M][C], const uint32_t (&rowbits)[M])
{
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < M; i++)
#pragma unroll
        for (int c = 0; c < C; c++)
            s += ((rowbits[i] >> c) & 1u) ? __uint_as_float(a[i][c]) : 0.f;
    return s;
}

}  // namespace tmask
