// Per-block solvers working on the strip layout (see tmask_device.hpp).
//   approx_keep   : Algorithm 1 of arXiv 2102.08124 (Sec. 4) in rank form
//   exact24_block : Eq. 3 optimum for 2:4 over all 90 feasible patterns (factored enumeration)
//   best_permutation4 : Eq. 3 optimum for 1:4 and 3:4 over the 24 permutations
//   exact_costs / exact_priced_start / exact_search : the pieces of the Eq. 3 optimum for M = 8, 16 by successive
//                   shortest augmenting paths on the bipartite row/column network of Fig. 3 (put together in
//                   tmask_exact_balance.hpp)
#pragma once
#include <type_traits>

#include "tmask_device.hpp"
#include "tmask_networks.hpp"

namespace tmask {

// =================================================================================================
// Algorithm 1 in rank form.
//
// Under the strict total order (magnitude key, then row-major index) the greedy sweep of
// Algorithm 1 -- take an entry while its row or its column has fewer than K taken entries --
// ends with exactly the entries that are among the K lightest of their row or of their column:
// the n-th lightest entry of a line (n <= K) meets fewer than K taken entries in that line when it
// is visited, and an entry outside the K lightest of both its lines finds both saturated.
// So  keep(i,j) <=> rank_in_row(i,j) >= K  and  rank_in_column(i,j) >= K,
// where rank = number of entries of the line that precede (i,j) in the order.  Because positions
// are static, "precedes" is `<=` against earlier positions and `<` against later ones.
// =================================================================================================

// rank bookkeeping for one ordered pair: `first` precedes `second` iff le.  Up to M = 8 the compare
// result stays a lane mask and feeds two add-with-carry instructions; at M = 16 that form costs
// registers and occupancy, plain 0/1 arithmetic is faster there.
template <int M>
__device__ __forceinline__ void rank_pair(bool le, uint32_t &r_first, uint32_t &r_second)
{
    if constexpr (M <= 8) {
        const lanemask_t m = lm(le);
        lm_inc(r_second, m);
        lm_inc(r_first, ~m);
    } else {
        const uint32_t v = le ? 1u : 0u;
        r_second += v;
        r_first += 1u - v;
    }
}

template <int M>
__device__ __forceinline__ void rank_one(bool precedes, uint32_t &r)
{
    if constexpr (M <= 8)
        lm_inc(r, lm(precedes));
    else
        r += precedes ? 1u : 0u;
}

// Column direction: all M rows of a column live in the lane.
// PIN: merge every flag into its row's bits at once.  Wanted at M = 16 when the flags are stored as bit masks:
// left alone the compiler carries all the compare results as lane masks to the place where the flags are
// stored (hundreds of spilled scalar registers, one wavefront per SIMD).  With byte masks the freer schedule is
// the faster one.
template <int M, int C, bool PIN = false>
__device__ __forceinline__ void col_rank_keep(const uint32_t (&a)[M][C], uint32_t K, uint32_t (&bits)[M])
{
#pragma unroll
    for (int i = 0; i < M; i++)
        bits[i] = 0;
#pragma unroll
    for (int c = 0; c < C; c++) {
        uint32_t r[M];
#pragma unroll
        for (int i = 0; i < M; i++)
            r[i] = 0;
#pragma unroll
        for (int i = 0; i < M; i++)
#pragma unroll
            for (int i2 = i + 1; i2 < M; i2++) {
                rank_pair<M>(a[i][c] <= a[i2][c], r[i], r[i2]);   // row i precedes row i2
            }
#pragma unroll
        for (int i = 0; i < M; i++) {
            bits[i] |= (r[i] >= K ? 1u : 0u) << c;
            if constexpr (PIN)
                asm volatile("" : "+v"(bits[i]));
        }
    }
}

// Row direction: a block-row is spread over G lanes (CL columns each); B blocks share a lane.
// gpos = position of the lane inside its group of G.  bits[i] &= row-keep.
template <int M, int C, int G, int B, bool PIN = false>
__device__ __forceinline__ void row_rank_keep(const uint32_t (&a)[M][C], uint32_t K, uint32_t gpos,
                                              uint32_t (&bits)[M])
{
    constexpr int CL = C / B;
#pragma unroll
    for (int i = 0; i < M; i++) {
        uint32_t keep = 0;
#pragma unroll
        for (int b = 0; b < B; b++) {
            uint32_t r[CL];
#pragma unroll
            for (int c = 0; c < CL; c++)
                r[c] = 0;
#pragma unroll
            for (int c = 0; c < CL; c++)
#pragma unroll
                for (int c2 = c + 1; c2 < CL; c2++) {
                    rank_pair<M>(a[i][b * CL + c] <= a[i][b * CL + c2], r[c], r[c2]);
                }
            if constexpr (G >= 2) {
                // keys are < 2^31, so "theirs <= mine" is "theirs < mine + 1"
                const uint32_t pb1 = ((gpos ^ 1u) < gpos) ? 1u : 0u;
#pragma unroll
                for (int c2 = 0; c2 < CL; c2++) {
                    const uint32_t t = quad_xor<1>(a[i][c2]);
#pragma unroll
                    for (int c = 0; c < CL; c++)
                        rank_one<M>(t < a[i][c] + pb1, r[c]);
                }
            }
            if constexpr (G == 4) {
                const uint32_t pb2 = ((gpos ^ 2u) < gpos) ? 1u : 0u;
                const uint32_t pb3 = ((gpos ^ 3u) < gpos) ? 1u : 0u;
#pragma unroll
                for (int c2 = 0; c2 < CL; c2++) {
                    const uint32_t t2 = quad_xor<2>(a[i][c2]);
                    const uint32_t t3 = quad_xor<3>(a[i][c2]);
#pragma unroll
                    for (int c = 0; c < CL; c++) {
                        rank_one<M>(t2 < a[i][c] + pb2, r[c]);
                        rank_one<M>(t3 < a[i][c] + pb3, r[c]);
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < CL; c++)
                keep |= (r[c] >= K ? 1u : 0u) << (b * CL + c);
        }
        bits[i] &= keep;
        if constexpr (PIN)
            asm volatile("" : "+v"(bits[i]));
    }
}

template <int DT, int M, bool PIN = false>
__device__ __forceinline__ void approx_keep(const uint32_t (&a)[M][Geo<DT, M>::C], uint32_t K, uint32_t gpos,
                                            uint32_t (&bits)[M])
{
    using Ge = Geo<DT, M>;
    col_rank_keep<M, Ge::C, PIN>(a, K, bits);
    row_rank_keep<M, Ge::C, Ge::G, Ge::B, PIN>(a, K, gpos, bits);
}

// =================================================================================================
// Exact 2:4: all 0/1 4x4 matrices with two ones in every row and column (there are 90), fp32 sums.
// A row pattern is a pair of columns; pairs are numbered 0..5 = {01,02,03,12,13,23}.
// =================================================================================================

struct Patterns24 {
    uint8_t p[90][4];
    int n;
};

constexpr int kPairX[6] = {0, 0, 0, 1, 1, 2};
constexpr int kPairY[6] = {1, 2, 3, 2, 3, 3};

constexpr uint32_t pair_bits(int p) { return (1u << kPairX[p]) | (1u << kPairY[p]); }

constexpr Patterns24 make_patterns24()
{
    Patterns24 t{};
    t.n = 0;
    for (int p0 = 0; p0 < 6; p0++)
        for (int p1 = 0; p1 < 6; p1++)
            for (int p2 = 0; p2 < 6; p2++)
                for (int p3 = 0; p3 < 6; p3++) {
                    bool ok = true;
                    for (int c = 0; c < 4; c++) {
                        int s = ((pair_bits(p0) >> c) & 1) + ((pair_bits(p1) >> c) & 1) +
                                ((pair_bits(p2) >> c) & 1) + ((pair_bits(p3) >> c) & 1);
                        ok = ok && (s == 2);
                    }
                    if (ok) {
                        t.p[t.n][0] = (uint8_t)p0; t.p[t.n][1] = (uint8_t)p1;
                        t.p[t.n][2] = (uint8_t)p2; t.p[t.n][3] = (uint8_t)p3;
                        t.n++;
                    }
                }
    return t;
}

constexpr Patterns24 kPatterns24 = make_patterns24();
static_assert(kPatterns24.n == 90, "a 4x4 block has 90 feasible 2:4 transposable patterns");

constexpr uint32_t pattern_mask16(int k)
{
    return pair_bits(kPatterns24.p[k][0]) | (pair_bits(kPatterns24.p[k][1]) << 4) |
           (pair_bits(kPatterns24.p[k][2]) << 8) | (pair_bits(kPatterns24.p[k][3]) << 12);
}

// The 90 patterns factor through the column-count vector left by rows 0 and 1: a pattern is a pair
// (p0, p1) for rows 0,1 with column counts v, and a pair (p2, p3) for rows 2,3 with counts 2 - v.
// There are 19 such vectors (6 of type 2200 reached by one pair of pairs, 12 of type 2110 reached by
// two, 1 of type 1111 reached by six: 6*1*1 + 12*2*2 + 1*6*6 = 90), so the optimum is
//     max over v of  best01[v] + best23[2 - v],
// with best01 / best23 the best pair sums of the upper / lower two rows for each vector: 72 sums and
// 19 combinations instead of 90 four-term sums.
struct Halves24 {
    int vec_of[36];      // (p, q) -> index of the count vector of pair_bits(p) + pair_bits(q)
    int first_of[36];    // 1 if (p, q) is the first pair of pairs with that vector (enumeration order)
    int compl_of[19];    // index of the vector 2 - v
    int n_vec;
};

constexpr int count_code(int p, int q)
{
    int code = 0, mul = 1;
    for (int c = 0; c < 4; c++) {
        code += mul * (int)(((pair_bits(p) >> c) & 1u) + ((pair_bits(q) >> c) & 1u));
        mul *= 3;
    }
    return code;
}

constexpr Halves24 make_halves24()
{
    Halves24 h{};
    int codes[36] = {};
    h.n_vec = 0;
    for (int k = 0; k < 36; k++) {
        const int code = count_code(k / 6, k % 6);
        int idx = -1;
        for (int j = 0; j < h.n_vec; j++)
            if (codes[j] == code)
                idx = j;
        h.first_of[k] = idx < 0 ? 1 : 0;
        if (idx < 0) {
            idx = h.n_vec;
            codes[h.n_vec++] = code;
        }
        h.vec_of[k] = idx;
    }
    for (int j = 0; j < h.n_vec; j++) {
        const int want = 80 - codes[j];       // (2,2,2,2) in base 3 is 80; digits never borrow
        h.compl_of[j] = -1;
        for (int i = 0; i < h.n_vec; i++)
            if (codes[i] == want)
                h.compl_of[j] = i;
    }
    return h;
}

constexpr Halves24 kHalves24 = make_halves24();
static_assert(kHalves24.n_vec == 19, "rows 0,1 of a 2:4 pattern leave 19 possible column-count vectors");

// Best pair of row patterns per count vector for rows (r, r+1): value and 8-bit mask (row r in bits 0..3).
__device__ __forceinline__ void best_pairs24(const float (&pa)[6], const float (&pb)[6], float (&val)[19],
                                             uint32_t (&msk)[19])
{
#pragma unroll
    for (int k = 0; k < 36; k++) {
        const int idx = kHalves24.vec_of[k];
        const float s = pa[k / 6] + pb[k % 6];
        const uint32_t m = pair_bits(k / 6) | (pair_bits(k % 6) << 4);
        if (kHalves24.first_of[k]) {
            val[idx] = s;
            msk[idx] = m;
        } else {
            const bool better = s > val[idx];     // false for NaN: a feasible choice stays in place
            val[idx] = better ? s : val[idx];
            msk[idx] = better ? m : msk[idx];
        }
    }
}

// v[r][c] = |W| of one 4x4 block.  Returns the 16-bit keep mask (row r in bits 4r..4r+3) of an
// optimal pattern (the first one in a fixed evaluation order) and its kept sum in `best`.
__device__ __forceinline__ uint32_t exact24_block(const float (&v)[4][4], float &best)
{
    float ps[4][6];
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
        for (int p = 0; p < 6; p++)
            ps[r][p] = v[r][kPairX[p]] + v[r][kPairY[p]];
    float top[19], bot[19];
    uint32_t topm[19], botm[19];
    best_pairs24(ps[0], ps[1], top, topm);
    best_pairs24(ps[2], ps[3], bot, botm);
    uint32_t bm = 0;
#pragma unroll
    for (int j = 0; j < 19; j++) {
        const int jc = kHalves24.compl_of[j];
        const float s = top[j] + bot[jc];
        const uint32_t m = topm[j] | (botm[jc] << 8);
        if (j == 0) {
            best = s;
            bm = m;
        } else {
            const bool better = s > best;
            best = better ? s : best;
            bm = better ? m : bm;
        }
    }
    return bm;
}

// 1:4 and 3:4: one entry per row and per column is kept (1:4) or pruned (3:4), i.e. the pattern is one of the 24
// permutations.  v[r][c] = |W| of one 4x4 block.  Returns the 16-bit mask (row r in bits 4r..4r+3) of the permutation
// with the largest (LARGEST) or smallest sum, the first one in a fixed evaluation order, and that sum in `best`.  Rows
// 0 and 1 take an ordered pair of columns (12 ways); rows 2 and 3 share the two columns left and take the better of
// their two assignments.
template <bool LARGEST>
__device__ __forceinline__ uint32_t best_permutation4(const float (&v)[4][4], float &best)
{
    uint32_t bm = 0;
    bool first = true;
#pragma unroll
    for (int c0 = 0; c0 < 4; c0++)
#pragma unroll
        for (int c1 = 0; c1 < 4; c1++) {
            if (c1 == c0)
                continue;
            int x = -1, y = -1;
#pragma unroll
            for (int c = 0; c < 4; c++)
                if (c != c0 && c != c1) {
                    if (x < 0)
                        x = c;
                    else
                        y = c;
                }
            const float top = v[0][c0] + v[1][c1];
            const float b1 = v[2][x] + v[3][y], b2 = v[2][y] + v[3][x];
            const bool swap = LARGEST ? b2 > b1 : b2 < b1;
            const float s = top + (swap ? b2 : b1);
            const uint32_t m = (1u << c0) | (1u << (4 + c1)) |
                               (swap ? ((1u << (8 + y)) | (1u << (12 + x))) : ((1u << (8 + x)) | (1u << (12 + y))));
            const bool better = first || (LARGEST ? s > best : s < best);
            best = better ? s : best;
            bm = better ? m : bm;
            first = false;
        }
    return bm;
}

// =================================================================================================
// Exact, general (N, M): min-cost flow on the network of Fig. 3 (source -> rows, rows -> columns
// with unit capacity and cost |W_ij|, columns -> sink), solved by successive shortest paths.
//
// Costs are integers: c_ij = |W_ij| scaled by a power of two so that the block maximum lies in
// [2^(S-1), 2^S) and truncated.  Integer arithmetic makes every path sum exact, so the residual
// network never shows a negative cycle, label-correcting search converges, and the predecessor
// graph is a forest; truncation costs less than M*K*2^-(S-1) of the block maximum in retained L1
// (S = 27 for M <= 8, 26 for M = 16).
//
// Start: every column prunes the K rows that are lightest under row prices (exact_priced_start) -- a flow that
// saturates the column->sink edges and
// is cheapest among all flows with the same row imbalances.  Then, while some row has more than K
// pruned entries, find the cheapest alternating path from any such row to a row with fewer than K
// (row r -> column j through a pruned entry (r,j), column j -> row r' through an unpruned entry
// (r',j)) with a label-correcting search over row labels, and flip the entries along it.
//
// The start works on the strip layout (a block in G lanes, CL columns each, every lane busy); the few blocks that it
// leaves unbalanced are handed to the searches through LDS, one column and row per lane.
// =================================================================================================

constexpr int kInfDist = 0x70000000;   // unreachable label; kInfDist - 2^S is still above kReachable
constexpr int kReachable = 0x40000000; // every real label is below this: |label| <= (M-1) * 2^S < 2^30
constexpr uint32_t kNoPred = 0xFFFFFFFFu;

constexpr int exact_cost_bits(int M) { return (M == 16) ? 26 : 27; }

// |W| keys (fp32 bit patterns) of one block -> integer costs, see above; as floats (which hold every cost: 24 significant bits)
// or integers.
template <int M, int CL, int G, typename T>
__device__ __forceinline__ void exact_costs(const uint32_t (&key)[M][CL], T (&cost)[M][CL])
{
    constexpr int S = exact_cost_bits(M);
    static_assert((M - 1) * (1ll << S) < kReachable, "labels must stay below the reachability threshold");
    // ---- integer costs ----
    uint32_t kmax = 0;
#pragma unroll
    for (int i = 0; i < M; i++)
#pragma unroll
        for (int c = 0; c < CL; c++)
            kmax = key[i][c] > kmax ? key[i][c] : kmax;
    if constexpr (G >= 2) {
        const uint32_t o = quad_xor<1>(kmax);
        kmax = o > kmax ? o : kmax;
    }
    if constexpr (G >= 4) {
        const uint32_t o = quad_xor<2>(kmax);
        kmax = o > kmax ? o : kmax;
    }
    if constexpr (G >= 8) {                                     // the quads hold one value each by now: any pairing of them will do
        const uint32_t o = dpp_read<kRowHalfMirror>(kmax);
        kmax = o > kmax ? o : kmax;
    }
    if constexpr (G == 16) {
        const uint32_t o = dpp_read<kRowRor8>(kmax);
        kmax = o > kmax ? o : kmax;
    }
    const uint32_t emax = (kmax >> 23) ? (kmax >> 23) : 1u;
    // |w| 2^k for the k that brings the block's maximum to [2^(S-1), 2^S): exact, then truncated.  Infinities and NaN count as
    // the magnitudes whose bits follow the largest finite one's; a block that has any takes its exponents one lower.
    const int shift = S + 126 - (int)emax + (emax == 255u ? 1 : 0);
    uint32_t k[M][CL];
#pragma unroll
    for (int i = 0; i < M; i++)
#pragma unroll
        for (int c = 0; c < CL; c++)
            k[i][c] = key[i][c];
    if (__any(emax == 255u)) {                                  // not an instruction for each weight of the others
        const uint32_t lower = emax == 255u ? 0x800000u : 0u;
#pragma unroll
        for (int i = 0; i < M; i++)
#pragma unroll
            for (int c = 0; c < CL; c++) {
                k[i][c] = __builtin_elementwise_sub_sat(k[i][c], lower);
                asm volatile("" : "+v"(k[i][c]));
            }
    }
#pragma unroll
    for (int i = 0; i < M; i++)
#pragma unroll
        for (int c = 0; c < CL; c++) {
            const float scaled = __builtin_ldexpf(__uint_as_float(k[i][c]), shift);
            if constexpr (std::is_same_v<T, float>)
                cost[i][c] = __builtin_truncf(scaled);
            else
                cost[i][c] = (int)scaled;
        }
}

// Start with row prices: column c prunes the K rows with the smallest cost + price (ties: by position, see below).
// Whatever the prices, the result is the cheapest pruning for the row counts it has: the price
// term of any pruning with those counts is the same sum over rows of price x count, so being cheapest under
// cost + price means being cheapest under cost alone.  That is all the augmenting searches ask of their
// start, so prices can even out the row counts before the first search.
//
// The prices come from a few rounds of ascent on the dual of the row constraints, smoothed: instead of counting the
// entries of a row below their column's threshold, each entry adds 0 ... 1 by where its key lies in a window of
// width w around the middle between the column's K-th and (K+1)-th smallest key (one fused multiply-add with the
// hardware's clamp and one addition, what a compare and a count cost), and a row's price moves by step x (that sum),
// with some momentum (kept in units of the round's step: a price moves by step x v, v <- sum + momentum / step_next x v, two
// instructions); w and step shrink from round to round.  A count says by how many entries a row is out of
// balance, the smoothed sum also how far away the balance is: blocks of N(0,1) entries left unbalanced, by emulation,
// 2.5 % after 8 rounds at M = 8 and 6 % after 13 at M = 16, where 12 and 20 rounds on counts left 12 % and 14 %.
// Schedules were settled by a search in emulation, the numbers of rounds by timing on the device (6 ... 10 and
// 10 ... 18 are within 5 % of each other: more rounds, fewer searches).  Windows and steps are multiples of the block's
// mean cost or, if that is less, of sqrt(2) times the mean difference of two entries of a column half a block apart, row
// means taken off: blocks whose rows, or columns, resemble one another differ by a small part of their mean, which windows
// of that size cannot tell apart (columns equal up to 1 %: excess left at 8:16 47 -> 2.4; 2048^2 fp32 1760 -> 300 us).  The
// prices start at what makes the row means equal, or a quarter less where these differ no more than three times what
// chance gives, which keeps heavy-tailed blocks as good.  All of it is fp32: the prices need no more, and every cost is a
// float exactly (24 significant bits, as the weights have).  The prices are then rounded to integers and the choice
// itself is taken on integer keys.
//
// Keys of that choice are (cost + price + 2^(S-1)) << 4 | tie-break with |price| < 2^(S-1): below 2^(S+5) <= 2^32 for
// costs < 2^S.  The tie-break of entry (i, j) is (i - j) mod M, not the row alone: columns with equal costs (blocks of an
// unstructured-sparse matrix are full of zeros) then prune different rows, a band, instead of all the same ones,
// which no row price could tell apart.  In such blocks prices that differ by little undo the band, so a wavefront in
// which a block has an excess of more than two left tries its blocks without prices as well and keeps the better
// choice (hardly ever on blocks of random values; 90 % zeros at 4:8: excess 10 -> 2.2).
// xcol: the pruned rows of every column; the return value: the excess they leave.
// GENERAL: any 0 < K < M, the same in every lane (the thresholds then come from a full sort of the column's keys and
// register reads at those indexes; 24 instead of 16 instructions at M = 8, 91 instead of 72 at M = 16); otherwise
// K = M/2.

// clamp(a * b + c, 0, 1)
__device__ __forceinline__ float fma_clamp01(float a, float b, float c)
{
    float r;
    asm("v_fma_f32 %0, %1, %2, %3 clamp" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// v + the value of lane (lane ^ X) within the quad, the move folded into the addition
template <int X>
__device__ __forceinline__ float quad_xor_sum(float v)
{
    constexpr int ctrl = (X == 1) ? 0xB1 : (X == 2) ? 0x4E : 0x1B;
    return v + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), ctrl, 0xF, 0xF, true));
}

// Schedule of the smoothed rounds: window and step in units of the block's mean cost, factors per round.
template <int M>
struct PriceSchedule;
template <>
struct PriceSchedule<8> {
    static constexpr int rounds = 8;
    static constexpr float window = 0.527f, window_next = 0.62f, step = 0.2325f, step_next = 0.66f, momentum = 0.22f;
};
template <>
struct PriceSchedule<16> {
    static constexpr int rounds = 13;
    static constexpr float window = 0.445f, window_next = 0.703f, step = 0.192f, step_next = 0.736f, momentum = 0.2f;
};

// A column of a round: x[i] = 0 ... 1 by where key k[i] (a positive float, which compares as its bits) lies in a window of
// width -1 / slope around the middle between the K-th and the (K+1)-th smallest key.
template <int M, bool GENERAL>
__device__ __forceinline__ void price_window(const uint32_t (&k)[M], float slope, uint32_t K, float (&x)[M])
{
    constexpr int H = M / 2;
    float both;                                                 // the two, added
    if constexpr (GENERAL) {
        uint32_t srt[M];
#pragma unroll
        for (int i = 0; i < M; i++)
            srt[i] = k[i];
        sort_asc<M>(srt);
        both = __uint_as_float(srt[(K - 1u) & (uint32_t)(M - 1)]) + __uint_as_float(srt[K & (uint32_t)(M - 1)]);
    } else if constexpr (M == 8) {
        const Eight e = columns_of_8(k);
        both = __uint_as_float(fourth_of_8(e)) + __uint_as_float(fifth_of_8(e));
    } else {
        uint32_t lo[H], hi[H], below = 0u, above = 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < H; i++) {
            lo[i] = k[i];
            hi[i] = k[H + i];
        }
        sort_asc<H>(lo);
        sort_asc<H>(hi);
#pragma unroll
        for (int i = 0; i < H; i += 2) {
            const uint32_t b0 = lo[i] < hi[H - 1 - i] ? lo[i] : hi[H - 1 - i], b1 = lo[i + 1] < hi[H - 2 - i] ? lo[i + 1] : hi[H - 2 - i];
            const uint32_t a0 = lo[i] < hi[H - 1 - i] ? hi[H - 1 - i] : lo[i], a1 = lo[i + 1] < hi[H - 2 - i] ? hi[H - 2 - i] : lo[i + 1];
            below = max3u(below, b0, b1);
            above = min3u(above, a0, a1);
        }
        both = __uint_as_float(below) + __uint_as_float(above);
    }
    const float at = 0.5f - (0.5f * slope) * both;              // clamp((middle - key) / w + 1/2)
#pragma unroll
    for (int i = 0; i < M; i++)
        x[i] = fma_clamp01(__uint_as_float(k[i]), slope, at);
}

// What the rounds of a block start with: the part of the row means that its prices make equal, and slope (of the windows) and step.
// mean: of the block's costs; spread: of two entries of a column half a block apart, row means taken off; row_dev: sum of what
// the row means differ from the mean by.
template <int M>
struct PriceScale {
    float part, slope, step;

    __device__ __forceinline__ PriceScale(float mean, float spread, float row_dev)
    {
        using Sched = PriceSchedule<M>;
        // three times what chance makes of the row means of independent entries, against what they are
        const float chance = 3.f * spread * (M == 16 ? 2.828427f : 2.f) * __builtin_amdgcn_rcpf(row_dev);      // sqrt(M / 2) M / M
        part = 1.f - 0.25f * (chance < 1.f ? chance : 1.f);
        float unit = 1.414214f * spread;
        unit = unit < mean ? unit : mean;
        unit = unit > 1.f ? unit : 1.f;                         // blocks of zeros, and of costs that rows and columns explain
        slope = -(1.f / Sched::window) * __builtin_amdgcn_rcpf(unit);
        step = Sched::step * unit;
    }
};

template <int M, int CL, int G, bool GENERAL = false>
__device__ __forceinline__ uint32_t exact_priced_start(const float (&cost)[M][CL], uint32_t gpos, uint32_t (&xcol)[CL],
                                                       uint32_t k_general = 0)
{
    constexpr int H = M / 2;
    const int K = GENERAL ? (int)__builtin_amdgcn_readfirstlane(k_general) : M / 2;
    constexpr int S = exact_cost_bits(M);
    constexpr float kOffset = (float)(1 << S);                  // added to the prices of the rounds: keys stay positive
    using Sched = PriceSchedule<M>;
    float cf[M][CL], pr[M], vel[M];
    float mean = 0.f;
#pragma unroll
    for (int i = 0; i < M; i++) {
        float sum = 0.f;
#pragma unroll
        for (int c = 0; c < CL; c++) {
            cf[i][c] = cost[i][c];
            asm volatile("" : "+v"(cf[i][c]));                  // the weights end here
            sum += cf[i][c];
        }
        if constexpr (G >= 2)
            sum = quad_xor_sum<1>(sum);
        if constexpr (G == 4)
            sum = quad_xor_sum<2>(sum);
        pr[i] = sum;
        mean += sum;
    }
    mean = mean * (1.f / (M * M));
    // how far the row means lie apart (their deviations go to pr), and, row means taken off, two entries of a column half a
    // block apart
    float row_dev = 0.f, spread = 0.f;
#pragma unroll
    for (int i = 0; i < M; i++) {
        pr[i] = mean - pr[i] * (1.f / M);
        row_dev += __builtin_fabsf(pr[i]);
    }
#pragma unroll
    for (int i = 0; i < H; i++) {
        const float rows = pr[i] - pr[H + i];
#pragma unroll
        for (int c = 0; c < CL; c++)
            spread += __builtin_fabsf((cf[i][c] - cf[H + i][c]) + rows);
    }
    if constexpr (G >= 2)
        spread = quad_xor_sum<1>(spread);
    if constexpr (G == 4)
        spread = quad_xor_sum<2>(spread);
    spread *= 2.f / (M * M);
    const PriceScale<M> scale(mean, spread, row_dev);
#pragma unroll
    for (int i = 0; i < M; i++) {
        pr[i] = kOffset + scale.part * pr[i];
        vel[i] = 0.f;
    }
    float slope = scale.slope, step = scale.step;
    float drift = 0.f;                                          // what K per row and round adds to every price
    float dvel = 0.f;
    constexpr float kCarry = Sched::momentum / Sched::step_next;
#pragma unroll 1
    for (int round = 0; round < Sched::rounds; round++) {
        float f[M];
#pragma unroll
        for (int c = 0; c < CL; c++) {
            uint32_t k[M];                                      // positive floats compare as integers
#pragma unroll
            for (int i = 0; i < M; i++)
                k[i] = __float_as_uint(pr[i] + cf[i][c]);
            float x[M];
            price_window<M, GENERAL>(k, slope, (uint32_t)K, x);
#pragma unroll
            for (int i = 0; i < M; i++)
                f[i] = c == 0 ? x[i] : f[i] + x[i];
            if constexpr (CL > 4 || M == 16)
                __builtin_amdgcn_sched_barrier(0);   // one column at a time: interleaving them costs M registers each
        }
        // all rows a step at a time: a value that was just written cannot be read across lanes for two wait states
        if constexpr (G >= 2) {
#pragma unroll
            for (int i = 0; i < M; i++)
                f[i] = quad_xor_sum<1>(f[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (G == 4) {
#pragma unroll
            for (int i = 0; i < M; i++)
                f[i] = quad_xor_sum<2>(f[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < M; i++) {
            // in place: as an expression it is an accumulation into f and a move
            asm("v_fma_f32 %0, %1, %0, %2" : "+v"(vel[i]) : "s"(kCarry), "v"(f[i]));
            pr[i] = __builtin_fmaf(step, vel[i], pr[i]);
        }
        dvel = __builtin_fmaf(kCarry, dvel, (float)K);
        drift = __builtin_fmaf(step, dvel, drift);
        slope *= 1.f / Sched::window_next;
        step *= Sched::step_next;
    }

    // ---- the choice under the prices reached, on integer keys ----
    constexpr int PMIN = 1, PMAX = (1 << S) - 1;                // price + 2^(S-1)
    int pi[M];
    auto choose = [&](auto priced, uint32_t (&x)[CL]) -> uint32_t {     // returns twice the excess
        uint32_t n[M];
#pragma unroll
        for (int i = 0; i < M; i++)
            n[i] = 0;
#pragma unroll
        for (int c = 0; c < CL; c++) {
            uint32_t k[M], lo[H], hi[H];
#pragma unroll
            for (int i = 0; i < M; i++) {
                const uint32_t v = (uint32_t)(int)cf[i][c] + (decltype(priced)::value ? (uint32_t)pi[i] : 1u << (S - 1));
                k[i] = (v << 4) | (((uint32_t)i - (gpos * (uint32_t)CL + (uint32_t)c)) & (uint32_t)(M - 1));
            }
            uint32_t t;
            if constexpr (GENERAL) {
                uint32_t srt[M];
#pragma unroll
                for (int i = 0; i < M; i++)
                    srt[i] = k[i];
                sort_asc<M>(srt);
                t = srt[(uint32_t)K & (uint32_t)(M - 1)];       // the (K+1)-th smallest; the index is the same in every lane
            } else {
#pragma unroll
                for (int i = 0; i < H; i++) {
                    lo[i] = k[i];
                    hi[i] = k[H + i];
                }
                t = upper_half_min<H>(lo, hi);
            }
            x[c] = 0u;
#pragma unroll
            for (int i = M - 1; i >= 0; i--) {
                const lanemask_t m = lm(k[i] < t);
                lm_inc(n[i], m);
                lm_shift_in(x[c], m);
            }
            __builtin_amdgcn_sched_barrier(0);       // the columns' keys one after the other
        }
        uint32_t e2 = 0;
#pragma unroll
        for (int i = 0; i < M; i++) {
            if constexpr (G >= 2)
                n[i] = quad_xor_sum<1>(n[i]);
            if constexpr (G == 4)
                n[i] = quad_xor_sum<2>(n[i]);
            e2 = __builtin_amdgcn_sad_u8(n[i], (uint32_t)K, e2);      // counts are below 256: |n - K| of the low byte
        }
        return e2;
    };
    // opaque: else the integer costs and tie-breaks of the choice are computed ahead of the rounds and held through them
#pragma unroll
    for (int i = 0; i < M; i++)
#pragma unroll
        for (int c = 0; c < CL; c++)
            asm volatile("" : "+v"(cf[i][c]));
    asm volatile("" : "+v"(gpos));
#pragma unroll
    for (int i = 0; i < M; i++) {
        const float p = pr[i] - drift - (kOffset - (float)(1 << (S - 1)));
        pi[i] = (int)__builtin_amdgcn_fmed3f(p, (float)PMIN, (float)(PMAX - 64));     // (float)PMAX would be 2^S
    }
    uint32_t e2 = choose(std::true_type{}, xcol);
    if (__any(e2 > 4u)) {
        uint32_t x[CL];
        const uint32_t e = choose(std::false_type{}, x);
        const bool better = e < e2 && e2 > 4u;      // a block's own excess decides, not its neighbours'
        e2 = better ? e : e2;
#pragma unroll
        for (int c = 0; c < CL; c++)
            xcol[c] = better ? x[c] : xcol[c];
    }
    return e2 >> 1;
}

// LDS of one wavefront's searches: the predecessors of the rows and columns of its 64 / M blocks, the chain that each
// row would take and the row it starts from, and the entries that the chains flip.
struct SearchLds {
    uint32_t prow[64], pcol[64];
    uint32_t chain[64], start[64], flip_row[64], flip_col[64];
};

// Augments until every row of the block has exactly K pruned entries (after at most M*M searches).  M lanes hold a
// block, a wavefront 64 / M of them: lane j of the block holds column j (ccol, xcol: bit i = entry (i, j) pruned) and row
// j (crow, xrow: bit c = entry (j, c) pruned).  All lanes of the wavefront take part; lanes with `active` false hold no block.
//
// A search labels the rows from those with excess, alternating a column step (lane j: the cheapest way into column j
// through a pruned entry of a reached row) and a row step (lane j: the cheapest way into row j out of a column through an
// unpruned entry).  Labels pass between the lanes of a block by DPP, and which entries are pruned is a lane mask for each
// row and column: four vector instructions an entry (eight through LDS with the bits tested in place, and the reads' latency).  Labels only
// ever fall, and a predecessor changes only when its label falls strictly: with exact integer sums and no negative cycle the
// predecessor graph is then a forest, also among entries of equal cost.
//
// At convergence every predecessor edge is tight (label of the head = label of the tail + edge cost), so flipping along any
// set of chains with no column in common keeps the pruning cheapest for its row counts.  The first reachable row that
// lacks pruned entries takes its chain; at M = 16, when three or more rows of the block have excess, as in blocks of tied values, every
// such row does whose chain is still free.  All of it depends on the block alone, not on those that share the wavefront: among equally
// good masks it finds the same one in every call.  (2048^2 8:16 with 50 % zeros 242 ->
// 200 us, three levels 207 -> 172; at M = 8 the second walk costs more than it saves, 70 -> 75 us with 70 % zeros.  Four or more rows of any
// block of the wavefront, until no block found two / three or more of the block's own: 4096^2 8:16 50 % zeros 307 / 292, three levels
// 326 / 324, 13:16 273 / 264 and 284 / 269, random values 75.5 / 75.5.)
template <int M>
__device__ __forceinline__ void exact_search(const int (&ccol)[M], const int (&crow)[M], uint32_t &xcol, uint32_t xrow,
                                             bool active, uint32_t K, SearchLds &lds)
{
    static_assert(M <= 16, "a chain's rows and columns share a word");
    constexpr bool SEVERAL = M == 16;
    const uint32_t lane = threadIdx.x & 63u, j = lane % M, base = lane - j;     // base: first lane of the block
    constexpr uint32_t kSeg = (uint32_t)((1ull << M) - 1ull);
    auto mine = [&](lanemask_t m) { return (uint32_t)(m >> base) & kSeg; };     // the block's bits of a ballot
    auto fence = []() {                                          // LDS accesses of a wavefront happen in program order
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
    };
    uint32_t cnt = active ? (uint32_t)__builtin_popcount(xrow) : K;
#pragma unroll 1
    for (int search = 0; search < M * M; search++) {
        const lanemask_t excess = lm(cnt > K);
        if (excess == 0)
            break;
        uint32_t over = mine(excess);
        int drow = cnt > K ? 0 : kInfDist, dcol = kInfDist;
        uint32_t prow = kNoPred, pcol = 0;
        lanemask_t in[M], out[M];                                // entry (i, j) is pruned, entry (j, i) is not
#pragma unroll
        for (int i = 0; i < M; i++) {
            in[i] = lm((xcol >> i) & 1u);
            out[i] = ~lm((xrow >> i) & 1u);
        }
#pragma unroll 1
        for (int it = 0; it <= M; it++) {
            // from a row that is not reached: above every label, and not a label itself
            each_of<M>([&](auto c) {
                constexpr int i = decltype(c)::value;
                const int v = (int)of_lane<M, i>((uint32_t)drow) - ccol[i];
                const bool better = lm_test(lm(v < dcol) & in[i]);
                dcol = better ? v : dcol;
                pcol = better ? (uint32_t)i : pcol;
            });
            dcol = dcol < kReachable ? dcol : kInfDist;
            const int before = drow;
            each_of<M>([&](auto c) {
                constexpr int i = decltype(c)::value;
                const int v = (int)of_lane<M, i>((uint32_t)dcol) + crow[i];      // from an unreached column: above every label
                const bool better = lm_test(lm(v < drow) & out[i]);
                drow = better ? v : drow;
                prow = better ? (uint32_t)i : prow;
            });
            if (lm(drow != before) == 0)
                break;
        }
        fence();
        lds.prow[lane] = prow;
        lds.pcol[lane] = pcol;
        fence();
        const bool lacks = cnt < K && drow < kReachable;
        uint32_t cand = mine(lm(lacks));
        if (lm(cand != 0u) == 0)
            break;                      // cannot happen for 0 < K < M; guards against looping on corrupt state
        const bool wide = SEVERAL && __builtin_popcount(over) >= 3;
        if (lm(wide) == 0) {
            // the first reachable row takes its chain
            const uint32_t target = cand != 0u ? (uint32_t)__builtin_ctz(cand) : 0u;
            uint32_t r = target, src = kNoPred;
            bool walking = cand != 0u;
#pragma unroll 1
            for (int step = 0; step <= M && lm(walking) != 0; step++) {
                if (walking) {
                    const uint32_t c = lds.prow[base + r];
                    if (c == kNoPred) {
                        src = r;                                 // the row with excess that the chain starts from
                        walking = false;
                    } else {
                        const uint32_t f = lds.pcol[base + c];   // (r, c) becomes pruned, (f, c) becomes unpruned
                        if (j == c)
                            xcol ^= (1u << r) | (1u << f);
                        if (j == r || j == f)
                            xrow ^= 1u << c;
                        r = f;
                    }
                }
            }
            if (src != kNoPred)
                cnt += (j == target ? 1u : 0u) - (j == src ? 1u : 0u);
        } else if constexpr (SEVERAL) {
            // every reachable row walks its chain, a lane each ...
            uint32_t r = j, chain = 0u, start = kNoPred;
            bool walking = lacks;
            lds.flip_row[lane] = 0u;
            lds.flip_col[lane] = 0u;
#pragma unroll 1
            for (int step = 0; step <= M && lm(walking) != 0; step++) {
                if (walking) {
                    const uint32_t c = lds.prow[base + r];
                    if (c == kNoPred) {
                        start = r;
                        walking = false;
                    } else {
                        chain |= 1u << r | 0x10000u << c;
                        r = lds.pcol[base + c];
                    }
                }
            }
            lds.chain[lane] = chain;
            lds.start[lane] = start;
            fence();
            // ... the lowest takes it, and so does, in a wide block, each after it that shares no row or column with those taken and
            // whose first row has excess left
            uint32_t used = 0u;
            bool taken = false;
            cand = wide ? cand : cand & (0u - cand);
#pragma unroll 1
            while (lm(cand != 0u) != 0) {
                over = mine(lm(cnt > K));
                const uint32_t t = cand != 0u ? (uint32_t)__builtin_ctz(cand) : 0u;
                const uint32_t ch = lds.chain[base + t], s = lds.start[base + t];
                if (cand != 0u && s < (uint32_t)M && (ch & used) == 0u && (over >> (s & 31u) & 1u)) {
                    used |= ch;
                    taken = taken || j == t;
                    cnt += (j == t ? 1u : 0u) - (j == s ? 1u : 0u);
                }
                cand &= cand - 1u;
            }
            r = j;
#pragma unroll 1
            for (int step = 0; step <= M && lm(taken) != 0; step++) {
                if (taken) {
                    const uint32_t c = lds.prow[base + r];
                    if (c == kNoPred) {
                        taken = false;
                    } else {
                        const uint32_t f = lds.pcol[base + c];
                        lds.flip_col[base + c] = 1u << r | 1u << f;      // no other chain has this column
                        atomicXor(&lds.flip_row[base + r], 1u << c);
                        atomicXor(&lds.flip_row[base + f], 1u << c);     // several chains may start from one row
                        r = f;
                    }
                }
            }
            fence();
            xcol ^= lds.flip_col[lane];
            xrow ^= lds.flip_row[lane];
        }
    }
}

}  // namespace tmask
