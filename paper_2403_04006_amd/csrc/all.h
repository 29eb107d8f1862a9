// Every output amplitude of one input pattern (passive linear optics): the
// Glynn sum runs over the input side S, and one term's column sums serve
// every output pattern T at once,
//   perm(U_{T,S}) = 2^{-(n-1)} sum_delta w(delta) prod_i c_i(delta)^{t_i},
//   c_i(delta) = sum_j delta_j U[i][j]  (i over all m output modes,
//                                         j over the input modes with s_j > 0),
// delta_j = s_j - 2 d_j with d_j in 0..s_j for free groups and 0..s_f - 1 for
// the fixed group f (the one with the smallest occupation), and
// w = prod_j (-1)^{d_j} C(mu'_j, d_j) with mu'_f = s_f - 1, mu'_j = s_j.
//
// Outputs are the C(n+m-1, n) occupation vectors T with sum n, in ascending
// lexicographic order of (T_0, ..., T_{m-1}) (T = (0, ..., 0, n) first).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/pq.h"
#include "pq_common.h"

namespace pq {

constexpr int kAllMaxModes = 64;
constexpr int kAllMaxPhotons = 48;
constexpr int kAllTile = 32;              // delta terms staged in LDS at a time
constexpr uint64_t kAllMaxTerms = 1ull << 20;
constexpr int64_t kAllMaxOutputs = PQ_ALL_MAX_OUTPUTS;

// Column sums and weights of every delta term (one thread per (term, mode)).
struct AllSumsArgs {
    const cplx* U;
    int64_t ldu;
    int32_t m;
    int32_t k;                          // input groups (distinct modes with s_j > 0)
    int32_t in_mode[kAllMaxPhotons];    // group modes, fixed group first
    int32_t in_mult[kAllMaxPhotons];    // s_j
    int32_t radix[kAllMaxPhotons];      // s_f for the fixed group, s_j + 1 otherwise
    uint64_t terms;                     // product of the radices
    cplx* csum;                         // [terms][m]
    cplx* csum_t;                       // [m][terms], may be null (the contraction's tables read it)
    double* w;                          // [terms]
};

// Every output: one thread per T.
struct AllOutArgs {
    const cplx* csum;
    const double* w;
    const uint64_t* count;   // [m][n+1]: compositions of nn into mm+1 parts at [mm][nn]
    uint64_t terms;
    int64_t outputs;
    int32_t m, n;
    double scale;            // 2^{-(n-1)}
    double norm_s;           // 1 / sqrt(prod S!)
    cplx* perm;
    cplx* amp;               // may be null
};

// The ladder form: photon by photon instead of a signed sum.  With the input
// photons in modes j_1, ..., j_n, expanding along the last column gives
//   perm_k(T) = sum_{i: t_i > 0} t_i U[i][j_k] perm_{k-1}(T - e_i),
// so every level's values are short sums over the level below: at most
// min(k, m) complex multiply-adds per output (6 on average at 10 photons in 16
// modes) where the signed sum takes one per Gray term (512), and no term
// larger than the result's own scale.  An output is its photons' modes in
// ascending order, q the mode counted from the last: with G(r, q) =
// C(r + q - 1, r) (the ways to put r photons into the last q modes), photons
// p = 0..k-1 and r_p = k - p,
//   rank(T) = sum_p G(r_p, q_p),
//   rank(T without photon p) = sum_{p' < p} G(r_p' - 1, q_p') + sum_{p' > p} G(r_p', q_p'),
// so ranks need no per-output tables, and since every output is at photon p
// in the same step, the searches for q_p and the loads run without branches.
// One workgroup runs the levels of a few thousand values in LDS, one launch
// each of the others; two levels below the outputs live in workspace.
// The first level needs none below: levels 1 to 3 directly, and s photons in one
// input mode j at once,
//   perm_s(T) = s! prod_i U[i][j]^{t_i},
// so the input mode of the most photons goes first where these are four or more.
// Whole calls (sweep or contraction -> ladder): 23 -> 16 us at 5 photons in 12
// modes, 47 -> 31 us at 8 in 12, 97 -> 44 us at 8 in 16, 1268 -> 111 us at 11 in
// 14 and 850 -> 112 us at 10 in 16.  Photons of one input mode: 16 in 8 modes
// 35 -> 17 us, 48 in 3 70 -> 28, 10 in 16 187 -> 49 (92, 362 and 119 when every
// photon was a level).  What is slower than the sweep are many photons of two input
// modes in few modes, where that has few terms: 7 + 7 in 6 modes 41 -> 58 us, 8 + 8
// in 8 61 -> 70; its sums cancel there (5e-15 of the value against 6e-16), so by
// default the ladder is taken whenever its two lower levels fit kAllLadderBytes.
constexpr uint64_t kAllLadderBytes = 1ull << 30;   // workspace of the two lower levels
constexpr int kAllLadderSmall = 2048;              // values of a level kept in LDS
constexpr int kAllLadderFirst = 4096;              // values of the last level that the small kernel takes
constexpr int kAllLadderCols = 512;                // modes x levels of the small kernel
constexpr int kAllLadderBlock = 1024;              // threads of the small levels' workgroup
static_assert(kAllMaxPhotons <= kRankMaxPhotons, "the rank table holds every level");

struct AllLadderArgs {
    const cplx* U;
    int64_t ldu;
    int32_t m, n;
    int32_t s1;                        // photons of the first input mode where they make the first level, or 0
    int32_t k0;                        // last level of the first kernel (0: there is none)
    uint8_t col[kAllMaxPhotons];       // input mode of photon k + 1
    double norm_s;                     // 1 / sqrt(prod S!)
    cplx* perm;
    cplx* amp;                         // may be null
};

// Level k from level k - 1 (in); out: the level's values, or the outputs when
// k == n (perm and amp of AllLadderArgs).
struct AllLevelArgs {
    AllLadderArgs a;
    int32_t k;                         // (a.s1: the first level, which has no input)
    uint32_t count;                    // outputs of level k
    uint32_t run;                      // consecutive outputs per workgroup, a multiple of kBlock
    const cplx* in;
    cplx* out;
};

hipError_t launch_all_ladder_small(const AllLadderArgs& a, cplx* out, hipStream_t s);
hipError_t launch_all_ladder_level(const AllLevelArgs& a, hipStream_t s);

// The contraction form (on request, or where the ladder's levels do not fit;
// its tables have to fit kAllGemmTableBytes):
// split the output modes into a = 0..ma-1 and b = ma..m-1, T = (T_a, T_b).
// Then prod_i c_i^{t_i} = M_a(delta, T_a) M_b(delta, T_b) with M the
// monomials of each half, and for |T_a| = k
//   perm(U_{T,S}) = 2^{-(n-1)} sum_delta [w M_a](delta, T_a) M_b(delta, T_b),
// one complex matrix product per k: (compositions of k into ma parts) x
// (compositions of n - k into m - ma parts), inner dimension the delta terms.
// The monomial tables are rows over delta (per composition, grouped by
// degree, ascending lexicographic order within a degree); the products land
// in a block-ordered buffer and a scatter puts each row of T_b's at its
// T_a's place in the output order.
constexpr uint64_t kAllGemmTableBytes = 1ull << 30;
// without the ladder, the contraction from this many (term, output) pairs on: below
// it the sweep is faster (the contraction's launches and stream joins cost
// about 0.2 ms; 8 photons in 16 modes, 6.3e7 pairs: sweep 0.10 ms,
// contraction 0.22 ms; 10 photons in 16 modes, 1.7e9 pairs: 1.9 ms and
// 0.85 ms)
constexpr uint64_t kAllGemmMinPairs = 1ull << 29;
constexpr int kAllMaxBlocks = kAllMaxPhotons + 1;

// The monomial tables, one row of terms per composition (half a weighted).
// A thread keeps its term's column sums of one half in registers and writes
// kAllTableRun consecutive compositions of that half.
constexpr int kAllTableRun = 64;
struct AllTableArgs {
    const cplx* csum_t;          // [m][terms]
    const double* w;             // [terms]
    const uint8_t* exps;         // [entries][stride]: a composition's exponents
    int32_t stride;
    int64_t entries_a;           // entries [0, entries_a) are half a (weighted), the rest half b
    int64_t entries;
    int64_t runs_a;              // ceil(entries_a / kAllTableRun)
    int32_t m, ma;
    uint32_t terms;
    uint32_t term_blocks;        // ceil(terms / kBlock)
    cplx* table;                 // [entries][terms]
};

struct AllScatterArgs {
    const cplx* prod;            // the products, block after block, rows of T_b's
    const int64_t* base;         // [entries_a]: output position of (T_a, first T_b)
    const double* fnorm;         // [entries]: 1 / sqrt(prod T!) of each half's composition
    int32_t nblocks;
    int64_t off[kAllMaxBlocks];  // first product of block b
    int64_t cols[kAllMaxBlocks]; // T_b's per row of block b
    int64_t ia0[kAllMaxBlocks];  // first half-a entry of block b
    int64_t ib0[kAllMaxBlocks];  // first half-b entry of block b
    int64_t outputs;
    double scale, norm_s;
    cplx* perm;
    cplx* amp;                   // may be null
};

// A thin block (at most kAllThinMax T_a's or T_b's): one wavefront per four
// entries of the long side, its lanes splitting the terms, the products
// written in the block's layout.  A 64 x 64 matrix-core tile would compute up
// to 64 times the needed products there.
constexpr int kAllThinMax = 8;
struct AllThinArgs {
    const cplx* table;           // [entries][terms]
    uint32_t terms;
    int64_t long0, short0;       // first table row of the long and of the short side
    int64_t nlong;
    int32_t nshort;              // 1..kAllThinMax
    int32_t long_is_col;         // 1: long side = T_b (product [v][u]); 0: T_a (product [u][v])
    int64_t cols;                // T_b's per row of the block
    cplx* prod;                  // the block's first product
};
hipError_t launch_all_thin(const AllThinArgs& a, hipStream_t s);

hipError_t launch_all_table(const AllTableArgs& a, hipStream_t s);
hipError_t launch_all_scatter(const AllScatterArgs& a, hipStream_t s);

}  // namespace pq
