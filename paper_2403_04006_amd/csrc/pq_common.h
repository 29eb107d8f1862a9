// Shared host/device definitions of the permanent engine: kernel argument
// blocks and the reflected mixed-radix Gray code used by the generalised
// BB/FG (Glynn) sum.
//
// Generalised BB/FG formula with repeated rows (Benchmarks / Boson Sampling:
// n-ary Gray code, digits from zero to the occupation of each mode).  With
// compact matrix B (r distinct iterated rows of multiplicity mu_i, NC distinct
// columns of multiplicity kappa_j), digit d_i and delta_i = mu_i - 2 d_i:
//
//   perm = 2^{-(n-1)} sum_d  prod_i (-1)^{d_i} C(rho_i - 1, d_i)
//                            * prod_j ( sum_i delta_i B_ij )^{kappa_j}
//
// where rho_i = mu_i + 1 is the radix of a free row, and the fixed row f
// ("halving": one delta pinned) has radix rho_f = mu_f (its first copy is
// pinned to +1, the other mu_f - 1 copies are summed).
//
// A digit increment d_i -> d_i + 1 changes every column sum by -2 B_ij, a
// decrement by +2 B_ij; one digit changes per step of a reflected Gray code.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define PQ_HD __host__ __device__ inline
#else
#define PQ_HD inline
#endif

namespace pq {

constexpr int kMaxDim = 48;        // distinct rows / columns / photons
constexpr int kMaxLaneDigits = 6;  // lane digits: product of radices <= 64
constexpr int kMaxInner = 4096;    // entries of the per-step table
constexpr int kBlock = 256;        // threads per workgroup (4 wavefronts)
constexpr int kWavesPerBlock = kBlock / 64;
// reverse-sweep walk variant used unless pq_walk_variant / PQ_WALK say
// otherwise: 2 (register flip digits - 1) + (quad exchanges via ds_swizzle)
constexpr int kWalkDefaultVariant = 4;   // 3 register digits, DPP

struct cplx { double re, im; };

// One entry of the per-step table of the inner (table-driven) digits.
//   off: complex-element offset of the +-2B row applied on the step from
//        position p-1 to p (relative to the start of the time rows of the
//        +-2B table); unused at p = 0.
//   w:   signed binomial weight of the inner digits' state at position p.
struct StepEntry {
    int32_t off;
    int32_t pad;
    double w;
};

// Argument block of the forward sweep kernels (passed by value).
// Power structure of prod_j c_j^{kap_j} over columns sorted by ascending power
// (see product_grouped): bit j of step[q] is set when the power rises by more
// than q from column j-1 to column j; low is the power of column 0.  general
// is 1 when a rise exceeds 3 or low exceeds 4 (the per-column loops are used).
struct PowSteps {
    uint64_t step[3];
    int32_t low;
    int32_t general;
};

template <class KapT>
inline void make_pow_steps(const KapT* kap, int n, PowSteps& ps) {
    ps.step[0] = ps.step[1] = ps.step[2] = 0;
    ps.low = n > 0 ? (int)kap[0] : 1;
    ps.general = (ps.low < 1 || ps.low > 4) ? 1 : 0;
    for (int j = 1; j < n; ++j) {
        const int d = (int)kap[j] - (int)kap[j - 1];
        if (d < 0 || d > 3) ps.general = 1;
        for (int q = 0; q < d && q < 3; ++q) ps.step[q] |= 1ull << j;
    }
}

struct GlynnArgs {
    const cplx* B;        // [r][NC]   compact matrix, iterated rows in digit order
    const cplx* rows2;    // [r][2][NC] per row: -2B (digit up), +2B (digit down)
    const cplx* base;     // [NC]      column sums at all-zero digits: sum_i mu_i B_ij
    const StepEntry* tab_fwd;   // [M_in] inner table, forward traversal
    const StepEntry* tab_bwd;   // [M_in] inner table, reflected traversal
    double* partials;     // [gridDim.x][4]: double-double (re_hi, re_lo, im_hi, im_lo)
    uint64_t time_states; // states swept in time (all time digits)
    uint32_t waves;       // active wavefronts (the range is split evenly among them)
    int32_t n_lane;       // lane digits: rows 0 .. n_lane-1
    int32_t lane_states;  // product of lane radices (<= 64); lanes beyond are idle
    int32_t n_time;       // time digits: rows n_lane .. n_lane+n_time-1 (least significant first)
    int32_t n_inner;      // the first n_inner time digits are table-driven
    int32_t m_inner;      // product of inner radices
    int32_t lane_radix[kMaxLaneDigits];
    int32_t time_radix[kMaxDim];
    int32_t kap[kMaxDim]; // column powers (ascending)
    PowSteps pw;          // their structure for product_grouped
    // mixed digits: column sums and weight of every lane's digits with the time
    // digits at zero, and the inverses of the time radices (digit_inverse)
    const cplx* lane_sums;    // [NC][64]
    const double* lane_w;     // [64]
    uint64_t time_inv[kMaxDim];
};

// Pair sweep (k_pair_impl.h).  Its table, in complex values for P pairs, W = 2 P
// columns (sums 1 and rows 0 in a padded one):
//   [W]                 column sums, lane and higher time digits at zero, the
//                       three lowest time digits at their middle
//   [kMaxLaneDigits][W] -2B of the lane digits
//   [P][4]              a_k b_k
//   [P][4][2]           a_k, b_k
//   [n_outer][2][P][6]  steps of the higher time digits (up, down): moves of the
//                       pair's sums, then of O_0 .. O_3
struct PairArgs {
    const cplx* tab;
    double* partials;            // [groups][4]
    uint64_t blocks;             // blocks of eight time states
    uint32_t groups;             // workgroups (the blocks are split evenly among them)
    int32_t n_lane, lane_states;
    int32_t n_outer;             // time digits above the three lowest (1 at least)
};

PQ_HD size_t pair_table_size(int pairs, int n_outer) {
    return (size_t)pairs * (size_t)(2 + 2 * kMaxLaneDigits + 4 + 8 + 12 * n_outer);
}

struct PairPrepArgs {
    const cplx* U;
    int64_t ldu;
    cplx* tab;
    int32_t r, nc, pairs;
    int32_t transposed;          // as in PrepArgs
    int32_t n_lane, n_outer;     // rows: lane digits, three time digits, n_outer time digits, constant rows
    int32_t row_mode[kMaxDim];   // iterated modes in digit order
    int32_t row_mu[kMaxDim];
    int32_t col_mode[kMaxDim];
};

// Prep kernel arguments: gather the compact matrix from U and build the
// +-2B rows and the base column sums.
struct PrepArgs {
    const cplx* U;
    int64_t ldu;
    cplx* B;
    cplx* rows2;
    cplx* base;
    int32_t r, nc;
    int32_t transposed;          // 0: B[i][j] = U[row_mode[i]][col_mode[j]]; 1: U[col_mode[j]][row_mode[i]]
    int32_t row_mode[kMaxDim];   // iterated modes in digit order
    int32_t row_mu[kMaxDim];
    int32_t col_mode[kMaxDim];
    // mixed digits: the inner digits' Gray sequence, and the lanes' sums and
    // weights (GlynnArgs); m_inner 0 otherwise
    StepEntry* tab_fwd;
    StepEntry* tab_bwd;
    cplx* lane_sums;
    double* lane_w;
    int32_t n_inner;
    int32_t m_inner;
    int32_t n_lane, lane_states;
    int32_t lane_radix[kMaxLaneDigits];
    int32_t radix[16];
};

// Finalisation: double-double sum of the workgroup partials, scaled by
// 2^{-(n-1)}, times the normaliser for the amplitude.
struct FinalArgs {
    const double* partials;
    int32_t count;
    double scale;                // 2^{-(n-1)}
    double norm;                 // 1 / sqrt(prod S! prod T!)
    cplx* perm;                  // may be null
    cplx* amp;                   // may be null
};

// A whole permanent in one launch (k_fused_impl.h).
constexpr int kTickets = 4;
struct FusedArgs {
    const cplx* U;
    int64_t ldu;
    cplx* perm;                  // may be null
    cplx* amp;                   // may be null
    double scale;                // 2^{-(n-1)}
    double norm;                 // 1 / sqrt(prod S! prod T!)
    double* partials;            // [grid][4]
    uint32_t* tickets;           // [kTickets], zero between launches
    uint32_t turn;               // the one this launch counts in
    uint32_t time_states;
    uint32_t waves;
    int32_t r, nc;
    int32_t transposed;          // as in PrepArgs
    int32_t n_lane, lane_states, n_time;
    int32_t row_mode[kMaxDim];   // iterated modes in digit order
    int32_t col_mode[kMaxDim];
    int8_t row_mu[kMaxDim];
    int8_t radix[kMaxDim];       // of the lane digits, then the time digits
    PowSteps pw;                 // of the padded columns
};

// ---------------------------------------------------------------- Gray code
// Reflected mixed-radix Gray code, digits least significant first.  With
// counter digits a_k of the rank, the Gray digit k is a_k when the digits
// above it sum to an even number and rho_k - 1 - a_k otherwise; moving from
// rank t to t+1 changes exactly one Gray digit (the lowest counter digit that
// does not wrap), by +1 or -1.
PQ_HD void gray_unrank(int d, const int32_t* radix, uint64_t rank, int32_t* g, int parity_in = 0) {
    int32_t a[kMaxDim];
    for (int k = 0; k < d; ++k) {
        if (rank >> 32) {
            a[k] = (int32_t)(rank % (uint64_t)radix[k]);
            rank /= (uint64_t)radix[k];
        } else {
            // a 64-bit division costs a kernel six times a 32-bit one
            const uint32_t r = (uint32_t)rank, q = r / (uint32_t)radix[k];
            a[k] = (int32_t)(r - q * (uint32_t)radix[k]);
            rank = q;
        }
    }
    int par = parity_in;
    for (int k = d - 1; k >= 0; --k) {
        g[k] = par ? radix[k] - 1 - a[k] : a[k];
        par ^= (g[k] & 1);
    }
}

// x / d for a divisor d of x (odd ones by their inverse modulo 2^64).
PQ_HD uint64_t exact_div(uint64_t x, uint32_t d) {
    switch (d) {
        case 1: return x;
        case 2: return x >> 1;
        case 3: return x * 0xAAAAAAAAAAAAAAABull;
        case 4: return x >> 2;
        case 5: return x * 0xCCCCCCCCCCCCCCCDull;
        case 6: return (x >> 1) * 0xAAAAAAAAAAAAAAABull;
        default: return x / d;
    }
}

// x / y and x mod y where the quotient is small (below 2^20).
PQ_HD uint32_t small_quotient(uint64_t x, uint64_t y, uint64_t& rem) {
#if defined(__HIP_DEVICE_COMPILE__)
    // an estimate that is off by one at most, then corrected
    uint32_t q = (uint32_t)((double)x * __builtin_amdgcn_rcp((double)y));
    int64_t r = (int64_t)(x - (uint64_t)q * y);
    if (r < 0) {
        --q;
        r += (int64_t)y;
    } else if (r >= (int64_t)y) {
        ++q;
        r -= (int64_t)y;
    }
    rem = (uint64_t)r;
    return q;
#else
    rem = x % y;
    return (uint32_t)(x / y);
#endif
}

// The same digits without a digit array: f(k, g_k) for k = d-1 down to 0,
// with radix(k) the radix of digit k.  Each digit is the quotient by the
// product of the radices below it, so every value stays wavefront-uniform.
// Ranks and products stay below 2^62.  Returns the parity of the digit sum
// (with parity_in).  Plain 64-bit divisions here (three a digit, about 150
// instructions each) were most of a short sweep: 84 us of 2 x 15 rows.
template <class Radix, class F>
PQ_HD int gray_digits_desc(int d, Radix radix, uint64_t rank, int parity_in, F&& f) {
    uint64_t below = 1;
    for (int k = 0; k < d; ++k) below *= (uint64_t)radix(k);
    int par = parity_in;
    for (int k = d - 1; k >= 0; --k) {
        const uint32_t rk = (uint32_t)radix(k);
        below = exact_div(below, rk);
        const int a = (int)small_quotient(rank, below, rank);
        const int g = par ? (int)rk - 1 - a : a;
        par ^= g & 1;
        f(k, g);
    }
    return par;
}

// Quotients by a radix rho of 2..49 through its inverse, exact below 2^58 (the
// error of the inverse, less than rho / 2^64, stays below 1 / rho).
inline uint64_t digit_inverse(uint32_t rho) { return ~(uint64_t)0 / rho + 1; }

// The same digits from digit 0 up: a digit runs downward where the quotient by
// the radices up to it is odd (every step moves one digit by one, so a digit
// sum's parity is its rank's).  On scalar registers alone, where
// gray_digits_desc takes some 25 vector instructions a digit.
template <class Radix, class Inv, class F>
PQ_HD void gray_digits_asc(int d, Radix radix, Inv inv, uint64_t rank, F&& f) {
    for (int k = 0; k < d; ++k) {
        const uint32_t rk = (uint32_t)radix(k);
#if defined(__HIP_DEVICE_COMPILE__)
        const uint64_t q = __umul64hi(rank, inv(k));
#else
        const uint64_t q = (uint64_t)(((unsigned __int128)rank * inv(k)) >> 64);
#endif
        const int a = (int)((uint32_t)rank - (uint32_t)q * rk);
        f(k, (q & 1) ? (int)rk - 1 - a : a);
        rank = q;
    }
}

// C(a, b) for small non-negative integers, exact in double (a <= 48).
PQ_HD double binom_d(int a, int b) {
    if (b < 0 || b > a) return 0.0;
    if (b > a - b) b = a - b;
    if (b == 0) return 1.0;
    double r = (double)(a - b + 1);
    for (int k = 2; k <= b; ++k) r = r * (double)(a - b + k) / (double)k;   // C(a - b + k, k): exact
    return r;
}

// (-1)^d C(rho - 1, d): the weight of digit value d of a row with radix rho.
PQ_HD double digit_weight(int rho, int d) {
    double w = binom_d(rho - 1, d);
    return (d & 1) ? -w : w;
}

// One state of a Gray block of n digits (M states, at most 2^16): its signed
// binomial weight w, and the digits that move on the steps into it, from rank
// q - 1 (fwd, q >= 1) and from rank q + 1 (bwd, q <= M - 2): the lowest counter
// digit that does not wrap, up or down by the parity of the digits above it.
struct GrayStep {
    double w;
    int fwd, bwd;            // digit
    int fwd_up, bwd_up;      // 1: the digit rises
};

template <class Radix>
PQ_HD GrayStep gray_step(int n, Radix radix, int M, int q) {
    GrayStep e{1.0, 0, 0, 0, 0};
    uint32_t below = (uint32_t)M, rem = (uint32_t)q;
    int par = 0;
    for (int k = n - 1; k >= 0; --k) {
        const uint32_t rk = (uint32_t)radix(k);
        below /= rk;
        const uint32_t a = rem / below;
        rem -= a * below;
        if (a != 0) {
            e.fwd = k;
            e.fwd_up = !par;
        }
        if (a != rk - 1) {
            e.bwd = k;
            e.bwd_up = par;
        }
        const int g = par ? (int)(rk - 1 - a) : (int)a;
        e.w *= digit_weight((int)rk, g);
        par ^= g & 1;
    }
    return e;
}

// Rank table of photon vectors (ladder.h): G[r][q] = C(r + q - 1, r), the ways
// to put r photons into the last q modes, for 1 <= q < m; rows of P, the power
// of two from m on.  The 64 lanes of a wavefront make rows 0..63 together:
// lane r has F(q, r) = C(q + r, r) = F(q - 1, r) + F(q, r - 1) at step q + r,
// `left` being its neighbour's value of the step before (0 in lane 0).  The last
// lane's value is also what row 64 adds at the same q.
constexpr int kRankMaxPhotons = 64;
struct RankLane {
    uint32_t v, next;   // F(q, lane); in the last lane also F(q, 64)
};

PQ_HD int rank_table_steps(int m, int n) { return m - 1 + (n < kRankMaxPhotons ? n : kRankMaxPhotons - 1); }

PQ_HD void rank_table_step(RankLane& x, int lane, uint32_t left, int s, int m, int n, int P, uint32_t* G) {
    const int q = s - lane;
    if (lane > n || q < 0 || q >= m - 1) return;
    x.v = lane == 0 || q == 0 ? 1u : x.v + left;
    G[lane * P + q + 1] = x.v;
    if (lane == kRankMaxPhotons - 1 && n == kRankMaxPhotons) {
        x.next = q == 0 ? 1u : x.next + x.v;
        G[kRankMaxPhotons * P + q + 1] = x.next;
    }
}

// Even split of [0, total) over `parts`: [start, start + count) of part w.
PQ_HD void split_range(uint64_t total, uint32_t parts, uint32_t w, uint64_t& start, uint64_t& count) {
    uint64_t q = total / parts, rem = total % parts;
    start = (uint64_t)w * q + (w < rem ? (uint64_t)w : rem);
    count = q + (w < rem ? 1u : 0u);
}

}  // namespace pq
