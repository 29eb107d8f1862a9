// Long collision-free permanents: eight terms at a time over pairs of columns,
// a term's columns shared by the two wavefronts of a workgroup.
//
// The three lowest time digits stand at their middle and move the sums of a
// pair of columns by +-(a_k, b_k), k = 0..3 (the sign patterns up to a common
// sign; first k, then -k).  With centre sums c, d the pair's products are
//   (c + a_k)(d + b_k) = E_k + O_k,   (c - a_k)(d - b_k) = E_k - O_k,
//   E_k = c d + a_k b_k,              O_k = c b_k + d a_k.
// The constants a_k b_k are the same everywhere, and a step of a higher digit by
// (x, y) moves O_k by the constant x b_k + y a_k, so the four O_k of every pair
// stay in registers: 8 adds for the step of O, 4 for c and d, 4 for c d, 8 for E
// and 16 for the eight factors, 2.5 instructions per column and term where the
// one-by-one walk takes 2 for the row and 4 for the product of every column.
// With the 4 per pair and term of the product: 4.5 instead of 6.
//
// A pair keeps 12 doubles a lane.  Eight pairs and the eight running products
// fill half the registers of a SIMD's lane, so two wavefronts (on two SIMDs)
// take the pairs of one term, and exchange products through LDS once a block of
// eight terms; two workgroups' wavefronts on a SIMD cover the exchange.  The
// second wavefront finishes the terms; its wait and half of its reads lie
// before its last pair's work.  Row constants come through scalar loads ahead of
// their use: 160 bytes a pair and block, where the one-by-one walk reads 256.
//
// Bound by FP64 issue at the clock that the card's power allows under it: 30
// photons 1052 FP64 instructions a block of eight terms and lane (1,480 one by
// one), 2.86 -> 2.26 ms; 28 photons 698 -> 540 us; 32 photons 13.0 -> 9.7 ms.
// Exchanging through a ring of four blocks with counters instead of a barrier
// was no faster (2.33 ms at 30).
#pragma once
#include <hip/hip_runtime.h>

#include "device.h"
#include "kernels.h"

namespace pq {

typedef const __attribute__((address_space(4))) cplx pair_kc;

// One pair's moves of a step (of its two sums and of O), and its a_k b_k.
struct PairMove {
    cplx x, y, o[4];
};
struct PairProd {
    cplx e[4];
};

__device__ __forceinline__ cplx pair_load(pair_kc* v) { return cplx{v->re, v->im}; }

__device__ __forceinline__ PairMove pair_move(pair_kc* step, int p) {
    PairMove r{pair_load(step + 6 * p), pair_load(step + 6 * p + 1), {}};
#pragma unroll
    for (int k = 0; k < 4; ++k) r.o[k] = pair_load(step + 6 * p + 2 + k);
    return r;
}

__device__ __forceinline__ PairProd pair_prod(pair_kc* prod, int p) {
    PairProd r;
#pragma unroll
    for (int k = 0; k < 4; ++k) r.e[k] = pair_load(prod + 4 * p + k);
    return r;
}

// The wavefront ROLE of a workgroup: pairs [FIRST, FIRST + N).
template <int PA, int PB, int ROLE>
__device__ __forceinline__ void pair_walk(const PairArgs& a, int lane, cplx (*buf)[8][64], double* half) {
    constexpr int P = PA + PB, W = 2 * P;
    constexpr int N = ROLE ? PB : PA, FIRST = ROLE ? PA : 0;
    // With eight pairs of its own wavefront 1 has no registers left to finish all
    // terms: 0 then takes the +k terms and 1 the -k terms.
    constexpr bool EVEN = PB == 8;
    constexpr int T0 = EVEN && ROLE ? 4 : 0, TERMS = EVEN ? 4 : (ROLE ? 8 : 0);   // finished here
    constexpr int EARLY = EVEN ? 0 : 4;   // of the other's products, read before the last pair's work
    const cplx* lrow = a.tab + W;
    const cplx* prod = lrow + kMaxLaneDigits * W;
    const cplx* dev = prod + 4 * P;
    const cplx* steps = dev + 8 * P;

    uint64_t start, count;
    split_range(a.blocks, a.groups, blockIdx.x, start, count);
    cplx c[N], d[N], o[N][4];
    {
        pair_kc* b = (pair_kc*)(a.tab + 2 * FIRST);
#pragma unroll
        for (int p = 0; p < N; ++p) {
            c[p] = cplx{b[2 * p].re, b[2 * p].im};
            d[p] = cplx{b[2 * p + 1].re, b[2 * p + 1].im};
        }
        for (int i = 0; i < a.n_lane; ++i) {
            pair_kc* l = (pair_kc*)(lrow + (size_t)i * W + 2 * FIRST);
            const double bit = (lane >> i) & 1 ? 1.0 : 0.0;
#pragma unroll
            for (int p = 0; p < N; ++p) {
                c[p].re = __builtin_fma(bit, l[2 * p].re, c[p].re);
                c[p].im = __builtin_fma(bit, l[2 * p].im, c[p].im);
                d[p].re = __builtin_fma(bit, l[2 * p + 1].re, d[p].re);
                d[p].im = __builtin_fma(bit, l[2 * p + 1].im, d[p].im);
            }
        }
        const uint64_t g = start ^ (start >> 1);
        for (int i = 0; i < a.n_outer; ++i)
            if ((g >> i) & 1ull) {
                pair_kc* s = (pair_kc*)(steps + ((size_t)i * 2 * P + FIRST) * 6);
#pragma unroll
                for (int p = 0; p < N; ++p) {
                    cadd_to(c[p], cplx{s[6 * p].re, s[6 * p].im});
                    cadd_to(d[p], cplx{s[6 * p + 1].re, s[6 * p + 1].im});
                }
            }
        pair_kc* v = (pair_kc*)(dev + 8 * FIRST);
#pragma unroll
        for (int p = 0; p < N; ++p)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const cplx ak{v[8 * p + 2 * k].re, v[8 * p + 2 * k].im};
                const cplx bk{v[8 * p + 2 * k + 1].re, v[8 * p + 2 * k + 1].im};
                o[p][k] = cmul(c[p], bk);
                cmadd(o[p][k], d[p], ak);
            }
    }

    auto meet = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    };
    cplx acc{0.0, 0.0};
    pair_kc* const base = (pair_kc*)(steps + (size_t)FIRST * 6);
    pair_kc* const pk0 = (pair_kc*)(prod + 4 * FIRST);
    PairProd pe = pair_prod(pk0, 0);
    const uint32_t end = (uint32_t)(start + count);
    for (uint32_t t = (uint32_t)start + 1; t <= end; ++t) {
        // the step to block t; past the last block one of the last digit, whose
        // sums are not used
        int i = __builtin_ctz(t);
        i = i < a.n_outer ? i : a.n_outer - 1;
        pair_kc* const step = base + (uint32_t)(2 * i + (int)((t >> i) >> 1 & 1)) * (uint32_t)(6 * P);
        // kept from being hoisted out of the loop, where they do not fit
        pair_kc* pk = pk0;
        asm("" : "+s"(pk));
        cplx (*const s)[64] = buf[t & 1];
        cplx pr[8], q[8];
        if constexpr (EVEN) pe = pair_prod(pk, 0);
#pragma unroll
        for (int p = 0; p < N; ++p) {
            // The moves are needed at the end of this pair's work, the constants
            // of the next pair at its start.  (EVEN: all of a pair's one pair
            // ahead, none over the loop's end; what spills least)
            const PairProd re = pe;
            const PairMove r = pair_move(step, p);
            if (!EVEN || p + 1 < N) pe = pair_prod(pk, p + 1 < N ? p + 1 : 0);
            if constexpr (!EVEN && ROLE) {
                // the other wavefront's products, behind the last pair's work
                if (p == N - 1) {
                    meet();
#pragma unroll
                    for (int k = 0; k < EARLY; ++k) q[k] = s[k][lane];
                }
            }
            const cplx e0 = cmul(c[p], d[p]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const cplx e{e0.re + re.e[k].re, e0.im + re.e[k].im};
                const cplx f{e.re + o[p][k].re, e.im + o[p][k].im};
                const cplx h{e.re - o[p][k].re, e.im - o[p][k].im};
                pr[k] = p ? cmul(pr[k], f) : f;
                pr[4 + k] = p ? cmul(pr[4 + k], h) : h;
                cadd_to(o[p][k], r.o[k]);
            }
            cadd_to(c[p], r.x);
            cadd_to(d[p], r.y);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the terms that the other wavefront finishes
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k < T0 || k >= T0 + TERMS) s[k][lane] = pr[k];
        if constexpr (EVEN || !ROLE) meet();
        if constexpr (TERMS > 0) {
            // +k terms and -k terms have opposite signs
            cplx up{0.0, 0.0}, dn{0.0, 0.0};
#pragma unroll
            for (int k = T0; k < T0 + TERMS; ++k) {
                if (k >= EARLY) q[k] = s[k][lane];
                cmadd(k < 4 ? up : dn, pr[k], q[k]);
            }
            // block t - 1: a step changes the sign
            const double w = (t & 1) ? 1.0 : -1.0;
            acc.re = __builtin_fma(w, up.re - dn.re, acc.re);
            acc.im = __builtin_fma(w, up.im - dn.im, acc.im);
        }
    }
    if constexpr (TERMS == 0) return;
    // sign of the lane digits (block 0 of the walk has every higher digit at zero)
    const double wl = lane < a.lane_states ? ((__builtin_popcount(lane) & 1) ? -1.0 : 1.0) : 0.0;
    cdd sum = wave_reduce(to_cdd(cplx{acc.re * wl, acc.im * wl}));
    if constexpr (EVEN) {
        if (ROLE == 0 && lane == 0) {
            half[0] = sum.re.hi;
            half[1] = sum.re.lo;
            half[2] = sum.im.hi;
            half[3] = sum.im.lo;
        }
        meet();
        if constexpr (ROLE == 0) return;
        sum = cdd_add(cdd{{half[0], half[1]}, {half[2], half[3]}}, sum);
    }
    if (lane == 0) {
        double* out = a.partials + 4 * (size_t)blockIdx.x;
        out[0] = sum.re.hi;
        out[1] = sum.re.lo;
        out[2] = sum.im.hi;
        out[3] = sum.im.lo;
    }
}

template <int PA, int PB>
__global__ __launch_bounds__(128, 2) void pair_kernel(const PairArgs a) {
    // products on their way, two blocks in turn
    __shared__ cplx buf[2][8][64];
    __shared__ double half[4];
    const int lane = threadIdx.x & 63;
    if (__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) == 0) pair_walk<PA, PB, 0>(a, lane, buf, half);
    else pair_walk<PA, PB, 1>(a, lane, buf, half);
}

#define PQ_PINST(P)                                                                                  \
    hipError_t launch_pair_##P(const PairArgs& a, hipStream_t s) {                                   \
        hipLaunchKernelGGL((pair_kernel<(P + 1) / 2, P / 2>), dim3(a.groups), dim3(128), 0, s, a);   \
        return hipGetLastError();                                                                    \
    }                                                                                                \
    int occupancy_pair_##P() {                                                                       \
        int nb = 0;                                                                                  \
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(                           \
            &nb, pair_kernel<(P + 1) / 2, P / 2>, 128, 0);                                           \
        return e == hipSuccess ? nb : 0;                                                             \
    }

}  // namespace pq
