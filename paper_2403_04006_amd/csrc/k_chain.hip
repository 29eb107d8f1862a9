// Chain-rule boson sampling on the device (Clifford & Clifford's algorithm A,
// named in the Boson Sampling benchmark section): one workgroup runs one
// sample's whole draw sequence.
//
// Step k (k = 1..n) with rows r_1..r_{k-1} drawn so far and the first k input
// modes of the sample's order c_0..c_{k-1}: the permanents of every next row l,
//   out_l = perm(U_{r + l, c}) = sum_j U[l, c_j] M_j,
//   M_j = 2^{-(k-1)} sum_delta (prod delta) delta_j prod_{i < k} v_i(delta),
//   v_i = sum_j delta_j U[r_i, c_j],
// over the signs of the k columns with delta_0 = 1; r_k is the first l whose
// cumulative |out|^2 (in mode order) exceeds u_k times the total.
//
// Signs over the columns, not over the rows: the sum has twice the terms of the
// row form (2^{k-1}), but a term is one product of k - 1 factors where the row
// form needs every leave-one-out product of k (three complex products a
// column), and delta_j is constant per lane (columns 1..6), per wavefront (the
// next two or three) or follows from the running sum of the terms at each flip
// (the time columns): with P(t) the sum up to state t,
//   sum_t delta_j(t) g(t) = delta_j(end) P(end) + 2 sum_flips dd P(before),
// dd = +1 where delta_j goes from +1 to -1.  Per term and lane: 2 adds a row,
// 4 (k - 2) for the product, 4 for the sums.
//
// The step's column (k - 1 values, the same for every lane) is read once by
// each row of 16 lanes, lane i value i, and enters the sums as a DPP operand
// (v_fmac_f64 with row_newbcast): two LDS reads a step instead of one a row,
// which the LDS could not deliver to four wavefronts.
//
// Bound by FP64 vector instructions: 1.93e9 wavefront instructions for 1000
// samples of 20 photons in 400 modes, 80 % of the issue slots at the 1.9 GHz that
// the card holds under them.  4.7 ms against 6.3 for the row form with four lanes
// a term; 100 such samples (eight wavefronts each) 1.00 ms against 2.12, 529 of 12
// photons 70 us against 104 (there the draws, which one thread made mode by mode).
// Small calls are level, or a little slower: one sample of 8 photons in 16 modes
// 41 us against 37, in 30 modes 41 against 43.
//
// Every term sums over all k columns, so the M_j carry an error relative to the
// largest column's; the columns of an interferometer, lossless or dilated, are
// unit vectors.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "chain.h"
#include "device.h"
#include "lane_column.h"
#include "sweep_common.h"

namespace pq {

constexpr int kChainRows = 32;   // rows of a column in LDS (drawn rows, then zeros)

// Sums over the 64 lanes of N (a power of two) values per lane by recursive
// halving: lane l ends with value (l / (64 / N)) in x[0].
template <int N, int M = 32>
__device__ __forceinline__ void halve_sums(cplx* x, int lane) {
    if constexpr (N > 1) {
        constexpr int H = N / 2;
        const bool up = (lane & M) != 0;
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const cplx keep = up ? x[i + H] : x[i], give = up ? x[i] : x[i + H];
            x[i] = cplx{keep.re + shfl_xor_d(give.re, M), keep.im + shfl_xor_d(give.im, M)};
        }
        halve_sums<H, M / 2>(x, lane);
    } else if constexpr (M >= 1) {
        x[0].re += shfl_xor_d(x[0].re, M);
        x[0].im += shfl_xor_d(x[0].im, M);
        halve_sums<1, M / 2>(x, lane);
    }
}

// Slots of the per-wavefront sums: the terms' sum, the six lane columns, then
// the time columns.
constexpr int kChainSums = 32;

// The sums of step k over at most R drawn rows, LW wavefront columns.
template <int R, int LW>
__device__ __forceinline__ void chain_sweep(const cplx (*sB)[kChainRows], int k, int lane, int wv, cplx* sums) {
    constexpr int T = R - 6 - LW > 0 ? R - 6 - LW : 0;   // most time columns
    const int nfree = k - 1;
    const int nl = nfree < 6 ? nfree : 6;
    const int nw = nfree - nl < LW ? nfree - nl : LW;
    const int nt = nfree - nl - nw;
    double w = lane < (1 << nl) && wv < (1 << nw) ? 1.0 : 0.0;
    cplx v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = cplx{i < nfree ? 0.0 : 1.0, 0.0};   // rows not drawn yet: factors of 1
    for (int j = 0; j < k; ++j) {
        // column 0 is fixed, columns 1..nl are lane, the next nw wavefront columns
        const int bit = j >= 1 && j <= nl ? (lane >> (j - 1)) & 1 : (j > nl && j <= nl + nw ? (wv >> (j - 1 - nl)) & 1 : 0);
        add_column(v, load_column<R>(sB[j], lane), bit ? -1.0 : 1.0);
        if (bit) w = -w;
    }
    cplx P{0.0, 0.0};
    cplx A[T > 0 ? T : 1];
#pragma unroll
    for (int i = 0; i < (T > 0 ? T : 1); ++i) A[i] = cplx{0.0, 0.0};
    if constexpr (T > 0) {
        const cplx(*sT)[kChainRows] = sB + (1 + nl + nw);   // the time columns
        // one step: the term of the current state, then the flip of column q
        // in direction dd (2: from +1 to -1) and its share of the sums
        auto step = [&](auto q, double sign, double dd) {
            constexpr int Q = decltype(q)::value;
            const LaneColumn b = load_column<R>(sT[Q], lane);
            cfma_to(P, sign, row_product(v));
            cfma_to(A[Q], dd, P);
            add_column(v, b, -dd);
        };
        using std::integral_constant;
        if (nt >= 3) {
            if constexpr (T >= 3) {
                // blocks of eight states: every step but the last flips one of
                // the first three columns, in a direction known here (column
                // 2's alternates by block), and the term's sign alternates
                const int blocks = T == 3 ? 1 : 1 << (nt - 3);
#pragma unroll 1
                for (int blk = 0; blk < blocks; ++blk) {
                    step(integral_constant<int, 0>{}, 1.0, 2.0);
                    step(integral_constant<int, 1>{}, -1.0, 2.0);
                    step(integral_constant<int, 0>{}, 1.0, -2.0);
                    step(integral_constant<int, 2>{}, -1.0, blk & 1 ? -2.0 : 2.0);
                    step(integral_constant<int, 0>{}, 1.0, 2.0);
                    step(integral_constant<int, 1>{}, -1.0, -2.0);
                    step(integral_constant<int, 0>{}, 1.0, -2.0);
                    const int i = __builtin_ctz(blk + 1);   // column 3 + i, unless this was the last block
                    const bool more = blk + 1 < blocks;
                    const LaneColumn b = load_column<R>(sT[more ? 3 + i : 0], lane);
                    cfma_to(P, -1.0, row_product(v));
                    if (more) {
                        const double dd = ((blk + 1) >> (i + 1)) & 1 ? -2.0 : 2.0;
                        flip_sums<3, T>(A, 3 + i, dd, P);
                        add_column(v, b, -dd);
                    }
                }
            }
        } else {
            const int states = 1 << nt;
#pragma unroll 1
            for (int t = 1; t < states; ++t) {
                const double sign = t & 1 ? 1.0 : -1.0;
                if (t & 1) step(integral_constant<int, 0>{}, sign, t & 2 ? -2.0 : 2.0);
                else if constexpr (T >= 2) step(integral_constant<int, 1>{}, sign, 2.0);
            }
            cfma_to(P, nt > 0 ? -1.0 : 1.0, row_product(v));
        }
        // the last state has only its top digit set
#pragma unroll
        for (int q = 0; q < T; ++q)
            if (q < nt) cfma_to(A[q], q == nt - 1 ? -1.0 : 1.0, P);
    } else {
        P = row_product(v);
    }
    constexpr int N = T <= 1 ? 8 : (T <= 9 ? 16 : kChainSums);
    cplx x[N];
    x[0] = cplx{w * P.re, w * P.im};
#pragma unroll
    for (int i = 1; i < N; ++i) {
        if (i <= 6) {
            const double s = (lane >> (i - 1)) & 1 ? -1.0 : 1.0;
            x[i] = cplx{s * x[0].re, s * x[0].im};
        } else {
            x[i] = i - 7 < T ? cplx{w * A[i - 7 < T ? i - 7 : 0].re, w * A[i - 7 < T ? i - 7 : 0].im} : cplx{0.0, 0.0};
        }
    }
    halve_sums<N>(x, lane);
    if ((lane & (64 / N - 1)) == 0) sums[lane / (64 / N)] = x[0];
}

// Step k by the sweep for the next even number of rows.
template <int R, int RMAX, int LW>
__device__ __forceinline__ void chain_step(const cplx (*sB)[kChainRows], int k, int lane, int wv, cplx* sums) {
    if constexpr (R >= RMAX) {
        chain_sweep<RMAX, LW>(sB, k, lane, wv, sums);
    } else {
        if (k - 1 <= R) chain_sweep<R, LW>(sB, k, lane, wv, sums);
        else chain_step<R + 2, RMAX, LW>(sB, k, lane, wv, sums);
    }
}

template <int RMAX, int LW>
__global__ __launch_bounds__(64 << LW, LW == 2 ? 3 : 2) void chain_kernel(const ChainArgs a) {
    constexpr int NT = 64 << LW, W = 1 << LW;
    __shared__ cplx sB[RMAX + 2][kChainRows];      // U[r_i, c_j] at [j][i]
    __shared__ cplx sSum[W][kChainSums];
    __shared__ cplx sM[RMAX + 2];
    __shared__ double sW[kChainMaxModes];
    __shared__ int sCol[RMAX + 2];
    __shared__ int sBad, sPick;
    const int s = (int)blockIdx.x;
    if (s >= a.samples) return;
    const int tid = (int)threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int n = a.n, m = a.m;
    if (tid == 0) sBad = 0;
    for (int e = tid; e < (RMAX + 2) * kChainRows; e += NT) sB[e / kChainRows][e % kChainRows] = cplx{0.0, 0.0};
    __syncthreads();
    // the input modes come from device memory the host cannot check: an entry
    // outside [0, m) marks the sample (every draw -1) and the call's status,
    // and no row of U is read through it
    for (int j = tid; j < n; j += NT) {
        int c = a.order[(size_t)s * n + j];
        if (c < 0 || c >= m) {
            atomicOr(&sBad, 1);
            c = 0;
        }
        sCol[j] = c;
    }
    __syncthreads();
    if (sBad) {
        for (int j = tid; j < n; j += NT) a.out[(size_t)s * n + j] = -1;
        if (tid == 0) __hip_atomic_fetch_or(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    for (int k = 1; k <= n; ++k) {
        if (k == 1) {
            if (tid == 0) sM[0] = cplx{1.0, 0.0};
        } else {
            chain_step<2, RMAX, LW>(sB, k, lane, wv, sSum[wv]);
            __syncthreads();
            // the columns' sums over the wavefronts (their columns' signs included)
            if (tid < k) {
                const int nl = k - 1 < 6 ? k - 1 : 6;
                const int nw = k - 1 - nl < LW ? k - 1 - nl : LW;
                const int slot = tid <= nl ? tid : (tid <= nl + nw ? 0 : 7 + tid - 1 - nl - nw);
                cplx M{0.0, 0.0};
#pragma unroll
                for (int x = 0; x < W; ++x) {
                    const double d = tid > nl && tid <= nl + nw && ((x >> (tid - 1 - nl)) & 1) ? -1.0 : 1.0;
                    cfma_to(M, d, sSum[x][slot]);
                }
                const double scale = ldexp(1.0, -(k - 1));
                sM[tid] = cplx{M.re * scale, M.im * scale};
            }
        }
        __syncthreads();
        // weights of the next mode
        for (int l = tid; l < m; l += NT) {
            const cplx* Ul = a.U + (size_t)l * (size_t)a.ldu;
            double re = 0.0, im = 0.0;
            for (int j = 0; j < k; ++j) {
                const cplx u = Ul[sCol[j]];
                const cplx L = sM[j];
                re = __builtin_fma(u.re, L.re, re);
                re = __builtin_fma(-u.im, L.im, re);
                im = __builtin_fma(u.re, L.im, im);
                im = __builtin_fma(u.im, L.re, im);
            }
            sW[l] = re * re + im * im;
        }
        __syncthreads();
        // the draw, by the first wavefront: each lane sums a run of modes, a
        // scan over the lanes finds the run that holds the target
        if (wv == 0) {
            const int run = (m + 63) / 64;
            const int l0 = lane * run < m ? lane * run : m, l1 = l0 + run < m ? l0 + run : m;
            double mine = 0.0;
            for (int l = l0; l < l1; ++l) mine += sW[l];
            double upto = mine;
#pragma unroll
            for (int h = 1; h < 64; h <<= 1) {
                const double o = __shfl_up(upto, h, 64);
                if (lane >= h) upto += o;
            }
            const double total = __shfl(upto, 63, 64);
            double before = __shfl_up(upto, 1, 64);
            if (lane == 0) before = 0.0;
            const double target = a.uniforms[(size_t)s * n + (k - 1)] * total;
            // a lane of zero weights is passed over: the scan's order of additions
            // differs by lane, so its sum can exceed the target by rounding alone;
            // where that leaves none, the last mode of any weight is taken, and
            // the last mode of all where the target is not below the total
            const unsigned long long some = __ballot(mine > 0.0), hit = some & __ballot(upto > target);
            const int who = hit ? __builtin_ctzll(hit) : (some && target < total ? 63 - __builtin_clzll(some) : -1);
            if (who < 0) {
                if (lane == 0) sPick = m - 1;
            } else if (lane == who) {
                int pick = m - 1;
                for (int l = l0; l < l1; ++l) {
                    before += sW[l];
                    if (sW[l] > 0.0) {
                        pick = l;   // where rounding leaves the run's sum at the target: its last mode
                        if (before > target) break;
                    }
                }
                sPick = pick;
            }
            if (lane == 0) a.out[(size_t)s * n + (k - 1)] = sPick;
        }
        __syncthreads();
        if (tid < n && k < n) sB[tid][k - 1] = a.U[(size_t)sPick * (size_t)a.ldu + sCol[tid]];
        __syncthreads();
    }
}

template <int RMAX>
static void launch_chain_rows(const ChainArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)(a.samples > 0 ? a.samples : 1));
    // eight wavefronts a sample while every sample still has a CU of its own
    // (they need the registers of one)
    if (a.samples <= 256) hipLaunchKernelGGL((chain_kernel<RMAX, 3>), grid, dim3(512), 0, s, a);
    else hipLaunchKernelGGL((chain_kernel<RMAX, 2>), grid, dim3(256), 0, s, a);
}

hipError_t launch_chain(const ChainArgs& a, hipStream_t s) {
    // n - 1 rows at the last step
    if (a.n <= 9) launch_chain_rows<8>(a, s);
    else if (a.n <= 13) launch_chain_rows<12>(a, s);
    else if (a.n <= 17) launch_chain_rows<16>(a, s);
    else if (a.n <= 21) launch_chain_rows<20>(a, s);
    else if (a.n <= kChainMaxPhotons) launch_chain_rows<24>(a, s);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace pq
