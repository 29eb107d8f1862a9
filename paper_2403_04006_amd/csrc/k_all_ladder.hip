// Kernels of the all-outputs ladder (see all.h).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "all.h"
#include "device.h"
#include "ladder.h"

namespace pq {

// Value of the output of rank `idx` at level k: the sum over its photons of
// U[mode][j_k] times the level below without that photon.  u is the column
// j_k by q; rs[c] = 1 / sqrt(c), whose product over the photons (c the
// photon's place among those of its mode) is 1 / sqrt(prod t_i!).  Four
// photons' loads are issued before the first is used.
template <bool LAST>
__device__ __forceinline__ cplx ladder_value(int k, int P, const uint32_t* G, const cplx* u, const double* rs,
                                             const cplx* in, uint32_t idx, double& nrm) {
    uint32_t rank = idx, at = idx;
    int qlast = -1, run = 0;
    cplx v{0.0, 0.0};
    for (int p0 = 0; p0 < k; p0 += 4) {
        cplx x[4];
        int qs[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if (p0 + g < k) {
                const uint32_t* row = G + (k - p0 - g) * P;
                const int q = ladder_mode(row, P, rank);
                const uint32_t f = row[q];
                x[g] = in[at - f];
                at += row[q - P] - f;
                rank -= f;
                qs[g] = q;
                if (LAST) {
                    run = q == qlast ? run + 1 : 1;
                    qlast = q;
                    nrm *= rs[run];
                }
            }
        }
#pragma unroll
        for (int g = 0; g < 4; ++g)
            if (p0 + g < k) cmadd(v, u[qs[g]], x[g]);
    }
    return v;
}

// Levels 1, 2 and 3 directly: the permanent of k rows of the columns u[0..k).
template <bool LAST>
__device__ __forceinline__ cplx ladder_first(int k, int m, int P, const uint32_t* G, const cplx* u, const double* rs,
                                             uint32_t idx, double& nrm) {
    int q[3];
    uint32_t rank = idx;
    int run = 0;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        if (p < k) {
            const uint32_t* row = G + (k - p) * P;
            q[p] = ladder_mode(row, P, rank);
            rank -= row[q[p]];
            if (LAST) {
                run = p > 0 && q[p] == q[p - 1] ? run + 1 : 1;
                nrm *= rs[run];
            }
        }
    }
    const cplx *u0 = u, *u1 = u + m, *u2 = u + 2 * m;
    if (k == 1) return u0[q[0]];
    cplx s{0.0, 0.0};
    cmadd(s, u0[q[0]], u1[q[1]]);
    cmadd(s, u0[q[1]], u1[q[0]]);
    if (k == 2) return s;
    cplx v = cmul(u2[q[2]], s);
    s = cplx{0.0, 0.0};
    cmadd(s, u0[q[0]], u1[q[2]]);
    cmadd(s, u0[q[2]], u1[q[0]]);
    cmadd(v, u2[q[1]], s);
    s = cplx{0.0, 0.0};
    cmadd(s, u0[q[1]], u1[q[2]]);
    cmadd(s, u0[q[2]], u1[q[1]]);
    cmadd(v, u2[q[0]], s);
    return v;
}

// The first level where its k photons are in one input mode: k! times the product
// of its column u over the output's photons (the factors of k! one by one, so that
// nothing over- or underflows that the value itself does not).
template <bool LAST>
__device__ __forceinline__ cplx ladder_direct(int k, int P, const uint32_t* G, const cplx* u, const double* rs,
                                              uint32_t idx, double& nrm) {
    uint32_t rank = idx;
    int qlast = -1, run = 0;
    cplx v{1.0, 0.0};
    for (int p = 0; p < k; ++p) {
        const uint32_t* row = G + (k - p) * P;
        const int q = ladder_mode(row, P, rank);
        rank -= row[q];
        const cplx f = u[q];
        const double c = (double)(p + 1);
        v = cmul(v, cplx{c * f.re, c * f.im});
        if (LAST) {
            run = q == qlast ? run + 1 : 1;
            qlast = q;
            nrm *= rs[run];
        }
    }
    return v;
}

// Levels up to k0 by one workgroup in LDS (at most kAllLadderSmall values, the
// last one, which goes to `out` or the outputs, kAllLadderFirst).  Bound by the
// latency of its dependent rounds, not by work: 11 us for the first four levels
// of 16 modes (17 us before the table was made by lane shifts and the photons'
// searches lost their branches).
__global__ __launch_bounds__(kAllLadderBlock) void all_ladder_small_kernel(const AllLadderArgs a, cplx* out) {
    __shared__ cplx buf[2][kAllLadderSmall];
    __shared__ cplx u[kAllLadderCols];
    __shared__ uint32_t G[(kAllMaxPhotons + 1) * kAllMaxModes];
    __shared__ double rs[kAllMaxPhotons + 1];
    const int tid = (int)threadIdx.x;
    const int m = a.m, n = a.n, P = ladder_stride(m);
    if (tid < 64) ladder_table(m, a.k0, P, tid, G);
    else if (tid < 64 + a.k0) rs[tid - 63] = 1.0 / sqrt((double)(tid - 63));
    else if (tid >= 128)
        for (int e = tid - 128; e < m * a.k0; e += kAllLadderBlock - 128) {
            const int k = e / m, q = e - k * m;
            u[e] = a.U[(size_t)(m - 1 - q) * (size_t)a.ldu + a.col[k]];
        }
    __syncthreads();
    const int first = a.s1 ? a.s1 : (a.k0 < 3 ? a.k0 : 3);
    for (int k = first; k <= a.k0; ++k) {
        // vectors of k photons in m modes: those of the last m - 1 with at
        // most k, i.e. the sum of a column of G
        uint32_t count = 0;
        for (int r = 0; r <= k; ++r) count += m > 1 ? G[r * P + m - 1] : 0;
        if (m == 1) count = 1;
        const cplx* in = buf[(k - 1) & 1];
        for (uint32_t idx = (uint32_t)tid; idx < count; idx += kAllLadderBlock) {
            double nrm = a.norm_s;
            const cplx* uk = u + (k - 1) * m;
            auto value = [&](auto last) {
                constexpr bool LAST = decltype(last)::value;
                if (k > first) return ladder_value<LAST>(k, P, G, uk, rs, in, idx, nrm);
                return a.s1 ? ladder_direct<LAST>(k, P, G, u, rs, idx, nrm) : ladder_first<LAST>(k, m, P, G, u, rs, idx, nrm);
            };
            const cplx v = k < n ? value(std::false_type{}) : value(std::true_type{});
            if (k == n) {
                a.perm[idx] = v;
                if (a.amp) a.amp[idx] = cplx{v.re * nrm, v.im * nrm};
            } else if (k < a.k0) {
                buf[k & 1][idx] = v;
            } else {
                out[idx] = v;
            }
        }
        __syncthreads();
    }
}

// One level: a workgroup takes `run` consecutive outputs, whose inputs lie in
// at most m nearly consecutive stretches of the level below.  Workgroups are
// dealt to the 8 XCDs in turn, so the run index is permuted to give every XCD
// (its own L2) one contiguous eighth of the level.  Bound by vector
// instructions (about 35 per photon: the search, two table reads, the load and
// four multiply-adds), then by the reads of the level below and the write of
// the outputs: 52 us for the 3,268,760 outputs of 10 photons in 16 modes
// (2.0 TB/s written).  Walking the modes instead of the photons took 79 us, the
// wavefronts splitting at every mode.
template <bool LAST, bool FIRST>
__global__ __launch_bounds__(kBlock) void all_ladder_level_kernel(const AllLevelArgs p) {
    extern __shared__ double lds[];
    const AllLadderArgs& a = p.a;
    const int tid = (int)threadIdx.x;
    const int m = a.m, P = ladder_stride(m);
    cplx* u = (cplx*)lds;
    double* rs = (double*)(u + m);
    uint32_t* G = (uint32_t*)(rs + p.k + 1);
    if (tid < 64) {
        ladder_table(m, p.k, P, tid, G);
    } else {
        for (int q = tid - 64; q < m; q += kBlock - 64) u[q] = a.U[(size_t)(m - 1 - q) * (size_t)a.ldu + a.col[p.k - 1]];
        if (LAST)
            for (int c = tid - 64; c <= p.k; c += kBlock - 64) rs[c] = c > 0 ? 1.0 / sqrt((double)c) : 1.0;
    }
    __syncthreads();
    const uint32_t per = (gridDim.x + 7) / 8;
    const uint64_t chunk = (uint64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
    const uint64_t first = chunk * p.run;
    const uint64_t last = first + p.run < p.count ? first + p.run : p.count;
    for (uint64_t e = first + (uint64_t)tid; e < last; e += kBlock) {
        const uint32_t idx = (uint32_t)e;
        double nrm = a.norm_s;
        cplx v;
        if constexpr (FIRST) v = ladder_direct<LAST>(p.k, P, G, u, rs, idx, nrm);
        else v = ladder_value<LAST>(p.k, P, G, u, rs, p.in, idx, nrm);
        if (LAST) {
            a.perm[idx] = v;
            if (a.amp) a.amp[idx] = cplx{v.re * nrm, v.im * nrm};
        } else {
            p.out[idx] = v;
        }
    }
}

hipError_t launch_all_ladder_small(const AllLadderArgs& a, cplx* out, hipStream_t s) {
    if (a.m < 1 || a.m > kAllMaxModes || a.n < 1 || a.n > kAllMaxPhotons || a.k0 < 1 || a.k0 > a.n ||
        a.s1 > a.k0 || a.m * a.k0 > kAllLadderCols || (a.k0 < a.n && !out))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(all_ladder_small_kernel, dim3(1), dim3(kAllLadderBlock), 0, s, a, out);
    return hipGetLastError();
}

hipError_t launch_all_ladder_level(const AllLevelArgs& a, hipStream_t s) {
    const bool first = a.k == a.a.s1;
    if (a.run == 0 || a.run % kBlock || a.k < 2 || a.k > a.a.n || (!first && !a.in)) return hipErrorInvalidValue;
    // whole eighths, so that the permuted run index covers every run (runs
    // past the last output are empty)
    const uint64_t runs = ((uint64_t)a.count + a.run - 1) / a.run;
    const dim3 grid((unsigned)((runs + 7) / 8 * 8)), block(kBlock);
    const size_t k = (size_t)a.k, m = (size_t)a.a.m;
    const size_t lds = sizeof(cplx) * m + sizeof(double) * (k + 1) + sizeof(uint32_t) * (size_t)ladder_stride(a.a.m) * (k + 1);
    if (first && a.k == a.a.n) hipLaunchKernelGGL((all_ladder_level_kernel<true, true>), grid, block, lds, s, a);
    else if (first) hipLaunchKernelGGL((all_ladder_level_kernel<false, true>), grid, block, lds, s, a);
    else if (a.k == a.a.n) hipLaunchKernelGGL((all_ladder_level_kernel<true, false>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((all_ladder_level_kernel<false, false>), grid, block, lds, s, a);
    return hipGetLastError();
}

}  // namespace pq
