// Kernels of the hafnian table built level by level (see haf.h).
#include <hip/hip_runtime.h>

#include "haf.h"
#include "ladder.h"

namespace pq {

// LDS of a workgroup: compact matrix [d][d] and loop weights [d], both by q
// (the mode counted from the last), then the rank table up to `top` photons.
struct HafLadderLds {
    cplx* A;
    cplx* gamma;
    uint32_t* G;
};

__host__ __device__ inline size_t haf_ladder_lds(int d, int top) {
    return sizeof(cplx) * (size_t)(d * d + d) + sizeof(uint32_t) * (size_t)(top + 1) * (size_t)ladder_stride(d);
}

__device__ __forceinline__ HafLadderLds haf_ladder_setup(const HafLadderArgs& a, char* mem, int top, int nthreads) {
    HafLadderLds L;
    const int d = a.d, tid = (int)threadIdx.x;
    L.A = (cplx*)mem;
    L.gamma = L.A + d * d;
    L.G = (uint32_t*)(L.gamma + d);
    if (tid < 64) {
        ladder_table(d, top, ladder_stride(d), tid, L.G);
    } else {
        for (int e = tid - 64; e < d * d + d; e += nthreads - 64) {
            if (e < d * d) {
                const int mi = a.mode[d - 1 - e / d], mj = a.mode[d - 1 - e % d];
                // only the upper triangle of A is read
                L.A[e] = mi < mj ? a.A[(size_t)mi * (size_t)a.lda + mj] : a.A[(size_t)mj * (size_t)a.lda + mi];
            } else {
                L.gamma[e - d * d] = a.gamma ? a.gamma[a.mode[d - 1 - (e - d * d)]] : cplx{0.0, 0.0};
            }
        }
    }
    return L;
}

// h of the vector of rank idx at level s from levels s - 1 (h1, loops only)
// and s - 2 (h2).  Four photons' loads are issued before the first is used.
__device__ __forceinline__ cplx haf_ladder_value(const HafLadderLds& L, int d, int P, int s, bool loops,
                                                 const cplx* h1, const cplx* h2, uint32_t idx) {
    const uint32_t* row0 = L.G + s * P;
    const int q0 = ladder_mode(row0, P, idx);
    uint32_t rank = idx - row0[q0];
    const cplx* Aq = L.A + q0 * d;
    cplx v{0.0, 0.0};
    if (loops) cmadd(v, L.gamma[q0], h1[rank]);
    uint32_t at = rank;
    for (int p0 = 1; p0 < s; p0 += 4) {
        cplx x[4];
        int qs[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if (p0 + g < s) {
                const uint32_t* row = L.G + (s - p0 - g) * P;
                const int q = ladder_mode(row, P, rank);
                const uint32_t f = row[q];
                x[g] = h2[at - f];
                at += row[q - P] - f;
                rank -= f;
                qs[g] = q;
            }
        }
#pragma unroll
        for (int g = 0; g < 4; ++g)
            if (p0 + g < s) cmadd(v, Aq[qs[g]], x[g]);
    }
    return v;
}

// Value of pattern p: its rank among the vectors of its photon number.
__device__ __forceinline__ void haf_ladder_read(const HafLadderArgs& a, const uint32_t* G, int P, int p) {
    const uint8_t* r = a.reps + (size_t)p * (size_t)a.d;
    int s = 0;
    for (int i = 0; i < a.d; ++i) s += r[i];
    if (!a.gamma && (s & 1)) {
        a.out[p] = cplx{0.0, 0.0};
        return;
    }
    uint32_t rank = 0;
    int rem = s;
    for (int i = 0; i < a.d; ++i) {
        const int c = r[i];
        for (int e = 0; e < c; ++e) rank += G[(rem--) * P + a.d - 1 - i];
    }
    a.out[p] = a.h[a.off[s] + rank];
}

// The levels up to s0 by one workgroup, the last three kept in LDS; when s0 is
// the last level, the patterns' values as well.  Bound by the latency of its
// dependent rounds: 11 us for levels 2 to 8 of 6 modes.
__global__ __launch_bounds__(kHafLadderBlock) void haf_ladder_small_kernel(const HafLadderArgs a) {
    extern __shared__ double mem[];
    __shared__ cplx ring[3][kHafLadderSmall];
    const int tid = (int)threadIdx.x;
    const int P = ladder_stride(a.d);
    const bool loops = a.gamma != nullptr;
    const HafLadderLds L = haf_ladder_setup(a, (char*)mem, a.s0, kHafLadderBlock);
    if (tid == 0) {
        ring[0][0] = cplx{1.0, 0.0};
        a.h[a.off[0]] = cplx{1.0, 0.0};
    }
    __syncthreads();
    for (int s = loops ? 1 : 2; s <= a.s0; s += loops ? 1 : 2) {
        const uint32_t count = a.off[s + 1] - a.off[s];
        const cplx* h1 = ring[(s - 1) % 3];
        const cplx* h2 = ring[s >= 2 ? (s - 2) % 3 : 0];
        for (uint32_t idx = (uint32_t)tid; idx < count; idx += kHafLadderBlock) {
            const cplx v = haf_ladder_value(L, a.d, P, s, loops, h1, h2, idx);
            ring[s % 3][idx] = v;
            a.h[a.off[s] + idx] = v;
        }
        __syncthreads();
    }
    if (a.s0 >= a.N)
        for (int p = tid; p < a.npat; p += kHafLadderBlock) haf_ladder_read(a, L.G, P, p);
}

// One level, one thread per vector.  Bound by the latency of its photons'
// searches and loads (5 to 10 us a level up to 20,349 vectors of 16 photons).
__global__ __launch_bounds__(kBlock) void haf_ladder_level_kernel(const HafLadderArgs a, int s) {
    extern __shared__ double mem[];
    const int P = ladder_stride(a.d);
    const bool loops = a.gamma != nullptr;
    const HafLadderLds L = haf_ladder_setup(a, (char*)mem, s, kBlock);
    __syncthreads();
    const uint32_t count = a.off[s + 1] - a.off[s];
    const cplx* h1 = a.h + a.off[s - 1];
    const cplx* h2 = a.h + a.off[s - 2];
    for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < count; e += (uint64_t)gridDim.x * kBlock)
        a.h[a.off[s] + (uint32_t)e] = haf_ladder_value(L, a.d, P, s, loops, h1, h2, (uint32_t)e);
}

__global__ __launch_bounds__(kBlock) void haf_ladder_gather_kernel(const HafLadderArgs a) {
    extern __shared__ double mem[];
    uint32_t* G = (uint32_t*)mem;
    const int P = ladder_stride(a.d);
    if (threadIdx.x < 64) ladder_table(a.d, a.N, P, (int)threadIdx.x, G);
    __syncthreads();
    const int p = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (p < a.npat) haf_ladder_read(a, G, P, p);
}

static bool haf_ladder_ok(const HafLadderArgs& a) {
    return a.d >= 1 && a.d <= kHafLadderModes && a.N >= 1 && a.N <= kHafMaxN && a.npat >= 1;
}

hipError_t launch_haf_ladder_small(const HafLadderArgs& a, hipStream_t s) {
    if (!haf_ladder_ok(a) || a.s0 < 0 || a.s0 > a.N) return hipErrorInvalidValue;
    hipLaunchKernelGGL(haf_ladder_small_kernel, dim3(1), dim3(kHafLadderBlock), haf_ladder_lds(a.d, a.s0), s, a);
    return hipGetLastError();
}

hipError_t launch_haf_ladder_level(const HafLadderArgs& a, int level, hipStream_t s) {
    if (!haf_ladder_ok(a) || level < 2 || level > a.N) return hipErrorInvalidValue;
    const uint32_t count = a.off[level + 1] - a.off[level];
    const uint32_t blocks = (count + kBlock - 1) / kBlock;
    const unsigned grid = blocks < 4096 ? (blocks > 0 ? blocks : 1) : 4096;
    hipLaunchKernelGGL(haf_ladder_level_kernel, dim3(grid), dim3(kBlock), haf_ladder_lds(a.d, level), s, a, level);
    return hipGetLastError();
}

hipError_t launch_haf_ladder_gather(const HafLadderArgs& a, hipStream_t s) {
    if (!haf_ladder_ok(a)) return hipErrorInvalidValue;
    const size_t lds = sizeof(uint32_t) * (size_t)(a.N + 1) * (size_t)ladder_stride(a.d);
    hipLaunchKernelGGL(haf_ladder_gather_kernel, dim3((unsigned)((a.npat + kBlock - 1) / kBlock)), dim3(kBlock), lds, s, a);
    return hipGetLastError();
}

}  // namespace pq
