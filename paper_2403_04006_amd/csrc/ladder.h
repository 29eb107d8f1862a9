// Ranks of photon vectors, shared by the kernels that build a level of
// photon-number vectors from the levels below (all outputs, hafnian tables).
// The vectors of k photons in m modes are in ascending lexicographic order of
// (T_0, ..., T_{m-1}); a vector is its photons' modes in ascending order, q the
// mode counted from the last, and rank(T) = sum_p G(k - p, q_p) over its
// photons p = 0..k-1.
#pragma once
#include <hip/hip_runtime.h>

#include "device.h"

namespace pq {

// The rank table (RankLane): 0 at q = 0 and no rank at all from q = m on.
constexpr uint32_t kNoRank = 0xffffffffu;

__host__ __device__ inline int ladder_stride(int m) {
    int p = 1;
    while (p < m) p *= 2;
    return p;
}

// G for at most n photons (kRankMaxPhotons at most) by one wavefront, without
// divisions or memory reads.
__device__ __forceinline__ void ladder_table(int m, int n, int P, int lane, uint32_t* G) {
    for (int e = lane; e < (n + 1) * P; e += 64) G[e] = (e & (P - 1)) == 0 ? 0u : kNoRank;
    RankLane x{0, 0};
    const int steps = rank_table_steps(m, n);
    for (int s = 0; s < steps; ++s) {
        const uint32_t left = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x.v, 0x138 /* wave_shr:1 */, 0xf, 0xf, true);
        rank_table_step(x, lane, left, s, m, n, P, G);
    }
}

// The mode of the next photon of an output, counted from the last mode: with
// rem photons left and the output at place `rank` among the ways to put them
// into the remaining modes, the largest q whose row entry does not exceed it.
// Every lane is at the same photon, so all search the same row.
__device__ __forceinline__ int ladder_mode(const uint32_t* row, int P, uint32_t rank) {
    int q = 0;
    for (int b = P >> 1; b; b >>= 1)
        if (row[q + b] <= rank) q += b;
    return q;
}

}  // namespace pq
