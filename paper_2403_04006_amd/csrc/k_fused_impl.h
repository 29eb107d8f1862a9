// A short permanent in one launch: every workgroup gathers the compact matrix
// into LDS, its wavefronts sweep their shares of the time states, and the last
// workgroup to finish adds the workgroups' sums in order.  The three or four
// launches of the longer sweeps (gather, step tables, sweep, final sum) cost 4
// to 6 us each where the sweep itself takes as little.
//
// The row of a step is the same for every lane; it is read from LDS once per 16
// columns and added through DPP (lane_column.h).  Mixed radices need no step
// table: on the step to state t the digit that moves is the lowest whose
// counter does not wrap, upward when t divided by the radices up to it is even,
// and the digits below it stand at 0 or at their top, where their binomials are
// 1; so the weight follows from the product over the digits above, which lane k
// keeps for digit k.
//
// Bound by the host's part of a call up to about 16 photons (13 us for 6 photons in
// 12 modes, where the kernel takes 4); at 20 photons in 40 modes the two are level
// (16.4 us to submit a call, 16 to 16.6 for the kernel).  The kernel is bound by
// latency: the launch, one round of loads of U, a start-up of r rows' additions (as
// long as seven steps at 20 rows) and the ticket.
#pragma once
#include <hip/hip_runtime.h>

#include "device.h"
#include "kernels.h"
#include "lane_column.h"
#include "sweep_common.h"

namespace pq {

// NC: columns, padded to an even number (sums 1, rows 0).  MIX: mixed radices
// or powers; otherwise every digit binary and every power 1.
template <int NC, bool MIX>
__global__ __launch_bounds__(kBlock) void fused_kernel(const FusedArgs a) {
    constexpr int W = NC <= 16 ? 16 : 32;    // row stride in LDS
    extern __shared__ double lds[];
    __shared__ double sred[kWavesPerBlock][4];
    __shared__ int slast;
    cplx* rows = (cplx*)lds;                 // [r][W]
    const int tid = (int)threadIdx.x, lane = tid & 63;
    for (int e = tid; e < a.r * W; e += kBlock) {
        const int i = e / W, j = e - i * W;
        // (the padding by selects on the values: on the address, it would go
        // through scratch memory)
        const int out = a.transposed ? a.col_mode[j] : a.row_mode[i];
        const int in = a.transposed ? a.row_mode[i] : a.col_mode[j];
        const bool on = j < a.nc;
        const cplx u = a.U[on ? (size_t)out * (size_t)a.ldu + (size_t)in : 0];
        rows[e] = cplx{on ? u.re : 0.0, on ? u.im : 0.0};
    }
    __syncthreads();
    const uint32_t wave = wave_id_uniform();
    cplx acc{0.0, 0.0};
    if (wave < a.waves) {
        uint64_t start64, count64;
        split_range(a.time_states, a.waves, wave, start64, count64);
        const uint32_t start = (uint32_t)start64, count = (uint32_t)count64;
        cplx v[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) v[j] = cplx{j < a.nc ? 0.0 : 1.0, 0.0};
        double wl = lane < a.lane_states ? 1.0 : 0.0;
        int rest = lane;
        for (int i = 0; i < a.n_lane; ++i) {
            int d;
            if constexpr (MIX) {
                const int rho = a.radix[i];
                d = rest % rho;
                rest /= rho;
                wl *= digit_weight(rho, d);
            } else {
                d = rest & 1;
                rest >>= 1;
                if (d) wl = -wl;
            }
            add_column(v, load_column<NC>(rows + i * W, lane), (double)(a.row_mu[i] - 2 * d));
        }
        for (int i = a.n_lane + a.n_time; i < a.r; ++i) add_column(v, load_column<NC>(rows + i * W, lane), (double)a.row_mu[i]);
        const cplx* trows = rows + a.n_lane * W;
        // lane k: digit k's value and the product of the binomials of the
        // digits from k on
        int myg = 0;
        double myw = 1.0, w = 1.0;
        if constexpr (MIX) {
            gray_digits_desc(a.n_time, [&](int k) { return (int)a.radix[a.n_lane + k]; }, start, 0, [&](int k, int g) {
                w *= binom_d(a.radix[a.n_lane + k] - 1, g);
                if (lane == k) {
                    myg = g;
                    myw = w;
                }
                add_column(v, load_column<NC>(trows + k * W, lane), (double)(a.row_mu[a.n_lane + k] - 2 * g));
            });
        } else {
            const uint32_t g = start ^ (start >> 1);
            for (int k = 0; k < a.n_time; ++k)
                add_column(v, load_column<NC>(trows + k * W, lane), (g >> k) & 1u ? -1.0 : 1.0);
        }
        // the sign of a term is the parity of its state's rank (every step
        // moves one digit by one)
        if (start & 1u) w = -w;
        const uint32_t end = start + count;
        for (uint32_t t = start + 1; t < end; ++t) {
            int k;
            bool down;
            if constexpr (MIX) {
                uint32_t x = t;
                k = 0;
                for (;;) {
                    const uint32_t rk = (uint32_t)a.radix[a.n_lane + k], q = x / rk;
                    const uint32_t rem = x - q * rk;
                    x = q;
                    if (rem) break;
                    ++k;
                }
                k = uniform_int(k);
                down = uniform_int((int)(x & 1u)) != 0;
            } else {
                k = __builtin_ctz(t);
                down = (t >> (k + 1)) & 1u;
            }
            const LaneColumn b = load_column<NC>(trows + k * W, lane);
            if constexpr (MIX) cfma_to(acc, w, product_grouped(v, a.pw));
            else cfma_to(acc, w, row_product(v));
            add_column(v, b, down ? 2.0 : -2.0);
            if constexpr (MIX) {
                const int g = __builtin_amdgcn_readlane(myg, k) + (down ? -1 : 1);
                const double above = k + 1 < a.n_time
                    ? __longlong_as_double(((long long)__builtin_amdgcn_readlane((int)(__double_as_longlong(myw) >> 32), k + 1) << 32) |
                                           (unsigned)__builtin_amdgcn_readlane((int)__double_as_longlong(myw), k + 1))
                    : 1.0;
                const double nw = above * binom_d(a.radix[a.n_lane + k] - 1, g);
                if (lane <= k) myw = nw;
                if (lane == k) myg = g;
                w = t & 1u ? -nw : nw;
            } else {
                w = -w;
            }
        }
        if constexpr (MIX) cfma_to(acc, w, product_grouped(v, a.pw));
        else cfma_to(acc, w, row_product(v));
        acc.re *= wl;
        acc.im *= wl;
    }
    cdd s = wave_reduce(to_cdd(acc));
    if (lane == 0) {
        double* o = sred[tid >> 6];
        o[0] = s.re.hi;
        o[1] = s.re.lo;
        o[2] = s.im.hi;
        o[3] = s.im.lo;
    }
    __syncthreads();
    s = cdd{{sred[0][0], sred[0][1]}, {sred[0][2], sred[0][3]}};
    for (int x = 1; x < kWavesPerBlock; ++x) s = cdd_add(s, cdd{{sred[x][0], sred[x][1]}, {sred[x][2], sred[x][3]}});
    if (gridDim.x > 1) {
        // every workgroup's sum, then its ticket; the last one sees them all.
        // Consecutive calls take turns through the counters, and the last
        // workgroup clears its own and the one two turns on: even two calls
        // racing against the rules leave nothing behind for later ones.
        if (tid == 0) {
            double* o = a.partials + 4 * (size_t)blockIdx.x;
            __hip_atomic_store(o, s.re.hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(o + 1, s.re.lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(o + 2, s.im.hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(o + 3, s.im.lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            const uint32_t got = __hip_atomic_fetch_add(a.tickets + a.turn, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            slast = got + 1 == gridDim.x;
        }
        __syncthreads();
        if (!slast) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        s = cdd{{0.0, 0.0}, {0.0, 0.0}};
        for (uint32_t b = (uint32_t)tid; b < gridDim.x; b += kBlock) {
            const double* o = a.partials + 4 * (size_t)b;
            cdd x;
            x.re.hi = __hip_atomic_load(o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            x.re.lo = __hip_atomic_load(o + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            x.im.hi = __hip_atomic_load(o + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            x.im.lo = __hip_atomic_load(o + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s = cdd_add(s, x);
        }
        s = wave_reduce(s);
        __syncthreads();
        if (lane == 0) {
            double* o = sred[tid >> 6];
            o[0] = s.re.hi;
            o[1] = s.re.lo;
            o[2] = s.im.hi;
            o[3] = s.im.lo;
        }
        __syncthreads();
        s = cdd{{sred[0][0], sred[0][1]}, {sred[0][2], sred[0][3]}};
        for (int x = 1; x < kWavesPerBlock; ++x) s = cdd_add(s, cdd{{sred[x][0], sred[x][1]}, {sred[x][2], sred[x][3]}});
        if (tid < 2) __hip_atomic_store(a.tickets + (a.turn + 2 * tid) % kTickets, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (tid == 0) {
        const double re = (s.re.hi + s.re.lo) * a.scale;
        const double im = (s.im.hi + s.im.lo) * a.scale;
        if (a.perm) a.perm[0] = cplx{re, im};
        if (a.amp) a.amp[0] = cplx{re * a.norm, im * a.norm};
    }
}

template <int NC>
hipError_t launch_fused_nc(bool mix, const FusedArgs& a, int grid, hipStream_t s) {
    const size_t lds = sizeof(cplx) * (size_t)a.r * (NC <= 16 ? 16 : 32);
    if (mix) {
        hipLaunchKernelGGL((fused_kernel<NC, true>), dim3(grid), dim3(kBlock), lds, s, a);
    } else {
        // (collision-free patterns go by pairs of columns from there on)
        if constexpr (NC < kPairMinCols) hipLaunchKernelGGL((fused_kernel<NC, false>), dim3(grid), dim3(kBlock), lds, s, a);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

#define PQ_FINST(NC) \
    hipError_t launch_fused_##NC(bool mix, const FusedArgs& a, int grid, hipStream_t s) { return launch_fused_nc<NC>(mix, a, grid, s); }

}  // namespace pq
