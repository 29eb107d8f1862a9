// EXTEND_ROW jobs whose columns all have multiplicity 1, swept over the signs
// of the columns instead of the rows: with k columns c_j and the drawn rows i
// (multiplicity t_i),
//   perm(U_{T + e_l, S}) = sum_j U[l, c_j] M_j,
//   M_j = 2^{-(k-1)} sum_delta (prod delta) delta_j prod_i v_i(delta)^{t_i},
//   v_i = sum_j delta_j U[i, c_j].
// A term is one product, where the row form needs the leave-one-out products of
// all columns (three complex products a column, on half as many terms), and the
// M_j follow from the running sum P of the terms: delta_j is a lane's sign, or
// constant over the chunk, or moves with one of the chunk's digits, for which
//   sum_t delta_j(t) g(t) = delta_j(end) P(end) + sum_flips 2 dd P(before).
// A chunk is an aligned run of 2^q time states (q <= kExtColDigits), one
// wavefront each; its slot holds every column's double-double sum.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "k_batch_impl.h"
#include "many.h"

namespace pq {

// Double-double sums over the 64 lanes of N (a power of two) values per lane
// by recursive halving, in a fixed order: lane l ends with value
// l / (64 / N) in x[0].
template <int N, int M = 32>
__device__ __forceinline__ void extcol_halve(cdd* x, int lane) {
    if constexpr (M >= 1) {
        constexpr int H = N > 1 ? N / 2 : 1;
        const bool up = (lane & M) != 0;
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const cdd keep = N > 1 && up ? x[i + (N > 1 ? H : 0)] : x[i];
            const cdd give = N > 1 && !up ? x[i + (N > 1 ? H : 0)] : x[i];
            cdd o;
            o.re.hi = shfl_xor_d(give.re.hi, M);
            o.re.lo = shfl_xor_d(give.re.lo, M);
            o.im.hi = shfl_xor_d(give.im.hi, M);
            o.im.lo = shfl_xor_d(give.im.lo, M);
            x[i] = cdd_add(keep, o);
        }
        extcol_halve<H, M / 2>(x, lane);
    }
}

// Bound by FP64 vector instructions (2 adds a row, 4 a product factor, 4 for
// the sums per term and lane); rows come through scalar loads as in the forward
// sweep.
template <int NC, bool UNIT>
__global__ __launch_bounds__(64, NC <= 12 ? 4 : (NC <= 20 ? 3 : 2)) void extcol_kernel(const ManyArgs a) {
    constexpr int T = kExtColDigits;
    static_assert(T >= 3, "blocks of eight states");
    const int lane = threadIdx.x & 63;
    const int ci = (int)blockIdx.x;
    if (ci >= a.nchunks) return;
    if (a.cancel && ci >= a.poll_from) {
        if (ci % kExtColPollEvery == 0) {
            if (cancel_requested(a.cancel, lane)) {
                if (lane == 0) __hip_atomic_store(a.stop, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return;
            }
        } else {
            unsigned stop = 0;
            if (lane == 0) stop = __hip_atomic_load(a.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (__builtin_amdgcn_readfirstlane((int)stop)) return;
        }
    }
    typedef const __attribute__((address_space(4))) MChunk kchunk;
    kchunk& ch = *(kchunk*)(a.chunks + ci);
    // the descriptor and the rows are written by earlier work only: through the
    // constant address space, so they stay in scalar registers
    kjob& J = *(kjob*)(a.jobs + ch.pat);
    PowSteps pw;
    for (int k = 0; k < 3; ++k) {
        const uint64_t v = J.pw.step[k];
        pw.step[k] = ((uint64_t)(uint32_t)uniform_int((int)(v >> 32)) << 32) | (uint32_t)uniform_int((int)v);
    }
    pw.low = uniform_int(J.pw.low);
    pw.general = 0;
    const cplx* mat = a.mat + J.mat_off;
    const cplx* rows2 = mat + (size_t)J.r * NC;
    const cplx* base = rows2 + (size_t)J.r * 2 * NC;
    const cplx* trows = rows2 + (size_t)J.n_lane * 2 * NC;
    const int nt = J.n_time, q = __builtin_ctzll(ch.count);   // whole powers of two
    const uint64_t start = ch.start;
    cplx c[NC];
    const double wl = lane_init_at<NC, true>(base, rows2, J.n_lane, J.lane_states, J.lane_radix, lane, c);
    const uint64_t g0 = start ^ (start >> 1);
    for (int k = 0; k < nt; ++k)
        if ((g0 >> k) & 1ull) add_row_at<NC, true>(c, trows, (size_t)k * 2 * NC);
    const double w0 = (__builtin_popcountll(g0) & 1) ? -wl : wl;   // weight of the first state, this lane's
    cplx P{0.0, 0.0};
    cplx A[T];
#pragma unroll
    for (int i = 0; i < T; ++i) A[i] = cplx{0.0, 0.0};
    auto term = [&]() -> cplx {
        if constexpr (UNIT) return product_unit_powers(c);
        else return product_grouped(c, pw);
    };
    // the term of the current state, then the flip of digit Q on the step to
    // state t (sel 0: the digit rises, delta from +1 to -1)
    auto step = [&](auto qc, double sign, int sel) {
        constexpr int Q = decltype(qc)::value;
        cfma_to(P, sign, term());
        cfma_to(A[Q], sel ? -2.0 : 2.0, P);
        // the row is loaded anew on every step: kept for the digit's next flip
        // it would spill (40 doubles a row), two moves a value
        const cplx* tr = trows;
#if defined(__HIP_DEVICE_COMPILE__)
        asm("" : "+s"(tr));
#endif
        add_row_at<NC, true>(c, tr, ((size_t)Q * 2 + sel) * NC);
    };
    using std::integral_constant;
    if (q >= 3) {
        const int blocks = 1 << (q - 3);
#pragma unroll 1
        for (int b = 0; b < blocks; ++b) {
            const uint64_t t = start + 8 * (uint64_t)b;
            step(integral_constant<int, 0>{}, 1.0, 0);
            step(integral_constant<int, 1>{}, -1.0, 0);
            step(integral_constant<int, 0>{}, 1.0, 1);
            step(integral_constant<int, 2>{}, -1.0, (int)((t >> 3) & 1u));
            step(integral_constant<int, 0>{}, 1.0, 0);
            step(integral_constant<int, 1>{}, -1.0, 1);
            step(integral_constant<int, 0>{}, 1.0, 1);
            cfma_to(P, -1.0, term());
            if (b + 1 < blocks) {
                const int i = 3 + __builtin_ctz(b + 1);
                const int sel = (int)(((t + 8) >> (i + 1)) & 1u);
                flip_sums<3, T>(A, i, sel ? -2.0 : 2.0, P);
                add_row_at<NC, true>(c, trows, ((size_t)i * 2 + sel) * NC);
            }
        }
    } else {
        const int states = 1 << q;
#pragma unroll 1
        for (int t = 1; t < states; ++t) {
            if (t & 1) step(integral_constant<int, 0>{}, 1.0, (t >> 1) & 1);
            else step(integral_constant<int, 1>{}, -1.0, 0);
        }
        cfma_to(P, q > 0 ? -1.0 : 1.0, term());
    }
    const uint64_t end = start + ch.count - 1, ge = end ^ (end >> 1);
    P = cplx{w0 * P.re, w0 * P.im};
    cdd x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        cplx v{0.0, 0.0};
        if (i == 0) {
            v = P;
        } else if (i <= 6) {
            const double s = (lane >> (i - 1)) & 1 ? -1.0 : 1.0;
            v = cplx{s * P.re, s * P.im};
        } else if (i - 7 < T) {
            const double d = (ge >> (i - 7)) & 1u ? -1.0 : 1.0;
            v.re = __builtin_fma(w0, A[i - 7].re, d * P.re);
            v.im = __builtin_fma(w0, A[i - 7].im, d * P.im);
        }
        x[i] = to_cdd(v);
    }
    static_assert(7 + T <= 16, "sums per lane");
    extcol_halve<16>(x, lane);
    // lane 4 v holds sum v: 0 the terms, 1..6 the lane columns, 7.. the digits;
    // columns that are constant over the chunk take +-sum 0
    __shared__ double sx[16][4];
    if ((lane & 3) == 0) {
        double* o = sx[lane >> 2];
        o[0] = x[0].re.hi;
        o[1] = x[0].re.lo;
        o[2] = x[0].im.hi;
        o[3] = x[0].im.lo;
    }
    __syncthreads();
    double* slot = a.partials + (size_t)ch.slot * a.slot_doubles;
    for (int e = lane; e < 4 * J.r; e += 64) {
        const int i = e >> 2, k = i - J.n_lane;   // iterated column: lane digits, time digits, the fixed one
        double v;
        if (k < 0) v = sx[1 + i][e & 3];
        else if (k < q) v = sx[7 + k][e & 3];
        else v = k < nt && ((ge >> k) & 1u) ? -sx[0][e & 3] : sx[0][e & 3];
        slot[e] = v;
    }
}

template <int NC>
hipError_t launch_extcol(int var, const ManyArgs& a, hipStream_t s) {
    const dim3 grid(a.nchunks > 0 ? a.nchunks : 1), block(64);
    // (the classes that either variant has, PQ_XCLASS)
    if (var & 1) {
        if constexpr (NC >= 12) hipLaunchKernelGGL((extcol_kernel<NC, true>), grid, block, 0, s, a);
        else return hipErrorInvalidValue;
    } else {
        if constexpr (NC <= 12) hipLaunchKernelGGL((extcol_kernel<NC, false>), grid, block, 0, s, a);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

#define PQ_XINST(NC) \
    hipError_t launch_extcol_##NC(int var, const ManyArgs& a, hipStream_t s) { return launch_extcol<NC>(var, a, s); }

}  // namespace pq
