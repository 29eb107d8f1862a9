// Adding a vector that is the same for every lane to per-lane sums: the vector
// is held across the lanes (lane i of every 16 holds entries i and 16 + i) and
// enters each sum as a DPP operand, v_fmac_f64 with row_newbcast, at the rate of
// a plain fused multiply-add.  One LDS read per 16 entries instead of one per
// entry, and no scalar registers.
#pragma once
#include <hip/hip_runtime.h>

#include "device.h"

namespace pq {

// v[i0 + i] += s * (value i of the 16 held across the lanes), i = 0..N-1.  The
// leading s_nop separates a copy of the operands, which the compiler may place
// right before, from the first DPP read.
template <int I0, int N, int R>
__device__ __forceinline__ void add_lanes(cplx (&v)[R], const cplx& b, double s) {
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (N == 8) {
        asm("s_nop 1\n\t"
            "v_fmac_f64_dpp %0, %16, %18 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %1, %17, %18 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %2, %16, %18 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %3, %17, %18 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %4, %16, %18 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %5, %17, %18 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %6, %16, %18 row_newbcast:%22 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %7, %17, %18 row_newbcast:%22 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %8, %16, %18 row_newbcast:%23 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %9, %17, %18 row_newbcast:%23 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %10, %16, %18 row_newbcast:%24 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %11, %17, %18 row_newbcast:%24 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %12, %16, %18 row_newbcast:%25 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %13, %17, %18 row_newbcast:%25 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %14, %16, %18 row_newbcast:%26 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %15, %17, %18 row_newbcast:%26 row_mask:0xf bank_mask:0xf"
            : "+v"(v[I0].re), "+v"(v[I0].im), "+v"(v[I0 + 1].re), "+v"(v[I0 + 1].im), "+v"(v[I0 + 2].re),
              "+v"(v[I0 + 2].im), "+v"(v[I0 + 3].re), "+v"(v[I0 + 3].im), "+v"(v[I0 + 4].re), "+v"(v[I0 + 4].im),
              "+v"(v[I0 + 5].re), "+v"(v[I0 + 5].im), "+v"(v[I0 + 6].re), "+v"(v[I0 + 6].im), "+v"(v[I0 + 7].re),
              "+v"(v[I0 + 7].im)
            : "v"(b.re), "v"(b.im), "v"(s), "n"(I0 & 15), "n"((I0 + 1) & 15), "n"((I0 + 2) & 15), "n"((I0 + 3) & 15),
              "n"((I0 + 4) & 15), "n"((I0 + 5) & 15), "n"((I0 + 6) & 15), "n"((I0 + 7) & 15));
    } else if constexpr (N == 4) {
        asm("s_nop 1\n\t"
            "v_fmac_f64_dpp %0, %8, %10 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %1, %9, %10 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %2, %8, %10 row_newbcast:%12 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %3, %9, %10 row_newbcast:%12 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %4, %8, %10 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %5, %9, %10 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %6, %8, %10 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %7, %9, %10 row_newbcast:%14 row_mask:0xf bank_mask:0xf"
            : "+v"(v[I0].re), "+v"(v[I0].im), "+v"(v[I0 + 1].re), "+v"(v[I0 + 1].im), "+v"(v[I0 + 2].re),
              "+v"(v[I0 + 2].im), "+v"(v[I0 + 3].re), "+v"(v[I0 + 3].im)
            : "v"(b.re), "v"(b.im), "v"(s), "n"(I0 & 15), "n"((I0 + 1) & 15), "n"((I0 + 2) & 15), "n"((I0 + 3) & 15));
    } else {
        static_assert(N == 2, "rows come in eights, fours and twos");
        asm("s_nop 1\n\t"
            "v_fmac_f64_dpp %0, %4, %6 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %1, %5, %6 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %2, %4, %6 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f64_dpp %3, %5, %6 row_newbcast:%8 row_mask:0xf bank_mask:0xf"
            : "+v"(v[I0].re), "+v"(v[I0].im), "+v"(v[I0 + 1].re), "+v"(v[I0 + 1].im)
            : "v"(b.re), "v"(b.im), "v"(s), "n"(I0 & 15), "n"((I0 + 1) & 15));
    }
#else
    (void)v;
    (void)b;
    (void)s;
#endif
}

// A column's values across the lanes: lane i of every 16 holds rows i and
// 16 + i (the second part only when R > 16).
struct LaneColumn {
    cplx lo, hi;
};

template <int R>
__device__ __forceinline__ LaneColumn load_column(const cplx* col, int lane) {
    LaneColumn b;
    b.lo = col[lane & 15];
    if constexpr (R > 16) b.hi = col[16 + (lane & 15)];
    else b.hi = cplx{0.0, 0.0};
    return b;
}

template <int I0, int R>
__device__ __forceinline__ void add_from(cplx (&v)[R], const LaneColumn& b, double s) {
    if constexpr (I0 < R) {
        constexpr int N = R - I0 >= 8 ? 8 : (R - I0 >= 4 ? 4 : 2);
        add_lanes<I0, N>(v, I0 < 16 ? b.lo : b.hi, s);
        add_from<I0 + N>(v, b, s);
    }
}

// v += s * column; every lane of the wavefront has to be active.
template <int R>
__device__ __forceinline__ void add_column(cplx (&v)[R], const LaneColumn& b, double s) {
    static_assert(R % 2 == 0, "an even number of rows");
    add_from<0>(v, b, s);
}

template <int R>
__device__ __forceinline__ cplx row_product(const cplx (&v)[R]) {
    cplx p0 = v[0], p1 = v[1];
#pragma unroll
    for (int i = 2; i < R; i += 2) {
        p0 = cmul(p0, v[i]);
        p1 = cmul(p1, v[i + 1]);
    }
    return cmul(p0, p1);
}

}  // namespace pq
