// Set-up kernels of a job list: gather of every job's compact matrix, and the
// inner-digit step tables.
#include <hip/hip_runtime.h>

#include "batch.h"
#include "batch_kernels.h"
#include "device.h"

namespace pq {

// One workgroup per job: B[i][j] (padded columns: 0), rows2 = (-2B, +2B),
// base_j = sum_i mu_i B_ij (padded columns: 1, so they leave products alone).
__device__ __forceinline__ void prep_job(const BPrepArgs& a, const BJob& J) {
    if (J.nchunks == 0) return;
    const int W = J.ncmax;
    cplx* B = a.mat + J.mat_off;
    cplx* rows2 = B + (size_t)J.r * W;
    cplx* base = rows2 + (size_t)J.r * 2 * W;
    const int32_t* rmode = a.idx + J.idx_off;
    const int32_t* rmu = rmode + J.r;
    const int32_t* cmode = rmu + J.r;
    for (int e = threadIdx.x; e < J.r * W; e += blockDim.x) {
        const int i = e / W, j = e % W;
        cplx v{0.0, 0.0};
        if (j < J.nc) {
            const int out = J.transposed ? cmode[j] : rmode[i];
            const int in = J.transposed ? rmode[i] : cmode[j];
            v = a.U[(size_t)out * (size_t)a.ldu + (size_t)in];
        }
        B[(size_t)i * W + j] = v;
        rows2[((size_t)i * 2 + 0) * W + j] = cplx{-2.0 * v.re, -2.0 * v.im};
        rows2[((size_t)i * 2 + 1) * W + j] = cplx{2.0 * v.re, 2.0 * v.im};
    }
    for (int j = threadIdx.x; j < W; j += blockDim.x) {
        if (j >= J.nc) {
            base[j] = cplx{1.0, 0.0};
            continue;
        }
        double re = 0.0, im = 0.0;
#pragma unroll 8
        for (int i = 0; i < J.r; ++i) {
            const int out = J.transposed ? cmode[j] : rmode[i];
            const int in = J.transposed ? rmode[i] : cmode[j];
            const cplx v = a.U[(size_t)out * (size_t)a.ldu + (size_t)in];
            re = __builtin_fma((double)rmu[i], v.re, re);
            im = __builtin_fma((double)rmu[i], v.im, im);
        }
        base[j] = cplx{re, im};
    }
}

// The same for the jobs swept over column signs (ext_cols), whose iterated rows i
// are columns of U, each of multiplicity 1.  Their sweep sums over the columns,
// and a column far larger than the others would drown them: its leave-one-out sum
// does not hold its values at all, but every term does (one column of 16 ten times
// as large cost six digits).  Each column is therefore scaled by a power of two to
// a largest entry in [1, 2).  What undoes it (the exponents of the other columns,
// which enter once each; and whether one of them is zero in these rows, which makes
// the sum zero where its terms would leave their rounding) is put in the place of
// B, which that sweep does not read.
//
// One wavefront a job, lane (h, j) its iterated rows h, h + 2, ... of column j: every
// load in flight at once and no barrier.  13,000 jobs of up to 14 photons take 21.0 us
// (a workgroup a job 44, and 21.6 without the scales).
__device__ __forceinline__ void prep_ext_job(const BPrepArgs& a, const BJob& J) {
    constexpr int N = kMaxExtendCols / 2;
    static_assert(kMaxExtendCols <= 32, "a column a lane");
    const int lane = (int)threadIdx.x & 63, h = lane >> 5, j = lane & 31;
    const int W = J.ncmax, r = J.r;
    cplx* scales = a.mat + J.mat_off;
    cplx* rows2 = scales + (size_t)r * W;
    cplx* base = rows2 + (size_t)r * 2 * W;
    const int32_t* col = a.idx + J.idx_off;
    const bool on = j < J.nc;
    const cplx* row = a.U + (size_t)(on ? col[2 * r + j] : 0) * (size_t)a.ldu;
    cplx v[N];
#pragma unroll
    for (int x = 0; x < N; ++x) {
        const int i = 2 * x + h;
        v[x] = on && i < r ? row[col[i]] : cplx{0.0, 0.0};
    }
    int mine = 0, sum = 0, zeros = 0;
    bool zero = false, finite = true;
    cplx s{0.0, 0.0};
#pragma unroll
    for (int x = 0; x < N; ++x) {
        if (2 * x >= r) continue;
        const int i = 2 * x + h;
        // the moduli's upper halves, ordered as they are (1: not zero, but nothing
        // above the lower half)
        auto key = [](double y) {
            const unsigned long long b = (unsigned long long)__double_as_longlong(fabs(y));
            return (int)(b >> 32) | ((int)(b >> 32) == 0 && b != 0 ? 1 : 0);
        };
        int top = max(key(v[x].re), key(v[x].im));
#pragma unroll
        for (int m = 16; m >= 1; m >>= 1) top = max(top, __shfl_xor(top, m, 64));
        const int b = top >> 20;
        const int e = b == 0 || b >= 0x7ff ? 0 : b - 1023;   // zero, tiny or not finite: as it is
        finite = finite && b < 0x7ff;
        if (j == x) {
            mine = e;
            zero = top == 0;
        }
        sum += e;
        zeros += i < r && top == 0;
        const cplx d{ldexp(v[x].re, 1 - e), ldexp(v[x].im, 1 - e)};
        cadd_to(s, d);
        if (i < r && j < W) {
            rows2[((size_t)i * 2 + 0) * W + j] = cplx{-d.re, -d.im};
            rows2[((size_t)i * 2 + 1) * W + j] = d;
        }
    }
    sum += __shfl_xor(sum, 32, 64);
    zeros += __shfl_xor(zeros, 32, 64);
    finite = __all(finite);
    s.re += shfl_xor_d(s.re, 32);
    s.im += shfl_xor_d(s.im, 32);
    if (h == 0 && j < W) base[j] = on ? cplx{0.5 * s.re, 0.5 * s.im} : cplx{1.0, 0.0};
    if (2 * j + h < r) scales[2 * j + h] = cplx{(double)(sum - mine), finite && zeros > (zero ? 1 : 0) ? 1.0 : 0.0};
}

// EXT: some jobs are swept over column signs.  The others' workgroups come first,
// by the list of them, then one for every four jobs.
template <bool EXT>
__global__ __launch_bounds__(kBlock) void bprep_kernel(const BPrepArgs a) {
    const int b = (int)blockIdx.x;
    if constexpr (EXT) {
        if (b >= a.nlist) {
            const int jb = __builtin_amdgcn_readfirstlane((b - a.nlist) * kWavesPerBlock + (int)(threadIdx.x >> 6));
            if (jb >= a.njobs) return;
            const BJob& J = a.jobs[jb];
            if (J.nchunks > 0 && J.ext_cols) prep_ext_job(a, J);
            return;
        }
        prep_job(a, a.jobs[a.list[b]]);
    } else if (b < a.njobs) {
        prep_job(a, a.jobs[b]);
    }
}

hipError_t launch_bprep(const BPrepArgs& a, hipStream_t s) {
    if (a.njobs < 1) return hipSuccess;
    if (a.list) {
        const int n = a.nlist + (a.njobs + kWavesPerBlock - 1) / kWavesPerBlock;
        hipLaunchKernelGGL(bprep_kernel<true>, dim3((unsigned)n), dim3(kBlock), 0, s, a);
    } else {
        hipLaunchKernelGGL(bprep_kernel<false>, dim3((unsigned)a.njobs), dim3(kBlock), 0, s, a);
    }
    return hipGetLastError();
}

// Same construction as the single-permanent table kernel, for every signature
// (n_inner, m_inner, ncmax, radices): forward entries at tabs + t*2*kMaxInner,
// reflected entries kMaxInner further.
__global__ __launch_bounds__(kBlock) void btable_kernel(const BTableArgs a) {
    const int t = blockIdx.y;
    if (t >= a.ntab) return;
    const int32_t* sg = a.sig + (size_t)t * kSigInts;
    const int n_inner = sg[0], M = sg[1], nc = sg[2];
    StepEntry* tf = a.tabs + (size_t)t * 2 * kMaxInner;
    StepEntry* tb = tf + kMaxInner;
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < M; q += gridDim.x * blockDim.x) {
        const GrayStep e = gray_step(n_inner, [&](int k) { return sg[3 + k]; }, M, q);
        tf[q] = StepEntry{q > 0 ? (2 * e.fwd + (e.fwd_up ? 0 : 1)) * nc : 0, 0, e.w};
        tb[M - 1 - q] = StepEntry{q < M - 1 ? (2 * e.bwd + (e.bwd_up ? 0 : 1)) * nc : 0, 0, e.w};
    }
}

hipError_t launch_btable(const BTableArgs& a, hipStream_t s) {
    if (a.ntab <= 0) return hipSuccess;
    hipLaunchKernelGGL(btable_kernel, dim3(kMaxInner / kBlock, a.ntab), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

}  // namespace pq
