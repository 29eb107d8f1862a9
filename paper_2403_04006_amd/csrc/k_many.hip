// Reduction and scatter kernels of the many-pattern entry points, and the
// class dispatch.
#include <hip/hip_runtime.h>

#include "device.h"
#include "many_kernels.h"

namespace pq {

// Final step of distinct pattern p, run by one whole wavefront (t = lane):
// add its chunk slots in slot order and write the value to every copy's
// output.  L and C are LDS scratch of kMaxExtendCols entries (extend-row jobs).
__device__ __forceinline__ void final_pattern(const ManyFinalArgs& a, int p, int t, cplx* L, int* C) {
    const int cls = a.pat_class[p];
    const int q0 = a.dup_off[p], q1 = a.dup_off[p + 1];
    if (a.adjoint && t == 0) {
        // the copies' cotangents, summed in pattern order
        double re = 0.0, im = 0.0;
        for (int q = q0; q < q1; ++q) {
            const cplx g = a.gperm[a.dup_pat[q]];
            re += g.re;
            im += g.im;
        }
        a.gsum[p] = cplx{re, im};
    }
    if (cls < 0) {
        for (int q = q0 + t; q < q1; q += 64) {
            if (a.perm) a.perm[a.dup_out[q]] = a.trivial[p];
            if (a.amp) a.amp[a.dup_out[q]] = a.trivial[p];
        }
        return;
    }
    const BJob& J = a.jobs[p];
    const int sd = a.class_sd[cls];
    const double* base = a.partials + a.class_off[cls] + (size_t)a.pat_slot[p] * sd;
    if (J.op == kOpPerm) {
        // thread t adds slots t, t + 64, ... in order, then a fixed butterfly
        cdd s{{0.0, 0.0}, {0.0, 0.0}};
#pragma unroll 8
        for (int k = t; k < J.nchunks; k += 64) {
            const double* q = base + (size_t)k * sd;
            s = cdd_add(s, cdd{{q[0], q[1]}, {q[2], q[3]}});
        }
        s = wave_reduce(s);
        // lane 0's sum, for every lane
        const double rh = __shfl(s.re.hi, 0, 64), rl = __shfl(s.re.lo, 0, 64);
        const double ih = __shfl(s.im.hi, 0, 64), il = __shfl(s.im.lo, 0, 64);
        const double re = (rh + rl) * J.scale;
        const double im = (ih + il) * J.scale;
        for (int q = q0 + t; q < q1; q += 64) {
            if (a.perm) a.perm[a.dup_out[q]] = cplx{re, im};
            if (a.amp) a.amp[a.dup_out[q]] = cplx{re * J.norm, im * J.norm};
        }
        if (a.adjoint && J.nchunks <= a.fuse_dred) {
            // derivative part of the slots: entry e adds its chunks in order
            // (the same sums as the two reduction stages)
            const int nent = J.r * J.nc;
            for (int e = t; e < nent; e += 64) {
                double dre = 0.0, dim = 0.0;
#pragma unroll 8
                for (int k = 0; k < J.nchunks; ++k) {
                    dre += base[(size_t)k * sd + 4 + 2 * e];
                    dim += base[(size_t)k * sd + 4 + 2 * e + 1];
                }
                a.dpat[a.dpat_off[p] + e] = cplx{dre * J.scale, dim * J.scale};
            }
        }
        // (otherwise the derivative part of the slots is the stage-1 items')
    } else {
        // Laplace expansion: L_j from the chunk sums, then out[l] = sum_j U[l, C_j] L_j;
        // a sweep over the columns' signs has the columns on its iterated side
        const int ncol = J.ext_cols ? J.r : J.nc;
        // lane (g, j) adds slots g, g + G, ... of column j in order; the G groups
        // of a column are then added in order
        const int G = 64 / ncol, g = t / ncol, jj = t - g * ncol;
        if (t < ncol) {
            // the column, or its row among the transposed ones
            const int c = a.idx[J.idx_off + (J.ext_cols ? 0 : 2 * J.r) + t];
            C[t] = a.UT ? a.ut_at[c] : c;
        }
        // the other columns' scales (prep_ext_job)
        const cplx others = J.ext_cols && t < ncol ? a.mat[J.mat_off + t] : cplx{0.0, 0.0};
        cdd s{{0.0, 0.0}, {0.0, 0.0}};
        if (g < G)
            for (int k = g; k < J.nchunks; k += G) {
                const double* q = base + (size_t)k * sd + 4 * jj;
                s = cdd_add(s, cdd{{q[0], q[1]}, {q[2], q[3]}});
            }
        for (int h = 1; h < G; ++h) {
            const int from = h * ncol + jj;
            const cdd o{{__shfl(s.re.hi, from, 64), __shfl(s.re.lo, from, 64)},
                        {__shfl(s.im.hi, from, 64), __shfl(s.im.lo, from, 64)}};
            if (g == 0) s = cdd_add(s, o);
        }
        if (t < ncol) {
            const int e = (int)others.re;
            const cplx v{(s.re.hi + s.re.lo) * J.scale, (s.im.hi + s.im.lo) * J.scale};
            L[t] = others.im != 0.0 ? cplx{0.0, 0.0} : cplx{ldexp(v.re, e), ldexp(v.im, e)};
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        for (int l = t; l < J.m_out; l += 64) {
            const cplx* Ul = a.U + (size_t)l * (size_t)a.ldu;
            double re = 0.0, im = 0.0;
            for (int j = 0; j < ncol; ++j) {
                const cplx u = a.UT ? a.UT[(size_t)C[j] * (size_t)a.m + l] : Ul[C[j]];
                re = __builtin_fma(u.re, L[j].re, re);
                re = __builtin_fma(-u.im, L[j].im, re);
                im = __builtin_fma(u.re, L[j].im, im);
                im = __builtin_fma(u.im, L[j].re, im);
            }
            if (a.perm)
                for (int q = q0; q < q1; ++q) a.perm[a.dup_out[q] + l] = cplx{re, im};
        }
    }
    // L is reused by the next call on this wavefront
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Stage-1 item of the derivative reduction (see DRedItem).  Bound by the
// latency of its strided reads: with 16 of them in flight, and beside the
// patterns' values instead of after them, one 23-photon pattern's reductions
// (18 MB of slots) take 14 us in two launches, 48 in three before.
__device__ __forceinline__ void reduce_slots(const ManyFinalArgs& a, const DRedItem& it, int t) {
    const BJob& J = a.jobs[it.pat];
    const int nent = J.r * J.nc;
    const int e = it.eb * 64 + t;
    if (e >= nent) return;
    const int cls = a.pat_class[it.pat];
    const int sd = a.class_sd[cls];
    const double* base = a.partials + a.class_off[cls] + (size_t)a.pat_slot[it.pat] * sd + 4 + 2 * e;
    const int k0 = it.cb * 64;
    const int k1 = J.nchunks < k0 + 64 ? J.nchunks : k0 + 64;
    double re = 0.0, im = 0.0;
#pragma unroll 16
    for (int k = k0; k < k1; ++k) {
        re += base[(size_t)k * sd];
        im += base[(size_t)k * sd + 1];
    }
    if (it.ncb == 1) a.dpat[a.dpat_off[it.pat] + e] = cplx{re * J.scale, im * J.scale};
    else a.red_part[it.part_off + (int64_t)it.cb * nent + e] = cplx{re, im};
}

// One workgroup per distinct pattern, then one per stage-1 item.
__global__ __launch_bounds__(64) void many_final_kernel(const ManyFinalArgs a) {
    __shared__ cplx L[kMaxExtendCols];
    __shared__ int C[kMaxExtendCols];
    const int p = blockIdx.x;
    if (p < a.npat) final_pattern(a, p, (int)threadIdx.x, L, C);
    else if (p - a.npat < a.nred) reduce_slots(a, a.red[p - a.npat], (int)threadIdx.x);
}

__global__ __launch_bounds__(64) void dred_kernel(const DRedArgs a) {
    const DRedItem it = a.items[blockIdx.x];
    const BJob& J = a.jobs[it.pat];
    const int nent = J.r * J.nc;
    const int e = it.eb * 64 + (int)threadIdx.x;
    if (e >= nent) return;
    double re = 0.0, im = 0.0;
#pragma unroll 8
    for (int cb = 0; cb < it.ncb; ++cb) {
        const cplx v = a.part[it.part_off + (int64_t)cb * nent + e];
        re += v.re;
        im += v.im;
    }
    a.dpat[a.dpat_off[it.pat] + e] = cplx{re * J.scale, im * J.scale};
}

hipError_t launch_dred(const DRedArgs& a, int nitems, hipStream_t s) {
    if (nitems <= 0) return hipSuccess;
    hipLaunchKernelGGL(dred_kernel, dim3(nitems), dim3(64), 0, s, a);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void transpose_kernel(const TransposeArgs a) {
    __shared__ cplx tile[16][17];
    const int x = threadIdx.x & 15, y = threadIdx.x >> 4;
    const int r = blockIdx.x * 16 + y, c = blockIdx.y * 16 + x;
    if (r < a.m && c < a.n) tile[y][x] = a.U[(size_t)r * (size_t)a.ldu + (size_t)a.col[c]];
    __syncthreads();
    const int tr = blockIdx.y * 16 + y, tc = blockIdx.x * 16 + x;
    if (tr < a.n && tc < a.m) a.UT[(size_t)tr * (size_t)a.m + tc] = tile[x][y];
}

hipError_t launch_transpose(const TransposeArgs& a, hipStream_t s) {
    if (a.m < 1 || a.n < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(transpose_kernel, dim3((unsigned)((a.m + 15) / 16), (unsigned)((a.n + 15) / 16)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_many_final(const ManyFinalArgs& a, hipStream_t s) {
    const int n = a.npat + a.nred;
    hipLaunchKernelGGL(many_final_kernel, dim3(n > 0 ? n : 1), dim3(64), 0, s, a);
    return hipGetLastError();
}

// dU[a][b] = sum_p g_p conj(d perm_p / d U_ab): one wavefront per entry; lane
// L adds items L, L+64, ... in order, then a fixed-order butterfly.
__global__ __launch_bounds__(256) void grad_scatter_kernel(const GradScatterArgs a) {
    const int e = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int nent = a.m * a.m;
    if (e >= nent) return;
    const int beg = a.offsets[e], end = a.offsets[e + 1];
    double re = 0.0, im = 0.0;
    for (int k = beg + lane; k < end; k += 64) {
        const int p = a.items[2 * k];
        const cplx d = a.dpat[a.items[2 * k + 1]];
        const cplx g = a.gperm[p];
        // g * conj(d)
        re = __builtin_fma(g.re, d.re, re);
        re = __builtin_fma(g.im, d.im, re);
        im = __builtin_fma(g.im, d.re, im);
        im = __builtin_fma(-g.re, d.im, im);
    }
#pragma unroll
    for (int msk = 32; msk >= 1; msk >>= 1) {
        re += __shfl_xor(re, msk, 64);
        im += __shfl_xor(im, msk, 64);
    }
    if (lane == 0) a.dU[(size_t)(e / a.m) * (size_t)a.lddu + (e % a.m)] = cplx{re, im};
}

hipError_t launch_grad_scatter(const GradScatterArgs& a, hipStream_t s) {
    const int n = a.m * a.m;
    hipLaunchKernelGGL(grad_scatter_kernel, dim3((n + 3) / 4 > 0 ? (n + 3) / 4 : 1), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Zero the queue counters (graph-safe: a kernel, not a memset node).
__global__ __launch_bounds__(64) void queue_prep_kernel(const QueuePrepArgs a) {
    for (int k = threadIdx.x; k < a.nzero; k += blockDim.x) a.zero[k] = 0u;
}

hipError_t launch_queue_prep(const QueuePrepArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(queue_prep_kernel, dim3(1), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_queue(int mode, int ncmax, int var, const QueueArgs& q, int grid, hipStream_t s) {
    switch (mode * 64 + ncmax) {
#define PQ_QCASE(MODE, NC) case MODE * 64 + NC: return launch_queue_##MODE##_##NC(var, q, grid, s);
        PQ_MCLASS_FWD(PQ_QCASE)
        PQ_MCLASS_EXT(PQ_QCASE)
#undef PQ_QCASE
        default: return hipErrorInvalidValue;
    }
}

int occupancy_queue(int mode, int ncmax, int var) {
    int blocks = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (mode * 64 + ncmax) {
#define PQ_QCASE(MODE, NC) case MODE * 64 + NC: e = occupancy_queue_##MODE##_##NC(var, &blocks); break;
        PQ_MCLASS_FWD(PQ_QCASE)
        PQ_MCLASS_EXT(PQ_QCASE)
#undef PQ_QCASE
        default: break;
    }
    return e == hipSuccess ? blocks : 0;
}

hipError_t launch_many(int mode, int ncmax, int var, const ManyArgs& a, hipStream_t s) {
    if (mode == kModeExtCol) {
        switch (ncmax) {
#define PQ_XCASE(NC) case NC: return launch_extcol_##NC(var, a, s);
            PQ_XCLASS(PQ_XCASE)
#undef PQ_XCASE
            default: return hipErrorInvalidValue;
        }
    }
    if (mode == kModeAdjWalk) {
        switch (ncmax) {
#define PQ_WCASE(NC) case NC: return launch_adjw_##NC(var, a, s);
            PQ_WCLASS(PQ_WCASE)
#undef PQ_WCASE
            default: return hipErrorInvalidValue;
        }
    }
    switch (mode * 64 + ncmax) {
#define PQ_MCASE(MODE, NC) case MODE * 64 + NC: return launch_many_##MODE##_##NC(var, a, s);
        PQ_MCLASS_FWD(PQ_MCASE)
        PQ_MCLASS_EXT(PQ_MCASE)
        PQ_MCLASS_ADJ(PQ_MCASE)
#undef PQ_MCASE
        default: return hipErrorInvalidValue;
    }
}

int occupancy_walk(int ncmax, int variant) {
    int blocks = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (ncmax) {
#define PQ_WOCC(NC) case NC: e = occupancy_adjw_##NC(variant, &blocks); break;
        PQ_WCLASS(PQ_WOCC)
#undef PQ_WOCC
        default: break;
    }
    return e == hipSuccess ? blocks : 0;
}

}  // namespace pq
