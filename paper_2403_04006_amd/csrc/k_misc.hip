// Small kernels around the forward sweep: gather of the compact matrix with the
// inner digits' step tables, the final double-double reduction, and a
// constant fill for the trivial cases.
#include <hip/hip_runtime.h>

#include "device.h"
#include "kernels.h"

namespace pq {

// B[i][j] = U[out][in] for iterated row i and power column j; rows2 holds
// -2B_i (a digit increment lowers delta_i by 2) and +2B_i; base_j = sum_i mu_i B_ij
// (column sums with every digit at zero, delta_i = mu_i).  For mixed digits
// also the per-step table of the inner digits and the lanes' sums and weights,
// by workgroups of their own.
// Table, forward traversal: position q is the Gray state of rank q.  Reflected
// traversal: position p is the state of rank M-1-p (the inner code run
// backwards).  Entry p holds the row offset of the step from position p-1 to p
// (digit up -> -2B row, down -> +2B row) and the signed binomial weight of state p.
__global__ __launch_bounds__(kBlock) void prep_kernel(const PrepArgs a, const int nprep, const int ntab) {
    auto at = [&](int i, int j) {
        const int out = a.transposed ? a.col_mode[j] : a.row_mode[i];
        const int in = a.transposed ? a.row_mode[i] : a.col_mode[j];
        return a.U[(size_t)out * (size_t)a.ldu + (size_t)in];
    };
    if ((int)blockIdx.x >= nprep + ntab) {
        const int e = ((int)blockIdx.x - nprep - ntab) * kBlock + (int)threadIdx.x;
        const int j = e >> 6, lane = e & 63;
        if (j > a.nc) return;
        // digits of the lane: delta_i = mu_i - 2 d_i
        int d[kMaxLaneDigits];
        double w = lane < a.lane_states ? 1.0 : 0.0;
        int rest = lane;
#pragma unroll
        for (int i = 0; i < kMaxLaneDigits; ++i) {
            const int rho = i < a.n_lane ? a.lane_radix[i] : 1;
            d[i] = rest % rho;
            rest /= rho;
            if (i < a.n_lane) w *= digit_weight(rho, d[i]);
        }
        if (j == a.nc) {
            a.lane_w[lane] = w;
            return;
        }
        cplx s{0.0, 0.0};
#pragma unroll 8
        for (int i = 0; i < a.r; ++i) cfma_to(s, (double)a.row_mu[i], at(i, j));
#pragma unroll
        for (int i = 0; i < kMaxLaneDigits; ++i)
            if (i < a.n_lane) cfma_to(s, -2.0 * (double)d[i], at(i, j));
        a.lane_sums[e] = s;
        return;
    }
    if ((int)blockIdx.x >= nprep) {
        const int q = ((int)blockIdx.x - nprep) * kBlock + (int)threadIdx.x;
        if (q >= a.m_inner) return;
        const GrayStep e = gray_step(a.n_inner, [&](int k) { return a.radix[k]; }, a.m_inner, q);
        const int32_t of = (int32_t)((2 * e.fwd + (e.fwd_up ? 0 : 1)) * a.nc);
        const int32_t ob = (int32_t)((2 * e.bwd + (e.bwd_up ? 0 : 1)) * a.nc);
        a.tab_fwd[q] = StepEntry{q > 0 ? of : 0, 0, e.w};
        a.tab_bwd[a.m_inner - 1 - q] = StepEntry{q < a.m_inner - 1 ? ob : 0, 0, e.w};
        return;
    }
    const int total = a.r * a.nc;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += nprep * blockDim.x) {
        const int i = e / a.nc, j = e % a.nc;
        const cplx v = at(i, j);
        a.B[(size_t)i * a.nc + j] = v;
        a.rows2[((size_t)i * 2 + 0) * a.nc + j] = cplx{-2.0 * v.re, -2.0 * v.im};
        a.rows2[((size_t)i * 2 + 1) * a.nc + j] = cplx{2.0 * v.re, 2.0 * v.im};
    }
    if (blockIdx.x == 0 && a.m_inner == 0) {
        for (int j = threadIdx.x; j < a.nc; j += blockDim.x) {
            cplx s{0.0, 0.0};
#pragma unroll 8
            for (int i = 0; i < a.r; ++i) cfma_to(s, (double)a.row_mu[i], at(i, j));
            a.base[j] = s;
        }
    }
}

hipError_t launch_prep(const PrepArgs& a, hipStream_t s) {
    const int total = a.r * a.nc;
    int grid = (total + kBlock - 1) / kBlock;
    if (grid < 1) grid = 1;
    if (grid > 64) grid = 64;
    const int ntab = (a.m_inner + kBlock - 1) / kBlock;
    const int nlane = a.m_inner > 0 ? (64 * (a.nc + 1) + kBlock - 1) / kBlock : 0;
    hipLaunchKernelGGL(prep_kernel, dim3(grid + ntab + nlane), dim3(kBlock), 0, s, a, grid, ntab);
    return hipGetLastError();
}

// The pair sweep's table (layout at PairArgs): one thread per pair of columns and
// digit row (row 0 also takes the pair's constants), then one wavefront per
// column for the column sums, each lane a row.
__global__ __launch_bounds__(64) void pair_prep_kernel(const PairPrepArgs a, const int main_blocks) {
    const int P = a.pairs, W = 2 * P;
    const int e = blockIdx.x * 64 + (int)threadIdx.x;
    const int i = e / P, p = e - i * P;
    const int n_rows = a.n_lane + 3 + a.n_outer;
    auto at = [&](int row, int col) {
        if (col >= a.nc) return cplx{0.0, 0.0};
        const int out = a.transposed ? a.col_mode[col] : a.row_mode[row];
        const int in = a.transposed ? a.row_mode[row] : a.col_mode[col];
        return a.U[(size_t)out * (size_t)a.ldu + (size_t)in];
    };
    if ((int)blockIdx.x >= main_blocks) {
        const int col = (int)blockIdx.x - main_blocks, row = (int)threadIdx.x;
        cplx s{0.0, 0.0};
        if (row < a.r) {
            // the middle of a low digit is one unit of its row below digit zero
            const bool low = row >= a.n_lane && row < a.n_lane + 3;
            cfma_to(s, (double)(a.row_mu[row] - (low ? 1 : 0)), at(row, col));
        }
#pragma unroll
        for (int h = 32; h >= 1; h >>= 1) {
            s.re += shfl_xor_d(s.re, h);
            s.im += shfl_xor_d(s.im, h);
        }
        if (row == 0) a.tab[col] = col < a.nc ? s : cplx{1.0, 0.0};
        return;
    }
    if (i >= n_rows) return;
    cplx* lrow = a.tab + W;
    cplx* prod = lrow + kMaxLaneDigits * W;
    cplx* dev = prod + 4 * P;
    cplx* steps = dev + 8 * P;
    // sign patterns of the three lowest digits, up to a common sign
    const double sign[4][3] = {{1, 1, 1}, {1, -1, -1}, {-1, 1, -1}, {-1, -1, 1}};
    cplx ak[4], bk[4];
    cplx la[3], lb[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        la[q] = at(a.n_lane + q, 2 * p);
        lb[q] = at(a.n_lane + q, 2 * p + 1);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        ak[k] = bk[k] = cplx{0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            cfma_to(ak[k], sign[k][q], la[q]);
            cfma_to(bk[k], sign[k][q], lb[q]);
        }
    }
    if (i < a.n_lane) {
        const cplx x = at(i, 2 * p), y = at(i, 2 * p + 1);
        lrow[i * W + 2 * p] = cplx{-2.0 * x.re, -2.0 * x.im};
        lrow[i * W + 2 * p + 1] = cplx{-2.0 * y.re, -2.0 * y.im};
    } else if (i >= a.n_lane + 3) {
        const cplx x = at(i, 2 * p), y = at(i, 2 * p + 1);
        cplx* s = steps + ((size_t)(i - a.n_lane - 3) * 2 * P + p) * 6;
#pragma unroll
        for (int sel = 0; sel < 2; ++sel) {
            const double f = sel ? 2.0 : -2.0;
            const cplx sx{f * x.re, f * x.im}, sy{f * y.re, f * y.im};
            cplx* o = s + (size_t)sel * P * 6;
            o[0] = sx;
            o[1] = sy;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const cplx u = cmul(sx, bk[k]), v = cmul(sy, ak[k]);
                o[2 + k] = cplx{u.re + v.re, u.im + v.im};
            }
        }
    }
    if (i == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            prod[4 * p + k] = cmul(ak[k], bk[k]);
            dev[8 * p + 2 * k] = ak[k];
            dev[8 * p + 2 * k + 1] = bk[k];
        }
    }
}

hipError_t launch_pair_prep(const PairPrepArgs& a, hipStream_t s) {
    if (a.r > 64) return hipErrorInvalidValue;
    const int blocks = (a.pairs * (a.n_lane + 3 + a.n_outer) + 63) / 64;
    hipLaunchKernelGGL(pair_prep_kernel, dim3(blocks + 2 * a.pairs), dim3(64), 0, s, a, blocks);
    return hipGetLastError();
}

// One workgroup: every thread adds a strided subset of the partials in a
// fixed order, then a fixed tree over the threads.
__global__ __launch_bounds__(kBlock) void final_kernel(const FinalArgs a) {
    __shared__ double sh[kBlock][4];
    cdd s{{0.0, 0.0}, {0.0, 0.0}};
#pragma unroll 8
    for (int k = threadIdx.x; k < a.count; k += kBlock) {
        const double* p = a.partials + 4 * (size_t)k;
        s = cdd_add(s, cdd{{p[0], p[1]}, {p[2], p[3]}});
    }
    sh[threadIdx.x][0] = s.re.hi;
    sh[threadIdx.x][1] = s.re.lo;
    sh[threadIdx.x][2] = s.im.hi;
    sh[threadIdx.x][3] = s.im.lo;
    __syncthreads();
    for (int h = kBlock / 2; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) {
            cdd x{{sh[threadIdx.x][0], sh[threadIdx.x][1]}, {sh[threadIdx.x][2], sh[threadIdx.x][3]}};
            cdd y{{sh[threadIdx.x + h][0], sh[threadIdx.x + h][1]}, {sh[threadIdx.x + h][2], sh[threadIdx.x + h][3]}};
            x = cdd_add(x, y);
            sh[threadIdx.x][0] = x.re.hi;
            sh[threadIdx.x][1] = x.re.lo;
            sh[threadIdx.x][2] = x.im.hi;
            sh[threadIdx.x][3] = x.im.lo;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double re = (sh[0][0] + sh[0][1]) * a.scale;
        const double im = (sh[0][2] + sh[0][3]) * a.scale;
        if (a.perm) a.perm[0] = cplx{re, im};
        if (a.amp) a.amp[0] = cplx{re * a.norm, im * a.norm};
    }
}

hipError_t launch_final(const FinalArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(final_kernel, dim3(1), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

__global__ void fill_kernel(cplx* perm, cplx* amp, cplx v) {
    if (threadIdx.x == 0) {
        if (perm) perm[0] = v;
        if (amp) amp[0] = v;
    }
}

hipError_t launch_fill(cplx* perm, cplx* amp, cplx value, hipStream_t s) {
    hipLaunchKernelGGL(fill_kernel, dim3(1), dim3(64), 0, s, perm, amp, value);
    return hipGetLastError();
}

// --------------------------------------------------------------- dispatch
typedef hipError_t (*launch_fn)(int, const GlynnArgs&, int, hipStream_t);
typedef int (*occ_fn)(int);

#define PQ_LAUNCH_PTR(NC) &launch_glynn_##NC,
#define PQ_OCC_PTR(NC) &occupancy_glynn_##NC,
static const launch_fn g_launch[kMaxDim] = {PQ_NC_LIST(PQ_LAUNCH_PTR)};
static const occ_fn g_occ[kMaxDim] = {PQ_NC_LIST(PQ_OCC_PTR)};

hipError_t launch_fused(bool mix, const FusedArgs& a, int grid, hipStream_t s) {
    if (a.nc < 1 || a.r < 1 || a.r > kMaxDim || grid < 1) return hipErrorInvalidValue;
    switch ((a.nc + 1) / 2 * 2) {
#define PQ_FCASE(NC) case NC: return launch_fused_##NC(mix, a, grid, s);
        PQ_FCLASS(PQ_FCASE)
#undef PQ_FCASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_pair(int nc, const PairArgs& a, hipStream_t s) {
    if (a.groups < 1 || a.n_outer < 1 || a.blocks != 1ull << a.n_outer) return hipErrorInvalidValue;
    switch ((nc + 1) / 2) {
#define PQ_PCASE(P) case P: return launch_pair_##P(a, s);
        PQ_PCLASS(PQ_PCASE)
#undef PQ_PCASE
        default: return hipErrorInvalidValue;
    }
}

int occupancy_pair(int nc) {
    switch ((nc + 1) / 2) {
#define PQ_PCASE(P) case P: return occupancy_pair_##P();
        PQ_PCLASS(PQ_PCASE)
#undef PQ_PCASE
        default: return 0;
    }
}

hipError_t launch_glynn(int kind, int nc, const GlynnArgs& a, int grid, hipStream_t s) {
    if (nc < 1 || nc > kMaxDim || kind < 0 || kind > 2) return hipErrorInvalidValue;
    return g_launch[nc - 1](kind, a, grid, s);
}

int occupancy_glynn(int kind, int nc) {
    if (nc < 1 || nc > kMaxDim || kind < 0 || kind > 2) return 0;
    return g_occ[nc - 1](kind);
}

}  // namespace pq
