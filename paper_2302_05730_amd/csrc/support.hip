// Small kernels around V-Sample: fixed-order reduction of the block partials,
// the iteration combination, the VEGAS grid refinement, the three in one
// launch, and fills.
#include <math.h>

#include "support_impl.h"

namespace mcubes {

namespace {

__global__ void fill_kernel(double *__restrict__ d, int64_t n, double value) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) d[i] = value;
}

// E_j[i] = i / nb on every axis.
__global__ void init_grid_kernel(double *__restrict__ grid, int dim, int nb) {
    const int n = dim * (nb + 1);
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) {
        const int i = q % (nb + 1);
        grid[q] = (double)i / (double)nb;
    }
}

// I_t and var_t from the block partials (one block, fixed order).
__global__ __launch_bounds__(kReduceThreads) void reduce_kernel(
    const double *__restrict__ partials, int nparts, double n_samples, double var_denom,
    double *__restrict__ est) {
    __shared__ ReduceLds lds;
    const double2 sv = reduce_partials(partials, 0, (uint32_t)nparts, lds);
    if (threadIdx.x == 0) {
        est[0] = sv.x / n_samples;
        est[1] = sv.y / var_denom;
    }
}

// Inverse-variance combination of the recorded iterations skip..t (one block;
// at most MCUBES_MAX_ITERATIONS entries).
__global__ __launch_bounds__(64) void combine_kernel(const double *__restrict__ est,
                                                     double *__restrict__ state, uint32_t t,
                                                     int skip, double rel_tol) {
    __shared__ CombineLds lds;
    combine_block(est[0], est[1], state, t, skip, rel_tol, lds);
}

// VEGAS rebinning, one block per axis.
__global__ __launch_bounds__(kRefineThreads) void refine_kernel(const double *__restrict__ grid,
                                                                const double *__restrict__ bins,
                                                                double *__restrict__ grid_out,
                                                                int nb, double alpha) {
    __shared__ RefineLds lds;
    const int j = blockIdx.x;
    refine_axis(grid + (size_t)j * (nb + 1), const_cast<double *>(bins) + (size_t)j * nb,
                grid_out + (size_t)j * (nb + 1), nb, alpha, false, lds);
}

// What follows V-Sample in an iteration, in one launch: block j < dim refines
// (or copies) axis j, the last block reduces the partials and combines.  The
// two sides read nothing the other writes.  As separate kernels they took
// 3.8 + 3.1 + 17 us at 8-D and 500 bins and a launch gap each.
__global__ __launch_bounds__(kRefineThreads) void iteration_end_kernel(const IterationEnd P) {
    // an earlier iteration ended the integration: nothing to do (the word is
    // written by the launch of the iteration that ends it, with that number,
    // so a block that reads it meanwhile decides alike)
    if (P.stop && *P.stop < P.t) return;
    __shared__ union {
        RefineLds refine;
        struct {
            ReduceLds reduce;
            CombineLds combine;
        } sums;
    } lds;
    const int nb = P.nb;
    if (blockIdx.x < (unsigned)P.dim) {
        const int j = blockIdx.x;
        const double *row = P.grid + (size_t)j * (nb + 1);
        double *out = P.grid_out + (size_t)j * (nb + 1);
        if (P.bins)
            refine_axis(row, P.bins + (size_t)j * nb, out, nb, P.alpha, P.clear_bins, lds.refine);
        else if ((int)threadIdx.x <= nb)
            out[threadIdx.x] = row[threadIdx.x];
        return;
    }
    const double2 sv = reduce_partials(P.partials, 0, (uint32_t)P.nparts, lds.sums.reduce);
    __shared__ double est[2];
    if (threadIdx.x == 0) {
        est[0] = sv.x / P.n_samples;
        est[1] = sv.y / P.var_denom;
        P.est[0] = est[0];
        P.est[1] = est[1];
    }
    __syncthreads();
    const bool ended =
        combine_block(est[0], est[1], P.state, P.t, P.skip, P.rel_tol, lds.sums.combine);
    if (ended && P.stop) *P.stop = P.t;
}

// The start of an integration: uniform grid, zeroed state and bins, no stop.
__global__ void integrate_init_kernel(double *__restrict__ grid, int dim, int nb,
                                      double *__restrict__ zero, int64_t nzero,
                                      uint32_t *__restrict__ stop) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (int64_t)dim * (nb + 1)) grid[i] = (double)(i % (nb + 1)) / (double)nb;
    if (i < nzero) zero[i] = 0.0;
    if (i == 0) *stop = UINT32_MAX;
}

}  // namespace

hipError_t launch_fill(double *d, int64_t n, double value, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, d, n, value);
    return hipGetLastError();
}

hipError_t launch_init_grid(double *grid, int dim, int nb, hipStream_t stream) {
    const int n = dim * (nb + 1);
    hipLaunchKernelGGL(init_grid_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, grid, dim, nb);
    return hipGetLastError();
}

hipError_t launch_reduce(const double *partials, int nparts, double n_samples, double var_denom,
                         double *est, hipStream_t stream) {
    hipLaunchKernelGGL(reduce_kernel, dim3(1), dim3(kReduceThreads), 0, stream, partials, nparts, n_samples,
                       var_denom, est);
    return hipGetLastError();
}

hipError_t launch_combine(const double *est, double *state, uint32_t iteration, int skip,
                          double rel_tol, hipStream_t stream) {
    hipLaunchKernelGGL(combine_kernel, dim3(1), dim3(64), 0, stream, est, state, iteration, skip,
                       rel_tol);
    return hipGetLastError();
}

hipError_t launch_refine(const double *grid, const double *bins, double *grid_out, int dim, int nb,
                         double alpha, hipStream_t stream) {
    hipLaunchKernelGGL(refine_kernel, dim3(dim), dim3(kRefineThreads), 0, stream, grid, bins,
                       grid_out, nb, alpha);
    return hipGetLastError();
}

hipError_t launch_iteration_end(const IterationEnd &P, hipStream_t stream) {
    // a grid that stays as and where it is needs no blocks of its own
    IterationEnd Q = P;
    if (!Q.bins && Q.grid == Q.grid_out) Q.dim = 0;
    hipLaunchKernelGGL(iteration_end_kernel, dim3(Q.dim + 1), dim3(kRefineThreads), 0, stream, Q);
    return hipGetLastError();
}

hipError_t launch_integrate_init(double *grid, int dim, int nb, double *zero, int64_t nzero,
                                 uint32_t *stop, hipStream_t stream) {
    const int64_t ng = (int64_t)dim * (nb + 1), n = ng > nzero ? ng : nzero;
    hipLaunchKernelGGL(integrate_init_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                       stream, grid, dim, nb, zero, nzero, stop);
    return hipGetLastError();
}

}  // namespace mcubes
