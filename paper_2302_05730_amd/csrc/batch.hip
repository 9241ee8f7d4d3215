// Support kernels of the batched form: the start of a run and the end of an
// iteration (per-integrand reduction of the tile partials, combination,
// refinement and the iteration counter).  They read the iteration number and
// the done flags from device memory, so one captured graph serves every
// iteration of a batch.
#include <algorithm>

#include "support_impl.h"

namespace mcubes {

namespace {

// The start of a run, in one launch: uniform grids E_j[k] = k / nb (block q <
// naxes the row axes[q], and zeroed sums of its bins), zeroed states, no
// integrand done, iteration 0.  A kernel rather than memsets, so that it can
// sit in a captured graph.
__global__ __launch_bounds__(256) void batch_init_kernel(const BatchInit P) {
    if (blockIdx.x < (unsigned)P.naxes) {
        const uint2 ax = P.axes[blockIdx.x];
        const BatchItem &B = P.items[ax.x];
        const int nb = B.nb;
        double *row = P.grids + B.grid_off + (size_t)ax.y * (nb + 1);
        double *sum = P.bins + B.bins_off + (size_t)ax.y * nb;
        for (int k = threadIdx.x; k <= nb; k += blockDim.x) {
            row[k] = (double)k / (double)nb;
            if (k < nb) sum[k] = 0.0;
        }
    }
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t q = tid; q < P.state_len; q += stride) P.states[q] = 0.0;
    for (int64_t q = tid; q <= P.n; q += stride) P.done[q] = 0u;  // and the ticket
    if (tid == 0) *P.iter = 0u;
}

// Sums, estimate and variance of integrand i from its tiles' partials, in the
// fixed order of the single-integrand form; in thread 0.
__device__ __forceinline__ double2 item_estimate(const BatchItem &B,
                                                 const double *__restrict__ partials,
                                                 ReduceLds &L) {
    const double2 sv = reduce_partials(partials, B.part_begin, B.part_end, L);
    return make_double2(sv.x / B.n_samples, sv.y / B.var_denom);
}

// What follows V-Sample in an iteration, in one launch.  Block i < n reduces
// the partials of integrand i and combines, and marks it done (iteration + 1)
// when it converged or its estimate is not finite; block n + q refines the row
// axes[q] in place and zeroes its bin sums, if its integrand recorded this
// iteration (one that converges in it is refined once more, as the
// single-integrand loop does) with a finite estimate, for which it forms the
// sums itself: no block waits for another.  The last one to end counts the
// iteration.  A chain of launches, not of work: as fill, reduction,
// combination, refinement, counter and the copy of the flags, six launches,
// 46 us of an iteration of 48 integrands; in one, 18.
__global__ __launch_bounds__(kRefineThreads) void batch_end_kernel(const BatchEnd P) {
    __shared__ union {
        RefineLds refine;
        CombineLds combine;
    } lds;
    __shared__ ReduceLds sums;
    __shared__ double est[2];
    const bool refines = blockIdx.x >= (unsigned)P.n;
    const uint2 ax = refines ? P.axes[blockIdx.x - P.n] : make_uint2(blockIdx.x, 0u);
    const uint32_t t = *P.iter;
    // written by this launch with t + 1 only, so a block that reads it
    // meanwhile decides alike
    const uint32_t done = P.done[ax.x];
    if (done == 0u || done == t + 1u) {
        const BatchItem &B = P.items[ax.x];
        const double2 e = item_estimate(B, P.partials, sums);
        if (threadIdx.x == 0) {
            est[0] = e.x;
            est[1] = e.y;
        }
        __syncthreads();
        if (refines) {
            const int nb = B.nb;
            double *row = P.grids + B.grid_off + (size_t)ax.y * (nb + 1);
            if (isfinite(est[0]) && isfinite(est[1]))
                refine_axis(row, P.bins + B.bins_off + (size_t)ax.y * nb, row, nb, P.alpha, true,
                            lds.refine);
        } else {
            double *state = P.states + (size_t)ax.x * MCUBES_STATE_LEN;
            if (combine_block(est[0], est[1], state, t, P.skip, P.rel_tol, lds.combine)) {
                P.done[ax.x] = t + 1u;
                P.host_done[ax.x] = t + 1u;
            }
        }
    }
    __syncthreads();  // every thread has read the iteration
    if (threadIdx.x == 0 && atomicAdd(P.done + P.n, 1u) == gridDim.x - 1u) {
        P.done[P.n] = 0u;
        *P.iter = t + 1u;
    }
}

// One iteration on given grids: block q refines the row axes[q] of its
// integrand, whatever its estimate; block q of an integrand's first axis
// writes the estimate too.
__global__ __launch_bounds__(kRefineThreads) void batch_step_end_kernel(
    const BatchItem *__restrict__ items, const uint2 *__restrict__ axes, double *__restrict__ grids,
    double *__restrict__ bins, const double *__restrict__ partials, double alpha,
    double *__restrict__ est) {
    __shared__ RefineLds refine;
    __shared__ ReduceLds sums;
    const uint2 ax = axes[blockIdx.x];
    const BatchItem &B = items[ax.x];
    const int nb = B.nb;
    if (ax.y == 0u) {
        const double2 e = item_estimate(B, partials, sums);
        if (threadIdx.x == 0) {
            est[2 * ax.x] = e.x;
            est[2 * ax.x + 1] = e.y;
        }
    }
    double *row = grids + B.grid_off + (size_t)ax.y * (nb + 1);
    refine_axis(row, bins + B.bins_off + (size_t)ax.y * nb, row, nb, alpha, false, refine);
}

// out <- values [offset, offset + width) of the states, row by row, `count` in
// all.  The host then takes one contiguous copy: a pitched one to pageable
// memory moves row by row, 350 us for 48 integrands' results and as much for
// their traces, where this and the copy take 25 us.
__global__ __launch_bounds__(256) void batch_gather_kernel(const double *__restrict__ states,
                                                           int64_t offset, int64_t width,
                                                           int64_t count,
                                                           double *__restrict__ out) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < count; q += stride)
        out[q] = states[q / width * MCUBES_STATE_LEN + offset + q % width];
}

}  // namespace

hipError_t launch_batch_init(const BatchInit &P, hipStream_t stream) {
    const int64_t blocks = std::max<int64_t>(P.naxes, std::min<int64_t>((P.state_len + 255) / 256, 4096));
    hipLaunchKernelGGL(batch_init_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, P);
    return hipGetLastError();
}

hipError_t launch_batch_end(const BatchEnd &P, bool refine, hipStream_t stream) {
    hipLaunchKernelGGL(batch_end_kernel, dim3(P.n + (refine ? P.naxes : 0)), dim3(kRefineThreads), 0,
                       stream, P);
    return hipGetLastError();
}

hipError_t launch_batch_step_end(const BatchItem *items, const uint2 *axes, int naxes,
                                 double *grids, double *bins, const double *partials, double alpha,
                                 double *est, hipStream_t stream) {
    hipLaunchKernelGGL(batch_step_end_kernel, dim3(naxes), dim3(kRefineThreads), 0, stream, items,
                       axes, grids, bins, partials, alpha, est);
    return hipGetLastError();
}

hipError_t launch_batch_gather(const double *states, int64_t offset, int64_t width, int64_t count,
                               double *out, hipStream_t stream) {
    const int64_t blocks = std::min<int64_t>((count + 255) / 256, 4096);
    hipLaunchKernelGGL(batch_gather_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, states,
                       offset, width, count, out);
    return hipGetLastError();
}

}  // namespace mcubes
