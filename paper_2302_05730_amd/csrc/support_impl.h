// Device bodies shared by the single-integrand and the batched support
// kernels: the fixed-order reduction of partial sums, the inverse-variance
// combination of the iteration estimates and the VEGAS rebinning of one axis.
#pragma once

#include <math.h>

#include "mcubes_internal.h"

namespace mcubes {

constexpr int kRefineThreads = 512;  // block of the refinement: more than kMaxBins

// Records (It, Vt) as iteration t in `state` (layout of mcubes_combine) and
// recombines iterations skip..t.  If no recorded iteration has zero variance
// the estimate is the inverse-variance weighted mean, its error (sum
// 1/var)^-1/2 and chi^2 the weighted squared deviations; an iteration with
// zero variance is exact and its estimate is taken as is.  By a whole block:
// the quotients of the iterations in parallel, their sums by thread 0 in
// iteration order.  Returns true in thread 0 when the iteration converged or
// is not finite.
struct CombineLds {
    double a[MCUBES_MAX_ITERATIONS], b[MCUBES_MAX_ITERATIONS];
    double mean;
    int exact;
};

__device__ __forceinline__ bool combine_block(double It, double Vt, double *__restrict__ state,
                                              uint32_t t, int skip, double rel_tol,
                                              CombineLds &L) {
    double *hist = state + MCUBES_STATE_HEADER;
    const int T = (int)t + 1, n = T - skip;
    // skip may be any int: only below T is it an index (and skip + a thread one)
    const int first = n >= 1 ? skip : T;
    if (threadIdx.x == 0) {
        hist[2 * t] = It;
        hist[2 * t + 1] = Vt;
        L.exact = -1;
    }
    __syncthreads();
    for (int q = first + (int)threadIdx.x; q < T; q += blockDim.x) {
        const double I = q == (int)t ? It : hist[2 * q], v = q == (int)t ? Vt : hist[2 * q + 1];
        if (v == 0.0) atomicMax(&L.exact, q);
        L.a[q] = 1.0 / v;
        L.b[q] = I / v;
    }
    __syncthreads();
    const int exact = L.exact;
    double sw = 0.0;
    if (threadIdx.x == 0 && n >= 1) {
        double swi = 0.0;
        for (int q = skip; q < T; ++q) {
            sw = sw + L.a[q];
            swi = swi + L.b[q];
        }
        L.mean = swi / sw;
    }
    __syncthreads();
    if (exact < 0) {
        const double mean = L.mean;
        for (int q = first + (int)threadIdx.x; q < T; q += blockDim.x) {
            const double I = q == (int)t ? It : hist[2 * q], v = q == (int)t ? Vt : hist[2 * q + 1];
            const double dv = I - mean;
            L.a[q] = dv * dv / v;
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return false;
    double Ibar = 0.0, sigma = INFINITY, chi2dof = 0.0;
    if (n >= 1) {
        if (exact >= 0) {  // zero variance: exact, the latest one counts
            Ibar = exact == (int)t ? It : hist[2 * exact];
            sigma = 0.0;
        } else {
            Ibar = L.mean;
            double chi2 = 0.0;
            for (int q = skip; q < T; ++q) chi2 = chi2 + L.a[q];
            sigma = 1.0 / sqrt(sw);
            chi2dof = n > 1 ? chi2 / (double)(n - 1) : 0.0;
        }
    }
    const bool bad = !isfinite(It) || !isfinite(Vt);
    const bool converged = n >= 1 && sigma <= rel_tol * fabs(Ibar);
    if (bad) state[6] = 1.0;
    state[4] = (double)T;
    state[0] = Ibar;
    state[1] = sigma;
    state[2] = chi2dof;
    state[3] = n >= 1 ? (double)(n - 1) : 0.0;
    state[5] = converged ? 1.0 : 0.0;
    return bad || converged;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sums of the pairs (S, V) in partials[2 b], partials[2 b + 1], b in [begin,
// end), by the first kReduceThreads threads of the block: strided sums, wave
// butterflies, then the waves in order, so the order depends on the count
// only.  Every thread of the block calls it (it synchronises); the sums are
// returned in thread 0.
constexpr int kReduceThreads = 256;
struct ReduceLds {
    double s[kReduceThreads / 64], v[kReduceThreads / 64];
};

__device__ __forceinline__ double2 reduce_partials(const double *__restrict__ partials,
                                                   uint32_t begin, uint32_t end, ReduceLds &L) {
    double s = 0.0, v = 0.0;
    if (threadIdx.x < kReduceThreads) {
        for (uint32_t b = begin + threadIdx.x; b < end; b += kReduceThreads) {
            s += partials[2 * (size_t)b];
            v += partials[2 * (size_t)b + 1];
        }
        s = wave_sum(s);
        v = wave_sum(v);
        if ((threadIdx.x & 63) == 0) {
            L.s[threadIdx.x >> 6] = s;
            L.v[threadIdx.x >> 6] = v;
        }
    }
    __syncthreads();
    s = v = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < kReduceThreads / 64; ++w) {
            s += L.s[w];
            v += L.v[w];
        }
    }
    return make_double2(s, v);
}

struct RefineLds {
    double E[kMaxBins + 1], d[kMaxBins], r[kMaxBins], R[kMaxBins + 1];
    double part[2][kRefineThreads / 64];
};

// VEGAS rebinning of one axis by a block of kRefineThreads > nb threads, one
// thread per bin.  New edge k lies in the first old bin i whose cumulative
// damped weight reaches k T, found by binary search between prefixes R with
// R_i < k T <= R_i+1.  The old edges are read into LDS before any new edge is
// written, so En may be the same row as E; with `clear` the bin sums are
// zeroed once read.
//
// A chain of latencies, not of work: the total and the cumulative weights are
// wave scans (six shuffles) and a pass over eight waves' totals, where one
// thread adding 500 values from LDS, twice, took 11 of 17 us at 500 bins; the
// default damping exponent 3/2 is x sqrt(x) instead of pow.
__device__ __forceinline__ void refine_axis(const double *E, double *dj, double *En, int nb,
                                            double alpha, bool clear, RefineLds &L) {
    const int k = threadIdx.x, lane = k & 63, wave = k >> 6;
    constexpr int kWaves = kRefineThreads / 64;
    double *sE = L.E, *sd = L.d, *sr = L.r, *sR = L.R;

    if (k <= nb) sE[k] = E[k];
    if (k < nb) {
        sd[k] = dj[k];
        if (clear) dj[k] = 0.0;
    }
    __syncthreads();
    double s = 0.0;
    if (k < nb) {
        if (k == 0)
            s = (sd[0] + sd[1]) / 2.0;
        else if (k == nb - 1)
            s = (sd[nb - 2] + sd[nb - 1]) / 2.0;
        else
            s = (sd[k - 1] + sd[k] + sd[k + 1]) / 3.0;
    }
    const double ws = wave_sum(s);
    if (lane == 0) L.part[0][wave] = ws;
    __syncthreads();
    double S = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) S += L.part[0][w];
    if (!(S > 0.0)) {  // no weight on this axis: keep it
        if (k <= nb) En[k] = sE[k];
        return;
    }
    double r = 0.0;
    if (k < nb) {
        const double rho = s / S;
        if (s == 0.0) {
            r = 0.0;
        } else if (rho == 1.0) {
            r = 1.0;
        } else {
            const double x = (rho - 1.0) / log(rho);
            r = alpha == 1.5 ? x * sqrt(x) : pow(x, alpha);
        }
        sr[k] = r;
    }
    double R = r;  // inclusive prefix over the wave
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double t = __shfl_up(R, off, 64);
        if (lane >= off) R += t;
    }
    if (lane == 63) L.part[1][wave] = R;
    __syncthreads();
    double before = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves - 1; ++w) before += w < wave ? L.part[1][w] : 0.0;
    if (k == 0) sR[0] = 0.0;
    if (k < nb) sR[k + 1] = before + R;
    __syncthreads();
    const double T = sR[nb] / (double)nb;
    if (k == 0) {
        En[0] = 0.0;
        En[nb] = 1.0;
    } else if (k < nb) {
        const double target = (double)k * T;
        // q in [1, nb] with R[q - 1] < target <= R[q] (nb if none), bin i = q - 1
        int lo = 1, hi = nb;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sR[mid] >= target)
                hi = mid;
            else
                lo = mid + 1;
        }
        const int i = lo - 1;
        const double W = sE[i + 1] - sE[i];
        double frac = (target - sR[i]) / sr[i];
        if (frac > 1.0) frac = 1.0;
        const double e = sE[i] + frac * W;
        En[k] = e < sE[i + 1] ? e : sE[i + 1];
    }
}

}  // namespace mcubes
