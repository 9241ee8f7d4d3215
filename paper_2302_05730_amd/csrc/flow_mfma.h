// The flow on the BF16 matrix cores, what its kernels share: the layout of the
// weight fragments (v_mfma_f32_32x32x16_bf16, see flow_bf16.hip for how the
// products chain) and the bodies of the kernels that run 64 samples per wave
// through a given evaluation of the flow.
#pragma once

#include "flow_impl.h"
#include "stratum.h"
#include "vsample_impl.h"

namespace mcubes {
namespace flow {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// fragments per layer: first product 2 row tiles x 6 K steps, second 2 x 4,
// third 4 x 4 (99 outputs padded to 128)
constexpr int G1T = 2, G1K = 6, G2T = 2, G2K = 4, G3T = 4, G3K = 4;
constexpr int OFF_G1 = 0, OFF_G2 = OFF_G1 + G1T * G1K, OFF_G3 = OFF_G2 + G2T * G2K;
constexpr int FRAGS = OFF_G3 + G3T * G3K;  // 36
// biases per layer in accumulator order: [tile][lane half][register]
constexpr int BOFF_1 = 0, BOFF_2 = BOFF_1 + G1T * 32, BOFF_3 = BOFF_2 + G2T * 32;
constexpr int BIAS = BOFF_3 + G3T * 32;  // 256

// row of the third product's 4 x 32 -> output: tile t < 3 holds the first 32 of
// the 33 spline outputs of mapped coordinate t, tile 3 the three last ones (row
// b: coordinate b's), so that one coordinate's outputs are one row tile and a
// value; -1 for the padding rows
__host__ __device__ constexpr int out_feature(int row) {
    return row < 32 * NB ? RAW * (row / 32) + row % 32
                         : (row < 32 * NB + NB ? RAW * (row - 32 * NB) + RAW - 1 : -1);
}

// feature held by accumulator register r of lane half h in row tile t
__host__ __device__ constexpr int acc_feature(int t, int r, int h) {
    return 32 * t + 8 * (r / 4) + 4 * h + (r % 4);
}

// Eight consecutive biases (16-byte aligned: every run starts at a multiple
// of 8 floats) as two 16-byte loads.
__device__ __forceinline__ void load_bias8(const float *__restrict__ p, float b[8]) {
    const float4 x = *reinterpret_cast<const float4 *>(p);
    const float4 y = *reinterpret_cast<const float4 *>(p + 4);
    b[0] = x.x; b[1] = x.y; b[2] = x.z; b[3] = x.w;
    b[4] = y.x; b[5] = y.y; b[6] = y.z; b[7] = y.w;
}

// Eight floats rounded to BF16 (nearest even): four v_cvt_pk_bf16_f32, where
// rounding with integer adds took about 4.5 instructions per value and a
// third of the sampling kernels' issue slots.
__device__ __forceinline__ bf16x8 pack8(const float v[8]) {
    typedef float f32x8 __attribute__((ext_vector_type(8)));
    f32x8 f;
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = v[i];
    return __builtin_convertvector(f, bf16x8);
}

// exp(x) for finite x below the overflow threshold, as 2^n 2^f: x log2(e) in two
// parts (the product's rounding error and the constant's low part in the second:
// Dekker's product by a fused multiply-add), n the integer nearest the first, the
// reduction of Cody and Waite (1980) in base 2.  The values expf gives (all but 4
// of 4e6 between -87 and 0), without its range checks.
__device__ __forceinline__ float exp_bounded(float x) {
    constexpr double kLog2e = 1.44269504088896340736;
    constexpr float kHi = (float)kLog2e, kLo = (float)(kLog2e - (double)kHi);
    const float p = x * kHi, q = __fmaf_rn(x, kLo, __fmaf_rn(x, kHi, -p));
    const float n = __builtin_rintf(p);
    return __builtin_ldexpf(__builtin_amdgcn_exp2f((p - n) + q), (int)n);
}

// Where the parameters sit in the packed forms (indices into theta over all
// layers; -1 for padding).  Bias entry gid (< L BIAS) of the accumulator-
// order bias array:
__device__ __forceinline__ int bias_param(int gid) {
    const int l = gid / BIAS, q = gid % BIAS;
    int off, t;
    if (q < BOFF_2) {
        off = OFF_B1; t = q / 32;
    } else if (q < BOFF_3) {
        off = OFF_B2; t = (q - BOFF_2) / 32;
    } else {
        off = OFF_B3; t = (q - BOFF_3) / 32;
    }
    const int w = q % 32, h = w / 16, r = w % 16;
    const int row = acc_feature(t, r, h), f = q < BOFF_3 ? row : out_feature(row);
    return f >= 0 ? l * LP + off + f : -1;
}

// element e of forward fragment slot gid = (layer, fragment, lane): the 8
// BF16 weights lane `lane` feeds to the matrix core
__device__ __forceinline__ int fwd_param(int gid, int e) {
    const int lane = gid % 64, fr = (gid / 64) % FRAGS, l = gid / (64 * FRAGS);
    const int row = lane % 32, h = lane / 32;
    if (fr < OFF_G2) {  // first product: natural K order over the 96 one-blob inputs
        const int t = fr / G1K, ks = fr % G1K;
        return l * LP + OFF_W1 + (16 * ks + 8 * h + e) * HID + 32 * t + row;
    }
    // second and third: K order of the previous accumulator registers
    const bool third = fr >= OFF_G3;
    const int q = fr - (third ? OFF_G3 : OFF_G2);
    const int t = q / 4, ks = q % 4;
    const int o = 32 * t + row;
    const int k = acc_feature(ks / 2, 8 * (ks % 2) + e, h);
    if (third) return out_feature(o) >= 0 ? l * LP + OFF_W3 + k * OUT + out_feature(o) : -1;
    return l * LP + OFF_W2 + k * HID + o;
}

// n / d, correctly rounded, for normal n, d and quotients: the reciprocal by one
// Newton step, the quotient by two corrections with its exact residual (Markstein
// 1990).  No scaling and no special cases: eight instructions instead of eleven.
__device__ __forceinline__ float div_normal(float n, float d) {
    float r = __builtin_amdgcn_rcpf(d);
    r = __fmaf_rn(__fmaf_rn(-d, r, 1.0f), r, r);
    float q = n * r;
    q = __fmaf_rn(__fmaf_rn(-d, q, n), r, q);
    return __fmaf_rn(__fmaf_rn(-d, q, n), r, q);
}

// Eight consecutive bumps of the one-blob encoding, k = k0 .. k0 + 7:
// e_k = exp(-(t - k)^2 / 2) with t = 32 u - 1/2.  The first directly, the
// rest by the ratio e_{k+1} / e_k = exp(t - k - 1/2), which itself shrinks
// by the constant exp(-1) per step: 2 exponentials and 14 multiplications
// instead of 8 exponentials.  The eighth bump stands behind 28 roundings (seven
// products by ratios that carry 21) and half a unit of x, up to 84: off by up to
// 5e-6 (3.3e-6 for |t - k| <= 3, 1e-6 rms), far under the BF16 rounding, 2e-3,
// that these inputs receive.  Starting
// at k0 keeps the first term representable whenever any of the eight
// matters: |t - k0| <= 13 if some |t - k| <= 6 (exp(-84.5) > FLT_MIN).
__device__ __forceinline__ void blob8(float u, int k0, float e[8]) {
    // (zero below half of the least subnormal number, as expf rounds: the ratio
    // would lift a subnormal first term to 1e-12 by the eighth)
    constexpr float kLeast = -149.0f * 0.69314718055994530942f;
    const float d = u * (float)BLOBS - 0.5f - (float)k0, x = -0.5f * d * d;
    e[0] = x < kLeast ? 0.0f : exp_bounded(x);
    float r = exp_bounded(d - 0.5f);
#pragma unroll
    for (int i = 1; i < 8; ++i) {
        e[i] = e[i - 1] * r;
        r *= 0.36787944117144233f;
    }
}

// One thread per (layer, fragment, lane): its 8 BF16 weights, and the biases
// in accumulator order.
__device__ __forceinline__ void pack_fwd(int gid, const float *__restrict__ theta,
                                         bf16x8 *__restrict__ frags, float *__restrict__ bias) {
    if (gid < L * BIAS) {
        const int p = bias_param(gid);
        bias[gid] = p >= 0 ? theta[p] : 0.0f;
    }
    if (gid >= L * FRAGS * 64) return;
    float v[8];
    for (int e = 0; e < 8; ++e) {
        const int p = fwd_param(gid, e);
        v[e] = p >= 0 ? theta[p] : 0.0f;
    }
    frags[gid] = pack8(v);
}

// relu(acc + b) of a product's two row tiles as the four operands of the
// next, b the biases in accumulator order; the maximum on the rounded bits
// (as 16-bit integers negative values are negative), two at a time.
__device__ __forceinline__ void relu_ops(const f32x16 (&acc)[2], const float *__restrict__ b,
                                         bf16x8 (&op)[4]) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        float bb[8];
        load_bias8(b + (ks / 2) * 32 + 8 * (ks % 2), bb);
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 8 * (ks % 2) + 2 * i;
            const f32x2 v = {acc[ks / 2][r] + bb[2 * i], acc[ks / 2][r + 1] + bb[2 * i + 1]};
            const bf16x2 c = __builtin_convertvector(v, bf16x2);
            w[i] = __builtin_bit_cast(
                uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, c), s16x2{}));
        }
        op[ks] = __builtin_bit_cast(bf16x8, w);
    }
}

// a of the column samples of both sample blocks: the lane's column l % 32 of
// block 0 in lo, of block 1 in hi
__device__ __forceinline__ void columns(float a, float &lo, float &hi) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(a), false,
                                                     false);
    lo = __uint_as_float(sw[0]);
    hi = __uint_as_float(sw[1]);
}

// A coordinate for the flow.  Beyond 64 every value maps alike (all bumps are
// zero, the spline's end), infinities too, whose differences and quotients in
// the spline would not be numbers.
__device__ __forceinline__ float flow_input(double v) {
    const float u = (float)v;
    return fabsf(u) > 64.0f ? copysignf(64.0f, u) : u;
}

// z (n x 6) -> x, log q, 64 samples per wave, flow(u) mapping a lane's sample in
// place and returning log q; lanes past n work on a copy of the last sample
// and store nothing.
template <class Flow>
__device__ __forceinline__ void map_samples(const Flow &flow, const double *__restrict__ z,
                                            int64_t n, double *__restrict__ x,
                                            double *__restrict__ logq) {
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    const int64_t wid = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    for (int64_t base = wid * 64; base < n; base += waves * 64) {
        const int64_t s = base + lane < n ? base + lane : n - 1;
        float u[D];
#pragma unroll
        for (int j = 0; j < D; ++j) u[j] = flow_input(z[s * D + j]);
        const float lq = flow(u);
        if (base + lane < n) {
#pragma unroll
            for (int j = 0; j < D; ++j) x[s * D + j] = (double)u[j];
            logq[s] = (double)lq;
        }
    }
}

// The flow-mapped iteration: 64 consecutive samples per wave, sample q = cube
// q / p, index q % p (p divides 64, so a cube's samples share a wave);
// per-cube statistics by butterfly sums over the p lanes of a cube.  Blocks of
// 256 threads.
template <int F, class Flow>
__device__ __forceinline__ void flow_iteration(const Flow &flow, const VsArgs &A,
                                               uint32_t stream_word, double *__restrict__ partials,
                                               uint32_t *__restrict__ whist) {
    constexpr int NBLK = (D + 3) / 4;
    __shared__ uint32_t hist[WH_BINS];
    wh_clear(hist);
    __syncthreads();
    const uint64_t N = (uint64_t)A.m * A.p;
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    const uint64_t wid = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int p = (int)A.p, log2p = __ffs(p) - 1;  // p divides 64
    double tS = 0.0, tV = 0.0;
    for (uint64_t base = wid * 64; base < N; base += waves * 64) {
        const uint64_t q = base + lane;
        const bool live = q < N;
        const uint32_t c = live ? (uint32_t)(q >> log2p) : 0u;
        const uint32_t k = live ? (uint32_t)q & (uint32_t)(p - 1) : 0u;
        float u[D];
        uint32_t rest = c;
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            uint32_t r[4];
            philox10(c, stream_word, k * NBLK + b, A.iteration, A.key0, A.key1, r);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = 4 * b + i;
                if (j < D) {
                    u[j] = stratum_coordinate(rest % A.g, r[i], A.g);
                    rest /= A.g;
                }
            }
        }
        const float lq = flow(u);
        Acc acc = Family<F, D>::begin(A.phase);
#pragma unroll
        for (int j = 0; j < D; ++j) Family<F, D>::axis(acc, A.ca[j], A.cu[j], (double)u[j]);
        const double w = Family<F, D>::end(acc, A) / exp((double)lq);
        if (live) wh_add(hist, w);
        // per-cube sums over the p lanes of the cube, shifted by its first sample
        const int first = lane & ~(p - 1);
        const double w0 = __shfl(w, first);
        const double dlt = w - w0;
        double S = w, D1 = dlt, D2 = dlt * dlt;
        for (int off = 1; off < p; off <<= 1) {
            S += __shfl_xor(S, off);
            D1 += __shfl_xor(D1, off);
            D2 += __shfl_xor(D2, off);
        }
        if (live && lane == first) {
            tS += S;
            tV += (D2 - D1 * D1 * A.inv_p) * A.inv_pm1;
        }
    }
    __shared__ double red[2][4];
    tS = wave_sum(tS);
    tV = wave_sum(tV);
    if (lane == 0) {
        red[0][threadIdx.x >> 6] = tS;
        red[1][threadIdx.x >> 6] = tV;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0, v = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
            s += red[0][w];
            v += red[1][w];
        }
        partials[2 * blockIdx.x] = s;
        partials[2 * blockIdx.x + 1] = v;
    }
    wh_flush(hist, whist);
}

// n plain (unstratified) samples of the flow with their weights w = f / q:
// sample i draws z from Philox counter (i, stream word, block, iteration); 64
// samples per wave, lanes past n work on a copy of the last sample and store
// nothing.
template <int F, class Flow>
__device__ __forceinline__ void draw_samples(const Flow &flow, const VsArgs &A,
                                             uint32_t stream_word, uint32_t n,
                                             double *__restrict__ xs, double *__restrict__ ws) {
    constexpr int NBLK = (D + 3) / 4;
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    const uint64_t wid = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    for (uint64_t base = wid * 64; base < n; base += waves * 64) {
        const bool live = base + lane < n;
        const uint32_t i = live ? (uint32_t)(base + lane) : n - 1;
        float u[D];
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            uint32_t r[4];
            philox10(i, stream_word, b, A.iteration, A.key0, A.key1, r);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (4 * b + t < D) u[4 * b + t] = (float)__fma_rn((double)r[t], 0x1p-32, 0x1p-33);
        }
        const float lq = flow(u);
        if (!live) continue;
        Acc acc = Family<F, D>::begin(A.phase);
#pragma unroll
        for (int j = 0; j < D; ++j) {
            Family<F, D>::axis(acc, A.ca[j], A.cu[j], (double)u[j]);
            xs[(uint64_t)i * D + j] = (double)u[j];
        }
        ws[i] = Family<F, D>::end(acc, A) / exp((double)lq);
    }
}

}  // namespace flow
}  // namespace mcubes
