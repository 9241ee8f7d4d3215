// The FP32 flow on the BF16 matrix cores: density, sampling and the draw of
// training samples.
//
// Every FP32 operand of a product is split into three BF16 parts, v = hi + mid
// + lo, exactly (rounded to nearest: mid and lo have either sign, up to 2^-8 and
// 2^-17 of v), and a product is the sum of six of the nine partial products,
// hi hi, hi mid, mid hi, mid mid, hi lo, lo hi, accumulated in FP32.  Of the
// three left out mid lo and lo mid reach 2^-25 of the product each, together
// what rounding it to FP32 may cost, and the matrix cores' sums are truncated
// where a multiply-add rounds: a product by itself is off by up to 3 x 2^-24,
// by a multiply-add 2^-24.  But a sum of 96 is rounded 36 times instead of 96,
// and the flow as a whole comes out closer to 64 bits: log q of networks as
// training leaves them 3.9e-7 rms (multiply-adds 4.3e-7), of steeper ones
// 2.2e-6 and 1.7e-5 (2.8e-6, 2.3e-5).  With mid lo and lo mid it is 2.1e-6 and
// 1.7e-5, and a fifth slower.  Six matrix instructions at 16 times the FP32 rate.
//
// Waves, fragments and the chaining of the products as in flow_bf16.hip; the
// fragments of a layer hold the three parts one after the other.  The matrix
// cores take 14,000 cycles per layer and 64 samples, the vector ALU about
// 17,000 (the encoding's 96 exponentials, splitting 224 values, the splines),
// so the two overlap between the two waves of a SIMD.
#include "flow_mfma.h"

namespace mcubes {

namespace {

using namespace flow;

constexpr int PARTS = 3;

struct Split {
    bf16x8 p[PARTS];  // hi, mid, lo
};

__device__ __forceinline__ float bf16_low(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_high(uint32_t w) {
    return __uint_as_float(w & 0xffff0000u);
}

__device__ __forceinline__ Split split8(const float v[8]) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    float r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = v[i];
    Split s;
#pragma unroll
    for (int q = 0; q < PARTS; ++q) {
        s.p[q] = pack8(r);
        const u32x4 w = __builtin_bit_cast(u32x4, s.p[q]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r[2 * i] -= bf16_low(w[i]);
            r[2 * i + 1] -= bf16_high(w[i]);
        }
    }
    return s;
}

// One thread per (layer, fragment, lane): the three parts of its 8 weights,
// and the biases in accumulator order.
__global__ void pack_fp32_kernel(const float *__restrict__ theta, bf16x8 *__restrict__ frags,
                                 float *__restrict__ bias) {
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
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
    const Split s = split8(v);
#pragma unroll
    for (int q = 0; q < PARTS; ++q) frags[((gid / 64) * PARTS + q) * 64 + gid % 64] = s.p[q];
}

// An Adam step that writes the new parameters into the fragments and biases as
// well (inv: where each sits, see launch_flow_inverse_map), as pack_fp32_kernel
// would: a launch less, 7.2 us a step and not 9.1.
__global__ __launch_bounds__(256) void adam_pack_fp32_kernel(
    float *__restrict__ theta, float *__restrict__ m, float *__restrict__ v,
    const float *__restrict__ grad, float lr, float beta1, float beta2, float eps, float c1,
    float c2, const int *__restrict__ inv, uint16_t *__restrict__ frags,
    float *__restrict__ bias) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= flow::PARAMS) return;
    const float t = adam_update(theta, m, v, i, grad[i], lr, beta1, beta2, eps, c1, c2);
    const int pf = inv[3 * i], pz = inv[3 * i + 2];
    if (pz >= 0) bias[pz] = t;
    if (pf < 0) return;
    const int gid = pf / 8;
    float r = t;
#pragma unroll
    for (int q = 0; q < PARTS; ++q) {
        const __bf16 part = (__bf16)r;
        frags[(((gid / 64) * PARTS + q) * 64 + gid % 64) * 8 + pf % 8] =
            __builtin_bit_cast(uint16_t, part);
        r -= (float)part;
    }
}

// acc += f x, smallest partial products first; F points at the lane's entry of
// the fragment's first part.
template <int NSB>
__device__ __forceinline__ void split_product(const bf16x8 *__restrict__ F, const Split (&x)[NSB],
                                              f32x16 (&acc)[NSB]) {
    const bf16x8 hi = F[0], mid = F[64], lo = F[128];
#define TERM(W, X)                                                                               \
    _Pragma("unroll") for (int sb = 0; sb < NSB; ++sb) acc[sb] =                                 \
        __builtin_amdgcn_mfma_f32_32x32x16_bf16(W, x[sb].p[X], acc[sb], 0, 0, 0)
    TERM(lo, 0);
    TERM(hi, 2);
    TERM(mid, 1);
    TERM(mid, 0);
    TERM(hi, 1);
    TERM(hi, 0);
#undef TERM
}

// exp(x) for finite x <= 0, to 1.3 ulp (expf: 0.9): the hardware 2^p with the
// rounding error of p = x log2(e) put back to first order.  0 below 2^-126.
__device__ __forceinline__ float exp_neg(float x) {
    constexpr double kLog2e = 1.44269504088896340736;
    constexpr float kHi = (float)kLog2e, kLo = (float)(kLog2e - (double)kHi);
    const float p = x * kHi, q = __fmaf_rn(x, kLo, __fmaf_rn(x, kHi, -p));
    const float e = __builtin_amdgcn_exp2f(p);
    return __fmaf_rn(e, q * (float)0.69314718055994530942, e);
}

// 2^32 exp(x), alike: 0 below 2^-158, where expf is below 2^-149.
__device__ __forceinline__ float exp_neg32(float x) {
    constexpr double kLog2e = 1.44269504088896340736;
    constexpr float kHi = (float)kLog2e, kLo = (float)(kLog2e - (double)kHi);
    const float p = __fmaf_rn(x, kHi, 32.0f), q = __fmaf_rn(x, kLo, __fmaf_rn(x, kHi, 32.0f - p));
    const float e = __builtin_amdgcn_exp2f(p);
    return __fmaf_rn(e, q * (float)0.69314718055994530942, e);
}

// The spline of raw outputs at v, forward (a coordinate to its CDF) or inverse,
// on unnormalised widths w_i and heights E_i: with s the sum of the widths, X_k
// the vertices times s and C_k = sum_{i<k} (E_i + E_{i+1}) w_i (twice the mass
// left of vertex k), the bin is the last with X_k <= v s (forward) or C_k <= v
// C_16 (inverse); inside it, a being the fraction of the bin,
//   C(a) = C_k + w (2 a E_0 + a^2 dE),  density = 2 (E_0 + a dE) s / C_16.
// Only results are divided by totals, and the bin is found by halving: each
// level keeps half of the widths and heights.  Returns the log density.
//
// Heights may lie anywhere below the highest, to 2^-149 of it and further, and so
// may the density.  (The hardware's 2^x and log2 flush subnormals: with heights
// from 1 down log q was -inf in a bin 2^-126 of the highest.)  So the heights
// here are 2^32 times theirs, normal down to 2^-158, the totals too, and the
// logarithm is that of the whole range.  A width below 2^-126 of the largest is 0,
// a bin without a point.  Numerators are held to the bin, so that every quotient
// is normal.  100,000 densities 110 us; with subnormal heights, expf and plain
// divisions 116, without them 103.
template <bool INVERSE>
__device__ __forceinline__ float spline_raw(const float raw[RAW], float v, float &out) {
    float mw = raw[0], mv = raw[BINS];
#pragma unroll
    for (int i = 1; i < BINS; ++i) mw = fmaxf(mw, raw[i]);
#pragma unroll
    for (int i = 1; i <= BINS; ++i) mv = fmaxf(mv, raw[BINS + i]);
    float w[BINS], E[BINS + 1];
#pragma unroll
    for (int i = 0; i < BINS; ++i) w[i] = exp_neg(raw[i] - mw);
#pragma unroll
    for (int i = 0; i <= BINS; ++i) E[i] = exp_neg32(raw[BINS + i] - mv);
    float c = 0.0f, x = 0.0f, cq[4], xq[4];
#pragma unroll
    for (int i = 0; i < BINS; ++i) {
        c = __fmaf_rn(E[i] + E[i + 1], w[i], c);
        x += w[i];
        if (i % 4 == 3) {
            cq[i / 4] = c;
            xq[i / 4] = x;
        }
    }
    const float t = v * (INVERSE ? c : x);
    // halves, then quarters, by the stored prefixes
    bool in = (INVERSE ? cq[1] : xq[1]) <= t;
    float C = in ? cq[1] : 0.0f, X = in ? xq[1] : 0.0f;
    float Cm = in ? cq[2] : cq[0], Xm = in ? xq[2] : xq[0];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = in ? w[8 + i] : w[i];
#pragma unroll
    for (int i = 0; i <= 8; ++i) E[i] = in ? E[8 + i] : E[i];
    in = (INVERSE ? Cm : Xm) <= t;
    C = in ? Cm : C;
    X = in ? Xm : X;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = in ? w[4 + i] : w[i];
#pragma unroll
    for (int i = 0; i <= 4; ++i) E[i] = in ? E[4 + i] : E[i];
    // pairs, then the bin, by prefixes formed again in the same order
    Cm = __fmaf_rn(E[1] + E[2], w[1], __fmaf_rn(E[0] + E[1], w[0], C));
    Xm = (X + w[0]) + w[1];
    in = (INVERSE ? Cm : Xm) <= t;
    C = in ? Cm : C;
    X = in ? Xm : X;
#pragma unroll
    for (int i = 0; i < 2; ++i) w[i] = in ? w[2 + i] : w[i];
#pragma unroll
    for (int i = 0; i <= 2; ++i) E[i] = in ? E[2 + i] : E[i];
    Cm = __fmaf_rn(E[0] + E[1], w[0], C);
    Xm = X + w[0];
    in = (INVERSE ? Cm : Xm) <= t;
    C = in ? Cm : C;
    X = in ? Xm : X;
    const float wb = in ? w[1] : w[0], E0 = in ? E[1] : E[0], E1 = in ? E[2] : E[1];
    const float dE = E1 - E0;
    float a;
    if (INVERSE) {
        // (t - C) / wb, at most E0 + E1 <= 2^33 inside the cube
        const float n = t - C, q = div_normal(n > 0x1p33f * wb ? 0x1p33f * wb : n, wb);
        const float den = E0 + sqrtf(fmaxf(__fmaf_rn(dE, q, E0 * E0), 0.0f));
        const float ad = div_normal(q > den ? den : q, den);  // (in any case: no branch)
        a = fminf(fmaxf(den > 0.0f ? ad : 0.0f, 0.0f), 1.0f);
        out = div_normal(__fmaf_rn(a, wb, X), x);
    } else {
        const float n = t - X;
        a = fminf(fmaxf(div_normal(n > wb ? wb : n, wb), 0.0f), 1.0f);
        out = div_normal(__fmaf_rn(wb * a, __fmaf_rn(a, dE, 2.0f * E0), C), c);
    }
    return logf(__fmaf_rn(a, dE, E0) * div_normal(2.0f * x, c));
}

// eight bumps k0 .. k0 + 7 of the one-blob encoding of both sample blocks
__device__ __forceinline__ void encode(const float (&ua)[2], int k0, Split (&op)[2]) {
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
        float e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float t = __fmaf_rn(ua[sb], (float)BLOBS, -0.5f - (float)(k0 + i));
            e[i] = exp_neg(-0.5f * t * t);
        }
        op[sb] = split8(e);
    }
}

// relu(acc + b) of a product's two row tiles, split, as the four operands of
// the next; b the biases in accumulator order
__device__ __forceinline__ void relu_split(const f32x16 (&acc)[2], const float *__restrict__ b,
                                           int sb, Split (&op)[4][2]) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        float v[8], bb[8];
        load_bias8(b + (ks / 2) * 32 + 8 * (ks % 2), bb);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = fmaxf(acc[ks / 2][8 * (ks % 2) + i] + bb[i], 0.0f);
        op[ks][sb] = split8(v);
    }
}

// 64 samples through the flow (or its inverse): lane s holds sample s in u[]
// and returns log q.  All 64 lanes must be active.
template <bool INVERSE>
__device__ __forceinline__ float flow_wave(const bf16x8 *__restrict__ frags,
                                           const float *__restrict__ bias, float u[D]) {
    const int lane = threadIdx.x & 63, h = lane >> 5;
    float lq = 0.0f;
#pragma unroll 1
    for (int step = 0; step < L; ++step) {
        const int l = INVERSE ? L - 1 - step : step;
        const bf16x8 *F = frags + (size_t)l * FRAGS * PARTS * 64 + lane;
        const float *Bs = bias + l * BIAS + h * 16;
        f32x16 acc[2][2];  // [row tile][sample block]
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t][0] = acc[t][1] = f32x16{};
        float ua[NA][2];
#pragma unroll
        for (int a = 0; a < NA; ++a) columns(getu(u, a_idx(l, a)), ua[a][0], ua[a][1]);
        // the operands of a step are formed while the step before multiplies
        Split op[2];
        encode(ua[0], 8 * h, op);
#pragma unroll
        for (int ks = 0; ks < G1K; ++ks) {
            Split next[2];
            if (ks + 1 < G1K) encode(ua[(ks + 1) / 2], 16 * ((ks + 1) % 2) + 8 * h, next);
#pragma unroll
            for (int t = 0; t < G1T; ++t)
                split_product<2>(F + (OFF_G1 + t * G1K + ks) * PARTS * 64, op, acc[t]);
            if (ks + 1 < G1K) {
                op[0] = next[0];
                op[1] = next[1];
            }
        }
        Split h1[G2K][2], h2[G3K][2];
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
            const f32x16 a2[2] = {acc[0][sb], acc[1][sb]};
            relu_split(a2, Bs + BOFF_1, sb, h1);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t][0] = acc[t][1] = f32x16{};
#pragma unroll
        for (int ks = 0; ks < G2K; ++ks)
#pragma unroll
            for (int t = 0; t < G2T; ++t)
                split_product<2>(F + (OFF_G2 + t * G2K + ks) * PARTS * 64, h1[ks], acc[t]);
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
            const f32x16 a2[2] = {acc[0][sb], acc[1][sb]};
            relu_split(a2, Bs + BOFF_2, sb, h2);
        }
        // one row tile of the third product, both sample blocks, and every lane
        // handed its own sample's rows (those of lane half 0 in o[0], of half 1
        // in o[1]), biases added
        const float *B3 = bias + l * BIAS + BOFF_3;
        const auto third = [&](int t, f32x16 (&o)[2]) {
            o[0] = o[1] = f32x16{};
#pragma unroll
            for (int ks = 0; ks < G3K; ++ks)
                split_product<2>(F + (OFF_G3 + t * G3K + ks) * PARTS * 64, h2[ks], o);
        };
        const auto own = [&](int t, int r, f32x16 (&o)[2]) {
            const auto sw = __builtin_amdgcn_permlane32_swap(
                __float_as_uint(o[0][r]), __float_as_uint(o[1][r]), false, false);
            o[0][r] = __uint_as_float(sw[0]) + B3[32 * t + r];
            o[1][r] = __uint_as_float(sw[1]) + B3[32 * t + 16 + r];
        };
        f32x16 o[2], ahead[2];
        third(NB, ahead);
        third(0, o);
        float last[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            own(NB, b, ahead);
            last[b] = ahead[0][b];
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            // the next coordinate's outputs multiply while this one's spline runs
            if (b + 1 < NB) third(b + 1, ahead);
            float raw[RAW];
#pragma unroll
            for (int r = 0; r < 16; ++r) own(b, r, o);
#pragma unroll
            for (int k = 0; k < RAW - 1; ++k) raw[k] = o[(k / 4) % 2][4 * (k / 8) + k % 4];
            raw[RAW - 1] = last[b];
            const int j = b_idx(l, b);
            float v;
            lq += spline_raw<INVERSE>(raw, getu(u, j), v);
            setu(u, j, v);
            o[0] = ahead[0];
            o[1] = ahead[1];
        }
    }
    return lq;
}

// two waves per SIMD (256 registers)
#define FP32_WAVES __attribute__((amdgpu_waves_per_eu(2)))

template <bool INVERSE>
__global__ __launch_bounds__(256) FP32_WAVES void map_fp32_kernel(
    const bf16x8 *__restrict__ frags, const float *__restrict__ bias,
    const double *__restrict__ in, int64_t n, double *__restrict__ out,
    double *__restrict__ logq) {
    map_samples([&](float u[D]) { return flow_wave<INVERSE>(frags, bias, u); }, in, n, out, logq);
}

template <int F>
__global__ __launch_bounds__(256) FP32_WAVES void flow_draw_fp32_kernel(
    const bf16x8 *__restrict__ frags, const float *__restrict__ bias, const VsArgs A,
    uint32_t stream_word, uint32_t n, double *__restrict__ xs, double *__restrict__ ws) {
    draw_samples<F>([&](float u[D]) { return flow_wave<true>(frags, bias, u); }, A, stream_word, n,
                    xs, ws);
}

unsigned map_blocks(int64_t n) {
    const int64_t blocks = (n + 255) / 256;
    return (unsigned)(blocks < 8192 ? blocks : 8192);
}

}  // namespace

int64_t flow_fp32_frag_bytes() { return (int64_t)L * FRAGS * PARTS * 64 * sizeof(bf16x8); }
int64_t flow_fp32_bias_floats() { return (int64_t)L * BIAS; }

hipError_t launch_flow_pack_fp32(const float *theta, void *frags, float *bias, hipStream_t s) {
    hipLaunchKernelGGL(pack_fp32_kernel, dim3((L * FRAGS * 64 + 255) / 256), dim3(256), 0, s, theta,
                       (bf16x8 *)frags, bias);
    return hipGetLastError();
}

hipError_t launch_flow_adam_pack_fp32(float *theta, float *m, float *v, const float *grad, float lr,
                                      float beta1, float beta2, float eps, float c1, float c2,
                                      const int *inv, void *frags, float *bias, hipStream_t s) {
    hipLaunchKernelGGL(adam_pack_fp32_kernel, dim3((flow::PARAMS + 255) / 256), dim3(256), 0, s,
                       theta, m, v, grad, lr, beta1, beta2, eps, c1, c2, inv, (uint16_t *)frags,
                       bias);
    return hipGetLastError();
}

hipError_t launch_flow_map_fp32(bool inverse, const void *frags, const float *bias,
                                const double *in, int64_t n, double *out, double *logq,
                                hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (inverse)
        hipLaunchKernelGGL(map_fp32_kernel<true>, dim3(map_blocks(n)), dim3(256), 0, s,
                           (const bf16x8 *)frags, bias, in, n, out, logq);
    else
        hipLaunchKernelGGL(map_fp32_kernel<false>, dim3(map_blocks(n)), dim3(256), 0, s,
                           (const bf16x8 *)frags, bias, in, n, out, logq);
    return hipGetLastError();
}

namespace {

template <int F>
hipError_t launch_draw_f(const void *frags, const float *bias, const VsArgs &A,
                         uint32_t stream_word, uint32_t n, double *xs, double *ws, hipStream_t s) {
    hipLaunchKernelGGL((flow_draw_fp32_kernel<F>), dim3(map_blocks(n)), dim3(256), 0, s,
                       (const bf16x8 *)frags, bias, A, stream_word, n, xs, ws);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_flow_draw_fp32(int family, const void *frags, const float *bias,
                                 const VsArgs &A, uint32_t stream_word, uint32_t n, double *xs,
                                 double *ws, hipStream_t s) {
    if (n == 0) return hipSuccess;
    switch (family) {
    case MCUBES_OSCILLATORY: return launch_draw_f<MCUBES_OSCILLATORY>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_PRODUCT_PEAK: return launch_draw_f<MCUBES_PRODUCT_PEAK>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_CORNER_PEAK: return launch_draw_f<MCUBES_CORNER_PEAK>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_GAUSSIAN: return launch_draw_f<MCUBES_GAUSSIAN>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_C0: return launch_draw_f<MCUBES_C0>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_DISCONTINUOUS: return launch_draw_f<MCUBES_DISCONTINUOUS>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_ADDITION: return launch_draw_f<MCUBES_ADDITION>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_MIXTURE: return launch_draw_f<MCUBES_MIXTURE>(frags, bias, A, stream_word, n, xs, ws, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mcubes
