// The flow on the BF16 matrix cores (gfx950 v_mfma_f32_32x32x16_bf16, FP32
// accumulation): sampling and the flow-mapped iteration (the proposal's hot
// loop).
//
// A wave carries 64 samples, one per lane for the per-sample work (Philox,
// spline inversion, integrand), and runs each conditioner as three chained
// matrix products in transposed form, out^T = W^T in^T: features are the
// matrix rows (M), the 64 samples two blocks of 32 columns (N).  With that
// orientation the accumulator of one product (lane l holds column l % 32 and
// rows 8 (r/4) + 4 (l/32) + r%4 of a 32-row tile, r = 0..15) is, after bias,
// ReLU and rounding to BF16, already the B operand of the next product (lane
// l holds K values 8 (l/32) .. +7 of column l % 32) provided the K order of a
// step is the one the accumulator registers hold: the weight fragments are
// packed with that order, so activations never leave the registers.  The
// one-blob inputs of the first product are computed directly in operand
// order.  At the end, one v_permlane32_swap per accumulator register gives
// every lane all 99 outputs of its own sample.
//
// Rounding: weights and the inputs of every product are BF16 (round to
// nearest even), biases and accumulation FP32, the splines FP32, the
// integrand and weights FP64.
#include "flow_mfma.h"

namespace mcubes {

namespace {

using namespace flow;

__global__ void pack_kernel(const float *__restrict__ theta, bf16x8 *__restrict__ frags,
                            float *__restrict__ bias) {
    pack_fwd(blockIdx.x * blockDim.x + threadIdx.x, theta, frags, bias);
}

constexpr float kLn2 = 0.69314718055994530942f;

// spline_setup and spline_inverse in one, by the hardware's exponential (a few
// ulp, where the raw outputs carry the BF16 products' 1e-3) and logarithm: the
// bin is found by halving, where each level keeps half of the widths and heights
// (42 selects, against 75 and a compare per bin in a scan), on prefixes that are
// formed in the scan's order; the halves in the masses 0.5 (V_i + V_i+1) W_i
// are left to the end of each sum (exact: a power of two).  About 400 issue
// slots against 570.  y -> u, log2 of the density returned.
__device__ __forceinline__ float spline_inverse_raw(const float raw[RAW], float y, float &u) {
    float mw = raw[0], mv = raw[BINS];
#pragma unroll
    for (int i = 1; i < BINS; ++i) mw = fmaxf(mw, raw[i]);
#pragma unroll
    for (int i = 1; i <= BINS; ++i) mv = fmaxf(mv, raw[BINS + i]);
    float W[BINS], V[BINS + 1], sw = 0.0f, Z = 0.0f;
#pragma unroll
    for (int i = 0; i < BINS; ++i) {
        W[i] = __expf(raw[i] - mw);
        sw += W[i];
    }
    const float inv = div_normal(1.0f, sw);
#pragma unroll
    for (int i = 0; i < BINS; ++i) W[i] *= inv;
#pragma unroll
    for (int i = 0; i <= BINS; ++i) V[i] = __expf(raw[BINS + i] - mv);
#pragma unroll
    for (int i = 0; i < BINS; ++i) Z += (V[i] + V[i + 1]) * W[i];
    const float iz = div_normal(1.0f, 0.5f * Z);
#pragma unroll
    for (int i = 0; i <= BINS; ++i) V[i] *= iz;
    // C: twice the CDF at the vertices, X: the vertices; at 4, 8 and 12
    float C = 0.0f, X = 0.0f, Cq[3], Xq[3];
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        C += (V[i] + V[i + 1]) * W[i];
        X += W[i];
        if (i % 4 == 3) {
            Cq[i / 4] = C;
            Xq[i / 4] = X;
        }
    }
    const float t = y + y;
    bool in = Cq[1] <= t;
    C = in ? Cq[1] : 0.0f;
    X = in ? Xq[1] : 0.0f;
    float Cm = in ? Cq[2] : Cq[0], Xm = in ? Xq[2] : Xq[0];
#pragma unroll
    for (int i = 0; i < 8; ++i) W[i] = in ? W[8 + i] : W[i];
#pragma unroll
    for (int i = 0; i <= 8; ++i) V[i] = in ? V[8 + i] : V[i];
    in = Cm <= t;
    C = in ? Cm : C;
    X = in ? Xm : X;
#pragma unroll
    for (int i = 0; i < 4; ++i) W[i] = in ? W[4 + i] : W[i];
#pragma unroll
    for (int i = 0; i <= 4; ++i) V[i] = in ? V[4 + i] : V[i];
    Cm = (C + (V[0] + V[1]) * W[0]) + (V[1] + V[2]) * W[1];
    Xm = (X + W[0]) + W[1];
    in = Cm <= t;
    C = in ? Cm : C;
    X = in ? Xm : X;
#pragma unroll
    for (int i = 0; i < 2; ++i) W[i] = in ? W[2 + i] : W[i];
#pragma unroll
    for (int i = 0; i <= 2; ++i) V[i] = in ? V[2 + i] : V[i];
    Cm = C + (V[0] + V[1]) * W[0];
    Xm = X + W[0];
    in = Cm <= t;
    C = in ? Cm : C;
    X = in ? Xm : X;
    const float Wb = in ? W[1] : W[0], V0 = in ? V[1] : V[0], V1 = in ? V[2] : V[1];
    const float r = y - 0.5f * C, dV = V1 - V0;
    const float disc = fmaxf(V0 * V0 + div_normal(2.0f * dV * r, Wb), 0.0f);
    const float den = Wb * (V0 + sqrtf(disc));
    float a = den > 0.0f ? div_normal(2.0f * r, den) : 0.0f;
    a = fminf(fmaxf(a, 0.0f), 1.0f);
    u = X + a * Wb;
    return __builtin_amdgcn_logf(V0 + a * dV);
}

// 64 samples through the inverse flow: lane s holds sample s in u[] and
// returns log q.  All 64 lanes must be active.
//
// Bound by the vector ALU (the splines' exponentials and selects, the bumps,
// the rounding between products), not by the matrix cores.  The third
// product runs one row tile at a time, a coordinate's 32 outputs (the 33rds
// first, in a tile of their own), so 32 accumulators live instead of 128 and
// three waves fit a SIMD where one did: while one waits for its fragments or
// its matrix products the others' splines issue.  With the cheaper spline and
// rounding a 2^24-sample iteration takes 4.50 ms (7.00 before; about 2,400
// issue slots per layer, exponentials counted as four, which is 85% of the
// time), 300,000 samples 106 us (186).  Four waves (128 registers, more
// spills) take 4.72 ms and 122 us.
__device__ __forceinline__ float sample_wave(const bf16x8 *__restrict__ frags,
                                             const float *__restrict__ bias, float u[D]) {
    const int lane = threadIdx.x & 63, h = lane >> 5;
    float lq = 0.0f;
#pragma unroll 1
    for (int l = L - 1; l >= 0; --l) {
        const bf16x8 *F = frags + (size_t)l * FRAGS * 64 + lane;
        const float *Bs = bias + l * BIAS + h * 16;
        f32x16 acc[2][2];  // [sample block][row tile]
#pragma unroll
        for (int t = 0; t < G1T; ++t) acc[0][t] = acc[1][t] = f32x16{};
#pragma unroll
        for (int a = 0; a < NA; ++a) {
            float ua[2];
            columns(getu(u, a_idx(l, a)), ua[0], ua[1]);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                bf16x8 op[2];
#pragma unroll
                for (int sb = 0; sb < 2; ++sb) {
                    float e[8];
                    blob8(ua[sb], 16 * k + 8 * h, e);
                    op[sb] = pack8(e);
                }
#pragma unroll
                for (int t = 0; t < G1T; ++t) {
                    const bf16x8 f = F[(OFF_G1 + t * G1K + 2 * a + k) * 64];
#pragma unroll
                    for (int sb = 0; sb < 2; ++sb)
                        acc[sb][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, op[sb], acc[sb][t],
                                                                             0, 0, 0);
                }
            }
        }
        bf16x8 h1[2][G2K], h2[2][G3K];
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) relu_ops(acc[sb], Bs + BOFF_1, h1[sb]);
#pragma unroll
        for (int t = 0; t < G2T; ++t) acc[0][t] = acc[1][t] = f32x16{};
#pragma unroll
        for (int ks = 0; ks < G2K; ++ks)
#pragma unroll
            for (int t = 0; t < G2T; ++t) {
                const bf16x8 f = F[(OFF_G2 + t * G2K + ks) * 64];
#pragma unroll
                for (int sb = 0; sb < 2; ++sb)
                    acc[sb][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, h1[sb][ks], acc[sb][t],
                                                                         0, 0, 0);
            }
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) relu_ops(acc[sb], Bs + BOFF_2, h2[sb]);
        // one row tile of the third product, both sample blocks
        const auto third = [&](int t, f32x16 (&o)[2]) {
            o[0] = o[1] = f32x16{};
#pragma unroll
            for (int ks = 0; ks < G3K; ++ks) {
                const bf16x8 f = F[(OFF_G3 + t * G3K + ks) * 64];
#pragma unroll
                for (int sb = 0; sb < 2; ++sb)
                    o[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, h2[sb][ks], o[sb], 0, 0, 0);
            }
        };
        // hands every lane its own sample: lanes 32..63 of block 0 <-> lanes
        // 0..31 of block 1; afterwards o[0] holds the rows of lane half 0 and
        // o[1] those of half 1, biases added
        const float *B3 = bias + l * BIAS + BOFF_3;
        const auto own = [&](f32x16 (&o)[2], int t, int r) {
            const auto sw = __builtin_amdgcn_permlane32_swap(
                __float_as_uint(o[0][r]), __float_as_uint(o[1][r]), false, false);
            o[0][r] = __uint_as_float(sw[0]) + B3[32 * t + r];
            o[1][r] = __uint_as_float(sw[1]) + B3[32 * t + 16 + r];
        };
        float last[NB];
        {
            f32x16 o[2];
            third(NB, o);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                own(o, NB, b);
                last[b] = o[0][b];
            }
        }
#pragma unroll 1
        for (int b = 0; b < NB; ++b) {
            f32x16 o[2];
            third(b, o);
#pragma unroll
            for (int r = 0; r < 16; ++r) own(o, b, r);
            float raw[RAW];
#pragma unroll
            for (int k = 0; k < RAW - 1; ++k) raw[k] = o[(k / 4) % 2][4 * (k / 8) + k % 4];
            raw[RAW - 1] = b == 0 ? last[0] : (b == 1 ? last[1] : last[2]);
            const int j = b_idx(l, b);
            float v;
            lq += spline_inverse_raw(raw, getu(u, j), v);
            setu(u, j, v);
        }
    }
    return lq * kLn2;
}

// three waves per SIMD (168 registers) in the kernels that run sample_wave
#define SAMPLING_WAVES __attribute__((amdgpu_waves_per_eu(3)))

__global__ __launch_bounds__(256) SAMPLING_WAVES void sample_bf16_kernel(
    const bf16x8 *__restrict__ frags, const float *__restrict__ bias,
    const double *__restrict__ z, int64_t n, double *__restrict__ x, double *__restrict__ logq) {
    map_samples([&](float u[D]) { return sample_wave(frags, bias, u); }, z, n, x, logq);
}

template <int F>
__global__ __launch_bounds__(256) SAMPLING_WAVES void flow_vsample_bf16_kernel(
    const bf16x8 *__restrict__ frags, const float *__restrict__ bias, const VsArgs A,
    uint32_t stream_word, double *__restrict__ partials, uint32_t *__restrict__ whist) {
    flow_iteration<F>([&](float u[D]) { return sample_wave(frags, bias, u); }, A, stream_word,
                      partials, whist);
}

template <int F>
__global__ __launch_bounds__(256) SAMPLING_WAVES void flow_draw_bf16_kernel(
    const bf16x8 *__restrict__ frags, const float *__restrict__ bias, const VsArgs A,
    uint32_t stream_word, uint32_t n, double *__restrict__ xs, double *__restrict__ ws) {
    draw_samples<F>([&](float u[D]) { return sample_wave(frags, bias, u); }, A, stream_word, n, xs,
                    ws);
}

template <int F>
hipError_t launch_bf16_f(const void *frags, const float *bias, const VsArgs &A,
                         uint32_t stream_word, double *partials, uint32_t *whist, int blocks,
                         hipStream_t s) {
    hipLaunchKernelGGL((flow_vsample_bf16_kernel<F>), dim3(blocks), dim3(256), 0, s,
                       (const bf16x8 *)frags, bias, A, stream_word, partials, whist);
    return hipGetLastError();
}

}  // namespace

int64_t flow_bf16_frag_bytes() { return (int64_t)L * FRAGS * 64 * sizeof(bf16x8); }
int64_t flow_bf16_bias_floats() { return (int64_t)L * BIAS; }

hipError_t launch_flow_pack_bf16(const float *theta, void *frags, float *bias, hipStream_t s) {
    const int n = L * FRAGS * 64;
    hipLaunchKernelGGL(pack_kernel, dim3((n + 255) / 256), dim3(256), 0, s, theta,
                       (bf16x8 *)frags, bias);
    return hipGetLastError();
}

template <int F>
hipError_t launch_draw_bf16_f(const void *frags, const float *bias, const VsArgs &A,
                              uint32_t stream_word, uint32_t n, double *xs, double *ws,
                              hipStream_t s) {
    int64_t blocks = ((int64_t)n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL((flow_draw_bf16_kernel<F>), dim3((unsigned)blocks), dim3(256), 0, s,
                       (const bf16x8 *)frags, bias, A, stream_word, n, xs, ws);
    return hipGetLastError();
}

hipError_t launch_flow_draw_bf16(int family, const void *frags, const float *bias,
                                 const VsArgs &A, uint32_t stream_word, uint32_t n, double *xs,
                                 double *ws, hipStream_t s) {
    if (n == 0) return hipSuccess;
    switch (family) {
    case MCUBES_OSCILLATORY: return launch_draw_bf16_f<MCUBES_OSCILLATORY>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_PRODUCT_PEAK: return launch_draw_bf16_f<MCUBES_PRODUCT_PEAK>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_CORNER_PEAK: return launch_draw_bf16_f<MCUBES_CORNER_PEAK>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_GAUSSIAN: return launch_draw_bf16_f<MCUBES_GAUSSIAN>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_C0: return launch_draw_bf16_f<MCUBES_C0>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_DISCONTINUOUS: return launch_draw_bf16_f<MCUBES_DISCONTINUOUS>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_ADDITION: return launch_draw_bf16_f<MCUBES_ADDITION>(frags, bias, A, stream_word, n, xs, ws, s);
    case MCUBES_MIXTURE: return launch_draw_bf16_f<MCUBES_MIXTURE>(frags, bias, A, stream_word, n, xs, ws, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_flow_sample_bf16(const void *frags, const float *bias, const double *z,
                                   int64_t n, double *x, double *logq, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(sample_bf16_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                       (const bf16x8 *)frags, bias, z, n, x, logq);
    return hipGetLastError();
}

hipError_t launch_flow_vsample_bf16(int family, const void *frags, const float *bias,
                                    const VsArgs &A, uint32_t stream_word, double *partials,
                                    uint32_t *whist, int blocks, hipStream_t s) {
    switch (family) {
    case MCUBES_OSCILLATORY: return launch_bf16_f<MCUBES_OSCILLATORY>(frags, bias, A, stream_word, partials, whist, blocks, s);
    case MCUBES_PRODUCT_PEAK: return launch_bf16_f<MCUBES_PRODUCT_PEAK>(frags, bias, A, stream_word, partials, whist, blocks, s);
    case MCUBES_CORNER_PEAK: return launch_bf16_f<MCUBES_CORNER_PEAK>(frags, bias, A, stream_word, partials, whist, blocks, s);
    case MCUBES_GAUSSIAN: return launch_bf16_f<MCUBES_GAUSSIAN>(frags, bias, A, stream_word, partials, whist, blocks, s);
    case MCUBES_C0: return launch_bf16_f<MCUBES_C0>(frags, bias, A, stream_word, partials, whist, blocks, s);
    case MCUBES_DISCONTINUOUS: return launch_bf16_f<MCUBES_DISCONTINUOUS>(frags, bias, A, stream_word, partials, whist, blocks, s);
    case MCUBES_ADDITION: return launch_bf16_f<MCUBES_ADDITION>(frags, bias, A, stream_word, partials, whist, blocks, s);
    case MCUBES_MIXTURE: return launch_bf16_f<MCUBES_MIXTURE>(frags, bias, A, stream_word, partials, whist, blocks, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mcubes
