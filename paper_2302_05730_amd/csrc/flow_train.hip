// BF16 training of the flow on the matrix cores: the forward and backward
// pass of the weighted negative log-likelihood and the weight gradients in
// one kernel, and the fixed-order sum of the gradients with Adam's step.
//
// A workgroup of eight waves takes 256 samples, 32 to a wave: lane l works on
// sample l % 32 of its wave, the two lane halves on the two halves of every
// feature set (see flow_bf16.hip for how the products chain in registers).
// Two waves share a SIMD, so a wave's loads, barriers and products are covered
// by the other's splines; one 64-sample wave per SIMD waited 40% of its life.
//
// The weight gradients are products over samples, inputs^T deltas, and want
// eight consecutive samples of one feature per lane where the passes hold one
// sample's features: each layer's inputs and deltas go through an LDS tile
// [feature][sample] of the workgroup's 256 samples, one product at a time, and
// the waves share out its 32 x 32 or 16 x 16 blocks.  Nothing of the fields
// goes to memory (a step of 65,536 samples wrote 289 MB of them and read 311
// MB back); what does are h1 and h2 as operands, 128 BF16 values per sample
// and layer, between the passes, and each workgroup's gradient.  The gradient
// of 65,536 samples takes 186 us, every launch counted; as a pass of 194 us
// that stored the fields, a kernel of 93 us over them and five small launches
// it took 357.
//
// Rounding: weights and product operands BF16, biases, accumulation and
// splines FP32; the forward pass is value for value that of the sampling
// kernels' spline and encoding.
#include "flow_mfma.h"

namespace mcubes {

namespace {

using namespace flow;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The backward products run through the transposed weights in the same
// orientation (features = rows, samples = columns): dh2 = W3 draw, dh1 = W2
// d2, de = W1 d1.  Their fragments: through W3, 2 row tiles (hidden units) x 7
// K steps over the 99 spline outputs; through W2, 2 x 4; through W1, 3 row
// tiles (one coordinate's 32 bumps each) x 4; the last two in the K order of
// the accumulator registers, like the forward products.
constexpr int B3T = 2, B3K = 7, B2T = 2, B2K = 4, B1T = 3, B1K = 4;
constexpr int OFF_B3F = 0, OFF_B2F = OFF_B3F + B3T * B3K, OFF_B1F = OFF_B2F + B2T * B2K;
constexpr int BFRAGS = OFF_B1F + B1T * B1K;  // 34

// K order of the product through W3: the outputs as the lanes hold them.  The
// low lane half runs the spline of mapped coordinate 0, the high half that of
// 1, both that of 2: steps 0-3 take eight outputs of each half's own
// coordinate, steps 4 and 5 coordinate 2's first 32 split between the halves,
// step 6 the three 33rd outputs.  -1: padding.
__host__ __device__ constexpr int bwd_out(int ks, int h, int e) {
    if (ks < 4) return RAW * h + 8 * ks + e;
    if (ks < 6) return 2 * RAW + 16 * (ks - 4) + 8 * h + e;
    if (e == 0) return RAW * h + RAW - 1;
    return e == 1 && h == 0 ? 3 * RAW - 1 : -1;
}

// Row order of the product through W1: row r of a lane half's accumulators is
// the bump the half encodes as element r % 8 of its octet r / 8.
__host__ __device__ constexpr int bump_row(int row) {
    const int r = 4 * (row / 8) + row % 4, h = (row / 4) % 2;
    return 16 * (r / 8) + 8 * h + r % 8;
}

// element e of backward fragment slot gid = (layer, fragment, lane)
__device__ __forceinline__ int bwd_param(int gid, int e) {
    const int lane = gid % 64, fr = (gid / 64) % BFRAGS, l = gid / (64 * BFRAGS);
    const int row = lane % 32, h = lane / 32;
    if (fr < OFF_B2F) {
        const int t = fr / B3K, ks = fr % B3K, i = 32 * t + row, k = bwd_out(ks, h, e);
        return k >= 0 ? l * LP + OFF_W3 + i * OUT + k : -1;
    }
    if (fr < OFF_B1F) {
        const int q = fr - OFF_B2F, t = q / B2K, ks = q % B2K, i = 32 * t + row;
        return l * LP + OFF_W2 + i * HID + acc_feature(ks / 2, 8 * (ks % 2) + e, h);
    }
    const int q = fr - OFF_B1F, t = q / B1K, ks = q % B1K, r = 32 * t + bump_row(row);
    return l * LP + OFF_W1 + r * HID + acc_feature(ks / 2, 8 * (ks % 2) + e, h);
}

__device__ __forceinline__ void pack_bwd(int gid, const float *__restrict__ theta,
                                         bf16x8 *__restrict__ frags) {
    if (gid >= L * BFRAGS * 64) return;
    float v[8];
    for (int e = 0; e < 8; ++e) {
        const int p = bwd_param(gid, e);
        v[e] = p >= 0 ? theta[p] : 0.0f;
    }
    frags[gid] = pack8(v);
}

// The inverse of the three maps: inv[3 p], inv[3 p + 1], inv[3 p + 2] = the
// BF16 element of the forward fragments, of the backward fragments and the
// bias entry that hold parameter p (-1 where none; the caller fills inv with
// -1 first).  Every weight sits in exactly one forward and one backward
// element, every bias in one bias entry, so the three are well defined.
__global__ void inverse_map_kernel(int *__restrict__ inv) {
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    const int nf = L * FRAGS * 64, nb = L * BFRAGS * 64;
    if (gid < nf) {
        for (int e = 0; e < 8; ++e) {
            const int p = fwd_param(gid, e);
            if (p >= 0) inv[3 * p] = 8 * gid + e;
        }
    } else if (gid < nf + nb) {
        const int g = gid - nf;
        for (int e = 0; e < 8; ++e) {
            const int p = bwd_param(g, e);
            if (p >= 0) inv[3 * p + 1] = 8 * g + e;
        }
    }
    if (gid < L * BIAS) {
        const int p = bias_param(gid);
        if (p >= 0) inv[3 * p + 2] = gid;
    }
}

// The end of a training step in one launch: the gradient's slice sum, the Adam
// step (as adam_kernel), and the new parameter written through the inverse map
// into both fragment sets and the bias array, the values prepare_kernel would
// write from the new theta.  The next step's pass then starts without
// repacking.
__global__ __launch_bounds__(kSumThreads) void sum_adam_pack_kernel(
    const float *__restrict__ part, int slices, float *__restrict__ theta, float *__restrict__ m,
    float *__restrict__ v, float *__restrict__ grad, float lr, float beta1, float beta2, float eps,
    float c1, float c2, const int *__restrict__ inv, uint16_t *__restrict__ frags,
    uint16_t *__restrict__ bfrags, float *__restrict__ bias) {
    __shared__ SumLds lds;
    float g;
    const int i = slice_sum(part, slices, lds, g);
    if (i < 0) return;
    grad[i] = g;
    const float t = adam_update(theta, m, v, i, g, lr, beta1, beta2, eps, c1, c2);
    const int pf = inv[3 * i], pb = inv[3 * i + 1], pz = inv[3 * i + 2];
    const uint16_t bits = __builtin_bit_cast(uint16_t, (__bf16)t);
    if (pf >= 0) frags[pf] = bits;
    if (pb >= 0) bfrags[pb] = bits;
    if (pz >= 0) bias[pz] = t;
}

// What a pass needs first, in one launch: forward and backward fragments and
// biases from theta (threads [0, nf) the forward ones), and in the last block,
// when wsum is not NULL, the sum of the n weights.
__global__ __launch_bounds__(1024) void prepare_kernel(
    const float *__restrict__ theta, bf16x8 *__restrict__ frags, float *__restrict__ bias,
    bf16x8 *__restrict__ bfrags, int nf, const double *__restrict__ w, int64_t n,
    double *__restrict__ wsum) {
    if (wsum && blockIdx.x == gridDim.x - 1) {
        __shared__ double red[16];
        const double a = block_sum(w, n, red);
        if (threadIdx.x == 0) *wsum = a;
        return;
    }
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    if (gid < nf)
        pack_fwd(gid, theta, frags, bias);
    else
        pack_bwd(gid - nf, theta, bfrags);
}

// ---- splines

// spline_setup as the sampling kernels have it, value for value (the hardware's
// exponential, the halves of Z's terms left to the end).
__device__ __forceinline__ void normalise(const float raw[RAW], Spline &s) {
    float mw = raw[0], mv = raw[BINS];
#pragma unroll
    for (int i = 1; i < BINS; ++i) mw = fmaxf(mw, raw[i]);
#pragma unroll
    for (int i = 1; i <= BINS; ++i) mv = fmaxf(mv, raw[BINS + i]);
    float sw = 0.0f, Z = 0.0f;
#pragma unroll
    for (int i = 0; i < BINS; ++i) {
        s.W[i] = __expf(raw[i] - mw);
        sw += s.W[i];
    }
    const float inv = div_normal(1.0f, sw);
#pragma unroll
    for (int i = 0; i < BINS; ++i) s.W[i] *= inv;
#pragma unroll
    for (int i = 0; i <= BINS; ++i) s.E[i] = __expf(raw[BINS + i] - mv);
#pragma unroll
    for (int i = 0; i < BINS; ++i) Z += (s.E[i] + s.E[i + 1]) * s.W[i];
    s.Z = 0.5f * Z;
    const float iz = div_normal(1.0f, s.Z);
#pragma unroll
    for (int i = 0; i <= BINS; ++i) s.V[i] = s.E[i] * iz;
}

// The bin of u (the last with left edge <= u): its edge X, CDF value A left of
// it, width, heights and index, by halving, on prefixes in the order of a scan.
__device__ __forceinline__ Bin locate(const Spline &s, float u) {
    const float *Win = s.W, *Vin = s.V;
    float C = 0.0f, X = 0.0f, Cq[3], Xq[3];  // C: twice the CDF
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        C += (Vin[i] + Vin[i + 1]) * Win[i];
        X += Win[i];
        if (i % 4 == 3) {
            Cq[i / 4] = C;
            Xq[i / 4] = X;
        }
    }
    float W[8], V[9];
    bool in = Xq[1] <= u;
    int k = in ? 8 : 0;
    C = in ? Cq[1] : 0.0f;
    X = in ? Xq[1] : 0.0f;
    float Cm = in ? Cq[2] : Cq[0], Xm = in ? Xq[2] : Xq[0];
#pragma unroll
    for (int i = 0; i < 8; ++i) W[i] = in ? Win[8 + i] : Win[i];
#pragma unroll
    for (int i = 0; i <= 8; ++i) V[i] = in ? Vin[8 + i] : Vin[i];
    in = Xm <= u;
    k += in ? 4 : 0;
    C = in ? Cm : C;
    X = in ? Xm : X;
#pragma unroll
    for (int i = 0; i < 4; ++i) W[i] = in ? W[4 + i] : W[i];
#pragma unroll
    for (int i = 0; i <= 4; ++i) V[i] = in ? V[4 + i] : V[i];
    Cm = (C + (V[0] + V[1]) * W[0]) + (V[1] + V[2]) * W[1];
    Xm = (X + W[0]) + W[1];
    in = Xm <= u;
    k += in ? 2 : 0;
    C = in ? Cm : C;
    X = in ? Xm : X;
#pragma unroll
    for (int i = 0; i < 2; ++i) W[i] = in ? W[2 + i] : W[i];
#pragma unroll
    for (int i = 0; i <= 2; ++i) V[i] = in ? V[2 + i] : V[i];
    Cm = C + (V[0] + V[1]) * W[0];
    Xm = X + W[0];
    in = Xm <= u;
    k += in ? 1 : 0;
    C = in ? Cm : C;
    X = in ? Xm : X;
    return Bin{X, 0.5f * C, in ? W[1] : W[0], in ? V[1] : V[0], in ? V[2] : V[1], k};
}

// spline_forward in the bin of u; returns the density
__device__ __forceinline__ float map_in_bin(const Bin &b, float u, float &y) {
    const float a = fminf(fmaxf(div_normal(u - b.X, b.W), 0.0f), 1.0f);
    const float dV = b.V1 - b.V0;
    y = b.A + b.W * (a * b.V0 + 0.5f * a * a * dV);
    return b.V0 + a * dV;
}

// y = the mapped u; returns log2 of the density
__device__ __forceinline__ float spline_map(const float raw[RAW], float u, float &y) {
    Spline s;
    normalise(raw, s);
    return __builtin_amdgcn_logf(map_in_bin(locate(s, u), u, y));
}

// Derivatives at u, given gy = dL/dy and c = dL/dlog pdf.
__device__ __forceinline__ void spline_grad(const float raw[RAW], float u, float gy, float c,
                                            float graw[RAW], float &gu) {
    Spline s;
    normalise(raw, s);
    const Bin b = locate(s, u);
    float y;
    const float pdf = map_in_bin(b, u, y);
    spline_backward(s, b, u, gy, c / pdf, graw, gu);
}

// ---- the pass

constexpr int kWaves = 8, kThreads = kWaves * 64, kPass = kWaves * 32;  // samples per pass
constexpr int kMaxBlocks = 256;
constexpr int H_OPS = G2K + G3K;                   // stored operands of h1 and h2
constexpr int SLOT = G3T * G3K + BFRAGS;           // 50 fragments >= FRAGS
constexpr int TROWS = HID + OUT, TLD = kPass + 8;  // tile: rows, padded row length
static_assert(TROWS >= 2 * HID && TROWS >= IN + HID, "tile rows");

// Copies FR fragments (FR x 64 lanes of 16 bytes) from src to dst, the
// workgroup's threads striding over them, every load issued before the first
// LDS write.
template <int FR>
__device__ __forceinline__ void stage_frags(bf16x8 *dst, const bf16x8 *__restrict__ src) {
    constexpr int N = FR * 64, PER = (N + kThreads - 1) / kThreads;
    bf16x8 v[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = threadIdx.x + k * kThreads;
        if (i < N) v[k] = src[i];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = threadIdx.x + k * kThreads;
        if (i < N) dst[i] = v[k];
    }
}

// A value of each half for both: lo = the low half's a, hi = the high half's.
__device__ __forceinline__ void both_halves(float a, float &lo, float &hi) { columns(a, lo, hi); }

// acc[t] += F[t][ks] x[ks] over T row tiles and K steps
template <int T, int K>
__device__ __forceinline__ void product(const bf16x8 *F, const bf16x8 (&x)[K], f32x16 (&acc)[T]) {
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = f32x16{};
#pragma unroll
    for (int ks = 0; ks < K; ++ks)
#pragma unroll
        for (int t = 0; t < T; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(F[(t * K + ks) * 64], x[ks], acc[t],
                                                             0, 0, 0);
}

// The third product, and every lane given the 33 outputs of its own
// coordinates of its sample, biases added: the low half coordinate 0's and the
// high half 1's in ra, coordinate 2's in rb on both.
__device__ __forceinline__ void outputs(const bf16x8 *F, const bf16x8 (&h2)[G3K],
                                        const float *__restrict__ B3, int h, float ra[RAW],
                                        float rb[RAW]) {
    f32x16 o[G3T];
    product<G3T, G3K>(F, h2, o);
    const float *Ba = B3 + 32 * h;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int k = 8 * (r / 4) + r % 4;  // raw index of half 0's row; half 1's is k + 4
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[0][r]),
                                                        __float_as_uint(o[1][r]), false, false);
        ra[k] = __uint_as_float(s[0]) + Ba[r];
        ra[k + 4] = __uint_as_float(s[1]) + Ba[16 + r];
        const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[2][r]),
                                                        __float_as_uint(o[2][r]), false, false);
        rb[k] = __uint_as_float(q[0]) + B3[64 + r];
        rb[k + 4] = __uint_as_float(q[1]) + B3[64 + 16 + r];
    }
    float l0, l1, l2, unused;
    both_halves(o[3][0], l0, unused);
    both_halves(o[3][1], l1, unused);
    both_halves(o[3][2], l2, unused);
    ra[RAW - 1] = (h ? l1 : l0) + (h ? B3[96 + 1] : B3[96]);
    rb[RAW - 1] = l2 + B3[96 + 2];
}

// the operand's elements (bf16 bits) of the lane's sample into tile rows
// row(i), column col
__device__ __forceinline__ uint16_t elem(const bf16x8 &v, int i) {
    const __bf16 e = v[i];
    return __builtin_bit_cast(uint16_t, e);
}

// rows of a hidden layer's operands (accumulator order)
__device__ __forceinline__ void hidden_rows(uint16_t *T, const bf16x8 (&op)[4], int h, int col) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int i = 0; i < 8; ++i)
            T[acc_feature(ks / 2, 8 * (ks % 2) + i, h) * TLD + col] = elem(op[ks], i);
}

// acc where the stored activation (>= 0) is not zero, as the four operands of
// the next product (an activation below 2^-134 is stored as zero, adds nothing
// to the product after it and counts as off)
__device__ __forceinline__ void masked_ops(const f32x16 (&acc)[2], const bf16x8 (&act)[4],
                                           bf16x8 (&op)[4]) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        float v[8];
        const u32x4 a = __builtin_bit_cast(u32x4, act[ks]);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t bits = i % 2 ? a[i / 2] >> 16 : a[i / 2] & 0xffffu;
            v[i] = bits ? acc[ks / 2][8 * (ks % 2) + i] : 0.0f;
        }
        op[ks] = pack8(v);
    }
}

__device__ __forceinline__ bf16x8 tile8(const uint16_t *T, int row, int s) {
    typedef uint16_t u16x8 __attribute__((ext_vector_type(8), may_alias));
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(T + row * TLD + s));
}

__device__ __forceinline__ bf16x8 ones8() {
    const float v[8] = {1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f};
    return pack8(v);
}

// the workgroup's partial gradient: set in its first pass, added to in later ones
__device__ __forceinline__ void put(float *G, float v, bool add) { *G = add ? *G + v : v; }

// Gradient of W3 and b3 from the tile (rows 0-63 h2, 64-162 the deltas): wave
// w the 32 x 32 block of rows 32 (w % 2) and columns 32 (w / 2) (the last of
// three columns); the column sums by a product with ones.
__device__ __forceinline__ void grad_w3(const uint16_t *T, float *G, int wave, int lane,
                                        bool add) {
    const int idx = lane & 31, h = lane >> 5, rt = wave & 1, ct = wave >> 1, C = 32 * ct + idx;
    const bool live = C < OUT;
    const int ra = 32 * rt + idx, rb = HID + (live ? C : 0);
    const bf16x8 one = ones8();
    f32x16 acc = f32x16{}, sum = f32x16{};
#pragma unroll 4
    for (int s = 0; s < kPass; s += 16) {
        const bf16x8 a = tile8(T, ra, s + 8 * h), b = tile8(T, rb, s + 8 * h);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
        if (rt == 0) sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(one, b, sum, 0, 0, 0);
    }
    if (!live) return;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        put(G + OFF_W3 + (32 * rt + acc_feature(0, r, h)) * OUT + C, acc[r], add);
    if (rt == 0 && h == 0) put(G + OFF_B3 + C, sum[0], add);
}

// Gradient of a 64-column matrix and its biases from the tile (rows [0, 32 RT)
// the inputs, then 64 deltas): wave w the 16 x 16 blocks of columns 16 (w % 4)
// and rows 16 (RT (w / 4) + 0 .. RT - 1).
template <int RT>
__device__ __forceinline__ void grad_hidden(const uint16_t *T, float *GW, float *GB, int wave,
                                            int lane, bool add) {
    const int idx = lane & 15, g = lane >> 4, C = 16 * (wave & 3) + idx, r0 = RT * (wave >> 2);
    const bf16x8 one = ones8();
    f32x4 acc[RT], sum = f32x4{};
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = f32x4{};
#pragma unroll 4
    for (int s = 0; s < kPass; s += 32) {
        const bf16x8 b = tile8(T, 32 * RT + C, s + 8 * g);
#pragma unroll
        for (int t = 0; t < RT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                tile8(T, 16 * (r0 + t) + idx, s + 8 * g), b, acc[t], 0, 0, 0);
        if (r0 == 0) sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(one, b, sum, 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            put(GW + (16 * (r0 + t) + 4 * g + r) * HID + C, acc[t][r], add);
    if (r0 == 0 && g == 0) put(GB + C, sum[0], add);
}

// Forward and backward pass and weight gradients.  loss += sum c log q with c =
// -w / sum w; part[block] <- the block's gradient.  Lanes past n work on a copy
// of the last sample with c = 0, which adds nothing to any sum.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void
train_bf16_kernel(const bf16x8 *__restrict__ frags, const bf16x8 *__restrict__ bfrags,
                  const float *__restrict__ bias, const double *__restrict__ x,
                  const double *__restrict__ w, int64_t n, const double *__restrict__ wsum,
                  float *__restrict__ part, bf16x8 *__restrict__ ops, double *__restrict__ loss) {
    __shared__ bf16x8 slot[SLOT * 64];
    __shared__ __align__(16) uint16_t T[TROWS * TLD];
    __shared__ float us[L][D][kPass];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane >> 5;
    const int col = 32 * wave + (lane & 31);  // the lane's sample in the workgroup
    float *G = part + (int64_t)blockIdx.x * PARAMS;
    const int64_t groups = (n + kPass - 1) / kPass * kWaves;
    double lsum = 0.0;
    bool add = false;
    for (int64_t base = (int64_t)blockIdx.x * kPass; base < n;
         base += (int64_t)gridDim.x * kPass) {
        const bool live = base + col < n;
        const int64_t s = live ? base + col : n - 1;
        // this wave's stored operands: [layer][group of 32 samples][operand][lane]
        bf16x8 *mine = ops + (base / 32 + wave) * H_OPS * 64 + lane;
        float u[D];
#pragma unroll
        for (int j = 0; j < D; ++j) u[j] = (float)x[s * D + j];
        const float c = live ? (float)(-w[s] / *wsum) : 0.0f;
        float lq = 0.0f;
        // ---- forward, x -> z
#pragma unroll 1
        for (int l = 0; l < L; ++l) {
#pragma unroll
            for (int j = 0; j < D; ++j) us[l][j][col] = u[j];
            __syncthreads();  // every wave is done with the previous fragments
            stage_frags<FRAGS>(slot, frags + (size_t)l * FRAGS * 64);
            __syncthreads();
            const bf16x8 *F = slot + lane;
            const float *Bs = bias + l * BIAS + h * 16;
            bf16x8 *keep = mine + (int64_t)l * groups * H_OPS * 64;
            bf16x8 e[G1K];
#pragma unroll
            for (int ks = 0; ks < G1K; ++ks) {
                float v[8];
                blob8(getu(u, a_idx(l, ks / 2)), 16 * (ks & 1) + 8 * h, v);
                e[ks] = pack8(v);
            }
            f32x16 acc[2];
            bf16x8 h1[G2K], h2[G3K];
            product<G1T, G1K>(F + OFF_G1 * 64, e, acc);
            relu_ops(acc, Bs + BOFF_1, h1);
#pragma unroll
            for (int ks = 0; ks < G2K; ++ks) keep[ks * 64] = h1[ks];
            product<G2T, G2K>(F + OFF_G2 * 64, h1, acc);
            relu_ops(acc, Bs + BOFF_2, h2);
#pragma unroll
            for (int ks = 0; ks < G3K; ++ks) keep[(G2K + ks) * 64] = h2[ks];
            float ra[RAW], rb[RAW];
            outputs(F + OFF_G3 * 64, h2, bias + l * BIAS + BOFF_3, h, ra, rb);
            const int j0 = b_idx(l, 0), j1 = b_idx(l, 1), j2 = b_idx(l, 2);
            float y, y0, y1, y2;
            lq += spline_map(ra, h ? getu(u, j1) : getu(u, j0), y);
            both_halves(y, y0, y1);
            const float d2 = spline_map(rb, getu(u, j2), y2);
            lq += h ? 0.0f : d2;
            setu(u, j0, y0);
            setu(u, j1, y1);
            setu(u, j2, y2);
        }
        lsum += (double)c * (double)(lq * 0.69314718055994530942f);
        // ---- backward; g = dL/du at the output of the current layer
        float g[D];
#pragma unroll
        for (int j = 0; j < D; ++j) g[j] = 0.0f;
#pragma unroll 1
        for (int l = L - 1; l >= 0; --l) {
            const bf16x8 *kept = mine + (int64_t)l * groups * H_OPS * 64;
            float *Gl = G + l * LP;
            bf16x8 h2[G3K];
#pragma unroll
            for (int ks = 0; ks < G3K; ++ks) h2[ks] = kept[(G2K + ks) * 64];
            float ul[D];
#pragma unroll
            for (int j = 0; j < D; ++j) ul[j] = us[l][j][col];
            __syncthreads();  // done with the previous fragments and tile
            stage_frags<G3T * G3K>(slot, frags + ((size_t)l * FRAGS + OFF_G3) * 64);
            stage_frags<BFRAGS>(slot + G3T * G3K * 64, bfrags + (size_t)l * BFRAGS * 64);
            __syncthreads();
            // spline deltas, as operands of the product through W3 and as rows
            // (after the 64 of h2) of the tile
            bf16x8 X[B3K];
            const int j0 = b_idx(l, 0), j1 = b_idx(l, 1), j2 = b_idx(l, 2);
            {
                float ra[RAW], rb[RAW], ga[RAW], gb[RAW], gu, gu0, gu1, gu2;
                outputs(slot + lane, h2, bias + l * BIAS + BOFF_3, h, ra, rb);
                spline_grad(ra, h ? getu(ul, j1) : getu(ul, j0),
                                    h ? getu(g, j1) : getu(g, j0), c, ga, gu);
                both_halves(gu, gu0, gu1);
                uint16_t *rows = T + (HID + RAW * h) * TLD + col;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    X[ks] = pack8(ga + 8 * ks);
#pragma unroll
                    for (int i = 0; i < 8; ++i) rows[(8 * ks + i) * TLD] = elem(X[ks], i);
                }
                spline_grad(rb, getu(ul, j2), getu(g, j2), c, gb, gu2);
                rows = T + (HID + 2 * RAW + 8 * h) * TLD + col;
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    float v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = h ? gb[16 * ks + 8 + i] : gb[16 * ks + i];
                    X[4 + ks] = pack8(v);
#pragma unroll
                    for (int i = 0; i < 8; ++i) rows[(16 * ks + i) * TLD] = elem(X[4 + ks], i);
                }
                const float v[8] = {ga[RAW - 1], h ? 0.0f : gb[RAW - 1], 0.0f, 0.0f,
                                    0.0f, 0.0f, 0.0f, 0.0f};
                X[6] = pack8(v);
                T[(HID + RAW * h + RAW - 1) * TLD + col] = elem(X[6], 0);
                if (h == 0) T[(HID + 3 * RAW - 1) * TLD + col] = elem(X[6], 1);
                setu(g, j0, gu0);
                setu(g, j1, gu1);
                setu(g, j2, gu2);
            }
            hidden_rows(T, h2, h, col);
            const bf16x8 *Br = slot + G3T * G3K * 64 + lane;
            f32x16 acc[2];
            bf16x8 h1[G2K], Y[B2K], Z[B1K];
#pragma unroll
            for (int ks = 0; ks < G2K; ++ks) h1[ks] = kept[ks * 64];
            // through W3 and the second ReLU
            product<B3T, B3K>(Br + OFF_B3F * 64, X, acc);
            masked_ops(acc, h2, Y);
            __syncthreads();
            grad_w3(T, Gl, wave, lane, add);
            __syncthreads();
            hidden_rows(T, h1, h, col);
            hidden_rows(T + HID * TLD, Y, h, col);
            // through W2 and the first ReLU
            product<B2T, B2K>(Br + OFF_B2F * 64, Y, acc);
            masked_ops(acc, h1, Z);
            __syncthreads();
            grad_hidden<2>(T, Gl + OFF_W2, Gl + OFF_B2, wave, lane, add);
            __syncthreads();
            hidden_rows(T + IN * TLD, Z, h, col);
            // through W1 to the one-blob inputs, then through the encoding, one
            // conditioning coordinate at a time: de_k/du = -32 e_k t_k
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                const float ua = getu(ul, a_idx(l, a));
                f32x16 d = f32x16{};
#pragma unroll
                for (int ks = 0; ks < B1K; ++ks)
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        Br[(OFF_B1F + a * B1K + ks) * 64], Z[ks], d, 0, 0, 0);
                float sum = 0.0f, half = -0.5f - 8.0f * (float)h;
                asm volatile("" : "+v"(half));  // 16 sums of it would be kept for the next a
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    // (directly: the forward pass's recurrence is off by up to 5e-6)
                    float e[8];
                    const int k0 = 16 * o + 8 * h;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float t = __fmaf_rn(ua, (float)BLOBS, half - (float)(16 * o + i));
                        e[i] = exp_bounded(-0.5f * t * t);
                        sum = __fmaf_rn(d[8 * o + i], e[i] * t, sum);
                    }
                    const bf16x8 eb = pack8(e);
#pragma unroll
                    for (int i = 0; i < 8; ++i) T[(32 * a + k0 + i) * TLD + col] = elem(eb, i);
                }
                sum *= -(float)BLOBS;
                sum += __shfl_xor(sum, 32);
                const int j = a_idx(l, a);
                setu(g, j, getu(g, j) + sum);
            }
            __syncthreads();
            grad_hidden<3>(T, Gl + OFF_W1, Gl + OFF_B1, wave, lane, add);
        }
        add = true;
    }
    const double v = wave_sum(lsum);
    if (lane == 0) unsafeAtomicAdd(loss, v);
}

int train_blocks(int64_t n, int cus) {
    const int64_t blocks = (n + kPass - 1) / kPass;
    const int64_t cap = cus > 0 && cus < kMaxBlocks ? cus : kMaxBlocks;
    return (int)(blocks < cap ? blocks : cap);
}

// floats of the blocks' partial gradients, a multiple of 4 so that the
// operands behind them are aligned
int64_t part_floats(int64_t n) {
    const int64_t f = (int64_t)train_blocks(n, kMaxBlocks) * PARAMS;
    return (f + 3) / 4 * 4;
}

}  // namespace

int64_t flow_bf16_bwd_frag_bytes() { return (int64_t)L * BFRAGS * 64 * sizeof(bf16x8); }

// the blocks' partial gradients, then h1 and h2 of every sample and layer
int64_t flow_bf16_train_floats(int64_t n) {
    return part_floats(n) + (n + kPass - 1) / kPass * kWaves * L * H_OPS * 64 * 4;
}

hipError_t launch_flow_train_bf16(const float *theta, void *frags, void *bfrags, float *bias,
                                  const double *x, const double *w, int64_t n, const double *wsum,
                                  double *own_wsum, float *scratch, double *loss, int cus,
                                  bool pack, hipStream_t s) {
    if (pack) {
        // the forward part covers the bias entries too (L BIAS < L FRAGS 64)
        const int nf = L * FRAGS * 64, nb = L * BFRAGS * 64;
        const int blocks = (nf + nb + 1023) / 1024;
        hipLaunchKernelGGL(prepare_kernel, dim3(blocks + (wsum ? 0 : 1)), dim3(1024), 0, s, theta,
                           (bf16x8 *)frags, bias, (bf16x8 *)bfrags, nf, w, n,
                           wsum ? nullptr : own_wsum);
    }
    hipLaunchKernelGGL(train_bf16_kernel, dim3(train_blocks(n, cus)), dim3(kThreads), 0, s,
                       (const bf16x8 *)frags, (const bf16x8 *)bfrags, bias, x, w, n,
                       wsum ? wsum : own_wsum, scratch, (bf16x8 *)(scratch + part_floats(n)), loss);
    return hipGetLastError();
}

hipError_t launch_flow_grad_bf16(const float *scratch, int64_t n, int cus, float *grad,
                                 double *wide, hipStream_t s) {
    return launch_flow_wgrad_sum(scratch, train_blocks(n, cus), grad, wide, s);
}

int64_t flow_bf16_inverse_map_ints() { return 3 * (int64_t)PARAMS; }

hipError_t launch_flow_inverse_map(int *inv, hipStream_t s) {
    const int threads = L * (FRAGS + BFRAGS) * 64;
    hipLaunchKernelGGL(inverse_map_kernel, dim3((threads + 255) / 256), dim3(256), 0, s, inv);
    return hipGetLastError();
}

hipError_t launch_flow_grad_adam_bf16(const float *scratch, int64_t n, int cus, float *theta,
                                      float *m, float *v, float *grad, float lr, float beta1,
                                      float beta2, float eps, float c1, float c2, const int *inv,
                                      void *frags, void *bfrags, float *bias, hipStream_t s) {
    hipLaunchKernelGGL(sum_adam_pack_kernel, dim3(kSumBlocks), dim3(kSumThreads), 0, s, scratch,
                       train_blocks(n, cus), theta, m, v, grad, lr, beta1, beta2, eps, c1, c2, inv,
                       (uint16_t *)frags, (uint16_t *)bfrags, bias);
    return hipGetLastError();
}

}  // namespace mcubes
