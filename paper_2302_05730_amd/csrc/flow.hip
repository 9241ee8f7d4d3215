// FP32 kernels of the learned proposal: the training pass (forward, then the
// backward pass into per-sample scratch fields), in a cooperative form with
// eight waves per 64 samples; the weight gradients as sums over the samples;
// Adam; the FP32 flow-mapped m-Cubes iteration (cooperative for p dividing 64,
// else one thread per cube); and the export of one plain iteration's own
// samples and weights.
#include "flow_impl.h"
#include "stratum.h"
#include "vsample_impl.h"

namespace mcubes {

namespace {

using namespace flow;

// Cooperative form: a workgroup of CW waves takes CS = 64 samples.  The matrix
// products run on the matrix cores in FP32 (16 x 16 x 4: 16 output features by
// 16 samples, a step of four inputs), whose result is that of one fused
// multiply-add per input in ascending order, bit for bit: the arithmetic is
// that of one thread running one sample.  The rest has a lane per sample.
//
// A wave takes the sample tile q % 4 and every other feature tile from q / 4.
// Activations stay in LDS, a row of 64 samples per feature, its four groups
// of 16 permuted by swz(row), so that the rows 4 s .. 4 s + 3 of a step (read)
// and the rows 4 k + r of the result (written) fall into different banks;
// weights come from memory, 16 consecutive features by four inputs.
//
// As FMAs with scalar weights, two waves per SIMD waiting for them, the
// training pass took 495 us at 20011 samples (one workgroup on most CUs), and
// takes 223; a flow-mapped iteration of 2^21 samples 5.4 ms, now 4.3 (at two
// workgroups per CU: at one, which leaves the matrix cores idle while the
// splines run on three waves, 5.6).
constexpr int CW = 8, CS = 64, CT = CW * CS;

// Transposed weights for the backward products, per layer:
// W1T[HID][IN], W2T[HID][HID], W3T[OUT][HID].
constexpr int T1 = 0, T2 = T1 + HID * IN, T3 = T2 + HID * HID, LPT = T3 + OUT * HID;

constexpr int ROWS = (OUT + 3) / 4 * 4;  // inputs of the widest product, in whole steps

struct Coop {
    float X[ROWS * CS], Y[ROWS * CS];  // activations of the current product
    float U[L + 1][D * CS];            // input of each step, then the output
    float G[2][D * CS];                // dL/du (training)
    float LQ[L * NB * CS];             // log spline density per step and coordinate
};
static_assert(sizeof(Coop) <= 65536, "cooperative LDS");

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int swz(int row) { return ((row ^ (row >> 2)) & 3) << 4; }
__device__ __forceinline__ int at(int row, int sample) { return row * CS + (sample ^ swz(row)); }

// What a lane of wave q reads and writes of an LDS array: in a product the
// rows 4 s + lane / 16 of its sample, at read[s % 4] + 4 CS s; of a result
// tile t the rows 32 t + feature + r, at write[r] + 32 CS t.
struct Lane {
    int sample, feature, read[4], write[4];
};
__device__ __forceinline__ Lane lane_of(int q, int lane) {
    Lane T;
    const int k = lane >> 4;
    T.sample = 16 * (q & 3) + (lane & 15);
    T.feature = 16 * (q >> 2) + 4 * k;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        T.read[r] = at(4 * r + k, T.sample) - 4 * CS * r;
        T.write[r] = at(T.feature + r, T.sample);
    }
    return T;
}

// acc[t] = the 16 x 16 tile of features 32 t + 16 (q / 4) .. by the wave's 16
// samples: sum_i W[i ld + feature] in[i][sample], i ascending from 0 to NI.
// Rows from NI on are zeros in `in`; their weights are those of the last row.
// The weights of four steps are loaded ahead of their products.
template <int CNT, int NI>
__device__ __forceinline__ void gemm_tiles(const float *__restrict__ W, int ld, const float *in,
                                           int q, int lane, const Lane &T, f32x4 acc[CNT]) {
    constexpr int K = (NI + 3) / 4, C = 4;  // steps, and of a chunk
    const int k = lane >> 4;
    const float *w = W + k * ld + 16 * (q >> 2) + (lane & 15);
    float a[2][C][CNT];
    const auto load = [&](int s0, float (&v)[C][CNT]) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int s = s0 + c;
            if (s >= K) break;
            const int row = NI % 4 && s == K - 1 ? min(4 * s + k, NI - 1) - k : 4 * s;
#pragma unroll
            for (int t = 0; t < CNT; ++t) v[c][t] = w[row * ld + 32 * t];
        }
    };
#pragma unroll
    for (int t = 0; t < CNT; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    load(0, a[0]);
#pragma unroll
    for (int s0 = 0; s0 < K; s0 += C) {
        if (s0 + C < K) load(s0 + C, a[(s0 / C + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int s = s0 + c;
            if (s >= K) break;
            const float b = in[T.read[s & 3] + 4 * CS * s];
#pragma unroll
            for (int t = 0; t < CNT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[(s0 / C) & 1][c][t], b, acc[t], 0, 0, 0);
        }
    }
}

// A hidden layer's tiles: bias and ReLU into `out`; with SAVE into the fields
// sc of 64 samples (stride n) as well.  Returns the signs, 8 bits.
template <bool SAVE>
__device__ __forceinline__ uint32_t relu_tiles(const f32x4 acc[2], const float *__restrict__ bias,
                                               const Lane &T, float *out, float *__restrict__ sc,
                                               int64_t n) {
    uint32_t mask = 0;
    float *field = sc + T.feature * n + T.sample;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float h = fmaxf(acc[t][r] + bias[T.feature + 32 * t + r], 0.0f);
            out[T.write[r] + 32 * CS * t] = h;
            if (SAVE) {
                field[(32 * t + r) * n] = h;
                mask |= h > 0.0f ? 1u << (4 * t + r) : 0u;
            }
        }
    }
    return mask;
}

// The deltas of a hidden layer: its tiles where the unit was on.
__device__ __forceinline__ void mask_tiles(const f32x4 acc[2], uint32_t mask, const Lane &T,
                                           float *out, float *__restrict__ sc, int64_t n) {
    float *field = sc + T.feature * n + T.sample;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float d = mask >> (4 * t + r) & 1u ? acc[t][r] : 0.0f;
            out[T.write[r] + 32 * CS * t] = d;
            field[(32 * t + r) * n] = d;
        }
    }
}

// Signs of the hidden units of the wave's tiles, 8 bits per layer.
struct Signs {
    uint32_t h1 = 0, h2 = 0;
};

// One coupling layer (P = its parameters) at step `step`: U[step] -> U[step+1].
// With SAVE the layer's input, hidden activations and spline parameters go
// to the scratch fields sc of the workgroup's samples (stride n), and the
// signs of the hidden units to `signs`.
template <bool INVERSE, bool SAVE>
__device__ __forceinline__ void coop_layer(const float *__restrict__ P, int l, int step, int q,
                                           int lane, Coop &S, float *__restrict__ sc, int64_t n,
                                           Signs &signs) {
    const float *Uin = S.U[step];
    float *Uout = S.U[step + 1];
    // one-blob encoding of u_A, rows a BLOBS + k; 12 rows per wave
#pragma unroll
    for (int i = 0; i < IN / CW; ++i) {
        const int r = (IN / CW) * q + i;
        S.X[at(r, lane)] = blob(Uin[a_idx(l, r / BLOBS) * CS + lane], r % BLOBS);
    }
    if (q == CW - 1) {
#pragma unroll
        for (int j = 0; j < D; ++j)
            if (SAVE) sc[(FS_U + j) * n + lane] = Uin[j * CS + lane];
#pragma unroll
        for (int t = 0; t < NA; ++t) {
            const int a = a_idx(l, t);
            Uout[a * CS + lane] = Uin[a * CS + lane];
        }
    }
    __syncthreads();
    const Lane T = lane_of(q, lane);
    f32x4 acc[4];
    gemm_tiles<2, IN>(P + OFF_W1, HID, S.X, q, lane, T, acc);
    signs.h1 |= relu_tiles<SAVE>(acc, P + OFF_B1, T, S.Y, sc + FS_H1 * n, n) << (8 * l);
    __syncthreads();
    gemm_tiles<2, HID>(P + OFF_W2, HID, S.Y, q, lane, T, acc);
    signs.h2 |= relu_tiles<SAVE>(acc, P + OFF_B2, T, S.X, sc + FS_H2 * n, n) << (8 * l);
    __syncthreads();
    // seven tiles of outputs: four and three (the last one's columns run past
    // OUT into the next row or b3: in the layer's parameters, and not kept)
    if (q < 4)
        gemm_tiles<4, HID>(P + OFF_W3, OUT, S.X, q, lane, T, acc);
    else
        gemm_tiles<3, HID>(P + OFF_W3, OUT, S.X, q, lane, T, acc);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int f = T.feature + 32 * t + r;
            if (f < OUT) S.Y[T.write[r] + 32 * CS * t] = acc[t][r] + P[OFF_B3 + f];
        }
    __syncthreads();
    if (q < NB) {
        float raw[RAW];
#pragma unroll
        for (int k = 0; k < RAW; ++k) {
            raw[k] = S.Y[at(q * RAW + k, lane)];
            if (SAVE) sc[(FS_DOUT + q * RAW + k) * n + lane] = raw[k];
        }
        Spline sp;
        spline_setup(raw, sp);
        const int j = b_idx(l, q);
        float v, pdf;
        if (INVERSE)
            spline_inverse(sp, Uin[j * CS + lane], v, pdf);
        else
            spline_forward(sp, Uin[j * CS + lane], v, pdf);
        Uout[j * CS + lane] = v;
        S.LQ[(step * NB + q) * CS + lane] = logf(pdf);
    }
    __syncthreads();
}

// Backward pass of layer l (PT = its transposed weights): dL/du at the
// layer's output G[gi] -> at its input G[gi ^ 1]; the deltas of the three
// products go to the scratch fields for the weight gradients.
__device__ __forceinline__ void coop_backward(const float *__restrict__ PT, int l, int q, int lane,
                                              Coop &S, float *__restrict__ sc, int64_t n, float c,
                                              int gi, const Signs &signs) {
    const float *Uin = S.U[l];
    const float *Gin = S.G[gi];
    float *Gout = S.G[gi ^ 1];
    if (q < NB) {
        float raw[RAW];
#pragma unroll
        for (int k = 0; k < RAW; ++k) raw[k] = sc[(FS_DOUT + q * RAW + k) * n + lane];
        Spline sp;
        spline_setup(raw, sp);
        const int j = b_idx(l, q);
        const float ub = Uin[j * CS + lane];
        float y, pdf, gu, graw[RAW];
        spline_forward(sp, ub, y, pdf);
        spline_backward(sp, find_bin<false>(sp, ub), ub, Gin[j * CS + lane], c / pdf, graw, gu);
        Gout[j * CS + lane] = gu;
#pragma unroll
        for (int k = 0; k < RAW; ++k) {
            S.X[at(q * RAW + k, lane)] = graw[k];
            sc[(FS_DOUT + q * RAW + k) * n + lane] = graw[k];
        }
    } else if (q == NB) {
#pragma unroll
        for (int r = OUT; r < ROWS; ++r) S.X[at(r, lane)] = 0.0f;
    }
    __syncthreads();
    const Lane T = lane_of(q, lane);
    f32x4 acc[3];
    // through W3 and the second ReLU
    gemm_tiles<2, OUT>(PT + T3, HID, S.X, q, lane, T, acc);
    mask_tiles(acc, signs.h2 >> (8 * l), T, S.Y, sc + FS_D2 * n, n);
    __syncthreads();
    // through W2 and the first ReLU
    gemm_tiles<2, HID>(PT + T2, HID, S.Y, q, lane, T, acc);
    mask_tiles(acc, signs.h1 >> (8 * l), T, S.X, sc + FS_D1 * n, n);
    __syncthreads();
    // through W1 to the one-blob inputs
    gemm_tiles<3, HID>(PT + T1, IN, S.X, q, lane, T, acc);
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) S.Y[T.write[r] + 32 * CS * t] = acc[t][r];
    __syncthreads();
    // and through the encoding into the conditioning coordinates
    if (q < NA) {
        const int j = a_idx(l, q);
        const float ux = Uin[j * CS + lane];
        float a = 0.0f;
#pragma unroll 4
        for (int k = 0; k < BLOBS; ++k) {
            const float t = (ux - ((float)k + 0.5f) * (1.0f / BLOBS)) * (float)BLOBS;
            a = __fmaf_rn(S.Y[at(q * BLOBS + k, lane)], -expf(-0.5f * t * t) * t * (float)BLOBS, a);
        }
        Gout[j * CS + lane] = Gin[j * CS + lane] + a;
    }
    __syncthreads();
}

// log q of the sample: the spline densities in the order they were met
__device__ __forceinline__ float coop_logq(const Coop &S, int lane) {
    float lq = 0.0f;
#pragma unroll
    for (int i = 0; i < L * NB; ++i) lq += S.LQ[i * CS + lane];
    return lq;
}

__device__ __forceinline__ int wave_index() {
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x / CS));
}

// transposed copies of the three weight matrices of every layer
__global__ void transpose_kernel(const float *__restrict__ theta, float *__restrict__ thetaT) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= L * LPT) return;
    const float *P = theta + (i / LPT) * LP;
    int r = i % LPT;
    float v;
    if (r < T2) {
        v = P[OFF_W1 + (r % IN) * HID + r / IN];
    } else if (r < T3) {
        r -= T2;
        v = P[OFF_W2 + (r % HID) * HID + r / HID];
    } else {
        r -= T3;
        v = P[OFF_W3 + (r % HID) * OUT + r / HID];
    }
    thetaT[i] = v;
}

// sum of the n weights
__global__ __launch_bounds__(1024) void wsum_kernel(const double *__restrict__ w, int64_t n,
                                                    double *__restrict__ out) {
    __shared__ double red[16];
    const double a = block_sum(w, n, red);
    if (threadIdx.x == 0) *out = a;
}

// Forward and backward pass of the weighted negative log-likelihood: loss
// contribution c log q(x) of each sample, c = -w / sum w.  The weight
// gradients are formed afterwards from the scratch fields.
__global__ __launch_bounds__(CT, 4) void train_kernel(const float *__restrict__ theta,
                                                   const float *__restrict__ thetaT,
                                                   const double *__restrict__ x,
                                                   const double *__restrict__ w, int64_t n,
                                                   const double *__restrict__ wsum,
                                                   float *__restrict__ scratch,
                                                   double *__restrict__ loss) {
    __shared__ Coop S;
    const int q = wave_index(), lane = threadIdx.x % CS;
    const int64_t s0 = (int64_t)blockIdx.x * CS, s = s0 + lane, ns = flow_scratch_stride(n);
    // samples past the last one run with weight 0: their deltas are zeros
    const bool live = s < n;
    Signs signs;
    const float c = live ? (float)(-w[s] / *wsum) : 0.0f;
    if (q == 0) {
#pragma unroll
        for (int j = 0; j < D; ++j) S.U[0][j * CS + lane] = live ? (float)x[s * D + j] : 0.5f;
    }
    if (q == 1) {
#pragma unroll
        for (int j = 0; j < D; ++j) S.G[0][j * CS + lane] = 0.0f;
    }
    __syncthreads();
#pragma unroll 1
    for (int l = 0; l < L; ++l)
        coop_layer<false, true>(theta + l * LP, l, l, q, lane, S,
                                scratch + (int64_t)l * FS * ns + s0, ns, signs);
    int gi = 0;
#pragma unroll 1
    for (int l = L - 1; l >= 0; --l) {
        coop_backward(thetaT + l * LPT, l, q, lane, S, scratch + (int64_t)l * FS * ns + s0, ns, c, gi,
                      signs);
        gi ^= 1;
    }
    if (q == 0) {
        const double v = wave_sum(live ? (double)c * (double)coop_logq(S, lane) : 0.0);
        if (lane == 0) unsafeAtomicAdd(loss, v);
    }
}

// Weight gradients as sums over the batch of inputs x deltas: per layer
// W1 (96 x 64, inputs the one-blob encoding), W2 (64 x 64, inputs h1) and W3
// (64 x 99, inputs h2), as FP32 matrix products with the samples as the summed
// index.  A wave takes 32 x 32 of them, a workgroup 64 x 64 of one matrix (its
// waves share the rows in L1); a lane loads eight consecutive samples of
// its feature, which are its terms of eight steps.  The batch is cut into slices of
// ks samples (blockIdx.y) whose partial sums land in part[slice][parameter]
// and are added in slice order afterwards, so the result does not depend on
// scheduling.  The waves whose rows start at 0 also sum their delta columns
// over the slice: the bias gradients.
//
// Through LDS, with 4 x 4 FMAs per thread, 146 us at 20011 samples; now 66.
constexpr int WKC = 32;     // samples per pass: whole 128-byte lines of a field
constexpr int TILES_L = 5;  // W1 rows 0-63 | W1 rows 64-95 | W2 | W3 cols 0-63 | W3 cols 64-98
constexpr int kMaxSlices = 64;

__global__ __launch_bounds__(256) void wgrad_kernel(const float *__restrict__ scratch, int64_t n,
                                                    int64_t ks, float *__restrict__ part) {
    const int l = blockIdx.x / TILES_L, tile = blockIdx.x % TILES_L;
    const int64_t s_begin = (int64_t)blockIdx.y * ks;
    const int64_t s_end = s_begin + ks < n ? s_begin + ks : n;
    const int64_t ns = flow_scratch_stride(n);
    int mat, r0, rows, c0, cols;
    switch (tile) {
    case 0: mat = 0; r0 = 0; rows = 64; c0 = 0; cols = HID; break;
    case 1: mat = 0; r0 = 64; rows = IN - 64; c0 = 0; cols = HID; break;
    case 2: mat = 1; r0 = 0; rows = HID; c0 = 0; cols = HID; break;
    case 3: mat = 2; r0 = 0; rows = HID; c0 = 0; cols = 64; break;
    default: mat = 2; r0 = 0; rows = HID; c0 = 64; cols = OUT - 64; break;
    }
    const int wave = wave_index(), lane = threadIdx.x & 63, i = lane & 15, k = lane >> 4;
    const int wr = 32 * (wave >> 1), wc = 32 * (wave & 1);
    if (wr >= rows || wc >= cols) return;
    r0 += wr;
    c0 += wc;
    cols -= wc;
    const float *sc = scratch + (int64_t)l * FS * ns + s_begin + 8 * k;
    const int bfield = mat == 0 ? FS_D1 : (mat == 1 ? FS_D2 : FS_DOUT);
    const float *pa[2], *pb[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        // (W1: the one coordinate whose bumps these rows are)
        const int row = mat == 0 ? FS_U + a_idx(l, r0 / BLOBS)
                                 : (mat == 1 ? FS_H1 : FS_H2) + r0 + 16 * g + i;
        pa[g] = sc + row * ns;
        pb[g] = sc + (bfield + c0 + 16 * g + i) * ns;  // past the last: other fields, not kept
    }
    f32x4 acc[2][2];
    float bsum[2] = {0.0f, 0.0f};
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[g][h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 na[2][2], nb[2][2];  // [group][half of the eight samples]
    const auto load = [&](int64_t off) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                na[g][e] = *reinterpret_cast<const f32x4 *>(pa[g] + off + 4 * e);
                nb[g][e] = *reinterpret_cast<const f32x4 *>(pb[g] + off + 4 * e);
            }
    };
    load(0);
    for (int64_t s0 = s_begin; s0 < s_end; s0 += WKC) {
        f32x4 a[2][2], b[2][2];
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                a[g][e] = na[g][e];
                b[g][e] = nb[g][e];
            }
        if (s0 + WKC < s_end) load(s0 + WKC - s_begin);
        if (mat == 0) {
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int c = 0; c < 4; ++c) a[g][e][c] = blob(a[g][e][c], 16 * g + i);
        }
        if (s0 + WKC > s_end) {  // samples of the next slice, or past the last
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool in = s0 + 8 * k + 4 * e + c < s_end;
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
                        a[g][e][c] = in ? a[g][e][c] : 0.0f;
                        b[g][e][c] = in ? b[g][e][c] : 0.0f;
                    }
                }
        }
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    bsum[h] += b[h][e][c];
#pragma unroll
                    for (int g = 0; g < 2; ++g)
                        acc[g][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[g][e][c], b[h][e][c],
                                                                         acc[g][h], 0, 0, 0);
                }
    }
    float *G = part + (int64_t)blockIdx.y * PARAMS + l * LP;
    if (r0 == 0) {
        const int boff = mat == 0 ? OFF_B1 : (mat == 1 ? OFF_B2 : OFF_B3);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float v = bsum[h];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (k == 0 && 16 * h + i < cols) G[boff + c0 + 16 * h + i] = v;
        }
    }
    const int off = mat == 0 ? OFF_W1 : (mat == 1 ? OFF_W2 : OFF_W3);
    const int ld = mat == 2 ? OUT : HID;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (16 * h + i < cols)
                    G[off + (r0 + 16 * g + 4 * k + r) * ld + c0 + 16 * h + i] = acc[g][h][r];
}

// grad[i] = sum over the slices, in slice order
__global__ __launch_bounds__(kSumThreads) void wgrad_sum_kernel(const float *__restrict__ part,
                                                                int slices,
                                                                float *__restrict__ grad,
                                                                double *__restrict__ wide) {
    __shared__ SumLds lds;
    float g;
    const int i = slice_sum(part, slices, lds, g);
    if (i < 0) return;
    grad[i] = g;
    if (wide) wide[i] = (double)g;
}

// one workgroup per minibatch: the sum of its weights (fixed order)
__global__ __launch_bounds__(1024) void batch_wsum_kernel(const double *__restrict__ w, int64_t n,
                                                          int64_t batch, double *__restrict__ out) {
    __shared__ double red[16];
    const int64_t b0 = (int64_t)blockIdx.x * batch;
    const double a = block_sum(w + b0, b0 + batch < n ? batch : n - b0, red);
    if (threadIdx.x == 0) out[blockIdx.x] = a;
}

__global__ void zero_u32_kernel(uint32_t *__restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Records (I_t, var_t) of flow-mapped iteration t in the combined state and
// recombines iterations 0..t with equal weights: they all sample the same
// proposal with the same number of points, so the plain mean is unbiased
// (variance weights would favour the iterations that missed the rare large
// weights).  Ibar = sum I / T, sigma = sqrt(sum var) / T, chi2/dof over the
// iterations with var > 0.  Header layout as for the plain combination.
__global__ void flow_combine_kernel(const double *__restrict__ est, double *__restrict__ state,
                                    uint32_t t, double rel_tol, int min_iters) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double *hist = state + MCUBES_STATE_HEADER;
    const double It = est[0], Vt = est[1];
    hist[2 * t] = It;
    hist[2 * t + 1] = Vt;
    if (!isfinite(It) || !isfinite(Vt)) state[6] = 1.0;
    const int T = (int)t + 1;
    double si = 0.0, sv = 0.0;
    for (int q = 0; q < T; ++q) {
        si = si + hist[2 * q];
        sv = sv + hist[2 * q + 1];
    }
    const double Ibar = si / (double)T;
    double chi2 = 0.0, ss = 0.0;
    for (int q = 0; q < T; ++q) {
        const double dv = hist[2 * q] - Ibar;
        ss = ss + dv * dv;
        const double v = hist[2 * q + 1];
        if (v > 0.0) chi2 = chi2 + dv * dv / v;
    }
    // the standard deviation of the mean, from the iterations' own variances
    // and from the scatter of their estimates; the larger is reported
    const double s_w = sqrt(sv) / (double)T;
    const double s_b = T > 1 ? sqrt(ss / ((double)T * (double)(T - 1))) : 0.0;
    const double sigma = s_b > s_w ? s_b : s_w;
    state[0] = Ibar;
    state[1] = sigma;
    state[2] = T > 1 ? chi2 / (double)(T - 1) : 0.0;
    state[3] = (double)(T - 1);
    state[4] = (double)T;
    state[5] = (T >= min_iters && sigma <= rel_tol * fabs(Ibar)) ? 1.0 : 0.0;
}

// Row j of the output is row (a j) mod n of the input (x: 6 doubles per row,
// w: one); with a coprime to n this is a permutation.
__global__ void shuffle_rows_kernel(const double *__restrict__ x, const double *__restrict__ w,
                                    int64_t n, uint64_t a, double *__restrict__ xo,
                                    double *__restrict__ wo) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int64_t src = (int64_t)(((uint64_t)j * a) % (uint64_t)n);
    const double *xi = x + src * flow::D;
    double *xj = xo + j * flow::D;
#pragma unroll
    for (int k = 0; k < flow::D; ++k) xj[k] = xi[k];
    wo[j] = w[src];
}

__global__ void pow_kernel(double *__restrict__ w, int64_t n, double power) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) w[i] = pow(w[i], power);
}

// One Adam step on the FP32 master parameters; c1 = 1 - beta1^t, c2 = 1 - beta2^t.
__global__ void adam_kernel(float *__restrict__ theta, float *__restrict__ m,
                            float *__restrict__ v, const float *__restrict__ grad, int count,
                            float lr, float beta1, float beta2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    adam_update(theta, m, v, i, grad[i], lr, beta1, beta2, eps, c1, c2);
}

// The flow as the map of an m-Cubes iteration: cube c's sample k draws u
// from Philox as V-Sample does (stream word with the high bit set), z_j =
// (c_j + u_j) / g, x = flow sample of z (FP32), w = f(x) / q(x) in FP64.  A
// persistent grid walks the cubes; per-block partials (sum S_c, sum var_c).
template <int F>
__global__ __launch_bounds__(256) void flow_vsample_kernel(const float *__restrict__ theta,
                                                           const VsArgs A, uint32_t stream_word,
                                                           double *__restrict__ partials,
                                                           uint32_t *__restrict__ whist) {
    constexpr int NBLK = (D + 3) / 4;
    __shared__ uint32_t hist[WH_BINS];
    wh_clear(hist);
    __syncthreads();
    const uint32_t T = gridDim.x * blockDim.x;
    double tS = 0.0, tV = 0.0;
    for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < A.m; c += T) {
        uint32_t dig[D];
        uint32_t rest = c;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            dig[j] = rest % A.g;
            rest /= A.g;
        }
        double S = 0.0, D1 = 0.0, D2 = 0.0, w0 = 0.0;
        for (uint32_t k = 0; k < A.p; ++k) {
            float u[D];
#pragma unroll
            for (int b = 0; b < NBLK; ++b) {
                uint32_t r[4];
                philox10(c, stream_word, k * NBLK + b, A.iteration, A.key0, A.key1, r);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int j = 4 * b + q;
                    if (j < D) u[j] = stratum_coordinate(dig[j], r[q], A.g);
                }
            }
            const float lq = sample(theta, u);
            Acc acc = Family<F, D>::begin(A.phase);
#pragma unroll
            for (int j = 0; j < D; ++j) Family<F, D>::axis(acc, A.ca[j], A.cu[j], (double)u[j]);
            const double w = Family<F, D>::end(acc, A) / exp((double)lq);
            wh_add(hist, w);
            S = S + w;
            if (k == 0) w0 = w;
            const double dlt = w - w0;
            D1 = D1 + dlt;
            D2 = D2 + dlt * dlt;
        }
        tS += S;
        tV += (D2 - D1 * D1 * A.inv_p) * A.inv_pm1;
    }
    __shared__ double red[2][4];
    tS = wave_sum(tS);
    tV = wave_sum(tV);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = tS;
        red[1][threadIdx.x >> 6] = tV;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0, v = 0.0;
        for (int q = 0; q < (int)(blockDim.x >> 6); ++q) {
            s += red[0][q];
            v += red[1][q];
        }
        partials[2 * blockIdx.x] = s;
        partials[2 * blockIdx.x + 1] = v;
    }
    wh_flush(hist, whist);
}

// The FP32 flow-mapped iteration in the cooperative form, for p dividing
// 64: each pass of a workgroup takes 64 consecutive samples q (cube q / p,
// sample q % p), so the p samples of a cube sit in one wave; the same
// counters and map as flow_vsample_kernel, the flow run by the eight waves
// together, and the per-cube sums by butterfly shuffles in wave 0.
template <int F>
__global__ __launch_bounds__(CT, 4) void flow_vsample_coop_kernel(const float *__restrict__ theta,
                                                               const VsArgs A,
                                                               uint32_t stream_word,
                                                               double *__restrict__ partials,
                                                               uint32_t *__restrict__ whist) {
    constexpr int NBLK = (D + 3) / 4;
    __shared__ Coop S;
    __shared__ uint32_t hist[WH_BINS];
    wh_clear(hist);
    const int q = wave_index(), lane = threadIdx.x % CS;
    const uint64_t N = (uint64_t)A.m * A.p;
    const int p = (int)A.p;
    Signs signs;  // not kept
    double tS = 0.0, tV = 0.0;
    for (uint64_t base = (uint64_t)blockIdx.x * CS; base < N; base += (uint64_t)gridDim.x * CS) {
        const uint64_t qs = base + lane;
        const bool live = qs < N;  // N is a multiple of p: a cube is live or not as a whole
        if (q == 0) {
            const uint32_t c = live ? (uint32_t)(qs / p) : 0u;
            const uint32_t k = live ? (uint32_t)(qs % p) : 0u;
            uint32_t rest = c;
#pragma unroll
            for (int b = 0; b < NBLK; ++b) {
                uint32_t r[4];
                philox10(c, stream_word, k * NBLK + b, A.iteration, A.key0, A.key1, r);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int j = 4 * b + i;
                    if (j < D) {
                        S.U[0][j * CS + lane] = stratum_coordinate(rest % A.g, r[i], A.g);
                        rest /= A.g;
                    }
                }
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int step = 0; step < L; ++step)
            coop_layer<true, false>(theta + (L - 1 - step) * LP, L - 1 - step, step, q, lane, S,
                                    nullptr, 0, signs);
        if (q == 0) {
            double w = 0.0;
            if (live) {
                Acc acc = Family<F, D>::begin(A.phase);
#pragma unroll
                for (int j = 0; j < D; ++j)
                    Family<F, D>::axis(acc, A.ca[j], A.cu[j], (double)S.U[L][j * CS + lane]);
                w = Family<F, D>::end(acc, A) / exp((double)coop_logq(S, lane));
                wh_add(hist, w);
            }
            // per-cube sums over the p lanes of the cube, shifted by its first sample
            const int first = lane - (lane % p);
            const double w0 = __shfl(w, first);
            const double dlt = w - w0;
            double Sc = w, D1 = dlt, D2 = dlt * dlt;
            for (int off = 1; off < p; off <<= 1) {
                Sc += __shfl_xor(Sc, off);
                D1 += __shfl_xor(D1, off);
                D2 += __shfl_xor(D2, off);
            }
            if (live && lane == first) {
                tS += Sc;
                tV += (D2 - D1 * D1 * A.inv_p) * A.inv_pm1;
            }
        }
        __syncthreads();  // S is reused by the next pass
    }
    if (q == 0) {
        tS = wave_sum(tS);
        tV = wave_sum(tV);
        if (lane == 0) {
            partials[2 * blockIdx.x] = tS;
            partials[2 * blockIdx.x + 1] = tV;
        }
    }
    wh_flush(hist, whist);
}

// The samples of work items [w0, w0 + count) of one plain iteration (cube
// (w mult) mod m, the order in which V-Sample's threads visit the cubes, so
// that a prefix of the work items is spread over the whole domain), with
// their weights w = f J: the same counters, bins and arithmetic as V-Sample,
// so these are samples that iteration draws.  x: (count p) x D, w: count p.
template <int F, int DIM>
__global__ __launch_bounds__(256) void dump_kernel(const VsArgs A, const double *__restrict__ grid,
                                                   uint32_t w0, uint32_t count,
                                                   double *__restrict__ xs,
                                                   double *__restrict__ ws) {
    constexpr int NBLK = (DIM + 3) / 4;
    const uint32_t q0 = blockIdx.x * blockDim.x + threadIdx.x;
    if (q0 >= count) return;
    const uint32_t c = (uint32_t)(((uint64_t)(w0 + q0) * A.mult) % A.m);
    const int nb = (int)A.nb;
    double cb[DIM];
    uint32_t rest = c;
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
        cb[j] = __fma_rn((double)(rest % A.g), 0x1p32, 0.5);
        rest /= A.g;
    }
    for (uint32_t k = 0; k < A.p; ++k) {
        Acc acc = Family<F, DIM>::begin(A.phase);
        double prod = 1.0;
        const uint64_t row = (uint64_t)q0 * A.p + k;
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            uint32_t r[4];
            philox10(c, A.stream_id, k * NBLK + b, A.iteration, A.key0, A.key1, r);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = 4 * b + q;
                if (j < DIM) {
                    const double z = ((double)r[q] + cb[j]) * A.zscale;
                    int i = (int)z;
                    double phi;
                    if constexpr (DIM >= 2) {
                        phi = __builtin_amdgcn_fract(z);
                    } else {
                        i = i < nb - 1 ? i : nb - 1;
                        phi = z - (double)i;
                    }
                    const double *e = grid + j * (nb + 1) + i;
                    const double W = e[1] - e[0];
                    const double x = __fma_rn(W, phi, e[0]);
                    prod = prod * W;
                    Family<F, DIM>::axis(acc, A.ca[j], A.cu[j], x);
                    xs[row * DIM + j] = x;
                }
            }
        }
        ws[row] = Family<F, DIM>::end(acc, A) * (A.nbd * prod);
    }
}

template <int F>
hipError_t launch_flow_vsample_f(const float *theta, const VsArgs &A, uint32_t stream_word,
                                 double *partials, uint32_t *whist, int blocks, hipStream_t s) {
    if (64 % A.p == 0)
        hipLaunchKernelGGL((flow_vsample_coop_kernel<F>), dim3(blocks), dim3(CT), 0, s, theta, A,
                           stream_word, partials, whist);
    else
        hipLaunchKernelGGL((flow_vsample_kernel<F>), dim3(blocks), dim3(256), 0, s, theta, A,
                           stream_word, partials, whist);
    return hipGetLastError();
}

template <int F>
hipError_t launch_dump_f(int dim, const VsArgs &A, const double *grid, uint32_t c0,
                         uint32_t count, double *xs, double *ws, hipStream_t s) {
    const dim3 grid_dim((count + 255) / 256);
#define DUMP_CASE(DD)                                                                            \
    case DD:                                                                                     \
        hipLaunchKernelGGL((dump_kernel<F, DD>), grid_dim, dim3(256), 0, s, A, grid, c0, count, \
                           xs, ws);                                                              \
        break;
    switch (dim) {
        DUMP_CASE(1) DUMP_CASE(2) DUMP_CASE(3) DUMP_CASE(4) DUMP_CASE(5)
        DUMP_CASE(6) DUMP_CASE(7) DUMP_CASE(8) DUMP_CASE(9) DUMP_CASE(10)
    default: return hipErrorInvalidValue;
    }
#undef DUMP_CASE
    return hipGetLastError();
}

}  // namespace

// FP32: per-sample fields, then the partial weight gradients of the slices
int64_t flow_scratch_floats(int64_t n) {
    const int64_t fp32 = (int64_t)L * FS * flow_scratch_stride(n) + (int64_t)kMaxSlices * PARAMS;
    const int64_t bf16 = flow_bf16_train_floats(n);
    return fp32 > bf16 ? fp32 : bf16;
}

hipError_t launch_flow_wgrad_sum(const float *part, int slices, float *grad, double *wide,
                                 hipStream_t s) {
    hipLaunchKernelGGL(wgrad_sum_kernel, dim3(kSumBlocks), dim3(kSumThreads), 0, s, part, slices,
                       grad, wide);
    return hipGetLastError();
}

int64_t flow_transposed_floats() { return (int64_t)L * LPT; }

hipError_t launch_flow_wsum(const double *w, int64_t n, double *wsum, hipStream_t s) {
    hipLaunchKernelGGL(wsum_kernel, dim3(1), dim3(1024), 0, s, w, n, wsum);
    return hipGetLastError();
}

hipError_t launch_flow_train_fp32(const float *theta, float *thetaT, const double *x,
                                  const double *w, int64_t n, const double *wsum, float *scratch,
                                  double *loss, hipStream_t s) {
    hipLaunchKernelGGL(transpose_kernel, dim3((L * LPT + 255) / 256), dim3(256), 0, s, theta,
                       thetaT);
    hipLaunchKernelGGL(train_kernel, dim3((unsigned)((n + CS - 1) / CS)), dim3(CT), 0, s, theta,
                       thetaT, x, w, n, wsum, scratch, loss);
    return hipGetLastError();
}

hipError_t launch_flow_wgrad(const float *scratch_in, int64_t n, float *grad, double *wide,
                             hipStream_t s) {
    float *scratch = const_cast<float *>(scratch_in);
    // slices of at least 512 samples, at most kMaxSlices of them
    int64_t slices = (n + 511) / 512;
    if (slices > kMaxSlices) slices = kMaxSlices;
    int64_t ks = (n + slices - 1) / slices;
    ks = (ks + WKC - 1) / WKC * WKC;
    slices = (n + ks - 1) / ks;
    float *part = scratch + (int64_t)L * FS * flow_scratch_stride(n);
    hipLaunchKernelGGL(wgrad_kernel, dim3(L * TILES_L, (unsigned)slices), dim3(256), 0, s, scratch,
                       n, ks, part);
    return launch_flow_wgrad_sum(part, (int)slices, grad, wide, s);
}

hipError_t launch_flow_batch_wsums(const double *w, int64_t n, int64_t batch, double *out,
                                   hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(batch_wsum_kernel, dim3((unsigned)((n + batch - 1) / batch)), dim3(1024), 0,
                       s, w, n, batch, out);
    return hipGetLastError();
}

hipError_t launch_zero_u32(uint32_t *p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_flow_combine(const double *est, double *state, uint32_t iteration,
                               double rel_tol, int min_iters, hipStream_t s) {
    hipLaunchKernelGGL(flow_combine_kernel, dim3(1), dim3(64), 0, s, est, state, iteration,
                       rel_tol, min_iters);
    return hipGetLastError();
}

hipError_t launch_flow_shuffle(const double *x, const double *w, int64_t n, uint64_t a,
                               double *xo, double *wo, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(shuffle_rows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x,
                       w, n, a, xo, wo);
    return hipGetLastError();
}

hipError_t launch_pow_weights(double *w, int64_t n, double power, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(pow_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, n, power);
    return hipGetLastError();
}

hipError_t launch_flow_adam(float *theta, float *m, float *v, const float *grad, float lr,
                            float beta1, float beta2, float eps, float c1, float c2,
                            hipStream_t s) {
    hipLaunchKernelGGL(adam_kernel, dim3((PARAMS + 255) / 256), dim3(256), 0, s, theta, m, v,
                       grad, PARAMS, lr, beta1, beta2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_flow_vsample(int family, const float *theta, const VsArgs &A,
                               uint32_t stream_word, double *partials, uint32_t *whist,
                               int blocks, hipStream_t s) {
    switch (family) {
    case MCUBES_OSCILLATORY: return launch_flow_vsample_f<MCUBES_OSCILLATORY>(theta, A, stream_word, partials, whist, blocks, s);
    case MCUBES_PRODUCT_PEAK: return launch_flow_vsample_f<MCUBES_PRODUCT_PEAK>(theta, A, stream_word, partials, whist, blocks, s);
    case MCUBES_CORNER_PEAK: return launch_flow_vsample_f<MCUBES_CORNER_PEAK>(theta, A, stream_word, partials, whist, blocks, s);
    case MCUBES_GAUSSIAN: return launch_flow_vsample_f<MCUBES_GAUSSIAN>(theta, A, stream_word, partials, whist, blocks, s);
    case MCUBES_C0: return launch_flow_vsample_f<MCUBES_C0>(theta, A, stream_word, partials, whist, blocks, s);
    case MCUBES_DISCONTINUOUS: return launch_flow_vsample_f<MCUBES_DISCONTINUOUS>(theta, A, stream_word, partials, whist, blocks, s);
    case MCUBES_ADDITION: return launch_flow_vsample_f<MCUBES_ADDITION>(theta, A, stream_word, partials, whist, blocks, s);
    case MCUBES_MIXTURE: return launch_flow_vsample_f<MCUBES_MIXTURE>(theta, A, stream_word, partials, whist, blocks, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_vsample_dump(int family, int dim, const VsArgs &A, const double *grid,
                               uint32_t c0, uint32_t count, double *xs, double *ws,
                               hipStream_t s) {
    if (count == 0) return hipSuccess;
    switch (family) {
    case MCUBES_OSCILLATORY: return launch_dump_f<MCUBES_OSCILLATORY>(dim, A, grid, c0, count, xs, ws, s);
    case MCUBES_PRODUCT_PEAK: return launch_dump_f<MCUBES_PRODUCT_PEAK>(dim, A, grid, c0, count, xs, ws, s);
    case MCUBES_CORNER_PEAK: return launch_dump_f<MCUBES_CORNER_PEAK>(dim, A, grid, c0, count, xs, ws, s);
    case MCUBES_GAUSSIAN: return launch_dump_f<MCUBES_GAUSSIAN>(dim, A, grid, c0, count, xs, ws, s);
    case MCUBES_C0: return launch_dump_f<MCUBES_C0>(dim, A, grid, c0, count, xs, ws, s);
    case MCUBES_DISCONTINUOUS: return launch_dump_f<MCUBES_DISCONTINUOUS>(dim, A, grid, c0, count, xs, ws, s);
    case MCUBES_ADDITION: return launch_dump_f<MCUBES_ADDITION>(dim, A, grid, c0, count, xs, ws, s);
    case MCUBES_MIXTURE: return launch_dump_f<MCUBES_MIXTURE>(dim, A, grid, c0, count, xs, ws, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mcubes
