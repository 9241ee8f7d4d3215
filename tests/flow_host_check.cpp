// CPU driver of the flow's host code (flow_api.hip), built and run by tests/test_flow_host.py: the
// HIP runtime and the kernel launches are stand-ins on host memory, of which any one can be made to
// fail.  An optimiser step adds 1 to the first parameter, a pack copies it into the packed forms, and
// the reading calls note the value they were given.  After every call that fails at any of its
// steps, and after it succeeds, each reading call has to see the parameters as they then are.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "flow_impl.h"

using namespace mcubes;

namespace {

int g_fail_at = 0, g_calls = 0;  // the g_fail_at-th call from here on fails (0: none)
float g_seen32 = 0, g_seen16 = 0;
const float *g_theta = nullptr;  // the flow's device parameters

hipError_t step() { return ++g_calls == g_fail_at ? hipErrorLaunchFailure : hipSuccess; }
void arm(int k) {
    g_calls = 0;
    g_fail_at = k;
}
void require(bool ok, const char *what, int k) {
    if (ok) return;
    printf("FAILED: %s, at step %d (theta %g, FP32 sees %g, BF16 sees %g)\n", what, k, *g_theta,
           g_seen32, g_seen16);
    exit(1);
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return step(); }
hipError_t hipStreamSynchronize(hipStream_t) { return step(); }
hipError_t hipMalloc(void **p, size_t n) { *p = calloc(n, 1); return hipSuccess; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    const hipError_t e = step();
    if (e == hipSuccess) memcpy(d, s, n);
    return e;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) {
    return hipMemcpy(d, s, n, k);
}
hipError_t hipMemset(void *d, int v, size_t n) {
    const hipError_t e = step();
    if (e == hipSuccess) memset(d, v, n);
    return e;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }
hipError_t hipEventCreate(hipEvent_t *) { return hipErrorUnknown; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorUnknown; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorUnknown; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorUnknown; }
const char *hipGetErrorString(hipError_t) { return "stand-in"; }
void mcubes_default_options(mcubes_options *o) { memset(o, 0, sizeof *o); }
int mcubes_iteration(const mcubes_plan *, uint32_t, const double *, double *, double *, double *,
                     double *, double *, double, void *) { return MCUBES_E_DEVICE; }
int mcubes_plan_create(int, const double *, int, int64_t, uint64_t, const mcubes_options *,
                       mcubes_plan **) { return MCUBES_E_DEVICE; }
void mcubes_plan_destroy(mcubes_plan *) {}
}

namespace mcubes {
int fail(int code, const char *, ...) { return code; }
int hip_fail(hipError_t, const char *) { return MCUBES_E_DEVICE; }
hipStream_t as_stream(void *s) { return (hipStream_t)s; }
int64_t flow_scratch_floats(int64_t) { return 64; }
int64_t flow_transposed_floats() { return 64; }
int64_t flow_bf16_frag_bytes() { return 64; }
int64_t flow_fp32_frag_bytes() { return 64; }
int64_t flow_bf16_bias_floats() { return 64; }
int64_t flow_fp32_bias_floats() { return 64; }
int64_t flow_bf16_bwd_frag_bytes() { return 64; }
int64_t flow_bf16_inverse_map_ints() { return 64; }
hipError_t launch_fill(double *, int64_t, double, hipStream_t) { return step(); }
hipError_t launch_init_grid(double *, int, int, hipStream_t) { return step(); }
hipError_t launch_reduce(const double *, int, double, double, double *, hipStream_t) { return step(); }
hipError_t launch_zero_u32(uint32_t *, int64_t, hipStream_t) { return step(); }
hipError_t launch_flow_combine(const double *, double *, uint32_t, double, int, hipStream_t) { return step(); }
hipError_t launch_flow_shuffle(const double *, const double *, int64_t, uint64_t, double *, double *,
                               hipStream_t) { return step(); }
hipError_t launch_pow_weights(double *, int64_t, double, hipStream_t) { return step(); }
hipError_t launch_flow_wsum(const double *, int64_t, double *, hipStream_t) { return step(); }
hipError_t launch_flow_batch_wsums(const double *, int64_t, int64_t, double *, hipStream_t) { return step(); }
hipError_t launch_flow_train_fp32(const float *, float *, const double *, const double *, int64_t,
                                  const double *, float *, double *, hipStream_t) { return step(); }
hipError_t launch_flow_wgrad(const float *, int64_t, float *, double *, hipStream_t) { return step(); }
hipError_t launch_flow_grad_bf16(const float *, int64_t, int, float *, double *, hipStream_t) { return step(); }
hipError_t launch_flow_inverse_map(int *, hipStream_t) { return step(); }
hipError_t launch_flow_vsample(int, const float *, const VsArgs &, uint32_t, double *, uint32_t *, int,
                               hipStream_t) { return step(); }
hipError_t launch_flow_vsample_bf16(int, const void *, const float *, const VsArgs &, uint32_t,
                                    double *, uint32_t *, int, hipStream_t) { return step(); }
hipError_t launch_flow_draw_bf16(int, const void *, const float *, const VsArgs &, uint32_t, uint32_t,
                                 double *, double *, hipStream_t) { return step(); }
hipError_t launch_vsample_dump(int, int, const VsArgs &, const double *, uint32_t, uint32_t, double *,
                               double *, hipStream_t) { return step(); }

hipError_t pack(const float *theta, void *frags) {
    const hipError_t e = step();
    g_theta = theta;
    if (e == hipSuccess) *(float *)frags = *theta;
    return e;
}
hipError_t launch_flow_pack_bf16(const float *theta, void *frags, float *, hipStream_t) { return pack(theta, frags); }
hipError_t launch_flow_pack_fp32(const float *theta, void *frags, float *, hipStream_t) { return pack(theta, frags); }
hipError_t launch_flow_train_bf16(const float *theta, void *frags, void *, float *, const double *,
                                  const double *, int64_t, const double *, double *, float *, double *,
                                  int, bool p, hipStream_t) { return p ? pack(theta, frags) : step(); }
hipError_t launch_flow_adam(float *theta, float *, float *, const float *, float, float, float, float,
                            float, float, hipStream_t) {
    const hipError_t e = step();
    if (e == hipSuccess) *theta += 1.0f;
    return e;
}
hipError_t launch_flow_adam_pack_fp32(float *theta, float *, float *, const float *, float, float,
                                      float, float, float, float, const int *, void *frags, float *,
                                      hipStream_t) {
    const hipError_t e = step();
    if (e == hipSuccess) *(float *)frags = *theta += 1.0f;
    return e;
}
hipError_t launch_flow_grad_adam_bf16(const float *, int64_t, int, float *theta, float *, float *,
                                      float *, float, float, float, float, float, float, const int *,
                                      void *frags, void *, float *, hipStream_t) {
    const hipError_t e = step();
    if (e == hipSuccess) *(float *)frags = *theta += 1.0f;
    return e;
}
hipError_t launch_flow_map_fp32(bool, const void *frags, const float *, const double *, int64_t,
                                double *, double *, hipStream_t) {
    g_seen32 = *(const float *)frags;
    return step();
}
hipError_t launch_flow_draw_fp32(int, const void *frags, const float *, const VsArgs &, uint32_t,
                                 uint32_t, double *, double *, hipStream_t) {
    g_seen32 = *(const float *)frags;
    return step();
}
hipError_t launch_flow_sample_bf16(const void *frags, const float *, const double *, int64_t, double *,
                                   double *, hipStream_t) {
    g_seen16 = *(const float *)frags;
    return step();
}
}  // namespace mcubes

namespace {

// every reading call sees the parameters as they are
void check_reads(mcubes_flow *F, const char *what, int k) {
    double x[6] = {}, y[6], q;
    arm(0);
    g_seen32 = g_seen16 = -1.0f;
    require(mcubes_flow_density(F, MCUBES_FP32, x, 1, y, &q, nullptr) == MCUBES_OK, "density", k);
    require(g_seen32 == *g_theta, what, k);
    g_seen32 = -1.0f;
    require(mcubes_flow_sample(F, MCUBES_FP32, x, 1, y, &q, nullptr) == MCUBES_OK, "sampling", k);
    require(g_seen32 == *g_theta, what, k);
    require(mcubes_flow_sample(F, MCUBES_BF16, x, 1, y, &q, nullptr) == MCUBES_OK, "sampling", k);
    require(g_seen16 == *g_theta, what, k);
}

// `call`, failing at its first, second, ... step until it succeeds
template <class Call>
int each_failure(mcubes_flow *F, const char *what, Call call) {
    for (int k = 1;; ++k) {
        arm(k);
        const int rc = call();
        const bool reached = g_calls >= k;
        require(reached == (rc != MCUBES_OK), "a failed step is reported", k);
        check_reads(F, what, k);
        if (!reached) return k;
    }
}

}  // namespace

int main() {
    std::vector<double> theta(flow::PARAMS, 0.5), other(flow::PARAMS, 7.0), x(6 * 10, 0.5), w(10, 1.0);
    mcubes_flow *F = nullptr;
    if (mcubes_flow_create(theta.data(), &F) != MCUBES_OK) return 2;
    int steps = 0;
    check_reads(F, "creation", 0);
    for (int precision : {(int)MCUBES_FP32, (int)MCUBES_BF16})
        for (int epochs : {0, 1, 3})
            for (int batch : {4, 10})
                for (bool losses : {false, true}) {
                    double l[3];
                    steps += each_failure(F, "training", [&] {
                        return mcubes_flow_train(F, precision, x.data(), w.data(), 10, epochs, batch,
                                                 1e-3, losses ? l : nullptr, nullptr);
                    });
                }
    steps += each_failure(F, "Adam step", [&] {
        return mcubes_flow_adam_step(F, 1e-3, 0.9, 0.999, 1e-8, nullptr);
    });
    steps += each_failure(F, "parameter upload", [&] { return mcubes_flow_set_params(F, other.data()); });
    mcubes_flow_destroy(F);
    printf("ok %d\n", steps);
    return 0;
}
