// af_step's status words on the host: the C ABI (af_api.hip) against stand-ins for the HIP
// calls that it makes (host memory, work done at once) and for the kernels' launchers.  A step of
// the stand-in adds one to every plane; step g_bad raises the CFL bit, step g_fail is not
// launched.  Prints nothing and returns 0 if every call's status and state are right.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "af.h"
#include "af_batch.h"
#include "af_internal.h"

static int g_step = 0, g_bad = -1, g_fail = -1;

namespace af {
static hipError_t step(const StepArgs& a) {
    const int s = g_step++;
    if (s == g_fail) return hipErrorOutOfMemory;
    const size_t n = (size_t)a.nx * a.ny;
    for (int k = 0; k < 16; ++k)
        for (size_t q = 0; q < n; ++q) ((double*)a.out[k])[q] = ((const double*)a.in[k])[q] + 1.0;
    if (s == g_bad) *a.status |= SB_CFL;
    return hipSuccess;
}
hipError_t launch_step_fused_f64(const StepArgs& a) { return step(a); }
hipError_t launch_step_fused_f32(const StepArgs&) { return hipErrorUnknown; }
hipError_t launch_step_multi_f64(const StepArgs&) { return hipErrorUnknown; }
hipError_t launch_step_split_f64(const StepArgs&) { return hipErrorUnknown; }
hipError_t launch_step_fc_f64(const StepArgs&) { return hipErrorUnknown; }
hipError_t launch_adjoint_f64(const StepArgs&, const void* const*, void* const*) { return hipErrorUnknown; }
hipError_t launch_adjoint_noalloc(StepArgs, const void* const*, void* const*) { return hipErrorUnknown; }
hipError_t noalloc_scratch_ptr(void**) { return hipErrorUnknown; }
hipError_t prepare_fused_f64(int, int) { return hipSuccess; }
hipError_t prepare_fused_f32(int, int) { return hipSuccess; }
hipError_t prepare_split_f64() { return hipSuccess; }
hipError_t prepare_adjoint_f64() { return hipSuccess; }
size_t scratch_bytes_multi_f64(int, int) { return 16; }
size_t scratch_bytes_split_f64(int, int) { return 16; }
size_t scratch_bytes_fc_f64(int, int) { return 16; }
size_t scratch_bytes_adjoint_f64(int, int) { return 16; }
hipError_t launch_diag(const void* const*, bool, const double*, int, int, double, double, double*, int, double*, hipStream_t) {
    return hipErrorUnknown;
}
const BatchTileCfg kBatchCfgs[kNumBatchCfgs] = {};
PolPert<float> pert_pol_f32(const double*, double) { return {}; }
hipError_t batch_occupancy(int, int, int*) { return hipErrorUnknown; }
hipError_t launch_batch(int, int, const BatchInst*, const int2*, int, int, unsigned*, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_batch_copy(const BatchInst*, int, hipStream_t) { return hipErrorUnknown; }
}  // namespace af

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
// the only kernel launched here is the copy of a state's planes: its first argument holds the
// pointers, its second the number of words
hipError_t hipLaunchKernel(const void*, dim3, dim3, void** args, size_t, hipStream_t) {
    struct { const void* src[16]; void* dst[16]; } c;
    size_t n;
    std::memcpy(&c, args[0], sizeof(c));
    std::memcpy(&n, args[1], sizeof(n));
    for (int k = 0; k < 16; ++k) std::memcpy(c.dst[k], c.src[k], n * 16);
    return hipSuccess;
}
}

static int bad = 0;

static void call(af_ctx* ctx, int nsteps, int bad_step, int fail_step, af_status want, double plus) {
    double* buf = (double*)std::aligned_alloc(64, 16 * 16 * sizeof(double));
    for (int q = 0; q < 256; ++q) buf[q] = q;
    af_state s;
    for (int k = 0; k < 4; ++k) { s.avg[k] = buf + 16 * k; s.V[k] = buf + 64 + 16 * k; s.EV[k] = buf + 128 + 16 * k; s.EH[k] = buf + 192 + 16 * k; }
    g_step = 0;
    g_bad = bad_step;
    g_fail = fail_step;
    const af_status st = af_step(ctx, &s, 0.1, nsteps);
    bool same = true;
    for (int q = 0; q < 256; ++q) same = same && (plus < 0.0 || buf[q] == q + plus);
    if (st != want || !same) {
        std::fprintf(stderr, "%d steps, bad %d, failed launch %d: status %d, expected %d; state %s\n", nsteps, bad_step, fail_step, st, want,
                     same ? "right" : "wrong");
        bad = 1;
    }
    std::free(buf);
}

int main() {
    af_config cfg{};
    cfg.nx = cfg.ny = 4;
    cfg.h = 1.0;
    cfg.gamma = 1.4;
    cfg.precision = AF_F64;
    cfg.flags = AF_CHECK;
    af_ctx* ctx = nullptr;
    if (af_init(&cfg, nullptr, &ctx) != AF_OK) return 2;
    for (int n : {1, 2, 15, 16, 17, 33}) {
        call(ctx, n, -1, -1, AF_OK, n);
        for (int b = 0; b < n; ++b) {
            call(ctx, n, b, -1, AF_ERR_ACOUSTIC_CFL, 0.0);
            call(ctx, n, -1, -1, AF_OK, n);
            call(ctx, n, -1, b, AF_ERR_HIP, -1.0);
            // a launch that fails after a bad step: the bad step's status, as the words are read in
            // order, the state of the call's input, and nothing left for the next call
            for (int f = b + 1; f < n; ++f) {
                call(ctx, n, b, f, AF_ERR_ACOUSTIC_CFL, 0.0);
                call(ctx, n, -1, -1, AF_OK, n);
            }
        }
    }
    af_destroy(ctx);
    return bad;
}
