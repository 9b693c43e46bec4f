// Driver for the CPU check of the host driver's error paths: mcubes_api.cpp and
// host.cpp on a stand-in for the HIP runtime and the kernels' launchers, which
// counts what is queued and not yet waited for and lets the n-th fallible
// call fail.  Every call has to return MC_EDEVICE then, with nothing queued that
// still reads the calling thread's buffers or the caller's tables.
// Usage: <program> <host|device|timed|pass|prepare> <tables: 0 or 1>
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "internal.hpp"
#include "mcubes.h"

namespace {
int calls = 0, fail_at = -1, queued = 0;
bool fails() { return calls++ == fail_at; }
hipError_t step() { return fails() ? hipErrorOutOfMemory : hipSuccess; }
hipError_t enqueue() {
    if (fails()) return hipErrorLaunchFailure;
    ++queued;
    return hipSuccess;
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return step(); }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 1; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    if (fails()) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { std::free(p); return step(); }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return step(); }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return enqueue(); }
hipError_t hipStreamSynchronize(hipStream_t) {
    if (fails()) { queued = 0; return hipErrorLaunchFailure; }  // (an error, but the work is over)
    queued = 0;
    return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) { return queued ? hipErrorNotReady : hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return step(); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return step(); }
hipError_t hipEventSynchronize(hipEvent_t) { return step(); }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 1.0f; return step(); }
}

namespace mcubes {
const void *sample_kernel(int, int, int, bool) { return &calls; }
hipError_t launch_sample(const void *, int, int, size_t, hipStream_t, const SampleArgs &) { return enqueue(); }
hipError_t launch_finalize(const double *, double *, int, int, int, int, uint32_t *, double *out, uint32_t *, uint32_t *done,
                           uint32_t seq, hipStream_t) {
    if (fails()) return hipErrorLaunchFailure;
    if (done) {  // all that was queued before is over once the word is there
        out[0] = out[1] = 1.0;
        out[2] = 0.0;
        *done = seq;
        queued = 0;
    } else {
        ++queued;
    }
    return hipSuccess;
}
hipError_t launch_upload(const double *, double *, int, hipStream_t) { return enqueue(); }
hipError_t launch_zero(double *, size_t, hipStream_t) { return enqueue(); }
hipError_t launch_run_init(RunState *, double *, double *, int, int, int, hipStream_t) { return enqueue(); }
hipError_t launch_steps(const StepsArgs &a, hipStream_t) {
    if (fails()) return hipErrorLaunchFailure;
    ++queued;
    a.ctl.host->k = a.ctl.it + 1;
    if (a.ctl.it + 1 == a.ctl.itmax) a.ctl.host->last = a.ctl.it;
    return hipSuccess;
}
hipError_t launch_refine(double *, const double *, int, int, int, double, hipStream_t) { return enqueue(); }
}  // namespace mcubes

int main(int, char **argv) {
    const std::string what = argv[1];
    const bool tables = argv[2][0] == '1';
    const int d = 4, nb = 8;
    std::vector<double> params(2 * d, 0.5), tab(2 * 65536, 1.0), lo(d, 0.0), hi(d, 1.0), grid(d * (nb + 1)), hist(d * nb);
    mc_problem p{};
    p.integrand = tables ? MC_F_GAUSS_TABLES : MC_F_GAUSS_PRODUCT;
    p.dim = d;
    p.params = params.data();
    p.n_params = 2 * d;
    p.tables = tables ? tab.data() : nullptr;
    p.n_tables = tables ? (int64_t)tab.size() : 0;
    p.lo = lo.data();
    p.hi = hi.data();
    p.maxcalls = 40'000'000;  // (launches of their own for the steps)
    p.nbins = nb;
    p.itmax = p.ita = 3;
    p.alpha = 1.5;
    p.device_steps = what == "device" || what == "timed";
    size_t bytes = 0;
    if (mc_workspace_bytes(&p, &bytes) != MC_OK) return 2;
    std::vector<char> ws(bytes);
    auto run = [&]() -> mc_status {
        mc_result r{};
        mc_timing t{};
        double out[2];
        if (what == "prepare") return mc_prepare(&p, ws.data(), bytes, nullptr);
        if (what == "pass")
            return mc_sample_iteration(&p, 0, 1, grid.data(), ws.data(), bytes, nullptr, out, hist.data(), nullptr, 0, 0, 0);
        return mc_integrate(&p, ws.data(), bytes, nullptr, &r, nullptr, grid.data(), what == "timed" ? &t : nullptr);
    };
    int bad = 0;
    for (int n = 0;; ++n) {
        calls = 0;
        fail_at = n;
        queued = 0;
        const mc_status st = run();
        if (calls <= n) {  // none failed any more
            if (st != MC_OK || queued != 0) std::printf("whole call: status %d queued %d\n", st, queued), ++bad;
            std::printf("%d places\n", n);
            return bad || n < 3;
        }
        if (st != MC_EDEVICE || queued != 0) std::printf("call %d failed: status %d queued %d\n", n, st, queued), ++bad;
    }
}
