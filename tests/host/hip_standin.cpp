// Stand-in for the HIP runtime, for host tests of the library's C entry points
// on machines without a GPU.  Device memory is host memory, copies and fills
// take effect at once, kernels do nothing.  Loaded with global symbols before
// libcteno.so, it takes the place of the runtime that the library is linked to.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <thread>
#include <unordered_map>

namespace {
std::mutex mu;
std::unordered_map<void *, size_t> blocks;
int64_t live = 0, peak = 0;
std::atomic<int64_t> n_malloc{0}, n_pinned{0}, n_capture{0}, n_instantiate{0}, n_graph{0}, n_graph_destroy{0},
    n_event{0}, n_event_destroy{0}, n_kernel{0}, n_foreign{0};
size_t fill_size = 0;
int32_t fill_value = 0;
std::atomic<int> fail_instantiate{0};     // this instantiation from now fails (0: none)
std::thread::id caller;
thread_local bool capturing = false;
std::atomic<uintptr_t> next_handle{0x1000};
template <class T> T handle() { return reinterpret_cast<T>(next_handle.fetch_add(16)); }
}  // namespace

extern "C" {
// what the tests read and set
int64_t standin_count(const char *what) {
    const auto is = [&](const char *s) { return std::strcmp(what, s) == 0; };
    if (is("malloc")) return n_malloc;
    if (is("pinned")) return n_pinned;
    if (is("capture")) return n_capture;
    if (is("instantiate")) return n_instantiate;
    if (is("graph_launch")) return n_graph;
    if (is("graph_alive")) return n_capture - n_graph_destroy;
    if (is("event_alive")) return n_event - n_event_destroy;
    if (is("kernel")) return n_kernel;
    if (is("foreign_copy")) return n_foreign;     // copies issued by other threads than standin_caller's
    std::lock_guard<std::mutex> lk(mu);
    if (is("live")) return live;
    if (is("peak")) return peak;
    return -1;
}
void standin_caller() { caller = std::this_thread::get_id(); }
void standin_fail_instantiate(int nth) { fail_instantiate = nth; }
// device allocations of this size hold that value instead of zeros
void standin_fill(size_t bytes, int32_t value) { fill_size = bytes; fill_value = value; }

void **__hipRegisterFatBinary(const void *) { static void *h = nullptr; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, dim3 *, dim3 *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st) {
    *g = *b = dim3(1);
    *s = 0;
    *st = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) {
    if (!capturing) ++n_kernel;
    return hipSuccess;
}

hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static char *buf = (char *)std::calloc(1, 64);
    *p = buf;
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n) {
    *p = std::calloc(1, n);
    if (!*p) return hipErrorOutOfMemory;
    for (size_t k = 0; n == fill_size && k < n / 4; ++k) ((int32_t *)*p)[k] = fill_value;
    ++n_malloc;
    std::lock_guard<std::mutex> lk(mu);
    blocks[*p] = n;
    live += (int64_t)n;
    peak = live > peak ? live : peak;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    {
        std::lock_guard<std::mutex> lk(mu);
        live -= (int64_t)blocks[p];
        blocks.erase(p);
    }
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    *p = std::calloc(1, n);
    ++n_pinned;
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *, const void *) { return hipErrorInvalidValue; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    if (std::this_thread::get_id() != caller) ++n_foreign;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = handle<hipStream_t>(); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = handle<hipEvent_t>(); ++n_event; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { ++n_event_destroy; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }

hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { capturing = true; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    capturing = false;
    ++n_capture;
    *g = handle<hipGraph_t>();
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { ++n_graph_destroy; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    ++n_instantiate;
    if (fail_instantiate > 0 && --fail_instantiate == 0) return hipErrorOutOfMemory;
    *x = handle<hipGraphExec_t>();
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { ++n_graph; return hipSuccess; }
}
