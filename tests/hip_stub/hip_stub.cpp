// A stand-in for the HIP runtime and for the kernels, for tests of the host
// runtime (dart_runtime, dart_server, dart_stream, dart_noalloc) on a CPU.
//
// Device memory is host memory (reserved, not touched), every stream runs its work
// at once, and kernels do nothing but what the host reads back: error words,
// descriptors, cleared words and totals.  Every call is first reported to the
// test's hook (name, two arguments); a non-zero answer is returned in place of
// running the call, which is how a test makes one fail, watches an order of calls,
// or acts in the middle of one.
#include <hip/hip_runtime.h>
#include <string.h>
#include <sys/mman.h>

#include <atomic>
#include <map>
#include <mutex>
#include <set>
#include <utility>
#include <vector>

#include "../../paper_2609_09322_amd/csrc/dart_internal.h"

namespace {

typedef int (*Hook)(const char *name, const void *a, const void *b);
std::atomic<Hook> g_hook{nullptr};
std::mutex g_mu;
std::map<void *, size_t> g_mem;     // device allocations
size_t g_held = 0, g_room = 256ull << 30;
std::set<void *> g_events;          // alive
std::atomic<uint64_t> g_bad{~0ull}; // the next load's first bad element
std::atomic<int> g_device{0};
std::atomic<bool> g_hold{false};
std::vector<std::pair<hipHostFn_t, void *>> g_host_funcs;

hipError_t ask(const char *name, const void *a = nullptr, const void *b = nullptr) {
    Hook h = g_hook.load();
    return h ? (hipError_t)h(name, a, b) : hipSuccess;
}

}  // namespace

#define ASK(...)                          \
    do {                                  \
        hipError_t e_ = ask(__VA_ARGS__); \
        if (e_ != hipSuccess) return e_;  \
    } while (0)

extern "C" {

void stub_hook(Hook h) { g_hook = h; }
void stub_room(size_t bytes) { g_room = bytes; }
void stub_bad_element(uint64_t bad) { g_bad = bad; }
void stub_hold_host_funcs(int on) { g_hold = on != 0; }
int stub_event_alive(void *e) {
    std::lock_guard<std::mutex> g(g_mu);
    return g_events.count(e) != 0;
}
size_t stub_held(void) {
    std::lock_guard<std::mutex> g(g_mu);
    return g_held;
}
// Runs the held completion callbacks.
void stub_run_host_funcs(void) {
    std::vector<std::pair<hipHostFn_t, void *>> f;
    {
        std::lock_guard<std::mutex> g(g_mu);
        f.swap(g_host_funcs);
    }
    for (auto &p : f) p.first(p.second);
}

hipError_t hipMalloc(void **p, size_t bytes) {
    ASK("hipMalloc", (const void *)bytes);
    std::lock_guard<std::mutex> g(g_mu);
    if (g_held + bytes > g_room) return hipErrorOutOfMemory;
    const size_t len = bytes ? bytes : 1;
    *p = mmap(nullptr, len, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (*p == MAP_FAILED) return hipErrorOutOfMemory;
    g_mem[*p] = len;
    g_held += len;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    ASK("hipFree", p);
    if (!p) return hipSuccess;
    std::lock_guard<std::mutex> g(g_mu);
    auto it = g_mem.find(p);
    if (it == g_mem.end()) return hipErrorInvalidValue;
    g_held -= it->second;
    munmap(p, it->second);
    g_mem.erase(it);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
    ASK("hipHostMalloc", (const void *)bytes);
    *p = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (*p == MAP_FAILED) return hipErrorOutOfMemory;
    std::lock_guard<std::mutex> g(g_mu);
    g_mem[*p] = bytes;
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    ASK("hipHostFree", p);
    std::lock_guard<std::mutex> g(g_mu);
    auto it = g_mem.find(p);
    if (it == g_mem.end()) return hipErrorInvalidValue;
    munmap(p, it->second);
    g_mem.erase(it);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *room, size_t *all) {
    ASK("hipMemGetInfo");
    std::lock_guard<std::mutex> g(g_mu);
    *room = g_room - g_held;
    *all = g_room;
    return hipSuccess;
}
// Device `at` of an address: device 1 above 2^60 (no memory there), else 0.
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    ASK("hipPointerGetAttributes", p);
    memset(a, 0, sizeof(*a));
    a->type = hipMemoryTypeDevice;
    a->device = (uint64_t)p >> 60 ? 1 : 0;
    a->devicePointer = (void *)p;
    return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) {
    ASK("hipMemcpy", dst, src);
    memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind k, hipStream_t s) {
    ASK("hipMemcpyAsync", dst, s);
    // (image copies of the stand-in kernels hold nothing; foreign addresses stay untouched)
    if (k != hipMemcpyDeviceToDevice) memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int, size_t, hipStream_t s) {
    ASK("hipMemsetAsync", p, s);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = g_device;
    return hipSuccess;
}
hipError_t hipSetDevice(int d) {
    g_device = d;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "success" : "stub error"; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static unsigned char scratch[64 << 20];
    *p = scratch;
    return hipSuccess;
}

hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    ASK("hipEventCreate");
    std::lock_guard<std::mutex> g(g_mu);
    *e = (hipEvent_t) new char;
    g_events.insert(*e);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
// (never given back to the allocator, so that a handle names one event)
hipError_t hipEventDestroy(hipEvent_t e) {
    {
        std::lock_guard<std::mutex> g(g_mu);
        g_events.erase(e);
    }
    return ask("hipEventDestroy", e);
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    ASK("hipEventRecord", e, s);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    ASK("hipEventQuery", e);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    ASK("hipEventSynchronize", e);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    ASK("hipEventElapsedTime");
    *ms = 1.0f;
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned flags) {
    ASK("hipStreamCreate", (const void *)(size_t)flags);
    *s = (hipStream_t) new char;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return ask("hipStreamDestroy", s); }
hipError_t hipStreamSynchronize(hipStream_t s) { return ask("hipStreamSynchronize", s); }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    return ask("hipStreamWaitEvent", s, e);
}
hipError_t hipLaunchHostFunc(hipStream_t s, hipHostFn_t f, void *arg) {
    ASK("hipLaunchHostFunc", s);
    if (g_hold) {
        std::lock_guard<std::mutex> g(g_mu);
        g_host_funcs.emplace_back(f, arg);
    } else {
        f(arg);
    }
    return hipSuccess;
}
// A stream named by an odd handle is under capture.
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c) {
    ASK("hipStreamIsCapturing", s);
    *c = ((size_t)s & 1) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    ASK("hipStreamBeginCapture", s);
    return ((size_t)s & 1) ? hipErrorIllegalState : hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
    ASK("hipStreamEndCapture", s);
    *g = (hipGraph_t) new char;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    ASK("hipGraphInstantiate");
    *x = (hipGraphExec_t) new char;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) { return ask("hipGraphLaunch", x, s); }

hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t s) {
    return ask("hipLaunchKernel", s);
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *,
                           dim3 *, dim3 *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}

}  // extern "C"

namespace dart {

hipError_t launch_plain(const RayView &v, const RenderSums &, hipStream_t s) {
    return ask("launch_plain", v.st.jplane, s);
}
hipError_t launch_batch(int, bool, int variant, const BatchLaunch &bl, int, hipStream_t s) {
    ASK("launch_batch", bl.views, (const void *)(size_t)variant);
    ASK("launch_batch parts", bl.parts, (const void *)(size_t)bl.n_tiles);
    return ask("launch_batch on", s);
}
hipError_t launch_finish(const RayView *, const Tile *, uint32_t, uint32_t, const double *,
                         hipStream_t s) {
    return ask("launch_finish", s);
}
hipError_t launch_mark(const RayView &, uint32_t *, int, bool, hipStream_t s) {
    return ask("launch_mark", s);
}
hipError_t launch_popcount(const uint32_t *, uint64_t, unsigned long long *out, hipStream_t s) {
    ASK("launch_popcount", s);
    *out = 0;
    return hipSuccess;
}
hipError_t launch_convert(int, int, const void *, const void *, int32_t, int32_t, const StackDev &,
                          void *data, void *plane, unsigned long long *err, hipStream_t) {
    ASK("launch_convert", data, plane);
    const uint64_t bad = g_bad.exchange(~0ull);
    if (bad < *err) *err = bad;
    return hipSuccess;
}
hipError_t launch_rebrick(int, const StackDev &, const StackDev &, void *dst, void *plane,
                          hipStream_t) {
    return ask("launch_rebrick", dst, plane);
}
hipError_t launch_read_epoch(const StackDev &, int32_t, void *, void *, hipStream_t s) {
    return ask("launch_read_epoch", s);
}
hipError_t launch_pack_j(int, const void *records, void *, uint64_t, hipStream_t s) {
    return ask("launch_pack_j", records, s);
}
hipError_t launch_pack_jplane(int, const void *records, void *, uint64_t, hipStream_t s) {
    return ask("launch_pack_jplane", records, s);
}
hipError_t launch_pack_pairs(const void *plane, void *, uint64_t, int32_t, hipStream_t s) {
    return ask("launch_pack_pairs", plane, s);
}
hipError_t launch_fill_u64(unsigned long long *p, uint64_t n, unsigned long long value,
                           hipStream_t s) {
    ASK("launch_fill_u64", p, s);
    for (uint64_t i = 0; i < n; i++) p[i] = value;
    return hipSuccess;
}
hipError_t launch_begin(unsigned long long *clear, size_t n_clear, void *dst, const void *src,
                        size_t n_copy, const Run *, size_t, Tile *, hipStream_t s) {
    ASK("launch_begin", n_copy ? dst : nullptr, s);
    if (n_copy) memcpy(dst, src, 8 * n_copy);
    if (n_clear) memset(clear, 0, 8 * n_clear);
    return hipSuccess;
}
hipError_t launch_totals(const RenderSums &, int32_t n, void *host, hipStream_t s) {
    ASK("launch_totals", s);
    memset(host, 0, 16 * (size_t)n);
    return hipSuccess;
}
hipError_t launch_copy(void *, const void *, uint64_t, hipStream_t s) {
    return ask("launch_copy", s);
}

}  // namespace dart
