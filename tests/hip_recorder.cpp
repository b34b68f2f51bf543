// Stands in for the HIP runtime on a machine without a GPU (preloaded by
// tests/test_call_order.py): device memory is host memory, kernels do nothing
// (but k_store_list, which copies its argument), and every call that orders work
// on a stream is written to a log.
#define __HIP_PLATFORM_AMD__ 1
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::string g_log, g_taken;
std::map<const void *, std::string> g_kernels;
bool g_ready = false;
hipStream_t g_capturing = nullptr;
uintptr_t g_next = 0x100;
struct { dim3 g, b; size_t sh; hipStream_t s; } g_config;

hipError_t note(const char *what, const void *a, const void *b = nullptr) {
    char line[256];
    std::snprintf(line, sizeof line, b ? "%s %lx %lx\n" : "%s %lx\n", what, (unsigned long)a, (unsigned long)b);
    g_log += line;
    return hipSuccess;
}

hipError_t alloc(void **p, size_t n) { return (*p = std::calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
}  // namespace

extern "C" {
// Lines since the last call; whether recorded events have finished; the stream under capture.
const char *rec_take() {
    g_taken.swap(g_log);
    g_log.clear();
    return g_taken.c_str();
}
void rec_events_ready(int ready) { g_ready = ready != 0; }
void rec_capturing(hipStream_t s) { g_capturing = s; }

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *fn, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *,
                           int *) {
    int st = 0;
    char *d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    std::string s = d ? d : name;
    std::free(d);
    const size_t at = s.find("k_");
    g_kernels[fn] = s.substr(at == std::string::npos ? 0 : at, s.find('(') - at);
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s) {
    g_config = {g, b, sh, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *s) {
    *g = g_config.g; *b = g_config.b; *sh = g_config.sh; *s = g_config.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3, dim3, void **args, size_t, hipStream_t s) {
    if (g_kernels[fn] == "k_store_list") std::memcpy(*(void **)args[0], args[2], *(int *)args[1] * size_t(16));
    return note(("launch " + g_kernels[fn]).c_str(), s);
}

hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 3; return hipSuccess; }
void *rec_symbol() { static void *m = std::calloc(1, 64 << 20); return m; }  // the library's static device array
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = rec_symbol(); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }

hipError_t hipMalloc(void **p, size_t n) { return alloc(p, n); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return alloc(p, n); }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
    std::memcpy(d, s, n);
    return note("copy", st);
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)(g_next += 0x10); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return note("sync", s); }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { return note("wait", s, e); }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) {
    *st = g_capturing && s == g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)(g_next += 0x10); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return g_ready ? hipSuccess : hipErrorNotReady; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return note("record", s, e); }
hipError_t hipEventSynchronize(hipEvent_t e) { return note("eventsync", e); }
}
