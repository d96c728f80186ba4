// Host-only stand-in for the HIP runtime, preloaded by tests/host_runtime.py: device memory is
// host memory, kernels do nothing, and every allocation, upload and launch is counted.  What the
// library asks of the device can then be checked without one.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<const void *, std::string> names;   // kernel stub -> mangled name
std::map<std::string, long> launches;        // by mangled name
std::map<void *, size_t> blocks;
long allocs, uploads, failed;
size_t held, peak, limit = ~(size_t)0;
hipError_t last = hipSuccess;                // until hipGetLastError takes it
struct { dim3 g, b; size_t lds; hipStream_t s; } conf;
}

extern "C" {
// the tests' side
long host_allocs() { return allocs; }
long host_uploads() { return uploads; }
long host_failed() { return failed; }
size_t host_held() { return held; }
size_t host_peak() { return peak; }
void host_limit(size_t bytes) { limit = bytes; }
void host_reset() { allocs = uploads = failed = 0; peak = held; launches.clear(); }
// launches of kernels whose mangled name holds `part`
long host_launches(const char *part)
{
    long n = 0;
    for (const auto &l : launches)
        if (l.first.find(part) != std::string::npos) n += l.second;
    return n;
}

// the library's side
void **__hipRegisterFatBinary(const void *) { static void *p; return &p; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *) { names[f] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) { conf = {g, b, lds, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) { *g = conf.g; *b = conf.b; *lds = conf.lds; *s = conf.s; return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t, hipStream_t)
{
    if (!g.x || !g.y || g.y > 65535 || !b.x || b.x > 1024) return hipErrorInvalidConfiguration;
    ++launches[names[f]];
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    *p = nullptr;
    if (n > limit || held > limit - n) { ++failed; return last = hipErrorOutOfMemory; }
    *p = calloc(1, n ? n : 1);
    blocks[*p] = n;
    held += n;
    if (held > peak) peak = held;
    ++allocs;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    auto it = blocks.find(p);
    if (it == blocks.end()) return p ? hipErrorInvalidValue : hipSuccess;
    held -= it->second;
    blocks.erase(it);
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { ++uploads; memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t *p, int) { memset(p, 0, sizeof *p); strcpy(p->gcnArchName, "host"); p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { *g = (hipGraph_t)8; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) { *e = (hipGraphExec_t)8; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 2; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static void *m = calloc(1, 1 << 22); *p = m; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
}
