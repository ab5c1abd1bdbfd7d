// A HIP runtime without a device, for host tests of the library's own objects: memory is host memory
// with a limit, kernels do nothing, copies copy, and a log holds what was called. A test sets what the
// next cooperative launch returns and what its workgroups report.
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

static std::map<void *, size_t> g_mem;
static size_t g_used, g_limit, g_base, g_peak;  // bytes: now, at most, at the last reset, most since
static std::string g_log;
static hipError_t g_last, g_coop = hipSuccess;
static bool g_report;
static unsigned int g_verdict[2], g_at;
static int g_fail_events;

extern "C" {
void host_reset(size_t limit) {
    g_limit = limit;
    g_last = hipSuccess;
    g_base = g_peak = g_used;
    g_log.clear();
    g_coop = hipSuccess;
    g_report = false;
    g_verdict[0] = g_verdict[1] = g_at = 0;
    g_fail_events = 0;
}
size_t host_used() { return g_used; }
size_t host_peak() { return g_peak - g_base; }
const char *host_log() { return g_log.c_str(); }
// The next cooperative launch returns e; the first read-back after it holds error and phases from word
// `at` on.
void host_coop(int e, unsigned int error, unsigned int phases, unsigned int at) {
    g_at = at;
    g_coop = (hipError_t)e;
    g_verdict[0] = error;
    g_verdict[1] = phases;
}
void host_fail_events(int n) { g_fail_events = n; }

static hipError_t ret(hipError_t e) {
    if (e != hipSuccess) g_last = e;
    return e;
}
hipError_t hipMalloc(void **p, size_t n) {
    if (g_used + n > g_limit) {
        g_log += "oom ";
        return ret(hipErrorOutOfMemory);
    }
    *p = calloc(n ? n : 1, 1);
    g_mem[*p] = n;
    g_used += n;
    if (g_used > g_peak) g_peak = g_used;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    g_log += "free ";
    g_used -= g_mem[p];
    g_mem.erase(p);
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned int) {
    *p = calloc(n, 1);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) {
    memcpy(d, s, n);
    if (k == hipMemcpyDeviceToHost && g_report && n >= 4 * g_at + sizeof g_verdict) {
        memcpy((char *)d + 4 * g_at, g_verdict, sizeof g_verdict);
        g_report = false;
    }
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) { return hipMemcpyAsync(d, s, n, k, nullptr); }
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) {
    memset(p, v, n);
    g_log += "set ";
    return hipSuccess;
}
hipError_t hipMemset(void *p, int v, size_t n) { return hipMemsetAsync(p, v, n, nullptr); }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) {
    g_log += "kernel ";
    return hipSuccess;
}
hipError_t hipLaunchCooperativeKernel(const void *, dim3, dim3, void **, unsigned int, hipStream_t) {
    g_log += "coop ";
    g_report = g_coop == hipSuccess;
    return ret(g_coop);
}
hipError_t hipStreamSynchronize(hipStream_t) {
    g_log += "wait ";
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipStreamSynchronize(nullptr); }
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "host test error"; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
int hipGetStreamDeviceId(hipStream_t) { return 0; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    p->warpSize = 64;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
    *n = 2;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static void *array = aligned_alloc(256, 64u << 20);
    *p = array;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    if (g_fail_events && g_fail_events-- == 1) return ret(hipErrorUnknown);
    *e = (hipEvent_t)malloc(1);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
    free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int) {
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return ret(hipErrorNotSupported); }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return ret(hipErrorNotSupported); }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return ret(hipErrorNotSupported); }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return ret(hipErrorNotSupported); }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

// what a compiled launch calls
static dim3 g_grid, g_block;
static size_t g_lds;
static hipStream_t g_stream;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    g_grid = grid;
    g_block = block;
    g_lds = lds;
    g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s) {
    *grid = g_grid;
    *block = g_block;
    *lds = g_lds;
    *s = g_stream;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned int, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
}
