// Host stand-in for the HIP runtime calls of libvms, for tests of the host side
// on a machine without a GPU: memory is host memory, copies are immediate,
// kernels do not run, and every call that orders streams is written to a log.
// Two kernels leave what the set-up needs: corner labels (1 for x at or beyond
// split_x) and the number of kept points of an INTERCEPTED element. A launch of a
// chosen kernel, or a chosen call, can be made to fail.
//
// Log lines: "launch STREAM KERNEL GRID", "record EVENT STREAM", "wait STREAM EVENT",
// "sync STREAM".
#include "kernels.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::string g_log, g_fail_kernel, g_fail_call;
int g_fail_nth = 0, g_split_x = 0, g_kept = 0;
hipError_t g_last = hipSuccess;
std::map<const void *, std::string> g_name;
dim3 g_grid, g_block;
size_t g_shmem;
hipStream_t g_stream;
uintptr_t g_next = 0x1000;

void note(const char *fmt, const void *a, const char *b) {
    char s[512];
    std::snprintf(s, sizeof s, fmt, (unsigned long)(uintptr_t)a, b);
    g_log += s;
}
// the chosen call fails the nth time it is made
hipError_t result(const char *call) {
    if (g_fail_call == call && g_fail_nth > 0 && --g_fail_nth == 0) return g_last = hipErrorUnknown;
    return hipSuccess;
}
std::string hex(const void *p) {
    char s[32];
    std::snprintf(s, sizeof s, "%lx", (unsigned long)(uintptr_t)p);
    return s;
}
}  // namespace

extern "C" {

const char *stand_in_log() { return g_log.c_str(); }
void stand_in_reset(const char *fail_kernel, const char *fail_call, int nth) {
    g_log.clear();
    g_fail_kernel = fail_kernel;
    g_fail_call = fail_call;
    g_fail_nth = nth;
    g_last = hipSuccess;
}
void stand_in_config(int split_x, int kept) {
    g_split_x = split_x;
    g_kept = kept;
}

void **__hipRegisterFatBinary(const void *) {
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *dev, const char *, unsigned, void *, void *, void *, void *, int *) {
    g_name[f] = dev;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
    g_grid = g; g_block = b; g_shmem = s; g_stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st) {
    *g = g_grid; *b = g_block; *s = g_shmem; *st = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t, hipStream_t st) {
    const std::string &k = g_name[f];
    if (!g_fail_kernel.empty() && k.find(g_fail_kernel) != std::string::npos && g_fail_nth > 0 && --g_fail_nth == 0)
        return g_last = hipErrorLaunchFailure;
    note("launch %lx %s", st, k.c_str());
    g_log += " " + std::to_string(grid.x) + "\n";
    if (k.find("k_vertex_labels") != std::string::npos) {
        const int64_t n = *(const int64_t *)args[2];
        const int32_t *ix = *(const int32_t *const *)args[3];
        uint8_t *lab = *(uint8_t *const *)args[6];
        for (int64_t i = 0; i < n; ++i) lab[i] = ix[i] >= g_split_x;
    } else if (k.find("k_subquad") != std::string::npos && *(const int *)args[3] == 0) {
        const vmsk::SubqArgs &a = *(const vmsk::SubqArgs *)args[2];
        for (int64_t i = 0; i < a.n; ++i) a.cnt[i] = g_kept;
    }
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n) { return (*p = std::calloc(1, n ? n : 1)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = nullptr; return hipErrorUnknown; }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)(g_next += 16); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { note("sync %lx%s\n", s, ""); return result("sync"); }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    const hipError_t r = result("wait");
    if (r == hipSuccess) note("wait %lx %s\n", s, hex(e).c_str());
    return r;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorUnknown; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorUnknown; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorUnknown; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorUnknown; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)(g_next += 16); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    const hipError_t r = result("record");
    if (r == hipSuccess) note("record %lx %s\n", e, hex(s).c_str());
    return r;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 0.f; return hipSuccess; }

hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *) {
    std::memset(a, 0, sizeof *a);
    a->sharedSizeBytes = 1024;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 12; return hipSuccess; }

}  // extern "C"
