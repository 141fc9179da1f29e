// A HIP runtime for tests on the CPU: libnf's host code runs against it, in
// order and at once, and every call that matters to it is written to a log.
// "Device" memory is host memory, kernels do nothing.
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

#include <string>

static std::string g_log;
static hipStream_t g_captured = nullptr;  // a caller's stream that is being captured
static hipStream_t g_own = nullptr;       // the library's stream under capture
static long g_next = 1;

static std::string g_grids;

static void note(const char* what) { (g_log += what) += '\n'; }
template <class T>
static T handle() { return (T)(g_next++ * 4096); }

extern "C" {
const char* stub_log(void) { return g_log.c_str(); }
const char* stub_grids(void) { return g_grids.c_str(); }  // of the launches, one number each
void stub_clear(void) { g_log.clear(); g_grids.clear(); }
void stub_capture(void* s) { g_captured = (hipStream_t)s; }

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
static dim3 g_grid, g_block;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) { g_grid = g; g_block = b; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* sh, hipStream_t* s)
{
    *g = g_grid; *b = g_block; *sh = 0; *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3, void**, size_t, hipStream_t)
{
    note(g_own ? "record" : "kernel");
    g_grids += std::to_string(grid.x) + ' ';
    return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t, hipEvent_t, hipEvent_t, int) { note("kernel"); return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
hipError_t hipDeviceSynchronize(void) { note("device synchronize"); return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = *t = (size_t)1 << 30; return hipSuccess; }

hipError_t hipMalloc(void** p, size_t n) { note("malloc"); *p = aligned_alloc(256, (n + 255) & ~(size_t)255); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { note("free"); free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { note("copy"); memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { note("copy"); memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { note("fill"); memset(d, v, n); return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = handle<hipStream_t>(); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { note("stream synchronize"); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st)
{
    *st = s && s == g_captured ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { g_own = s; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { g_own = nullptr; *g = handle<hipGraph_t>(); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) { *e = handle<hipGraphExec_t>(); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { note("graph launch"); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { note("graph destroy"); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { note("exec destroy"); return hipSuccess; }

hipError_t hipEventCreate(hipEvent_t* e) { *e = handle<hipEvent_t>(); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = handle<hipEvent_t>(); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { note("event record"); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { note("event synchronize"); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1; return hipSuccess; }
}
