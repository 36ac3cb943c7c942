// A HIP runtime without a device, for tests of the library's host side on the CPU: loaded with RTLD_GLOBAL before
// libclada.so it takes every runtime call the library makes.  Kernels are not run; their launches are written down, in
// order, as "name gridx gridy gridz blockx lane" (one per line; lane: 1 on a stream that the library made), and the n-th launch from now can be made to fail.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>

static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
static std::string g_log, g_out;
static long g_fail_in = -1;          // launches until one is refused, or -1
static int g_capture;                // what hipStreamIsCapturing answers
static int g_streams, g_events;      // created since they were last asked for
static hipError_t g_last = hipSuccess;
static struct { dim3 grid, block; size_t lds; hipStream_t st; } g_cfg;

static hipError_t refuse(hipError_t e) { g_last = e; return e; }
static hipError_t launch(const void *fn, dim3 g, dim3 b, hipStream_t st)
{
    if (g_fail_in >= 0 && g_fail_in-- == 0) return refuse(hipErrorLaunchFailure);
    char line[512];
    std::snprintf(line, sizeof(line), "%s %u %u %u %u %d\n", names()[fn].c_str(), g.x, g.y, g.z, b.x, st != nullptr);
    g_log += line;
    return hipSuccess;
}

extern "C" {
// controls of the tests
const char *fake_take_log(void) { g_out.swap(g_log); g_log.clear(); return g_out.c_str(); }
void fake_fail_launch(long n) { g_fail_in = n; }
void fake_capturing(int on) { g_capture = on; }
int fake_take_streams(void) { const int n = g_streams; g_streams = 0; return n; }
int fake_take_events(void) { const int n = g_events; g_events = 0; return n; }

// what the compiler emits around kernels
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names()[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) { g_cfg = {g, b, lds, st}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *st) { *g = g_cfg.grid; *b = g_cfg.block; *lds = g_cfg.lds; *st = g_cfg.st; return hipSuccess; }

hipError_t hipLaunchKernel(const void *fn, dim3 g, dim3 b, void **, size_t, hipStream_t st) { return launch(fn, g, b, st); }
hipError_t hipExtLaunchKernel(const void *fn, dim3 g, dim3 b, void **, size_t, hipStream_t st, hipEvent_t, hipEvent_t, int) { return launch(fn, g, b, st); }
hipError_t hipGetLastError(void) { const hipError_t e = g_last; g_last = hipSuccess; return e; }
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "refused by the test"; }

hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) { std::memset(p, 0, sizeof(*p)); p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { return posix_memalign(p, 256, n ? n : 256) ? refuse(hipErrorOutOfMemory) : hipSuccess; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { static char h; ++g_streams; *s = (hipStream_t)&h; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { static char h; ++g_events; *e = (hipEvent_t)&h; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 1; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **, const void *) { return refuse(hipErrorInvalidSymbol); }
}
