// The HIP runtime calls that libharvest makes, for tests of its host code on a machine without a GPU: device memory is host
// memory, kernels do not run, every call is written down in order, and any call can be told to fail.  Linked with the host half of
// harvest.hip (hipcc --offload-host-only); nothing here ever reaches a GPU or is part of the product library.
//
// The log has a line per call: its name and what it was about - stream and event numbers are handed out in the order of creation
// (stream 0 is the null stream), a launch names its kernel, its stream and its grid.
#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <vector>

namespace {
std::string g_log, g_taken, g_fail_call;
int g_fail_nth = 0, g_streams = 0, g_events = 0;
hipError_t g_last = hipSuccess;                          // of the latest launch
std::map<size_t, std::vector<void *>> g_pinned;
std::vector<unsigned char> g_symbol_store;
// filled by constructors of the other file, which may run before this one's
std::map<const void *, std::string> &kernels() { static std::map<const void *, std::string> m; return m; }
std::map<const void *, size_t> &symbols() { static std::map<const void *, size_t> m; return m; }
const void *g_capturing = nullptr;
hipStreamCaptureMode g_mode = hipStreamCaptureModeGlobal;
bool g_not_ready = false;
struct Config { dim3 grid, block; size_t shared; hipStream_t s; };
std::vector<Config> g_config;

struct Handle { int number; unsigned flags; };
int number_of(const void *h) { return h ? ((const Handle *)h)->number : 0; }

void say(const char *fmt, ...)
{
    char line[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(line, sizeof line, fmt, ap);
    va_end(ap);
    g_log += line;
    g_log += '\n';
}
hipError_t outcome(const char *call)
{
    if (g_fail_nth <= 0 || g_fail_call != call || --g_fail_nth) return hipSuccess;
    g_log += "  failed\n";
    return hipErrorUnknown;
}
void *memory(size_t bytes) { return aligned_alloc(256, (bytes + 255) & ~(size_t)255); }
hipError_t launch(const char *call, const void *f, dim3 g, dim3 b, hipStream_t s)
{
    say("%s %s stream %d grid %u,%u,%u block %u", call, kernels()[f].c_str(), number_of(s), g.x, g.y, g.z, b.x);
    return g_last = outcome(call);
}
}  // namespace

extern "C" {
// ---- what the tests call ----
const char *fake_log()                                   // the log since the last time it was asked for
{
    g_taken.swap(g_log);
    g_log.clear();
    return g_taken.c_str();
}
void fake_fail(const char *call, int nth) { g_fail_call = call; g_fail_nth = nth; }      // the nth such call from now on; 0: none
int fake_fail_pending() { return g_fail_nth > 0; }
void fake_capture(const void *stream) { g_capturing = stream; }                         // null: nothing is being recorded
void fake_not_ready(int yes) { g_not_ready = yes; }                                     // what events answer from now on
void *fake_stream() { return new Handle{ ++g_streams, 0 }; }
int fake_number(const void *handle) { return number_of(handle); }
void *fake_pinned(size_t bytes, size_t nth) { return nth < g_pinned[bytes].size() ? g_pinned[bytes][nth] : nullptr; }
size_t fake_pinned_count(size_t bytes) { return g_pinned[bytes].size(); }

// ---- what hipcc's host code calls ----
char HIP_FATBIN[8] __attribute__((visibility("hidden")));
void **__hipRegisterFatBinary(const void *) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    kernels()[host] = name;
}
void __hipRegisterVar(void **, void *var, char *, char *, int, size_t size, int, int) { symbols()[var] = size; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s)
{
    g_config.push_back({ grid, block, shared, s });
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *s)
{
    const Config c = g_config.back();
    g_config.pop_back();
    *grid = c.grid; *block = c.block; *shared = c.shared; *s = c.s;
    return hipSuccess;
}

// ---- the runtime ----
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "as the test asked for"; }
hipError_t hipGetLastError()
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
hipError_t hipGetSymbolAddress(void **ptr, const void *symbol)
{
    if (g_symbol_store.empty()) g_symbol_store.resize(symbols()[symbol] + 256);
    *ptr = (void *)(((uintptr_t)g_symbol_store.data() + 255) & ~(uintptr_t)255);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t bytes)
{
    if (hipError_t e = outcome("hipMalloc")) return e;
    *p = memory(bytes);
    return hipSuccess;
}
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned)
{
    if (hipError_t e = outcome("hipHostMalloc")) return e;
    *p = memory(bytes);
    g_pinned[bytes].push_back(*p);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned)
{
    *d = h;
    return outcome("hipHostGetDevicePointer");
}
hipError_t hipMemset(void *p, int v, size_t bytes)
{
    say("hipMemset");
    memset(p, v, bytes);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int v, size_t bytes, hipStream_t s)
{
    say("hipMemsetAsync stream %d", number_of(s));
    memset(p, v, bytes);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t bytes, hipMemcpyKind)
{
    memcpy(d, s, bytes);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *src, size_t bytes, hipMemcpyKind, hipStream_t s)
{
    say("hipMemcpyAsync stream %d", number_of(s));
    if (hipError_t e = outcome("hipMemcpyAsync")) return e;
    memcpy(d, src, bytes);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { say("hipDeviceSynchronize"); return outcome("hipDeviceSynchronize"); }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned flags)
{
    *s = (hipStream_t) new Handle{ ++g_streams, flags };
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { delete (Handle *)s; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s)
{
    say("hipStreamSynchronize stream %d", number_of(s));
    return outcome("hipStreamSynchronize");
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st)
{
    *st = g_capturing && s == g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    say("hipStreamWaitEvent stream %d event %d", number_of(s), number_of(e));
    return outcome("hipStreamWaitEvent");
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned flags)
{
    if (hipError_t r = outcome("hipEventCreateWithFlags")) return r;
    *e = (hipEvent_t) new Handle{ ++g_events, flags };
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Handle *)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    say("hipEventRecord stream %d event %d%s", number_of(s), number_of(e),
        ((Handle *)e)->flags & hipEventDisableSystemFence ? " no-system-fence" : "");
    return outcome("hipEventRecord");
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *mode)
{
    std::swap(*mode, g_mode);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e)
{
    say("hipEventQuery event %d%s", number_of(e), g_mode == hipStreamCaptureModeRelaxed ? " relaxed" : "");
    if (g_capturing && g_mode != hipStreamCaptureModeRelaxed) return g_last = hipErrorStreamCaptureUnsupported;
    return g_not_ready ? hipErrorNotReady : hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    say("hipEventSynchronize event %d%s", number_of(e), ((Handle *)e)->flags & hipEventDisableSystemFence ? " no-system-fence" : "");
    return outcome("hipEventSynchronize");
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t, hipStream_t s)
{
    return launch("hipLaunchKernel", f, grid, block, s);
}
hipError_t hipExtLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t, hipStream_t s, hipEvent_t, hipEvent_t, int)
{
    return launch("hipExtLaunchKernel", f, grid, block, s);
}
}  // extern "C"
