// Stand-in for the HIP runtime: memory is host memory, kernels do nothing, and
// every call is counted.  Calls can be made to block or to fail by name, so
// that tests see how the library's host code orders its calls, on several
// threads too, with no GPU.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <condition_variable>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>

namespace {
std::mutex mu;
std::condition_variable cv;
std::map<std::string, long> calls, failing;
std::map<std::string, bool> holding;
std::map<void *, int> events;   // times recorded
int held = 0, inside = 0, beside_cooperative = 0;
bool capturing = false;
long blocks = 0;                // of hipLaunchKernel
int occupancy = 1;
thread_local dim3 t_grid, t_block;
thread_local size_t t_shared;
thread_local hipStream_t t_stream;

struct Call {
    bool ok = true;
    explicit Call(const char *name)
    {
        std::unique_lock<std::mutex> g(mu);
        inside++;
        calls[name]++;
        if (holding[name]) {
            held++;
            cv.notify_all();
            cv.wait(g, [&] { return !holding[name]; });
            held--;
        }
        if (failing[name] > 0) {
            failing[name]--;
            ok = false;
        }
    }
    ~Call()
    {
        std::lock_guard<std::mutex> g(mu);
        inside--;
    }
};
}  // namespace

#define CALL()            \
    Call call(__func__);  \
    if (!call.ok) return hipErrorUnknown

extern "C" {
long stub_calls(const char *name) { std::lock_guard<std::mutex> g(mu); return calls[name]; }
long stub_blocks(void) { std::lock_guard<std::mutex> g(mu); return blocks; }
void stub_reset(void) { std::lock_guard<std::mutex> g(mu); calls.clear(); blocks = 0; beside_cooperative = 0; }
void stub_fail(const char *name, long n) { std::lock_guard<std::mutex> g(mu); failing[name] = n; }
void stub_hold(const char *name) { std::lock_guard<std::mutex> g(mu); holding[name] = true; }
void stub_wait_held(int n) { std::unique_lock<std::mutex> g(mu); cv.wait(g, [&] { return held >= n; }); }
void stub_release(const char *name) { { std::lock_guard<std::mutex> g(mu); holding[name] = false; } cv.notify_all(); }
void stub_capturing(int on) { std::lock_guard<std::mutex> g(mu); capturing = on != 0; }
void stub_occupancy(int n) { std::lock_guard<std::mutex> g(mu); occupancy = n; }
int stub_beside_cooperative(void) { std::lock_guard<std::mutex> g(mu); return beside_cooperative; }

hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st)
{
    t_grid = g, t_block = b, t_shared = s, t_stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st)
{
    *g = t_grid, *b = t_block, *s = t_shared, *st = t_stream;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { static void *p; return &p; }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { CALL(); *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { CALL(); return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static char mem[64 << 20]; *p = mem; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n)
{
    CALL();
    n = (n + 255) / 256 * 256;
    *p = aligned_alloc(256, n);
    return *p ? (memset(*p, 0, n), hipSuccess) : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { CALL(); free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { CALL(); *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { CALL(); free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { CALL(); memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { CALL(); memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { CALL(); memset(d, v, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { CALL(); *s = (hipStream_t)calloc(1, 64); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { CALL(); free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { CALL(); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { CALL(); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    CALL();
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { CALL(); return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { CALL(); *g = nullptr; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { CALL(); *e = (hipEvent_t)calloc(1, 64); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { CALL(); *e = (hipEvent_t)calloc(1, 64); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { CALL(); free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { CALL(); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { CALL(); return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { CALL(); *ms = 1.0f; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) { CALL(); *e = (hipGraphExec_t)calloc(1, 8); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { CALL(); free(e); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { CALL(); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { CALL(); return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { CALL(); *n = occupancy; return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3 g, dim3, void **, size_t, hipStream_t)
{
    CALL();
    std::lock_guard<std::mutex> l(mu);
    blocks += g.x;
    return hipSuccess;
}
hipError_t hipLaunchCooperativeKernel(const void *, dim3, dim3, void **, unsigned, hipStream_t)
{
    CALL();
    for (int i = 0; i < 20; i++) {
        std::this_thread::sleep_for(std::chrono::microseconds(50));
        std::lock_guard<std::mutex> g(mu);
        if (inside - 1 > beside_cooperative) beside_cooperative = inside - 1;
    }
    return hipSuccess;
}
}
