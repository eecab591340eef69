// The HIP calls of the library on host memory, for tests of its host code without a GPU: copies are
// done at once, kernels do nothing, and what the calls did is counted.  A stream that is being
// captured takes work without running it and refuses to be waited for.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>

struct ihipStream_t {
    bool capturing;
};
struct ihipEvent_t {
    int unused;
};

namespace {

std::mutex mu;
std::map<void *, size_t> device_memory, pinned_memory;
std::set<hipStream_t> streams;
std::set<hipEvent_t> events;
thread_local int device = 0;

// counters by name (stub_count)
long wrong_device, captured, launches, waits, copies;
int expected_device = -1;      // >= 0: calls that belong to a device are counted when it is not current
size_t malloc_limit = ~(size_t)0;

void belongs_to_device()
{
    if (expected_device >= 0 && device != expected_device) wrong_device++;
}

// whether work on the stream runs (it is captured otherwise)
bool runs(hipStream_t s)
{
    if (s && s->capturing) {
        captured++;
        return false;
    }
    return true;
}

size_t total(const std::map<void *, size_t> &m)
{
    size_t n = 0;
    for (auto &p : m) n += p.second;
    return n;
}

}  // namespace

extern "C" {

extern const char __hip_fatbin[8];
const char __hip_fatbin[8] = {0};

void *stub_stream()
{
    std::lock_guard<std::mutex> l(mu);
    hipStream_t s = new ihipStream_t{false};
    return s;
}
void stub_stream_free(void *s) { delete static_cast<hipStream_t>(s); }
void stub_capture(void *s, int on) { static_cast<hipStream_t>(s)->capturing = on != 0; }
void stub_expect_device(int d) { expected_device = d; }
void stub_malloc_limit(size_t n) { malloc_limit = n; }
void stub_reset() { wrong_device = captured = launches = waits = copies = 0; }
long stub_count(const char *what)
{
    std::lock_guard<std::mutex> l(mu);
    const std::map<std::string, long> c = {{"wrong_device", wrong_device},
                                           {"captured", captured},
                                           {"launches", launches},
                                           {"waits", waits},
                                           {"copies", copies},
                                           {"device_bytes", (long)total(device_memory)},
                                           {"pinned_bytes", (long)total(pinned_memory)},
                                           {"streams", (long)streams.size()},
                                           {"events", (long)events.size()}};
    return c.at(what);
}

hipError_t hipGetDevice(int *d)
{
    *d = device;
    return hipSuccess;
}
hipError_t hipSetDevice(int d)
{
    device = d;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetLastError() { return hipSuccess; }

hipError_t hipMalloc(void **p, size_t n)
{
    std::lock_guard<std::mutex> l(mu);
    belongs_to_device();
    if (n > malloc_limit) return hipErrorOutOfMemory;
    *p = std::calloc(1, n);
    device_memory[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::lock_guard<std::mutex> l(mu);
    device_memory.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    std::lock_guard<std::mutex> l(mu);
    belongs_to_device();
    *p = std::calloc(1, n);
    pinned_memory[*p] = n;
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    std::lock_guard<std::mutex> l(mu);
    pinned_memory.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    std::lock_guard<std::mutex> l(mu);
    copies++;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    std::lock_guard<std::mutex> l(mu);
    if (!runs(st)) return hipSuccess;
    copies++;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n)
{
    std::memset(d, v, n);
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    std::lock_guard<std::mutex> l(mu);
    belongs_to_device();
    *s = new ihipStream_t{false};
    streams.insert(*s);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    std::lock_guard<std::mutex> l(mu);
    streams.erase(s);
    delete s;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    std::lock_guard<std::mutex> l(mu);
    waits++;
    return s && s->capturing ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c)
{
    *c = s && s->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }

hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    std::lock_guard<std::mutex> l(mu);
    *e = new ihipEvent_t{};
    events.insert(*e);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    std::lock_guard<std::mutex> l(mu);
    events.erase(e);
    delete e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 0;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorNotSupported; }

hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t s)
{
    std::lock_guard<std::mutex> l(mu);
    belongs_to_device();
    if (runs(s)) launches++;
    return hipSuccess;
}
static thread_local struct {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
} call;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s)
{
    call = {g, b, sh, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *s)
{
    *g = call.grid;
    *b = call.block;
    *sh = call.shared;
    *s = call.stream;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}

}  // extern "C"
