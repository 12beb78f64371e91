// A stand-in for the HIP runtime, so that the library's host code can be run and watched without a GPU:
// it keeps the queues' order, says what was enqueued where, and runs no kernel.  A test decides when a
// stream's work has finished (`finish`, or a call of the library's that waits).
#pragma once
#include <cxxabi.h>
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

namespace fake {

struct Stream {
    unsigned flags = 0;
    uint64_t queued = 0, done = 0;      // operations
    bool capturing = false;
};
struct Event {
    Stream *stream = nullptr;
    uint64_t at = 0;
    bool fired() const { return !stream || stream->done >= at; }
};
struct Launch {
    std::string kernel;                 // name with its template arguments
    Stream *stream;
    dim3 grid, block;
    bool event;                         // a stop event rides on it
};

static Stream null_stream;
static std::vector<Launch> launches;
static std::vector<std::pair<Stream *, Event *>> records, waits;        // hipEventRecord, hipStreamWaitEvent
static void (*watch)(const Launch &, void **args);       // called with every launch, if set
static std::map<const void *, std::string> kernels;
static std::set<void *> device_memory;
static uint64_t mallocs, frees, waited;     // allocations and frees of device memory; waits of the host for unfinished kernels
static bool capture_broken;                 // a call that a capture in progress forbids was made
static int captures;                        // streams being captured (by this thread, in the default, strictest mode)
static thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;

inline Stream *of(hipStream_t s) { return s ? reinterpret_cast<Stream *>(s) : &null_stream; }
inline Event *of(hipEvent_t e) { return reinterpret_cast<Event *>(e); }
inline hipStream_t handle(Stream &s) { return reinterpret_cast<hipStream_t>(&s); }
inline void finish(Stream *s) { s->done = s->queued; }
inline void wait_for(Stream *s, uint64_t at) {
    if (s->done < at) {
        ++waited;
        s->done = at;
    }
}
inline void begin_capture(Stream &s) { s.capturing = true; ++captures; }
inline void end_capture(Stream &s) { s.capturing = false; --captures; }
// what may not be called while a stream is being captured, unless the thread has said that it knows (relaxed mode)
inline bool forbidden() {
    if (captures && mode != hipStreamCaptureModeRelaxed) capture_broken = true;
    return captures && mode != hipStreamCaptureModeRelaxed;
}
inline hipError_t launch(const void *f, dim3 grid, dim3 block, void **args, hipStream_t s, hipEvent_t stop) {
    Stream *st = of(s);
    launches.push_back(Launch{kernels[f], st, grid, block, stop != nullptr});
    if (watch) watch(launches.back(), args);
    if (!st->capturing) ++st->queued;
    if (stop) *of(stop) = Event{st, st->queued};
    return hipSuccess;
}

}  // namespace fake

extern "C" {

static dim3 fake_grid, fake_block;
static size_t fake_shared;
static hipStream_t fake_stream;
extern const char __hip_fatbin[1] = {0};

hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) {
    fake_grid = g; fake_block = b; fake_shared = m; fake_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s) {
    *g = fake_grid; *b = fake_block; *m = fake_shared; *s = fake_stream;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { static void *p; return &p; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *f, char *name, const char *, unsigned, void *, void *, dim3 *, dim3 *, int *) {
    int bad = 0;
    char *plain = abi::__cxa_demangle(name, nullptr, nullptr, &bad);
    fake::kernels[f] = plain ? plain : name;
    std::free(plain);
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t, hipStream_t s) { return fake::launch(f, g, b, a, s, nullptr); }
hipError_t hipExtLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t, hipStream_t s, hipEvent_t, hipEvent_t stop, int) {
    return fake::launch(f, g, b, a, s, stop);
}

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }

hipError_t hipMalloc(void **p, size_t n) {
    if (fake::forbidden()) return hipErrorStreamCaptureUnsupported;
    *p = std::malloc(n);
    fake::device_memory.insert(*p);
    ++fake::mallocs;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    fake::device_memory.erase(p);
    ++fake::frees;
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
// (a copy has ended when the call returns: only kernels can be unfinished here)
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) { a->type = hipMemoryTypeDevice; return hipSuccess; }
hipError_t hipMemGetAddressRange(hipDeviceptr_t *, size_t *, hipDeviceptr_t) { return hipErrorInvalidValue; }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned flags) {
    fake::Stream *st = new fake::Stream;
    st->flags = flags;
    *s = fake::handle(*st);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { delete fake::of(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { fake::wait_for(fake::of(s), fake::of(s)->queued); return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { ++fake::waited; return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t s) { return fake::of(s)->done < fake::of(s)->queued ? hipErrorNotReady : hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c) {
    *c = fake::of(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) { std::swap(*m, fake::mode); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    fake::Stream *st = fake::of(s);
    if (st->capturing) fake::capture_broken = true;         // an event from outside the capture
    fake::waits.emplace_back(st, fake::of(e));
    return hipSuccess;
}

hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = reinterpret_cast<hipEvent_t>(new fake::Event); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete fake::of(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    fake::Stream *st = fake::of(s);
    *fake::of(e) = fake::Event{st, ++st->queued};
    fake::records.emplace_back(st, fake::of(e));
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    if (fake::forbidden()) return hipErrorStreamCaptureUnsupported;
    return fake::of(e)->fired() ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    if (fake::of(e)->stream) fake::wait_for(fake::of(e)->stream, fake::of(e)->at);
    return hipSuccess;
}

}  // extern "C"
