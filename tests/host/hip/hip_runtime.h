// A HIP runtime of two devices for tests of the host code on the CPU: streams and events that
// know their device, copies that are made and counted, captures and graphs without content.
#pragma once

#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

enum hipError_t {
    hipSuccess = 0,
    hipErrorInvalidValue = 1,
    hipErrorOutOfMemory = 2,
    hipErrorInvalidHandle = 400,
    hipErrorStreamCaptureIsolation = 905,
    hipErrorUnknown = 999
};
struct ihipStream_t {
    int device;
    ihipStream_t *origin; // stream that began the capture it is in
};
struct ihipEvent_t {
    int device;
    ihipStream_t *origin;
};
struct ihipGraph {
};
using hipStream_t = ihipStream_t *;
using hipEvent_t = ihipEvent_t *;
using hipGraph_t = ihipGraph *;
using hipGraphExec_t = ihipGraph *;
using hipDevice_t = int;
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };
enum hipMemoryType { hipMemoryTypeUnregistered = 0, hipMemoryTypeHost = 1, hipMemoryTypeDevice = 2 };
struct hipPointerAttribute_t {
    hipMemoryType type;
};
enum hipStreamCaptureMode { hipStreamCaptureModeThreadLocal = 1 };
constexpr unsigned hipStreamNonBlocking = 1, hipEventDisableTiming = 2, hipHostMallocPortable = 1, hipHostMallocDefault = 0;
static const hipStream_t hipStreamLegacy = (hipStream_t)1, hipStreamPerThread = (hipStream_t)2;

namespace fake {
inline thread_local int device = 0;
struct Copy {
    const char *dst;
    size_t bytes;
};
inline std::recursive_mutex lock;
inline std::vector<Copy> copies;          // every hipMemcpyAsync
inline std::map<const char *, size_t> pinned, on_device; // live hipHostMalloc and hipMalloc allocations
inline std::vector<hipStream_t> graph_launches; // the stream of each
inline int streams = 0, events = 0, captures = 0, events_left = 1 << 30, streams_left = 1 << 30;
inline int device_of(hipStream_t s) { return (size_t)s <= 2 ? device : s->device; }
inline bool within(const std::map<const char *, size_t> &blocks, const void *p)
{
    std::lock_guard<std::recursive_mutex> l(lock);
    auto it = blocks.upper_bound((const char *)p);
    return it != blocks.begin() && (const char *)p < (--it)->first + it->second;
}
} // namespace fake

inline hipError_t hipGetDevice(int *d) { return *d = fake::device, hipSuccess; }
inline hipError_t hipSetDevice(int d) { return fake::device = d, hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t *d)
{
    if ((size_t)s <= 2) std::abort(); // only streams that were created
    return *d = s->device, hipSuccess;
}
inline hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    std::lock_guard<std::recursive_mutex> l(fake::lock);
    if (fake::streams_left-- <= 0) return hipErrorOutOfMemory;
    ++fake::streams;
    *s = (hipStream_t)std::malloc(sizeof(ihipStream_t));
    return **s = {fake::device, nullptr}, hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t s)
{
    std::lock_guard<std::recursive_mutex> l(fake::lock);
    --fake::streams;
    std::free(s);
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    std::lock_guard<std::recursive_mutex> l(fake::lock);
    if (fake::events_left-- <= 0) return hipErrorOutOfMemory;
    ++fake::events;
    *e = (hipEvent_t)std::malloc(sizeof(ihipEvent_t));
    return **e = {fake::device, nullptr}, hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e)
{
    std::lock_guard<std::recursive_mutex> l(fake::lock);
    --fake::events;
    std::free(e);
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    if (e->device != fake::device_of(s)) return hipErrorInvalidHandle;
    e->origin = (size_t)s <= 2 ? nullptr : s->origin;
    return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    if (s->origin && !e->origin) return hipErrorStreamCaptureIsolation;
    if (e->origin) s->origin = e->origin;
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(dst, src, n);
    std::lock_guard<std::recursive_mutex> l(fake::lock);
    fake::copies.push_back({(const char *)dst, n});
    return hipSuccess;
}
inline hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) { return std::memcpy(dst, src, n), hipSuccess; }
inline hipError_t hipMalloc(void **p, size_t n)
{
    std::lock_guard<std::recursive_mutex> l(fake::lock);
    *p = std::malloc(n);
    fake::on_device[(const char *)*p] = n;
    return hipSuccess;
}
inline hipError_t hipFree(void *p)
{
    std::lock_guard<std::recursive_mutex> l(fake::lock);
    fake::on_device.erase((const char *)p);
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    std::lock_guard<std::recursive_mutex> l(fake::lock);
    *p = std::malloc(n);
    fake::pinned[(const char *)*p] = n;
    return hipSuccess;
}
inline hipError_t hipHostFree(void *p)
{
    std::lock_guard<std::recursive_mutex> l(fake::lock);
    fake::pinned.erase((const char *)p);
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    a->type = fake::within(fake::pinned, p)      ? hipMemoryTypeHost
              : fake::within(fake::on_device, p) ? hipMemoryTypeDevice
                                                 : hipMemoryTypeUnregistered;
    return hipSuccess;
}
inline hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    ++fake::captures;
    return s->origin = s, hipSuccess;
}
inline hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g)
{
    --fake::captures;
    s->origin = nullptr;
    return *g = (ihipGraph *)std::malloc(1), hipSuccess;
}
inline hipError_t hipGraphDestroy(hipGraph_t g) { return std::free(g), hipSuccess; }
inline hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, void *, char *, size_t) { return *x = (ihipGraph *)std::malloc(1), hipSuccess; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t x) { return std::free(x), hipSuccess; }
inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return fake::graph_launches.push_back(s), hipSuccess; }
