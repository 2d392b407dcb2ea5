// A stand-in for the HIP runtime in tests of the library's host code on a machine without a GPU: "device" memory is host memory, events
// and streams do nothing, and whether a stream is being captured is what the test says.
#include "hip_host.h"

#include <cstdlib>
#include <map>
#include <mutex>

#include "taper_internal.h"

namespace hip_host {
std::atomic<int> capturing{0};
static std::mutex guard;
static std::map<char*, size_t> live;
bool inside_one_allocation(const void* first, const void* end) {
    std::lock_guard<std::mutex> l(guard);
    auto it = live.upper_bound((char*)first);
    if (it == live.begin()) return false;
    --it;
    return (char*)end >= (char*)first && (char*)end <= it->first + it->second;
}
size_t live_allocations() {
    std::lock_guard<std::mutex> l(guard);
    return live.size();
}
static hipError_t take(void** p, size_t n) {
    *p = std::calloc(1, n ? n : 1);
    if (!*p) return hipErrorOutOfMemory;
    std::lock_guard<std::mutex> l(guard);
    live[(char*)*p] = n;
    return hipSuccess;
}
static hipError_t give(void* p) {
    if (!p) return hipSuccess;
    std::lock_guard<std::mutex> l(guard);
    if (live.erase((char*)p) != 1) return hipErrorInvalidValue;
    std::free(p);
    return hipSuccess;
}
}  // namespace hip_host

extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMalloc(void** p, size_t n) { return hip_host::take(p, n); }
hipError_t hipFree(void* p) { return hip_host::give(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hip_host::take(p, n); }
hipError_t hipHostFree(void* p) { return hip_host::give(p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = hip_host::capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
}

namespace taper {
hipError_t static_scratch(int, void**) { return hipErrorNotSupported; }
hipError_t launch_upload(void*, const void*, size_t, int32_t*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_kv_append(const void*, const void*, const int64_t*, void*, int, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_stream_read(const void*, int64_t, int, unsigned*, hipStream_t) { return hipSuccess; }
hipError_t launch_resolve_slots(const StepArgs&, int64_t*, int64_t, hipStream_t) { return hipSuccess; }
}  // namespace taper
