// Device memory that belongs to no context and is never allocated: the scratch array behind
// taper_decode_step_attention_static (for callers that cannot allocate device memory).  Every GPU the
// library runs on holds its own copy of the array, at its own address, until the process ends.
#include "taper_internal.h"

namespace taper {

static __device__ __align__(256) unsigned char scratch[kStaticStartsBytes + kStaticScratchBytes];

// In host code the array's name is only a handle for the symbol, not a device address: what kernels,
// copies and fills are given is the address looked up here, once per device.
constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];

hipError_t static_scratch(int device, void** ptr) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // of the current device's copy
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = p;
    }
    *ptr = g_scratch_ptr[device];
    return hipSuccess;
}

// Brings a plan's image from pinned host memory to the device and clears the counters behind it: the lanes read host
// memory themselves.  A copy command would do the first part, but it runs on a copy engine, and the hand-overs from the
// kernels before it and to the kernels after it took longer than the 0.1-1 MB themselves (a decode step of four layers:
// 383 us with copy commands, 367 this way).  (Nor is a fill command used: the call may be recorded into a graph.)
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void upload_kernel(u32x4* __restrict__ dst, const u32x4* __restrict__ src, int64_t n,
                                                     int32_t* __restrict__ zero, int64_t n_zero) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = src[i];
    if (i < n_zero) zero[i] = 0;
}

hipError_t launch_upload(void* dst, const void* src, size_t bytes, int32_t* zero, int64_t n_zero, hipStream_t s) {
    const int64_t n = (int64_t)(bytes / 16), most = n > n_zero ? n : n_zero;
    if (most <= 0) return hipSuccess;
    hipLaunchKernelGGL(upload_kernel, dim3((unsigned)((most + 255) / 256)), dim3(256), 0, s, (u32x4*)dst, (const u32x4*)src, n, zero,
                       n_zero);
    return hipGetLastError();
}

}  // namespace taper
