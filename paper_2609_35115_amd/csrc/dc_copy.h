// Staging copies between a caller's device buffers and a state's fixed ones.
// Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dc {

template <typename V> static __global__ __launch_bounds__(256) void stage_kernel(V* dst, const V* src, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) dst[i] = src[i];
}

// Whether [p, p + bytes) is ordinary memory of device dev: inside one
// allocation, so a kernel may read or write it.
static inline bool device_range(const void* p, size_t bytes, int dev)
{
    hipPointerAttribute_t a{};
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipPointerGetAttributes(&a, p) != hipSuccess || a.type != hipMemoryTypeDevice || a.device != dev ||
        hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p) != hipSuccess) {
        (void)hipGetLastError();   // (an unknown pointer is no error of ours)
        return false;
    }
    return (uintptr_t)p - (uintptr_t)base + bytes <= size;
}

// hipMemcpyAsync, device to device, of `bytes` (a multiple of 4) on device dev
// (the current one), by a kernel of our own where both ranges are that
// device's memory: the runtime's copy puts barriers around its kernel, which
// cost more than these small copies (two of them and their barriers per call).
static inline hipError_t stage_async(void* dst, const void* src, size_t bytes, int dev, hipStream_t st)
{
    if (!bytes) return hipSuccess;
    if (!device_range(dst, bytes, dev) || !device_range(src, bytes, dev) || bytes % 4 ||
        ((uintptr_t)dst | (uintptr_t)src) % 4)
        return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, st);
    const bool wide = (((uintptr_t)dst | (uintptr_t)src | bytes) & 15) == 0;
    const int64_t n = (int64_t)(bytes / (wide ? 16 : 4));
    const unsigned blocks = (unsigned)(n < 256 * 2048 ? (n + 255) / 256 : 2048);
    // (hipLaunchKernel for its own status: hipGetLastError would report, and take,
    // an error of the caller's that has nothing to do with the copy)
    void* args[] = {&dst, &src, (void*)&n};
    return hipLaunchKernel(wide ? (const void*)&stage_kernel<uint4> : (const void*)&stage_kernel<uint32_t>, dim3(blocks),
                           dim3(256), args, 0, st);
}

}  // namespace dc
