// Host-side launch helper shared by the kernels that use more LDS than the default limit (internal).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

namespace climber {

// Dynamic LDS above 64 KiB has to be allowed per kernel; the attribute belongs to the function as loaded on the
// current device, so it is raised once per device (bytes: the most this kernel is ever launched with).
template <auto Kernel>
hipError_t raise_lds_limit(size_t bytes)
{
    constexpr int kMaxDevices = 64;
    static std::atomic<bool> raised[kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (raised[dev].load(std::memory_order_acquire)) return hipSuccess;
    e = hipFuncSetAttribute((const void *)Kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) raised[dev].store(true, std::memory_order_release);
    return e;
}

}  // namespace climber
