// A kernel that takes more than 64 KB of dynamic LDS says so once per device.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <initializer_list>

namespace fact {

struct LdsLimit {
    std::atomic<bool> set[64];                     // one flag per device; a static object of each launcher
};

// Sets the limit of `kernels` on the current device unless `limit` says that it is set.  (Two host threads may make a
// kernel's first launch at once: setting the limit twice is harmless.)
inline hipError_t raise_lds_limit(LdsLimit &limit, int bytes, std::initializer_list<const void *> kernels)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (limit.set[dev].load(std::memory_order_acquire)) return hipSuccess;
    for (const void *kernel : kernels) {
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
    }
    limit.set[dev].store(true, std::memory_order_release);
    return hipSuccess;
}

}  // namespace fact
