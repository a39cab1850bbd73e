// The limit of dynamic LDS of a kernel that needs more than a launch may ask for by default.
#pragma once
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdint>

namespace rtn {

// One per kernel (static).  The attribute belongs to the kernel on one device, so it is set at the first launch on each;
// threads that come first together set it twice, to the same value.
class LdsLimit {
public:
    hipError_t raise(const void* kernel, int bytes)
    {
        int dev = -1;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;  // (further devices: at every launch)
        if (done_.load(std::memory_order_acquire) & bit) return hipSuccess;
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e == hipSuccess) done_.fetch_or(bit, std::memory_order_release);
        return e;
    }

private:
    std::atomic<uint64_t> done_{0};  // bit = device
};

}  // namespace rtn
