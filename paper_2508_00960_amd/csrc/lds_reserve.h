// Dynamic LDS beyond what any launch may ask for has to be reserved for a kernel, once per device: the attribute belongs to the device's own copy of the
// kernel, and a thread may use several devices.  (Host code.)
#pragma once
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdint>

namespace phantom {

// One per kernel, static: which devices have the reservation.  Reserving twice, as two threads at once may, is harmless.
class LdsReserved {
public:
    // for the device that is current
    hipError_t reserve(const void *kernel, int bytes)
    {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;        // (a device past the word's end: on every launch)
        if (devices_.load(std::memory_order_acquire) & bit) return hipSuccess;
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e == hipSuccess) devices_.fetch_or(bit, std::memory_order_release);
        return e;
    }

private:
    std::atomic<uint64_t> devices_{0};
};

}  // namespace phantom
