// A kernel's limit on dynamic LDS.  The runtime keeps it per device (as it keeps the kernel), so it is raised on every device
// that a process launches the kernel on, once each; a call that fails is made again the next time.
#pragma once
#include <hip/hip_runtime.h>
#include <atomic>
#include <stdint.h>

namespace svdq {

struct LdsLimit {
    std::atomic<uint64_t> raised{0};      // one bit per device
    // on the current device; `bytes` is the same in every call for one kernel
    hipError_t raise(const void *kernel, int bytes) {
        int dev = -1;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;      // (further devices: every time)
        if (raised.load(std::memory_order_acquire) & bit) return hipSuccess;
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e == hipSuccess) raised.fetch_or(bit, std::memory_order_release);
        return e;
    }
};

}  // namespace svdq
