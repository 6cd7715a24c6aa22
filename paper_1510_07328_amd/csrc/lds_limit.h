// Dynamic LDS beyond 64 KB.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>

namespace lbm {

// Kernels with more than 64 KB of dynamic LDS need their limit raised, on each
// device they run on: once per device and kernel, under a lock.
constexpr int kMaxDevices = 64;
struct LdsLimit {
    std::mutex m;
    bool done[kMaxDevices] = {};
    hipError_t raise(const void *fn, int bytes) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
        std::lock_guard<std::mutex> lock(m);
        if (done[dev]) return hipSuccess;
        e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e == hipSuccess) done[dev] = true;
        return e;
    }
};

}  // namespace lbm
