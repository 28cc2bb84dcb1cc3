// Kernels with more dynamic LDS than a launch may ask for by default.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <atomic>
#include <cstddef>

namespace cmoe {

// Devices on which a kernel's limit has been raised: the limit belongs to the kernel's copy on one device, and several host
// threads may launch for the first time at once.  One per kernel, static in its launcher.
struct LdsLimit {
  std::atomic<uint64_t> raised{0};

  // Raise the limit of `kernel` on the current device, unless that has been done.
  hipError_t raise(const void* kernel, size_t bytes) {
    int device = -1;
    hipError_t err = hipGetDevice(&device);
    if (err != hipSuccess) return err;
    const uint64_t bit = device >= 0 && device < 64 ? (uint64_t)1 << device : 0;      // (any other: every time)
    if (raised.load(std::memory_order_acquire) & bit) return hipSuccess;
    err = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (err == hipSuccess) raised.fetch_or(bit, std::memory_order_release);
    return err;
  }
};

}  // namespace cmoe
