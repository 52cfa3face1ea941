// Dynamic LDS beyond the default limit of 64 KiB a workgroup.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

namespace edpc {

constexpr int kLdsBytes = 160 * 1024;  // of a CU

// Allows a kernel up to `bytes` of it.  A function's attributes are those of the
// current device, so this is asked for once on each device (one object a kernel,
// with the same bytes every time).
class LdsLimit {
 public:
  hipError_t raise(const void* kernel, int bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool counted = dev >= 0 && dev < 64;
    const uint64_t bit = counted ? (uint64_t)1 << dev : 0;
    if (raised_.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) raised_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<uint64_t> raised_{0};
};

}  // namespace edpc
