// A kernel's limit of dynamic LDS, which every device keeps for itself: raised once on each, by whichever
// thread launches there first.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstddef>
#include <cstdint>

namespace attt {

class LdsLimit {  // one per kernel
  std::atomic<uint64_t> raised_{0};  // bit d: done on device d

 public:
  // Lets `kernel` use `bytes` of dynamic LDS on the current device.
  hipError_t raise(const void* kernel, size_t bytes) {
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;  // others set it on every call
    if (raised_.load(std::memory_order_acquire) & bit) return hipSuccess;
    if (hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes)) return e;
    raised_.fetch_or(bit, std::memory_order_release);
    return hipSuccess;
  }
};

}  // namespace attt
