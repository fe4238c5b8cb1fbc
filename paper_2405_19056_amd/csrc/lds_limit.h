// A kernel's limit of dynamic LDS, raised once per device and size.
#pragma once

#include <stddef.h>

#include <atomic>
#include <mutex>

#include <hip/hip_runtime_api.h>

namespace gn {

// One per kernel (a function's static).  The attribute belongs to the function
// on one device: handles on several devices each need it there.  A failure is
// returned and not remembered.  Any thread.
class LdsLimit {
 public:
  // The current device's limit, at least `bytes`.
  hipError_t raise(const void *kernel, size_t bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kDevices)      // no record: set it every time
      return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (held_[dev].load(std::memory_order_acquire) >= bytes) return hipSuccess;
    std::lock_guard<std::mutex> lk(mu_);  // a smaller size must not follow a larger one
    if (held_[dev].load(std::memory_order_relaxed) >= bytes) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) held_[dev].store(bytes, std::memory_order_release);
    return e;
  }

 private:
  static constexpr int kDevices = 64;
  std::mutex mu_;
  std::atomic<size_t> held_[kDevices] = {};
};

}  // namespace gn
