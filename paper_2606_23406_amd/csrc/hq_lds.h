// The opt-in of kernels launched with more than 64 KB of dynamic LDS.
#ifndef HQ_LDS_H
#define HQ_LDS_H
#include <hip/hip_runtime_api.h>
#include <stddef.h>

#include <atomic>
#include <mutex>

// What one kernel has been opted in for, per device (the runtime keeps the
// opt-in per kernel and device); one static object per kernel.
struct hq_lds_granted {
  static constexpr int kDevices = 64;
  std::atomic<size_t> bytes[kDevices] = {};
  std::mutex mu;
};

// Lets `kernel` be launched on the current device with `bytes` of dynamic LDS.
// The runtime call is costly, so it is made only where the size exceeds the
// largest one so far on this device; under a lock, since a smaller size set
// later would take a larger one back.  Returns 0 or the runtime's error, which
// the launch's own error check finds too.
inline int hq_allow_lds(const void* kernel, size_t bytes, hq_lds_granted& g) {
  if (bytes <= 65536) return 0;
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= hq_lds_granted::kDevices)
    return (int)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  std::atomic<size_t>& most = g.bytes[dev];
  if (bytes <= most.load(std::memory_order_acquire)) return 0;
  std::lock_guard<std::mutex> lock(g.mu);
  if (bytes <= most.load(std::memory_order_relaxed)) return 0;
  const hipError_t set = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (set == hipSuccess) most.store(bytes, std::memory_order_release);
  return (int)set;
}

#endif
