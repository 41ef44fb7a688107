// Internal: dynamic LDS limits of kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

namespace s2 {

// A kernel's dynamic LDS limit is a per-device attribute: remember, per device, that it is set.
constexpr int kMaxDevices = 64;
struct SmemSet {
  std::atomic<unsigned char> done[kMaxDevices];
};

template <class K>
inline hipError_t set_smem(K kernel, size_t bytes, SmemSet& flags) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool tracked = dev >= 0 && dev < kMaxDevices;
  if (tracked && flags.done[dev].load(std::memory_order_acquire)) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)bytes);
  if (e == hipSuccess && tracked) flags.done[dev].store(1, std::memory_order_release);
  return e;
}

}  // namespace s2
