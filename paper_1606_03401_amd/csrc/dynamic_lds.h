// Dynamic LDS beyond the runtime's default limit.  Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstddef>

namespace mebptt {

// Lets `Kernel` be launched with up to `bytes` of dynamic LDS on the current device.  The runtime is asked once per
// kernel and device; safe from any thread (asking twice does no harm).
template <auto Kernel>
hipError_t allow_dynamic_lds(size_t bytes) {
  static std::atomic<unsigned> devices{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const unsigned bit = dev < 32 ? 1u << dev : 0u;   // a device past the 32nd is asked every time
  if (devices.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) devices.fetch_or(bit, std::memory_order_release);
  return e;
}

}  // namespace mebptt
