// Raising a kernel's limit of dynamic LDS above the default 64 KB.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

namespace seis {

// A setting to be made once on each device of the process, from any thread. A
// failure is not kept: the next call tries again.
class PerDevice {
 public:
  template <class F>
  hipError_t ensure(int device, F set) {
    const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return hipSuccess;
    const hipError_t st = set();
    if (st == hipSuccess) done_.fetch_or(bit, std::memory_order_release);
    return st;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

// kernel K may be launched with up to bytes of dynamic LDS on the current device
template <auto K>
hipError_t raise_lds_limit(int bytes) {
  static PerDevice limit;
  int device = -1;
  const hipError_t st = hipGetDevice(&device);
  if (st != hipSuccess) return st;
  return limit.ensure(device, [&] {
    return hipFuncSetAttribute((const void*)K, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  });
}

}  // namespace seis
