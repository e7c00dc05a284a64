// Dynamic LDS beyond the default limit, allowed per kernel and device.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

namespace sr {

// One per kernel (a static beside its launch).  The attribute belongs to the
// current device, so each device of a process needs it once; threads may launch
// at the same time, and setting it twice does no harm.
class LdsLimit {
 public:
  bool pending(int device) const { return device >= 64 || !((done_.load() >> device) & 1); }
  void set(int device) {
    if (device < 64) done_.fetch_or((uint64_t)1 << device);
  }
  hipError_t raise(const void* kernel, size_t lds) {
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess || !pending(device)) return e;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess) set(device);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace sr
