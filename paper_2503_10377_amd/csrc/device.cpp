// Facts about the current device that the launchers ask for.
#include <hip/hip_runtime.h>

#include <atomic>

#include "sppo_kernels.h"

namespace sppo {

int device_cus() {
  constexpr int kMaxDevices = 64;
  static std::atomic<int> known[kMaxDevices];
  int dev = -1, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  if ((n = known[dev].load(std::memory_order_relaxed)) > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) return 256;
  known[dev].store(n, std::memory_order_relaxed);
  return n;
}

}  // namespace sppo
