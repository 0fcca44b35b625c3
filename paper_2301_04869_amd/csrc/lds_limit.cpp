// Dynamic LDS limits of the kernels: a kernel's limit belongs to a device, is
// shared by every handle on it and must never drop below what an earlier
// handle's launches need, so the largest one set so far is kept per device and
// kernel, under a lock (handles are created from several threads).
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <utility>

#include "lds_limit.h"

namespace rkkt {

hipError_t raise_lds(const void* kernel, long long need) {
  static std::mutex mu;
  static std::map<std::pair<int, const void*>, long long> set;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  long long& cur = set[{dev, kernel}];
  if (need <= cur) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)need);
  if (e == hipSuccess) cur = need;
  return e;
}

}  // namespace rkkt
