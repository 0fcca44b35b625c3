// Host test program for lds_limit.cpp with a stand-in for the HIP runtime: prints
// "ok" if every launch that a handle prepared for is within its kernel's limit on
// its device, after handles on two devices and from several threads.
#include <atomic>
#include <cstdio>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include <hip/hip_runtime.h>

#include "lds_limit.h"

namespace {
thread_local int device = 0;
std::mutex mu;
std::map<std::pair<int, const void*>, int> limit;
std::atomic<int> sets{0}, bad{0};
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = device, hipSuccess; }
hipError_t hipFuncSetAttribute(const void* fn, hipFuncAttribute, int v) {
  ++sets;
  std::this_thread::yield();
  std::lock_guard<std::mutex> lock(mu);
  limit[{device, fn}] = v;
  return hipSuccess;
}
}

int main() {
  int kernels[3];
  auto handle = [&](int dev, int k, int need) {
    device = dev;
    if (rkkt::raise_lds(&kernels[k], need) != hipSuccess) ++bad;
    std::lock_guard<std::mutex> lock(mu);
    if (limit[{dev, &kernels[k]}] < need) ++bad;
  };
  handle(0, 0, 100);
  handle(1, 0, 100);   // the same kernel on a second device
  handle(0, 0, 50);    // never lowered
  if (sets != 2) ++bad;
  std::vector<std::thread> t;
  for (int i = 0; i < 8; ++i)
    t.emplace_back([&, i] {
      for (int n = 0; n < 2000; ++n) handle(i % 2, 1 + n % 2, 1 + (n * 37 + i * 11) % 5000);
    });
  for (auto& x : t) x.join();
  std::printf(bad ? "bad %d\n" : "ok\n", (int)bad);
  return bad != 0;
}
