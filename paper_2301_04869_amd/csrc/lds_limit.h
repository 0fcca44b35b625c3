#pragma once

#include <hip/hip_runtime_api.h>

namespace rkkt {

// Lets launches of `kernel` on the current device use `need` bytes of dynamic LDS.
hipError_t raise_lds(const void* kernel, long long need);

}  // namespace rkkt
