// Launch of a planned kernel.
#pragma once

#include <hip/hip_runtime.h>

#include "ops.hpp"

namespace ug {

// A refused launch is reported here and not again by a later call's
// hipGetLastError.
inline hipError_t submit(const OpPlan& p, void** args, hipStream_t s) {
  const hipError_t e = hipLaunchKernel(p.func, p.grid, p.block, args, p.lds, s);
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}

}  // namespace ug
