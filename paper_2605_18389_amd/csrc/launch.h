// What the kernel launchers share.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "per_device.h"
#include "shot_internal.h"

namespace shot {

constexpr size_t LDS_BYTES = 160 * 1024;  // of a compute unit

// Dynamic LDS beyond 64 KiB has to be enabled for a kernel, on each device.  The limit
// set is all that the kernel can have, never the size of the launch at hand: of two
// threads that launch one kernel with different sizes, the later one to set its own
// would leave the other's launches beyond the limit.
inline hipError_t allow_lds(const void* kernel, size_t lds, std::atomic<unsigned long long>& done) {
  if (lds <= 65536) return hipSuccess;
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return once_per_device(done, dev, [kernel]() -> hipError_t {
    hipFuncAttributes fa;
    const hipError_t g = hipFuncGetAttributes(&fa, kernel);
    if (g != hipSuccess) return g;
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(LDS_BYTES - fa.sharedSizeBytes));
  });
}

}  // namespace shot

// A launch, between the events set for it, if any (attached to the dispatch itself, so
// that they time the kernel's execution rather than the gap before it).
#define SHOT_LAUNCH(kernel, grid, block, lds, stream, ...)                                         \
  do {                                                                                             \
    hipEvent_t ev0, ev1;                                                                           \
    if (shot::take_launch_events(&ev0, &ev1))                                                      \
      hipExtLaunchKernelGGL(kernel, grid, block, lds, stream, ev0, ev1, 0, __VA_ARGS__);           \
    else                                                                                           \
      hipLaunchKernelGGL(kernel, grid, block, lds, stream, __VA_ARGS__);                           \
  } while (0)
