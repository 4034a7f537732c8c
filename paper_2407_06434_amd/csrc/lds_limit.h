// Dynamic LDS beyond the 64 KiB that every kernel may use.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace bomp {

// Raises `kernel`'s limit to `bytes` on the current device. The limit belongs to one kernel on
// one device, and kernels of one template share their type, so nothing is remembered between
// calls: this runs before every launch that needs it (the solves replay graphs, where it runs
// once per capture).
template <class K>
inline hipError_t lds_limit(K kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

}  // namespace bomp
