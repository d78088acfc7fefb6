// How the kernels that run many generations in one launch (ones_fused.hip, ones_resident.hip) exchange data between
// their workgroups: entries written and polled with relaxed atomics at device scope, which the hardware performs at
// the device's point of coherence instead of in the caches of one XCD.
#pragma once

#include "ones_device.h"

namespace ones {
namespace {

template <typename T>
__device__ __forceinline__ T shared_load(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void shared_store(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace
}  // namespace ones
