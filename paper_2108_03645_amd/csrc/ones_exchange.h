// What the kernels that run many generations in one launch exchange between their workgroups
// (ones_fused.hip, ones_resident.hip): 64-bit entries written and polled with relaxed atomics at device scope,
// which the hardware performs at the device's point of coherence instead of in the caches of one XCD.
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

// Tag of the n-th use (n = 0, 1, ..) of a pair of exchange buffers that start out zeroed: use n
// goes to buffer n & 1 and flips the tag that buffer's entries carried before.
__device__ __forceinline__ uint64_t use_tag(uint32_t n) { return static_cast<uint64_t>(((n >> 1) & 1u) ^ 1u) << 63; }
constexpr uint64_t kTagBit = 1ull << 63;

// Collects n published 64-bit entries: thread t of kThreads takes entries t, t + kThreads, ..., polls until every one
// is ready and hands it to take(e, v, now), which whole waves call together (now: the lane's entry has just become
// ready).  at(e): the address of entry e.  False when the polls ran out.  No branch around a load: a thread
// reads its entries again until the wave has all of its own.
template <int kPer, int kThreads, typename At, typename Ready, typename Take>
__device__ __forceinline__ bool gather_per(uint32_t n, uint32_t spin_limit, At at, Ready ready, Take take) {
  uint32_t pending = 0;
  const uint64_t *src[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t e = threadIdx.x + k * kThreads;
    if (e < n) pending |= 1u << k;
    src[k] = at(min(e, n - 1));
  }
  if (__ballot(pending != 0) == 0) return true;
  for (uint32_t spins = 0; spins < spin_limit; ++spins) {
    uint64_t v[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) v[k] = shared_load(src[k]);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const uint32_t e = threadIdx.x + k * kThreads;
      const bool now = ((pending >> k) & 1u) && ready(e, v[k]);
      take(e, v[k], now);
      if (now) pending &= ~(1u << k);
    }
    if (__ballot(pending != 0) == 0) return true;
  }
  return false;
}

}  // namespace
}  // namespace ones
