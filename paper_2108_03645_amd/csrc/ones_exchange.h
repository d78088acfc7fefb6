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

// All stores and loads of the workgroup are done when one thread goes on, whose fence at system scope then stands for all of
// them.  (A fence by every wave writes the cache back as often: 16 waves 6 us.)
__device__ __forceinline__ void all_arrived() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0);
  asm volatile("" ::: "memory");
  __syncthreads();
}
// Whether this workgroup is the last of the launch to come here; one thread of each asks, behind a fence for what it has stored.  The counter wraps to zero with the last
// one, so that a launch that was refused, or recorded into a graph and never run, leaves nothing to be made up for.
__device__ __forceinline__ bool last_to_arrive(uint32_t *arrived) {
  const uint32_t others = gridDim.x - 1;
  if (others == 0) return true;
  if (__builtin_amdgcn_atomic_inc32(arrived, others, __ATOMIC_RELAXED, "agent") != others) return false;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return true;
}
// The winner of a call, in genome row `row` of so many words, for the host.  Whole workgroup; w lies in the argument block.
template <typename Args>
__device__ __forceinline__ void publish_winner(const Args &w, const uint32_t *genes, uint32_t row_words, uint32_t row, const uint32_t *info, uint64_t score_bits) {
  const uint32_t n = w.n_slots;
  int32_t *batch = w.batch, *gpus = w.gpus;
  for (uint32_t j = threadIdx.x; j < n; j += blockDim.x) {
    const uint32_t at = gene_byte(j), code = (shared_load(genes + static_cast<size_t>(row) * row_words + at / 4) >> (8 * (at % 4))) & 0xFFu;
    batch[j] = static_cast<int32_t>(batch_of_code(code, info_blexp(info[j])));
    gpus[j] = static_cast<int32_t>((1u << code) >> 1);
  }
  if (threadIdx.x == 0) *w.fit = __longlong_as_double(static_cast<long long>(score_bits));
}
// Tells the host that the call is done: by the thread that knows that all its workgroups are.  err: the two error words.
template <typename Args>
__device__ __forceinline__ void signal_call_done(const Args &w, const uint32_t *err) {
  w.err[0] = shared_load(err);
  w.err[1] = shared_load(err + 1);
  *w.of = w.done.value;                                // (not before: the workgroups of a launch that gives up do not all arrive)
  __hip_atomic_store(w.done.flag, w.done.value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace
}  // namespace ones
