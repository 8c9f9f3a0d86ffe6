// Progress words of the strip streams: waves of a workgroup that take items (a
// strip of one alignment matrix over all its columns) round robin and wait for
// the item before, chunk by chunk, through words in LDS instead of barriers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/swdb.h"
#include "plans.h"

namespace swdb {

// A wave's progress: its item's number in the bits from kProgBits up (modulo
// 2^9), finished chunks below.  Compared by signed difference: a wave is at most
// kRing items ahead of the one that waits for it.
constexpr int kProgBits = 23;
static_assert((SW_MAX_LEN >> 2) + 2 < (1 << kProgBits), "chunks fit the progress word");

// A word of LDS that another wave publishes (acquire and release at workgroup
// scope: what that wave wrote before is seen), as a uniform value.
template <class T>
__device__ __forceinline__ int peek(const T* p) {
  return __builtin_amdgcn_readfirstlane(
      (int)__hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
}
template <class T>
__device__ __forceinline__ void publish(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Polling costs issue slots (sleeps of 64 cycles took 7 % of them, 1,024 cost
// nothing: a chunk takes some 5,000).
__device__ __forceinline__ void poll_pause() { __builtin_amdgcn_s_sleep(16); }

// Waits until the progress word at p, last read as `known`, has reached need.
__device__ __forceinline__ void wait_progress(const uint32_t* p, uint32_t& known, uint32_t need) {
  while ((int)(known - need) < 0) {
    known = (uint32_t)peek(p);
    if ((int)(known - need) < 0) poll_pause();
  }
}

typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));

}  // namespace swdb
