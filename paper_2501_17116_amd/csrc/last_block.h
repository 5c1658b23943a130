// What the workgroup that finishes last of a launch does with what all of them left: one launch instead of two.
#pragma once
#include "fp4_common.h"

#if defined(__HIPCC__)
// True for every thread of the workgroup that arrives last of `of`; *arrived starts at 0.  What the others leave for it
// must have been written with device-scope atomics and is read with load_device: those go past
// the XCDs' own L2s, so no cache is written back or invalidated here (a release fence of a whole L2 per workgroup cost more
// than a launch) and it is enough that this thread's have been acknowledged.  Nobody waits for anybody.
FP4_D bool last_workgroup(uint32_t* arrived, uint32_t of) {
  __shared__ bool s_last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) s_last = __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == of - 1;
  __syncthreads();
  return s_last;
}
template <class T>
FP4_D T load_device(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
#endif
