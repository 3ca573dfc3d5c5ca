// Partial results of several workgroups, added inside the launch by the one that arrives last.
//
// The workgroups may run on different XCDs, whose L2s are not coherent, so partials and arrival words are accessed with
// relaxed device-scope atomics (which bypass the L2), and "partials before arrival" comes from waiting for the
// stores' acknowledgement.
#pragma once
#include <hip/hip_runtime.h>

namespace mate {

template <bool kShared>
__device__ __forceinline__ void put_pair(float* p, float x, float y) {
  const unsigned long long v = (unsigned long long)__float_as_uint(x) | ((unsigned long long)__float_as_uint(y) << 32);
  if (kShared) __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *reinterpret_cast<unsigned long long*>(p) = v;
}
template <bool kShared>
__device__ __forceinline__ float2 get_pair(const float* p) {
  const unsigned long long* q = reinterpret_cast<const unsigned long long*>(p);
  const unsigned long long v = kShared ? __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *q;
  return make_float2(__uint_as_float((unsigned)v), __uint_as_float((unsigned)(v >> 32)));
}
// All of the workgroup's partials and words are where every XCD sees them from here on.
__device__ __forceinline__ void publish_partials() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// Who merges.  The workspace is uninitialised, so there is no counter to add to: every chunk has a
// word of its own and sets it to the call's ticket, a 64-bit number no earlier call has used; a
// workgroup that then finds every word of its group set is the one (or one of several, which write
// the same values: each sets its word before it reads the others', so at least one sees all).
// The words are cleared again afterwards, so that a captured launch, which is replayed with its
// old ticket, finds none of its own.
__device__ __forceinline__ bool completes_group(unsigned long long* words, int mine, int n_chunks,
                                                unsigned long long ticket, int* flag) {
  publish_partials();
  if (threadIdx.x < 64) {
    if (threadIdx.x == 0) __hip_atomic_store(words + mine, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    bool all = true;
    for (int j = threadIdx.x; j < n_chunks; j += 64)
      all &= __hip_atomic_load(words + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ticket;
    const bool every = __all(all);
    if (threadIdx.x == 0) *flag = every;
  }
  __syncthreads();
  return *flag != 0;
}

}  // namespace mate
