// Quotients of workgroup numbers.  (For the host too: a test compares them with exact ones.)
#pragma once
#include <hip/hip_runtime.h>

namespace mate {

// (float)x / d, nearly; wave-uniform
__host__ __device__ inline int nearly_quotient(int x, int d) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_readfirstlane((int)((float)x * __builtin_amdgcn_rcpf((float)d)));
#else
  return (int)((float)x * (1.f / (float)d));
#endif
}

// x / d and the remainder, both wave-uniform and not negative, for a quotient below 2^21: one float product and its
// correction, half the instructions of an integer division (scalar instructions wait for each other, and a workgroup's first
// microsecond is little else).
__host__ __device__ inline int uniform_div(int x, int d, int& rest) {
  int k = nearly_quotient(x, d);
  rest = x - k * d;
  const int below = rest >> 31;
  k += below;
  rest += below & d;
  const int above = rest >= d;
  k += above;
  rest -= above ? d : 0;
  return k;
}
// The same for any x: from 2^21 on the quotient may be too large for that (x as a float is off by two from 2^25 on).
__host__ __device__ inline int uniform_div_any(int x, int d, int& rest) {
  if (__builtin_expect(x < 1 << 21, 1)) return uniform_div(x, d, rest);
  rest = (int)((unsigned)x % (unsigned)d);
  return (int)((unsigned)x / (unsigned)d);
}

}  // namespace mate
