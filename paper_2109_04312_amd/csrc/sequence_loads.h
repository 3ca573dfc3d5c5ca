// A lane's kEach consecutive positions of a sequence's ids or flags, in one load; N is kEach at least.
//
// Near the end of a sequence a lane loads the last kEach positions instead and shifts them down afterwards, so no load
// is behind a branch: with one path for lanes inside the sequence and another for the rest, the compiler loaded word by
// word and waited in between.  (Any alignment that an int array and a byte array have: a sequence of odd length shifts
// the next one.)
#pragma once
#include <hip/hip_runtime.h>

namespace mate {

// First position that is loaded for a lane that begins at i0.
template <int kEach>
__device__ __forceinline__ int load_from(int i0, int N) { return min(i0, N - kEach); }

// (Vectors: an array whose elements are selected by the shift would end up in memory.)
template <int kEach>
struct Ids {
  typedef int type __attribute__((ext_vector_type(kEach)));
  typedef type loaded __attribute__((aligned(4)));
};
template <int kEach>
__device__ __forceinline__ typename Ids<kEach>::type load_ids(const int* ids, int i0, int N) {
  return *reinterpret_cast<const typename Ids<kEach>::loaded*>(ids + load_from<kEach>(i0, N));
}
template <int kEach>
__device__ __forceinline__ unsigned load_flags(const unsigned char* flags, int i0, int N) {  // a byte each
  static_assert(kEach == 1 || kEach == 2 || kEach == 4, "a word of bytes");
  unsigned word = 0;
  __builtin_memcpy(&word, flags + load_from<kEach>(i0, N), kEach);
  return word;
}
// What was loaded, moved so that element j is position i0 + j where that is below N (anything elsewhere).
template <int kEach>
__device__ __forceinline__ typename Ids<kEach>::type align_ids(typename Ids<kEach>::type id, int i0, int N) {
  const int shift = i0 - load_from<kEach>(i0, N);
#pragma unroll
  for (int by = 1; by < kEach; by *= 2)
#pragma unroll
    for (int j = 0; j + by < kEach; ++j) {
      const int here = id[j], further = id[j + by];
      id[j] = (shift & by) ? further : here;
    }
  return id;
}
template <int kEach>
__device__ __forceinline__ unsigned align_flags(unsigned word, int i0, int N) {
  return word >> (8 * ((i0 - load_from<kEach>(i0, N)) & 3));
}

}  // namespace mate
