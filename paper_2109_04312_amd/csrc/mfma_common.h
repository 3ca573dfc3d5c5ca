// Device helpers shared by the bf16 MFMA attention kernels (gfx950, wave64).
//
// MFMA used: v_mfma_f32_32x32x16_bf16.  Operand layout, lane l = 32*hl + m (m = l % 32):
//   A (32 x 16): lane holds row m,    k = 8*hl .. 8*hl+7   (8 bf16 = 16 bytes)
//   B (16 x 32): lane holds column m, k = 8*hl .. 8*hl+7
//   C (32 x 32): lane holds column m, register c = 4*g + r  <->  row 8*g + 4*hl + r
// and, in the backward, the short dense forward and the projections, v_mfma_f32_16x16x32_bf16, lane l = 16*q + r (r = l % 16):
//   A (16 x 32): lane holds row r,    k = 8*q .. 8*q+7
//   B (32 x 16): lane holds column r, k = 8*q .. 8*q+7
//   C (16 x 16): lane holds column r, register e  <->  row 4*q + e
// Every kernel here computes "transposed" score tiles (rows = keys or queries of the streamed
// tile, columns = the rows the wavefront owns), so each lane owns one of the wavefront's rows
// and per-row softmax statistics are per-lane scalars.
#pragma once
#include <hip/hip_runtime.h>

#include "division.h"

namespace mate {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kD = 64;             // head size
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ inline f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The same for a start that the result does not simply replace (a start of two products, a chain outside a loop).  The compiler may give a
// four-register result half of the registers of a start that nothing reads again; its assembler refuses that for longer results only.  Eight
// such instructions agreed with the oracle wherever they ran, but a variant of the weight gradient that had one was wrong, and what made it wrong was
// not found.  Here the start is kept until the result is there, so that the library has none (a test reads the built code).
__device__ __forceinline__ f32x4 mfma16_apart(bf16x8 a, bf16x8 b, f32x4 start) {
  f32x4 c = mfma16(a, b, start);
  asm("" : "+v"(c) : "v"(start));
  return c;
}

__device__ inline f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}

// Registers c0 .. c0+7 of a C tile, rounded to bf16 (nearest even), as an MFMA operand.
__device__ inline bf16x8 pack8(const f32x16& x, int c0) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (__bf16)x[c0 + e];
  return r;
}

// Rows of a result, sixteen bytes a lane.  kThrough: written through the L2 (sc1, agent scope) instead of left dirty in it.
// A kernel is not over before the dirty lines of all eight L2s, up to 32 MB, are in memory, which takes some 6 us that nothing
// overlaps; written through, a result travels while other workgroups still compute, and the next kernel finds it in the memory-side
// cache either way.  us, left and through: dense forward and backward of 32 x 128, 12 heads 22.5 and 20.8, forward and backward of
// 32 x 512, 12 heads 111 and 103.3, layer training of 8 x 512 138 and 133, of 2 x 8192 580 and 574.  (Non-temporal stores, which pass that
// cache as well, gain another 3 % where nothing reads the result, and cost a layer 1 to 3 %.)  Where a launch writes a few hundred
// kilobytes there is nothing to overlap, and it waits for memory instead of the L2: see result_through and the other callers.
// Offsets from `base` are below 4 GB: a (sequence, head)'s rows, or a tile's.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
template <bool kThrough = true>
struct ResultRows {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ explicit ResultRows(void* base /* wave-uniform */) : rsrc(__builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00027000)) {}
  __device__ void store(unsigned byte_off, u32x4 v) const { __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, byte_off, 0, kThrough ? 16 : 0); }
};

// A value that is the same in all lanes, in a scalar register.
__device__ inline float uniform(float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); }

// c ? x : y of values (of two variables the operator yields a variable, which the compiler then looks for in memory)
template <class T>
__device__ __forceinline__ T pick(bool c, T x, T y) { return c ? x : y; }

// max / sum of a per-row value across the two lane halves that share the row (lanes l, l ^ 32):
// v_permlane32_swap exchanges the upper half of its first operand with the lower half of the
// second, so after swapping (x, x) every lane holds both halves' values.
__device__ inline float half_max(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float half_sum(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The same across the four lane quarters of a 16 x 16 tile's column (lanes l, l ^ 16, l ^ 32, l ^ 48).
__device__ inline float quad_max(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return half_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ inline float quad_sum(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return half_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// Lanes m and m + 32 hold row m's value of 32 rows: those of rows r and 16 + r (r = lane % 16).
struct RowPair { unsigned v[2]; };
__device__ inline RowPair row_pair(unsigned x) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return {{r[0], r[1]}};
}

// Sum of the eight bf16 values of an operand, added to acc (v_dot2 against ones): the row sum
// of exactly the rounded probabilities that go into the second contraction.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ inline float sum8(bf16x8 p, float acc) {
  const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const bf16x2 pr = {p[2 * e], p[2 * e + 1]};
    acc = __builtin_amdgcn_fdot2_f32_bf16(pr, one, acc, false);
  }
  return acc;
}

// The same for two values in a word.
__device__ inline float sum2(unsigned p, float acc) {
  const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p), one, acc, false);
}

__device__ inline bf16x8 as_bf16x8(uint4 v) {
  union { uint4 u; bf16x8 b; } x;
  x.u = v;
  return x.b;
}

// Two values rounded to bf16 in one word, x in the low half (one instruction).
__device__ inline unsigned pack2(float x, float y) {
  const bf16x2 r = {(__bf16)x, (__bf16)y};
  return __builtin_bit_cast(unsigned, r);
}

}  // namespace mate
