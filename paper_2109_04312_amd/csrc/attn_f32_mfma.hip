// fp32 MATE attention on the matrix cores: the path for dtype f32, forward and backward.
//
// Products are formed from splits (the published three-part bfloat16 scheme of Henry, Tang and Heinecke, 2019, "Leveraging
// the bfloat16 artificial intelligence datatype for higher-precision computations"): x = x1 + x2 + x3 with bf16 parts of 8
// significant bits each, which together hold all 24 bits of an fp32 value, and
// x y = x1 y1 + (x1 y2 + x2 y1) + (x1 y3 + x2 y2 + x3 y1).  What is left out, x2 y3 + x3 y2 + x3 y3, is at most
// (2^-24 + 2^-34) |x y| (x2 of 2^-8 and x3 of 2^-17 of the power of two below x, the most that rounding to nearest leaves) and
// 2^-27.5 |x y| rms, where an fp32 rounding of the sum that it goes into is up to 2^-24 of that sum.
// Six v_mfma_f32_32x32x16_bf16 (32 cycles, 16 of the contraction) take the place of eight v_mfma_f32_32x32x2_f32 (64 cycles, 2 of it): 192 cycles for 512.
// Sums are fp32 as before, and fewer of them are rounded (a matrix instruction adds sixteen products at once).
// (A value above the largest bf16, 3.39e38, has no such split, nor has an infinity or a NaN: see accumulate_special.  For
// values below 2^-103 see kLeast.)
//
// Same pattern, tables and work units as the bf16 kernels (stream_plan.h), other proportions: no shared tiles and no
// barriers in the loop.  A workgroup owns 32 rows (a quarter of a unit), its four wavefronts take every fourth
// 32-row tile of the other side, each through LDS of its own, and their results are added in LDS at the end.
// Small units also mean that a batch of short sequences fills the chip.
//
// A tile is loaded in whole rows (16 lanes x 16 bytes) into registers, is split there, and passes through LDS into
// operand order: three planes of 32 rows x 128 bytes, laid out and read like the tiles of the bf16 kernels (d2l.h).
//
// Measured (4 sequences of 512 tokens, 12 heads), with the fp32 instruction and with splits: forward 22.8 -> 18.3 us, backward
// 62.4 -> 46.5 (3 of it from one launch), a training step 91.3 -> 69; one sequence of 128, 4 heads 7.4 -> 7.5.  Errors against
// 64 bits (relative 2-norm, and the largest in units of the rms; means of 12 seeds at that shape): O 2.6e-7 -> 1.4e-7 and
// 5.2e-6 -> 2.7e-6, LSE 4.7e-8 -> 4.5e-8 and 2.0e-7 -> 1.8e-7, dQ 3.9e-7 -> 3.0e-7 and 7.4e-6 -> 5.5e-6, dK 4.1e-7 -> 3.2e-7
// and 1.09e-5 -> 0.81e-5, dV 3.9e-7 -> 3.1e-7 and 9.3e-6 -> 7.3e-6; smaller at seven other shapes of 64 to 1024 tokens and with
// Q and K three times as large, too.
// What bounds it: a tile is 440 to 510 vector instructions (224 of them the splits of two tensors, 56 those of P or dS) beside
// 1536 (forward) to 3072 cycles of matrix pipe; question-token owners have four tiles per wavefront and end last, and 74 KB of LDS
// leave room for two workgroups on a CU.  (The splits interleaved with the matrix instructions of the tile before: 17.5 ->
// 19.9 and 46 -> 64, most wavefronts have one or two tiles and would split one that nobody meets.)
//
// Operand layouts are those of the bf16 kernels; the second contraction's operand of P or dS is C registers 8 tt .. 8 tt + 7.
#include <hip/hip_runtime.h>

#include "d2l.h"
#include "launch.h"
#include "mfma_common.h"
#include "stream_plan.h"
#include "tile_bodies.h"

namespace mate {
namespace {

constexpr int kRows = 32;                  // owned rows of a workgroup, rows of a streamed tile
constexpr int kWaves = kThreads / 64;

__device__ __forceinline__ f32x16 mfma1(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// The three planes of a tile, and a wavefront's piece of LDS.
constexpr int kPlane = kRows * 128;
constexpr int kPlanes = 3 * kPlane;

// Tiles of whole fp32 values (accumulate_special, and results on their way out): 32 rows of 64 floats and a pad of 4, which spreads row accesses (16 bytes of 16 rows at
// once) over the 64 banks; column reads (rows r and r + 4 at once) overlap in a quarter of them, which
// the matrix pipe hides.
constexpr int kStride = kD + 4;
static_assert(kRows * kStride * 4 <= kPlanes, "a wavefront's piece holds either form");

// Two values as three words of bf16 parts (rounded to nearest, so that what is left has a sign of its own).  A dot product with
// (-1, 0) or (0, -1) takes a part off its value in one instruction, exactly.
__device__ __forceinline__ void split2(float x, float y, unsigned (&w)[3]) {
  // (-1, 0) and (0, -1), in scalar registers: written as constants, one becomes the instruction's inline -1.0, which the
  // hardware reads as 32 bits, that is as the other
  unsigned one = 0x0000bf80u, other = 0xbf800000u;
  asm("" : "+s"(one), "+s"(other));
  const bf16x2 minus_x = __builtin_bit_cast(bf16x2, one), minus_y = __builtin_bit_cast(bf16x2, other);
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    w[p] = pack2(x, y);
    if (p == 2) break;
    const bf16x2 part = __builtin_bit_cast(bf16x2, w[p]);
    x = __builtin_amdgcn_fdot2_f32_bf16(part, minus_x, x, false);
    y = __builtin_amdgcn_fdot2_f32_bf16(part, minus_y, y, false);
  }
}
// ---- values whose parts would not all be normal numbers -----------------------------------------------------------
// A value of kLeast or more has its last bit at 2^-126 or above, so its parts are zeros or normal numbers.  Smaller ones
// would lose up to kLost of themselves.  Results in which that could show are computed with whole values, in the second
// pass that infinities have too.  No streamed value is looked at for it (that took 3 % of a backward and 5 % of a forward,
// this takes 2 %):
//  * P and dS are small by themselves (a score 87 below the largest is 2^-126): they are split times kLift.
//  * A sum of weights times rows of V, K or Q is off by at most kLost times the sum of the weights, which is known (the
//    forward's row sum) or bounded by the largest (dS).  Only where a result is less than 2^25 times that are the
//    rows looked at.  (Zeros in a result, from a column of zeros, cost that look; small values the second pass.)
//  * A score matters as it is, not against its size: from exact owned rows of at most kLarge it is off by less than 2^-54
//    before the scale.  Owned rows that hold small or large values have the second pass, and so have large scales.
//  * dP matters against delta, which shows what small values of V could cost; those of dO: see delta_f32_kernel.
constexpr float kLeast = 0x1p-103f, kLost = 0x1p-125f, kLarge = 0x1p64f, kLargeScale = 0x1p20f, kLift = 0x1p24f;
constexpr float kVisible = kLost * 0x1p25f;        // times the sum of weights: a result above it has lost nothing
constexpr float kMostRows = 16384;                 // MATE_MAX_N
// Is x small and not zero?
__device__ __forceinline__ bool is_small(float x) { return __float_as_uint(fabsf(x)) - 1u < __float_as_uint(kLeast) - 1u; }
template <int kCount>
__device__ __forceinline__ bool any_small(const f32x4 (&v)[kCount]) {
  bool small = false;
#pragma unroll
  for (int i = 0; i < kCount; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) small |= is_small(v[i][e]);
  return __any(small);
}

// 16 bytes of a row to the planes at `tile`: piece = dims 4 piece .. + 3 of row `row`.
__device__ __forceinline__ void put_split(char* tile, int row, int piece, const f32x4& v) {
  unsigned a[3], b[3];
  split2(v.x, v.y, a);
  split2(v.z, v.w, b);
  char* at = tile + row * 128 + (((piece >> 1) ^ swz(row & 15)) << 4) + 8 * (piece & 1);
#pragma unroll
  for (int p = 0; p < 3; ++p) *reinterpret_cast<uint2*>(at + p * kPlane) = make_uint2(a[p], b[p]);
}

// A lane's window of the tile's rows.  (Compared per pair: the matrix pipe bounds these kernels, and their registers are
// full.)
struct SlotWindow {
  int d0, len;  // the tile's first slot + 4 hl - the window's, and its length
  __device__ __forceinline__ bool in(int c) const { return (unsigned)(d0 + 8 * (c >> 2) + (c & 3)) < (unsigned)len; }
  // tile row `row`, whichever lane half holds its score
  __device__ __forceinline__ bool meets(int row, int hl) const { return (unsigned)(d0 - 4 * hl + row) < (unsigned)len; }
};

// Piece l % 16 of a row; X is wave-uniform and the offset in it below 2^32 bytes, which is the form of a load that takes
// no 64-bit arithmetic.
__device__ __forceinline__ f32x4 load_piece(const float* X, int tok, int lane) {
  return *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(X) + ((unsigned)tok * (kD * 4u) + (unsigned)(lane & 15) * 16u));
}

// A tile on its way from global memory: lane l holds piece l % 16 of rows l / 16 + 4 i.
struct TileRegs {
  f32x4 v[8];
  // `tok`: lanes m and m + 32 hold the token of tile row m
  __device__ __forceinline__ void load(const float* X, int tok, int lane) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = load_piece(X, __shfl(tok, (lane >> 4) + 4 * i, 64), lane);
  }
  __device__ __forceinline__ void split(char* tile, int lane) const {
#pragma unroll
    for (int i = 0; i < 8; ++i) put_split(tile, (lane >> 4) + 4 * i, lane & 15, v[i]);
  }
  __device__ __forceinline__ void put(float* tile, int lane) const {
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<f32x4*>(tile + ((lane >> 4) + 4 * i) * kStride + 4 * (lane & 15)) = v[i];
  }
};
// The owned rows of a tensor into planes: every wavefront brings eight of them.
struct OwnedRows {
  f32x4 v[2];
  __device__ __forceinline__ void load(const float* X, int pos, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = load_piece(X, __shfl(pos, 8 * wave + 4 * i + (lane >> 4), 64), lane);
  }
  __device__ __forceinline__ void split(char* tile, int wave, int lane) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) put_split(tile, 8 * wave + 4 * i + (lane >> 4), lane & 15, v[i]);
  }
  // Is there a value that is zero, small or large?
  __device__ __forceinline__ bool suspect() const {
    float least = kLeast, most = kLarge;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        least = fminf(fminf(least, fabsf(v[i][e])), fabsf(v[i][e + 1]));
        most = fmaxf(fmaxf(most, fabsf(v[i][e])), fabsf(v[i][e + 1]));
      }
    return least < kLeast || most > kLarge;
  }
  __device__ __forceinline__ bool inexact() const {
    bool large = false;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) large |= fabsf(v[i][e]) > kLarge;
    return any_small(v) || __any(large);
  }
};

// Over dims: rows of the tile against rows of an owned one, both in planes.  (The small products have a sum of their own, which
// rounds them against each other and not against the large ones.)  kOwned: which of the workgroup's owned tiles.
template <int kOwned = 0>
__device__ __forceinline__ f32x16 contract(const PlainAddr& a, const PlainAddr& b) {
  f32x16 sum = zero16(), small = zero16();
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    bf16x8 x[3], y[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      x[p] = read_plain(a.a[ks] + p * kPlane);
      y[p] = read_plain(b.a[ks] + kOwned * kPlanes + p * kPlane);
    }
    small = mfma(x[2], y[0], small);
    sum = mfma(x[0], y[0], sum);
    small = mfma(x[0], y[2], small);
    small = mfma(x[1], y[1], small);
    small = mfma(x[1], y[0], small);
    small = mfma(x[0], y[1], small);
  }
#pragma unroll
  for (int c = 0; c < 16; ++c) sum[c] += small[c];
  return sum;
}
// Over tile rows: the tile's columns against C registers.
__device__ __forceinline__ void accumulate(f32x16 (&acc)[2], const TransposedAddr& t, const f32x16& p) {
#pragma unroll
  for (int tt = 0; tt < 2; ++tt) {
    unsigned w[4][3];
#pragma unroll
    for (int e = 0; e < 4; ++e) split2(p[8 * tt + 2 * e], p[8 * tt + 2 * e + 1], w[e]);
    bf16x8 y[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) y[i] = as_bf16x8(make_uint4(w[0][i], w[1][i], w[2][i], w[3][i]));
    bf16x8 x[2][3];
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int i = 0; i < 3; ++i) x[db][i] = read_transposed(t.lo[db] + i * kPlane + tt * 2048, t.hi[db] + i * kPlane + tt * 2048);
    constexpr int kX[6] = {2, 0, 1, 1, 0, 0}, kY[6] = {0, 2, 1, 0, 1, 0};  // smallest products first
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int db = 0; db < 2; ++db) acc[db] = mfma(x[db][kX[i]], y[kY[i]], acc[db]);
  }
}

// The same with whole fp32 values.  Over dims: row m of the tile, and an owned row in registers (dims 8 j + 4 hl + e).
__device__ __forceinline__ void load_row(f32x4 (&b)[8], const float* X, int pos, int hl) {
#pragma unroll
  for (int j = 0; j < 8; ++j) b[j] = *reinterpret_cast<const f32x4*>(X + (unsigned)pos * kD + 8 * j + 4 * hl);
}
__device__ __forceinline__ f32x16 contract(const float* a_tile, const f32x4 (&b)[8], int m, int hl) {
  f32x16 c = zero16();
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(a_tile + m * kStride + 8 * j + 4 * hl);
#pragma unroll
    for (int e = 0; e < 4; ++e) c = mfma1(a[e], b[j][e], c);
  }
  return c;
}
// Over tile rows: columns m and 32 + m of the tile against C registers.
__device__ __forceinline__ void accumulate(f32x16 (&acc)[2], const float* tile, int m, int hl, const f32x16& p) {
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const float* row = tile + c_row(c, hl) * kStride + m;
    acc[0] = mfma1(row[0], p[c], acc[0]);
    acc[1] = mfma1(row[32], p[c], acc[1]);
  }
}

// For a tile that may hold an infinity or a NaN, or a value that has no split.  The matrix instruction multiplies every weight with
// every row, and 0 x Inf is NaN: such a row would reach the owned rows that do not meet it.  So these rows
// go through the vector ALU, owned rows that meet them only, and are cleared for the matrix instruction.
// A wavefront whose results are not all finite when its loop ends does its tiles again this way, without splits or a
// prefetch.  (Looking for such values
// in every tile instead of in the results: 88.8 us a training step for 85.6.)
__device__ __forceinline__ void accumulate_special(f32x16 (&acc)[2], float* tile, int m, int hl, f32x16& p,
                                                   const SlotWindow& mask) {
  const int lane = 32 * hl + m;
#pragma unroll 1
  for (int row = 0; row < kRows; ++row) {
    float* const x = tile + row * kStride;
    if (!__any((__float_as_uint(x[lane]) & 0x7fffffffu) >= 0x7f800000u)) continue;
    const int reg = 4 * (row >> 3) + (row & 3), half = (row >> 2) & 1;  // where the row's weights are: c_row(reg, half)
    float w = 0.f;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      w = c == reg ? p[c] : w;
      p[c] = c == reg && hl == half ? 0.f : p[c];
    }
    w = __shfl(w, 32 * half + m, 64);
    const bool in = mask.meets(row, hl);
#pragma unroll
    for (int c = 0; c < 16; c += 4)
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(x + 32 * db + 2 * c + 4 * hl);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[db][c + e] = in ? fmaf(w, v[e], acc[db][c + e]) : acc[db][c + e];
      }
    x[lane] = 0.f;
  }
  accumulate(acc, tile, m, hl, p);
}

// Is any value infinite or NaN?  (v_maximum3 keeps a NaN; assembly, because the build lets the compiler assume that
// there is none.  The compiler does not know that assembly may read a matrix result too early, so the chain
// starts with an instruction of its own that waits for both accumulators.)
__device__ __forceinline__ bool any_special(const f32x16 (&acc)[2]) {
  float x = __uint_as_float(max(__float_as_uint(acc[0][0]) & 0x7fffffffu, __float_as_uint(acc[1][0]) & 0x7fffffffu));
#pragma unroll
  for (int i = 0; i < 32; i += 2)
    asm("v_maximum3_f32 %0, |%1|, |%2|, %0" : "+v"(x) : "v"(acc[i >> 4][i & 15]), "v"(acc[i >> 4][(i & 15) + 1]));
  return __any(__float_as_uint(x) >= 0x7f800000u);
}

// Is any value's size below the lane's bound?
__device__ __forceinline__ bool any_below(const f32x16 (&acc)[2], float bound) {
  float least = fabsf(acc[0][0]);
#pragma unroll
  for (int i = 1; i < 31; i += 2) least = fminf(fminf(least, fabsf(acc[i >> 4][i & 15])), fabsf(acc[(i + 1) >> 4][(i + 1) & 15]));
  return __any(fminf(least, fabsf(acc[1][15])) < bound);
}
__device__ __forceinline__ void most_of(float& most, const f32x16& x) {
#pragma unroll
  for (int c = 0; c < 16; c += 2) most = fmaxf(fmaxf(most, fabsf(x[c])), fabsf(x[c + 1]));
}
// What the four wavefronts found in the owned rows that they loaded.
__device__ __forceinline__ int any_of(const int (&flags)[kWaves]) {
  int any = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) any |= flags[w];
  return any;
}

// Loads and stores stay on their side of this (the compiler sinks a prefetch to its first use otherwise).
__device__ __forceinline__ void keep_order() { asm volatile("" ::: "memory"); }

// A workgroup's share of the unit list: a quarter of a unit (the four quarters of one unit on one XCD).
// Consecutive workgroups of an XCD go to its four shader engines in rotation, and many units have
// fewer than four quarters with rows, so the quarters' order rotates from unit to unit: with a fixed
// order the first quarters all sat on one engine and half of the launch waited for it (dQ 44 us).
struct Quarter {
  Work w;
  int sub;
  int turn;  // which wavefront takes the first tile: the ones that get a tile more than the others
             // should not all sit on the same SIMD
};
template <bool kOwnersFirst, bool kMany>
__device__ inline bool take_quarter(const UnitLists& l, const AttnArgs& a, unsigned block, Quarter& q) {
  q.sub = ((block >> 3) + (block >> 5)) & 3;
  q.turn = block >> 5;
  const int unit = ((block >> 5) << 3) | (block & 7);
  if (kMany ? !take_unit_of_many<kOwnersFirst, false>(a, unit, q.w) : !take_unit<kOwnersFirst, false>(l, a, unit, q.w)) return false;
  const UnitPlan& u = q.w.u;
  if (u.kind == UNIT_PAD) return true;
  // (a chunked question-token owner: its first unit streams everything, there are no partials here)
  if (u.part >= 0 && u.t_begin != 0) return false;
  if (u.t0 + kRows * q.sub >= u.own_count) return false;
  // Question-token owners stream the whole sequence and end last: they go first on a shared SIMD
  // (with the fp32 instruction, beside two other wavefronts, their tiles took 7.8 us each, 2.6 us of it their own).
  if (u.kind == UNIT_GLOBAL) __builtin_amdgcn_s_setprio(3);
  return true;
}

// The owned row of a lane and the tiles its workgroup streams.
struct Rows {
  int pos, lo, hi;         // token of row m, its window of table slots
  bool valid;
  const int *gidx, *list;  // question tokens [0, G), then slots [s_lo, s_hi) of list
  int G, s_lo, s_hi, nG, n;
  __device__ __forceinline__ Rows(const Quarter& q, int m) {
    const UnitPlan& u = q.w.u;
    const int first = u.t0 + kRows * q.sub, slot = min(first + m, u.own_count - 1);
    valid = first + m < u.own_count;
    pos = u.own_list[slot];
    lo = 0;
    hi = u.L;
    if (u.kind == UNIT_LOCAL) {
      const int2 g = q.w.slot_rng[slot];
      lo = g.x;
      hi = g.y;
    }
    gidx = q.w.global_idx;
    list = u.str_list;
    G = u.G;
    s_lo = __builtin_amdgcn_readlane(lo, 0);  // windows are monotone in the slot
    s_hi = __builtin_amdgcn_readlane(hi, 31);
    nG = (G + kRows - 1) / kRows;
    n = nG + (s_hi - s_lo + kRows - 1) / kRows;
  }
  // token of row m of tile t (the last valid one past the end of a list); tiles past n repeat the last
  __device__ __forceinline__ int token(int t, int m) const {
    t = min(t, n - 1);
    return t < nG ? gidx[min(kRows * t + m, G - 1)] : list[min(s_lo + kRows * (t - nG) + m, s_hi - 1)];
  }
  __device__ __forceinline__ SlotWindow mask(int t, int hl) const {
    const bool part0 = t < nG;
    const int base = part0 ? kRows * t : s_lo + kRows * (t - nG);
    return {base + 4 * hl - (part0 ? 0 : lo), part0 ? G : hi - lo};
  }
};

// Has X a small value in this wavefront's tiles?
__device__ __forceinline__ bool any_small_row(const float* X, const Rows& r, int t0, int m, int lane) {
  bool small = false;
#pragma unroll 1
  for (int t = t0; t < r.n && !small; t += kWaves) {
    TileRegs x;
    x.load(X, r.token(t, m), lane);
    small = any_small(x.v);
  }
  return small;
}

// Sum of the four wavefronts' accumulators, stored as whole rows: lane m's column is owned row m.
// `lds` = the wavefronts' pieces, `row_tok` = the owned rows' tokens.
// kThrough: see ResultRows (the backward: with the forward 66.0 us for 4 x 512, 12 heads, and 65.2 through) and result_through.
__device__ __forceinline__ float* piece_of(char* lds, int wave) { return reinterpret_cast<float*>(lds + wave * kPlanes); }
template <bool kThrough>
__device__ __forceinline__ void store_sum(const f32x16 (&acc)[2], float mul, char* lds, const int* row_tok, float* out,
                                          int wave, int m, int hl) {
  float* mine = piece_of(lds, wave);
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 x = {acc[db][4 * g] * mul, acc[db][4 * g + 1] * mul, acc[db][4 * g + 2] * mul, acc[db][4 * g + 3] * mul};
      *reinterpret_cast<f32x4*>(mine + m * kStride + 32 * db + 8 * g + 4 * hl) = x;
    }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (threadIdx.x >> 4) + 16 * i, piece = threadIdx.x & 15, tok = row_tok[row];
    f32x4 s = *reinterpret_cast<const f32x4*>(piece_of(lds, 0) + row * kStride + 4 * piece);
#pragma unroll
    for (int w = 1; w < kWaves; ++w) s += *reinterpret_cast<const f32x4*>(piece_of(lds, w) + row * kStride + 4 * piece);
    if (tok >= 0) ResultRows<kThrough>(out).store((unsigned)tok * (kD * 4) + 16 * piece, __builtin_bit_cast(u32x4, s));
  }
}

// A quarter of a pad unit: zero rows (16 lanes each), and zeros in up to one per-position array.
template <int kTensors>
__device__ __forceinline__ void zero_pads(const Quarter& q, float* const (&out)[kTensors], float* per_row) {
  const UnitPlan& u = q.w.u;
  constexpr int kShare = kPadSlots / 4;
  const int first = u.t0 + kShare * q.sub, last = min(first + kShare, u.own_count), piece = threadIdx.x & 15;
  for (int r0 = first + (threadIdx.x >> 4); r0 < last; r0 += kThreads) {
    int tok[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) tok[i] = r0 + 16 * i < last ? u.own_list[r0 + 16 * i] : -1;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (tok[i] >= 0) {
#pragma unroll
        for (int x = 0; x < kTensors; ++x)
          ResultRows<>(out[x]).store((unsigned)tok[i] * (kD * 4) + 16 * piece, u32x4{0, 0, 0, 0});
        if (per_row && piece == 0) per_row[tok[i]] = 0.f;
      }
  }
}

// ======================================================================================
// forward
// ======================================================================================
template <bool kOwnersFirst, bool kThrough>
__global__ __launch_bounds__(kThreads, 2) void fwd_f32_kernel(MATE_UNIT_LISTS, AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds[kWaves * kPlanes];
  __shared__ __attribute__((aligned(1024))) char own[kPlanes];
  __shared__ float2 stat[kWaves][kRows];
  __shared__ int row_tok[kRows], inexact[kWaves];
  Quarter q;
  if (!take_quarter<kOwnersFirst, false>({hdr, gunit, unit_row, unit_col, B, H, N, n_col}, a, blockIdx.x, q)) return;
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, hl = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t bh = (size_t)q.w.bh * a.N;
  const float* Q = static_cast<const float*>(a.q) + bh * kD;
  const float* K = static_cast<const float*>(a.k) + bh * kD;
  const float* V = static_cast<const float*>(a.v) + bh * kD;
  float* O = static_cast<float*>(a.out) + bh * kD;
  if (q.w.u.kind == UNIT_PAD) {
    float* const outs[1] = {O};
    zero_pads<1>(q, outs, a.lse + bh);
    return;
  }
  const Rows r(q, m);
  if (tid < kRows) row_tok[tid] = r.valid ? r.pos : -1;
  const int t0 = (wave + q.turn) & (kWaves - 1);
  int tok = r.token(t0, m), tok_next = r.token(t0 + kWaves, m);
  TileRegs key, val;
  OwnedRows q_rows;
  q_rows.load(Q, r.pos, wave, lane);
  key.load(K, tok, lane);
  val.load(V, tok, lane);
  keep_order();
  q_rows.split(own, wave, lane);
  inexact[wave] = __any(q_rows.suspect()) && q_rows.inexact();
  __syncthreads();
  const int own_inexact = any_of(inexact);
  keep_order();
  char* const tile = lds + wave * kPlanes;
  const OperandLanes lanes(lane);
  const PlainAddr tile_rows(lanes, lds_addr(tile)), own_rows(lanes, lds_addr(own));
  const TransposedAddr tile_cols(lanes, lds_addr(tile));

  const float sc = a.scale * kLog2e;  // scores are kept raw; exp2(s sc - m sc)
  f32x16 o[2] = {zero16(), zero16()};
  float m_run = -INFINITY, l_run = 0.f;
  // S^T -> P^T of a tile, O and the row sum rescaled
  auto probs = [&](f32x16& s, const SlotWindow& mask, float lift) {
#pragma unroll
    for (int c = 0; c < 16; ++c) s[c] = mask.in(c) ? s[c] : -INFINITY;
    float mx = s[0];
#pragma unroll
    for (int c = 1; c < 16; ++c) mx = fmaxf(mx, s[c]);
    const float m_new = fmaxf(m_run, half_max(mx));
    const float msc = m_new == -INFINITY ? 0.f : m_new * sc;
    const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_run - m_new) * sc);
    m_run = m_new;
    l_run *= alpha;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      o[0][c] *= alpha;
      o[1][c] *= alpha;
      s[c] = __builtin_amdgcn_exp2f(fmaf(s[c], sc, -msc));
      l_run += s[c];
      s[c] *= lift;
    }
  };
  for (int t = t0; t < r.n; t += kWaves) {
    const int tok_after = r.token(t + 2 * kWaves, m);
    key.split(tile, lane);
    key.load(K, tok_next, lane);                          // the next tile's keys land during this one
    keep_order();
    f32x16 s = contract(tile_rows, own_rows);             // S^T = K Q^T
    keep_order();
    val.split(tile, lane);                                // (the keys have been read)
    val.load(V, tok_next, lane);
    keep_order();
    probs(s, r.mask(t, hl), kLift);
    accumulate(o, tile_cols, s);                          // O^T += V^T P^T
    keep_order();
    tok_next = tok_after;
  }
  float l_tot = half_sum(l_run);
  bool whole = any_special(o) || __builtin_amdgcn_readfirstlane(own_inexact) || a.scale > kLargeScale;
  if (__builtin_expect(any_below(o, l_tot * (kLift * kVisible)), 0)) whole |= any_small_row(V, r, t0, m, lane);
  if (__builtin_expect(whole, 0)) {
    o[0] = o[1] = zero16();
    m_run = -INFINITY;
    l_run = 0.f;
    float* const x = piece_of(lds, wave);
    f32x4 q_own[8];
    load_row(q_own, Q, r.pos, hl);
    for (int t = t0; t < r.n; t += kWaves) {
      tok = r.token(t, m);
      key.load(K, tok, lane);
      key.put(x, lane);
      keep_order();
      f32x16 s = contract(x, q_own, m, hl);
      keep_order();
      val.load(V, tok, lane);
      val.put(x, lane);
      keep_order();
      const SlotWindow mask = r.mask(t, hl);
      probs(s, mask, 1.f);
      accumulate_special(o, x, m, hl, s, mask);
      keep_order();
    }
    l_tot = half_sum(l_run);
  }
  // the wavefronts' maxima and sums, then their sum of O scaled to the common maximum
  if (hl == 0) stat[wave][m] = make_float2(m_run, l_tot);
  __syncthreads();
  // (a wavefront without a maximum has a sum of zero, or of NaN if it met scores of NaN only)
  auto weight = [&](float mx, float m_all) { return mx == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((mx - m_all) * sc); };
  float m_all = -INFINITY, l_all = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) m_all = fmaxf(m_all, stat[w][m].x);
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float2 ml = stat[w][m];
    l_all += ml.y * weight(ml.x, m_all);
  }
  if (wave == 0 && hl == 0 && r.valid) a.lse[bh + r.pos] = (m_all * sc + __builtin_amdgcn_logf(l_all)) * kLn2;
  float mul = weight(m_run, m_all) / l_all;
  if (!whole) {  // (where the product of both would be too small, one after the other)
    if (__builtin_expect(__any(mul < kLeast), 0))
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        o[0][c] *= 1.f / kLift;
        o[1][c] *= 1.f / kLift;
      }
    else
      mul *= 1.f / kLift;
  }
  store_sum<kThrough>(o, mul, lds, row_tok, O, wave, m, hl);
}

// ======================================================================================
// dQ
// ======================================================================================
// LDS of a backward workgroup.
struct BwdLds {
  char tiles[kWaves * kPlanes];
  char own[2 * kPlanes];        // Q, dO; or K, V
  float stat[kWaves][2][kRows]; // dK/dV, of the wavefront's tile: lse in base 2, delta
  int row_tok[kRows];
  int inexact[kWaves];          // Q; or K
};

// What delta_f32_kernel leaves for a row whose delta is zero though its dO is not (-0).
constexpr unsigned kZeroDelta = 0x80000000u;

// delta = rowsum(dO * O) of the token of row m, in the second pass: lanes m and m + 32 have half of the dims each.
__device__ __forceinline__ float row_delta(const float* dO, const float* O, int tok, int hl) {
  f32x4 g[8], o[8];
  load_row(g, dO, tok, hl);
  load_row(o, O, tok, hl);
  float d = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) d = fmaf(g[j][e], o[j][e], d);
  return half_sum(d);
}

__device__ __forceinline__ void dq_quarter(const AttnArgs& a, const Quarter& q, BwdLds& shared) {
  char *const lds = shared.tiles, *const own = shared.own;
  int* const row_tok = shared.row_tok;
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, hl = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t bh = (size_t)q.w.bh * a.N;
  const float* Q = static_cast<const float*>(a.q) + bh * kD;
  const float* K = static_cast<const float*>(a.k) + bh * kD;
  const float* V = static_cast<const float*>(a.v) + bh * kD;
  const float *dO = static_cast<const float*>(a.dout) + bh * kD, *O = static_cast<const float*>(a.o) + bh * kD;
  float* dQ = static_cast<float*>(a.dq) + bh * kD;
  if (q.w.u.kind == UNIT_PAD) {
    float* const outs[1] = {dQ};
    zero_pads<1>(q, outs, nullptr);
    return;
  }
  const Rows r(q, m);
  if (tid < kRows) row_tok[tid] = r.valid ? r.pos : -1;
  const int t0 = (wave + q.turn) & (kWaves - 1);
  int tok = r.token(t0, m), tok_next = r.token(t0 + kWaves, m);
  const float lse2 = a.lse[bh + r.pos] * kLog2e, sc = a.scale * kLog2e;
  float delta = a.delta[bh + r.pos];
  TileRegs key, val;
  {  // owned Q and dO rows to LDS
    OwnedRows g, qr;
    g.load(dO, r.pos, wave, lane);
    qr.load(Q, r.pos, wave, lane);
    val.load(V, tok, lane);
    key.load(K, tok, lane);
    keep_order();
    g.split(own + kPlanes, wave, lane);
    qr.split(own, wave, lane);
    shared.inexact[wave] = __any(qr.suspect()) && qr.inexact();
  }
  __syncthreads();
  char* const tile = lds + wave * kPlanes;
  const OperandLanes lanes(lane);
  const PlainAddr tile_rows(lanes, lds_addr(tile)), own_rows(lanes, lds_addr(own));
  const TransposedAddr tile_cols(lanes, lds_addr(tile));

  f32x16 dq[2] = {zero16(), zero16()};
  auto dscores = [&](f32x16& s, const f32x16& dp, const SlotWindow& mask, float lift) {  // S^T -> dS^T
#pragma unroll
    for (int c = 0; c < 16; ++c)
      s[c] = mask.in(c) ? __builtin_amdgcn_exp2f(fmaf(s[c], sc, -lse2)) * fmaf(dp[c], lift, -delta * lift) : 0.f;
  };
  float most = 0.f;  // of |dS|
  for (int t = t0; t < r.n; t += kWaves) {
    const int tok_after = r.token(t + 2 * kWaves, m);
    val.split(tile, lane);
    val.load(V, tok_next, lane);
    keep_order();
    const f32x16 dp = contract<1>(tile_rows, own_rows);  // dP^T = V dO^T
    keep_order();
    key.split(tile, lane);
    key.load(K, tok_next, lane);
    keep_order();
    f32x16 s = contract<0>(tile_rows, own_rows);         // S^T  = K Q^T
    dscores(s, dp, r.mask(t, hl), kLift);
    most_of(most, s);
    accumulate(dq, tile_cols, s);                   // dQ^T += K^T dS^T
    keep_order();
    tok_next = tok_after;
  }
  float mul = a.scale * (1.f / kLift);
  bool whole = any_special(dq) || __builtin_amdgcn_readfirstlane(any_of(shared.inexact)) || mul < kLeast || a.scale > kLargeScale;
  if (__builtin_expect(any_below(dq, half_max(most) * (kMostRows * kVisible)), 0)) whole |= any_small_row(K, r, t0, m, lane);
  if (__builtin_expect(__any(__float_as_uint(delta) == kZeroDelta), 0)) whole |= any_small_row(V, r, t0, m, lane);
  if (__builtin_expect(whole, 0)) {
    dq[0] = dq[1] = zero16();
    mul = a.scale;
    delta = row_delta(dO, O, r.pos, hl);
    float* const x = piece_of(lds, wave);
    for (int t = t0; t < r.n; t += kWaves) {
      tok = r.token(t, m);
      f32x4 own[8];
      load_row(own, dO, r.pos, hl);
      val.load(V, tok, lane);
      val.put(x, lane);
      keep_order();
      const f32x16 dp = contract(x, own, m, hl);
      keep_order();
      load_row(own, Q, r.pos, hl);
      key.load(K, tok, lane);
      key.put(x, lane);
      keep_order();
      f32x16 s = contract(x, own, m, hl);
      const SlotWindow mask = r.mask(t, hl);
      dscores(s, dp, mask, 1.f);
      accumulate_special(dq, x, m, hl, s, mask);
      keep_order();
    }
  }
  __syncthreads();
  store_sum<true>(dq, mul, lds, row_tok, dQ, wave, m, hl);
}

// ======================================================================================
// dK, dV: the owned rows are keys, the streamed ones the queries that see them (the same lists and
// windows as in the forward, read the other way round)
// ======================================================================================
__device__ __forceinline__ void dkv_quarter(const AttnArgs& a, const Quarter& q, BwdLds& shared) {
  char *const lds = shared.tiles, *const own = shared.own;
  int* const row_tok = shared.row_tok;
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, hl = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t bh = (size_t)q.w.bh * a.N;
  const float* Q = static_cast<const float*>(a.q) + bh * kD;
  const float* K = static_cast<const float*>(a.k) + bh * kD;
  const float* V = static_cast<const float*>(a.v) + bh * kD;
  const float *dO = static_cast<const float*>(a.dout) + bh * kD, *O = static_cast<const float*>(a.o) + bh * kD;
  float* dK = static_cast<float*>(a.dk) + bh * kD;
  float* dV = static_cast<float*>(a.dv) + bh * kD;
  if (q.w.u.kind == UNIT_PAD) {
    float* const outs[2] = {dK, dV};
    zero_pads<2>(q, outs, nullptr);
    return;
  }
  const Rows r(q, m);
  if (tid < kRows) row_tok[tid] = r.valid ? r.pos : -1;
  const int t0 = (wave + q.turn) & (kWaves - 1);
  int tok = r.token(t0, m), tok_next = r.token(t0 + kWaves, m);
  const float *lse = a.lse + bh, *delta = a.delta + bh;
  float row_lse = lse[tok], row_d = delta[tok];  // of tile row m
  TileRegs qry, grad;
  {
    OwnedRows k_rows, v_rows;
    k_rows.load(K, r.pos, wave, lane);
    v_rows.load(V, r.pos, wave, lane);
    grad.load(dO, tok, lane);
    qry.load(Q, tok, lane);
    keep_order();
    k_rows.split(own, wave, lane);
    v_rows.split(own + kPlanes, wave, lane);
    shared.inexact[wave] = __any(k_rows.suspect()) && k_rows.inexact();
  }
  __syncthreads();
  char* const tile = lds + wave * kPlanes;
  const OperandLanes lanes(lane);
  const PlainAddr tile_rows(lanes, lds_addr(tile)), own_rows(lanes, lds_addr(own));
  const TransposedAddr tile_cols(lanes, lds_addr(tile));
  const float sc = a.scale * kLog2e;

  f32x16 dk[2] = {zero16(), zero16()}, dv[2] = {zero16(), zero16()};
  float* const my_stat = &shared.stat[wave][0][0];
  bool zero_delta = false;
  auto put_stat = [&]() {
    zero_delta |= __float_as_uint(row_d) == kZeroDelta;
    if (hl == 0) {
      my_stat[m] = row_lse * kLog2e;
      my_stat[kRows + m] = row_d;
    }
  };
  // S -> P, dP -> dS.  (A pair outside the pattern has P = 0 and so dS = 0, unless a value is not finite: then dS is
  // masked as well, in the second pass.)
  auto dscores = [&](f32x16& s, f32x16& dp, const SlotWindow& mask, float lift, bool mask_ds) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 l = *reinterpret_cast<const f32x4*>(my_stat + 8 * g + 4 * hl);
      const f32x4 d = *reinterpret_cast<const f32x4*>(my_stat + kRows + 8 * g + 4 * hl);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = 4 * g + e;
        s[c] = mask.in(c) ? __builtin_amdgcn_exp2f(fmaf(s[c], sc, -l[e])) * lift : 0.f;
        dp[c] = s[c] * (dp[c] - d[e]);
        if (mask_ds) dp[c] = mask.in(c) ? dp[c] : 0.f;
      }
    }
  };
  float most = 0.f;  // of |dS|
  for (int t = t0; t < r.n; t += kWaves) {
    const int tok_after = r.token(t + 2 * kWaves, m);
    // (One tile of planes at a time, so that two workgroups fit a CU; the gradients are split twice for it.)
    grad.split(tile, lane);
    put_stat();
    keep_order();
    f32x16 dp = contract<1>(tile_rows, own_rows);  // dP = dO V^T
    keep_order();
    qry.split(tile, lane);
    qry.load(Q, tok_next, lane);
    keep_order();
    f32x16 s = contract<0>(tile_rows, own_rows);   // S  = Q K^T
    dscores(s, dp, r.mask(t, hl), kLift, false);
    most_of(most, dp);
    row_lse = lse[tok_next];
    row_d = delta[tok_next];
    accumulate(dk, tile_cols, dp);            // dK^T += Q^T dS
    keep_order();
    grad.split(tile, lane);
    grad.load(dO, tok_next, lane);
    keep_order();
    accumulate(dv, tile_cols, s);             // dV^T += dO^T P
    keep_order();
    tok_next = tok_after;
  }
  float mul_k = a.scale * (1.f / kLift), mul_v = 1.f / kLift;
  bool whole = any_special(dk) || any_special(dv) || __builtin_amdgcn_readfirstlane(any_of(shared.inexact)) || mul_k < kLeast ||
               a.scale > kLargeScale;
  if (__builtin_expect(any_below(dk, half_max(most) * (kMostRows * kVisible)), 0)) whole |= any_small_row(Q, r, t0, m, lane);
  if (__builtin_expect(__any(zero_delta), 0)) {
    f32x4 own[8];
    load_row(own, V, r.pos, hl);
    whole |= any_small(own);
  }
  if (__builtin_expect(whole, 0)) {
    mul_k = a.scale;
    mul_v = 1.f;
    dk[0] = dk[1] = dv[0] = dv[1] = zero16();
    float* const x = piece_of(lds, wave);
    for (int t = t0; t < r.n; t += kWaves) {
      tok = r.token(t, m);
      row_lse = lse[tok];
      row_d = row_delta(dO, O, tok, hl);
      f32x4 own[8];
      load_row(own, V, r.pos, hl);
      grad.load(dO, tok, lane);
      grad.put(x, lane);
      put_stat();
      keep_order();
      f32x16 dp = contract(x, own, m, hl);
      keep_order();
      load_row(own, K, r.pos, hl);
      qry.load(Q, tok, lane);
      qry.put(x, lane);
      keep_order();
      f32x16 s = contract(x, own, m, hl);
      const SlotWindow mask = r.mask(t, hl);
      dscores(s, dp, mask, 1.f, true);
      accumulate_special(dk, x, m, hl, dp, mask);
      keep_order();
      grad.put(x, lane);
      keep_order();
      accumulate_special(dv, x, m, hl, s, mask);
      keep_order();
    }
  }
  __syncthreads();
  store_sum<true>(dk, mul_k, lds, row_tok, dK, wave, m, hl);
  __syncthreads();
  store_sum<true>(dv, mul_v, lds, row_tok, dV, wave, m, hl);
}

// ======================================================================================
// The backward: delta = rowsum(dO * O), then both of the above
// ======================================================================================
// One after the other, dQ and dK/dV each ended with a last round of workgroups that left most of the chip idle (two fit on
// a CU, 4 sequences of 512 tokens with 12 heads are 1.6 rounds) or were one round of latency.  In one launch, a unit's dK/dV beside its dQ, they
// fill each other's; delta, which both need, comes from a launch of its own and is not computed by dQ.  us, backward as
// dQ and dK/dV and now: one sequence of 128, 4 heads 22.7 -> 15.3; 12 heads, one of 512 37.7 -> 25.6, of 1024 66.8 -> 42.7,
// 4 x 512 48.4 -> 46.0, 8 x 512 82.2 -> 78.0, 16 x 1024 331 -> 328.  (All of dK/dV first: 16.5, 25.9, 43.7, 46.8, 79.7, 330.)
//
// delta is NaN, which sends those that meet the row into their second pass (they compute it themselves there), where dO has
// a small value, and where it is so small against dO that dP - delta could show what dP loses with small values of V:
// at most kLost times the sum of |dO|, so 2^-35 of delta where delta is at least 2^-84 times the largest |dO|.  A delta of zero
// (V is zero where dO is not) becomes kZeroDelta instead: those that meet the row look at V, and a second pass follows if
// it has small values (4 x 512, 12 heads with V = 0 108.0 us in the second pass, 48.6 with the look, 64.7 with the fp32 instruction).
constexpr int kDeltaRows = 64;   // of a workgroup, 16 lanes of four dims each
template <int kDpp>
__device__ __forceinline__ void row_reduce(float& sum, float& most) {
  auto other = [](float x) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), kDpp, 0xf, 0xf, true));
  };
  sum += other(sum);
  most = fmaxf(most, other(most));
}
__global__ __launch_bounds__(kThreads) void delta_f32_kernel(AttnArgs a) {
  const size_t rows = (size_t)a.B * a.H * a.N, first = (size_t)blockIdx.x * kDeltaRows + (threadIdx.x >> 4);
  const int piece = threadIdx.x & 15;
  f32x4 g[4], o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const size_t at = min(first + 16 * i, rows - 1) * kD + 4 * piece;
    g[i] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.dout) + at);
    o[i] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.o) + at);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float d = g[i].x * o[i].x + g[i].y * o[i].y + g[i].z * o[i].z + g[i].w * o[i].w, most = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) most = is_small(g[i][e]) ? INFINITY : fmaxf(most, fabsf(g[i][e]));
    row_reduce<0xb1>(d, most);   // lanes ^ 1, ^ 2, and the other half of eight and of sixteen
    row_reduce<0x4e>(d, most);
    row_reduce<0x141>(d, most);
    row_reduce<0x140>(d, most);
    unsigned bits = __float_as_uint(d);
    if (fabsf(d) < most * 0x1p-84f) bits = d == 0.f && most < INFINITY ? kZeroDelta : 0x7fc00000u;
    if (piece == 0 && first + 16 * i < rows) reinterpret_cast<unsigned*>(a.delta)[first + 16 * i] = bits;
  }
}
template <bool kOwnersFirst, bool kMany>
__global__ __launch_bounds__(kThreads, 2) void bwd_f32_kernel(MATE_UNIT_LISTS, AttnArgs a, unsigned first) {
  __shared__ __attribute__((aligned(1024))) BwdLds lds;
  const unsigned block = first + blockIdx.x;
  Quarter q;
  // (32 workgroups are the quarters of eight units, one on each XCD)
  if (!take_quarter<kOwnersFirst, kMany>({hdr, gunit, unit_row, unit_col, B, H, N, n_col}, a, ((block >> 6) << 5) | (block & 31), q)) return;
  if (block & 32) dq_quarter(a, q, lds);
  else dkv_quarter(a, q, lds);
}

}  // namespace

// Question-token owners before column-head units in the forward: where the quarters of table-token units are more than the 512
// that fit the chip at once.  An owner streams the whole sequence alone, and one that starts in the second round ends long
// after everything else.  us, after and before the columns: 12 heads, 4 x 1024 47.2 -> 43.5 and (14 columns) 40.3 -> 31.4, 8 x 512
// 31.4 -> 30.7 and 27.3 -> 25.3, one sequence of 2048 53.8 -> 44.1, 2 x 1500 48.7 -> 36.0, 16 x 1024 132.6 -> 132.9; 8 heads, 2 x
// 2100 77.1 -> 52.2 (66.6 with the fp32 instruction), one of 8192 301 -> 207.  Launches that fit: one of 512 14.6 -> 15.0, 2 x
// 512 15.9 -> 16.1, one of 1000 24.6 -> 24.5.  With two or three tiles of owners a sequence the chain is short and most
// of the workgroups in front are empty: from 1024 on (8 x 300 23.5 -> 23.1, 16 x 250 30.5 -> 29.7, but 6 x 232 12.0 -> 13.1, 4 x
// 300 14.2 -> 15.1, 5 x 300 17.2 -> 17.7; one tile: 11 x 100 14.5 -> 14.2, 16 x 128 19.2 -> 19.0).
static bool owners_first(int B, int H, int N) {
  const int T = owner_slots(N);
  return 4l * B * H * T > (T == 2 || T == 3 ? 1024 : 512);
}

// The same in the backward, where an owner of dK and dV takes 22 us of 4 x 512's launch and owners began at 13: sequences of four tiles and
// more whose quarters, two for each, are more than the 512 that fit at once.  us, columns first and owners first: 12 heads, 4 x 512 42.3 -> 38.7, 3 x
// 512 40.3 -> 33.7, 2 x 478 31.5 -> 25.4, 2 x 847 65 -> 54.6, one of 847 48.6 -> 40.8, of 2048 86.9 -> 59.5, of 4096 190 -> 139, 16 x 512 137.2 -> 136.9, 16 x
// 1024 291.6 -> 291.7; 8 heads, 3 x 858 68.2 -> 56.9, 8 x 512 49.2 -> 48.7, 10 x 550 86.2 -> 86.6.  Below: 2 x 400, 8 heads 21.8 -> 23.3, one of 701
// 33.8 -> 34.1; three tiles: 2 x 377, 12 heads 22.5 -> 23.9, 10 x 301, 4 heads 22.8 -> 23.5.
static bool bwd_owners_first(int B, int H, int N) {
  const int T = owner_slots(N);
  return T > 3 && 8l * B * H * T > 512;
}

hipError_t launch_fwd_f32(const AttnArgs& a, hipStream_t stream) {
  const dim3 grid(4 * unit_grid(a.B, a.H, a.N, a.n_col)), block(kThreads);
  const bool owners = owners_first(a.B, a.H, a.N);
  const auto kernel = result_through(a.B, a.H, a.N, 4) ? (owners ? fwd_f32_kernel<true, true> : fwd_f32_kernel<false, true>)
                                                       : (owners ? fwd_f32_kernel<true, false> : fwd_f32_kernel<false, false>);
  hipLaunchKernelGGL(kernel, grid, block, 0, stream, MATE_UNIT_LISTS_VALUES(a), a);
  return hipGetLastError();
}

hipError_t launch_bwd_f32(const AttnArgs& a, hipStream_t stream) {
  const size_t rows = (size_t)a.B * a.H * a.N;
  hipLaunchKernelGGL(delta_f32_kernel, dim3((unsigned)((rows + kDeltaRows - 1) / kDeltaRows)), dim3(kThreads), 0, stream, a);
  hipError_t e = hipGetLastError();
  const unsigned blocks = 2 * 4 * (unsigned)unit_grid(a.B, a.H, a.N, a.n_col), most = 1u << 23;  // (a launch has less than 2^32 threads)
  // Step by step (see kManyRecords) from 40 rounds of workgroups on.  us, in one round trip and so, 16 heads unless said, lengths that differ: 20 x
  // 936 203.8 and 196.2, 15 x 653 131.5 and 128.6, 12 x 637 97.9 and 95.7, 18 x 846, 12 heads 142.7 and 137.9; full sequences: 29 x 315 225 and 223, 19 x
  // 652, 12 heads 241 and 237.5, 9 x 1325 421 and 424.  With fewer, full ones are up to 3 % longer (3 x 1073, 12 heads 87.7 and 90.9).  (The forward
  // gains by the round trip at any size, up to 5 %.)
  // (There the order of owners and columns makes no difference.)
  const auto kernel = blocks > 20000                      ? bwd_f32_kernel<false, true>
                      : bwd_owners_first(a.B, a.H, a.N) ? bwd_f32_kernel<true, false>
                                                        : bwd_f32_kernel<false, false>;
  for (unsigned first = 0; first < blocks && e == hipSuccess; first += most) {
    hipLaunchKernelGGL(kernel, dim3(min(most, blocks - first)), dim3(kThreads), 0, stream, MATE_UNIT_LISTS_VALUES(a), a, first);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace mate
