// What a wavefront does with ONE streamed 64-row tile, shared by the segment kernels and the
// dense-mask kernels: the arithmetic is the same in both (Section 3 head equation: scores,
// one softmax, weighted sum; and its derivative), only the rule that says which (owned row,
// streamed row) pairs belong to the attention pattern differs.  That rule is the Mask argument:
//
//   mask.full(blk)     wave-uniform: every pair of the 32-row block blk belongs to the pattern (no masking)
//   mask.skip(blk)     wave-uniform: no pair of the 32-row block blk belongs to the pattern
//   mask.load(blk)     fetch what keep() needs for the 32-row block blk of the tile
//   mask.keep(c, x, o) x if the pair (this lane's owned row, streamed row c_row(c) of the loaded
//                      block) belongs to the pattern, else o.  c = accumulator register 0..15
//   Mask::kPairs       the mask also has load_pairs(blk) and pair_mask(i): ones where registers 2 i (low half of the
//                      word) and 2 i + 1 belong to the pattern, for words of two bf16 values
//
// Layout everywhere: C tiles have rows = streamed rows, columns = the wavefront's 32 owned rows
// (lane m = owned row, lane half hl), so per-owned-row quantities are per-lane scalars.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "d2l.h"
#include "mfma_common.h"

namespace mate {

// Segment path: the owned row meets the streamed sorted slots [lo, hi); the tile's first row is
// slot `base`.  (For the question-token part of a stream lo = 0, hi = G.)
//
// The window of a block is one word of bits per lane, and a pair costs a bit-field extract (0 or -1) and
// a bitwise select: no compare, whose result would travel through a scalar register pair (with the wait
// that takes between two vector instructions).  Add, compare and select per pair before: see fwd_tile.
struct WindowMask {
  const int base, hl;   // the tile's first slot (wave-uniform), the lane's half
  const bool all;       // wave-uniform: every row's window is [0, end) (the question-token part of a stream)
  const int lo, hi;     // else this lane's
  const int end;
  const int u_lo, u_hi, a_lo, a_hi;  // wave-uniform, relative to base: union and intersection of the rows' windows
  static constexpr bool kPairs = true;
  int one = 1;         // width of the extract; its value is hidden from the compiler, which would turn extract
                       // and select into test, compare and conditional move
  unsigned bits = 0;   // bit 8 (c >> 2) + (c & 3): register c of the loaded block is inside
  // [u0, u1) = union, [a0, a1) = intersection of the windows of the wavefront's rows, in the same slot
  // numbering as base.  (What a lane needs is computed where a block is masked: most blocks are not.)
  __device__ __forceinline__ WindowMask(int base_, int hl_, bool all_, int end_, int lo_, int hi_, int u0, int u1, int a0, int a1)
      : base(base_), hl(hl_), all(all_), lo(lo_), hi(hi_), end(end_), u_lo(u0 - base_), u_hi(u1 - base_), a_lo(a0 - base_),
        a_hi(a1 - base_) {
    asm("" : "+s"(one));
  }
  // base + 4 hl - lo, and the window's length
  __device__ __forceinline__ int d0() const { return base + 4 * hl - (all ? 0 : lo); }
  __device__ __forceinline__ int len() const { return all ? end : hi - lo; }
  __device__ __forceinline__ bool full(int blk) const { return 32 * blk >= a_lo && 32 * blk + 32 <= a_hi; }
  __device__ __forceinline__ bool skip(int blk) const { return 32 * blk >= u_hi || 32 * blk + 32 <= u_lo; }
  __device__ __forceinline__ void load(int blk) {
    // (31 of 32 bits are enough: the highest one asked for is 27)
    const int d = d0(), first = min(max(-d - 32 * blk, 0), 31), last = min(max(len() - d - 32 * blk, 0), 31);
    bits = ((1u << last) - 1u) & ~((1u << first) - 1u);
  }
  // Two values rounded to bf16 share a word, and so do the two halves of its mask: the signs of a word's two
  // halves, spread over them by one byte permutation, from a register that has every pair's bits 16 apart.  For P and dS four
  // instructions per pair of each where masking them one by one takes six (dK/dV of 8 x 2048 with long cells 77.0 -> 75.0 us, of
  // 2 x 8192 82.0 -> 79.7, of 16 ragged sequences of 4096 228 -> 222); for dS or P alone three where it takes four,
  // which gained nothing.
  unsigned pairs[2];   // of registers 0..7 and 8..15: bit 8 g + 2 i and that + 16: pair i of group g
  __device__ __forceinline__ void load_pairs(int blk) {
    load(blk);
    pairs[0] = (bits & 0xffffu) | ((bits << 15) & 0xffff0000u);
    pairs[1] = (bits >> 16) | ((bits >> 1) & 0xffff0000u);
  }
  __device__ __forceinline__ unsigned pair_mask(int i) const {
    return __builtin_amdgcn_perm(0u, pairs[i >> 2] << (15 - 8 * ((i >> 1) & 1) - 2 * (i & 1)), 0x09090808u);
  }
  __device__ __forceinline__ float keep(int c, float x, float other) const {
    const unsigned in = (unsigned)__builtin_amdgcn_sbfe((int)bits, 8 * (c >> 2) + (c & 3), one);
    return __uint_as_float((__float_as_uint(x) & in) | (__float_as_uint(other) & ~in));
  }
};

// Forward: S^T = K Q^T, mask, online softmax in base 2 (reference score m_run of the raw scores, this lane
// half's share l_run of the row sum), P rounded to bf16, O^T += V^T P^T.
//
// Softmax needs a reference near the row's maximum, not the maximum: any other changes neither the
// relative rounding of P in bf16 nor the accuracy of the fp32 sums, as long as nothing overflows.  So
// only a tile that finds a row without a reference takes the maximum of its scores (and rescales what
// was summed so far); the others use the reference as it is and look at the sum of the tile's
// probabilities afterwards.  Where one exceeds 2^13 (one score more than 8 to 13 bits above the reference)
// the tile starts again with the maximum, and from there on this wavefront's reference follows the maximum in
// every tile, without the trial: rows whose scores have risen once tend to rise again.  (Starting again each
// time cost inputs of widely spread scores, standard deviation 60 before the scale, up to two fifths of the
// forward: B = 2, N = 8192, H = 16 67 us, now 57.3, and 51.2 at standard-normal inputs; dense 8 x 1024, H = 12
// 61, now 48.8, and 43.9.  Scaling sums and rounded probabilities by a power of two instead is as fast, but the
// largest probability is then a rounded one and not 1, and the mean error of such rows' LSE five times as large.)
// Vector and matrix instructions of the resident wavefronts mostly take turns here, and under full load the
// chip lowers its clock (2.4 to 1.95 GHz), so every instruction left out counts: without the 16 three-operand
// maxima and the rescaling decision per tile, with two instructions per masked pair instead of three and a wait,
// and with single blocks, B = 2, N = 8192, H = 16 takes 54 instead of 57 us, B = 8, N = 2048 49 instead of 53.
constexpr float kMaxTileSum = 8192.f;
// A wavefront's reference: missing for one of its rows, as the first tiles left it, or following the maximum.
enum Reference { kMissing, kFixed, kFollows };
// P^T of the tile as the second contraction's operands, [32-key block][half of it], two bf16 values in a word.  (Words,
// because the compiler takes vectors of bf16 that live across a branch apart and converts every value twice.)
typedef unsigned Probs[2][2][4];
// A tile of which only one 32-key block is visible is done with that block alone (kBlocks = 1); branching
// around the blocks inside one body would cost the interleaving of their instruction streams.
//
// S^T = K Q^T of kBlocks 32-key blocks from block blk0 on: rows = keys, columns = this wave's queries; -inf
// outside the pattern.
template <int kBlocks, class Mask>
__device__ __forceinline__ void fwd_scores(int blk0, const PlainAddr& k, const bf16x8 (&qf)[4], Mask& mask, f32x16 (&s)[kBlocks]) {
#pragma unroll
  for (int jb = 0; jb < kBlocks; ++jb) {
    s[jb] = zero16();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) s[jb] = mfma(read_plain(k.a[ks] + jb * 32 * 128), qf[ks], s[jb]);
  }
  if constexpr (kBlocks == 2) {  // six of the eight operands ahead: all eight do not fit the registers
    __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
  }
  // wave-uniform: some (query, key) pairs are outside the pattern
  if (!(mask.full(blk0) && mask.full(blk0 + kBlocks - 1))) {
#pragma unroll
    for (int jb = 0; jb < kBlocks; ++jb) {
      mask.load(blk0 + jb);
#pragma unroll
      for (int c = 0; c < 16; ++c) s[jb][c] = mask.keep(c, s[jb][c], -INFINITY);
    }
  }
}
// P^T = exp2(S^T sc - msc), rounded to bf16; returns the sum of the rounded values
template <int kBlocks>
__device__ __forceinline__ float fwd_probs(f32x16 (&s)[kBlocks], float sc, float msc, Probs& pb) {
  float l[kBlocks];
#pragma unroll
  for (int jb = 0; jb < kBlocks; ++jb) {
    l[jb] = 0.f;
#pragma unroll
    for (int c = 0; c < 16; ++c) s[jb][c] = __builtin_amdgcn_exp2f(fmaf(s[jb][c], sc, -msc));
#pragma unroll
    for (int c = 0; c < 16; c += 2) {
      unsigned& w = pb[jb][c >> 3][(c >> 1) & 3];
      w = pack2(s[jb][c], s[jb][c + 1]);
      l[jb] = sum2(w, l[jb]);
    }
  }
  return kBlocks == 2 ? l[0] + l[kBlocks - 1] : l[0];
}
template <int kBlocks, class Mask>
__device__ __forceinline__ float fwd_probs_new_max(int blk0, const PlainAddr& k, const bf16x8 (&qf)[4], Mask& mask, float sc,
                                                   float& m_run, Probs& pb) {
  f32x16 s[kBlocks];
  fwd_scores<kBlocks>(blk0, k, qf, mask, s);
  float mx = s[0][0];
#pragma unroll
  for (int jb = 0; jb < kBlocks; ++jb)
#pragma unroll
    for (int c = 0; c < 16; c += 2) mx = fmaxf(fmaxf(mx, s[jb][c]), s[jb][c + 1]);
  m_run = fmaxf(m_run, half_max(mx));
  return fwd_probs<kBlocks>(s, sc, (m_run == -INFINITY ? 0.f : m_run) * sc, pb);
}
// `tile`: LDS address of the K tile; the V tile follows.
template <class Mask>
__device__ __forceinline__ void fwd_tile(unsigned tile, const bf16x8 (&qf)[4], const OperandLanes& lanes, float sc, Mask&& mask,
                                         f32x16 (&o_acc)[2], float& m_run, float& l_run, Reference& ref) {
  const bool skip0 = mask.skip(0), skip1 = mask.skip(1);
  if (skip0 && skip1) return;
  // (a word: a condition that lives across the branches below would go through a vector register)
  const int both = __builtin_amdgcn_readfirstlane(!skip0 && !skip1);
  const int blk0 = skip0 ? 1 : 0;
  tile += blk0 * 32 * 128;
  const PlainAddr k(lanes, tile);
  // O^T += V^T P^T
  auto add = [&](const Probs& pb, float l_tile) {
    l_run += l_tile;
    const TransposedAddr v(lanes, tile + kTileBytes);
    auto block = [&](int jb) {
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        const int at = (jb * 32 + tt * 16) * 128;
        const bf16x8 p = as_bf16x8(make_uint4(pb[jb][tt][0], pb[jb][tt][1], pb[jb][tt][2], pb[jb][tt][3]));
#pragma unroll
        for (int db = 0; db < 2; ++db) o_acc[db] = mfma(read_transposed(v.lo[db] + at, v.hi[db] + at), p, o_acc[db]);
      }
    };
    block(0);
    if (both) block(1);
  };
  if (ref == kFixed) {
    Probs pb;
    float l_tile;
    if (both) {
      f32x16 s[2];
      fwd_scores<2>(0, k, qf, mask, s);
      l_tile = fwd_probs<2>(s, sc, m_run * sc, pb);
    } else {
      f32x16 s[1];
      fwd_scores<1>(blk0, k, qf, mask, s);
      l_tile = fwd_probs<1>(s, sc, m_run * sc, pb);
    }
    if (__all(l_tile <= kMaxTileSum)) return add(pb, l_tile);
    ref = kFollows;
  }
  Probs pb;
  const float m_old = m_run;
  const float l_tile = both ? fwd_probs_new_max<2>(0, k, qf, mask, sc, m_run, pb)
                            : fwd_probs_new_max<1>(blk0, k, qf, mask, sc, m_run, pb);
  if (__any(m_old != -INFINITY)) {  // (not for a wavefront's first tile: there is nothing to scale)
    const float alpha = m_run == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((m_old - m_run) * sc);
    l_run *= alpha;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int c = 0; c < 16; ++c) o_acc[db][c] *= alpha;
  }
  if (ref == kMissing && !__any(m_run == -INFINITY)) ref = kFixed;
  add(pb, l_tile);
}

// dQ: P = exp2(S sc - lse2), dP^T = V dO^T, dS = P (dP - delta), dQ^T += K^T dS^T; one 32-key block
// at a time, so only one block's scores are live.
template <class Mask>
__device__ __forceinline__ void dq_tile(unsigned tile, const bf16x8 (&qf)[4], const bf16x8 (&gf)[4], const OperandLanes& lanes,
                                        float sc, float lse2, float delta, Mask&& mask, f32x16 (&dq_acc)[2]) {
  const PlainAddr p(lanes, tile);  // K; V follows it
  const TransposedAddr kt(lanes, tile);
#pragma unroll
  for (int jb = 0; jb < 2; ++jb) {
    if (mask.skip(jb)) continue;
    f32x16 s = zero16(), dp = zero16();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      s = mfma(read_plain(p.a[ks] + jb * 32 * 128), qf[ks], s);                 // S^T  = K Q^T
      dp = mfma(read_plain(p.a[ks] + kTileBytes + jb * 32 * 128), gf[ks], dp);  // dP^T = V dO^T
    }
#pragma unroll
    for (int c = 0; c < 16; ++c)
      s[c] = __builtin_amdgcn_exp2f(fmaf(s[c], sc, -lse2)) * (dp[c] - delta);
    if (!mask.full(jb)) {  // wave-uniform: zero the pairs outside the pattern
      mask.load(jb);
#pragma unroll
      for (int c = 0; c < 16; ++c) s[c] = mask.keep(c, s[c], 0.f);
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const bf16x8 ds8 = pack8(s, 8 * tt);
      const int at = (jb * 32 + tt * 16) * 128;
#pragma unroll
      for (int db = 0; db < 2; ++db) dq_acc[db] = mfma(read_transposed(kt.lo[db] + at, kt.hi[db] + at), ds8, dq_acc[db]);
    }
  }
}

// dK, dV: rows of the tile are the streamed queries.  The accumulators start at the rows'
// -lse / scale and -delta (from LDS, four consecutive rows per group of four registers), so the
// contractions deliver S - lse / scale and dP - delta directly: P = exp2(that sc), dS = P (dP - delta);
// dV^T += dO^T P, dK^T += Q^T dS.
template <class Mask>
__device__ __forceinline__ void dkv_tile(unsigned tile, const float* lse_row, const float* delta_row, const bf16x8 (&kf)[4],
                                         const bf16x8 (&vf)[4], const OperandLanes& lanes, float sc, int hl, Mask&& mask,
                                         f32x16 (&dk_acc)[2], f32x16 (&dv_acc)[2]) {
  const PlainAddr p(lanes, tile);  // Q; dO follows it
  const TransposedAddr t(lanes, tile);
#pragma unroll
  for (int ib = 0; ib < 2; ++ib) {
    if (mask.skip(ib)) continue;
    f32x16 s, dp;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int row0 = ib * 32 + 8 * g + 4 * hl;
      const float4 l4 = *reinterpret_cast<const float4*>(lse_row + row0);
      const float4 d4 = *reinterpret_cast<const float4*>(delta_row + row0);
      s[4 * g] = l4.x; s[4 * g + 1] = l4.y; s[4 * g + 2] = l4.z; s[4 * g + 3] = l4.w;
      dp[4 * g] = d4.x; dp[4 * g + 1] = d4.y; dp[4 * g + 2] = d4.z; dp[4 * g + 3] = d4.w;
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      s = mfma(read_plain(p.a[ks] + ib * 32 * 128), kf[ks], s);                 // S  = Q K^T
      dp = mfma(read_plain(p.a[ks] + kTileBytes + ib * 32 * 128), vf[ks], dp);  // dP = dO V^T
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      s[c] = __builtin_amdgcn_exp2f(s[c] * sc);  // P
      dp[c] *= s[c];                             // dS
    }
    // wave-uniform: zero the pairs outside the pattern
    constexpr bool kPairs = std::remove_reference<Mask>::type::kPairs;
    if (!kPairs && !mask.full(ib)) {
      mask.load(ib);
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        s[c] = mask.keep(c, s[c], 0.f);
        dp[c] = mask.keep(c, dp[c], 0.f);
      }
    }
    unsigned pw[8], dw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      pw[i] = pack2(s[2 * i], s[2 * i + 1]);
      dw[i] = pack2(dp[2 * i], dp[2 * i + 1]);
    }
    if constexpr (kPairs)
      if (!mask.full(ib)) {
        mask.load_pairs(ib);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const unsigned in = mask.pair_mask(i);
          pw[i] &= in;
          dw[i] &= in;
        }
      }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const bf16x8 p8 = as_bf16x8(make_uint4(pw[4 * tt], pw[4 * tt + 1], pw[4 * tt + 2], pw[4 * tt + 3]));
      const bf16x8 ds8 = as_bf16x8(make_uint4(dw[4 * tt], dw[4 * tt + 1], dw[4 * tt + 2], dw[4 * tt + 3]));
      const int q_at = (ib * 32 + tt * 16) * 128, g_at = q_at + kTileBytes;
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        dv_acc[db] = mfma(read_transposed(t.lo[db] + g_at, t.hi[db] + g_at), p8, dv_acc[db]);   // dV^T += dO^T P
        dk_acc[db] = mfma(read_transposed(t.lo[db] + q_at, t.hi[db] + q_at), ds8, dk_acc[db]);  // dK^T += Q^T dS
      }
    }
  }
}

}  // namespace mate
