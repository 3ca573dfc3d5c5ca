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
// and in the backward, in place of the last two:
//   mask.load_pairs(blk)
//   mask.pair_mask(cb, i)  for words of two bf16 values: ones where the lane's streamed rows 2 i (low half) and 2 i + 1
//                          belong to the pattern for its owned row of block cb
//
// Layout everywhere: C tiles have rows = streamed rows, columns = owned rows, so per-owned-row quantities are per-lane
// scalars.  The forward has 32 x 32 tiles (lane m = owned row, lane half hl), the backward 16 x 16 ones (lane 16 q + r owns
// rows r and 16 + r of the wavefront's 32, blocks cb = 0, 1, and holds streamed rows 8 q .. 8 q + 7 of 32: see QuadLanes).
#pragma once
#include <hip/hip_runtime.h>

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
  __device__ __forceinline__ float keep(int c, float x, float other) const {
    const unsigned in = (unsigned)__builtin_amdgcn_sbfe((int)bits, 8 * (c >> 2) + (c & 3), one);
    return __uint_as_float((__float_as_uint(x) & in) | (__float_as_uint(other) & ~in));
  }
};

// The same in the backward.  A masked value is already rounded to bf16, two in a word, and so are the two halves of its mask:
// the signs of a word's two halves, spread over them by one byte permutation, from a register that has every pair's bits 16
// apart.  For P and dS four instructions per pair of each where masking them one by one takes six (dK/dV of 8 x 2048 with
// long cells 77.0 -> 75.0 us, of 16 ragged sequences of 4096 228 -> 222).
struct PairWindowMask {
  const int base, lane;
  const bool all;
  const RowPair& rng;   // of the lane's two rows: first slot | end << 16 (both are below 2^15)
  const int end;
  const int u_lo, u_hi, a_lo, a_hi;
  unsigned pairs = 0;   // bit 8 cb + 2 i and that + 16: streamed rows 2 i and 2 i + 1 of the lane's eight
  __device__ __forceinline__ PairWindowMask(int base_, int lane_, bool all_, int end_, const RowPair& rng_, int u0, int u1, int a0, int a1)
      : base(base_), lane(lane_), all(all_), rng(rng_), end(end_), u_lo(u0 - base_), u_hi(u1 - base_), a_lo(a0 - base_),
        a_hi(a1 - base_) {}
  __device__ __forceinline__ bool full(int blk) const { return 32 * blk >= a_lo && 32 * blk + 32 <= a_hi; }
  __device__ __forceinline__ bool skip(int blk) const { return 32 * blk >= u_hi || 32 * blk + 32 <= u_lo; }
  __device__ __forceinline__ void load_pairs(int blk) {
    int l = lane;
    asm volatile("" : "+v"(l));  // (the lane's first row is worked out here, not kept in a register through the loop)
    const int at = base + 32 * blk + 8 * (l >> 4);
    unsigned bits = 0;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      const unsigned r = all ? (unsigned)end << 16 : rng.v[cb];
      const int first = min(max((int)(r & 0xffffu) - at, 0), 8), last = min(max((int)(r >> 16) - at, 0), 8);
      bits |= (((1u << last) - 1u) & ~((1u << first) - 1u)) << (8 * cb);
    }
    pairs = bits | ((bits << 15) & 0xffff0000u);
  }
  __device__ __forceinline__ unsigned pair_mask(int cb, int i) const {
    return __builtin_amdgcn_perm(0u, pairs << (15 - 8 * cb - 2 * i), 0x09090808u);
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

// The backward's tiles are 16 x 16 (16x16x32 instructions).  They move half as many accumulator bytes per operation; a lane's four registers of a
// row block can all start at the same value, so dP - delta comes out of dQ's product too; and -lse / scale and -delta of a block are read once for both
// blocks of owned rows.  Operand reads are told to go ahead of the products: left to itself the compiler reads one operand of the second
// contraction, waits, multiplies and reads the next.  us by the kernel trace, both in turn, with 32 x 32 tiles and so: 2 x 8192, 16 heads dQ 61.9 -> 58.4
// and dK/dV 76.9 -> 73.9, 8 x 2048 with long cells 58.5 -> 55.1 and 73.0 -> 69.0, 16 ragged sequences of 4096 166.9 -> 160.3 and 220.7 -> 211.5, 32 x
// 512, 12 heads 32.9 -> 32.6 and 37.0 -> 36.3.  By the counters of 2 x 8192 wavefronts wait less (41.1 to 33.1 million of dK/dV's cycle counts) with as many
// vector instructions (11.6 million without the matrix ones); the kernels are 1 and 2 % shorter in cycles (109 and 137 thousand), and the rest is clock, which
// matrix instructions that move fewer bytes leave higher.  220 launches of 257 to 9000 tokens a sequence: 2.2 % shorter in the mean, up to 4 % longer where dQ and
// dK/dV are one launch (3 x 428, 12 heads, 57 question tokens 13.15 and 13.55, 5 x 381, 16 heads 14.7 and 15.1; run one after the other both kernels are
// shorter there too, and single sequences are 4 to 5 % shorter in one launch).  (The forward, whose vector part is larger, gains 2 % at 2 x 8192 and loses 1 to 3 %
// elsewhere: half of its instructions are exponentials and their sums, and a short unit's beginning and end take longer.)
//
// dQ: P = exp2(S sc - lse2), dP^T - delta = V dO^T - delta, dS = P (dP - delta), dQ^T += K^T dS^T; one 32-key block
// at a time, so only one block's scores are live.
template <class Mask>
__device__ __forceinline__ void dq_tile(unsigned tile, const bf16x8 (&qf)[2][2], const bf16x8 (&gf)[2][2], const QuadLanes& lanes,
                                             float sc, const float (&lse2)[2], const f32x4 (&ndelta)[2], Mask&& mask, f32x4 (&dq_acc)[4][2]) {
  const QuadAddr at(lanes, tile);
#pragma unroll
  for (int jb = 0; jb < 2; ++jb) {
    __builtin_amdgcn_sched_barrier(0);  // (where a mask brings no branches: blocks and their two contractions one after the other, or the registers do not do)
    if (mask.skip(jb)) continue;
    const unsigned k_at = jb * kBlockBytes, v_at = k_at + kTileBytes;
    f32x4 s[2][2], dp[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const bf16x8 k = read_quad(at, k_at, h, ks), v = read_quad(at, v_at, h, ks);
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          s[h][cb] = mfma16(k, qf[ks][cb], ks ? s[h][cb] : f32x4{0.f, 0.f, 0.f, 0.f});  // S^T  = K Q^T
          dp[h][cb] = mfma16(v, gf[ks][cb], ks ? dp[h][cb] : ndelta[cb]);               // dP^T = V dO^T
        }
      }
    unsigned dw[2][4];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int e = 0; e < 4; ++e) s[h][cb][e] = __builtin_amdgcn_exp2f(fmaf(s[h][cb][e], sc, -lse2[cb])) * dp[h][cb][e];
#pragma unroll
        for (int i = 0; i < 2; ++i) dw[cb][2 * h + i] = pack2(s[h][cb][2 * i], s[h][cb][2 * i + 1]);
      }
    if (!mask.full(jb)) {  // wave-uniform: zero the pairs outside the pattern
      mask.load_pairs(jb);
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) dw[cb][i] &= mask.pair_mask(cb, i);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const bf16x8 k = read_quad_transposed(at, k_at, d);
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
        dq_acc[d][cb] = mfma16(k, as_bf16x8(make_uint4(dw[cb][0], dw[cb][1], dw[cb][2], dw[cb][3])), dq_acc[d][cb]);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
  }
}
// dK, dV: rows of the tile are the streamed queries.  The accumulators start at the rows'
// -lse / scale and -delta (from LDS, four consecutive rows per block h), so the
// contractions deliver S - lse / scale and dP - delta directly: P = exp2(that sc), dS = P (dP - delta);
// dV^T += dO^T P, dK^T += Q^T dS.
template <class Mask>
__device__ __forceinline__ void dkv_tile(unsigned tile, const float* lse_row, const float* delta_row, const bf16x8 (&kf)[2][2],
                                              const bf16x8 (&vf)[2][2], const QuadLanes& lanes, float sc, int q, Mask&& mask,
                                              f32x4 (&dk_acc)[4][2], f32x4 (&dv_acc)[4][2]) {
  const QuadAddr at(lanes, tile);
#pragma unroll
  for (int ib = 0; ib < 2; ++ib) {
    __builtin_amdgcn_sched_barrier(0);
    if (mask.skip(ib)) continue;
    const unsigned q_at = ib * kBlockBytes, g_at = q_at + kTileBytes;
    f32x4 s[2][2], dp[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4 l4 = *reinterpret_cast<const f32x4*>(lse_row + ib * 32 + 8 * q + 4 * h);
      const f32x4 d4 = *reinterpret_cast<const f32x4*>(delta_row + ib * 32 + 8 * q + 4 * h);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const bf16x8 x = read_quad(at, q_at, h, ks), g = read_quad(at, g_at, h, ks);
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          s[h][cb] = mfma16_apart(x, kf[ks][cb], ks ? s[h][cb] : l4);    // S  = Q K^T
          dp[h][cb] = mfma16_apart(g, vf[ks][cb], ks ? dp[h][cb] : d4);  // dP = dO V^T
        }
      }
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    unsigned pw[2][4], dw[2][4];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[h][cb][e] = __builtin_amdgcn_exp2f(s[h][cb][e] * sc);  // P
          dp[h][cb][e] *= s[h][cb][e];                             // dS
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          pw[cb][2 * h + i] = pack2(s[h][cb][2 * i], s[h][cb][2 * i + 1]);
          dw[cb][2 * h + i] = pack2(dp[h][cb][2 * i], dp[h][cb][2 * i + 1]);
        }
      }
    if (!mask.full(ib)) {  // wave-uniform: zero the pairs outside the pattern
      mask.load_pairs(ib);
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const unsigned in = mask.pair_mask(cb, i);
          pw[cb][i] &= in;
          dw[cb][i] &= in;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 p8[2], ds8[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      p8[cb] = as_bf16x8(make_uint4(pw[cb][0], pw[cb][1], pw[cb][2], pw[cb][3]));
      ds8[cb] = as_bf16x8(make_uint4(dw[cb][0], dw[cb][1], dw[cb][2], dw[cb][3]));
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const bf16x8 g = read_quad_transposed(at, g_at, d), x = read_quad_transposed(at, q_at, d);
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        dv_acc[d][cb] = mfma16(g, p8[cb], dv_acc[d][cb]);   // dV^T += dO^T P
        dk_acc[d][cb] = mfma16(x, ds8[cb], dk_acc[d][cb]);  // dK^T += Q^T dS
      }
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
  }
}

}  // namespace mate
