// The projections either side of the attention and their gradients, bf16 MFMA (gfx950):
//   QKV:  q[b,i,k,:] = W_Q^i x[b,k,:], likewise K and V -- the W^i X_k of the head equation of
//         Section 3 for all heads at once, written straight into the [B, H, N, 64] layout the
//         attention kernels read (the head split costs nothing);
//   out:  y[b,k,:] = W_O concat_i o[b,i,k,:], reading the attention output head by head in the
//         layout it was written in (no concatenation pass);
//   dX, d_o: the same products with the weight matrix transposed, read through transposing LDS
//         reads from the matrix as it is;
//   dW:   contracts over tokens, dW[f, e] = sum_tok G[tok, f] X[tok, e].
// Pad tokens are not computed when a whole token tile is padding, and are stored as zeros.
//
// All are one main loop over two operands: C[b, a] = sum_k B[b, k] A[a, k], a contiguous in the
// output (features, or columns of dW), so that the MFMA accumulator layout (rows = a: a lane holds
// four consecutive a of one b) turns into 16-byte stores without a detour through LDS.  Operands are
// streamed in tiles of 64 rows x 128 bytes straight from global memory into LDS (global_load_lds_dwordx4),
// XOR-swizzled so that plain 16-byte operand reads and transposing 8-byte ones are both free of bank
// conflicts, through a ring of stages with explicit vmcnt waits.  A tile is either "plain" (rows =
// operand rows, 64 of k per stage) or "transposed" (rows = 64 of k, columns = operand rows: whatever
// contracts over tokens, and the weights of dX and d_o).
//
// v_mfma_f32_16x16x32_bf16 rather than 32x32x16: at these sizes the chip is limited by power, and the
// smaller instruction moves half as many accumulator bytes per operation (16384 x 3072 x 1024: 97 us
// against 104 us, everything else equal).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "arrival.h"
#include "d2l.h"
#include "launch.h"
#include "mfma_common.h"
#include "tile_deal.h"

namespace mate {
namespace {

// A pointer the compiler can keep in scalar registers (the value is the same in every lane).
__device__ inline const char* uniform_ptr(const void* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return reinterpret_cast<const char*>(((unsigned long long)hi << 32) | lo);
}

// Workgroup shape: kA x 64 rows of operand A by kB x 64 rows of operand B, kWA x kWB wavefronts; kGroups such
// sets of wavefronts share the contraction (stage k belongs to group k mod kGroups, each group has its own
// ring of stages) and add their accumulators at the end.
//
// Two groups are for products with so few tiles that a CU has one: alone, four wavefronts read LDS and
// multiply in turns (0.6 us a stage of 128 x 128 where the matrix pipe needs 0.2), and two workgroups on a
// CU drift apart so that one reads while the other multiplies.  Two groups of one workgroup would read at the
// same time, because every stage has a barrier; so they are kept half a stage apart (kAlternate): a second
// barrier between reading and multiplying, and group 1 one barrier behind.  dX at 8 x 512 tokens and 768
// wide 26.4 -> 21.8 us, its weight gradient 35.3 -> 32.9, that of the output projection 29.2 -> 24.6; in
// step they gained 0 to 2.  (The 128 x 64 shape with its shorter stages, three of them, is better in step.)
//
// Eight wavefronts on one tile (256 x 256) are kept apart in the same way, the upper four half a slice behind
// the lower four, where the weights' products use them: 1024 -> 3072 features at 2 x 8192 tokens 97.5 -> 93.0
// us, 3072 -> 1024 81.7 -> 78.5.  In the weight gradient, whose operands are both read through the slower
// transposing reads, the reads of one half outlast the products of the other: 111 -> 117 us, so not there.
template <int kA_, int kB_, int kWA_, int kWB_, int kStages_, int kPerCU_, int kGroups_ = 1>
struct Shape {
  static constexpr int kA = kA_, kB = kB_, kWA = kWA_, kWB = kWB_, kStages = kStages_, kPerCU = kPerCU_, kGroups = kGroups_;
  static constexpr int kWaves = kWA * kWB, kAllWaves = kWaves * kGroups, kThreads = 64 * kAllWaves;
  static constexpr int kRowsA = 64 * kA, kRowsB = 64 * kB;
  static constexpr int kFA = 4 * kA / kWA, kFB = 4 * kB / kWB;  // 16-row blocks of a wavefront
  static constexpr int kOutB = kFB / kGroups;                   // and those of B that it stores
  static constexpr bool kAlternate = kGroups == 2 && kStages == 2;
  static constexpr int kStageBytes = (kA + kB) * kTileBytes, kRingBytes = kStages * kStageBytes, kLds = kGroups * kRingBytes;
  static constexpr int kLoadsA = 8 * kA / kWaves, kLoadsB = 8 * kB / kWaves, kLoads = kLoadsA + kLoadsB;
  static_assert(8 * kA % kWaves == 0 && 8 * kB % kWaves == 0, "loads must divide evenly");
  static_assert(4 * kA % kWA == 0 && 4 * kB % kWB == 0 && kFA % 2 == 0 && kFB % kGroups == 0, "blocks must divide evenly");
  static_assert(kGroups == 1 || kGroups == 2, "the exchange is between two groups");
};

// Load instruction i of a wavefront brings eight rows of one tile: which tile, which row this lane's
// 16 bytes belong to, and which 16-byte chunk of it.
struct LoadUnit {
  int tile, row, chunk;
};
template <int kWaves>
__device__ __forceinline__ LoadUnit load_unit(int wave, int lane, int i) {
  const int u = wave + kWaves * i;
  LoadUnit l;
  l.tile = u >> 3;
  l.row = (u & 7) * 8 + (lane >> 3);
  l.chunk = (lane & 7) ^ swz(l.row & 15);
  return l;
}
template <int kWaves>
__device__ __forceinline__ int load_dst(int wave, int i) {
  const int u = wave + kWaves * i;
  return (u >> 3) * kTileBytes + (u & 7) * 8 * 128;
}

// Operand fragment of 16 rows and 32 of k.  Lane l = 16 q + r: row r, k = 8 q .. 8 q + 7.
struct FragOffsets {
  int plain[2];      // per 32-wide k slice
  int trans[2][4];   // [first / second four of k][16-column block of a tile]; a k slice is 32 rows further
};
template <bool kTransposed>
__device__ __forceinline__ void frag_offsets(FragOffsets& f, int lane) {
  const int r = lane & 15, q = lane >> 4;
  if (!kTransposed) {
#pragma unroll
    for (int k = 0; k < 2; ++k) f.plain[k] = r * 128 + (((4 * k + q) ^ swz(r)) << 4);
  } else {
    // 16 lanes read 4 rows x 16 columns: lane i addresses row i / 4, columns 4 (i % 4) .., and receives
    // column i of the four rows
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int row = 8 * q + 4 * h + (r >> 2);
#pragma unroll
      for (int c = 0; c < 4; ++c)
        f.trans[h][c] = row * 128 + (((2 * c + ((r & 3) >> 1)) ^ swz(row & 15)) << 4) + ((r & 1) << 3);
    }
  }
}
template <bool kTransposed>
__device__ __forceinline__ bf16x8 read_frag(const char* tiles, const FragOffsets& f, int block, int k) {
  if (!kTransposed) return read_plain(tiles + block * 16 * 128, f.plain[k]);
  const char* t = tiles + (block >> 2) * kTileBytes + k * 32 * 128;
  return read_transposed(t, f.trans[0][block & 3], f.trans[1][block & 3]);
}

// One stage (64 of k): two slices of 32.
// `issue` starts the loads of a later stage.  Where the stage's operands are plain it does so behind the operand
// reads: its instructions (eight for 256 x 256, each with an address and m0) then cost the wavefront time in which its
// reads travel, not time before them.  256 x 256 at 16384 x 3072 x 1024 2590 -> 2539 cycles a stage (2885 while the reads had bank
// conflicts); whole products in 128 x 64 with two groups 5 to 9 % shorter, 128 x 128 with two groups 2 to 5, 192 x 128 1 to 2.
// Transposing reads are twice as many instructions, and behind them the loads come too late: all gradients with `issue` behind
// the reads take 3 to 6 % more in the mean.  And 128 x 128 with one group: 5 % less to 7 % more, none in the mean.
// kHalves: `next_landed` is called where this wavefront's share of the next stage must have landed.
// kAlternate: `reading` is called while the fragments travel and the other group multiplies.
template <class S, bool kTA, bool kTB, bool kHalves, class Issue, class PerSlice, class Next, class Reading>
__device__ __forceinline__ void contract_stage(const char* stage, const FragOffsets& fa, const FragOffsets& fb, int wa,
                                               int wb, f32x4 (&acc)[S::kFA][S::kFB], Issue&& issue, PerSlice&& per_slice,
                                               Next&& next_landed, Reading&& reading) {
  const char* ta = stage + (kTA ? 0 : wa * S::kFA * 16 * 128);
  const char* tb = stage + S::kA * kTileBytes + (kTB ? 0 : wb * S::kFB * 16 * 128);
  constexpr bool kIssueLate = !kTA && (S::kGroups > 1 || S::kFA * S::kFB != 16);
  bf16x8 a[2][S::kFA], b[2][S::kFB];
  auto read_slice = [&](int k) {
#pragma unroll
    for (int i = 0; i < S::kFA; ++i) a[k][i] = read_frag<kTA>(ta, fa, (kTA ? wa * S::kFA : 0) + i, k);
#pragma unroll
    for (int j = 0; j < S::kFB; ++j) b[k][j] = read_frag<kTB>(tb, fb, (kTB ? wb * S::kFB : 0) + j, k);
  };
  if (!kIssueLate) issue();
  if constexpr (kHalves) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (k) barrier_no_fence();
      __builtin_amdgcn_sched_barrier(0);
      read_slice(k);
      if (kIssueLate && !k) issue();
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (k) next_landed();
      __builtin_amdgcn_sched_barrier(0);
      barrier_no_fence();  // from here on the other half reads
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < S::kFA; ++i)
#pragma unroll
        for (int j = 0; j < S::kFB; ++j) acc[i][j] = mfma16(a[k][i], b[k][j], acc[i][j]);
      per_slice(b[k]);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(0);
    }
    return;
  }
  read_slice(0);
  if constexpr (S::kAlternate) {
    read_slice(1);
    if (kIssueLate) issue();
    reading();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    barrier_no_fence();  // from here on the other group reads
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (k == 0 && !S::kAlternate) {
      read_slice(1);  // the second slice travels while the first is contracted
      if (kIssueLate) issue();
    }
#pragma unroll
    for (int i = 0; i < S::kFA; ++i)
#pragma unroll
      for (int j = 0; j < S::kFB; ++j) acc[i][j] = mfma16(a[k][i], b[k][j], acc[i][j]);
    if constexpr (!S::kAlternate) per_slice(b[k]);
  }
  if constexpr (S::kAlternate) {
    per_slice(b[0]);
    per_slice(b[1]);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
  }
}
// The two groups' accumulators: each wavefront gives half of its blocks of B to its counterpart in the
// other group, through LDS, and keeps the sum of the other half.  (Group 0 stores blocks 0 .. kOutB - 1.)
template <class S>
__device__ __forceinline__ void add_groups(f32x4 (&acc)[S::kFA][S::kFB], f32x4 (&out)[S::kFA][S::kOutB], char* lds, int group,
                                           int wave, int lane) {
  if constexpr (S::kGroups == 1) {
#pragma unroll
    for (int i = 0; i < S::kFA; ++i)
#pragma unroll
      for (int j = 0; j < S::kOutB; ++j) out[i][j] = acc[i][j];
  } else {
    constexpr int kBlocks = S::kFA * S::kOutB;
    static_assert(2 * S::kWaves * kBlocks * 1024 <= S::kLds, "the exchange must fit the stages");
    f32x4* x = reinterpret_cast<f32x4*>(lds) + lane;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < S::kFA; ++i)
#pragma unroll
      for (int j = 0; j < S::kOutB; ++j)
        x[((group * S::kWaves + wave) * kBlocks + i * S::kOutB + j) * 64] = group ? acc[i][j] : acc[i][j + S::kOutB];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < S::kFA; ++i)
#pragma unroll
      for (int j = 0; j < S::kOutB; ++j) {
        const f32x4 other = x[(((1 - group) * S::kWaves + wave) * kBlocks + i * S::kOutB + j) * 64];
        out[i][j] = group ? other + acc[i][j + S::kOutB] : acc[i][j] + other;
      }
  }
}

// Partial sums of a weight gradient (one fp32 matrix per token range, see below), added in range order
// by the workgroups behind the tiles of the product that follows: a launch of its own took 11 to 14 us
// on the benchmark layer, 5 of them the launch, while the product leaves compute units idle at its end.
struct RangeSums {
  const float* part;       // [splits][n] partial sums, n a multiple of 4
  const float* part_bias;  // [splits][n_bias]
  float *out, *out_bias;   // out_bias may be null
  size_t n;
  int n_bias, splits, blocks;  // blocks: workgroups that share the work (0: nothing to add)
};
__device__ __forceinline__ void add_ranges(const RangeSums& s, int block, int threads) {
  const size_t stride = (size_t)s.blocks * threads, first = (size_t)block * threads + threadIdx.x;
  const f32x4* part = reinterpret_cast<const f32x4*>(s.part);
  for (size_t i = first; i < s.n / 4; i += stride) {
    f32x4 v = part[i];
    for (int k0 = 1; k0 < s.splits; k0 += 4) {  // four at a time, all loaded before the first is added
      f32x4 x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = part[(size_t)min(k0 + e, s.splits - 1) * (s.n / 4) + i];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k0 + e < s.splits) v += x[e];
    }
    reinterpret_cast<f32x4*>(s.out)[i] = v;
  }
  if (s.out_bias)
    for (size_t i = first; i < (size_t)s.n_bias; i += stride) {
      float v = s.part_bias[i];
      for (int k = 1; k < s.splits; ++k) v += s.part_bias[(size_t)k * s.n_bias + i];
      s.out_bias[i] = v;
    }
}

// ======================================================================================
// Products with the weights: forward, dX, d_o
// ======================================================================================
// What a tile's first loads need: kernel arguments of their own, the first ones, because plain values arrive in registers with
// the wavefront.
struct ProjStart {
  const unsigned short* w;       // plain: [F][K] row-major; transposed: [K][F]
  const unsigned short* tok;     // flat tokens: [B*N][K] row-major (x, or dy in the backward)
  const unsigned char* flags;    // [B][N]
  int N;
  int F, K;                      // features, contraction length
  TileDeal deal;
};
struct ProjArgs : ProjStart {
  const unsigned short* tok3[3]; // head tokens: [B][H][N][64] tensors whose heads are the k steps, one
                                 // after the other (o; or dq, dk, dv in the backward)
  const float* bias;             // [F] or null
  unsigned short* out[3];        // head layout: q, k, v (or d_o) [B][H][N][64];  flat: [B][N][F] in out[0]
  int B, H;
  int lazy_tiles;                // the tiles before this one leave their results in the L2
  RangeSums ranges;
};

// kHeadTok: the token operand comes from head-layout tensors and the output is flat; else the reverse.
// kTransposedW: the weight operand is read transposed.
template <class S, bool kHeadTok, bool kTransposedW, bool kBeside>
__device__ __forceinline__ void product_tile(const ProjStart& p, const ProjArgs& a, char* lds, int b, int n0, int f0, bool through) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave_id / S::kWaves, wave = wave_id - group * S::kWaves;
  const int wa = wave / S::kWB, wb = wave - wa * S::kWB;
  const int r = lane & 15, quarter = lane >> 4;
  char* const ring = lds + group * S::kRingBytes;

  const int rows = min(S::kRowsB, p.N - n0), feats = min(S::kRowsA, p.F - f0);

  // ---- operand streams: per load a wave-uniform base and a 32-bit lane offset -----------------------
  unsigned off[S::kLoads];
#pragma unroll
  for (int i = 0; i < S::kLoadsA; ++i) {
    const LoadUnit l = load_unit<S::kWaves>(wave, lane, i);
    // (features past F repeat the last 64-column block or the last row, and are not stored)
    off[i] = kTransposedW ? (unsigned)l.row * (unsigned)p.F * 2 + (unsigned)min(64 * l.tile, feats - 64) * 2 + l.chunk * 16
                          : (unsigned)min(64 * l.tile + l.row, feats - 1) * (unsigned)p.K * 2 + l.chunk * 16;
  }
#pragma unroll
  for (int i = 0; i < S::kLoadsB; ++i) {  // (tokens past the end repeat the last one)
    const LoadUnit l = load_unit<S::kWaves>(wave, lane, i);
    off[S::kLoadsA + i] = (unsigned)min(64 * l.tile + l.row, rows - 1) * (kHeadTok ? kD * 2u : (unsigned)p.K * 2) + l.chunk * 16;
  }
  const unsigned short *tok3_1 = a.tok3[1], *tok3_2 = a.tok3[2];
  const size_t w_step = kTransposedW ? (size_t)64 * p.F * 2 : 128;
  const char* w_ptr = reinterpret_cast<const char*>(kTransposedW ? p.w + f0 : p.w + (size_t)f0 * p.K) + group * w_step;  // of the next stage
  const size_t head0 = (((size_t)b * a.H) * p.N + n0) * kD * 2, t_step = kHeadTok ? (size_t)p.N * kD * 2 : 128;
  const char* t_ptr = kHeadTok ? reinterpret_cast<const char*>(a.tok3[0]) + head0
                               : reinterpret_cast<const char*>(p.tok + ((size_t)b * p.N + n0) * p.K);
  t_ptr += group * t_step;
  int head = group, tensor = 0;
  auto issue_stage = [&](int g) {
    char* st = ring + (g % S::kStages) * S::kStageBytes;
    const char *w_base = uniform_ptr(w_ptr), *t_base = uniform_ptr(t_ptr);
#pragma unroll
    for (int i = 0; i < S::kLoadsA; ++i) load_to_lds_16(w_base, off[i], st + load_dst<S::kWaves>(wave, i));
#pragma unroll
    for (int i = 0; i < S::kLoadsB; ++i)
      load_to_lds_16(t_base, off[S::kLoadsA + i], st + S::kA * kTileBytes + load_dst<S::kWaves>(wave, i));
    w_ptr += S::kGroups * w_step;
    t_ptr += S::kGroups * t_step;
    if (kHeadTok && (head += S::kGroups) >= a.H) {  // the next tensor's heads (H is even)
      head -= a.H;
      ++tensor;
      t_ptr = reinterpret_cast<const char*>(pick(tensor == 1, tok3_1, tok3_2)) + head0 + head * t_step;
    }
  };
  constexpr bool kHalves = S::kGroups == 1 && S::kWaves == 8 && S::kStages == 2;
  const int nk = p.K / 64 / S::kGroups;  // this group's stages (K is a multiple of 128)
#pragma unroll
  for (int s = 0; s < S::kStages - 1; ++s)
    if (s < nk) issue_stage(s);

  // While the first stages travel: is any token of the tile not padding (every wavefront looks at all of
  // them), which of this lane's are, and the bias of this lane's features.
  const unsigned char* fl = p.flags + (size_t)b * p.N + n0;
  bool any = false;
#pragma unroll
  for (int i = 0; i < S::kB; ++i) any |= fl[min(64 * i + lane, rows - 1)] < 2;
  const int j0 = wb * S::kFB + group * S::kOutB;  // first block of tokens that this wavefront stores
  int row[S::kOutB];
  unsigned pad_bits = 0;
#pragma unroll
  for (int j = 0; j < S::kOutB; ++j) {
    row[j] = min((j0 + j) * 16 + r, rows - 1);
    pad_bits |= (unsigned)(fl[row[j]] >= 2) << j;
  }
  f32x4 bias[S::kFA];
#pragma unroll
  for (int i = 0; i < S::kFA; ++i) bias[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (a.bias)   // (one branch around all loads: a branch each had a wait each)
#pragma unroll
    for (int i = 0; i < S::kFA; ++i) bias[i] = *reinterpret_cast<const f32x4*>(a.bias + f0 + min((wa * S::kFA + i) * 16, feats - 16) + 4 * quarter);

  f32x4 acc[S::kFA][S::kFB];
#pragma unroll
  for (int i = 0; i < S::kFA; ++i)
#pragma unroll
    for (int j = 0; j < S::kFB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (__any(any)) {  // (a tile of padding only is stored as zeros without arithmetic)
    FragOffsets fa, fb;
    frag_offsets<kTransposedW>(fa, lane);
    frag_offsets<false>(fb, lane);
    // the second half, or group, follows one barrier behind
    const bool apart = kHalves || S::kAlternate, second = kHalves ? wave >= 4 : group == 1;
    if (kHalves) wait_vmcnt_le<0>(0);
    if (apart && second) barrier_no_fence();
    for (int ks = 0; ks < nk; ++ks) {
      // stage ks has landed: everything but the younger stages' loads (fewer near the end)
      if (!kHalves) wait_vmcnt_le<S::kLoads * (S::kStages - 2)>(min(S::kStages - 2, nk - 1 - ks) * S::kLoads);
      barrier_no_fence();  // ... for every wavefront, and everyone is done with stage ks - 1
      contract_stage<S, kTransposedW, false, kHalves>(ring + (ks % S::kStages) * S::kStageBytes, fa, fb, wa, wb, acc,
                                                      [&]() { if (ks + S::kStages - 1 < nk) issue_stage(ks + S::kStages - 1); },
                                                      [](const bf16x8 (&)[S::kFB]) {}, []() { wait_vmcnt_le<0>(0); }, []() {});
    }
    if (apart && !second) barrier_no_fence();
  }
  f32x4 sum[S::kFA][S::kOutB];
  add_groups<S>(acc, sum, lds, group, wave, lane);

  unsigned short *const out_0 = a.out[0], *const out_1 = a.out[1], *const out_2 = a.out[2];
  // ---- epilogue: + bias, round to bf16.  A lane holds features 16 i + 4 quarter .. + 3 of token 16 j + r;
  // after exchanging quarters between neighbouring blocks it holds eight consecutive ones and stores
  // 16 bytes, 64 of a token's bytes per instruction. ------------------------------------------------
  auto store = [&](auto through) {
#pragma unroll
    for (int i = 0; i < S::kFA; i += 2) {
      const int fw = (wa * S::kFA + i) * 16;       // first feature of the block pair in the tile
      if (fw >= feats) break;                      // (F is a multiple of 64: a pair is inside or outside)
      unsigned short* dst;
      if (kHeadTok) dst = out_0 + ((size_t)b * p.N + n0) * p.F + f0 + fw;
      else {
        const int head_slot = (f0 + fw) >> 6, x = head_slot / a.H, h = head_slot - x * a.H;
        dst = pick(x == 0, out_0, pick(x == 1, out_1, out_2)) + (((size_t)b * a.H + h) * p.N + n0) * kD + (fw & 63);
      }
      const ResultRows<true> past_l2(dst);
      const ResultRows<false> in_l2(dst);
      const unsigned token_bytes = (kHeadTok ? (unsigned)p.F : (unsigned)kD) * 2;   // between consecutive tokens
#pragma unroll
      for (int j = 0; j < S::kOutB; ++j) {
        unsigned u[2][2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const f32x4 c = sum[i + p][j] + bias[i + p];
          u[p][0] = pack2(c[0], c[1]);
          u[p][1] = pack2(c[2], c[3]);
        }
        const auto lo = __builtin_amdgcn_permlane16_swap(u[0][0], u[1][0], false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(u[0][1], u[1][1], false, false);
        u32x4 v = {lo[0], hi[0], lo[1], hi[1]};
        if ((pad_bits >> j) & 1u) v = u32x4{0, 0, 0, 0};
        if ((j0 + j) * 16 + r < rows) {
          const unsigned at = (unsigned)row[j] * token_bytes + ((quarter & 1) * 16 + (quarter >> 1) * 8) * 2;
          if (through) past_l2.store(at, v);
          else in_l2.store(at, v);
        }
      }
    }
  };
  // Two groups: one copy of this, with a branch at every store; one group, or beside a weight gradient: a copy for each.  us, with two copies and
  // with one: d_o 256 x 256 at 33 tokens 4.88 and 4.43, output 768 x 768 at 7 x 97 7.37 and 7.14, QKV there 8.6 and 8.3, over 1000 products in two
  // groups 2 to 5 % shorter in the mean; one group, d_o 128 x 128 at 40 tokens 3.50 and 3.91; both gradients of 512 x 512 at 51 12.4 and 12.8.
  if constexpr (S::kGroups == 2 && !kBeside) store(through);
  else if (through) store(std::true_type());
  else store(std::false_type());
}

template <class S, bool kHeadTok, bool kTransposedW, bool kBeside = false>
__device__ __forceinline__ void dealt_product(const ProjStart& p, const ProjArgs& a, char* lds, int x, int y) {
  int token_tile, feature_tile, tile;
  if (!dealt_tile(p.deal, x, y, token_tile, feature_tile)) return;
  const int b = sequence_of(token_tile, (p.N + S::kRowsB - 1) / S::kRowsB, tile);
  product_tile<S, kHeadTok, kTransposedW, kBeside>(p, a, lds, b, tile * S::kRowsB, feature_tile * S::kRowsA, y * p.deal.grid_x() + x >= a.lazy_tiles);
}

template <class S, bool kHeadTok, bool kTransposedW>
__global__ __launch_bounds__(S::kThreads, S::kAllWaves / 4 * S::kPerCU) void proj_kernel(
    const unsigned short* w, const unsigned short* tok, const unsigned char* flags, int N, int F, int K, int token_tiles, int feature_tiles,
    int whole_rows, int by_feature, ProjArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const ProjStart p = {w, tok, flags, N, F, K, {token_tiles, feature_tiles, whole_rows, by_feature}};
  const int x = blockIdx.x, y = blockIdx.y + kMostGridY * blockIdx.z, behind = y - p.deal.grid_y();
  if (behind < 0) dealt_product<S, kHeadTok, kTransposedW>(p, a, lds, x, y);
  else if (behind * p.deal.grid_x() < a.ranges.blocks) add_ranges(a.ranges, behind * p.deal.grid_x() + x, S::kThreads);  // behind the tiles: partial sums of a weight gradient
}

// Tiles of a product, and how many a CU takes one after the other.
template <class S>
long tiles_of(const ProjArgs& a) {
  return (long)a.B * ((a.N + S::kRowsB - 1) / S::kRowsB) * ((a.F + S::kRowsA - 1) / S::kRowsA);
}
long rounds(long tiles) { return (tiles + 255) / 256; }

template <class S>
void deal_tiles(ProjArgs& a) {
  TileDeal& d = a.deal;
  d.tokens = a.B * ((a.N + S::kRowsB - 1) / S::kRowsB);
  d.features = (a.F + S::kRowsA - 1) / S::kRowsA;
  // every XCD reads all of the other operand: the smaller one (us by token tiles and by feature tiles: 1024 -> 3072 at 600
  // tokens 12.1 and 9.8, at 1200 13.8 and 12.5, at 1700 16.8 and 16.5; 2048 -> 6144 at 1000 33.5 and 32.0).  Fewer than eight
  // feature tiles would all be dealt one by one, and each be read by every XCD: dX 640 wide (five) at 3 x 173 tokens 12.9 and 13.5,
  // 768 wide (six) at 295 15.1 and 15.5, where 1024 wide (eight) at 512 takes 20.5 and 18.9; QKV and output of five and six gain 0 to 1 %.
  d.by_feature = a.F > (long)a.B * a.N && d.features >= 8;
  d.rows = (d.by_feature ? d.features : d.tokens) / 8;
}

// How many tiles, the first ones, leave their part of the result in the L2 (see ResultRows): all that do not fit it at the end anyway.
// The last 32 MB are what the L2s hold.  us, left, through for the last 64 MB, and for the last 32: 768 -> 2304 at 6 x 8447 tokens, 30 %
// padding (233 MB) 169.8, 175.8, 171.9, 1024 -> 3072 at 8 x 4096 (201 MB) 190.6, 191.9, 187.2, at 14566 (89 MB) 89.4, 86.9, 86.7, 768 ->
// 2304 at 2 x 11434 (105 MB) 77.6, 76.3, 75.8, 1024 -> 1024 at 8 x 4096 (67 MB) 61.5, 60.4, 59.6; 768 -> 768 at 8 x 2048 (25 MB) 19.9 and,
// through, 18.1.  The gradients
// behind a weight gradient lose by the last 64 MB of a long result what they gain by a short one: dX (and dW) at 2 x 8192, 1024 wide (34
// MB) 140 and 138, at 4 x 10584 217 and 222, at 16 x 4096 (101 MB) 334 and 343, d_o there 138 and 143.
template <class S, bool kTransposedW>
int lazy_tiles(const ProjArgs& a) {
  const size_t tiles = (size_t)a.deal.tokens * a.deal.features, bytes = tiles * (S::kRowsA * S::kRowsB * 2);
  if (kTransposedW) return bytes <= (48u << 20) ? 0 : (int)tiles;
  return (int)(tiles - std::min(tiles, (size_t)(32u << 20) / (S::kRowsA * S::kRowsB * 2)));
}

template <class S, bool kHeadTok, bool kTransposedW>
hipError_t launch_proj(ProjArgs a, int kernel_id, hipStream_t stream) {
  deal_tiles<S>(a);
  a.lazy_tiles = lazy_tiles<S, kTransposedW>(a);
  const int x = a.deal.grid_x();
  int range_rows = 0;
  if (a.ranges.splits) {
    range_rows = (int)(std::max<size_t>(1, std::min<size_t>(1024 * 256 / S::kThreads, a.ranges.n / 4 / S::kThreads)) + x - 1) / x;
    a.ranges.blocks = range_rows * x;
  }
  const int y = a.deal.grid_y() + range_rows;
  const dim3 grid(x, std::min(y, kMostGridY), (y + kMostGridY - 1) / kMostGridY);
  const hipError_t e = allow_lds<&proj_kernel<S, kHeadTok, kTransposedW>>(S::kLds);
  if (e != hipSuccess) return e;
  ProfileScope prof(kernel_id, stream);
  hipLaunchKernelGGL((proj_kernel<S, kHeadTok, kTransposedW>), grid, dim3(S::kThreads),
                     S::kLds, stream, a.w, a.tok, a.flags, a.N, a.F, a.K, a.deal.tokens, a.deal.features, a.deal.rows, a.deal.by_feature, a);
  return hipGetLastError();
}

// Which shape.  A compute unit that gets n tiles of a shape needs about (k / 64) (c2 for every two tiles, c1 for
// an odd last one) + e n us, so the shape with the smallest such sum wins, n being the rounds of tiles:
// large tiles once they fill the chip, smaller ones where they fit its units better.  The constants were fitted
// to the times of six shapes for 912 products when n was the rounds of the busiest of eight XCDs, which no deal of tiles evened out; with the
// present deal, n and nine shapes, over 7148 products (64 to 40000 tokens, widths 128 to 4096, 2 to 32 heads, no padding), the shape that they
// choose takes 0.5 % more than the fastest one on average, more than 5 % in one of 26 and 27 % at most (short contractions of 128 and 256
// terms and many tokens, where larger tiles than the chosen ones would be faster).  For
// instance, us, 256 x 256, 192 x 128, 128 x 128, with two groups, 128 x 64, with two groups: 2048 -> 6144 at 900
// tokens 47, 39, 34, 40, 55, 61, at 8 x 512 98, 116, 111, 132, 216, 225; 1024 -> 3072 at 512 tokens 27, 17, 15, 12, 11, 11.
// 192 x 128 with two groups came later, fitted to 186 products (128 to 16384 tokens, widths 128 to 2048): it is for
// the few sizes whose tiles fill most of one round and no more, where a unit that has the same tile to itself waits
// at every stage.  us, before and with it: 768 -> 2304 at 1999 tokens 15.4 and 14.6, 1024 -> 3072 at 1500 19.0 and
// 17.2, 1536 -> 4608 at 1000 28.2 and 24.0, 768 -> 768 at 8192 15.6 and 14.4; in a second round it loses (768 -> 2304
// at 2300 tokens 16.2 and 25.4), which its constant for two tiles says.
// 192 x 256 and 256 x 192, eight wavefronts, read 0.9 of what a CU loads for as many products in 192 x 128 and have a third more
// tiles than 256 x 256: for sizes whose tiles are one round.  us, before and with them: 768 -> 2304 at 8 x 512 23.1 -> 22.1, at
// 5 x 929 22.7 -> 21.3, 1024 -> 3072 at 4000 28.1 -> 25.3, 1024 -> 1024 at 2 x 4344 28.0 -> 23.5, at 10752 29.4 -> 26.4, d_o
// there with dW 55.5 -> 52.2.  Their constants (1.0 a stage, 6.8) were read off these times and are the same for both; where both are
// one round, 256 x 192 is taken if it has fewer tiles, which compute less past the last feature and the last token, and 192 x 256 has more than 200.  With
// fewer than that a fifth of the CUs is idle in either, and a tile of 256 tokens has more of them past the end of a short sequence, which cost it nothing.
// us, 192 x 256 and 256 x 192: 2048 -> 6144 at 4 x 295 (256 and 192 tiles) 39.9 and 36.2, 1536 -> 1536 at 16 x 324 31.5 and 28.3, 768 -> 2304 at 4 x 1058
// (240 and 216) 18.6 and 17.0, 1280 -> 3840 at 12 x 192 (240 and 180) 26.5 and 27.7; of 270 products with fewer tiles of 256 x 192 the 206 with more than
// 200 of 192 x 256 are 1.9 % shorter in the mean, 11 % at best, 4 % longer at worst, the others 1.6 % longer, 6 % at worst (1024 -> 3072 at 12 x
// 192, 192 and 144 tiles, 20.0 and 21.2, 1536 -> 4608 at 8 x 164 27.0 and 28.9).  As many
// tiles: 22 products, equal in the mean (768 -> 2304 at 8 x 512, 192 and 216 tiles, 17.6 and 18.1, at 3 x 1511 19.1 and 21.2, 1536 -> 4608 at 3 x
// 593 33.9 and 31.7); more tiles: 17, 0.5 % longer.
//                        features x tokens, wavefronts, stages, workgroups per CU, groups
using Proj256 = Shape<4, 4, 2, 4, 2, 1>;      // 256 x 256
using Proj192x256 = Shape<3, 4, 2, 4, 2, 1>;  // 192 x 256  (plain weights, as below)
using Proj256x192 = Shape<4, 3, 4, 2, 2, 1>;  // 256 x 192
using Proj192 = Shape<3, 2, 2, 2, 2, 2>;      // 192 x 128  (plain weights; its wavefronts' 96 features are not whole tiles)
using Proj192x2 = Shape<3, 2, 2, 2, 2, 1, 2>; // (all 160 KB of a compute unit's LDS)
using Proj128 = Shape<2, 2, 2, 2, 2, 2>;      // 128 x 128
using Proj128x2 = Shape<2, 2, 2, 2, 2, 1, 2>;
using Proj64 = Shape<2, 1, 2, 2, 3, 2>;       // 128 x  64
using Proj64x2 = Shape<2, 1, 2, 2, 3, 1, 2>;
template <class S>
double proj_cost(const ProjArgs& a, double c1, double c2, double e) {
  const long n = rounds(tiles_of<S>(a));
  return (a.K / 64) * ((n / 2) * c2 + (n % 2) * c1) + e * n;
}

typedef hipError_t (*ProjLaunch)(ProjArgs, int, hipStream_t);
struct ProjChoice {
  double cost;
  ProjLaunch launch;
  int groups;   // shapes with as many groups add up a product's stages in the same order
};
template <bool kHeadTok, bool kTransposedW>
ProjChoice choose_proj(const ProjArgs& a) {
  ProjChoice best = {1e30, nullptr, 0};
  auto offer = [&](double cost, ProjLaunch launch, int groups) {
    if (cost < best.cost) best = {cost, launch, groups};
  };
  offer(proj_cost<Proj256>(a, 1.37, 3.14, 5.33), launch_proj<Proj256, kHeadTok, kTransposedW>, 1);
  // In one round only: in a second one, where sequences end in padding, 256 x 256 has skipped enough tiles to need none (1024 ->
  // 3072 at 12000 tokens, a fifth of them padding, 65.7 and 71.4 us).  dX, whose weights are four times as long, gains nothing.
  // And where 128 x 128 needs more than the two tiles that a CU takes at once: long products in those take less than their
  // constants say (us, 128 x 128 and these: 4096 -> 6144 at 8 x 76 tokens 55.0 and 74.7, 3456 -> 3840 at 1988 52.2 and 64.5, 4096 -> 2304 at 2 x
  // 1769 65.9 and 80.1, d_o of 1536 from 3584 at 11 x 248 46.4 and 60.2; shorter ones are told apart by the costs).
  const bool large = tiles_of<Proj128>(a) > 512;
  if constexpr (!kTransposedW)
    if (large && tiles_of<Proj192x256>(a) <= std::min(256l, std::max(200l, tiles_of<Proj256x192>(a))))
      offer(proj_cost<Proj192x256>(a, 1.0, 0, 6.8), launch_proj<Proj192x256, kHeadTok, kTransposedW>, 1);
  if constexpr (!kTransposedW || !kHeadTok)
    if (large && tiles_of<Proj256x192>(a) <= 256) offer(proj_cost<Proj256x192>(a, 1.0, 0, 6.8), launch_proj<Proj256x192, kHeadTok, kTransposedW>, 1);
  if constexpr (!kTransposedW)
    // (beyond 4608 features it takes up to 23 % more than its constants say)
    if (a.F % Proj192::kRowsA == 0 && a.F <= 4608) {
      offer(proj_cost<Proj192>(a, 1.17, 1.52, 0.86), launch_proj<Proj192, kHeadTok, kTransposedW>, 1);
      offer(proj_cost<Proj192x2>(a, 0.8, 1.5, 4.6), launch_proj<Proj192x2, kHeadTok, kTransposedW>, 2);
    }
  offer(proj_cost<Proj128>(a, 0.62, 1.09, 1.1), launch_proj<Proj128, kHeadTok, kTransposedW>, 1);
  offer(proj_cost<Proj128x2>(a, 0.47, 1.2, 1.86), launch_proj<Proj128x2, kHeadTok, kTransposedW>, 2);
  offer(proj_cost<Proj64>(a, 0.46, 0.74, 0.53), launch_proj<Proj64, kHeadTok, kTransposedW>, 1);
  offer(proj_cost<Proj64x2>(a, 0.39, 0.8, 0.71), launch_proj<Proj64x2, kHeadTok, kTransposedW>, 2);
  return best;
}

// ======================================================================================
// Gradient with respect to the weights
// ======================================================================================
// Both operands are token-major, so their 64-token x 64-column tiles go into LDS as they are and both
// are read transposed.  A workgroup owns a tile of dW and a range of the token blocks; partial sums of
// the ranges are added in a fixed order afterwards (no atomics: the result is bit-reproducible).  The bias gradient (column sums of G) rides along in the workgroups of the first
// column tile.  Rows of pad tokens are cleared in LDS after a block has landed, and blocks of padding
// only are skipped.

// Token-major matrix whose 64-column blocks are either columns of a flat [B*N][ld] matrix or
// heads of up to three [B][H][N][64] tensors (column block c <-> tensor c / H, head c % H).
struct TokMat {
  const unsigned short* p[3];
  int heads;          // 1: head layout, 0: flat
  int ld;             // flat: elements per row
};
struct WgradArgs {
  TokMat g, x;                    // G [tok][F-side], X [tok][E-side]
  const unsigned char* flags;     // [B][N]
  float* out;                     // [F][E] (final when splits == 1)
  float* out_bias;                // [F] or null
  float* part;                    // [splits][F][E] partial sums (splits > 1)
  float* part_bias;               // [splits][F]
  unsigned long long* arrived;    // [tiles][kMaxRanges], where the ranges are added in the launch
  unsigned long long ticket;
  int B, N, H;
  int F, E;                       // rows and columns of dW
  int blocks_per_seq;             // ceil(N / 64)
  int splits, per_split;          // token-block ranges
  int want_bias;
};
constexpr int kMaxRange = 1024;   // token blocks of one range
constexpr int kMaxRanges = 8;     // of a launch that adds them itself

// Which of the 64 tokens from position n0 of the sequence at flags[seq] on are padding (or past its end):
// one bit each.  `total` = bytes of the flags array, which is read 64 bytes at a time.
__device__ __forceinline__ unsigned long long pad_mask(const unsigned char* flags, size_t total, size_t seq, int n0, int N) {
  const int n = min(64, N - n0);
  const size_t first = seq + n0;
  unsigned long long bits = 0;
  if (total >= 64) {
    const size_t at = first < total - 64 ? first : total - 64;  // the 64 bytes must lie inside the array
    unsigned w[16];
    __builtin_memcpy(w, flags + at, 64);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const unsigned two = w[i] & 0xfefefefeu;  // a byte of 2 or more leaves a bit here: collect it in bit 7
      const unsigned pad = (((two & 0x7f7f7f7fu) + 0x7f7f7f7fu) | two) & 0x80808080u;
      bits |= (unsigned long long)(((pad >> 7) * 0x10204080u) >> 28) << (4 * i);
    }
    bits >>= (int)(first - at);
  } else {
    for (int i = 0; i < n; ++i) bits |= (unsigned long long)(flags[first + i] >= 2) << i;
  }
  return n < 64 ? bits | ~0ull << n : bits;
}

// kList: token blocks of one range at most.  kChain > 0: a group's accumulators go into a second set after every
// kChain blocks, so that a long range is no less exact than the sum of short ones.
// kMerge: the range of a tile that is done last adds them all (otherwise another launch does).  Partial sums of a range are
// then whole tiles, one after the other, so F and E must be whole tiles as well.
// kThrough: see ResultRows; not where another launch of the same tiles follows (8 x 2048 tokens, 768 wide gain 1.5 %, 4 x 10584
// and 16 x 4096 lose 1.5 %).
template <class S, int kList, int kChain, bool kMerge, bool kThrough>
__device__ __forceinline__ void wgrad_tile(WgradArgs a, char* lds, int block) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave_id / S::kWaves, wave = wave_id - group * S::kWaves;
  char* const ring = lds + group * S::kRingBytes;
  const int e_tiles = (a.E + S::kRowsA - 1) / S::kRowsA, tiles = ((a.F + S::kRowsB - 1) / S::kRowsB) * e_tiles;
  // Workgroup -> (token range, tile): XCD q = block % 8 takes a contiguous piece of the list
  // ordered by token range first, so the workgroups that stream the same tokens share an L2
  // (dealt round-robin, every XCD would fetch all of G from memory: 8 x the traffic).
  const int total = tiles * a.splits, per_xcd = (total + 7) >> 3;
  const int q = block & 7, jx = block >> 3, idx = q * per_xcd + jx;
  if (jx >= per_xcd || idx >= total) return;
  const int split = idx / tiles, tile = idx - split * tiles;
  const int ft = tile / e_tiles, et = tile - ft * e_tiles;
  const int f0 = ft * S::kRowsB, e0 = et * S::kRowsA;
  const int wa = wave / S::kWB, wb = wave - wa * S::kWB;
  const int total_blocks = a.B * a.blocks_per_seq;
  // Up to kList token blocks: every workgroup lists all of them and takes its share of the live ones
  // (with ranges of equal length the padding at the end of the sequences left some ranges half empty:
  // 52 live blocks in the longest of five where 41 would do).  More: ranges of equal length.
  const bool share = total_blocks <= kList;
  const int s_begin = share ? 0 : split * a.per_split, s_end = share ? total_blocks : min(total_blocks, s_begin + a.per_split);

  // ---- the blocks with a non-pad row, in order, and their pad masks, listed in LDS before the
  // loop (looked up one by one inside it, every step waited for dependent loads: 3 us a step where the
  // contractions need 0.9) ----
  __shared__ unsigned long long live_mask[kList];
  __shared__ uint2 live_at[kList];  // where the block begins in X and G, in units of 128 bytes
  __shared__ int wave_live[S::kAllWaves], first_tail;
  int n_live = 0;
  const unsigned x_stride = a.x.heads ? kD * 2 : (unsigned)a.x.ld * 2, g_stride = a.g.heads ? kD * 2 : (unsigned)a.g.ld * 2;
  const unsigned x_seq = (unsigned)((a.x.heads ? (size_t)a.H * a.N * kD * 2 : (size_t)a.N * x_stride) / 128);
  const unsigned g_seq = (unsigned)((a.g.heads ? (size_t)a.H * a.N * kD * 2 : (size_t)a.N * g_stride) / 128);
  if (tid == 0) first_tail = kList;  // (the loop's first barrier comes before anyone else's turn)
  for (int s0 = s_begin; s0 < s_end; s0 += S::kThreads) {  // one block per thread, its 64 flags at once
    const int s = s0 + tid, b = s / a.blocks_per_seq;
    const unsigned long long mask = s < s_end ? pad_mask(a.flags, (size_t)a.B * a.N, (size_t)b * a.N, (s - b * a.blocks_per_seq) * 64, a.N) : ~0ull;
    const unsigned long long ballot = __ballot(mask != ~0ull);
    if (lane == 0) wave_live[wave_id] = __popcll(ballot);
    __syncthreads();
    int at = n_live + __popcll(ballot & ((1ull << lane) - 1));
#pragma unroll
    for (int w = 0; w < S::kAllWaves; ++w) {
      if (w < wave_id) at += wave_live[w];
      n_live += wave_live[w];
    }
    if (mask != ~0ull) {
      const unsigned n0 = (unsigned)(s - b * a.blocks_per_seq) * 64;
      live_mask[at] = mask;
      live_at[at] = make_uint2(b * x_seq + n0 * (x_stride / 128), b * g_seq + n0 * (g_stride / 128));
      if ((size_t)a.B * a.N - ((size_t)b * a.N + n0) < 64) atomicMin(&first_tail, at);
    }
    __syncthreads();
  }
  n_live = __builtin_amdgcn_readfirstlane(n_live);
  const int i_begin = share ? n_live * split / a.splits : 0, i_end = share ? n_live * (split + 1) / a.splits : n_live;

  // ---- operand streams: X tiles (columns e0 ..) then G tiles (columns f0 ..) ------------------------
  // The bases are wave-uniform and move with the block; the lane offsets are those of a whole block.  A sequence's
  // last, shorter block reads into the rows that follow, which are cleared like pad rows; only where fewer than 64 rows
  // are left before memory may end (the end of the last sequence, or of the last few if they are short) does it
  // repeat its last row instead.
  constexpr int kTilesX = S::kA, kTilesG = S::kB;
  const char* base[kTilesX + kTilesG];
#pragma unroll
  for (int t = 0; t < kTilesX + kTilesG; ++t) {
    const bool is_x = t < kTilesX;
    const TokMat& mat = is_x ? a.x : a.g;
    // (column blocks past the last one repeat it and are not stored)
    const int c = is_x ? min(e0 / 64 + t, a.E / 64 - 1) : min(f0 / 64 + t - kTilesX, a.F / 64 - 1);
    const int x = c / a.H, h = c - x * a.H;
    const unsigned short* tensor = !mat.heads || x == 0 ? mat.p[0] : x == 1 ? mat.p[1] : mat.p[2];
    base[t] = uniform_ptr(tensor + (mat.heads ? (size_t)h * a.N * kD : (size_t)c * 64));
  }
  unsigned off[S::kLoads];
#pragma unroll
  for (int i = 0; i < S::kLoads; ++i) {
    const LoadUnit l = load_unit<S::kWaves>(wave, lane, i < S::kLoadsA ? i : i - S::kLoadsA);
    off[i] = (unsigned)l.row * (i < S::kLoadsA ? x_stride : g_stride) + l.chunk * 16;
  }
  const int tail = __builtin_amdgcn_readfirstlane(first_tail), tail_rows = a.N % 64;
  auto issue_stage = [&](int i_live, uint2 at, int slot) {
    char* st = ring + slot * S::kStageBytes;
    const size_t x_at = (size_t)(unsigned)__builtin_amdgcn_readfirstlane(at.x) * 128;
    const size_t g_at = (size_t)(unsigned)__builtin_amdgcn_readfirstlane(at.y) * 128;
    auto issue = [&](auto whole) {
#pragma unroll
      for (int i = 0; i < S::kLoads; ++i) {
        const bool is_x = i < S::kLoadsA;
        const int y = is_x ? i : i - S::kLoadsA, tile = S::kWaves * y / 8;
        unsigned o = off[i];
        if (!decltype(whole)::value)
          o -= (unsigned)max(0, load_unit<S::kWaves>(wave, lane, y).row - (tail_rows - 1)) * (is_x ? x_stride : g_stride);
        load_to_lds_16(base[is_x ? tile : kTilesX + tile] + (is_x ? x_at : g_at), o,
                       st + (is_x ? 0 : S::kA * kTileBytes) + load_dst<S::kWaves>(wave, y));
      }
    };
    if (__builtin_expect(i_live >= tail, 0)) issue(std::false_type());
    else issue(std::true_type());
  };

  f32x4 acc[S::kFA][S::kFB];
#pragma unroll
  for (int i = 0; i < S::kFA; ++i)
#pragma unroll
    for (int j = 0; j < S::kFB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 chains[S::kFA][S::kFB];  // (the first chain sets it: zeroing it took short ranges 0.3 us)
  float bias_acc[S::kFB];
#pragma unroll
  for (int j = 0; j < S::kFB; ++j) bias_acc[j] = 0.f;
  const bool do_bias = a.want_bias && et == 0 && wa == 0;
  FragOffsets fo;
  frag_offsets<true>(fo, lane);

  // this group's blocks: i_begin + group, + kGroups, ...
#pragma unroll
  for (int k = 0; k + 1 < S::kStages; ++k)
    if (i_begin + group + k * S::kGroups < i_end)
      issue_stage(i_begin + group + k * S::kGroups, live_at[i_begin + group + k * S::kGroups], k);
  // My share of block i has landed: everything but the loads of the blocks after it that were issued.  Its pad
  // rows are cleared (0 x anything = 0 then).
  auto land = [&](int i, int it) {
    wait_vmcnt_le<S::kLoads * (S::kStages - 2)>(max(0, min(S::kStages - 2, (i_end - 1 - i) / S::kGroups)) * S::kLoads);
    // (an odd last block leaves group 1 a block of padding only)
    const unsigned long long padmask = S::kGroups == 1 || i < i_end ? live_mask[i] : ~0ull;
    if (padmask) {
      char* st = ring + (it % S::kStages) * S::kStageBytes;
#pragma unroll
      for (int l = 0; l < S::kLoads; ++l) {
        const int y = l < S::kLoadsA ? l : l - S::kLoadsA;
        if ((padmask >> load_unit<S::kWaves>(wave, lane, y).row) & 1ull)
          *reinterpret_cast<uint4*>(st + (l < S::kLoadsA ? 0 : S::kA * kTileBytes) + load_dst<S::kWaves>(wave, y) + lane * 16) =
              make_uint4(0, 0, 0, 0);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
  };
  if (S::kAlternate && group == 1) barrier_no_fence();  // group 1 follows one barrier behind
  for (int i0 = i_begin, it = 0; i0 < i_end; i0 += S::kGroups, ++it) {
    const int i = i0 + group, ahead = i + (S::kStages - 1) * S::kGroups;
    const uint2 next = live_at[min(ahead, i_end - 1)];
    land(i, it);
    barrier_no_fence();          // landed for everyone; and everyone is done with the block before it
    contract_stage<S, true, true, false>(ring + (it % S::kStages) * S::kStageBytes, fo, fo, wa, wb, acc,
                                  [&]() { if (ahead < i_end) issue_stage(ahead, next, (it + S::kStages - 1) % S::kStages); },
                                  [&](const bf16x8 (&g)[S::kFB]) {
                                    if (do_bias) {
#pragma unroll
                                      for (int j = 0; j < S::kFB; ++j) bias_acc[j] = sum8(g[j], bias_acc[j]);
                                    }
                                  },
                                  []() {},
                                  [&]() {
                                    if constexpr (kChain > 0)
                                      if (it % kChain == 0 && it)
#pragma unroll
                                        for (int y = 0; y < S::kFA; ++y)
#pragma unroll
                                          for (int j = 0; j < S::kFB; ++j) {
                                            chains[y][j] = it == kChain ? acc[y][j] : chains[y][j] + acc[y][j];
                                            acc[y][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                                          }
                                  });
  }
  if (S::kAlternate && group == 0) barrier_no_fence();
  if constexpr (kChain > 0)
    if (i_end - i_begin > kChain * S::kGroups)
#pragma unroll
      for (int i = 0; i < S::kFA; ++i)
#pragma unroll
        for (int j = 0; j < S::kFB; ++j) acc[i][j] += chains[i][j];
  f32x4 sum[S::kFA][S::kOutB];
  add_groups<S>(acc, sum, lds, group, wave, lane);

  const int r = lane & 15, quarter = lane >> 4;
  float bias_sum[S::kFB];   // of row 16 j + r, in group 0's wavefronts of the first columns
  if (a.want_bias && et == 0) {
    if (S::kGroups > 1) {  // the other group's column sums
      float* x = reinterpret_cast<float*>(lds);
      __syncthreads();
      if (do_bias && group)
#pragma unroll
        for (int j = 0; j < S::kFB; ++j) x[(wb * S::kFB + j) * 64 + lane] = bias_acc[j];
      __syncthreads();
      if (do_bias && !group)
#pragma unroll
        for (int j = 0; j < S::kFB; ++j) bias_acc[j] += x[(wb * S::kFB + j) * 64 + lane];
    }
#pragma unroll
    for (int j = 0; j < S::kFB; ++j) {
      bias_sum[j] = bias_acc[j] + __shfl_xor(bias_acc[j], 16, 64);
      bias_sum[j] += __shfl_xor(bias_sum[j], 32, 64);
    }
  }
  const bool has_bias = do_bias && !group;
  if constexpr (kMerge) {
    if (a.splits > 1) {
      // Ranges are added in pairs, pairs of pairs and so on: of two, the one that comes first leaves its registers
      // as they are ([wavefront][block][half][lane] pairs, in the place of its lowest range) and ends, the other adds
      // them to its own.  (One workgroup that adds all of them waits for 64 KB of far memory per range.)
      constexpr int kTile = S::kRowsA * S::kRowsB, kBlocks = S::kFA * S::kOutB;
      static_assert(kTile == S::kAllWaves * kBlocks * 256, "the registers are the tile");
      __shared__ int second;
      for (int level = 0; (1 << level) < a.splits; ++level) {
        const int node = split >> level, other = (node ^ 1) << level;
        if (other >= a.splits) continue;
        unsigned long long* const word = a.arrived + (size_t)tile * kMaxRanges + (kMaxRanges - (kMaxRanges >> level)) + (node >> 1);
        auto place = [&](int range) { return a.part + ((size_t)range * tiles + tile) * kTile + wave_id * kBlocks * 256 + lane * 2; };
        auto bias_place = [&](int range) { return a.part_bias + (size_t)range * a.F + f0 + wb * S::kFB * 16 + r; };
        if (tid == 0) second = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.ticket;
        __syncthreads();
        if (!second) {
          float* const mine = place(node << level);
#pragma unroll
          for (int y = 0; y < kBlocks; ++y)
#pragma unroll
            for (int h = 0; h < 2; ++h)
              put_pair<true>(mine + y * 256 + h * 128, sum[y / S::kOutB][y % S::kOutB][2 * h], sum[y / S::kOutB][y % S::kOutB][2 * h + 1]);
          if (has_bias && quarter == 0)
#pragma unroll
            for (int j = 0; j < S::kFB; ++j)
              __hip_atomic_store(bias_place(node << level) + j * 16, bias_sum[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          publish_partials();
          if (tid == 0) second = __hip_atomic_exchange(word, a.ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.ticket;
          __syncthreads();
          if (!second) return;
        }
        const float* const theirs = place(other);
        float2 v[kBlocks][2];
#pragma unroll
        for (int y = 0; y < kBlocks; ++y)
#pragma unroll
          for (int h = 0; h < 2; ++h) v[y][h] = get_pair<true>(theirs + y * 256 + h * 128);
#pragma unroll
        for (int y = 0; y < kBlocks; ++y) sum[y / S::kOutB][y % S::kOutB] += f32x4{v[y][0].x, v[y][0].y, v[y][1].x, v[y][1].y};
        if (has_bias)
#pragma unroll
          for (int j = 0; j < S::kFB; ++j)
            bias_sum[j] += __hip_atomic_load(bias_place(other) + j * 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // (cleared again, so that a captured launch, which is replayed with its old ticket, finds none of its own)
        if (tid == 0) __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();  // (everyone has looked at `second`)
      }
    }
  }
  const bool partial = !kMerge && a.splits > 1;
  // a lane holds columns 16 i + 4 quarter .. + 3 of row 16 j + r
  const ResultRows<kThrough> rows((partial ? a.part + (size_t)split * a.F * a.E : a.out) + (size_t)f0 * a.E);
#pragma unroll
  for (int j = 0; j < S::kOutB; ++j) {
    const int f = (wb * S::kFB + group * S::kOutB + j) * 16 + r;
#pragma unroll
    for (int i = 0; i < S::kFA; ++i) {
      const int e = e0 + (wa * S::kFA + i) * 16 + 4 * quarter;
      if (f < a.F - f0 && e < a.E) rows.store(((unsigned)f * a.E + e) * 4, __builtin_bit_cast(u32x4, sum[i][j]));
    }
  }
  if (has_bias) {
    float* bd = partial ? a.part_bias + (size_t)split * a.F : a.out_bias;
#pragma unroll
    for (int j = 0; j < S::kFB; ++j) {
      const int f = f0 + (wb * S::kFB + j) * 16 + r;
      if (quarter == 0 && f < a.F) bd[f] = bias_sum[j];
    }
  }
}
template <class S>
__global__ __launch_bounds__(S::kThreads, S::kAllWaves / 4 * S::kPerCU) void proj_wgrad_kernel(WgradArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  wgrad_tile<S, kMaxRange, 0, false, false>(a, lds, blockIdx.x);
}

// For a weight gradient that no product follows.
__global__ __launch_bounds__(256) void add_ranges_kernel(RangeSums s) { add_ranges(s, blockIdx.x, 256); }

//                         columns x rows of dW
using Wgrad256 = Shape<4, 4, 2, 4, 2, 1>;      // 256 x 256
using Wgrad128 = Shape<2, 2, 2, 2, 2, 1, 2>;   // 128 x 128, two groups

size_t align256(size_t n) { return (n + 255) & ~size_t(255); }
struct WgradPlan {
  int blocks_per_seq, splits, per_split, tile;
  double cost;
  size_t bias_off, total;
};
// F x E = shape of the weight gradient.
WgradPlan plan_wgrad(int B, int N, int F, int E) {
  WgradPlan p;
  p.blocks_per_seq = (N + 63) / 64;
  const int total_blocks = B * p.blocks_per_seq;
  // Large tiles read half as much per contraction, small ones need fewer token ranges to fill the chip, and
  // every range leaves an fp32 partial matrix that is written and read again.  In us, as measured on 768
  // and 1024 wide layers of 257 to 16384 tokens, one workgroup per CU: 1.9 a token block for 256 x 256, 0.7 for
  // 128 x 128 with two groups, 1 per 5.2 MB of partial sums.  (3072 x 1024 at 4096 tokens: 50 against 47,
  // at 8192 70 against 85, at 1024 37 against 19.)
  constexpr int kSlots = 256;
  for (int tile : {256, 128}) {
    const int tiles = ((F + tile - 1) / tile) * ((E + tile - 1) / tile);
    // enough workgroups for the chip, but ranges of at least eight token blocks
    const int want = std::max({1, std::min(std::max(1, kSlots / tiles), total_blocks / 8), (total_blocks + kMaxRange - 1) / kMaxRange});
    const int per = (total_blocks + want - 1) / want, splits = (total_blocks + per - 1) / per;
    const double rounds = (double)((tiles * splits + kSlots - 1) / kSlots);
    const double cost = rounds * per * (tile == 256 ? 1.9 : 0.7) + (splits > 1 ? splits * 8.0 * F * E / 5.2e6 : 0.0);
    if (tile == 256 || cost < p.cost) {
      p.cost = cost;
      p.tile = tile;
      p.per_split = per;
      p.splits = splits;
    }
  }
  p.bias_off = p.splits > 1 ? align256((size_t)p.splits * F * E * 4) : 0;
  p.total = p.bias_off + (p.splits > 1 ? align256((size_t)p.splits * F * 4) : 0) + 256;
  return p;
}

template <class S>
hipError_t launch_wgrad(const WgradArgs& a, int kernel_id, hipStream_t stream) {
  const int tiles = ((a.F + S::kRowsB - 1) / S::kRowsB) * ((a.E + S::kRowsA - 1) / S::kRowsA);
  const hipError_t e = allow_lds<&proj_wgrad_kernel<S>>(S::kLds);
  if (e != hipSuccess) return e;
  ProfileScope prof(kernel_id, stream);
  hipLaunchKernelGGL(proj_wgrad_kernel<S>, dim3(8 * ((tiles * a.splits + 7) / 8)), dim3(S::kThreads), S::kLds, stream, a);
  return hipGetLastError();
}

// Leaves in `sums` what is still to be added up.
hipError_t run_wgrad(WgradArgs a, const WgradPlan& p, char* ws, int kernel_id, RangeSums& sums, hipStream_t stream) {
  a.blocks_per_seq = p.blocks_per_seq;
  a.splits = p.splits;
  a.per_split = p.per_split;
  a.part = reinterpret_cast<float*>(ws);
  a.part_bias = reinterpret_cast<float*>(ws + p.bias_off);
  sums = {};
  if (p.splits > 1) sums = {a.part, a.part_bias, a.out, a.out_bias, (size_t)a.F * a.E, a.F, p.splits, 0};
  return p.tile == 256 ? launch_wgrad<Wgrad256>(a, kernel_id, stream) : launch_wgrad<Wgrad128>(a, kernel_id, stream);
}
hipError_t add_ranges_alone(RangeSums s, hipStream_t stream) {
  if (!s.splits) return hipSuccess;
  s.blocks = (int)std::max<size_t>(1, std::min<size_t>(1024, s.n / 4 / 256));
  hipLaunchKernelGGL(add_ranges_kernel, dim3(s.blocks), dim3(256), 0, stream, s);
  return hipGetLastError();
}

// ---- both gradients of a projection in one launch ------------------------------------------------------------
// A small layer's gradients are two launches that leave compute units idle (dW 2304 x 768 has 108 tiles, dX at 8 x 512
// tokens 192), and partial sums that the second has to read.  Here the tiles of dW go first, each over all token
// blocks or a few ranges of them, and those of the other gradient take the units that are left; ranges are added by
// the workgroups themselves.
constexpr int kOneLaunchBlocks = 160;  // token blocks, at most (beyond, two launches are as fast)
// The shortest ranges of two launches give each group four blocks; with chains of that length the error of dW (rms
// against 64 bits, of its own rms) is 0.7e-7 to 1.1e-7 where it was up to 2.1e-7, and would be up to 3.4e-7 without.
// Adding them up after the multiplication cost 8 % of a long range, while the next fragments travel half of that.
constexpr int kOneLaunchChain = 4;
template <class S, bool kHeadTok>
__global__ __launch_bounds__(S::kThreads, S::kAllWaves / 4) void proj_bwd_kernel(WgradArgs w, ProjArgs a, int w_blocks) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  static_assert(S::kThreads == Wgrad128::kThreads, "one workgroup size for both");
  if ((int)blockIdx.x < w_blocks) wgrad_tile<Wgrad128, kOneLaunchBlocks, kOneLaunchChain, true, true>(w, lds, blockIdx.x);
  else {
    int x;
    const int y = uniform_div(blockIdx.x - w_blocks, a.deal.grid_x(), x);
    dealt_product<S, kHeadTok, true, true>(a, a, lds, x, y);
  }
}

// The product's tiles there, eight wavefronts each.  Those of one group and those of two add up a product's stages in
// different orders; which of them, is as for the product alone, so that it comes in the same bits from either.
using Both256 = Proj256;
using Both128 = Shape<4, 2, 4, 2, 2, 1>;   // 256 x 128
using Both128x2 = Proj128x2;
using Both64x2 = Proj64x2;

int wgrad_tiles128(int F, int E) { return (F + 127) / 128 * ((E + 127) / 128); }

// When the last of `first` workgroups of t1 us and then `second` ones of t2 us ends, one at a time on each unit.
double end_of_both(int first, double t1, long second, double t2) {
  constexpr int kUnits = 256;
  const int late = first % kUnits, early = kUnits - late;   // units that end the first kind a round later, or not
  double early_at = first / kUnits * t1, late_at = early_at + t1, end = late ? late_at : early_at;
  while (second > 0) {
    const bool use_early = !late || early_at <= late_at;
    double& at = use_early ? early_at : late_at;
    at += t2;
    second -= use_early ? early : late;
    end = std::max(end, at);
  }
  return end;
}

struct BwdPlan {
  double cost;       // us
  double wgrad;      // of that, until dW is there
  int ranges;        // of token blocks; 0: not in one launch
  bool large;        // the larger or the smaller tiles of the product
  size_t bias_off, words_off, total;
};
template <class S>
void offer_bwd(BwdPlan& best, ProjArgs a, bool large, int tiles, int blocks, int ranges, double per_step, double rest) {
  deal_tiles<S>(a);
  const int first = (tiles * ranges + 7) / 8 * 8, per_range = (blocks + ranges - 1) / ranges;
  double t1 = (0.44 + 0.12 * std::min(1.0, first / 256.0)) * per_range + 5.1;
  for (int r = 1; r < ranges; r *= 2) t1 += 2.7;   // one addition of pairs
  // (padding, which this leaves out, shortens long ranges most: several must be worth 16 %)
  const double cost = (ranges > 1 ? 1.16 : 1.0) * (4.4 + end_of_both(first, t1, a.deal.tokens * a.deal.features, per_step * (a.K / 64) + rest));
  if (cost < best.cost) {
    best.cost = cost;
    best.wgrad = t1;
    best.ranges = ranges;
    best.large = large;
  }
}
// Where the partial sums of dW's ranges lie in the workspace, for `tiles` tiles of dW.
void lay_out(BwdPlan& p, const WgradArgs& w, int ranges, int tiles) {
  p.bias_off = align256((size_t)ranges * w.F * w.E * 4);
  p.words_off = p.bias_off + align256((size_t)ranges * w.F * 4);
  p.total = p.words_off + (size_t)tiles * kMaxRanges * 8 + 16;   // (the caller's address may be any)
}
void place_ranges(WgradArgs& w, const BwdPlan& p, char* ws) {
  ws += -reinterpret_cast<uintptr_t>(ws) & 15;
  w.blocks_per_seq = (w.N + 63) / 64;
  w.splits = p.ranges;
  w.per_split = w.B * w.blocks_per_seq;
  w.part = reinterpret_cast<float*>(ws);
  w.part_bias = reinterpret_cast<float*>(ws + p.bias_off);
  w.arrived = reinterpret_cast<unsigned long long*>(ws + p.words_off);
}
// `groups`: of the product's shape if it were alone; `room`: bytes of the workspace, which are those that two launches need.
BwdPlan plan_bwd(const WgradArgs& w, const ProjArgs& a, int groups, size_t room) {
  BwdPlan p = {1e30, 0, 0, false, 0, 0, 0};
  const int tiles = wgrad_tiles128(w.F, w.E), blocks = w.B * ((w.N + 63) / 64);
  // (Ranges that are added in the launch leave whole tiles and whole tiles' bias rows in space for F x E and F values: see
  // wgrad_tile.  The callers allow no other sizes today.)
  if (blocks > kOneLaunchBlocks || w.F % Wgrad128::kRowsB || w.E % Wgrad128::kRowsA) return p;
  for (int ranges = 1; ranges <= kMaxRanges && tiles * ranges <= 256 && (ranges == 1 || blocks >= 8 * ranges); ++ranges) {
    lay_out(p, w, ranges, tiles);
    if (ranges > 1 && p.total > room) break;
    if (groups == 2) {
      offer_bwd<Both128x2>(p, a, true, tiles, blocks, ranges, 0.38, 3.1);
      offer_bwd<Both64x2>(p, a, false, tiles, blocks, ranges, 0.35, 1.8);
    } else {
      offer_bwd<Both256>(p, a, true, tiles, blocks, ranges, 1.3, 5.3);
      offer_bwd<Both128>(p, a, false, tiles, blocks, ranges, 0.75, 5.0);
    }
  }
  lay_out(p, w, p.ranges, tiles);
  return p;
}

template <class S, bool kHeadTok>
hipError_t launch_bwd(WgradArgs w, ProjArgs a, const BwdPlan& p, char* ws, int wgrad_id, int proj_id, hipStream_t stream) {
  deal_tiles<S>(a);
  a.lazy_tiles = lazy_tiles<S, true>(a);
  place_ranges(w, p, ws);
  const int w_blocks = (wgrad_tiles128(w.F, w.E) * p.ranges + 7) / 8 * 8;  // (whole rounds of XCDs, so the products' tiles are dealt as ever)
  constexpr int kLds = std::max(S::kLds, Wgrad128::kLds);
  const hipError_t e = allow_lds<&proj_bwd_kernel<S, kHeadTok>>(kLds);
  if (e != hipSuccess) return e;
  ProfileScope prof(wgrad_id, stream, proj_id);
  hipLaunchKernelGGL((proj_bwd_kernel<S, kHeadTok>), dim3(w_blocks + a.deal.grid_x() * a.deal.grid_y()), dim3(S::kThreads), kLds, stream, w, a, w_blocks);
  return hipGetLastError();
}

// dW alone, in the same bits: the same ranges, groups and chains for each element, in tiles small enough that
// they spread over the chip, which no product fills.  The smallest tile whose workgroups are one round; us for 128 x 128 (as
// beside a product), 128 x 64 and 64 x 64: 512 wide, 512 tokens 11.1, 8.6, 8.1, 2048 tokens in two ranges 19.8, 15.6,
// 15.6; 768 wide, 512 tokens 11.6, 9.5, 10.4, 8 x 512 36.4, 29.1, 30.1; with more than 128 workgroups of 128 x 128, 16 to
// 64 blocks each, 23.2, 34.0, 36.2.
using Wgrad64 = Shape<2, 1, 2, 2, 2, 1, 2>;
using Wgrad64x64 = Shape<1, 1, 2, 2, 2, 1, 2>;
template <class S, bool kThrough>
__global__ __launch_bounds__(S::kThreads, S::kAllWaves / 4 * S::kPerCU) void proj_wgrad_alone_kernel(WgradArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  wgrad_tile<S, kOneLaunchBlocks, kOneLaunchChain, true, kThrough>(a, lds, blockIdx.x);
}
// kThrough: dW of more than 1 MB (us, left and through: 256 x 256 at 47 tokens 6.45 and 6.65, 512 x 512 at 2 x 101 6.5 and 6.65; of 240 sizes
// up to 0.7 MB take 1.5 % longer through, 0.75 to 1 MB 1 %, 1.1 to 2 MB 0.3 % less, 2.2 to 3 MB 1.7 %, 4.5 to 9 MB 5 %; beside a product there
// is no difference up to 1 MB).
template <class S, bool kThrough>
hipError_t launch_wgrad_alone(WgradArgs w, const BwdPlan& p, char* ws, int kernel_id, hipStream_t stream) {
  place_ranges(w, p, ws);
  const hipError_t e = allow_lds<&proj_wgrad_alone_kernel<S, kThrough>>(S::kLds);
  if (e != hipSuccess) return e;
  const int tiles = ((w.F + S::kRowsB - 1) / S::kRowsB) * ((w.E + S::kRowsA - 1) / S::kRowsA);
  ProfileScope prof(kernel_id, stream);
  hipLaunchKernelGGL((proj_wgrad_alone_kernel<S, kThrough>), dim3((tiles * p.ranges + 7) / 8 * 8), dim3(S::kThreads), S::kLds, stream, w);
  return hipGetLastError();
}
hipError_t run_wgrad_alone(const WgradArgs& w, BwdPlan p, char* ws, size_t room, int kernel_id, hipStream_t stream) {
  const int tiles = wgrad_tiles128(w.F, w.E);
  int cut = 4;   // tiles made of one
  for (;; cut /= 2) {
    lay_out(p, w, p.ranges, tiles * cut);
    if (cut == 1 || (tiles * p.ranges * cut <= 256 && (p.ranges == 1 || p.total <= room))) break;
  }
  const auto run = [&](auto through) {
    constexpr bool kThrough = decltype(through)::value;
    const auto launch = cut == 4   ? launch_wgrad_alone<Wgrad64x64, kThrough>
                        : cut == 2 ? launch_wgrad_alone<Wgrad64, kThrough>
                                   : launch_wgrad_alone<Wgrad128, kThrough>;
    return launch(w, p, ws, kernel_id, stream);
  };
  return (size_t)w.F * w.E > (256u << 10) ? run(std::true_type()) : run(std::false_type());
}

// dW (unless w.out is null) and the other gradient (unless a.out[0] is).  One launch if these costs say that it is
// faster.  They were fitted to 130 pairs of gradients (64 to 16384 tokens, 256 to 1536 wide) in up to fifteen forms;
// over them the rule gained 16 %, lost 5 % at most and was 1.5 % behind the best form of each.  Over 1800 pairs of up to 40000 tokens, with the
// present deal of tiles, what it takes is 0.2 % behind the better of two launches and the best one launch in the mean, 16 % at most (1536 wide at
// 2453 tokens 43.6 and 50.2).  us, as two launches and
// as one, gradients of QKV and of the output projection, 768 wide: 512 tokens 27.1 -> 16.8 and 17.8 -> 11.1, 2048 tokens
// 32.5 -> 23.5 and 22.4 -> 18.7, 8 x 512 44 -> 39.5 and 26.4 -> 23.0, 3 x 1999 64 -> 53.5 and 32 -> 27;
// 1024 wide, 1024 tokens 35.8 -> 25 and 22.9 -> 15.3, 8 x 512 61 -> 60.5 and 35 -> 27.5.
// dW alone follows the same rule up to kSameBits token blocks, so that it is the same bits whether or not the other gradient
// is wanted (us, as two launches and as one: 512 tokens 11.1 -> 9.5 and 10.6 -> 7.8, 2048 tokens 23.0 -> 18.2 and 18.3 ->
// 14.9, 8 x 512 27 -> 29.1 and 22.3 -> 18.8; at worst, 512 wide with 8 heads at 13 x 134, 18.8 -> 22.6, where both gradients are 24.3 ->
// 22.1).  Beyond, the form that is
// faster beside a product can take 1.2 times as long without one (768 wide, 15 x 512 39 -> 48.3), and dW alone has two
// unless its tiles of 128 x 128 nearly fill the chip (1024 wide, 3 x 1999 58.2 -> 53.6).
constexpr int kSameBits = 64;
template <bool kHeadTok>
hipError_t run_bwd(const WgradArgs& w, ProjArgs a, char* ws, int wgrad_id, int proj_id, hipStream_t stream) {
  const WgradPlan alone = plan_wgrad(w.B, w.N, w.F, w.E);
  const ProjChoice product = choose_proj<kHeadTok, true>(a);
  const BwdPlan both = plan_bwd(w, a, product.groups, alone.total);
  const bool want_w = w.out, want_a = a.out[0];
  const bool same = want_a || w.B * ((w.N + 63) / 64) <= kSameBits ||
                    (wgrad_tiles128(w.F, w.E) * both.ranges > 128 && both.wgrad + 3 < alone.cost);
  if (want_w && same && both.cost < 13.4 + 0.66 * alone.cost + 0.88 * product.cost) {
    if (!want_a) return run_wgrad_alone(w, both, ws, alone.total, wgrad_id, stream);
    const auto launch = product.groups == 2 ? (both.large ? launch_bwd<Both128x2, kHeadTok> : launch_bwd<Both64x2, kHeadTok>)
                                            : (both.large ? launch_bwd<Both256, kHeadTok> : launch_bwd<Both128, kHeadTok>);
    return launch(w, a, both, ws, wgrad_id, proj_id, stream);
  }
  if (want_w) {
    const hipError_t e = run_wgrad(w, alone, ws, wgrad_id, a.ranges, stream);
    if (e != hipSuccess) return e;
  }
  return want_a ? product.launch(a, proj_id, stream) : add_ranges_alone(a.ranges, stream);
}

}  // namespace

hipError_t launch_qkv_project(const void* x, const void* w_qkv, const float* bias,
                              const unsigned char* flags, int B, int N, int H, int E, void* q,
                              void* k, void* v, hipStream_t stream) {
  ProjArgs a = {};
  a.w = static_cast<const unsigned short*>(w_qkv);
  a.tok = static_cast<const unsigned short*>(x);
  a.bias = bias;
  a.flags = flags;
  a.out[0] = static_cast<unsigned short*>(q);
  a.out[1] = static_cast<unsigned short*>(k);
  a.out[2] = static_cast<unsigned short*>(v);
  a.B = B; a.N = N; a.H = H;
  a.F = 3 * H * kD;
  a.K = E;
  return choose_proj<false, false>(a).launch(a, 8, stream);
}

hipError_t launch_out_project(const void* o, const void* w_o, const float* bias,
                              const unsigned char* flags, int B, int N, int H, int E, void* y,
                              hipStream_t stream) {
  ProjArgs a = {};
  a.w = static_cast<const unsigned short*>(w_o);
  a.tok3[0] = static_cast<const unsigned short*>(o);
  a.bias = bias;
  a.flags = flags;
  a.out[0] = static_cast<unsigned short*>(y);
  a.B = B; a.N = N; a.H = H;
  a.F = E;
  a.K = H * kD;
  return choose_proj<true, false>(a).launch(a, 9, stream);
}

namespace {
// The sizes of both gradients: dW [F][E] and the product over K.
void bwd_sizes(WgradArgs& w, ProjArgs& a, int B, int N, int H, int F, int E, int features, int K) {
  w = {};
  a = {};
  w.B = a.B = B; w.N = a.N = N; w.H = a.H = H;
  w.F = F; w.E = E;
  a.F = features; a.K = K;
}
void qkv_bwd_sizes(WgradArgs& w, ProjArgs& a, int B, int N, int H, int E) { bwd_sizes(w, a, B, N, H, 3 * H * kD, E, E, 3 * H * kD); }
void out_bwd_sizes(WgradArgs& w, ProjArgs& a, int B, int N, int H, int E) { bwd_sizes(w, a, B, N, H, E, H * kD, H * kD, E); }
}  // namespace

size_t qkv_project_bwd_workspace(int B, int N, int H, int E) { return plan_wgrad(B, N, 3 * H * kD, E).total; }
size_t out_project_bwd_workspace(int B, int N, int H, int E) { return plan_wgrad(B, N, E, H * kD).total; }

hipError_t launch_qkv_project_bwd(const void* x, const void* w_qkv, const unsigned char* flags,
                                  const void* dq, const void* dk, const void* dv, int B, int N, int H,
                                  int E, void* dx, float* dw, float* dbias, void* workspace,
                                  unsigned long long ticket, hipStream_t stream) {
  WgradArgs g;
  ProjArgs a;
  qkv_bwd_sizes(g, a, B, N, H, E);
  g.g.p[0] = static_cast<const unsigned short*>(dq);
  g.g.p[1] = static_cast<const unsigned short*>(dk);
  g.g.p[2] = static_cast<const unsigned short*>(dv);
  g.g.heads = 1;
  g.x.p[0] = static_cast<const unsigned short*>(x);
  g.x.heads = 0;
  g.x.ld = E;
  g.flags = flags;
  g.out = dw;
  g.out_bias = dbias;
  g.want_bias = dbias != nullptr;
  g.ticket = ticket;
  // dx[tok, :] = sum over the 3 H heads of dq, dk, dv [tok, head] . w_qkv[head rows, :]
  a.w = static_cast<const unsigned short*>(w_qkv);  // [F][E], contracted over its rows
  a.tok3[0] = static_cast<const unsigned short*>(dq);
  a.tok3[1] = static_cast<const unsigned short*>(dk);
  a.tok3[2] = static_cast<const unsigned short*>(dv);
  a.flags = flags;
  a.out[0] = static_cast<unsigned short*>(dx);
  return run_bwd<true>(g, a, static_cast<char*>(workspace), 11, 10, stream);
}

hipError_t launch_out_project_bwd(const void* o, const void* w_o, const unsigned char* flags,
                                  const void* dy, int B, int N, int H, int E, void* d_o, float* dw,
                                  float* dbias, void* workspace, unsigned long long ticket, hipStream_t stream) {
  WgradArgs g;
  ProjArgs a;
  out_bwd_sizes(g, a, B, N, H, E);
  g.g.p[0] = static_cast<const unsigned short*>(dy);
  g.g.heads = 0;
  g.g.ld = E;
  g.x.p[0] = static_cast<const unsigned short*>(o);
  g.x.heads = 1;
  g.flags = flags;
  g.out = dw;
  g.out_bias = dbias;
  g.want_bias = dbias != nullptr;
  g.ticket = ticket;
  // d_o[tok, head i] = dy[tok, :] . w_o[:, head i columns], written head by head
  a.w = static_cast<const unsigned short*>(w_o);  // [E][H*64], contracted over its rows
  a.tok = static_cast<const unsigned short*>(dy);
  a.flags = flags;
  a.out[0] = static_cast<unsigned short*>(d_o);
  return run_bwd<false>(g, a, static_cast<char*>(workspace), 13, 12, stream);
}

}  // namespace mate
