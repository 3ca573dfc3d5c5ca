// fp32 MATE attention on the matrix cores (v_mfma_f32_32x32x2_f32: exact fp32 products, fp32
// accumulation): the path for dtype f32, forward and backward.
//
// Same pattern, tables and work units as the bf16 kernels (stream_plan.h), other proportions: the
// fp32 matrix instruction does 1/16 of the bf16 one's work per cycle (150 TFLOP/s measured), so a
// 32 x 32 block of scores costs 2048 cycles of matrix pipe per contraction and everything else --
// loads, softmax, masks -- hides behind it.  So no shared tiles and no barriers in the loop: a
// workgroup owns 32 rows (a quarter of a unit), its four wavefronts take every fourth 32-row tile of
// the other side, each through LDS of its own, and their results are added in LDS at the end.
// Small units also mean that a batch of short sequences fills the chip.
//
// A tile is loaded in whole rows (16 lanes x 16 bytes), one tile ahead, into registers and passes
// through LDS into operand order.  Operands loaded straight from global memory (16 bytes of 64
// different rows per instruction) touched four times as many cache lines per instruction, and the
// first tiles of a launch took 10 us to arrive.
//
// Measured (training step of 4 sequences of 512 tokens, 12 heads: tables, forward, dQ, dK/dV):
// 90 us, 1390 us with one wavefront per query and dot products on the vector ALU.  Kernels 23, 28 and
// 34 us: question-token owners (four tiles per wavefront) end last, the rest is over after 20 us.
//
// Operand layout of the instruction: lane l = 32 hl + m holds row (A) or column (B) m at k = hl; the
// C tile is that of the bf16 instruction.  The order of a contraction is free:
//   over dims      lane half hl takes dims 8 j + 4 hl + e: 16-byte loads, 32 contiguous bytes per row
//   over tile rows step c pairs rows c_row(c, 0) and c_row(c, 1): the B operand is C register c itself
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

typedef float f32x4 __attribute__((ext_vector_type(4)));  // (arrays of HIP's float4 class end up in scratch memory)

__device__ __forceinline__ f32x16 mfma1(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// LDS tiles: 32 rows of 64 floats and a pad of 4, which spreads row accesses (16 bytes of 16 rows at
// once) over the 64 banks; column reads (rows r and r + 4 at once) overlap in a quarter of them, which
// the matrix pipe hides.  The pad of an owned tile keeps the row's token and its delta.  (An XOR
// swizzle needs no pad, but its addresses are not base + constant: 30 registers more, and spills.)
constexpr int kStride = kD + 4;
constexpr int kTileFloats = kRows * kStride;
constexpr int kTokAt = kD, kDeltaAt = kD + 1;

// A lane's window of the tile's rows.  (Compared per pair: the matrix pipe bounds these kernels, and their registers are
// full.)
struct SlotWindow {
  int d0, len;  // the tile's first slot + 4 hl - the window's, and its length
  __device__ __forceinline__ bool in(int c) const { return (unsigned)(d0 + 8 * (c >> 2) + (c & 3)) < (unsigned)len; }
  // tile row `row`, whichever lane half holds its score
  __device__ __forceinline__ bool meets(int row, int hl) const { return (unsigned)(d0 - 4 * hl + row) < (unsigned)len; }
};

// A tile on its way from global memory: lane l holds piece l % 16 of rows l / 16 + 4 i.
struct TileRegs {
  f32x4 v[8];
  // `tok`: lanes m and m + 32 hold the token of tile row m
  __device__ __forceinline__ void load(const float* X, int tok, int lane) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      v[i] = *reinterpret_cast<const f32x4*>(X + (unsigned)__shfl(tok, (lane >> 4) + 4 * i, 64) * kD + 4 * (lane & 15));
  }
  __device__ __forceinline__ void put(float* tile, int lane) const {
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<f32x4*>(tile + ((lane >> 4) + 4 * i) * kStride + 4 * (lane & 15)) = v[i];
  }
};
// The owned rows of a tensor into an LDS tile: every wavefront brings eight of them.
__device__ __forceinline__ void put_owned(float* tile, const float* X, int pos, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = 8 * wave + 4 * i + (lane >> 4);
    *reinterpret_cast<f32x4*>(tile + row * kStride + 4 * (lane & 15)) =
        *reinterpret_cast<const f32x4*>(X + (unsigned)__shfl(pos, row, 64) * kD + 4 * (lane & 15));
  }
}

// Over dims: row m of the wavefront's tile and of an owned one.
__device__ __forceinline__ f32x16 contract(const float* a_tile, const float* b_tile, int m, int hl, f32x16 c) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(a_tile + m * kStride + 8 * j + 4 * hl);
    const f32x4 b = *reinterpret_cast<const f32x4*>(b_tile + m * kStride + 8 * j + 4 * hl);
#pragma unroll
    for (int e = 0; e < 4; ++e) c = mfma1(a[e], b[e], c);
  }
  return c;
}
__device__ __forceinline__ f32x16 contract(const float* a_tile, const f32x4 (&b)[8], int m, int hl, f32x16 c) {
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

// The same for a tile that may hold an infinity or a NaN.  The matrix instruction multiplies every weight with
// every row, and 0 x Inf is NaN: such a row would reach the owned rows that do not meet it.  So these rows
// go through the vector ALU, owned rows that meet them only, and are cleared for the matrix instruction.
// In the main loops this would take 30 to 40 registers that are not there; a wavefront whose results are
// not all finite when its loop ends does its tiles again this way, without a prefetch.  (Looking for such values
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
__device__ inline bool take_quarter(const AttnArgs& a, Quarter& q) {
  q.sub = ((blockIdx.x >> 3) + (blockIdx.x >> 5)) & 3;
  q.turn = blockIdx.x >> 5;
  if (!take_unit<false, false>(a, ((blockIdx.x >> 5) << 3) | (blockIdx.x & 7), q.w)) return false;
  const UnitPlan& u = q.w.u;
  if (u.kind == UNIT_PAD) return true;
  // (a chunked question-token owner: its first unit streams everything, there are no partials here)
  if (u.part >= 0 && u.t_begin != 0) return false;
  if (u.t0 + kRows * q.sub >= u.own_count) return false;
  // Question-token owners stream the whole sequence and end last: they go first on a shared SIMD
  // (their tiles took 7.8 us each beside two other wavefronts, 2.6 us of it their own).
  if (u.kind == UNIT_GLOBAL) __builtin_amdgcn_s_setprio(3);
  return true;
}

// The owned row of a lane and the tiles its workgroup streams.
struct Rows {
  int pos, lo, hi;         // token of row m, its window of table slots
  bool valid;
  const int *gidx, *list;  // question tokens [0, G), then slots [s_lo, s_hi) of list
  int G, s_lo, s_hi, nG, n;
  __device__ __forceinline__ Rows(const AttnArgs& a, const Quarter& q, int m) {
    const UnitPlan& u = q.w.u;
    const int b = q.w.b, first = u.t0 + kRows * q.sub, slot = min(first + m, u.own_count - 1);
    valid = first + m < u.own_count;
    pos = u.own_list[slot];
    lo = 0;
    hi = u.L;
    if (u.kind == UNIT_LOCAL) {
      const int2 g = a.seg.slot_rng[q.w.view][(size_t)b * a.N + slot];
      lo = g.x;
      hi = g.y;
    }
    gidx = a.seg.global_idx + (size_t)b * a.N;
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

// Sum of the four wavefronts' accumulators, stored as whole rows: lane m's column is owned row m.
// `lds` = the wavefronts' tiles, `own` = the owned tile that keeps the rows' tokens.
__device__ __forceinline__ void store_sum(const f32x16 (&acc)[2], float mul, float* lds, const float* own, float* out,
                                          int wave, int m, int hl) {
  float* mine = lds + wave * kTileFloats;
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
    const int row = (threadIdx.x >> 4) + 16 * i, piece = threadIdx.x & 15, tok = __float_as_int(own[row * kStride + kTokAt]);
    f32x4 s = *reinterpret_cast<const f32x4*>(lds + row * kStride + 4 * piece);
#pragma unroll
    for (int w = 1; w < kWaves; ++w) s += *reinterpret_cast<const f32x4*>(lds + w * kTileFloats + row * kStride + 4 * piece);
    if (tok >= 0) *reinterpret_cast<f32x4*>(out + (size_t)tok * kD + 4 * piece) = s;
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
          *reinterpret_cast<float4*>(out[x] + (size_t)tok[i] * kD + 4 * piece) = make_float4(0.f, 0.f, 0.f, 0.f);
        if (per_row && piece == 0) per_row[tok[i]] = 0.f;
      }
  }
}

// ======================================================================================
// forward
// ======================================================================================
__global__ __launch_bounds__(kThreads, 3) void fwd_f32_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) float lds[kWaves * kTileFloats], own[kTileFloats];
  __shared__ float2 stat[kWaves][kRows];
  Quarter q;
  if (!take_quarter(a, q)) return;
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
  const Rows r(a, q, m);
  if (tid < kRows) own[tid * kStride + kTokAt] = __int_as_float(r.valid ? r.pos : -1);
  const int t0 = (wave + q.turn) & (kWaves - 1);
  int tok = r.token(t0, m), tok_next = r.token(t0 + kWaves, m);
  TileRegs key, val;
  key.load(K, tok, lane);
  put_owned(own, Q, r.pos, wave, lane);
  val.load(V, tok, lane);
  keep_order();
  __syncthreads();
  float* tile = lds + wave * kTileFloats;

  const float sc = a.scale * kLog2e;  // scores are kept raw; exp2(s sc - m sc)
  f32x16 o[2] = {zero16(), zero16()};
  float m_run = -INFINITY, l_run = 0.f;
  // S^T -> P^T of a tile, O and the row sum rescaled
  auto probs = [&](f32x16& s, const SlotWindow& mask) {
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
    }
  };
  for (int t = t0; t < r.n; t += kWaves) {
    const int tok_after = r.token(t + 2 * kWaves, m);
    key.put(tile, lane);
    key.load(K, tok_next, lane);                          // the next tile's keys land during this one
    keep_order();
    f32x16 s = contract(tile, own, m, hl, zero16());      // S^T = K Q^T
    val.put(tile, lane);                                  // (the keys have been read)
    val.load(V, tok_next, lane);
    keep_order();
    probs(s, r.mask(t, hl));
    accumulate(o, tile, m, hl, s);                        // O^T += V^T P^T
    tok_next = tok_after;
  }
  if (__builtin_expect(any_special(o), 0)) {
    o[0] = o[1] = zero16();
    m_run = -INFINITY;
    l_run = 0.f;
    for (int t = t0; t < r.n; t += kWaves) {
      tok = r.token(t, m);
      key.load(K, tok, lane);
      key.put(tile, lane);
      f32x16 s = contract(tile, own, m, hl, zero16());
      val.load(V, tok, lane);
      val.put(tile, lane);
      const SlotWindow mask = r.mask(t, hl);
      probs(s, mask);
      accumulate_special(o, tile, m, hl, s, mask);
    }
  }
  // the wavefronts' maxima and sums, then their sum of O scaled to the common maximum
  const float l_tot = half_sum(l_run);
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
  const float mul = weight(m_run, m_all) / l_all;
  store_sum(o, mul, lds, own, O, wave, m, hl);
}

// ======================================================================================
// dQ, and delta = rowsum(dO * O) for the dK/dV kernel
// ======================================================================================
__global__ __launch_bounds__(kThreads, 3) void bwd_dq_f32_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) float lds[kWaves * kTileFloats], own_q[kTileFloats], own_g[kTileFloats];
  Quarter q;
  if (!take_quarter(a, q)) return;
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, hl = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t bh = (size_t)q.w.bh * a.N;
  const float* Q = static_cast<const float*>(a.q) + bh * kD;
  const float* K = static_cast<const float*>(a.k) + bh * kD;
  const float* V = static_cast<const float*>(a.v) + bh * kD;
  const float* O = static_cast<const float*>(a.o) + bh * kD;
  const float* dO = static_cast<const float*>(a.dout) + bh * kD;
  float* dQ = static_cast<float*>(a.dq) + bh * kD;
  if (q.w.u.kind == UNIT_PAD) {
    float* const outs[1] = {dQ};
    zero_pads<1>(q, outs, nullptr);
    return;
  }
  const Rows r(a, q, m);
  if (tid < kRows) own_q[tid * kStride + kTokAt] = __int_as_float(r.valid ? r.pos : -1);
  const int t0 = (wave + q.turn) & (kWaves - 1);
  int tok = r.token(t0, m), tok_next = r.token(t0 + kWaves, m);
  const float lse2 = a.lse[bh + r.pos] * kLog2e, sc = a.scale * kLog2e;
  TileRegs key, val;
  val.load(V, tok, lane);
  {  // owned Q and dO rows to LDS; delta of the eight rows this wavefront brings, 16 lanes per row
    f32x4 g[2], o[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned off = (unsigned)__shfl(r.pos, 8 * wave + 4 * i + (lane >> 4), 64) * kD + 4 * (lane & 15);
      g[i] = *reinterpret_cast<const f32x4*>(dO + off);
      o[i] = *reinterpret_cast<const f32x4*>(O + off);
    }
    put_owned(own_q, Q, r.pos, wave, lane);
    key.load(K, tok, lane);
    keep_order();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = 8 * wave + 4 * i + (lane >> 4);
      *reinterpret_cast<f32x4*>(own_g + row * kStride + 4 * (lane & 15)) = g[i];
      float d = g[i].x * o[i].x + g[i].y * o[i].y + g[i].z * o[i].z + g[i].w * o[i].w;
#pragma unroll
      for (int x = 8; x >= 1; x >>= 1) d += __shfl_xor(d, x, 64);
      if ((lane & 15) == 0) own_g[row * kStride + kDeltaAt] = d;
    }
  }
  __syncthreads();
  const float delta = own_g[m * kStride + kDeltaAt];
  if (wave == 0 && hl == 0 && r.valid) a.delta[bh + r.pos] = delta;
  float* tile = lds + wave * kTileFloats;

  f32x16 dq[2] = {zero16(), zero16()};
  auto dscores = [&](f32x16& s, const f32x16& dp, const SlotWindow& mask) {  // S^T -> dS^T
#pragma unroll
    for (int c = 0; c < 16; ++c)
      s[c] = mask.in(c) ? __builtin_amdgcn_exp2f(fmaf(s[c], sc, -lse2)) * (dp[c] - delta) : 0.f;
  };
  for (int t = t0; t < r.n; t += kWaves) {
    const int tok_after = r.token(t + 2 * kWaves, m);
    val.put(tile, lane);
    val.load(V, tok_next, lane);
    keep_order();
    const f32x16 dp = contract(tile, own_g, m, hl, zero16());  // dP^T = V dO^T
    key.put(tile, lane);
    key.load(K, tok_next, lane);
    keep_order();
    f32x16 s = contract(tile, own_q, m, hl, zero16());         // S^T  = K Q^T
    dscores(s, dp, r.mask(t, hl));
    accumulate(dq, tile, m, hl, s);                            // dQ^T += K^T dS^T
    tok_next = tok_after;
  }
  if (__builtin_expect(any_special(dq), 0)) {
    dq[0] = dq[1] = zero16();
    for (int t = t0; t < r.n; t += kWaves) {
      tok = r.token(t, m);
      val.load(V, tok, lane);
      val.put(tile, lane);
      keep_order();
      const f32x16 dp = contract(tile, own_g, m, hl, zero16());
      keep_order();
      key.load(K, tok, lane);
      key.put(tile, lane);
      keep_order();
      f32x16 s = contract(tile, own_q, m, hl, zero16());
      const SlotWindow mask = r.mask(t, hl);
      dscores(s, dp, mask);
      accumulate_special(dq, tile, m, hl, s, mask);
    }
  }
  __syncthreads();
  store_sum(dq, a.scale, lds, own_q, dQ, wave, m, hl);
}

// ======================================================================================
// dK, dV: the owned rows are keys, the streamed ones the queries that see them (the same lists and
// windows as in the forward, read the other way round)
// ======================================================================================
__global__ __launch_bounds__(kThreads, 2) void bwd_dkv_f32_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) float lds[2 * kWaves * kTileFloats];
  __shared__ __attribute__((aligned(16))) float own_k[kTileFloats];
  Quarter q;
  if (!take_quarter(a, q)) return;
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, hl = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t bh = (size_t)q.w.bh * a.N;
  const float* Q = static_cast<const float*>(a.q) + bh * kD;
  const float* K = static_cast<const float*>(a.k) + bh * kD;
  const float* V = static_cast<const float*>(a.v) + bh * kD;
  const float* dO = static_cast<const float*>(a.dout) + bh * kD;
  float* dK = static_cast<float*>(a.dk) + bh * kD;
  float* dV = static_cast<float*>(a.dv) + bh * kD;
  if (q.w.u.kind == UNIT_PAD) {
    float* const outs[2] = {dK, dV};
    zero_pads<2>(q, outs, nullptr);
    return;
  }
  const Rows r(a, q, m);
  if (tid < kRows) own_k[tid * kStride + kTokAt] = __int_as_float(r.valid ? r.pos : -1);
  const int t0 = (wave + q.turn) & (kWaves - 1);
  int tok = r.token(t0, m), tok_next = r.token(t0 + kWaves, m);
  const float *lse = a.lse + bh, *delta = a.delta + bh;
  float row_lse = lse[tok], row_delta = delta[tok];  // of tile row m
  float *tile_q = lds + wave * kTileFloats, *tile_g = tile_q + kWaves * kTileFloats;
  TileRegs qry, grad;
  qry.load(Q, tok, lane);
  put_owned(own_k, K, r.pos, wave, lane);
  put_owned(lds, V, r.pos, wave, lane);  // passes through the first tile into registers: there is no room for both
  grad.load(dO, tok, lane);
  keep_order();
  __syncthreads();
  f32x4 v_own[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) v_own[j] = *reinterpret_cast<const f32x4*>(lds + m * kStride + 8 * j + 4 * hl);
  __syncthreads();
  const float sc = a.scale * kLog2e;

  f32x16 dk[2] = {zero16(), zero16()}, dv[2] = {zero16(), zero16()};
  // S -> P, dP -> dS.  (A pair outside the pattern has P = 0 and so dS = 0, unless a value is not finite: then dS is
  // masked as well, in the second pass.)
  auto dscores = [&](f32x16& s, f32x16& dp, const SlotWindow& mask, bool mask_ds) {
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const float l = __shfl(row_lse, c_row(c, hl), 64), d = __shfl(row_delta, c_row(c, hl), 64);
      s[c] = mask.in(c) ? __builtin_amdgcn_exp2f(fmaf(s[c], sc, -l * kLog2e)) : 0.f;
      dp[c] = s[c] * (dp[c] - d);
      if (mask_ds) dp[c] = mask.in(c) ? dp[c] : 0.f;
    }
  };
  for (int t = t0; t < r.n; t += kWaves) {
    const int tok_after = r.token(t + 2 * kWaves, m);
    qry.put(tile_q, lane);
    qry.load(Q, tok_next, lane);
    grad.put(tile_g, lane);
    grad.load(dO, tok_next, lane);
    keep_order();
    f32x16 s = contract(tile_q, own_k, m, hl, zero16());   // S  = Q K^T
    f32x16 dp = contract(tile_g, v_own, m, hl, zero16());  // dP = dO V^T
    dscores(s, dp, r.mask(t, hl), false);
    row_lse = lse[tok_next];
    row_delta = delta[tok_next];
    keep_order();
    accumulate(dv, tile_g, m, hl, s);                      // dV^T += dO^T P
    accumulate(dk, tile_q, m, hl, dp);                     // dK^T += Q^T dS
    tok_next = tok_after;
  }
  if (__builtin_expect(any_special(dk) || any_special(dv), 0)) {
    dk[0] = dk[1] = dv[0] = dv[1] = zero16();
    for (int t = t0; t < r.n; t += kWaves) {
      tok = r.token(t, m);
      row_lse = lse[tok];
      row_delta = delta[tok];
      qry.load(Q, tok, lane);
      qry.put(tile_q, lane);
      grad.load(dO, tok, lane);
      grad.put(tile_g, lane);
      f32x16 s = contract(tile_q, own_k, m, hl, zero16());
      f32x16 dp = contract(tile_g, v_own, m, hl, zero16());
      const SlotWindow mask = r.mask(t, hl);
      dscores(s, dp, mask, true);
      accumulate_special(dv, tile_g, m, hl, s, mask);
      accumulate_special(dk, tile_q, m, hl, dp, mask);
    }
  }
  __syncthreads();
  store_sum(dk, a.scale, lds, own_k, dK, wave, m, hl);
  store_sum(dv, 1.f, lds + kWaves * kTileFloats, own_k, dV, wave, m, hl);
}

}  // namespace

hipError_t launch_fwd_f32(const AttnArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(fwd_f32_kernel, dim3(4 * unit_grid(a.B, a.H, a.N, a.n_col)), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_bwd_f32(const AttnArgs& a, hipStream_t stream) {
  const dim3 grid(4 * unit_grid(a.B, a.H, a.N, a.n_col));
  hipLaunchKernelGGL(bwd_dq_f32_kernel, grid, dim3(kThreads), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(bwd_dkv_f32_kernel, grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace mate
