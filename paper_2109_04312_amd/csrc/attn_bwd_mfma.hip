// bf16 MFMA backward for MATE attention: the derivative of the forward (Section 3 head
// equation restricted to the attention pattern A^i_k) with respect to Q, K and V.
//
// No floating-point atomics, so results are bit-reproducible:
//   dq kernel  -- a workgroup owns 128 queries (sorted order of the head kind, or question
//                 tokens) and streams the key tiles they see, exactly like the forward:
//                 P = exp(S - LSE), dP = dO V^T, dS = P (dP - delta), dQ += dS K.
//                 It also produces delta_k = dO_k . O_k for its queries and leaves -delta and
//                 -LSE / scale for the next kernel.
//   dkv kernel -- a workgroup owns 128 keys and streams the query tiles that see them: the
//                 question tokens plus the table tokens of the keys' own segments (every
//                 non-pad token when the keys are question tokens):
//                 dV += P^T dO, dK += dS^T Q.
// Question-token owners stream the whole sequence, so their stream is cut into chunks run by
// separate workgroups, which leave fp32 partials that are added in chunk order: dQ's by the first
// workgroups of the dkv kernel, dK's and dV's by the chunk that arrives last.
// Small launches run the units of both kernels in one (see the end).
// Pairs (table query, table key) are therefore recomputed once in each of the first two.
#include <hip/hip_runtime.h>

#include "d2l.h"
#include "launch.h"
#include "mfma_common.h"
#include "stream_plan.h"
#include "tile_bodies.h"
#include "tile_stream.h"

namespace mate {
namespace {

// Adds the chunk partials of one owner tile of question tokens in chunk order and stores its rows of
// kTensors gradients; part[x] = the tile's first partial slot.  Items (32 rows x 32 dims of one tensor)
// are dealt to the four wavefronts.
template <int kTensors, bool kShared>
__device__ __forceinline__ void merge_chunks(const float* const (&part)[kTensors], unsigned short* const (&out)[kTensors],
                                             int rows, int n_chunks, char* stage, const int* row_tok, int wave, int lane) {
  const int items = 2 * ((min(rows, BM) + 31) / 32);
  for (int i = wave; i < items * kTensors; i += kThreads / 64) {
    const int x = i / items, item = i - x * items;
    const float* src = x == 0 ? part[0] : part[kTensors - 1];
    f32x4 acc[2][2] = {};  // register i of the item: [i / 8][i / 4 % 2][i % 4]
    for (int c0 = 0; c0 < n_chunks; c0 += kBatch) {
      float2 v[kBatch][8];
      load_items<kShared>(v, src, item, c0, n_chunks, lane);
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        const float w = c0 + e < n_chunks ? 1.f : 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          acc[k >> 2][(k >> 1) & 1][2 * (k & 1)] += w * v[e][k].x;
          acc[k >> 2][(k >> 1) & 1][2 * (k & 1) + 1] += w * v[e][k].y;
        }
      }
    }
#pragma unroll
    for (int d = 0; d < 2; ++d) stage_rows_quad(acc[d], 1.f, stage + x * (BM * 128), (item >> 1) * 32, 2 * (item & 1) + d, lane);
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < kTensors; ++x) flush_rows(out[x], stage + x * (BM * 128), row_tok, wave, lane);
}

// ======================================================================================
// dQ (and delta)
// ======================================================================================
constexpr int kDqStage = 2 * kTileBytes;          // K tile, V tile
constexpr int kDkvStage = 2 * kTileBytes + 512;   // Q tile, dO tile, -lse/scale[64], -delta[64]

// kOne: delta and -LSE / scale are there already, and chunks are merged here.
template <bool kOne>
__device__ __forceinline__ void bwd_dq_unit(const AttnArgs& a, const Work& w, char* lds, int (*idx_ring)[BN], int* q_tok, int* group_done) {
  const int N = a.N, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction
  const int m = lane & 31, hl = lane >> 5;
  const UnitPlan& u = w.u;

  const size_t bh = (size_t)w.bh * N;
  const unsigned short* Q = static_cast<const unsigned short*>(a.q) + bh * kD;
  const unsigned short* K = static_cast<const unsigned short*>(a.k) + bh * kD;
  const unsigned short* V = static_cast<const unsigned short*>(a.v) + bh * kD;
  const unsigned short* O = static_cast<const unsigned short*>(a.o) + bh * kD;
  const unsigned short* dO = static_cast<const unsigned short*>(a.dout) + bh * kD;
  unsigned short* dQ = static_cast<unsigned short*>(a.dq) + bh * kD;

  if (u.kind == UNIT_PAD) {
    unsigned short* const outs[1] = {dQ};
    zero_pad_rows<1>(outs, u, tid);
    return;
  }
  // First round trip: which rows this workgroup owns, and the token indices of the first tiles.
  // Second: the owned rows (registers) and the first K / V tiles (LDS), all in flight together.
  // K and V tiles stream through the LDS ring; K is read both plain (S^T = K Q^T) and
  // transposed (dQ^T += K^T dS^T), V plain (dP^T = V dO^T).
  TileStream<kDqStage, 1, true> stream(u, w.global_idx, lds, idx_ring, K, V, nullptr, 0, wave, lane);
  stream.begin();
  const OwnerSplit<1> split(u, wave);
  const OwnedRow me = owned_row(w, split.block, m);
  asm volatile("" ::"v"(me.pos), "v"(me.lo), "v"(me.hi), "v"(me.stage_tok));  // the owned rows are known from here on
  if (tid < BM) q_tok[tid] = me.stage_tok;
  // the dkv kernel counts the chunks of an owner tile in the word of its first one
  if (!kOne && tid == 0 && u.part >= 0) a.arrived[(size_t)w.bh * owner_slots(N) + u.part] = 0;
  stream.prime();

  // this lane's query rows and dO rows as B operands (columns r, k = dims), and delta
  OwnedTile q_rows, g_rows, o_rows;
  g_rows.load(dO, me.pos, lane);
  if (!kOne) o_rows.load(O, me.pos, lane);
  q_rows.load(Q, me.pos, lane);
  const float lse = a.lse[bh + me.pos];
  const float kept = kOne ? a.delta[bh + me.pos] : 0.f;
  bf16x8 qf[2][2], gf[2][2];
  g_rows.operands(gf, stream.room(), lane);
  const float delta = kOne ? -kept : row_delta(g_rows, o_rows, stream.room(), lane);
  q_rows.operands(qf, stream.room(), lane);
  // Everything loaded into registers so far is pinned as complete here, so that no load with a
  // register destination is pending inside the loop.
  asm volatile("" ::"v"(qf[0][0]), "v"(qf[0][1]), "v"(qf[1][0]), "v"(qf[1][1]), "v"(gf[0][0]), "v"(gf[0][1]),
               "v"(gf[1][0]), "v"(gf[1][1]), "v"(delta), "v"(lse));
  // every chunk of a question-token owner computes the same delta; the first one stores it
  // (stored negated, with -lse / scale beside it: the dK/dV kernel starts its accumulators there)
  if (!kOne && hl == 0 && me.valid && u.t_begin == 0 && split.writes(wave)) {
    a.delta[bh + me.pos] = -delta;
    a.nlse[bh + me.pos] = -lse / a.scale;
  }
  const RowPair l = row_pair(__float_as_uint(lse * kLog2e)), nd = row_pair(__float_as_uint(-delta));
  const float lse2[2] = {__uint_as_float(l.v[0]), __uint_as_float(l.v[1])};
  f32x4 ndelta[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) ndelta[i >> 2][i & 3] = __uint_as_float(nd.v[i >> 2]);
  const RowPair rng = row_pair(me.lo | me.hi << 16);
  const float sc = uniform(a.scale * kLog2e);

  const QuadLanes lanes(lane);

  QuadAcc dq_acc = {};
  for (int t = u.t_begin; t < u.t_end; ++t) {
    const unsigned tile = lds_addr(stream.acquire(t));
    const bool part0 = t < u.n_t0;
    const int base = part0 ? t * BN : u.s_lo + (t - u.n_t0) * BN;
    if (me.wave_active) {
      PairWindowMask mask(base, lane, part0, u.G, rng, split.first(base, part0 ? 0 : me.w_lo),
                      split.end(base, part0 ? u.G : me.w_hi), part0 ? 0 : me.a_lo, part0 ? u.G : me.a_hi);
      dq_tile(tile, qf, gf, lanes, sc, lse2, ndelta, mask, dq_acc);
    }
  }
  __syncthreads();  // all wavefronts are done reading the stages; reuse them for the epilogue
  int ln = lane;
  asm volatile("" : "+v"(ln));  // what follows is computed here, not kept in registers through the loop
  if (split.on) {  // add the other half of the streamed rows
    char* const mine = lds + BM * 128 + (wave & 1) * (kItemFloats * 2 * 4);  // (rows are staged below that)
    if (wave >= 2) put_items(mine, dq_acc, ln);
    __syncthreads();
    if (wave < 2) add_items(mine, dq_acc, 1.f, 1.f, ln);
  }
  if (u.part >= 0) {
    const size_t slot = (size_t)w.bh * owner_slots(N) + u.part;
    if (me.wave_active && split.writes(wave)) store_partial<kOne>(dq_acc, a.scale, a.part[0] + slot * BM * kD, wave, ln);
    if constexpr (kOne) {
      const size_t slot0 = slot - u.part % u.n_chunks;
      publish_partials();
      if (tid == 0)  // (the word of the second chunk; the first one's is dK/dV's)
        *group_done = __hip_atomic_fetch_add(a.arrived + slot0 + 1, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                      (unsigned long long)(u.n_chunks - 1);
      __syncthreads();
      if (*group_done) {
        const float* const parts[1] = {a.part[0] + slot0 * BM * kD};
        unsigned short* const grads[1] = {dQ};
        merge_chunks<1, true>(parts, grads, u.own_count - u.t0, u.n_chunks, lds, q_tok, wave, ln);
        if (tid == 0) __hip_atomic_store(a.arrived + slot0 + 1, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    return;
  }
  const QuadAcc* accs[1] = {&dq_acc};
  const float muls[1] = {a.scale};
  unsigned short* const outs[1] = {dQ};
  store_owned_rows<1>(accs, muls, outs, lds, q_tok, wave, ln);
}

// (four workgroups per CU: with three, the column-head units of the benchmark shape do not all
// fit at once and the stragglers double the kernel's critical path)
template <bool kJoin, bool kMany>
__global__ __launch_bounds__(kThreads, 4) void bwd_dq_mfma_kernel(MATE_UNIT_LISTS, AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds[kStages * kDqStage];
  __shared__ int idx_ring[kIdxSlots][BN];
  __shared__ int row_tok[BM];
  Work w;
  if (kMany ? !take_unit_of_many<true, kJoin>(a, blockIdx.x, w)
            : !take_unit<true, kJoin>({hdr, gunit, unit_row, unit_col, B, H, N, n_col}, a, blockIdx.x, w)) return;
  bwd_dq_unit<false>(a, w, lds, idx_ring, row_tok, nullptr);
}

// ======================================================================================
// dK, dV
// ======================================================================================
__device__ __forceinline__ void bwd_dkv_unit(const AttnArgs& a, const Work& w, char* lds, int (*idx_ring)[BN], int* k_tok, int* group_done) {
  const int N = a.N, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction
  const int m = lane & 31;
  const UnitPlan& u = w.u;

  const size_t bh = (size_t)w.bh * N;
  const unsigned short* Q = static_cast<const unsigned short*>(a.q) + bh * kD;
  const unsigned short* K = static_cast<const unsigned short*>(a.k) + bh * kD;
  const unsigned short* V = static_cast<const unsigned short*>(a.v) + bh * kD;
  const unsigned short* dO = static_cast<const unsigned short*>(a.dout) + bh * kD;
  unsigned short* dK = static_cast<unsigned short*>(a.dk) + bh * kD;
  unsigned short* dV = static_cast<unsigned short*>(a.dv) + bh * kD;

  if (u.kind == UNIT_PAD) {
    unsigned short* const outs[2] = {dK, dV};
    zero_pad_rows<2>(outs, u, tid);
    return;
  }
  // Q and dO tiles of the streamed queries go through the LDS ring, each read plain
  // (S = Q K^T, dP = dO V^T) and transposed (dK^T += Q^T dS, dV^T += dO^T P); wavefront 0
  // also brings the queries' -lse / scale, wavefront 1 their -delta (one float per row).
  // First round trip: the owned rows' positions and the first tiles' token indices; second:
  // the owned K / V rows (registers) and the first tiles (LDS).
  const float* row_src = wave == 0 ? a.nlse + bh : wave == 1 ? a.delta + bh : nullptr;
  TileStream<kDkvStage, 1, true> stream(u, w.global_idx, lds, idx_ring, Q, dO, row_src,
                               2 * kTileBytes + 256 * wave, wave, lane);
  stream.begin();
  // `me` is this lane's key; its window is the set of query slots that see it
  const OwnerSplit<1> split(u, wave);
  const OwnedRow me = owned_row(w, split.block, m);
  asm volatile("" ::"v"(me.pos), "v"(me.lo), "v"(me.hi), "v"(me.stage_tok));  // the owned rows are known from here on
  if (tid < BM) k_tok[tid] = me.stage_tok;
  stream.prime();

  OwnedTile k_rows, v_rows;
  k_rows.load(K, me.pos, lane);
  v_rows.load(V, me.pos, lane);
  bf16x8 kf[2][2], vf[2][2];  // this lane's key and value rows as B operands
  k_rows.operands(kf, stream.room(), lane);
  v_rows.operands(vf, stream.room(), lane);
  const float sc = uniform(a.scale * kLog2e);
  asm volatile("" ::"v"(kf[0][0]), "v"(kf[0][1]), "v"(kf[1][0]), "v"(kf[1][1]), "v"(vf[0][0]), "v"(vf[0][1]),
               "v"(vf[1][0]), "v"(vf[1][1]));

  const QuadLanes lanes(lane);
  const int quarter = lane >> 4;
  const RowPair rng = row_pair(me.lo | me.hi << 16);

  QuadAcc dk_acc = {}, dv_acc = {};
  for (int t = u.t_begin; t < u.t_end; ++t) {
    const char* Qst = stream.acquire(t);
    const float* lse_row = reinterpret_cast<const float*>(Qst + 2 * kTileBytes);
    const float* delta_row = lse_row + BN;
    const bool part0 = t < u.n_t0;
    const int base = part0 ? t * BN : u.s_lo + (t - u.n_t0) * BN;
    if (me.wave_active) {
      PairWindowMask mask(base, lane, part0, u.G, rng, split.first(base, part0 ? 0 : me.w_lo),
                      split.end(base, part0 ? u.G : me.w_hi), part0 ? 0 : me.a_lo, part0 ? u.G : me.a_hi);
      dkv_tile(lds_addr(Qst), lse_row, delta_row, kf, vf, lanes, sc, quarter, mask, dk_acc, dv_acc);
    }
  }
  __syncthreads();  // all wavefronts are done reading the stages; reuse them for the epilogue
  if (split.on) {  // add the other half of the streamed rows
    char* const mine = lds + (wave & 1) * (kItemFloats * 4 * 4);
    if (wave >= 2) {
      put_items(mine, dk_acc, lane);
      put_items(mine + kItemFloats * 2 * 4, dv_acc, lane);
    }
    __syncthreads();
    if (wave < 2) {
      add_items(mine, dk_acc, 1.f, 1.f, lane);
      add_items(mine + kItemFloats * 2 * 4, dv_acc, 1.f, 1.f, lane);
    }
    __syncthreads();
  }
  if (u.part >= 0) {
    const size_t slot = (size_t)w.bh * owner_slots(N) + u.part;
    const size_t slot0 = slot - u.part % u.n_chunks;
    if (me.wave_active && split.writes(wave)) {
      store_partial<true>(dk_acc, a.scale, a.part[1] + slot * BM * kD, wave, lane);
      store_partial<true>(dv_acc, 1.f, a.part[2] + slot * BM * kD, wave, lane);
    }
    publish_partials();
    if (tid == 0)
      *group_done = __hip_atomic_fetch_add(a.arrived + slot0, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                   (unsigned long long)(u.n_chunks - 1);
    __syncthreads();
    if (*group_done) {
      const float* const parts[2] = {a.part[1] + slot0 * BM * kD, a.part[2] + slot0 * BM * kD};
      unsigned short* const grads[2] = {dK, dV};
      merge_chunks<2, true>(parts, grads, u.own_count - u.t0, u.n_chunks, lds, k_tok, wave, lane);
    }
    return;
  }
  const QuadAcc* accs[2] = {&dk_acc, &dv_acc};
  const float muls[2] = {a.scale, 1.f};
  unsigned short* const outs[2] = {dK, dV};
  store_owned_rows<2>(accs, muls, outs, lds, k_tok, wave, lane);
}

// dQ rows of the question tokens of one (sequence, head) from the dq kernel's chunk partials.
template <bool kJoin>
__device__ __forceinline__ void merge_dq(const AttnArgs& a, int bh_i, char* stage, int* row_tok) {
  const int b = bh_i / a.H, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // header and counts in one scalar round trip (both lie inside the table buffer whatever it holds)
  const int* cnt = a.seg.counts + (size_t)b * kCountWords;
  const int h_magic = a.seg.hdr[0], h_B = a.seg.hdr[1], h_N = a.seg.hdr[2];
  const int G = cnt[C_G], L = cnt[C_L];
  if (h_magic != kMagic || h_B != a.B || h_N != a.N) return;
  GlobalSplit s = global_split(G, L, a.B, a.N);
  if (kJoin && s.n_st <= kLongStream) s.n_chunks = joined(s.n_chunks);
  if (s.n_chunks <= 1) return;
  unsigned short* const out[1] = {static_cast<unsigned short*>(a.dq) + (size_t)bh_i * a.N * kD};
  for (int gt = 0; gt < s.n_gt; ++gt) {
    const int row = gt * BM + tid;
    if (tid < BM) row_tok[tid] = row < G ? a.seg.global_idx[(size_t)b * a.N + row] : -1;
    const size_t slot0 = (size_t)bh_i * owner_slots(a.N) + (size_t)gt * s.n_chunks;
    const float* const part[1] = {a.part[0] + slot0 * BM * kD};
    merge_chunks<1, false>(part, out, G - gt * BM, s.n_chunks, stage, row_tok, wave, lane);
    __syncthreads();
  }
}

// The first `n_merge` workgroups (a multiple of eight, so that the unit queues keep their XCDs) merge
// dQ partials: a few microseconds each, out of the way before the kernel's own tail.
// (162 registers: three workgroups per CU; with two the kernel takes 15 to 20 % longer)
template <bool kJoin, bool kMany>
__global__ __launch_bounds__(kThreads, 3) void bwd_dkv_mfma_kernel(MATE_UNIT_LISTS, AttnArgs a, int n_merge) {
  __shared__ __attribute__((aligned(1024))) char lds[kStages * kDkvStage];
  __shared__ int idx_ring[kIdxSlots][BN];
  __shared__ int row_tok[BM];
  __shared__ int group_done;
  if ((int)blockIdx.x < n_merge) {
    if ((int)blockIdx.x < a.B * a.H) merge_dq<kJoin>(a, blockIdx.x, lds, row_tok);
    return;
  }
  Work w;
  if (kMany ? !take_unit_of_many<true, kJoin>(a, blockIdx.x - n_merge, w)
            : !take_unit<true, kJoin>({hdr, gunit, unit_row, unit_col, B, H, N, n_col}, a, blockIdx.x - n_merge, w)) return;
  bwd_dkv_unit(a, w, lds, idx_ring, row_tok, &group_done);
}

// ======================================================================================
// Small launches: both in one, and delta before it
// ======================================================================================
// A launch that does not fill the chip is as long as its longest unit, twice over; with dK/dV's units and dQ's in one
// launch the second time goes.  What dQ did for dK/dV (-delta, -LSE / scale, the cleared words) is a launch of its own
// then, and dQ's chunks are merged by the one that arrives last, counted in the word of the group's second chunk.
// us, backward as dQ and dK/dV and as delta and both: 12 heads, one sequence of 300 19.0 -> 13.8, 512 22.8 -> 16.1, 1024
// 24.4 -> 17.1, 4096 56.8 -> 43.3, 8 x 512 30.3 -> 24.9, 16 x 512 44.2 -> 42.8.
constexpr int kDeltaRows = 128;   // of a workgroup, eight lanes of eight dims each
__global__ __launch_bounds__(kThreads) void bwd_delta_kernel(AttnArgs a) {
  const size_t rows = (size_t)a.B * a.H * a.N, first = (size_t)blockIdx.x * kDeltaRows + (threadIdx.x >> 3);
  const int piece = threadIdx.x & 7;
  bf16x8 g[4], o[4];
  float lse[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const size_t row = min(first + 32 * i, rows - 1), at = row * kD + 8 * piece;
    g[i] = *reinterpret_cast<const bf16x8*>(static_cast<const unsigned short*>(a.dout) + at);
    o[i] = *reinterpret_cast<const bf16x8*>(static_cast<const unsigned short*>(a.o) + at);
    lse[i] = a.lse[row];
  }
  const size_t words = (size_t)a.B * a.H * owner_slots(a.N);
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < words; i += (size_t)gridDim.x * kThreads) a.arrived[i] = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float d = row_dot8(g[i], o[i]);
    if (piece == 0 && first + 32 * i < rows) {
      a.delta[first + 32 * i] = -d;
      a.nlse[first + 32 * i] = -lse[i] / a.scale;
    }
  }
}
template <bool kJoin, bool kMany>
__global__ __launch_bounds__(kThreads, 3) void bwd_both_mfma_kernel(MATE_UNIT_LISTS, AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds[kStages * kDkvStage];
  __shared__ int idx_ring[kIdxSlots][BN];
  __shared__ int row_tok[BM];
  __shared__ int group_done;
  const unsigned half = gridDim.x / 2;
  const bool dkv = blockIdx.x < half;
  Work w;
  const int unit = dkv ? blockIdx.x : blockIdx.x - half;
  if (kMany ? !take_unit_of_many<true, kJoin>(a, unit, w)
            : !take_unit<true, kJoin>({hdr, gunit, unit_row, unit_col, B, H, N, n_col}, a, unit, w)) return;
  if (dkv) bwd_dkv_unit(a, w, lds, idx_ring, row_tok, &group_done);
  else bwd_dq_unit<true>(a, w, lds, idx_ring, row_tok, &group_done);
}

}  // namespace

// Does a launch leave so much of the chip idle that dQ and dK/dV run at once?  dQ has four workgroups on a compute unit
// where the registers of dK/dV leave room for three, so two launches of one full round each are as fast as one of two.
// Measured over 500 launches of 64 to 8192 tokens, full sequences and such with a third of padding, 12 and 16 heads.  By units of
// 128 owners (a sequence's tiles and, per head, one for its question tokens) one launch is so many times as fast, mean and worst:
// up to two tiles a sequence 1.05 and 1.00 at 1000 units, 1.04 and 0.99 at 1080, 1.00 and 0.94 beyond; three to six tiles 1.11 and
// 0.99 at 640, 1.03 and 0.94 (12 x 512) at 760, 1.00 and 0.93 at 840, 0.98 and 0.92 at 1000; more tiles, where one long chain is
// most of a launch, 1.09 and 1.04 at 760, 1.05 and 0.97 at 860 (768 tiles), 1.0 at 1500.
static bool both_at_once(int B, int H, int N) {
  const int T = owner_slots(N);
  const long tiles = (long)B * H * T, units = tiles + (long)B * H;
  return T > 6 ? tiles <= 768 : units <= (T > 2 ? 760 : 1080);
}

template <bool kJoin>
static hipError_t launch_bwd(const AttnArgs& a, hipStream_t stream) {
  const dim3 grid(unit_grid(a.B, a.H, a.N, a.n_col)), block(kThreads);
  const bool many = (int)grid.x > kManyRecords;
  hipError_t e;
  if (both_at_once(a.B, a.H, a.N)) {
    const size_t rows = (size_t)a.B * a.H * a.N;
    hipLaunchKernelGGL(bwd_delta_kernel, dim3((unsigned)((rows + kDeltaRows - 1) / kDeltaRows)), block, 0, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    ProfileScope prof(4, stream, 3);
    // Sequences of one or two tiles, where half of the records or more are padding and empty ones: step by step (see kManyRecords) from one and a
    // half rounds of workgroups on.  us, in one round trip and so: 24 x 53, 8 heads 13.1 and 12.4, 15 x 39, 12 heads 12.4 and 11.65, 23 x 106, 8 heads
    // 15.9 and 15.3, 11 x 149 12.55 and 12.1, 16 x 128, 12 heads 15.6 and 15.4, 18 x 61 14.5 and 14.8; 66 such sizes 1.3 % shorter in the mean, 2 % longer at
    // worst.  With fewer workgroups the round trip is 1 % shorter, and with longer sequences up to 8 % either way, 0.3 % in the mean.
    const bool step_by_step = !kJoin && owner_slots(a.N) <= 2 && 2 * grid.x >= 1152;   // (chunks that are joined: seven tiles and more)
    const auto kernel = step_by_step ? bwd_both_mfma_kernel<false, true> : bwd_both_mfma_kernel<kJoin, false>;
    hipLaunchKernelGGL(kernel, dim3(2 * grid.x), block, 0, stream, MATE_UNIT_LISTS_VALUES(a), a);
    return hipGetLastError();
  }
  {
    ProfileScope prof(3, stream);
    const auto kernel = many ? bwd_dq_mfma_kernel<kJoin, true> : bwd_dq_mfma_kernel<kJoin, false>;
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, MATE_UNIT_LISTS_VALUES(a), a);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  ProfileScope prof(4, stream);
  const int n_merge = may_chunk(a.B, a.N) ? 8 * ((a.B * a.H + 7) / 8) : 0;
  const auto kernel = many ? bwd_dkv_mfma_kernel<kJoin, true> : bwd_dkv_mfma_kernel<kJoin, false>;
  hipLaunchKernelGGL(kernel, dim3(grid.x + n_merge), block, 0, stream, MATE_UNIT_LISTS_VALUES(a), a, n_merge);
  return hipGetLastError();
}
hipError_t launch_bwd_mfma(const AttnArgs& a, hipStream_t stream) {
  return joins_chunks(a.B, a.H, a.N) ? launch_bwd<true>(a, stream) : launch_bwd<false>(a, stream);
}

}  // namespace mate
