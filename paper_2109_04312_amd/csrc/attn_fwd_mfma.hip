// bf16 MFMA forward for MATE attention (Section 3: attention pattern and head equation;
// Section 3.1: per-head-kind ordering so that a token's keys are contiguous).
//
// A workgroup (4 wavefronts) owns 128 consecutive queries of one (sequence, head) in the head
// kind's sorted order -- or 128 question tokens, or 1024 pad tokens (zero fill).  It streams the
// keys those queries may see in 64-key tiles: first the question tokens (gathered through
// global_idx), then the sorted slots spanned by the queries' own row / column segments
// (gathered through perm; every table token for question-token owners, whose key stream is cut
// into chunks run by separate workgroups).  Each key tile goes straight from global memory
// into LDS once (K and V both as [key][dim]; V^T is produced by transposing LDS reads) and is
// used by all four wavefronts; scores are masked per element by "key slot inside this query's
// segment range", and one online softmax runs across
// the question-key and segment-key tiles, which is the single softmax over the union that the
// definition asks for.  Chunked owners leave (unnormalised O, max, sum) partials that the chunk
// arriving last merges with the usual log-sum-exp rule.
#include <hip/hip_runtime.h>

#include "d2l.h"
#include "launch.h"
#include "mfma_common.h"
#include "stream_plan.h"
#include "tile_bodies.h"
#include "tile_stream.h"

namespace mate {
namespace {

constexpr int kStageBytes = 2 * kTileBytes;   // K tile, V tile

// O = sum_c 2^(m_c - m) O_c / sum_c 2^(m_c - m) l_c over the chunks of one owner tile of question
// tokens; slot0 = the tile's first partial slot.  Items are dealt to the four wavefronts.
template <bool kThrough>
__device__ __forceinline__ void merge_chunks(const AttnArgs& a, const UnitPlan& u, size_t slot0, unsigned short* O,
                                             float* LSE, char* stage, const int* row_tok, int wave, int lane) {
  const int m = lane & 31, hl = lane >> 5;
  const float* part = a.part[0] + slot0 * BM * kD;
  const float* stat = a.part_ml + slot0 * BM * 2;
  for (int item = wave; item < 2 * BM / 32; item += kThreads / 64) {
    const int row = (item >> 1) * 32 + m;
    if (u.t0 + (item >> 1) * 32 >= u.own_count) break;  // no question token in this block
    f32x16 acc = zero16();
    float mx = -INFINITY, l = 0.f;
    for (int c0 = 0; c0 < u.n_chunks; c0 += kBatch) {
      float2 ml[kBatch], v[kBatch][8];
#pragma unroll
      for (int e = 0; e < kBatch; ++e) ml[e] = get_pair<true>(stat + ((size_t)min(c0 + e, u.n_chunks - 1) * BM + row) * 2);
      load_items<true>(v, part, item, c0, u.n_chunks, lane);
      float m_new = mx;
#pragma unroll
      for (int e = 0; e < kBatch; ++e) m_new = fmaxf(m_new, ml[e].x);  // (repeats of the last chunk change nothing)
      const float alpha = __builtin_amdgcn_exp2f(mx - m_new);          // every chunk has a key: m_new is finite
      mx = m_new;
      l *= alpha;
#pragma unroll
      for (int c = 0; c < 16; ++c) acc[c] *= alpha;
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        const float w = c0 + e < u.n_chunks ? __builtin_amdgcn_exp2f(ml[e].x - mx) : 0.f;
        l += w * ml[e].y;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          acc[2 * i] += w * v[e][i].x;
          acc[2 * i + 1] += w * v[e][i].y;
        }
      }
    }
    stage_rows(acc, 1.f / l, stage, row, item & 1, hl);
    if ((item & 1) == 0 && hl == 0 && row_tok[row] >= 0) LSE[row_tok[row]] = (mx + __builtin_amdgcn_logf(l)) * kLn2;
  }
  __syncthreads();
  flush_rows<kThrough>(O, stage, row_tok, wave, lane);
}

template <int kTiles>
struct FwdLds {
  __attribute__((aligned(1024))) char stages[kStages * kTiles * kStageBytes];
  int idx_ring[kIdxSlots][BN];  // [tile & 7][row] token positions
  int q_tok[BM];
  int group_done;
};

// kThrough: see result_through.
template <int kTiles, bool kThrough>
__device__ __forceinline__ void fwd_unit(const AttnArgs& a, const Work& w, FwdLds<kTiles>& s) {
  char* const lds = s.stages;
  int (&idx_ring)[kIdxSlots][BN] = s.idx_ring;
  int (&q_tok)[BM] = s.q_tok;
  int& group_done = s.group_done;
  const int N = a.N, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction
  const int m = lane & 31, hl = lane >> 5;
  const UnitPlan& u = w.u;

  const size_t bh = (size_t)w.bh * N;
  const unsigned short* Q = static_cast<const unsigned short*>(a.q) + bh * kD;
  const unsigned short* K = static_cast<const unsigned short*>(a.k) + bh * kD;
  const unsigned short* V = static_cast<const unsigned short*>(a.v) + bh * kD;
  unsigned short* O = static_cast<unsigned short*>(a.out) + bh * kD;
  float* LSE = a.lse + bh;

  if (u.kind == UNIT_PAD) {  // pad positions: O = 0, LSE = 0
    unsigned short* const outs[1] = {O};
    zero_pad_rows<1>(outs, u, tid);
    int tok[kPadSlots / kThreads];
#pragma unroll
    for (int i = 0; i < kPadSlots / kThreads; ++i) {
      const int row = u.t0 + tid + i * kThreads;
      tok[i] = row < u.own_count ? u.own_list[row] : -1;
    }
#pragma unroll
    for (int i = 0; i < kPadSlots / kThreads; ++i)
      if (tok[i] >= 0) LSE[tok[i]] = 0.f;
    return;
  }

  // First round trip: which rows this workgroup owns, and the token indices of the first tiles.
  // Second: the owned query rows (registers) and the first K / V tiles (LDS), all in flight
  // together.
  TileStream<kStageBytes, kTiles> stream(u, w.global_idx, lds, idx_ring, K, V, nullptr, 0, wave, lane);
  stream.begin();
  const OwnerSplit<kTiles> split(u, wave);
  const OwnedRow me = owned_row(w, split.block, m);
  asm volatile("" ::"v"(me.pos), "v"(me.lo), "v"(me.hi), "v"(me.stage_tok));  // the owned rows are known from here on
  if (tid < BM) q_tok[tid] = me.stage_tok;
  stream.prime();

  OwnedTile q_rows;
  q_rows.load(Q, me.pos, lane);
  bf16x8 qf[4];
  q_rows.operands(qf, stream.room(), lane);

  const float sc = uniform(a.scale * kLog2e);  // scores are kept raw; exp2(s * sc - m * sc)
  f32x16 o_acc[2] = {zero16(), zero16()};
  float m_run = -INFINITY, l_run = 0.f;  // reference of raw scores; this lane-half's share of the sum
  Reference ref = kMissing;

  const int tb = u.t_begin, te = u.t_end;
  // Everything loaded into registers so far is pinned as complete here, so that no load with a
  // register destination is pending inside the loop (the compiler would otherwise wait for
  // *all* outstanding loads, prefetches included, at the first use).
  asm volatile("" ::"v"(qf[0]), "v"(qf[1]), "v"(qf[2]), "v"(qf[3]));

  const OperandLanes lanes(lane);

  for (int t0 = tb; t0 < te; t0 += kTiles) {
    const unsigned stage = lds_addr(stream.acquire(t0));
#pragma unroll 1
    for (int j = 0; j < kTiles; ++j) {
      const int t = t0 + j;
      if (kTiles > 1 && (t >= te || !split.meets(j))) continue;
      // visible slot window for this tile: question keys [0,G), else this lane's segment range
      const bool part0 = t < u.n_t0;
      const int base = part0 ? t * BN : u.s_lo + (t - u.n_t0) * BN;
      if (me.wave_active) {
        WindowMask mask(base, hl, part0, u.G, me.lo, me.hi, split.first(base, part0 ? 0 : me.w_lo),
                        split.end(base, part0 ? u.G : me.w_hi), part0 ? 0 : me.a_lo, part0 ? u.G : me.a_hi);
        fwd_tile(stage + j * kStageBytes, qf, lanes, sc, mask, o_acc, m_run, l_run, ref);
      }
    }
  }
  __syncthreads();  // all wavefronts are done reading the stages; reuse them for the epilogue

  int ln = lane;
  asm volatile("" : "+v"(ln));  // what follows is computed here, not kept in registers through the loop
  const int row = wave * 32 + (ln & 31);
  if (split.on) {  // add the other half of the streamed rows: O = sum_h 2^(m_h - m) O_h, l likewise
    // (beyond the 16 KB the epilogue stages rows in; the statistics where the token indices were)
    char* const mine = lds + BM * 128 + (wave & 1) * (kItemFloats * 2 * 4);
    float* const stat = reinterpret_cast<float*>(&idx_ring[2 * (wave & 1)][0]);
    auto put = [&](char* items, float* st) {
      put_items(items, o_acc, ln);
      st[ln] = m_run;
      st[64 + ln] = l_run;
    };
    auto add = [&](const char* items, const float* st) {
      const float m2 = st[ln], m_new = fmaxf(m_run, m2);
      const float own = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_run - m_new) * sc);
      const float other = m2 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m2 - m_new) * sc);
      l_run = l_run * own + st[64 + ln] * other;
      m_run = m_new;
      add_items(items, o_acc, own, other, ln);
    };
    if (wave >= 2) put(mine, stat);
    __syncthreads();
    if (wave < 2) add(mine, stat);
    if (kTiles == 2 && split.four) {  // and the other tiles
      if (wave == 1) put(mine, stat);
      __syncthreads();
      if (wave == 0) add(lds + BM * 128 + kItemFloats * 2 * 4, reinterpret_cast<const float*>(&idx_ring[2][0]));
    }
  }
  const bool writes = me.wave_active && split.writes(wave);
  const float l_tot = half_sum(l_run);
  if (u.part >= 0) {
    // chunk of a question-token owner: leave (unnormalised O, max, sum); the last one merges
    const size_t slot = (size_t)w.bh * owner_slots(N) + u.part;
    const int mine = u.part % u.n_chunks;
    if (writes) {
      store_partial<true>(o_acc, 1.f, a.part[0] + slot * BM * kD, wave, ln);
      if (ln < 32)
        put_pair<true>(a.part_ml + (slot * BM + row) * 2, m_run == -INFINITY ? m_run : m_run * sc, l_tot);
    }
    unsigned long long* words = a.arrived + (slot - mine);
    if (completes_group(words, mine, u.n_chunks, a.ticket, &group_done)) {
      merge_chunks<kThrough>(a, u, slot - mine, O, LSE, lds, q_tok, wave, ln);
      const int c = wave * 64 + ln;
      if (c < u.n_chunks) __hip_atomic_store(words + c, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return;
  }
  if (ln < 32 && q_tok[row] >= 0) LSE[q_tok[row]] = (m_run * sc + __builtin_amdgcn_logf(l_tot)) * kLn2;
  const f32x16 (*accs[1])[2] = {&o_acc};
  const float muls[1] = {1.f / l_tot};
  unsigned short* const outs[1] = {O};
  store_owned_rows<1, kThrough>(accs, muls, outs, lds, q_tok, wave, ln);
}

template <bool kChunksFirst, bool kJoin, bool kMany>
__global__ __launch_bounds__(kThreads, 4) void fwd_mfma_kernel(MATE_UNIT_LISTS, AttnArgs a) {
  __shared__ FwdLds<1> s;
  Work w;
  if (kMany ? !take_unit_of_many<kChunksFirst, kJoin>(a, blockIdx.x, w)
            : !take_unit<kChunksFirst, kJoin>({hdr, gunit, unit_row, unit_col, B, H, N, n_col}, a, blockIdx.x, w)) return;
  fwd_unit<1, true>(a, w, s);
}
template <bool kChunksFirst, bool kThrough, bool kMany>
__global__ __launch_bounds__(kThreads, 2) void fwd_small_kernel(MATE_UNIT_LISTS, AttnArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char dynamic_lds[];
  Work w;
  if (kMany ? !take_unit_of_many<kChunksFirst, false>(a, blockIdx.x, w)
            : !take_unit<kChunksFirst, false>({hdr, gunit, unit_row, unit_col, B, H, N, n_col}, a, blockIdx.x, w)) return;
  if (OwnerSplit<2>(w.u, 0).four) fwd_unit<2, kThrough>(a, w, *reinterpret_cast<FwdLds<2>*>(dynamic_lds));
  else fwd_unit<1, kThrough>(a, w, *reinterpret_cast<FwdLds<1>*>(dynamic_lds));
}

}  // namespace

template <bool kChunksFirst, bool kThrough, bool kMany = false>
static hipError_t launch_small(const AttnArgs& a, dim3 grid, hipStream_t stream) {
  const hipError_t e = allow_lds<&fwd_small_kernel<kChunksFirst, kThrough, kMany>>(sizeof(FwdLds<2>));
  if (e != hipSuccess) return e;
  ProfileScope prof(2, stream);
  hipLaunchKernelGGL((fwd_small_kernel<kChunksFirst, kThrough, kMany>), grid, dim3(kThreads), sizeof(FwdLds<2>), stream, MATE_UNIT_LISTS_VALUES(a), a);
  return hipGetLastError();
}
hipError_t launch_fwd_mfma(const AttnArgs& a, hipStream_t stream) {
  const dim3 grid(unit_grid(a.B, a.H, a.N, a.n_col)), block(kThreads);
  const bool first = fwd_chunks_first(a.B, a.H, a.N), join = joins_chunks(a.B, a.H, a.N);
  if (small_forward(a.B, a.H, a.N)) {
    const bool owners = small_owners_first(a.B, a.H, a.N), through = result_through(a.B, a.H, a.N, 2);
    // Sequences of one tile whose records, half of them padding and empty ones, are more than the chip takes at once: step by step (see
    // kManyRecords).  us, in one round trip and so: 24 x 33, 8 heads 7.35 and 6.85, 14 x 45, 12 heads 7.3 and 6.8; 9 x 68, 16 heads (576 records)
    // 6.1 and 6.25, and longer sequences at as many records 0 to 2 % longer.
    if (owner_slots(a.N) == 1 && grid.x >= 640) return through ? launch_small<true, true, true>(a, grid, stream) : launch_small<true, false, true>(a, grid, stream);
    if (through) return owners ? launch_small<true, true>(a, grid, stream) : launch_small<false, true>(a, grid, stream);
    return owners ? launch_small<true, false>(a, grid, stream) : launch_small<false, false>(a, grid, stream);
  }
  ProfileScope prof(2, stream);
  const bool many = !first && (int)grid.x > kManyRecords;   // (chunks first: never that many)
  const auto kernel = first  ? (join ? fwd_mfma_kernel<true, true, false> : fwd_mfma_kernel<true, false, false>)
                      : many ? (join ? fwd_mfma_kernel<false, true, true> : fwd_mfma_kernel<false, false, true>)
                             : (join ? fwd_mfma_kernel<false, true, false> : fwd_mfma_kernel<false, false, false>);
  hipLaunchKernelGGL(kernel, grid, block, 0, stream, MATE_UNIT_LISTS_VALUES(a), a);
  return hipGetLastError();
}

}  // namespace mate
