// Dense-mask variant of the bf16 MFMA attention kernels for short sequences.
//
// Section 3.1 keeps two functionally equivalent implementations -- the reordered, windowed one and
// plain attention under the mask of Section 3 -- and picks the faster per use case, because at
// short lengths the cost of reordering outweighs the saved work.  Here the reordered path is
// mate_build_segments + mate_attn_fwd / mate_attn_bwd; this file is the other one: no segment
// tables, no sort, no gathers.  A workgroup has a whole (sequence, head) in LDS, up to 128 positions
// (192 for some numbers of pairs) in the forward and 256 in the backward; of longer sequences it owns 128
// consecutive positions and streams every 64-position tile.  Each (query, key) pair is
// scored and then kept or dropped by comparing the two tokens' codes
//     code = row id + 1 (row heads) / column id + 1 (column heads) for a table token,
//            0 for a question token, kPadCode for padding
//     allowed = both are not padding, and they are equal or one is a question token
// which is the attention pattern A^i_k of Section 3 written per pair.  The arithmetic (base-2
// softmax, online where keys are streamed and with one maximum where all are there, bf16 P and dS, fp32
// accumulation, accumulators of dK and dV started at -lse / scale and -delta) is that of the segment
// kernels, so both paths meet the same oracle.
#include <hip/hip_runtime.h>

#include "d2l.h"
#include "launch.h"
#include "mfma_common.h"
#include "stream_plan.h"
#include "tile_bodies.h"

namespace mate {
namespace {

constexpr int kStage = 2 * kTileBytes;        // two tensors' tiles
constexpr int kDkvStageD = kStage + 512;      // ... plus -lse/scale[64], -delta[64]

constexpr unsigned kPadCode = 0xffffffffu;

struct DenseUnit {
  int b, bh, view, tile;  // tile: which 128 positions are owned
};

// The first arguments of a kernel, plain values, which arrive in registers with the wavefront; N and H in one word.  With the
// head kinds as bits and the codes' loads ahead of the tiles' (a kind was a byte, a vector load that the ids, and
// so the first barrier, waited for): forward of 32 x 128, 12 heads 8.6 -> 8.1 us, 64 x 64 7.2 -> 6.9, 3 x 600 14.2 -> 13.4,
// backward of 64 x 64 11.7 -> 11.0, 8 x 256 18.0 -> 17.5.
inline int pack_sizes(int N, int H) { return N | H << 16; }
static_assert(kDenseMaxN < 1 << 16, "sixteen bits hold N");

__device__ __forceinline__ int head_view(const DenseArgs& a, int h) { return (int)(a.col_heads[h >> 5] >> (h & 31)) & 1; }
// Workgroup -> (sequence, head, owner tile); (sequence, head) pairs with equal index mod 8 share
// an XCD (consecutive workgroups go to consecutive XCDs), so their K / V tiles share an L2.
__device__ __forceinline__ bool dense_unit(const DenseArgs& a, int N, int H, int pairs, DenseUnit& u) {
  const int q = blockIdx.x & 7, r = blockIdx.x >> 3;
  u.bh = uniform_div(r, owner_slots(N), u.tile) * 8 + q;
  if (u.bh >= pairs) return false;
  int h;
  u.b = uniform_div_any(u.bh, H, h);
  u.view = head_view(a, h);
  return true;
}
inline int dense_grid(const DenseArgs& a) { return 8 * ((a.B * a.H + 7) / 8) * owner_slots(a.N); }

// (ids below 0 are not valid; -1 and less act as question tokens and padding)
__device__ inline unsigned token_code(bool in_range, int flag, int id) {
  if (!in_range || flag > 1 || (flag == 0 && id < -1)) return kPadCode;
  return flag == 1 ? 0u : (unsigned)id + 1u;
}

// Codes of all positions of the sequence (padded with kPadCode to a whole number of tiles), on their way into LDS.
struct DenseCodes {
  int flag[kDenseMaxN / kThreads], id[kDenseMaxN / kThreads];
  __device__ __forceinline__ void load(const int* row_ids, const int* col_ids, const unsigned char* flags, const DenseUnit& u, int N) {
    const int* ids = pick(u.view == 0, row_ids, col_ids) + (size_t)u.b * N;
    const unsigned char* fl = flags + (size_t)u.b * N;
#pragma unroll
    for (int i = 0; i < kDenseMaxN / kThreads; ++i)
      if (i * kThreads < N) {
        const int n = min((int)threadIdx.x + i * kThreads, N - 1);
        flag[i] = fl[n];
        id[i] = ids[n];
      }
  }
  __device__ __forceinline__ void put(unsigned* code, int N) const {
#pragma unroll
    for (int i = 0; i < kDenseMaxN / kThreads; ++i) {
      const int n = (int)threadIdx.x + i * kThreads;
      if (i * kThreads < N && n < ((N + BN - 1) / BN) * BN) code[n] = token_code(n < N, flag[i], id[i]);
    }
  }
};

// May the owned row (code mc) meet a streamed row with code kc?  min(kc, kc ^ mc) is 0 iff the streamed row is a
// question token or has the same code, and with mc = 0 it is kc; so one comparison with a limit that depends on
// the owned row says it: below 1 for a table token, below kPadCode for a question token (code 0), never for
// padding.  (Four instructions per pair where comparing the three cases took seven: training steps of 32
// sequences of 128, 12 heads 27.1 -> 25.5 us, of one 18.0 -> 15.5, with the loads below in one round trip.)
__device__ inline unsigned owner_limit(unsigned mc) { return mc == 0u ? kPadCode : mc == kPadCode ? 0u : 1u; }
__device__ inline bool allowed(unsigned kc, unsigned mc, unsigned limit) { return min(kc, kc ^ mc) < limit; }

// Owned row of a lane: position, code, and whether anything may be written for it.
struct DenseRow {
  int pos;     // clamped to N - 1
  bool in_range;
  unsigned code, limit;
};
__device__ inline DenseRow dense_row(int N, const DenseUnit& u, const unsigned* code, int wave, int m) {
  DenseRow r;
  const int p = u.tile * BM + wave * 32 + m;
  r.in_range = p < N;
  r.pos = min(p, N - 1);
  r.code = code[r.pos];
  r.limit = owner_limit(r.code);
  return r;
}

// Streams the sequence's 64-position tiles of two tensors through two LDS stages.
struct DenseStream {
  const unsigned short *X0, *X1;
  const float *rows0, *rows1;  // optional per-position floats (wavefront 0 / 1 load them)
  char* stages;
  int stage_bytes, N, wave, lane;
  LoadLane ll;
  __device__ void issue(int t) {
    char* st = stages + (t & 1) * stage_bytes;
    const int p0 = min(t * BN + ll.row0, N - 1), p1 = min(t * BN + ll.row0 + 8, N - 1);
    issue_tile(X0, p0, p1, ll, st, wave);
    issue_tile(X1, p0, p1, ll, st + kTileBytes, wave);
    const float* rs = wave == 0 ? rows0 : wave == 1 ? rows1 : nullptr;
    if (rs) issue_row_words(rs, min(t * BN + lane, N - 1), st + kStage + 256 * wave);
  }
  // both stages: tiles 0 and 1
  __device__ void begin(int n_tiles) {
    issue(0);
    if (n_tiles > 1) issue(1);
  }
  // tile t is complete for every wavefront and the other stage is free: start loading tile t + 1
  __device__ const char* acquire(int t, int n_tiles) {
    wait_vmcnt_le(0);
    barrier_no_fence();
    if (t > 0 && t + 1 < n_tiles) issue(t + 1);
    return stages + (t & 1) * stage_bytes;
  }
};

// The dense-mask rule as a Mask of tile_bodies.h: the pair is kept iff the two tokens' codes say
// so.  `codes` points at the tile's 64 codes in LDS, offset by this lane half's 4 hl.
struct CodeMask {
  const unsigned* codes;
  unsigned my_code, limit;
  unsigned k[16];
  __device__ __forceinline__ CodeMask(const unsigned* tile_codes, int hl, unsigned code, unsigned limit_)
      : codes(tile_codes + 4 * hl), my_code(code), limit(limit_) {}
  __device__ __forceinline__ void load(int blk) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const uint4 kc = *reinterpret_cast<const uint4*>(codes + blk * 32 + 8 * g);
      k[4 * g] = kc.x; k[4 * g + 1] = kc.y; k[4 * g + 2] = kc.z; k[4 * g + 3] = kc.w;
    }
  }
  __device__ __forceinline__ bool full(int) const { return false; }
  __device__ __forceinline__ bool skip(int) const { return false; }
  __device__ __forceinline__ bool in(int c) const { return allowed(k[c], my_code, limit); }
  __device__ __forceinline__ float keep(int c, float x, float other) const { return in(c) ? x : other; }
};

// The same in the backward: lane 16 q + r owns rows r and 16 + r, `codes` is offset by 8 q.
struct PairCodeMask {
  const unsigned* codes;
  const RowPair &mine, &limit;
  unsigned k[8];
  __device__ __forceinline__ PairCodeMask(const unsigned* tile_codes, int q, const RowPair& mine_, const RowPair& limit_)
      : codes(tile_codes + 8 * q), mine(mine_), limit(limit_) {}
  __device__ __forceinline__ bool full(int) const { return false; }
  __device__ __forceinline__ bool skip(int) const { return false; }
  __device__ __forceinline__ void load_pairs(int blk) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint4 kc = *reinterpret_cast<const uint4*>(codes + blk * 32 + 4 * h);
      k[4 * h] = kc.x; k[4 * h + 1] = kc.y; k[4 * h + 2] = kc.z; k[4 * h + 3] = kc.w;
    }
  }
  __device__ __forceinline__ unsigned pair_mask(int cb, int i) const {
    return (allowed(k[2 * i], mine.v[cb], limit.v[cb]) ? 0xffffu : 0u) | (allowed(k[2 * i + 1], mine.v[cb], limit.v[cb]) ? 0xffff0000u : 0u);
  }
};
// Rows r and 16 + r of a wavefront's 32 owned positions from `first` on, as operands of 16 x 16 tiles.
__device__ __forceinline__ void dense_operands(const unsigned short* X, int first, int N, int lane, bf16x8 (&f)[2][2]) {
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      f[ks][cb] = *reinterpret_cast<const bf16x8*>(X + (unsigned)min(first + 16 * cb + (lane & 15), N - 1) * kD + 32 * ks + 8 * (lane >> 4));
}
// Results of pad positions, and of rows past the end, are zeros.
__device__ __forceinline__ void live_rows(QuadAcc& acc, float mul, const RowPair& live) {
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[d][i >> 2][i & 3] = live.v[i >> 2] ? acc[d][i >> 2][i & 3] * mul : 0.f;
}

// ======================================================================================
// forward
// ======================================================================================
template <bool kThrough>
__global__ __launch_bounds__(kThreads) void fwd_dense_kernel(const void* q, const void* k, const void* v, const int* row_ids,
                                                             const int* col_ids, const unsigned char* flags, int sizes, int pairs,
                                                             DenseArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds[2 * kStage];
  __shared__ __attribute__((aligned(16))) unsigned code[kDenseMaxN];
  __shared__ int q_tok[BM];
  const int N = sizes & 0xffff, H = sizes >> 16, tid = threadIdx.x, lane = tid & 63;
  DenseUnit u;
  if (!dense_unit(a, N, H, pairs, u)) return;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 31, hl = lane >> 5;
  const size_t bh = (size_t)u.bh * N;
  const unsigned short* Q = static_cast<const unsigned short*>(q) + bh * kD;
  const unsigned short* K = static_cast<const unsigned short*>(k) + bh * kD;
  const unsigned short* V = static_cast<const unsigned short*>(v) + bh * kD;
  unsigned short* O = static_cast<unsigned short*>(a.out) + bh * kD;

  DenseStream stream{K, V, nullptr, nullptr, lds, kStage, N, wave, lane, make_load_lane(wave, lane)};
  // everything in one round trip: the owned rows, the first two tiles, the codes.  (Whole owned rows, which the backward
  // loads, have to pass through the place of the second tile first: 8.5 -> 8.2 us for 32 x 128, 12 heads, but 16.8 -> 17.4 for
  // 64 x 128, 16 heads, and 4.8 -> 5.1 for one sequence of 64.)
  const int n_tiles = (N + BN - 1) / BN;
  const int pos = min(u.tile * BM + wave * 32 + m, N - 1);
  bf16x8 qf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    qf[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(Q + (size_t)pos * kD + ks * 16 + hl * 8));
  DenseCodes codes;
  codes.load(row_ids, col_ids, flags, u, N);
  stream.begin(n_tiles);
  codes.put(code, N);
  if (tid < BM) q_tok[tid] = u.tile * BM + tid < N ? u.tile * BM + tid : -1;
  __syncthreads();
  DenseRow me = dense_row(N, u, code, wave, m);
  if (me.limit == 0) me.limit = kPadCode;  // (padding meets anything: its results are replaced, and every row has a maximum)
  asm volatile("" ::"v"(qf[0]), "v"(qf[1]), "v"(qf[2]), "v"(qf[3]));

  const float sc = uniform(a.scale * kLog2e);
  f32x16 o_acc[2] = {zero16(), zero16()};
  float m_run = -INFINITY, l_run = 0.f;
  Reference ref = kMissing;
  const OperandLanes lanes(lane);
  const bool wave_active = u.tile * BM + wave * 32 < N;

  for (int t = 0; t < n_tiles; ++t) {
    const unsigned tile = lds_addr(stream.acquire(t, n_tiles));
    if (!wave_active) continue;
    fwd_tile(tile, qf, lanes, sc, CodeMask(code + t * BN, hl, me.code, me.limit), o_acc, m_run, l_run, ref);
  }
  __syncthreads();
  const float l_tot = half_sum(l_run);
  const bool live = me.in_range && me.code != kPadCode;  // pad positions: O = 0, LSE = 0
  if (hl == 0 && me.in_range)
    a.lse[bh + me.pos] = live ? (m_run * sc + __builtin_amdgcn_logf(l_tot)) * kLn2 : 0.f;
  const float inv = live ? 1.f / l_tot : 0.f;
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int c = 0; c < 16; ++c) o_acc[db][c] = live ? o_acc[db][c] * inv : 0.f;
  const f32x16 (*accs[1])[2] = {&o_acc};
  const float muls[1] = {1.f};
  unsigned short* const outs[1] = {O};
  store_owned_rows<1, kThrough>(accs, muls, outs, lds, q_tok, wave, lane);
}

// ======================================================================================
// forward of up to 128 positions, and of up to 192 where launch_fwd_dense says so
// ======================================================================================
// One workgroup per (sequence, head), whose keys and values are in LDS at once; wavefront w owns queries 16 w .. 16 w + 15.  All scores
// of a query are there before the first is used, so there is one maximum and nothing to rescale, and one barrier.  Like the backward
// below, such a launch is as long as a wavefront's own chain.
// us, before (128 queries a workgroup, 32 a wavefront) and so: 80 x 64 positions, 16 heads 9.1 -> 6.0, 24 x 33, 4 heads 4.1 -> 3.0, one sequence of 53
// 4.05 -> 3.05; 128 positions, 1 x, 4 heads 5.2 -> 4.55, 32 x, 12 heads 7.6 -> 6.85, 48 x 9.3 -> 8.5, 64 x 10.8 -> 9.7, 86 x 16.0 -> 15.3, 64 x, 16
// heads 14.4 -> 14.2, 128 x 24.65 -> 24.4; 64 x 100, 12 heads 9.6 -> 8.8.  With scores that rise late, where the form before starts tiles again, 32 x 128 8.7 -> 6.7.
template <int NW>
struct ShortShape {
  static constexpr int kRows = 16 * NW;                   // most positions
  static constexpr int kBlocks = kRows / 32;              // 32-row blocks
  static constexpr int kBytes = kRows * 128;              // of one tensor
  // Backward: K tiles | Q tiles | dO tiles | V tiles; dS^T, 64 queries a tile, comes over the last three
  static constexpr int kBwdLds = (1 + ((kBlocks + 1) / 2 > 3 ? (kBlocks + 1) / 2 : 3)) * kBytes;
};
// The rows of X to LDS, eight per instruction (rows past N repeat the last).
template <int NW>
__device__ __forceinline__ void stream_short(const unsigned short* X, const char* tile, int N, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int g = wave + i * NW, row = 8 * g + (lane >> 3), chunk = (lane & 7) ^ swz_quad(row);
    load_to_lds_16(X, (unsigned)min(row, N - 1) * 128u + chunk * 16, tile + g * 1024);
  }
}
// Sixteen result rows of a wavefront, scaled and rounded to bf16, through 2 KB of LDS that no other wavefront uses.  (Registers e
// of lane 16 q + r: dims 16 d + 4 q + e of row r.)  Pad positions: zeros, whatever was computed for them.
template <bool kThrough>
__device__ __forceinline__ void store_short(const f32x4 (&acc)[4], float mul, bool live, char* st, unsigned short* out, int own, int N, int lane) {
  const int r = lane & 15, q = lane >> 4;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    uint2 w = make_uint2(pack2(acc[d][0] * mul, acc[d][1] * mul), pack2(acc[d][2] * mul, acc[d][3] * mul));
    if (!live) w = make_uint2(0, 0);
    *reinterpret_cast<uint2*>(st + r * 128 + (((2 * d + (q >> 1)) ^ (r & 7)) << 4) + 8 * (q & 1)) = w;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // LDS keeps a wavefront's accesses in order
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int row = it * 8 + (lane >> 3), piece = lane & 7;
    const u32x4 v = *reinterpret_cast<const u32x4*>(st + row * 128 + ((piece ^ (row & 7)) << 4));
    if (own + row < N) ResultRows<kThrough>(out).store((unsigned)(own + row) * (kD * 2) + piece * 16, v);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
template <int NW, bool kThrough>
__global__ __launch_bounds__(64 * NW, 4) void fwd_dense_short_kernel(const void* q, const void* k, const void* v, const int* row_ids,
                                                                     const int* col_ids, const unsigned char* flags, int sizes, DenseArgs a) {
  using S = ShortShape<NW>;
  __shared__ __attribute__((aligned(1024))) char kt[S::kBytes], vt[S::kBytes];
  __shared__ __attribute__((aligned(16))) char rows[NW * 2048];
  __shared__ __attribute__((aligned(16))) unsigned code[S::kRows];
  const int N = sizes & 0xffff, tid = threadIdx.x, lane = tid & 63, bh_i = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, quarter = lane >> 4, own = 16 * wave, pos = min(own + r, N - 1);
  const size_t bh = (size_t)bh_i * N;
  int h;
  const int b = uniform_div_any(bh_i, sizes >> 16, h), view = head_view(a, h);
  const int f = flags[(size_t)b * N + pos], id = (pick(view == 0, row_ids, col_ids) + (size_t)b * N)[pos];
  const unsigned short* Q = static_cast<const unsigned short*>(q) + bh * kD;
  bf16x8 qf[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(Q + (unsigned)pos * kD + 32 * ks + 8 * quarter);
  stream_short<NW>(static_cast<const unsigned short*>(k) + bh * kD, kt, N, wave, lane);
  stream_short<NW>(static_cast<const unsigned short*>(v) + bh * kD, vt, N, wave, lane);
  const unsigned my_code = token_code(true, f, id);
  // (padding meets anything: its results are replaced, and every row has a maximum)
  const unsigned my_limit = my_code == 0u || my_code == kPadCode ? kPadCode : 1u;
  if (lane < 16) code[own + r] = own + r < N ? my_code : kPadCode;
  wait_vmcnt_le<0>(0);
  __syncthreads();
  if (own >= N) return;
  const float sc = uniform(a.scale * kLog2e);
  const QuadLanes lanes(lane);   // (an address for each block: one for all of a tensor takes up to 8 registers more here)
  const unsigned k_at = lds_addr(kt), v_at = lds_addr(vt);
  f32x4 s[S::kBlocks][2];  // S^T: keys 8 q + 4 h + e of the block, query r
  float mx = -INFINITY;
#pragma unroll
  for (int ib = 0; ib < S::kBlocks; ++ib)
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      if (ib * 32 >= N) continue;
      f32x4 x = mfma16(read_quad(QuadAddr(lanes, k_at + ib * kBlockBytes), 0, hb, 0), qf[0], f32x4{0.f, 0.f, 0.f, 0.f});
      // (Four wavefronts have no such instruction by themselves, and with this take 2 % longer, one sequence of 64, 4 heads 3.02 and 3.09 us.)
      const bf16x8 k1 = read_quad(QuadAddr(lanes, k_at + ib * kBlockBytes), 0, hb, 1);
      x = NW > 4 ? mfma16_apart(k1, qf[1], x) : mfma16(k1, qf[1], x);
      const uint4 c4 = *reinterpret_cast<const uint4*>(code + ib * 32 + 8 * quarter + 4 * hb);
      const unsigned codes[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = allowed(codes[e], my_code, my_limit) ? x[e] : -INFINITY;
      mx = fmaxf(fmaxf(mx, x[0]), x[1]);
      mx = fmaxf(fmaxf(mx, x[2]), x[3]);
      s[ib][hb] = x;
    }
  mx = quad_max(mx);
  const float msc = mx * sc;
  float l = 0.f;
  f32x4 acc[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ib = 0; ib < S::kBlocks; ++ib) {
    if (ib * 32 >= N) continue;
    unsigned w[4];
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      f32x4& x = s[ib][hb];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = __builtin_amdgcn_exp2f(fmaf(x[e], sc, -msc));
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        w[2 * hb + i] = pack2(x[2 * i], x[2 * i + 1]);
        l = sum2(w[2 * hb + i], l);
      }
    }
    const bf16x8 p8 = as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
#pragma unroll
    for (int d = 0; d < 4; ++d) acc[d] = mfma16(read_quad_transposed(QuadAddr(lanes, v_at + ib * kBlockBytes), 0, d), p8, acc[d]);   // O^T += V^T P^T
  }
  l = quad_sum(l);
  const bool live = my_code != kPadCode;  // pad positions: O = 0, LSE = 0
  if (lane < 16 && own + r < N) a.lse[bh + own + r] = live ? (msc + __builtin_amdgcn_logf(l)) * kLn2 : 0.f;
  store_short<kThrough>(acc, 1.f / l, live, rows + wave * 2048, static_cast<unsigned short*>(a.out) + bh * kD, own, N, lane);
}

// ======================================================================================
// dQ (and -delta, -lse / scale for the dK/dV kernel)
// ======================================================================================
__global__ __launch_bounds__(kThreads, 3) void bwd_dq_dense_kernel(DenseArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds[2 * kStage];
  __shared__ __attribute__((aligned(16))) unsigned code[kDenseMaxN];
  __shared__ int q_tok[BM];
  DenseUnit u;
  if (!dense_unit(a, a.N, a.H, a.B * a.H, u)) return;
  const int N = a.N, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 31;
  const size_t bh = (size_t)u.bh * N;
  const unsigned short* Q = static_cast<const unsigned short*>(a.q) + bh * kD;
  const unsigned short* K = static_cast<const unsigned short*>(a.k) + bh * kD;
  const unsigned short* V = static_cast<const unsigned short*>(a.v) + bh * kD;
  const unsigned short* O = static_cast<const unsigned short*>(a.o) + bh * kD;
  const unsigned short* dO = static_cast<const unsigned short*>(a.dout) + bh * kD;
  unsigned short* dQ = static_cast<unsigned short*>(a.dq) + bh * kD;

  DenseStream stream{K, V, nullptr, nullptr, lds, kStage, N, wave, lane, make_load_lane<true>(wave, lane)};
  const int n_tiles = (N + BN - 1) / BN;
  DenseCodes codes;
  codes.load(a.row_ids, a.col_ids, a.flags, u, N);
  stream.begin(n_tiles);
  codes.put(code, N);
  if (tid < BM) q_tok[tid] = u.tile * BM + tid < N ? u.tile * BM + tid : -1;
  __syncthreads();
  const DenseRow me = dense_row(N, u, code, wave, m);
  const int first = u.tile * BM + wave * 32;
  bf16x8 qf[2][2], gf[2][2], of[2][2];
  dense_operands(Q, first, N, lane, qf);
  dense_operands(dO, first, N, lane, gf);
  dense_operands(O, first, N, lane, of);
  const float lse = a.lse[bh + me.pos];
  asm volatile("" ::"v"(qf[0][0]), "v"(qf[0][1]), "v"(qf[1][0]), "v"(qf[1][1]), "v"(gf[0][0]), "v"(gf[0][1]), "v"(gf[1][0]),
               "v"(gf[1][1]), "v"(of[0][0]), "v"(of[0][1]), "v"(of[1][0]), "v"(of[1][1]), "v"(lse));
  f32x4 ndelta[2];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    float d = 0.f;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) d = fmaf((float)gf[ks][cb][e], (float)of[ks][cb][e], d);
    d = -quad_sum(d);
    ndelta[cb] = f32x4{d, d, d, d};
  }
  if (lane < 32 && me.in_range) {   // (lane m < 32: row m)
    a.delta[bh + me.pos] = pick(lane < 16, ndelta[0][0], ndelta[1][0]);
    a.nlse[bh + me.pos] = -lse / a.scale;
  }
  const RowPair l = row_pair(__float_as_uint(lse * kLog2e)), mine = row_pair(me.code), limit = row_pair(me.limit);
  const float lse2[2] = {__uint_as_float(l.v[0]), __uint_as_float(l.v[1])}, sc = a.scale * kLog2e;
  const QuadLanes lanes(lane);
  const bool wave_active = u.tile * BM + wave * 32 < N;

  QuadAcc dq_acc = {};
  for (int t = 0; t < n_tiles; ++t) {
    const unsigned tile = lds_addr(stream.acquire(t, n_tiles));
    if (!wave_active) continue;
    dq_tile(tile, qf, gf, lanes, sc, lse2, ndelta, PairCodeMask(code + t * BN, lane >> 4, mine, limit), dq_acc);
  }
  __syncthreads();
  live_rows(dq_acc, a.scale, row_pair(me.in_range && me.code != kPadCode));
  const QuadAcc* accs[1] = {&dq_acc};
  const float muls[1] = {1.f};
  unsigned short* const outs[1] = {dQ};
  store_owned_rows<1>(accs, muls, outs, lds, q_tok, wave, lane);
}

// ======================================================================================
// dK, dV
// ======================================================================================
// (168 registers, three workgroups a compute unit; left to itself the compiler takes 182: 16 x 384, 16 heads, both kernels, 47.6 and 52.7 us)
__global__ __launch_bounds__(kThreads, 3) void bwd_dkv_dense_kernel(DenseArgs a) {
  __shared__ __attribute__((aligned(1024))) char lds[2 * kDkvStageD];
  __shared__ __attribute__((aligned(16))) unsigned code[kDenseMaxN];
  __shared__ int k_tok[BM];
  DenseUnit u;
  if (!dense_unit(a, a.N, a.H, a.B * a.H, u)) return;
  const int N = a.N, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 31;
  const size_t bh = (size_t)u.bh * N;
  const unsigned short* Q = static_cast<const unsigned short*>(a.q) + bh * kD;
  const unsigned short* K = static_cast<const unsigned short*>(a.k) + bh * kD;
  const unsigned short* V = static_cast<const unsigned short*>(a.v) + bh * kD;
  const unsigned short* dO = static_cast<const unsigned short*>(a.dout) + bh * kD;
  unsigned short* dK = static_cast<unsigned short*>(a.dk) + bh * kD;
  unsigned short* dV = static_cast<unsigned short*>(a.dv) + bh * kD;

  DenseStream stream{Q, dO, a.nlse + bh, a.delta + bh, lds, kDkvStageD, N, wave, lane,
                     make_load_lane<true>(wave, lane)};
  const int n_tiles = (N + BN - 1) / BN;
  DenseCodes codes;
  codes.load(a.row_ids, a.col_ids, a.flags, u, N);
  stream.begin(n_tiles);
  codes.put(code, N);
  if (tid < BM) k_tok[tid] = u.tile * BM + tid < N ? u.tile * BM + tid : -1;
  __syncthreads();
  const DenseRow me = dense_row(N, u, code, wave, m);  // this lane's key
  bf16x8 kf[2][2], vf[2][2];
  dense_operands(K, u.tile * BM + wave * 32, N, lane, kf);
  dense_operands(V, u.tile * BM + wave * 32, N, lane, vf);
  asm volatile("" ::"v"(kf[0][0]), "v"(kf[0][1]), "v"(kf[1][0]), "v"(kf[1][1]), "v"(vf[0][0]), "v"(vf[0][1]), "v"(vf[1][0]),
               "v"(vf[1][1]));
  const float sc = uniform(a.scale * kLog2e);
  const QuadLanes lanes(lane);
  const RowPair mine = row_pair(me.code), limit = row_pair(me.limit);
  const bool wave_active = u.tile * BM + wave * 32 < N;

  QuadAcc dk_acc = {}, dv_acc = {};
  for (int t = 0; t < n_tiles; ++t) {
    const char* Qst = stream.acquire(t, n_tiles);
    const float* lse_row = reinterpret_cast<const float*>(Qst + kStage);
    const float* delta_row = lse_row + BN;
    if (!wave_active) continue;
    dkv_tile(lds_addr(Qst), lse_row, delta_row, kf, vf, lanes, sc, lane >> 4, PairCodeMask(code + t * BN, lane >> 4, mine, limit), dk_acc, dv_acc);
  }
  __syncthreads();
  const RowPair live = row_pair(me.in_range && me.code != kPadCode);
  live_rows(dk_acc, a.scale, live);
  live_rows(dv_acc, 1.f, live);
  const QuadAcc* accs[2] = {&dk_acc, &dv_acc};
  const float muls[2] = {1.f, 1.f};
  unsigned short* const outs[2] = {dK, dV};
  store_owned_rows<2>(accs, muls, outs, lds, k_tok, wave, lane);
}

// ======================================================================================
// Backward of up to 256 positions in one launch
// ======================================================================================
// One workgroup per (sequence, head) that meets every pair, so S and dP are computed once for all three gradients (the two
// kernels above compute them twice, and of their 13 us each at B = 32, H = 12, N = 128 five are the launch): a wavefront's dK and dV
// accumulate in registers, the bf16 dS^T goes through LDS, and dQ^T = K^T dS^T with both operands read transposed (both permute
// the keys of a slice the same way).
//
// Here for 193 to 256 positions: wavefront w owns keys 32 w .. 32 w + 31, and queries come in two passes of 128.  (Shorter
// sequences: bwd_dense_short_kernel.)
//
// Per-lane LDS offsets of the operand reads: plain 16-byte reads for the four 16-wide k slices,
// transposing reads for the two 32-row blocks of the other operand (see d2l.h).
__device__ __forceinline__ void operand_offsets(int lane, int (&poff)[4], int (&toff)[2][2]) {
  const int m = lane & 31, hl = lane >> 5;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) poff[ks] = plain_off(m, hl, ks);
#pragma unroll
  for (int db = 0; db < 2; ++db) {
    toff[db][0] = tr_off(lane, db, 0);
    toff[db][1] = tr_off(lane, db, 1);
  }
}
struct SmallShape {
  static constexpr int kWaves = 8, kKeys = 32 * kWaves;  // most positions
  static constexpr int kBlocks = 4, kQueries = 32 * kBlocks, kPasses = 2;  // 32-query blocks of a pass
  static constexpr int kKeyBytes = kKeys * 128, kQryBytes = kQueries * 128;
  // K tiles | Q tiles | dO tiles | V tiles, then dS^T; dQ rows are staged over the Q tiles, dK and dV rows over the K tiles
  static constexpr int kLds = kKeyBytes + 2 * kQryBytes + kKeys * kQueries * 2;
};
template <bool kThrough>
__global__ __launch_bounds__(64 * SmallShape::kWaves, 2) void bwd_dense_small_kernel(
    const void* q, const void* k, const void* v, const void* o, const void* dout, int sizes, DenseArgs a) {
  using S = SmallShape;
  constexpr int NW = S::kWaves;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  __shared__ __attribute__((aligned(16))) unsigned code[S::kKeys];
  __shared__ __attribute__((aligned(16))) float nlse[S::kKeys], ndelta[S::kKeys];
  char *const kt = lds, *const qt = lds + S::kKeyBytes, *const gt = qt + S::kQryBytes;
  char *const vt = gt + S::kQryBytes, *const ds = vt;
  const int N = sizes & 0xffff, tid = threadIdx.x, lane = tid & 63, bh_i = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 31, hl = lane >> 5;
  const size_t bh = (size_t)bh_i * N;
  const unsigned short* Q = static_cast<const unsigned short*>(q) + bh * kD;
  const unsigned short* K = static_cast<const unsigned short*>(k) + bh * kD;
  const unsigned short* V = static_cast<const unsigned short*>(v) + bh * kD;
  const unsigned short* O = static_cast<const unsigned short*>(o) + bh * kD;
  const unsigned short* dO = static_cast<const unsigned short*>(dout) + bh * kD;
  unsigned short* dQ = static_cast<unsigned short*>(a.dq) + bh * kD;
  unsigned short* dK = static_cast<unsigned short*>(a.dk) + bh * kD;
  unsigned short* dV = static_cast<unsigned short*>(a.dv) + bh * kD;

  int h;
  const int b = uniform_div_any(bh_i, sizes >> 16, h), view = head_view(a, h);
  const int *row_ids = a.row_ids, *col_ids = a.col_ids;
  const unsigned char* flags = a.flags;
  // rows [first, first + rows) of X to LDS, eight per instruction (rows past N repeat the last)
  auto stream_rows = [&](const unsigned short* X, int first, auto rows, const char* tile) {
    static_assert(decltype(rows)::value % (8 * NW) == 0, "the wavefronts share the rows evenly");
#pragma unroll
    for (int i = 0; i < decltype(rows)::value / (8 * NW); ++i) {
      const int g = wave + i * NW, row = 8 * g + (lane >> 3), chunk = (lane & 7) ^ swz(row & 15);
      load_to_lds_16(X, (unsigned)min(first + row, N - 1) * 128u + chunk * 16, tile + g * 1024);
    }
  };
  const std::integral_constant<int, S::kKeys> keys;
  const std::integral_constant<int, S::kQueries> queries;
  stream_rows(K, 0, keys, kt);
  stream_rows(Q, 0, queries, qt);
  stream_rows(dO, 0, queries, gt);

  stream_rows(V, 0, keys, vt);

  // of this lane's row: delta and -lse / scale of the query, and the code.  (All rows are loaded whole, eight per
  // instruction.  With key, value, dO and O operands straight from global memory, sixteen loads that touch 32 lines each: 8 x 256,
  // 12 heads 20.4 us, now 18.1.)
  const int pos = min(32 * wave + m, N - 1);
  {
    OwnedTile g_rows, o_rows;
    g_rows.load(dO, pos, lane);
    o_rows.load(O, pos, lane);
    const float lse = a.lse[bh + pos];
    const int* ids = pick(view == 0, row_ids, col_ids) + (size_t)b * N;
    const int f = flags[(size_t)b * N + pos], id = ids[pos];
    const float delta = row_delta(g_rows, o_rows, reinterpret_cast<char*>(ndelta + 32 * wave), lane);
    if (hl == 0) {
      nlse[32 * wave + m] = -lse / a.scale;
      ndelta[32 * wave + m] = -delta;
      code[32 * wave + m] = token_code(32 * wave + m < N, f, id);
    }
  }
  bf16x8 kf[4], vf[4];  // this lane's key and value as B operands
  const float sc = uniform(a.scale * kLog2e);
  int poff[4], toff[2][2];
  operand_offsets(lane, poff, toff);
  const int n_blocks = (N + 31) / 32;  // wavefronts that own keys, and query blocks
  const bool active = wave < n_blocks;
  f32x16 dk_acc[2] = {zero16(), zero16()}, dv_acc[2] = {zero16(), zero16()};

  for (int p = 0; p < S::kPasses; ++p) {
    if (p > 0) {
      __syncthreads();  // the staged dQ rows of the pass before have been stored
      stream_rows(Q, p * S::kQueries, queries, qt);
      stream_rows(dO, p * S::kQueries, queries, gt);
    }
    wait_vmcnt_le<0>(0);
    __syncthreads();
    if (p == 0)  // (dS^T may come where V is, but of each wavefront over its own rows)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        kf[ks] = read_plain(kt + wave * 32 * 128, poff[ks]);
        vf[ks] = read_plain(vt + wave * 32 * 128, poff[ks]);
      }
    bf16x8 ds8[S::kBlocks][2];
    const unsigned my_code = code[32 * wave + m], my_limit = owner_limit(my_code);
    if (active)
#pragma unroll
      for (int ib = 0; ib < S::kBlocks; ++ib) {
        const int q0 = (p * S::kBlocks + ib) * 32;
        if (q0 >= N) continue;
        f32x16 s, dp;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 l4 = *reinterpret_cast<const float4*>(nlse + q0 + 8 * g + 4 * hl);
          const float4 d4 = *reinterpret_cast<const float4*>(ndelta + q0 + 8 * g + 4 * hl);
          s[4 * g] = l4.x; s[4 * g + 1] = l4.y; s[4 * g + 2] = l4.z; s[4 * g + 3] = l4.w;
          dp[4 * g] = d4.x; dp[4 * g + 1] = d4.y; dp[4 * g + 2] = d4.z; dp[4 * g + 3] = d4.w;
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          s = mfma(read_plain(qt + ib * 32 * 128, poff[ks]), kf[ks], s);     // S  = Q K^T
          dp = mfma(read_plain(gt + ib * 32 * 128, poff[ks]), vf[ks], dp);   // dP = dO V^T
        }
        CodeMask mask(code + q0, hl, my_code, my_limit);
        mask.load(0);
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          const bool in = mask.in(c);
          s[c] = in ? __builtin_amdgcn_exp2f(s[c] * sc) : 0.f;   // P
          dp[c] = in ? s[c] * dp[c] : 0.f;                       // dS
        }
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
          const bf16x8 p8 = pack8(s, 8 * tt);
          ds8[ib][tt] = pack8(dp, 8 * tt);
          const char *gr = gt + (ib * 32 + tt * 16) * 128, *qr = qt + (ib * 32 + tt * 16) * 128;
#pragma unroll
          for (int db = 0; db < 2; ++db) {
            dv_acc[db] = mfma(read_transposed(gr, toff[db][0], toff[db][1]), p8, dv_acc[db]);          // dV^T += dO^T P
            dk_acc[db] = mfma(read_transposed(qr, toff[db][0], toff[db][1]), ds8[ib][tt], dk_acc[db]);  // dK^T += Q^T dS
          }
        }
      }
    // dS^T: row = key, 64 queries per 128-byte row and tile, swizzled like the other tiles
    if (active)
#pragma unroll
      for (int ib = 0; ib < S::kBlocks; ++ib)
        if ((p * S::kBlocks + ib) * 32 < N)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            union { bf16x8 v; uint2 h[2]; } x;
            x.v = ds8[ib][g >> 1];
            const int row = 32 * wave + m, chunk = 4 * (ib & 1) + g;
            *reinterpret_cast<uint2*>(ds + (ib >> 1) * S::kKeys * 128 + row * 128 + ((chunk ^ swz(row & 15)) << 4) + 8 * hl) =
                x.h[g & 1];
          }
    __syncthreads();
    // dQ: 32 dims (block db) of query block qb
    const int qb = wave % S::kBlocks, db = wave / S::kBlocks;
    const bool has_block = (p * S::kBlocks + qb) * 32 < N;
    f32x16 dq_acc = zero16();
    if (has_block) {
      const char* dst = ds + (qb >> 1) * S::kKeys * 128;
      const int q_lo = qb & 1 ? toff[1][0] : toff[0][0], q_hi = qb & 1 ? toff[1][1] : toff[0][1];
      const int d_lo = db ? toff[1][0] : toff[0][0], d_hi = db ? toff[1][1] : toff[0][1];
      for (int kb = 0; kb < n_blocks; ++kb)
#pragma unroll
        for (int kk = 2 * kb; kk < 2 * kb + 2; ++kk) {
          const bf16x8 dsq = read_transposed(dst + kk * 16 * 128, q_lo, q_hi);
          dq_acc = mfma(read_transposed(kt + kk * 16 * 128, d_lo, d_hi), dsq, dq_acc);
        }
    }
    if (has_block) {
      const int q = (p * S::kBlocks + qb) * 32 + m;
      const bool live_q = code[q] != kPadCode;  // pad positions: zeros, whatever their rows held
      stage_rows(live_q ? dq_acc : zero16(), a.scale, qt, qb * 32 + m, db, hl);
    }
    __syncthreads();
    for (int g = wave; g < S::kQueries / 8; g += NW) {
      const int row = 8 * g + (lane >> 3), piece = lane & 7, q = p * S::kQueries + row;
      if (q < N) *reinterpret_cast<uint4*>(dQ + (size_t)q * kD + piece * 8) =
          *reinterpret_cast<const uint4*>(qt + row * 128 + ((piece ^ (row & 7)) << 4));
    }
  }
  __syncthreads();
  // dK, dV rows of this wavefront's keys, staged one after the other over its own rows of the K tiles:
  // nobody else touches them, and LDS keeps a wavefront's accesses in order
  if (!active) return;
  char* const st = kt + wave * 32 * 128;
  const bool live = code[32 * wave + m] != kPadCode;
  const auto flush = [&](unsigned short* out) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int row = it * 8 + (lane >> 3), piece = lane & 7, k = 32 * wave + row;
      const u32x4 v = *reinterpret_cast<const u32x4*>(st + row * 128 + ((piece ^ (row & 7)) << 4));
      if (k < N) ResultRows<kThrough>(out).store((unsigned)k * (kD * 2) + piece * 16, v);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
#pragma unroll
  for (int db = 0; db < 2; ++db) stage_rows(live ? dk_acc[db] : zero16(), a.scale, st, m, db, hl);
  flush(dK);
#pragma unroll
  for (int db = 0; db < 2; ++db) stage_rows(live ? dv_acc[db] : zero16(), 1.f, st, m, db, hl);
  flush(dV);
}

// The same for up to 192 positions: sixteen keys a wavefront in place of 32, in 16 x 16 x 32 instructions, all queries in one pass, and no
// barrier after dQ's.  Such a launch is one or two workgroups on a compute unit that load, compute and store at the same time, so it is
// as long as a wavefront's own chain, which is half as long here.  Every wavefront reads all of Q and dO, plain and transposed, so LDS
// reads double, and from 193 positions on those bound it (14 wavefronts: 1 x 224, 12 heads 15.4 -> 15.7, 32 x 224 35.5 -> 36.8).
// LDS banks: dS^T goes in by rows whose swizzle does not know bit 2, so those writes and the staged results meet in banks, 0.75 cycles per LDS instruction.
// us, 32 keys a wavefront and sixteen: 80 x 64 positions, 16 heads 17.7 -> 14.6, 64 x 64 13.3 -> 11.7, 48 x 64 9.4 -> 7.4, 17 x 64 7.4 -> 5.6, one sequence of 64,
// 4 heads 5.7 -> 4.25; 128 positions, 1 x, 4 heads 7.6 -> 7.0, 32 x, 12 heads 12.85 -> 11.75, 48 x 20.0 -> 18.6, 64 x, 16 heads
// 27.7 -> 26.1, 128 x 49.0 -> 48.6; 40 x 96, 16 heads 16.7 -> 14.4; 8 x 160, 12 heads 12.6 -> 10.1, 40 x 160, 16 heads 41.9 -> 35.9; 8 x 192, 12 heads 14.0 -> 12.1, 40 x 192, 16 heads
// 47.8 -> 43.7.
template <int NW, bool kThrough>
__global__ __launch_bounds__(64 * NW, 4) void bwd_dense_short_kernel(
    const void* q, const void* k, const void* v, const void* o, const void* dout, int sizes, DenseArgs a) {
  using S = ShortShape<NW>;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  __shared__ __attribute__((aligned(16))) unsigned code[S::kRows];
  __shared__ __attribute__((aligned(16))) float nlse[S::kRows], ndelta[S::kRows];
  char *const kt = lds, *const qt = lds + S::kBytes, *const gt = qt + S::kBytes, *const vt = gt + S::kBytes, *const ds = qt;
  const int N = sizes & 0xffff, tid = threadIdx.x, lane = tid & 63, bh_i = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, quarter = lane >> 4, q8 = 8 * quarter;
  const size_t bh = (size_t)bh_i * N;
  const unsigned short* Q = static_cast<const unsigned short*>(q) + bh * kD;
  const unsigned short* K = static_cast<const unsigned short*>(k) + bh * kD;
  const unsigned short* V = static_cast<const unsigned short*>(v) + bh * kD;
  const unsigned short* O = static_cast<const unsigned short*>(o) + bh * kD;
  const unsigned short* dO = static_cast<const unsigned short*>(dout) + bh * kD;
  unsigned short* dQ = static_cast<unsigned short*>(a.dq) + bh * kD;
  unsigned short* dK = static_cast<unsigned short*>(a.dk) + bh * kD;
  unsigned short* dV = static_cast<unsigned short*>(a.dv) + bh * kD;

  int h;
  const int b = uniform_div_any(bh_i, sizes >> 16, h), view = head_view(a, h);
  const int *row_ids = a.row_ids, *col_ids = a.col_ids;
  const unsigned char* flags = a.flags;
  stream_short<NW>(K, kt, N, wave, lane);
  stream_short<NW>(Q, qt, N, wave, lane);
  stream_short<NW>(dO, gt, N, wave, lane);
  stream_short<NW>(V, vt, N, wave, lane);

  // of this wavefront's rows: delta and -lse / scale of the queries, and the codes
  const int own = 16 * wave;
  {
    bf16x8 g[2], y[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned at = (unsigned)min(own + 8 * i + (lane >> 3), N - 1) * kD + 8 * (lane & 7);
      g[i] = *reinterpret_cast<const bf16x8*>(dO + at);
      y[i] = *reinterpret_cast<const bf16x8*>(O + at);
    }
    const int pos = min(own + r, N - 1);
    const float lse = a.lse[bh + pos];
    const int* ids = pick(view == 0, row_ids, col_ids) + (size_t)b * N;
    const int f = flags[(size_t)b * N + pos], id = ids[pos];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float d = row_dot8(g[i], y[i]);
      if ((lane & 7) == 0) ndelta[own + 8 * i + (lane >> 3)] = -d;
    }
    if (lane < 16) {
      nlse[own + r] = -lse / a.scale;
      code[own + r] = token_code(own + r < N, f, id);
    }
  }
  bf16x8 kf[2], vf[2];  // this lane's key and value as B operands
  const float sc = uniform(a.scale * kLog2e);
  const QuadLanes lanes(lane);
  const unsigned q_at = lds_addr(qt), g_at = lds_addr(gt), k_at = lds_addr(kt), ds_at = lds_addr(ds);
  // the wavefront owns a key, or its rows of dS^T are met together with those of one that does
  const bool active = (own & ~31) < N;
  f32x4 dk_acc[4], dv_acc[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) dk_acc[d] = dv_acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};

  wait_vmcnt_le<0>(0);
  __syncthreads();
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int row = own + r, at = row * 128 + (((4 * ks + quarter) ^ swz_quad(row)) << 4);
    kf[ks] = read_plain(kt, at);
    vf[ks] = read_plain(vt, at);
  }
  unsigned dw[S::kBlocks][4];   // dS of the block's queries 8 q .. 8 q + 7
  const unsigned my_code = code[own + r], my_limit = owner_limit(my_code);
  if (active)
#pragma unroll
    for (int ib = 0; ib < S::kBlocks; ++ib) {
      const int q0 = ib * 32;
      if (q0 >= N) continue;
      unsigned pw[4];
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        f32x4 s = *reinterpret_cast<const f32x4*>(nlse + q0 + q8 + 4 * hb), dp = *reinterpret_cast<const f32x4*>(ndelta + q0 + q8 + 4 * hb);
        const uint4 c4 = *reinterpret_cast<const uint4*>(code + q0 + q8 + 4 * hb);
        const unsigned codes[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          s = mfma16(read_quad(QuadAddr(lanes, q_at + ib * kBlockBytes), 0, hb, ks), kf[ks], s);     // S  = Q K^T
          dp = mfma16(read_quad(QuadAddr(lanes, g_at + ib * kBlockBytes), 0, hb, ks), vf[ks], dp);   // dP = dO V^T
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool in = allowed(codes[e], my_code, my_limit);
          s[e] = in ? __builtin_amdgcn_exp2f(s[e] * sc) : 0.f;   // P
          dp[e] = in ? s[e] * dp[e] : 0.f;                       // dS
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          pw[2 * hb + i] = pack2(s[2 * i], s[2 * i + 1]);
          dw[ib][2 * hb + i] = pack2(dp[2 * i], dp[2 * i + 1]);
        }
      }
      const bf16x8 p8 = as_bf16x8(make_uint4(pw[0], pw[1], pw[2], pw[3]));
      const bf16x8 ds8 = as_bf16x8(make_uint4(dw[ib][0], dw[ib][1], dw[ib][2], dw[ib][3]));
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        dv_acc[d] = mfma16(read_quad_transposed(QuadAddr(lanes, g_at + ib * kBlockBytes), 0, d), p8, dv_acc[d]);   // dV^T += dO^T P
        dk_acc[d] = mfma16(read_quad_transposed(QuadAddr(lanes, q_at + ib * kBlockBytes), 0, d), ds8, dk_acc[d]);  // dK^T += Q^T dS
      }
    }
  __syncthreads();  // everyone is done with the Q and dO tiles, and with its own rows of V
  // dS^T: row = key, 64 queries per 128-byte row and tile, swizzled like the other tiles
  if (active)
#pragma unroll
    for (int ib = 0; ib < S::kBlocks; ++ib)
      if (ib * 32 < N) {
        const int row = own + r, chunk = 4 * (ib & 1) + quarter;
        *reinterpret_cast<uint4*>(ds + (ib >> 1) * S::kBytes + row * 128 + ((chunk ^ swz_quad(row)) << 4)) =
            make_uint4(dw[ib][0], dw[ib][1], dw[ib][2], dw[ib][3]);
      }
  __syncthreads();
  // dQ of this wavefront's queries
  f32x4 dq_acc[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) dq_acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (own < N)
    for (int kb = 0; kb * 32 < N; ++kb) {
      const bf16x8 dsq = read_quad_transposed(QuadAddr(lanes, ds_at + (wave >> 2) * S::kBytes + kb * kBlockBytes), 0, wave & 3);
#pragma unroll
      for (int d = 0; d < 4; ++d) dq_acc[d] = mfma16(read_quad_transposed(QuadAddr(lanes, k_at + kb * kBlockBytes), 0, d), dsq, dq_acc[d]);
    }
  __syncthreads();  // dS^T and the K tiles have been read
  // Result rows of this wavefront, staged one tensor after the other over its own rows of the K tiles.
  if (own >= N) return;
  char* const st = kt + own * 128;
  const bool live = code[own + r] != kPadCode;
  store_short<kThrough>(dq_acc, a.scale, live, st, dQ, own, N, lane);
  store_short<kThrough>(dk_acc, a.scale, live, st, dK, own, N, lane);
  store_short<kThrough>(dv_acc, 1.f, live, st, dV, own, N, lane);
}

template <int NW, bool kThrough>
hipError_t launch_fwd_short(const DenseArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL((fwd_dense_short_kernel<NW, kThrough>), dim3(a.B * a.H), dim3(64 * NW), 0, stream, a.q, a.k, a.v, a.row_ids, a.col_ids,
                     a.flags, pack_sizes(a.N, a.H), a);
  return hipGetLastError();
}
template <int NW, bool kThrough>
hipError_t launch_bwd_short(const DenseArgs& a, hipStream_t stream) {
  const hipError_t e = allow_lds<&bwd_dense_short_kernel<NW, kThrough>>(ShortShape<NW>::kBwdLds);
  if (e != hipSuccess) return e;
  ProfileScope prof(7, stream, 6);
  hipLaunchKernelGGL((bwd_dense_short_kernel<NW, kThrough>), dim3(a.B * a.H), dim3(64 * NW), ShortShape<NW>::kBwdLds, stream, a.q, a.k, a.v, a.o,
                     a.dout, pack_sizes(a.N, a.H), a);
  return hipGetLastError();
}
template <bool kThrough>
hipError_t launch_bwd_small(const DenseArgs& a, hipStream_t stream) {
  const hipError_t e = allow_lds<&bwd_dense_small_kernel<kThrough>>(SmallShape::kLds);
  if (e != hipSuccess) return e;
  ProfileScope prof(7, stream, 6);
  hipLaunchKernelGGL((bwd_dense_small_kernel<kThrough>), dim3(a.B * a.H), dim3(64 * SmallShape::kWaves), SmallShape::kLds, stream, a.q, a.k,
                     a.v, a.o, a.dout, pack_sizes(a.N, a.H), a);
  return hipGetLastError();
}
template <bool kThrough>
hipError_t launch_bwd_one(const DenseArgs& a, hipStream_t stream) {
  return a.N <= 64    ? launch_bwd_short<4, kThrough>(a, stream)
         : a.N <= 128 ? launch_bwd_short<8, kThrough>(a, stream)
         : a.N <= 160 ? launch_bwd_short<10, kThrough>(a, stream)
         : a.N <= 192 ? launch_bwd_short<12, kThrough>(a, stream)
                      : launch_bwd_small<kThrough>(a, stream);
}

}  // namespace

hipError_t launch_fwd_dense(const DenseArgs& a, hipStream_t stream) {
  ProfileScope prof(5, stream);
  // The short form: up to 128 positions, and up to 192 where the general one has more workgroups than compute units and it has not (us,
  // 16 heads: 16 x 160 8.65 -> 6.65, 16 x 192 8.7 -> 7.35; 8 x 192, 12 heads 6.6 -> 7.3, 24 x 192 10.9 -> 10.75, 40 x 192, 16 heads 17.2 -> 17.2).
  const bool through = result_through(a.B, a.H, a.N, 2);
  if (a.N <= 64) return through ? launch_fwd_short<4, true>(a, stream) : launch_fwd_short<4, false>(a, stream);
  if (a.N <= 128) return through ? launch_fwd_short<8, true>(a, stream) : launch_fwd_short<8, false>(a, stream);
  if (a.N <= 192 && a.B * a.H > 128 && a.B * a.H <= 256)
    return through ? launch_fwd_short<12, true>(a, stream) : launch_fwd_short<12, false>(a, stream);
  const auto kernel = through ? fwd_dense_kernel<true> : fwd_dense_kernel<false>;
  hipLaunchKernelGGL(kernel, dim3(dense_grid(a)), dim3(kThreads), 0, stream, a.q, a.k, a.v, a.row_ids, a.col_ids, a.flags,
                     pack_sizes(a.N, a.H), a.B * a.H, a);
  return hipGetLastError();
}

hipError_t launch_bwd_dense(const DenseArgs& a, hipStream_t stream) {
  // one workgroup per (sequence, head) as long as its dS^T and K fit the LDS; the length says which kernel: see there
  const bool through = result_through(a.B, a.H, a.N, 3 * 2);
  if (a.N <= SmallShape::kKeys) return through ? launch_bwd_one<true>(a, stream) : launch_bwd_one<false>(a, stream);
  {
    ProfileScope prof(6, stream);
    hipLaunchKernelGGL(bwd_dq_dense_kernel, dim3(dense_grid(a)), dim3(kThreads), 0, stream, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  ProfileScope prof(7, stream);
  hipLaunchKernelGGL(bwd_dkv_dense_kernel, dim3(dense_grid(a)), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace mate
