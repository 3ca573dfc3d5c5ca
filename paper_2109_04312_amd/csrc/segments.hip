// Segment builder: the per-head-kind reordering of Section 3.1 (row-order / column-order
// traversal of the table tokens), computed as a stable sort of the table-token positions by id
// plus run boundaries.  Integer work only; all sorting lives in LDS.
//
// Two ways, chosen on the device from the ids themselves:
//   * ids all below 512 (every row and column number of a real table): the order is a counting
//     sort, slot(p) = first slot of id_p + number of earlier table tokens with the same id, and
//     everything else (segments, windows, work units) follows from the histogram of ids.  Up to
//     eight workgroups share a (sequence, view): each reads the whole sequence (a few KB),
//     builds the histogram and the part of it that lies before its own chunk of positions, and
//     ranks and writes only its chunk; one more workgroup has no chunk and lists the work units
//     instead (the longest single piece of work after the histogram).  Nothing is exchanged
//     between workgroups.
//   * otherwise workgroup 0 of the (sequence, view) sorts alone, as described next.
//
// Sort: table-token positions are first compacted in ascending order, then reordered by a
// least-significant-digit radix sort on their id, 9 bits per pass.  Each pass is stable (every
// wavefront owns a contiguous block of the current order, counts its digits, and ranks equal
// digits inside a 64-element batch in lane order with ballots), so ties keep ascending position.
// Passes whose digit is zero for every id are skipped: ids below 512 cost one pass.
//
// The kernel also lists the work units of the attention kernels per (sequence, view): pieces of
// up to 128 slots of the sorted order (cut so that none straddles the boundary of a long
// segment, listed longest streamed side first) with the window of sorted slots their segments
// span, then the pad tiles, and per sequence the chunks of the question-token owners.  The
// attention kernels map a workgroup index to one of these records with arithmetic alone.
//
// What bounds it: latency, not traffic -- load, classify, scan, rank, store, with a workgroup barrier
// between each.  So the counters are cleared while the inputs travel, prefix sums are DPP moves
// (six dependent shuffles were 2 us of the kernel), ids and segments are counted in one scan, and the
// classification, which the instruction issue bounds, takes four elements per lane.  us per launch in a row of
// them, against the version without these: one sequence of 128 positions 8.6 -> 5.0, of 512 9.3 -> 5.6, of 1999
// 10.3 -> 7.0, two of 8192 14.3 -> 11.0.  Since then a lane's inputs are one load each and leave before anything else is
// worked out (sequence_loads.h), all arguments arrive in registers, a slot's window is written by the token that takes the
// slot (it knows its segment; a binary search per slot before), and the unit list finds its segments in three rounds
// of reads instead of nine, in one wavefront without a barrier where it is short: 5.1 -> 4.3, 5.6 -> 4.4, 7.1 -> 5.4, 11.0 -> 9.1, one sequence of 16384 16.9 -> 13.7.
//
// Bucketed mode (the approximation of Section 3.1: a global part of at most G tokens, the rest
// of the head's order in buckets of R, a bucket meeting itself and its two neighbours): the
// question tokens past the first `max_global` are classified as table tokens, and every slot's
// window is its segment cut to the slots of buckets j - 1 .. j + 1 of its own bucket j.  The
// attention kernels read windows only, so the mode lives entirely in these tables.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "launch.h"
#include "seg_layout.h"
#include "sequence_loads.h"

namespace mate {

constexpr int kSegChunk = 1024;             // positions per workgroup, about
constexpr int kDigitBits = 9;               // radix digit: ids below 512 sort in one pass
constexpr unsigned kBins = 1u << kDigitBits;

// Workgroup barrier for data exchanged through LDS only: waits for this wavefront's LDS traffic,
// not for its global stores (a full fence would stall every phase on store round trips; nothing
// the kernel writes to global memory is read back inside it).
__device__ inline void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Inclusive prefix sums with DPP moves (a shuffle is a round trip through the LDS unit): over each row of
// sixteen lanes, and over the wavefront.
__device__ inline int row_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111 /* row_shr:1 */, 0xf, 0xf, false);  // lanes without a source add 0
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  return v;
}
__device__ inline int wave_scan(int v) {
  v = row_scan(v);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142 /* row_bcast:15 */, 0xa, 0xf, false);  // into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143 /* row_bcast:31 */, 0xc, 0xf, false);  // into rows 2 and 3
  return v;
}
// Bitwise or over the wavefront, in every lane.
__device__ inline int wave_or(int v) {
  v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return __builtin_amdgcn_readlane(v, 63);
}
// Sum of table[0 .. kWaves) before this wavefront's entry, and of all of it: one LDS read.
template <int kWaves>
__device__ inline int waves_before(const int* table, int wave, int& total) {
  static_assert(kWaves == 8 || kWaves == 16, "one DPP row holds the table");
  const int inc = row_scan(table[threadIdx.x & (kWaves - 1)]);
  total = __builtin_amdgcn_readlane(inc, kWaves - 1);
  return wave ? __builtin_amdgcn_readlane(inc, wave - 1) : 0;
}

// Exclusive prefix sum of one int per thread across the workgroup; `total` gets the sum.
// `tmp` is kWaves ints of LDS that no wavefront still reads; it may be written again after the next barrier.
template <int kWaves>
__device__ inline int block_exclusive_scan(int v, int* tmp, int& total) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int inc = wave_scan(v);
  if ((threadIdx.x & 63) == 63) tmp[wave] = inc;
  lds_barrier();
  return waves_before<kWaves>(tmp, wave, total) + inc - v;
}

// Number of set bits of `mask` that belong to lanes before this one (v_mbcnt).
__device__ inline int lanes_before(unsigned long long mask) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// Exclusive prefix count of one flag per thread; same contract.
template <int kWaves>
__device__ inline int block_flag_scan(bool flag, int* tmp, int& total) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned long long m = __ballot(flag);
  if ((threadIdx.x & 63) == 0) tmp[wave] = __popcll(m);
  lds_barrier();
  return waves_before<kWaves>(tmp, wave, total) + lanes_before(m);
}

// Lanes of the wavefront that hold the same digit as this lane (valid lanes only).  Only the
// bits of `vary` (wave-uniform: the bits in which the digits of this batch differ at all) need a
// ballot each.
__device__ inline unsigned long long match_digit(unsigned digit, bool valid, unsigned vary) {
  unsigned long long same = __ballot(valid);
  for (unsigned v = vary; v; v &= v - 1u) {
    const bool one = (digit >> (__ffs(v) - 1)) & 1u;
    const unsigned long long m = __ballot(one);
    same &= one ? m : ~m;
  }
  return same;
}
// Bits in which the digits of the valid lanes differ (wave-uniform).
__device__ inline unsigned varying_bits(unsigned digit, bool valid) {
  const unsigned long long vm = __ballot(valid);
  if (vm == 0) return 0u;
  const unsigned first = __builtin_amdgcn_readlane(digit, __ffsll((long long)vm) - 1);
  return (unsigned)wave_or(valid ? (int)(digit ^ first) : 0);
}

// Longest sequence and wavefronts of the workgroup: with 16, every step from the second barrier on is mostly the
// issue of their instructions, so up to 2048 positions take eight (one sequence of 512: 6.3 -> 5.6 us, of 2048 8.2 -> 7.6).
template <int P2, int kSegWaves>
__global__ __launch_bounds__(64 * kSegWaves) void build_segments_kernel(
    const int* __restrict__ row_ids, const int* __restrict__ col_ids,
    const unsigned char* __restrict__ flags, int B, int N, int max_global, int radius,
    int* __restrict__ seg, int K) {
  constexpr int kSegThreads = 64 * kSegWaves;
  constexpr int CHUNK = P2 / kSegWaves;  // consecutive elements owned by one wavefront
  constexpr int NB = CHUNK / 64;         // 64-element batches per wavefront
  constexpr int VE = NB < 4 ? NB : 4;    // consecutive elements per lane while classifying
  constexpr int NV = NB / VE;            // batches of 64 VE elements
  static_assert(NB >= 1, "P2 must be at least the workgroup size");
  __shared__ __attribute__((aligned(16))) int ids[P2];                  // id by token position; later: segment starts (ushort)
  __shared__ unsigned short buf_a[P2];     // current order of table-token positions
  __shared__ unsigned short buf_b[P2];     // next order; later: segment index by slot
  __shared__ __attribute__((aligned(16))) unsigned short hist[kSegWaves][kBins];  // per-wavefront digit counts -> first output slots
  __shared__ int scan_tmp[3][kSegWaves];
  __shared__ int wave_tot[3][kSegWaves];
  __shared__ int s_or, s_bad;
  // counting-sort path: how often every id is seen, anywhere and (<< 16) before this workgroup's
  // chunk (it lives in an order buffer, which only the general path uses, and later); first slot
  // (and << 16 one past the last) and segment index of every id; scratch for the work-unit list
  unsigned* const id_count = reinterpret_cast<unsigned*>(buf_b);
  __shared__ int start_v[kBins];
  __shared__ int seg_i[kBins];
  __shared__ int seg_tmp[2][kBins + 8];
  static_assert(P2 * sizeof(unsigned short) >= kBins * sizeof(int), "the histogram must fit an order buffer");

  const int b = blockIdx.x, view = blockIdx.y, tid = threadIdx.x;
  // Several workgroups per (sequence, view): K of them take a chunk of the positions each, one
  // more (k == K, no chunk) lists the work units.
  const int k = blockIdx.z;
  const int chunk = (((N + K - 1) / K) + 63) & ~63, c0 = k < K ? k * chunk : 0, c1 = min(N, c0 + chunk);
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int* id_src = (view == 0 ? row_ids : col_ids) + (size_t)b * N;
  const unsigned char* fl = flags + (size_t)b * N;
  // Element order everywhere below: a wavefront owns CHUNK consecutive elements and walks them in
  // batches of 64, lane = consecutive element, so that LDS and global accesses are unit-stride
  // and ranks inside a batch come from ballots.  Only the classification, which every workgroup
  // does for the whole sequence and which the instruction issue bounds, takes VE consecutive
  // elements per lane.
  const int w0 = wave * CHUNK;

  // All of this wavefront's inputs first, in one go: the loads travel together instead of one
  // dependent round trip per batch.
  typedef typename Ids<VE>::type idv;
  unsigned in_word[NV];
  idv in_id[NV];
#pragma unroll
  for (int e = 0; e < NV; ++e) {
    const int i0 = w0 + (e * 64 + lane) * VE;
    in_word[e] = load_flags<VE>(fl, i0, N);
    in_id[e] = load_ids<VE>(id_src, i0, N);
  }
  asm volatile("" ::: "memory");  // (where the tables lie is worked out while they travel)

  const SegLayout lay(B, N);
  int* counts = seg + lay.counts + (size_t)b * kCountWords;
  int* global_idx = seg + lay.global_idx + (size_t)b * N;
  int* pad_idx = seg + lay.pad_idx + (size_t)b * N;
  int* vbase = seg + lay.view0 + (size_t)view * lay.view_stride;
  int* perm = vbase + lay.perm + (size_t)b * N;
  int* seg_off = vbase + lay.seg_off + (size_t)b * (N + 1);
  int* seg_of_tok = vbase + lay.seg_of_tok + (size_t)b * N;
  int2* slot_rng = reinterpret_cast<int2*>(vbase + lay.slot_rng) + (size_t)b * N;
  int4* unit = reinterpret_cast<int4*>(vbase + lay.unit) + (size_t)b * lay.units * 2;
  int4* gunit = reinterpret_cast<int4*>(seg + lay.gunit) + (size_t)b * lay.tiles * 2;

  if (b == 0 && view == 0 && k == 0 && tid < kHdrWords)
    seg[tid] = tid == 0 ? kMagic : tid == 1 ? B : tid == 2 ? N : tid == 4 ? max_global : tid == 5 ? radius : 0;

  // (while they travel) clear the counters
  if (tid == 0) { s_or = 0; s_bad = 0; }
  if (tid < (int)kBins) id_count[tid] = 0;
  for (int i = tid; i < kSegWaves * (int)kBins / 8; i += kSegThreads)
    reinterpret_cast<uint4*>(&hist[0][0])[i] = make_uint4(0, 0, 0, 0);
  lds_barrier();

  unsigned char in_flag[NV][VE];
#pragma unroll
  for (int e = 0; e < NV; ++e) {
    const int i0 = w0 + (e * 64 + lane) * VE;
    if (w0 + CHUNK > N) {  // uniform
      in_word[e] = align_flags<VE>(in_word[e], i0, N);
      in_id[e] = align_ids<VE>(in_id[e], i0, N);
    }
#pragma unroll
    for (int j = 0; j < VE; ++j) in_flag[e][j] = (unsigned char)(in_word[e] >> (8 * j));
  }

  // ---- bucketed mode: question tokens past the first max_global join the table tokens ----------
  int q_at = 0;   // question tokens before this wavefront's block
  if (max_global < N) {  // uniform; a sequence has at most N question tokens
    int n_q = 0;
#pragma unroll
    for (int e = 0; e < NV; ++e)
#pragma unroll
      for (int j = 0; j < VE; ++j) {
        const int i = w0 + (e * 64 + lane) * VE + j;
        n_q += __popcll(__ballot(i < N && in_flag[e][j] == 1));
      }
    if (lane == 0) scan_tmp[0][wave] = n_q;
    lds_barrier();
    int all_q;
    q_at = waves_before<kSegWaves>(scan_tmp[0], wave, all_q);
  }

  // ---- classify; count the three kinds of position per wavefront ---------------------------
  int n_lg = 0, lg_bef = 0;   // my table tokens, and question tokens << 16; those before this workgroup's chunk
  int bad = 0, my_or = 0;
#pragma unroll
  for (int e = 0; e < NV; ++e) {
    const int i0 = w0 + (e * 64 + lane) * VE;
    const bool before = i0 < c0;   // (c0 is a multiple of 64)
    if (max_global < N) {
      int mine = 0;
#pragma unroll
      for (int j = 0; j < VE; ++j) mine += i0 + j < N && in_flag[e][j] == 1;
      const int upto = wave_scan(mine);
      int q = q_at + upto - mine;
#pragma unroll
      for (int j = 0; j < VE; ++j)
        if (i0 + j < N && in_flag[e][j] == 1 && q++ >= max_global) in_flag[e][j] = 0;
      q_at += __builtin_amdgcn_readlane(upto, 63);
    }
    idv code;
    int lg = 0;
    unsigned run = 0;
#pragma unroll
    for (int j = 0; j < VE; ++j) {
      unsigned f = in_flag[e][j];
      const int id = in_id[e][j];
      const bool have = i0 + j < N;
      const bool table = have && f == 0;
      bad |= have && (f > 2 || (f == 0 && id < 0));
      f = min(f, 2u);
      my_or |= table ? id : 0;
      lg += table ? 1 : have && f == 1 ? 1 << 16 : 0;
      code[j] = f == 0 ? id : -(int)f;   // table token: its id; question token -1; pad -2
      // histogram of the low digit, one LDS add per run of equal ids of this lane (ids of a
      // flattened table come in runs); only meaningful if every id turns out to be below kBins
      const int key = table ? id & (int)(kBins - 1u) : -1;
      const int next = j + 1 < VE && i0 + j + 1 < N && in_flag[e][j + 1] == 0 ? in_id[e][j + 1] & (int)(kBins - 1u) : -1;
      ++run;
      if (key != next || j + 1 == VE) {
        if (key >= 0) atomicAdd(&id_count[key], before ? run * 0x10001u : run);
        run = 0;
      }
    }
    if constexpr (VE == 1) ids[i0] = code[0];
    else *reinterpret_cast<idv*>(&ids[i0]) = code;
    n_lg += lg;
    if (before) lg_bef += lg;
  }
  my_or = wave_or(my_or);
  n_lg = wave_scan(n_lg);
  lg_bef = wave_scan(lg_bef);
  if (lane == 63) {
    if (my_or) atomicOr(&s_or, my_or);
    wave_tot[0][wave] = n_lg;
    wave_tot[1][wave] = lg_bef;
  }
  if (bad) s_bad = 1;
  lds_barrier();
  int lg_all, lg_before;
  const int lg_at = waves_before<kSegWaves>(wave_tot[0], wave, lg_all);
  waves_before<kSegWaves>(wave_tot[1], wave, lg_before);
  const int L = lg_all & 0xffff, G = lg_all >> 16, P = N - L - G;
  // kinds before this workgroup's chunk
  const int g_before = lg_before >> 16, p_before = c0 - (lg_before & 0xffff) - g_before;
  const unsigned all_bits = (unsigned)s_or;
  const float inv_radius = radius > 0 ? 1.0f / (float)radius : 0.f;
  const int n_pt = (P + kPadSlots - 1) / kPadSlots;
  const int n_t0 = (G + BN - 1) / BN;
  constexpr int kMaxUnits = kMaxTiles + kMaxTiles / 2 + 2;
  __shared__ unsigned short head_pos[kMaxUnits];
  __shared__ unsigned short unit_len[kMaxUnits];

  if ((all_bits & ~(kBins - 1u)) == 0) {
    // ============ counting-sort path: every id is below kBins, all workgroups ============
    constexpr int NBC = (P2 > 8 * kSegChunk ? 2 : 1) * kSegChunk / kSegThreads;   // 64-position batches of the chunk per wavefront
    // first slot and segment index of every id, from one scan (segments << 16)
    const unsigned count = tid < (int)kBins ? id_count[tid] : 0u;
    const int c_id = (int)(count & 0xffffu);
    int tot;
    const int at = block_exclusive_scan<kSegWaves>(c_id | (c_id > 0 ? 1 << 16 : 0), scan_tmp[1], tot);
    const int first_slot = at & 0xffff, seg_index = at >> 16, S = tot >> 16;
    if (tid < (int)kBins) {
      start_v[tid] = first_slot | (first_slot + c_id) << 16;
      seg_i[tid] = seg_index;
      if (c_id > 0) seg_tmp[0][seg_index] = first_slot;   // first slot of every segment, compact
    }
    if (tid == 0) seg_tmp[0][S] = L;
    lds_barrier();
    const int* sstart = seg_tmp[0];
    // A slot's window: its segment [lo, hi), in bucketed mode cut to the neighbouring buckets.  Slots are below 2^14, so the
    // bucket index comes exactly from one float multiply: (s + 0.5) / radius is at least 0.5 / radius away from an
    // integer and the rounding error is below 2e-7 s / radius.
    auto bounded = [&](int s, int lo, int hi) {
      if (radius > 0) {
        const int first = (int)(((float)s + 0.5f) * inv_radius) * radius;  // first slot of s's bucket
        lo = max(lo, first - radius);
        hi = min(hi, first + 2 * radius);
      }
      return make_int2(lo, hi);
    };

    // ---- this workgroup's chunk of positions: rank among equal ids, kind lists ----------------
    if (k < K) {
      int code[NBC], rank_w[NBC], g_rank[NBC], p_rank[NBC];
      int g_w = 0, p_w = 0;
#pragma unroll
      for (int j = 0; j < NBC; ++j) {
        const int p = c0 + (wave * NBC + j) * 64 + lane;
        code[j] = p < c1 ? ids[p] : -3;
        const bool local = code[j] >= 0;
        const unsigned dg = local ? (unsigned)code[j] : 0u;
        const unsigned long long same = match_digit(dg, local, varying_bits(dg, local));
        const int before = lanes_before(same);
        int old = 0;
        if (local && before == 0) {  // first lane of a group of equal ids
          old = hist[wave][dg];
          hist[wave][dg] = (unsigned short)(old + __popcll(same));
        }
        old = __shfl(old, local ? __ffsll((long long)same) - 1 : lane, 64);
        rank_w[j] = old + before;
        const unsigned long long mg = __ballot(code[j] == -1), mp = __ballot(code[j] == -2);
        g_rank[j] = g_w + lanes_before(mg);
        p_rank[j] = p_w + lanes_before(mp);
        g_w += __popcll(mg);
        p_w += __popcll(mp);
      }
      if (lane == 0) wave_tot[2][wave] = g_w | p_w << 16;
      lds_barrier();
      // (id, wavefront) counts -> tokens with that id before the wavefront's block
      if (tid < (int)kBins) {
        int c[kSegWaves], running = (int)(count >> 16);
#pragma unroll
        for (int w = 0; w < kSegWaves; ++w) c[w] = hist[w][tid];
#pragma unroll
        for (int w = 0; w < kSegWaves; ++w) {
          hist[w][tid] = (unsigned short)running;
          running += c[w];
        }
      }
      int gp_chunk;
      const int gp = waves_before<kSegWaves>(wave_tot[2], wave, gp_chunk);
      const int g_at_c = g_before + (gp & 0xffff), p_at_c = p_before + (gp >> 16);
      lds_barrier();
#pragma unroll
      for (int j = 0; j < NBC; ++j) {
        const int p = c0 + (wave * NBC + j) * 64 + lane;
        if (p < c1) {
          const int g_at = g_at_c + g_rank[j], p_at = p_at_c + p_rank[j];
          if (code[j] >= 0) {
            const int range = start_v[code[j]], lo = range & 0xffff, slot = lo + hist[wave][code[j]] + rank_w[j];
            perm[slot] = p;
            slot_rng[slot] = bounded(slot, lo, range >> 16);
            seg_of_tok[p] = seg_i[code[j]];
          } else {
            slot_rng[L + g_at + p_at] = make_int2(0, 0);  // (behind the last slot, one for every other token)
            seg_of_tok[p] = -1;
            if (view == 0) {
              if (code[j] == -1) global_idx[g_at] = p;
              else pad_idx[p_at] = p;
            }
          }
        }
      }
    }
    // ---- per-sequence and per-segment tables (first workgroup) -----------------------------------
    if (k == 0) {
      if (tid < (int)kBins && c_id > 0) seg_off[seg_index] = first_slot;
      if (tid == 0) {
        seg_off[S] = L;
        counts[C_SROW + view] = S;
        counts[5 + view] = s_bad;
        if (view == 0) { counts[C_G] = G; counts[C_L] = L; counts[C_P] = P; }
      }
    }
    if (k != K) return;
    // ---- work units of the attention kernels (the workgroup without a chunk) ---------------------
    // question-token owners (the same for both views), by the last wavefronts, which seldom list units
    constexpr int kFirst = kSegThreads - kMaxTiles;
    auto list_question_owners = [&]() {
      if (view != 0 || tid < kFirst || tid - kFirst >= lay.tiles) return;
      const int rec = tid - kFirst;
      const GlobalSplit gs = global_split(G, L, B, N);
      int4 q0 = make_int4(UNIT_NONE, 0, 0, 0), q1 = make_int4(0, 0, -1, 0);
      if (rec < gs.n_gt * gs.n_chunks) {
        const int gt = rec / gs.n_chunks, c = rec % gs.n_chunks;
        q0 = make_int4(UNIT_GLOBAL, gt * BM, 0, L);
        q1.x = c * gs.per;
        q1.y = min(gs.n_st, q1.x + gs.per);
        if (gs.n_chunks > 1) q1.z = rec;
        q1.w = gs.n_chunks;
      }
      gunit[2 * rec] = q0;
      gunit[2 * rec + 1] = q1;
    };
    // The record of the unit that owns slots [t0, end), without its place in the list.  Its first and last segments are the
    // last ones that begin at or before t0 and end - 1: rounds of seven reads at a time (three for up to 512 segments),
    // where a binary search is up to nine rounds, of 50 ns each.
    auto local_unit = [&](int t0, int end, auto first_step, int4& r0, int4& r1) {
      int first_seg = 0, last_seg = 0;
#pragma unroll
      for (int step = decltype(first_step)::value; step > 0; step /= 8) {
        int f[7], l[7];
#pragma unroll
        for (int j = 0; j < 7; ++j) {   // (sstart[S] = L is beyond every slot)
          f[j] = sstart[min(first_seg + (j + 1) * step, S)];
          l[j] = sstart[min(last_seg + (j + 1) * step, S)];
        }
        int f_n = 0, l_n = 0;
#pragma unroll
        for (int j = 0; j < 7; ++j) {
          f_n += f[j] <= t0;
          l_n += l[j] < end;
        }
        first_seg += f_n * step;
        last_seg += l_n * step;
      }
      const int lo = bounded(t0, sstart[first_seg], L).x, hi = bounded(end - 1, 0, sstart[last_seg + 1]).y;
      r0 = make_int4(UNIT_LOCAL, t0, lo, hi);
      r1.y = n_t0 + (hi - lo + BN - 1) / BN;
      r1.w = end;
    };
    // A run is a segment of at least kBigSegment slots, or the shorter segments between two such
    // segments; units are 128-slot pieces of runs (see the general path below for why).
    // Up to 64 records (5248 positions) and 128 segments: one wavefront lists them, without a barrier, kEach consecutive segments and one record to
    // a lane.  (us with the workgroup's scans below and with this: one sequence of 128 4.9 and 4.3, of 512 5.2 and 4.4, of 1999
    // with 100 rows 6.0 and 5.4, 8 of 2048 6.6 and 5.7; with eight segments to a lane, for up to 512, the scans are faster: 5.7 and 5.9.)
    auto list_units = [&](auto each) {
      constexpr int kEach = decltype(each)::value;
      int start[kEach + 1];
#pragma unroll
      for (int e = 0; e <= kEach; ++e) start[e] = sstart[min(kEach * lane + e, S)];
      const int before = sstart[max(min(kEach * lane, S) - 1, 0)];
      unsigned cuts = 0;
      int first_start = L;   // of the lane's first run
#pragma unroll
      for (int e = kEach - 1; e >= 0; --e) {
        const int i = kEach * lane + e, last = e ? start[e - 1] : before;
        if (i < S && (i == 0 || start[e + 1] - start[e] >= kBigSegment || start[e] - last >= kBigSegment)) {
          cuts |= 1u << e;
          first_start = start[e];
        }
      }
      const unsigned long long lanes = __ballot(cuts != 0), later = lane < 63 ? lanes >> (lane + 1) : 0;
      const int next_start = __shfl(first_start, later ? lane + __ffsll((long long)later) : lane, 64);
      int run_end = later ? next_start : L, units_of[kEach], mine = 0;
#pragma unroll
      for (int e = kEach - 1; e >= 0; --e) {
        const bool cut = (cuts >> e) & 1u;
        units_of[e] = cut ? (run_end - start[e] + kTileSlots - 1) / kTileSlots : 0;
        run_end = cut ? start[e] : run_end;
        mine += units_of[e];
      }
      const int upto = wave_scan(mine);
      int n_units = __builtin_amdgcn_readlane(upto, 63);
      if (n_units + n_pt <= lay.units) {
        int at = upto - mine;
#pragma unroll
        for (int e = 0; e < kEach; ++e)
          for (int i = 0; i < units_of[e]; ++i) head_pos[at++] = (unsigned short)(start[e] + i * kTileSlots);
      } else {  // more records than the buffer has: every 128 slots regardless of segments
        n_units = (L + kTileSlots - 1) / kTileSlots;
        if (lane < n_units) head_pos[lane] = (unsigned short)(lane * kTileSlots);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      int4 r0 = make_int4(UNIT_NONE, 0, 0, 0), r1 = make_int4(0, 0, -1, 0);
      if (lane < n_units) {
        const int t0 = min((int)head_pos[lane], L - 1);
        const int end = min(max(lane + 1 < n_units ? (int)head_pos[lane + 1] : L, t0 + 1), min(L, t0 + kTileSlots));
        local_unit(t0, end, std::integral_constant<int, kEach == 1 ? 8 : 64>(), r0, r1);
      } else if (lane < n_units + n_pt) {
        r0 = make_int4(UNIT_PAD, (lane - n_units) * kPadSlots, 0, 0);
      }
      int place = lane;
      if (lane < n_units) {   // longest streamed side first, ties in slot order
        place = 0;
        for (int j = 0; j < n_units; ++j) {
          const int other = __builtin_amdgcn_readlane(r1.y, j);
          place += other > r1.y || (other == r1.y && j < lane);
        }
      }
      if (lane < lay.units) {
        unit[2 * place] = r0;
        unit[2 * place + 1] = r1;
      }
    };
    if (lay.units <= 64 && S <= 128) {
      if (wave != 0) list_question_owners();
      else if (S <= 64) list_units(std::integral_constant<int, 1>());
      else list_units(std::integral_constant<int, 2>());
      return;
    }
    // More: the workgroup, a segment and a record to a thread.
    int* run_start = seg_tmp[1];
    bool cut = false;
    if (tid < S) {
      const int size = sstart[tid + 1] - sstart[tid];
      cut = tid == 0 || size >= kBigSegment || sstart[tid] - sstart[tid - 1] >= kBigSegment;
    }
    int n_runs;
    const int run_index = block_flag_scan<kSegWaves>(cut, scan_tmp[2], n_runs);
    if (cut) run_start[run_index] = sstart[tid];
    if (tid == 0) run_start[n_runs] = L;
    lds_barrier();
    const int run_units = tid < n_runs ? (run_start[tid + 1] - run_start[tid] + kTileSlots - 1) / kTileSlots : 0;
    int n_units;
    const int unit_base = block_exclusive_scan<kSegWaves>(run_units, scan_tmp[1], n_units);
    if (n_units + n_pt <= lay.units) {
      for (int i = 0; i < run_units; ++i) head_pos[unit_base + i] = (unsigned short)(run_start[tid] + i * kTileSlots);
    } else {  // more records than the buffer has: every 128 slots regardless of segments
      n_units = (L + kTileSlots - 1) / kTileSlots;
      if (tid < n_units) head_pos[tid] = (unsigned short)(tid * kTileSlots);
    }
    lds_barrier();
    int4 r0 = make_int4(UNIT_NONE, 0, 0, 0), r1 = make_int4(0, 0, -1, 0);
    if (tid < n_units) {
      const int t0 = min((int)head_pos[tid], L - 1);
      const int end = min(max(tid + 1 < n_units ? (int)head_pos[tid + 1] : L, t0 + 1), min(L, t0 + kTileSlots));
      static_assert(kBins == 8 * 8 * 8, "three digits");
      local_unit(t0, end, std::integral_constant<int, 64>(), r0, r1);
      unit_len[tid] = (unsigned short)r1.y;
    }
    lds_barrier();
    if (tid < lay.units) {
      int place = tid;
      if (tid < n_units) {   // longest streamed side first, ties in slot order
        place = 0;
        const int mine = r1.y;
#pragma unroll 8
        for (int j = 0; j < n_units; ++j) {
          const int other = unit_len[j];
          place += other > mine || (other == mine && j < tid);
        }
      } else if (tid < n_units + n_pt) {
        r0 = make_int4(UNIT_PAD, (tid - n_units) * kPadSlots, 0, 0);
      }
      unit[2 * place] = r0;
      unit[2 * place + 1] = r1;
    }
    list_question_owners();
    return;
  }
  if (k != 0) return;   // ids of 512 and more: the first workgroup sorts alone

  // ======================= general path: LSD radix sort in this workgroup =======================
  // ---- compact the three kinds in ascending position order ------------------------------------
  int l_at = lg_at & 0xffff, g_at = lg_at >> 16, p_at = min(w0, N) - l_at - g_at;
#pragma unroll
  for (int e = 0; e < NB; ++e) {
    const int i = w0 + e * 64 + lane;
    const unsigned char f = i < N ? fl[i] : (unsigned char)0;
    const unsigned long long mq = __ballot(i < N && f == 1);
    // (the question tokens kept come first)
    const bool question = i < N && f == 1 && g_at + lanes_before(mq) < max_global;
    const bool table = i < N && (f == 0 || (f == 1 && !question)), pad = i < N && f >= 2;
    const unsigned long long ml = __ballot(table), mg = __ballot(question), mp = __ballot(pad);
    if (table) buf_a[l_at + lanes_before(ml)] = (unsigned short)i;
    else if (i < N) seg_of_tok[i] = -1;
    if (view == 0) {
      if (question) global_idx[g_at + lanes_before(mg)] = i;
      if (pad) pad_idx[p_at + lanes_before(mp)] = i;
    }
    l_at += __popcll(ml);
    g_at += __popcll(mg);
    p_at += __popcll(mp);
  }
  if (view == 0) {
    // entries past G and P stay unwritten: nothing reads them (the export hook masks them)
    if (tid == 0) { counts[C_G] = G; counts[C_L] = L; counts[C_P] = P; }
  }
  if (tid == 0) counts[5 + view] = s_bad;
  lds_barrier();

  // ---- stable LSD radix sort of buf_a[0..L) by ids[position] --------------------------------
  unsigned short* cur = buf_a;
  unsigned short* nxt = buf_b;
  for (int shift = 0; shift < 32; shift += kDigitBits) {
    if (((all_bits >> shift) & (kBins - 1u)) == 0) continue;  // digit 0 everywhere: order unchanged
    for (int i = tid; i < kSegWaves * kBins / 2; i += kSegThreads) reinterpret_cast<int*>(&hist[0][0])[i] = 0;
    lds_barrier();
    // count digits per wavefront; every element learns its rank among the equal digits of its
    // wavefront's block (batches in order, lanes in order inside a batch)
    int pos[NB], rank_w[NB];
    unsigned dig[NB];
#pragma unroll
    for (int e = 0; e < NB; ++e) {
      const int s = w0 + e * 64 + lane;
      pos[e] = s < L ? cur[s] : 0;
      dig[e] = s < L ? ((unsigned)ids[pos[e]] >> shift) & (kBins - 1u) : 0u;
    }
#pragma unroll
    for (int e = 0; e < NB; ++e) {
      const bool valid = w0 + e * 64 + lane < L;
      const unsigned long long same = match_digit(dig[e], valid, varying_bits(dig[e], valid));
      const int before = lanes_before(same);
      int old = 0;
      if (valid && before == 0) {  // first lane of a group of equal digits
        old = hist[wave][dig[e]];
        hist[wave][dig[e]] = (unsigned short)(old + __popcll(same));
      }
      old = __shfl(old, valid ? __ffsll((long long)same) - 1 : lane, 64);
      rank_w[e] = old + before;
    }
    lds_barrier();
    // counts -> first output slot of (digit, wavefront): digits ascending, wavefronts ascending
    int first[kSegWaves], tot = 0;
    if (tid < kBins) {
#pragma unroll
      for (int w = 0; w < kSegWaves; ++w) first[w] = hist[w][tid];
#pragma unroll
      for (int w = 0; w < kSegWaves; ++w) {
        const int c = first[w];
        first[w] = tot;
        tot += c;
      }
    }
    int all;
    const int digit_base = block_exclusive_scan<kSegWaves>(tot, scan_tmp[0], all);
    if (tid < kBins) {
#pragma unroll
      for (int w = 0; w < kSegWaves; ++w) hist[w][tid] = (unsigned short)(first[w] + digit_base);
    }
    lds_barrier();
#pragma unroll
    for (int e = 0; e < NB; ++e)
      if (w0 + e * 64 + lane < L) nxt[hist[wave][dig[e]] + rank_w[e]] = (unsigned short)pos[e];
    lds_barrier();
    unsigned short* t = cur; cur = nxt; nxt = t;
  }

  // ---- run boundaries -> segment index per slot ----------------------------------------------
  unsigned head_bits = 0;  // bit e: my slot of batch e starts a segment
  int my_pos[NB];
  int n_head = 0;
#pragma unroll
  for (int e = 0; e < NB; ++e) {
    const int s = w0 + e * 64 + lane;
    my_pos[e] = s < L ? cur[s] : 0;
    const bool head = s < L && (s == 0 || ids[cur[s - 1]] != ids[my_pos[e]]);
    head_bits |= (unsigned)head << e;
    n_head += __popcll(__ballot(head));
  }
  if (lane == 0) wave_tot[0][wave] = n_head;
  lds_barrier();  // also: every wavefront is done reading ids[]
  int S = 0, seg_at = 0;
#pragma unroll
  for (int w = 0; w < kSegWaves; ++w) {
    const int c = wave_tot[0][w];
    if (w < wave) seg_at += c;
    S += c;
  }
  // ids[] and the spare order buffer are dead now: reuse them
  unsigned short* seg_start = reinterpret_cast<unsigned short*>(ids);  // [P2], entry S (== L) implied
  unsigned short* seg_of_slot = nxt;                                    // [P2]
#pragma unroll
  for (int e = 0; e < NB; ++e) {
    const int s = w0 + e * 64 + lane;
    const bool head = (head_bits >> e) & 1u;
    const unsigned long long mh = __ballot(head);
    const int seg_idx = seg_at + lanes_before(mh) + (head ? 1 : 0) - 1;  // heads up to and including me
    if (s < L) {
      perm[s] = my_pos[e];
      seg_of_tok[my_pos[e]] = seg_idx;
      seg_of_slot[s] = (unsigned short)seg_idx;
      if (head) { seg_start[seg_idx] = (unsigned short)s; seg_off[seg_idx] = s; }
    }  // perm past L, like seg_off past S, stays unwritten (masked by the export hook)
    seg_at += __popcll(mh);
  }
  if (tid == 0) { seg_off[S] = L; counts[C_SROW + view] = S; }
  lds_barrier();
  // window of slot s: its segment, in bucketed mode cut to the neighbouring buckets.  Slots are
  // below 2^14, so the bucket index comes exactly from one float multiply: (s + 0.5) / radius is
  // at least 0.5 / radius away from an integer and the rounding error is below 2e-7 s / radius.
  auto window = [&](int s) {
    const int g = seg_of_slot[s];
    int lo = seg_start[g], hi = g + 1 < S ? (int)seg_start[g + 1] : L;
    if (radius > 0) {
      const int first = (int)(((float)s + 0.5f) * inv_radius) * radius;  // first slot of s's bucket
      lo = max(lo, first - radius);
      hi = min(hi, first + 2 * radius);
    }
    return make_int2(lo, hi);
  };
#pragma unroll
  for (int e = 0; e < NB; ++e) {
    const int s = w0 + e * 64 + lane;
    if (s < N) slot_rng[s] = s < L ? window(s) : make_int2(0, 0);
  }

  // ---- work units of the attention kernels -------------------------------------------------
  // Table-token owners: up to 128 consecutive sorted slots each, streaming the question tokens
  // and then the slot window spanned by the segments those slots touch; pad owners after them.
  // A segment of at least kBigSegment slots starts a unit of its own ("cut"), and so does the
  // first slot after it, so no unit straddles the boundary of a long segment; if that would
  // need more records than the buffer has, the slots are cut every 128 regardless.
  auto seg_size = [&](int g) { return (g + 1 < S ? (int)seg_start[g + 1] : L) - (int)seg_start[g]; };
  unsigned cut_bits = 0;  // bit e: my slot of batch e is a cut
#pragma unroll
  for (int e = 0; e < NB; ++e) {
    const int s = w0 + e * 64 + lane;
    bool cut = false;
    if (s < L) {
      const int g = seg_of_slot[s];
      cut = s == (int)seg_start[g] &&
            (g == 0 || seg_size(g) >= kBigSegment || seg_size(g - 1) >= kBigSegment);
    }
    cut_bits |= (unsigned)cut << e;
  }
  int n_units = 0;
  for (int attempt = 0; attempt < 2; ++attempt) {  // 0: with cuts; 1: every 128 slots (rare)
    const bool use_cuts = attempt == 0;
    // last cut inside each wavefront's block -> the cut in force at the start of the next ones
    int last = -1;
#pragma unroll
    for (int e = 0; e < NB; ++e) {
      const unsigned long long m = __ballot(use_cuts && ((cut_bits >> e) & 1u));
      if (m) last = w0 + e * 64 + 63 - __clzll((long long)m);
    }
    if (lane == 0) wave_tot[1][wave] = last;
    lds_barrier();
    int running = 0;
#pragma unroll
    for (int w = 0; w < kSegWaves; ++w)
      if (w < wave) running = max(running, wave_tot[1][w]);
    unsigned hbits = 0;  // bit e: my slot of batch e starts a unit
    int n_head_w = 0;
#pragma unroll
    for (int e = 0; e < NB; ++e) {
      const int s = w0 + e * 64 + lane;
      const unsigned long long m = __ballot(use_cuts && ((cut_bits >> e) & 1u));
      const unsigned long long upto = m & (~0ull >> (63 - lane));  // cuts at lanes <= mine
      const int base = upto ? w0 + e * 64 + 63 - __clzll((long long)upto) : running;
      const bool head = s < L && ((s - base) & (kTileSlots - 1)) == 0;
      hbits |= (unsigned)head << e;
      n_head_w += __popcll(__ballot(head));
      if (m) running = w0 + e * 64 + 63 - __clzll((long long)m);
    }
    if (lane == 0) wave_tot[0][wave] = n_head_w;
    lds_barrier();
    int head_at = 0;
    n_units = 0;
#pragma unroll
    for (int w = 0; w < kSegWaves; ++w) {
      const int c = wave_tot[0][w];
      if (w < wave) head_at += c;
      n_units += c;
    }
    const bool fits = n_units + n_pt <= lay.units;  // always true without cuts
    if (fits) {
#pragma unroll
      for (int e = 0; e < NB; ++e) {
        const bool head = (hbits >> e) & 1u;
        const unsigned long long mh = __ballot(head);
        if (head) head_pos[head_at + lanes_before(mh)] = (unsigned short)(w0 + e * 64 + lane);
        head_at += __popcll(mh);
      }
    }
    lds_barrier();  // head_pos is complete; wave_tot may be written again
    if (fits) break;
  }
  // streamed length of every unit, then its place in the list: longest first (ties in slot
  // order), so that across a launch the long units start first and the short ones fill the end
  int4 r0 = make_int4(UNIT_NONE, 0, 0, 0), r1 = make_int4(0, 0, -1, 0);
  if (tid < n_units) {
    // (clamped so that a record can never name a slot outside [0, L), whatever else goes wrong)
    const int t0 = min((int)head_pos[tid], L - 1);
    const int end = min(max(tid + 1 < n_units ? (int)head_pos[tid + 1] : L, t0 + 1), min(L, t0 + kTileSlots));
    const int lo = window(t0).x, hi = window(end - 1).y;
    r0 = make_int4(UNIT_LOCAL, t0, lo, hi);
    r1.y = n_t0 + (hi - lo + BN - 1) / BN;
    r1.w = end;
    unit_len[tid] = (unsigned short)r1.y;
  }
  lds_barrier();
  if (tid < lay.units) {
    int place = tid;
    if (tid < n_units) {
      place = 0;
      const int mine = r1.y;
      for (int j = 0; j < n_units; ++j) {
        const int other = unit_len[j];
        place += other > mine || (other == mine && j < tid);
      }
    } else if (tid < n_units + n_pt) {
      r0 = make_int4(UNIT_PAD, (tid - n_units) * kPadSlots, 0, 0);
    }
    unit[2 * place] = r0;
    unit[2 * place + 1] = r1;
  }
  // question-token owners (the same for both views; written by the row view's workgroup)
  if (view == 0 && tid < lay.tiles) {
    const GlobalSplit gs = global_split(G, L, B, N);
    int4 r0 = make_int4(UNIT_NONE, 0, 0, 0), r1 = make_int4(0, 0, -1, 0);
    if (tid < gs.n_gt * gs.n_chunks) {
      const int gt = tid / gs.n_chunks, c = tid % gs.n_chunks;
      r0 = make_int4(UNIT_GLOBAL, gt * BM, 0, L);
      r1.x = c * gs.per;
      r1.y = min(gs.n_st, r1.x + gs.per);
      if (gs.n_chunks > 1) r1.z = tid;
      r1.w = gs.n_chunks;
    }
    gunit[2 * tid] = r0;
    gunit[2 * tid + 1] = r1;
  }
}

hipError_t launch_build_segments(const int* row_ids, const int* col_ids,
                                 const unsigned char* flags, int B, int N, int max_global,
                                 int radius, int* seg, hipStream_t stream) {
  // up to eight workgroups per (sequence, view) with about 1024 positions each, and a further one
  // for the work-unit list
  const int chunks = std::min(8, (N + kSegChunk - 1) / kSegChunk);
  dim3 grid(B, 2, chunks + 1);
  ProfileScope prof(1, stream);
#define MATE_SEG_CASE(MAX, P2, WAVES)                                                                     \
  if (N <= MAX) {                                                                                     \
    hipLaunchKernelGGL((build_segments_kernel<P2, WAVES>), grid, dim3(64 * WAVES), 0, stream, row_ids, \
                       col_ids, flags, B, N, max_global, radius, seg, chunks);                             \
    return hipGetLastError();                                                                         \
  }
  MATE_SEG_CASE(1, 1024, 16)   // (one position a lane)
  MATE_SEG_CASE(1024, 1024, 8)
  MATE_SEG_CASE(2048, 2048, 8)
  MATE_SEG_CASE(4096, 4096, 16)
  MATE_SEG_CASE(8192, 8192, 16)
  MATE_SEG_CASE(16384, 16384, 16)
#undef MATE_SEG_CASE
  return hipErrorInvalidValue;
}

}  // namespace mate
