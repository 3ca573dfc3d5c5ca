// Work decomposition shared by the bf16 MFMA forward / dQ / dK-dV kernels.
//
// Every kernel has the same shape: a workgroup OWNS 128 rows (queries, or keys for dK/dV) and
// STREAMS 64-row tiles of the other side.  By the attention pattern of Section 3 the two sides
// are symmetric: an owned table token meets the question tokens plus the table tokens of its
// own row / column segment; an owned question token meets every non-pad token.
//
// Units of one (sequence, head) -- listed by the segment builder, see seg_layout.h:
//   local   table-token owners, up to 128 consecutive slots of the head kind's sorted order
//           that never straddle the boundary of a long segment; listed longest stream first
//   pad     ceil(P / 1024) pad owners (zero fill)
//   global  question-token owners.  Their streamed side is the whole sequence, so it is cut into
//           chunks that run as separate units and leave partial results; the chunk that arrives
//           last merges them (where dQ has a launch of its own, its chunks are merged by the next kernel).
// Workgroup -> unit is arithmetic on the workgroup index plus one record read: no counters, no
// atomics, no dependent loads.  Workgroup i serves queue i mod 8 (consecutive workgroups go to
// consecutive XCDs, so a queue stays on one XCD and the units of one (sequence, head) pair
// share an L2).  Column-head pairs are numbered c = b n_col + i and belong to queue c mod 8, row-
// head pairs r = b n_row + i to queue (r + B n_col) mod 8.  Order inside a queue, longest units first:
//   1. column heads: record 0 (the longest unit) of every pair, record 1 of every pair, ... up
//      to record T - 1
//   2. the first T / 8 + 2 question-token unit records of all pairs, the same way (all of the
//      real ones unless a sequence has more than 128 question tokens)
//   3. row heads, as in 1
//   4. what is left of the three lists (real records only in the cases named above)
// The two backward kernels run 2 before 1: there the question-token chunks are as long as the
// column-head units, and more of both exist than workgroup slots, so whichever kind comes second
// has members that start late and end last; the chunks first measured 1-6 us better on four of
// the five benchmark shapes and the same on the fifth.  The forward does so when the streams are cut
// into chunks and the launch is a few rounds of the 1024 workgroup slots, where chunks that start
// second are the last to end (training steps: 2 x 8192, 16 heads 208.4 -> 204.5 us, bucketed 154.1 -> 148.8,
// 8 x 2048 201.0 -> 197.1); in longer launches, and where owners stream a few tiles, it is the
// column-head units that must not wait (16 x 4096 604 -> 613 with the chunks first, 32 x 512 114.5 -> 115.8).
// Records of kind "none" pad every pair to the same count; their workgroups exit at once.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "arrival.h"
#include "d2l.h"
#include "launch.h"
#include "mfma_common.h"

namespace mate {

constexpr int kThreads = 256;

struct UnitPlan {
  int kind;
  int t0;                // first owned slot in own_list
  const int* own_list;   // global_idx, perm[view] or pad_idx
  int own_count;
  const int* str_list;   // streamed table tokens: perm[view] (perm[0] for question owners)
  int s_lo, s_hi;        // streamed sorted-slot window
  int n_t0;              // streamed question-token tiles; table tiles follow
  int t_begin, t_end;    // streamed tiles of this unit
  int part;              // partial-result slot (unit index) or -1: results are final
  int n_chunks;          // question-token owners: chunks of this owner tile
  int G, L, P;
};

// ---- workgroup -> unit ---------------------------------------------------------------------
struct Work {
  int b, bh, view;
  const int* global_idx;  // of the sequence
  const int2* slot_rng;   // of the sequence and view
  UnitPlan u;
};

// Where the unit lists are, and the sizes that map a workgroup to one of them.  These are kernel arguments of their own, the
// first ones: plain values arrive in registers with the wavefront, a structure is loaded.
struct UnitLists {
  const int* hdr;   // the tables' header; the counts follow it
  const int4 *gunit, *unit_row, *unit_col;
  int B, H, N, n_col;
};
#define MATE_UNIT_LISTS const int *hdr, const int4 *gunit, const int4 *unit_row, const int4 *unit_col, int B, int H, int N, int n_col
#define MATE_UNIT_LISTS_VALUES(a) (a).seg.hdr, (a).seg.gunit, (a).seg.unit[0], (a).seg.unit[1], (a).B, (a).H, (a).N, (a).n_col

inline int unit_grid(int B, int H, int N, int n_col) {
  const int T = owner_slots(N), U = view_units(N), nc = (B * n_col + 7) / 8, nr = (B * (H - n_col) + 7) / 8;
  return 8 * ((nc + nr) * U + (nc + nr) * T);
}

// Question-token units before column-head units in the forward: see above.
inline bool fwd_chunks_first(int B, int H, int N) { return may_chunk(B, N) && (long)B * H * owner_slots(N) <= 3 * 1024; }

// A launch that is full although B N is small runs the short chunks that its tables list (see chunk_tiles) in pairs:
// an even chunk takes the odd one after it along, whose workgroup leaves.  (A template argument of the kernels: as a
// kernel argument it cost the short launches, which have none of it, 0.3 us each.)
inline bool joins_chunks(int B, int H, int N) {
  return may_chunk(B, N) && (long)B * N <= kSmallBatch && (long)B * H * owner_slots(N) > kFullLaunch;
}
__host__ __device__ inline int joined(int n_chunks) { return (n_chunks + 1) >> 1; }

// Small launches of the forward: a question-token owner of at most 32 rows is met by all four wavefronts, two tiles at a
// time (OwnerSplit).  That takes the LDS of two workgroups, so a launch must fit the chip twice over: at most two units a
// compute unit, with all the chunks that its sequences could have.  us, forward with 16 or 32 question tokens, one tile and
// two at a time: 12 heads, one sequence of 450 9.8 -> 8.5, of 2048 12.7 -> 11.7, 4 x 512 10.1 -> 9.5, 8 x 512 12.9 -> 11.3, 9 x 384
// 11.4 -> 10.7, 13 x 250 11.0 -> 10.8.  With more of them, which the host cannot know, two workgroups a compute unit cost 0 to
// 2 % (2 x 1000 with 64 11.3 -> 11.6) except where the order below gains.  Where owners stream three or four tiles (N up to 256)
// there is nothing to gain at fewer units (10 x 256 with 96 10.5 -> 10.75), and sequences of one tile of owners have pad
// owners as well, a unit in three: 20 x 128 8.1 -> 10.0, where 13 to 16 gain from the order (8.1 -> 7.8).
inline int forward_units(int B, int H, int N) { return B * H * (owner_slots(N) + (may_chunk(B, N) ? owner_slots(N) : 1)); }
inline bool small_forward(int B, int H, int N) {
  const long most = (long)B * H * owner_slots(N);
  if (most > 512) return false;
  const int units = forward_units(B, H, N);
  if (owner_slots(N) == 1) return units > 256 && units <= 384;
  if (owner_slots(N) == 2) return units > 416 && units <= 512;
  return units <= 512;
}
// Question-token units before column-head units there: where whole owners make some compute units get two (8 x 512 with 64
// question tokens 12.5 -> 11.4, with 96 14.8 -> 13.2, 10 x 384 with 96 12.9 -> 11.9; at 400 units and fewer 5 x 512 with 64 10.3 ->
// 10.65, 8 x 300 with 96 10.0 -> 11.0; with two tiles of owners 12 x 250 with 16 9.8 -> 10.4), and
// where chunks do (one sequence of 1500, 160 question tokens 16.6 -> 14.6, 2 x 900 14.4 -> 13.7; with up to 64 of them 1 to
// 4 % slower).
inline bool small_owners_first(int B, int H, int N) {
  if (owner_slots(N) == 1) return true;
  return owner_slots(N) > 2 && forward_units(B, H, N) > (may_chunk(B, N) ? 256 : 416);
}

template <bool kJoin>
__device__ __forceinline__ bool join_chunks(UnitPlan& u, bool glob) {  // false: the chunk before takes this one along
  if (kJoin && glob && u.part >= 0) {
    const int n_st = u.n_t0 + (u.L + BN - 1) / BN, gt = u.t0 / BM, c = u.part - gt * u.n_chunks;
    if (n_st <= kLongStream) {
      if (c & 1) return false;
      u.t_end = min(n_st, 2 * u.t_end - u.t_begin);
      u.n_chunks = joined(u.n_chunks);
      u.part = u.n_chunks > 1 ? gt * u.n_chunks + (c >> 1) : -1;
    }
  }
  return true;
}

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// Returns false if this workgroup has nothing to do.  Everything here is wave-uniform and
// stays in scalar registers.
//
// One round trip to memory: the place of the record is arithmetic on arguments that are in registers, and
// the record, the header and the counts are loaded together, the pointers that a unit's beginning needs during the
// arithmetic.  (Left to the compiler, every one of these was loaded where it is first used, behind the test of the one before:
// nine scalar round trips, three of them to memory, before the first index load.  us, before and now: f32 forward of one sequence of
// 128, 4 heads 12.7 -> 12.0, serving one of 512, 12 heads 16.4 -> 15.8, training at 2 x 8192, 16 heads 198.2 -> 197.3 and
// bucketed 142.4 -> 141.7, 8 x 2048 177.8 -> 175.3.)
template <bool kChunksFirst, bool kJoin>
__device__ __forceinline__ bool take_unit(UnitLists l, const AttnArgs& a, int block, Work& w) {
  const int *gidx = a.seg.global_idx, *pads = a.seg.pad_idx, *perm_row = a.seg.perm[0], *perm_col = a.seg.perm[1];
  const int2 *rng_row = a.seg.slot_rng[0], *rng_col = a.seg.slot_rng[1];
  const void *xq = a.q, *xk = a.k, *xv = a.v, *xo = a.o, *xg = a.dout, *out = a.out;
  const float* lse = a.lse;
  __builtin_amdgcn_sched_barrier(0);   // these loads are under way during the arithmetic
  const int N = l.N, T = owner_slots(N), U = view_units(N), n_col = l.n_col, n_row = l.H - n_col;
  const int q = block & 7;
  // row-head pairs are dealt to the queues starting where the column-head pairs stopped, so that
  // a handful of pairs still spreads over as many XCDs as possible
  const int qr = (q - l.B * n_col) & 7;
  const int nc = (l.B * n_col - q + 7) >> 3, nr = (l.B * n_row - qr + 7) >> 3;  // pairs of this queue
  // Records are listed longest first and the empty ones last, and how many are real is only
  // known on the device: a workgroup that finds an empty record leaves at once, but it still
  // took a slot for a microsecond, and a thousand of them ahead of real units delay those by
  // several.  So the early part of each list (where the real records are unless a sequence is
  // filled to the last position, resp. has more than 128 question tokens) comes first for all
  // three kinds of unit, the remainders after them.
  const int T1 = min(T, (T >> 3) + 2), n_all = nc + nr;
  // the first two regions: column heads then question-token owners (early parts), or the reverse
  const int len_a = kChunksFirst ? n_all * T1 : nc * T, len_b = kChunksFirst ? nc * T : n_all * T1;
  int t = block >> 3, k0 = 0, first = 0;
  bool glob = kChunksFirst;
  if (t >= len_a) { t -= len_a; glob = !kChunksFirst; }
  const bool rows = t >= len_b && glob != kChunksFirst;  // row heads, early part
  t -= rows ? len_b : 0;
  glob &= !rows;
  first = rows ? nc : 0;
  int pairs = rows ? nr : glob ? n_all : nc, per = glob ? T1 : T;
  if (__builtin_expect(rows && t >= nr * T, 0)) {  // the rest of the three lists
    t -= nr * T; first = 0; pairs = nc; k0 = T; per = U - T;          // column heads
    if (t >= nc * (U - T)) {
      t -= nc * (U - T); first = nc; pairs = nr;                      // row heads
      if (t >= nr * (U - T)) {
        t -= nr * (U - T); first = 0; pairs = n_all; k0 = T1; per = T - T1; glob = true;  // question-token owners
      }
    }
  }
  // (the pointers have arrived here)
  asm("" : "+s"(t) : "s"(gidx), "s"(pads), "s"(perm_row), "s"(perm_col), "s"(rng_row), "s"(rng_col), "s"(xq), "s"(xk), "s"(xv),
      "s"(xo), "s"(xg), "s"(out), "s"(lse));
  // The hardware hands consecutive workgroups of an XCD to its shader engines in rotation and
  // stalls when the engine whose turn it is has no room, so each engine must see the same mix
  // of units: the pair order rotates from sweep to sweep.
  int turn;
  const int kk = uniform_div(t, max(pairs, 1), turn);
  uniform_div(turn + kk, max(pairs, 1), turn);
  const bool real = pairs > 0 && kk < per;
  const int k = real ? k0 + kk : 0, j = real ? first + turn : 0;
  w.view = j < nc ? 1 : 0;
  const int pair = pick(j < nc, q + 8 * j, qr + 8 * (j - nc)), heads = max(pick(j < nc, n_col, n_row), 1);
  int b, i;
  if (__builtin_expect(l.B < 1 << 20, 1)) {
    b = uniform_div(pair, heads, i);
  } else {
    b = (int)((unsigned)pair / (unsigned)heads);
    i = pair - b * heads;
  }
  b = real ? b : 0;
  i = real ? i : 0;
  const int order = i + (real && j >= nc ? n_col : 0);
  w.b = b;
  const int4* list = pick<const int4*>(glob, l.gunit, pick<const int4*>(j < nc, l.unit_col, l.unit_row));
  // (A byte of the head order, indexed by a run-time value, would be fetched with a vector load; the
  // containing 32-bit word comes with the other kernel arguments.)
  unsigned heads4 = reinterpret_cast<const unsigned*>(a.head_order)[order >> 2];
  // The header is fetched together with the record: tables
  // built for another (B, N), or never built, make every workgroup leave before it uses a word
  // of them.  All of these reads stay inside the mate_segments_bytes(B, N) bytes the caller
  // must provide.
  i32x8 r = *reinterpret_cast<const i32x8*>(list + ((size_t)b * pick(glob, T, U) + k) * 2);
  i32x4 h = *reinterpret_cast<const i32x4*>(l.hdr);
  i32x4 cnt = *reinterpret_cast<const i32x4*>(l.hdr + kHdrWords + (size_t)b * kCountWords);
  asm("" : "+s"(h), "+s"(heads4) : "s"(r), "s"(cnt));
  w.bh = b * l.H + (int)((heads4 >> (8 * (order & 3))) & 0xffu);
  UnitPlan& u = w.u;
  u.kind = r[0];
  if (!real || h[0] != kMagic || h[1] != l.B || h[2] != N || u.kind == UNIT_NONE) return false;
  u.t0 = r[1];
  u.s_lo = r[2];
  u.s_hi = r[3];
  u.t_begin = r[4];
  u.t_end = r[5];
  u.part = r[6];
  u.n_chunks = r[7];
  u.G = cnt[C_G];
  u.L = cnt[C_L];
  u.P = cnt[C_P];
  u.n_t0 = (u.G + BN - 1) / BN;
  const size_t seq = (size_t)b * N;
  w.global_idx = gidx + seq;
  w.slot_rng = pick(j < nc, rng_col, rng_row) + seq;
  const int* perm_v = pick(j < nc, perm_col, perm_row) + seq;
  u.str_list = pick<const int*>(glob, perm_row + seq, perm_v);  // row order: the contiguous one
  u.own_list = pick<const int*>(glob, gidx + seq, pick<const int*>(r[0] == UNIT_LOCAL, perm_v, pads + seq));
  u.own_count = glob ? cnt[C_G] : r[0] == UNIT_LOCAL ? r[7] : cnt[C_P];
  return join_chunks<kJoin>(u, glob);
}

// The same for launches of many records: every step is loaded where it is first needed and an empty record asks for nothing more,
// which gains where most are empty, as they are where sequences differ in length.  us, the form above and this one.  Above the line, lengths
// that differ: forward of 13 sequences of up to 6512, 16 heads (26832 records) 97.4 and 94.5, 16 of 4096 (20992) 73.7 and 72.1, 32 of 2048, 12
// heads (16128) 55.8 and 54.9, backward there 240 and 235, 230 and 227, 170 and 168; full sequences: forward of 32 x 2048 118.8 and
// 117.7, 48 x 1024 (16896) 114.4 and 113.7, 8 x 8192 (20736) 209.8 and 209.2, 64 x 512 (12288) 74.2 and 74.2, backward the same within 0.5 %.
// Below it: forward and backward of 2 x 8192 (5184) 52.4 and 52.8, 147.1 and 148.8, forward of 4 x 8192 (10368) 103.5 and 103.4, of lengths
// that differ 36.9 and 37.5, of 16 x 2048 (8064) 29.4 and 29.7.  (A forward with its chunks first, may_chunk and B H T <= 3072, has
// 11880 records at most.)
constexpr int kManyRecords = 12000;
template <bool kChunksFirst, bool kJoin>
__device__ inline bool take_unit_of_many(const AttnArgs& a, int block, Work& w) {
  const int T = a.seg.tiles, U = a.seg.units, N = a.N, n_col = a.n_col, n_row = a.H - n_col;
  const int q = block & 7;
  const int qr = (q - a.B * n_col) & 7;
  const int nc = (a.B * n_col - q + 7) >> 3, nr = (a.B * n_row - qr + 7) >> 3;
  const int E = min(U, T), T1 = min(T, (T >> 3) + 2);
  int t = block >> 3;
  const int n_all = nc + nr;
  const int len_a = kChunksFirst ? n_all * T1 : nc * E, len_b = kChunksFirst ? nc * E : n_all * T1;
  bool glob = kChunksFirst;
  int first = 0, pairs = glob ? n_all : nc, k0 = 0, per = glob ? T1 : E;
  if (t >= len_a) {
    t -= len_a; glob = !kChunksFirst; pairs = glob ? n_all : nc; per = glob ? T1 : E;
    if (t >= len_b) {                      // row heads, early part
      t -= len_b; first = nc; pairs = nr; k0 = 0; per = E; glob = false;
      if (t >= nr * E) {                   // column heads, rest
        t -= nr * E; first = 0; pairs = nc; k0 = E; per = U - E;
        if (t >= nc * (U - E)) {           // row heads, rest
          t -= nc * (U - E); first = nc; pairs = nr;
          if (t >= nr * (U - E)) {         // question-token owners, rest
            t -= nr * (U - E); first = 0; pairs = n_all; k0 = T1; per = T - T1; glob = true;
          }
        }
      }
    }
  }
  if (pairs <= 0) return false;
  int at, i;
  const int kk = uniform_div(t, pairs, at), k = k0 + kk;
  if (kk >= per) return false;
  uniform_div(at + kk, pairs, at);
  const int j = first + at;
  w.view = j < nc ? 1 : 0;
  const int pair = w.view ? q + 8 * j : qr + 8 * (j - nc), heads = w.view ? n_col : n_row;
  int b;
  if (__builtin_expect(a.B < 1 << 20, 1)) {
    b = uniform_div(pair, heads, i);
  } else {
    b = (int)((unsigned)pair / (unsigned)heads);
    i = pair - b * heads;
  }
  const int order = w.view ? i : n_col + i;
  const unsigned heads4 = reinterpret_cast<const unsigned*>(a.head_order)[order >> 2];
  w.b = b;
  w.bh = b * a.H + (int)((heads4 >> (8 * (order & 3))) & 0xffu);
  const int4* rec = glob ? a.seg.gunit + ((size_t)b * T + k) * 2
                         : a.seg.unit[w.view] + ((size_t)b * U + k) * 2;
  const int h_magic = a.seg.hdr[0], h_B = a.seg.hdr[1], h_N = a.seg.hdr[2];
  const int4 r0 = rec[0], r1 = rec[1];
  const int* cnt = a.seg.counts + (size_t)b * kCountWords;
  UnitPlan& u = w.u;
  u.kind = r0.x;
  if (h_magic != kMagic || h_B != a.B || h_N != a.N) return false;
  if (u.kind == UNIT_NONE) return false;
  u.t0 = r0.y;
  u.s_lo = r0.z;
  u.s_hi = r0.w;
  u.t_begin = r1.x;
  u.t_end = r1.y;
  u.part = r1.z;
  u.n_chunks = r1.w;
  u.G = cnt[C_G];
  u.L = cnt[C_L];
  u.P = cnt[C_P];
  u.n_t0 = (u.G + BN - 1) / BN;
  const size_t seq = (size_t)b * N;
  w.global_idx = a.seg.global_idx + seq;
  w.slot_rng = a.seg.slot_rng[w.view] + seq;
  const int* perm_v = a.seg.perm[w.view] + seq;
  u.str_list = glob ? a.seg.perm[0] + seq : perm_v;  // row order: the contiguous one
  u.own_list = glob ? w.global_idx : u.kind == UNIT_LOCAL ? perm_v : a.seg.pad_idx + seq;
  u.own_count = glob ? u.G : u.kind == UNIT_LOCAL ? r1.w : u.P;
  return join_chunks<kJoin>(u, glob);
}

// Streamed tile t of a unit: which index list, first slot, last valid slot.
__device__ inline void tile_source(const UnitPlan& u, const int* global_idx, int t,
                                   const int*& list, int& base, int& last) {
  if (t < u.n_t0) { list = global_idx; base = t * BN; last = u.G - 1; }
  else { list = u.str_list; base = u.s_lo + (t - u.n_t0) * BN; last = u.s_hi - 1; }
}

// A unit of at most 64 rows has work for two wavefronts; the other two take half of it: wavefronts w and
// w + 2 own the same 32 rows, w meets the first 32 rows of every streamed tile and w + 2 the last 32, and the
// two results are added (through LDS) before anything is stored.  Most question-token owners are such units,
// and they are the longest chain of tiles of a small launch.  (One or two tiles are not worth the addition: forward /
// backward of one sequence of 64 with 12 heads 6.2/14.7 us split, 5.6/13.1 whole; from three on split is faster.)
//
// With kTiles = 2 tiles in a stage, a unit of at most 32 rows has work for all four: wavefronts 2 h + j meet half h of
// tile j of every stage.
template <int kTiles>
struct OwnerSplit {
  bool on;
  bool four;  // all four own the same 32 rows
  int block;  // the wavefront's 32-row block of owned rows
  int half;   // and of streamed rows
  int tile;   // and, if four, of the tiles
  __device__ inline OwnerSplit(const UnitPlan& u, int wave)
      : on(u.own_count - u.t0 <= BM / 2 && u.t_end - u.t_begin >= 3), four(kTiles == 2 && on && u.own_count - u.t0 <= BM / 4),
        block(four ? 0 : on ? wave & 1 : wave), half(wave >> 1), tile(wave & 1) {}
  __device__ inline bool meets(int j) const { return kTiles == 1 || !four || j == tile; }
  __device__ inline bool writes(int wave) const { return !on || wave < (kTiles == 2 && four ? 1 : 2); }
  // [first, end): the part of the slots [lo, hi) met in the tile that begins at slot `base`
  __device__ inline int first(int base, int lo) const { return on ? max(lo, base + 32 * half) : lo; }
  __device__ inline int end(int base, int hi) const { return on ? min(hi, base + 32 * half + 32) : hi; }
};

// Per-lane view of the owned row: position, and the streamed-slot window it may meet.
struct OwnedRow {
  int stage_tok;      // token position of owned row threadIdx.x (-1 past the end or past row 127):
                      // what the epilogue's row table holds, fetched together with `pos`
  int pos;            // token position (rows past the end repeat the last valid one)
  bool valid;
  int lo, hi;         // this row's window of streamed table slots
  int w_lo, w_hi;     // union over the wavefront's 32 rows
  int a_lo, a_hi;     // intersection over the wavefront's rows
  bool wave_active;   // the wavefront owns at least one valid row
};
__device__ inline OwnedRow owned_row(const Work& w, int wave, int m) {
  const UnitPlan& u = w.u;
  OwnedRow r;
  const int slot_raw = u.t0 + wave * 32 + m;
  const int slot = min(slot_raw, u.own_count - 1);
  r.valid = slot_raw < u.own_count;
  r.wave_active = u.t0 + wave * 32 < u.own_count;
  r.pos = u.own_list[slot];
  {
    const int row = u.t0 + (int)threadIdx.x;
    r.stage_tok = threadIdx.x < BM && row < u.own_count ? u.own_list[row] : -1;
  }
  r.lo = 0;
  r.hi = u.L;
  if (u.kind == UNIT_LOCAL) {
    const int2 g = w.slot_rng[slot];
    r.lo = g.x;
    r.hi = g.y;
  }
  r.w_lo = __builtin_amdgcn_readlane(r.lo, 0);   // wave-uniform, kept in scalar registers
  r.w_hi = __builtin_amdgcn_readlane(r.hi, 31);
  r.a_lo = __builtin_amdgcn_readlane(r.lo, 31);
  r.a_hi = __builtin_amdgcn_readlane(r.hi, 0);
  return r;
}

// The wavefront's 32 owned rows of a tensor on their way to operand order.  Whole rows are loaded, eight per
// instruction (lane l holds 16-byte piece l & 7 of row (l >> 3) + 8 i), and pass through 4 KB of LDS of the wavefront's
// own.  Operands loaded straight from global memory (lane m: 16 bytes of row m) touch 32 lines per instruction and
// each line four times, and at the start of a launch every wavefront of a CU wants its 4 (forward), 8 (dK/dV) or 12
// (dQ) such loads at once.  delta comes from the rows as they are loaded.  Training steps, us, four runs of each in turn: 2 x 8192,
// 16 heads 196.9 -> 195.7 (runs of one side differ by 0.7 %), bucketed 138.5 -> 136.1, 8 x 2048 with long cells 169.9 -> 168.0,
// 16 ragged sequences of 4096 554 -> 545, 32 x 512, 12 heads 106.9 -> 106.6; single sequences the same.
struct OwnedTile {
  bf16x8 v[4];  // (an array of HIP's uint4 class ends up in scratch memory)
  // `pos`: lane m and m + 32 hold the token of row m; X wave-uniform
  __device__ __forceinline__ void load(const unsigned short* X, int pos, int lane) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      v[i] = *reinterpret_cast<const bf16x8*>(X + (unsigned)__shfl(pos, (lane >> 3) + 8 * i, 64) * kD + 8 * (lane & 7));
  }
  // Operand order.  `room`: 4 KB that no other wavefront uses; LDS keeps a wavefront's accesses in order.
  // 32 x 32 tiles: lane m, half hl holds dims 16 ks + 8 hl .. + 7 of row m.
  __device__ __forceinline__ void operands(bf16x8 (&f)[4], char* room, int lane) const {
    through(room, lane, [&] {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) f[ks] = read_plain(room, plain_off(lane & 31, lane >> 5, ks));
    });
  }
  // 16 x 16 tiles: lane 16 q + r holds dims 32 ks + 8 q .. + 7 of rows r and 16 + r, [ks][which].
  __device__ __forceinline__ void operands(bf16x8 (&f)[2][2], char* room, int lane) const {
    through(room, lane, [&] {
      const int r = lane & 15;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) f[ks][cb] = read_plain(room, (16 * cb + r) * 128 + (((4 * ks + (lane >> 4)) ^ swz(r)) << 4));
    });
  }
  template <class Read>
  __device__ __forceinline__ void through(char* room, int lane, Read&& read) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = (lane >> 3) + 8 * i;
      *reinterpret_cast<bf16x8*>(room + row * 128 + (((lane & 7) ^ swz(row & 15)) << 4)) = v[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    read();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
};
// Sums of x over the eight lanes that hold one row of an OwnedTile.
__device__ __forceinline__ float row_sum8(float x) {
  auto add = [&](auto ctrl) {
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  add(std::integral_constant<int, 0xb1>{});   // lane ^ 1
  add(std::integral_constant<int, 0x4e>{});   // lane ^ 2
  add(std::integral_constant<int, 0x141>{});  // mirrored within eight lanes: the other four
  return x;
}
// x . y of a row, eight lanes of eight dims each.
__device__ __forceinline__ float row_dot8(const bf16x8& x, const bf16x8& y) {
  float d = 0.f;
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const bf16x2 u = {x[e], x[e + 1]}, v = {y[e], y[e + 1]};
    d = __builtin_amdgcn_fdot2_f32_bf16(u, v, d, false);
  }
  return row_sum8(d);
}
// delta = dO . O of the rows of two OwnedTiles: every lane gets its row m's.  `room` as above (128 bytes of it).
__device__ __forceinline__ float row_delta(const OwnedTile& g, const OwnedTile& o, char* room, int lane) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float d = row_dot8(g.v[i], o.v[i]);
    if ((lane & 7) == 0) reinterpret_cast<float*>(room)[(lane >> 3) + 8 * i] = d;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const float d = reinterpret_cast<const float*>(room)[lane & 31];
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return d;
}

// Final results: C tile pairs (columns = owned rows, registers = head dims) scaled, rounded to
// bf16, transposed through LDS and stored as whole 128-byte token rows.  `stage` needs 16 KB per
// tensor: 128 rows of 128 bytes whose 16-byte chunks are XOR-swizzled with the row number so
// that both the column-wise writes and the row-wise reads spread over all banks.  One barrier;
// the staging area must not be reused by the caller afterwards without another one.
// (stage_rows: one wavefront-slot's 32 rows x 32 dims; flush_rows: after a barrier, every wavefront its 32 rows)
__device__ __forceinline__ void stage_rows(const f32x16& a, float mul, char* stage, int wrow, int db, int hl) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    uint2 w;
    w.x = pack2(a[4 * g] * mul, a[4 * g + 1] * mul);
    w.y = pack2(a[4 * g + 2] * mul, a[4 * g + 3] * mul);
    *reinterpret_cast<uint2*>(stage + wrow * 128 + (((4 * db + g) ^ (wrow & 7)) << 4) + 8 * hl) = w;
  }
}
// The same of 16 x 16 tiles, [16 dims][16 owned rows]: register e of lane 16 q + r is dim 16 d + 4 q + e of row 16 cb + r.
// They stay quads of registers from the loop to the stores: gathered into sixteen neighbours each, dK and dV took 158 moves at the end of
// every unit (see QuadAddr for what the two cost together).
// (Rows r and r + 8 of a write meet in one bank.)
typedef f32x4 QuadAcc[4][2];
__device__ __forceinline__ void stage_rows_quad(const f32x4 (&a)[2], float mul, char* stage, int row0, int d, int lane) {
  const int r = lane & 15, q = lane >> 4;
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    const int row = row0 + 16 * cb + r;
    uint2 w;
    w.x = pack2(a[cb][0] * mul, a[cb][1] * mul);
    w.y = pack2(a[cb][2] * mul, a[cb][3] * mul);
    *reinterpret_cast<uint2*>(stage + row * 128 + (((2 * d + (q >> 1)) ^ (r & 7)) << 4) + 8 * (q & 1)) = w;
  }
}
template <bool kThrough = true>
__device__ __forceinline__ void flush_rows(unsigned short* out, const char* stage, const int* row_tok, int wave, int lane) {
  const ResultRows<kThrough> rows(out);
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = wave * 32 + it * 8 + (lane >> 3), piece = lane & 7;
    const int tok = row_tok[row];
    if (tok >= 0)
      rows.store((unsigned)tok * (kD * 2) + piece * 16, *reinterpret_cast<const u32x4*>(stage + row * 128 + ((piece ^ (row & 7)) << 4)));
  }
}
template <int kTensors, bool kThrough = true>
__device__ inline void store_owned_rows(const f32x16 (*acc[kTensors])[2], const float (&mul)[kTensors],
                                        unsigned short* const (&out)[kTensors], char* stage,
                                        const int* row_tok, int wave, int lane) {
#pragma unroll
  for (int x = 0; x < kTensors; ++x)
#pragma unroll
    for (int db = 0; db < 2; ++db)
      stage_rows((*acc[x])[db], mul[x], stage + x * (BM * 128), wave * 32 + (lane & 31), db, lane >> 5);
  __syncthreads();
#pragma unroll
  for (int x = 0; x < kTensors; ++x) flush_rows<kThrough>(out[x], stage + x * (BM * 128), row_tok, wave, lane);
}
template <int kTensors>
__device__ inline void store_owned_rows(const QuadAcc* (&acc)[kTensors], const float (&mul)[kTensors], unsigned short* const (&out)[kTensors],
                                        char* stage, const int* row_tok, int wave, int lane) {
#pragma unroll
  for (int x = 0; x < kTensors; ++x)
#pragma unroll
    for (int d = 0; d < 4; ++d) stage_rows_quad((*acc[x])[d], mul[x], stage + x * (BM * 128), wave * 32, d, lane);
  __syncthreads();
#pragma unroll
  for (int x = 0; x < kTensors; ++x) flush_rows(out[x], stage + x * (BM * 128), row_tok, wave, lane);
}

// ---- partial results of chunked question-token owners ------------------------------------------
// A chunk leaves its fp32 accumulators in the workspace in register order, [item][8][64 lanes] pairs
// with item = 2 wavefront + dim block, so every access is 512 contiguous bytes and the merge works on
// the same registers as the chunks did.  Merging adds the chunks in order, so the result does not
// depend on who merges, or when.
//
// Forward and dK/dV: the chunk of an owner tile that arrives last merges inside the same launch
// (a finalize kernel of its own cost 4.8 us in the forward and 6.4 us in the backward at B = 2,
// N = 8192, H = 16, nearly all of it the launch), and so does dQ's where all three gradients are one launch.  Where dQ has
// one of its own: merged by the first workgroups of the dK/dV kernel, behind the kernel boundary.
constexpr int kItemFloats = 16 * 64;  // one wavefront's accumulator of one dim block
// (Of 16 x 16 tiles an item is two of the four d, its register 8 (d & 1) + 4 cb + e.)
__device__ __forceinline__ float item_register(const f32x16 (&acc)[2], int item, int i) { return acc[item][i]; }
__device__ __forceinline__ float item_register(const QuadAcc& acc, int item, int i) { return acc[2 * item + (i >> 3)][(i >> 2) & 1][i & 3]; }
__device__ __forceinline__ void set_item_register(f32x16 (&acc)[2], int item, int i, float x) { acc[item][i] = x; }
__device__ __forceinline__ void set_item_register(QuadAcc& acc, int item, int i, float x) { acc[2 * item + (i >> 3)][(i >> 2) & 1][i & 3] = x; }
template <bool kShared, class Acc>
__device__ __forceinline__ void store_partial(const Acc& acc, float mul, float* __restrict__ part, int wave, int lane) {
  asm volatile("" : "+v"(lane));  // keeps the address arithmetic out of the tile loop's registers
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int i = 0; i < 8; ++i)
      put_pair<kShared>(part + (2 * wave + db) * kItemFloats + (i * 64 + lane) * 2, item_register(acc, db, 2 * i) * mul,
                        item_register(acc, db, 2 * i + 1) * mul);
}
// The same registers through LDS (two blocks of kItemFloats floats at p): acc = own acc + other p.
template <class Acc>
__device__ __forceinline__ void put_items(char* p, const Acc& acc, int lane) {
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int i = 0; i < 8; ++i)
      *reinterpret_cast<float2*>(p + ((x * 8 + i) * 64 + lane) * 8) = make_float2(item_register(acc, x, 2 * i), item_register(acc, x, 2 * i + 1));
}
template <class Acc>
__device__ __forceinline__ void add_items(const char* p, Acc& acc, float own, float other, int lane) {
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float2 v = *reinterpret_cast<const float2*>(p + ((x * 8 + i) * 64 + lane) * 8);
      set_item_register(acc, x, 2 * i, fmaf(v.x, other, item_register(acc, x, 2 * i) * own));
      set_item_register(acc, x, 2 * i + 1, fmaf(v.y, other, item_register(acc, x, 2 * i + 1) * own));
    }
}
// kBatch chunks of one item with all loads issued before the first use (the pin: left alone, the
// compiler keeps only a few in flight and the merge becomes a chain of memory round trips).
constexpr int kBatch = 4;
template <bool kShared>
__device__ __forceinline__ void load_items(float2 (&v)[kBatch][8], const float* part0, int item, int c0, int n_chunks, int lane) {
#pragma unroll
  for (int e = 0; e < kBatch; ++e)
#pragma unroll
    for (int i = 0; i < 8; ++i)
      v[e][i] = get_pair<kShared>(part0 + (size_t)min(c0 + e, n_chunks - 1) * (BM * kD) + item * kItemFloats + (i * 64 + lane) * 2);
#pragma unroll
  for (int e = 0; e < kBatch; ++e)
#pragma unroll
    for (int i = 0; i < 8; i += 4)
      asm volatile("" ::"v"(v[e][i].x), "v"(v[e][i].y), "v"(v[e][i + 1].x), "v"(v[e][i + 1].y), "v"(v[e][i + 2].x),
                   "v"(v[e][i + 2].y), "v"(v[e][i + 3].x), "v"(v[e][i + 3].y));
}
// Zero fill of the rows of a pad unit in kTensors tensors.  The positions of all the rows a
// thread will write are loaded first (independent loads, one round trip), then the stores go
// out back to back.
template <int kTensors>
__device__ inline void zero_pad_rows(unsigned short* const (&out)[kTensors], const UnitPlan& u, int tid) {
  constexpr int kRounds = kPadSlots * 8 / kThreads;  // rows of 8 pieces; 32 rows per round
  const int piece = tid & 7;
  int tok[kRounds];
#pragma unroll
  for (int i = 0; i < kRounds; ++i) {
    const int row = u.t0 + (tid >> 3) + i * (kThreads / 8);
    tok[i] = row < u.own_count ? u.own_list[row] : -1;
  }
#pragma unroll
  for (int x = 0; x < kTensors; ++x)
#pragma unroll
    for (int i = 0; i < kRounds; ++i)
      if (tok[i] >= 0)
        ResultRows<>(out[x]).store((unsigned)tok[i] * (kD * 2) + piece * 16, u32x4{0, 0, 0, 0});
}

// Workspace carving (float words).  Partial buffers are per (b,h): [UG][BM][64].
__host__ __device__ inline size_t part_words_per_bh(int N) { return (size_t)owner_slots(N) * BM * kD; }
__host__ __device__ inline size_t stat_words_per_bh(int N) { return (size_t)owner_slots(N) * BM * 2; }

}  // namespace mate
