// Streaming 64-row x 64-dim bf16 tiles from global memory straight into LDS (gfx950
// global_load_lds_dwordx4), and reading them back as MFMA operands, plain or transposed
// (ds_read_b64_tr_b16).  No registers are spent on staging, so several tiles can be in flight.
//
// LDS tile layout: 64 rows of 128 bytes, no padding; the eight 16-byte chunks of row r are
// stored XOR-swizzled, chunk c at slot c ^ swz(r), with swz(r) built from bits 1..3 of r:
//   * the 16 lanes of a plain 16-byte operand read that are served together hit 16 distinct
//     (bank-half, slot) pairs, whether the wavefront reads 32 rows at two chunk indexes (32x32x16) or
//     16 rows at four (16x16x32);
//   * 4 consecutive rows read at two adjacent chunks (transposing 8-byte reads) do too.
// Lanes served together are not 16 consecutive ones: a ds_read_b128 takes lanes 0-3, 12-15 and 20-27,
// then 4-11, 16-19 and 28-31, then the same of the upper 32.  So in a 16-row read rows 0-3 and 12-15 of one
// chunk meet rows 4-11 of the next one; with swz built for 16 consecutive lanes (bits 1, 2, 3 as they are)
// the conflict counter showed 4.0 cycles for each plain read of a product, half of its time, and now 0.0.
// A wave-wide load instruction deposits lane l's 16 bytes at (LDS base) + 16 l, i.e. rows
// l / 8 of an 8-row group, slot l % 8; the swizzle is applied by choosing which global chunk
// each lane fetches.
//
// Hardware facts this relies on (checked on the device with known data):
//   * global_load_lds_dwordx4: lane l's data lands at M0-base + 16 l.
//   * ds_read_b64_tr_b16: within each group of 16 lanes, lane i receives element (i & 3) of the
//     four 8-byte rows addressed by lanes (i >> 2), (i >> 2) + 4, + 8, + 12 of the group.
#pragma once
#include <hip/hip_runtime.h>

#include "mfma_common.h"

namespace mate {

constexpr int kTileBytes = 64 * 128;  // one streamed tile in LDS

__host__ __device__ inline int swz(int r) { return (((r >> 1) & 1) << 2) | ((((r >> 3) ^ (r >> 2)) & 1) << 1) | ((r >> 2) & 1); }
// The same for tiles that are read as QuadLanes says (below): rows 8 i + 4 h + j (i, j = 0 .. 3) at four chunk indexes,
// and rows 8 i + 4 h + j of two i at two adjacent ones.  Bit 2 of a row (h) is not part of it.
__host__ __device__ inline int swz_quad(int r) { return (((r >> 1) & 1) << 2) | ((((r >> 3) ^ (r >> 4)) & 1) << 1) | ((r >> 4) & 1); }

typedef short s16x4 __attribute__((ext_vector_type(4)));

// ---- issuing loads -------------------------------------------------------------------------
// A wavefront covers rows 16 w .. 16 w + 15 of a tile with two instructions (8 rows each).
struct LoadLane {
  int row0;    // this lane's row for instruction 0 (instruction 1: row0 + 8)
  int chunk0;  // global chunk this lane fetches for instruction 0 (instruction 1: chunk0 ^ 2)
};
template <bool kQuad = false>
__host__ __device__ inline LoadLane make_load_lane(int wave, int lane) {
  LoadLane l;
  l.row0 = 16 * wave + (lane >> 3);
  l.chunk0 = (lane & 7) ^ (kQuad ? swz_quad(l.row0) : swz(l.row0 & 15));  // of row0 + 8: ^ 2
  return l;
}

// The load instructions are written as inline assembly on purpose: the compiler then does not
// know that they write LDS, so it does not guard later LDS reads with "wait for every
// outstanding load" (which would drain the prefetches of later tiles on every iteration).
// Ordering against the LDS reads is by the explicit waits and barriers of the caller.  The
// compiler's own vmcnt bookkeeping for ordinary loads stays safe: loads it cannot see only make
// its waits stricter, since loads retire in issue order.
// (The low half of the generic address of LDS is the LDS offset; a cast to the LDS address space would add
// a comparison with the null pointer to every load.)
__device__ __forceinline__ unsigned lds_addr(const void* p) { return __builtin_amdgcn_readfirstlane((unsigned)(size_t)p); }
// Address form: 64-bit base in scalar registers (wave-uniform) plus a 32-bit byte offset per
// lane, so the per-lane address arithmetic is one shift-add.
__device__ inline void load_to_lds_16(const void* base /* wave-uniform */, unsigned byte_off,
                                      const void* lds_dst /* wave-uniform */) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(byte_off), "s"(base), "s"(lds_addr(lds_dst)) : "memory", "m0");
}
__device__ inline void load_to_lds_4(const void* base /* wave-uniform */, unsigned byte_off,
                                     const void* lds_dst /* wave-uniform */) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
               :: "v"(byte_off), "s"(base), "s"(lds_addr(lds_dst)) : "memory", "m0");
}

// Rows `tok0` / `tok1` (token positions of this lane's two rows) of tensor X (wave-uniform
// base; a (sequence, head) slice, so byte offsets fit 32 bits) into the tile at LDS address
// `tile` (wave-uniform).
__device__ inline void issue_tile(const unsigned short* X, int tok0, int tok1,
                                  const LoadLane& l, const char* tile, int wave) {
  const char* d0 = tile + (16 * wave) * 128;
  load_to_lds_16(X, (unsigned)tok0 * 128u + l.chunk0 * 16, d0);
  load_to_lds_16(X, (unsigned)tok1 * 128u + (l.chunk0 ^ 2) * 16, d0 + 8 * 128);
}

// One 32-bit word per lane, word `index` of the array at `base` (wave-uniform), to 64
// consecutive words at `dst` (wave-uniform LDS address): token indices, or per-row statistics,
// of a streamed tile.
__device__ inline void issue_row_words(const void* base, int index, const void* dst) {
  load_to_lds_4(base, (unsigned)index * 4u, dst);
}

// ---- waiting ------------------------------------------------------------------------------
// "At most n of my vector-memory loads still outstanding" (n wave-uniform, 0 <= n; values above
// kMax are treated as kMax).  Loads complete in issue order, so this retires everything issued
// before the last n.  n is rounded down to a value with an encoding below (waiting for more is
// always safe).
template <int kMax = 12>
__device__ inline void wait_vmcnt_le(int n) {
  if (kMax >= 12 && n >= 12) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
  else if (kMax >= 11 && n >= 11) asm volatile("s_waitcnt vmcnt(11)" ::: "memory");
  else if (kMax >= 10 && n >= 10) asm volatile("s_waitcnt vmcnt(10)" ::: "memory");
  else if (kMax >= 9 && n >= 9) asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
  else if (kMax >= 8 && n >= 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  else if (kMax >= 6 && n >= 6) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
  else if (kMax >= 5 && n >= 5) asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
  else if (kMax >= 4 && n >= 4) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Workgroup barrier without the release/acquire fence of __syncthreads (which would wait for
// every outstanding load, including the prefetches of later tiles).  The caller has already
// waited for exactly the loads that must be visible.
__device__ inline void barrier_no_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ---- reading operands -----------------------------------------------------------------------
// Plain operand: tile row = 32 blk + m, dims 16 ks + 8 hl .. + 7 (A operand with k = dims).
// plain_off(ks) is per lane; add blk * 32 * 128 bytes.
__host__ __device__ inline int plain_off(int m, int hl, int ks) {
  return m * 128 + (((2 * ks + hl) ^ swz(m & 15)) << 4);
}
__device__ inline bf16x8 read_plain(const char* tile, int off) {
  return *reinterpret_cast<const bf16x8*>(tile + off);
}

// Transposed operand: A row = dim 32 db + m, k = tile rows.  For a C tile computed with rows =
// tile rows (no permutation), the eight registers 8 tt .. 8 tt + 7 of a lane in half hl are tile
// rows 16 tt + 4 hl + {0..3} and 16 tt + 8 + 4 hl + {0..3} of the 32-row block: two transposing
// reads.  tr_off(db, half) is per lane; add (32 blk + 16 tt) * 128 bytes.
__host__ __device__ inline int tr_off(int lane, int db, int half) {
  const int i = lane & 15, g = lane >> 4, hl = g >> 1;
  const int jl = 4 * hl + (i >> 2) + 8 * half;              // row inside the 16-row group
  const int chunk = db * 4 + 2 * (g & 1) + ((i & 3) >> 1);  // dims 32 db + 16 (g & 1) + 4 (i & 3)
  return jl * 128 + ((chunk ^ swz(jl)) << 4) + ((i & 1) << 3);
}
__device__ inline bf16x8 read_transposed(const char* tile, int off_lo, int off_hi) {
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(tile + off_lo));
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(tile + off_hi));
  union { s16x4 h[2]; bf16x8 v; } u;
  u.h[0] = a;
  u.h[1] = b;
  return u.v;
}

// The same two reads from an LDS address (the low half of a generic address).  Tiles begin at multiples of 128 bytes, so
// all of a lane's addresses in a tile follow from three by exclusive or: one addition and one exclusive or each where
// address = tile + offset takes an addition and a register per offset.
typedef const __attribute__((address_space(3))) bf16x8* LdsOperand;
typedef __attribute__((address_space(3))) s16x4* LdsQuad;
__device__ inline bf16x8 read_plain(unsigned addr) { return *(LdsOperand)addr; }
__device__ inline bf16x8 read_transposed(unsigned addr_lo, unsigned addr_hi) {
  union { s16x4 h[2]; bf16x8 v; } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad)addr_lo);
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad)addr_hi);
  return u.v;
}
// A lane's part of the addresses: plain_off(0), tr_off(0, 0).
struct OperandLanes {
  unsigned plain, trans;
  __host__ __device__ explicit OperandLanes(int lane) : plain(plain_off(lane & 31, lane >> 5, 0)), trans(tr_off(lane, 0, 0)) {}
};
// Addresses of the operands in the tile at LDS address `tile` (wave-uniform).
struct PlainAddr {
  unsigned a[4];  // per 16-wide k slice
  __host__ __device__ PlainAddr(const OperandLanes& o, unsigned tile) {
    a[0] = tile + o.plain;
#pragma unroll
    for (int ks = 1; ks < 4; ++ks) a[ks] = a[0] ^ (ks << 5);
  }
};
// (The upper rows follow from the lower ones, eight rows on, and take no register of their own: with a tr_off(0, 1) that the compiler does
// not see to be the same, the dense forward takes 1 to 2.5 % longer, 1 x 1024, 4 heads 18.8 and 19.25 us.)
struct TransposedAddr {
  unsigned lo[2], hi[2];  // per 32-wide dim block
  __host__ __device__ TransposedAddr(const OperandLanes& o, unsigned tile) {
    lo[0] = tile + o.trans;
    lo[1] = lo[0] ^ 64;
    hi[0] = (lo[0] ^ 32) + 8 * 128;
    hi[1] = (lo[0] ^ 96) + 8 * 128;
  }
};

// Operands of v_mfma_f32_16x16x32_bf16 from a tile, lane 16 q + r.  The 32 rows of a block are two blocks of 16, row
// 8 i + 4 h + j being row 4 i + j of block h, so that in C tiles a lane holds rows 8 q .. 8 q + 7 of the 32: what the
// second contraction's operand holds, and two transposing reads bring of the other one.
struct QuadLanes {
  unsigned plain;  // row r of block 0, dims 8 q .. + 7 (the other 32 dims: ^ 64; block 1: + 512; the next 32 rows: + 4096)
  unsigned trans;  // rows 8 q .. + 3, columns 0 .. 15 (columns 16 d ..: ^ 32 d; rows 8 q + 4 .. + 7: + 512)
  __host__ __device__ explicit QuadLanes(int lane) {
    const int r = lane & 15, q = lane >> 4, row = 8 * (r >> 2) + (r & 3), row_t = 8 * q + (r >> 2);
    plain = row * 128 + ((q ^ swz_quad(row)) << 4);
    trans = row_t * 128 + ((((r & 3) >> 1) ^ swz_quad(row_t)) << 4) + ((r & 1) << 3);
  }
};
constexpr int kBlockBytes = 32 * 128, kHalfBlock = 4 * 128;  // in LDS: 32 rows, and from block 0 to block 1 of them
// A lane's two addresses in the tiles from LDS address `tile` on.  Blocks of 32 rows, halves of them and tensors one tile after the other lie multiples
// of 512 bytes apart, which the exclusive ors do not touch: immediate offsets (`at`).  us, backward, with an address of its own for each block and tensor and
// results gathered before they are stored (see QuadAcc), and so: 5 x 487, 12 heads 16.75 -> 16.35, 5 x 348, 16 heads 16.5 -> 15.95, 6 x 289, 12 heads
// 14.15 -> 13.95, 4 x 1024 25.5 -> 25.2, 2 x 8192, 16 heads 169.5 -> 164, dense 1 x 1024, 4 heads 54.15 -> 53.15, 8 x 300, 12 heads 32.0 -> 31.3.  (The first
// of these are what a short unit's beginning and end cost; with 32 x 32 tiles they were 16.2, 15.8, 13.75, 26.0, 173.5, 53.9 and 32.2.)
struct QuadAddr {
  unsigned plain, trans;
  __host__ __device__ __forceinline__ QuadAddr(const QuadLanes& l, unsigned tile) : plain(tile + l.plain), trans(tile + l.trans) {}
  __host__ __device__ __forceinline__ unsigned plain_at(unsigned at, int h, int k) const { return (plain ^ (64 * k)) + (at + h * kHalfBlock); }
  __host__ __device__ __forceinline__ unsigned trans_at(unsigned at, int d) const { return (trans ^ (32 * d)) + at; }
};
// Row r of block h of the 32 rows at `at`, dims 32 k + 8 q .. + 7.
__device__ __forceinline__ bf16x8 read_quad(const QuadAddr& a, unsigned at, int h, int k) { return read_plain(a.plain_at(at, h, k)); }
// Columns 16 d .. + 15 (operand rows) and rows 8 q .. + 7 (k) of the 32 rows at `at`.
__device__ __forceinline__ bf16x8 read_quad_transposed(const QuadAddr& a, unsigned at, int d) {
  return read_transposed(a.trans_at(at, d), a.trans_at(at + kHalfBlock, d));
}

// Tile row (0..31 inside a 32-row block) held in C register c of a lane in half hl when the A
// operand rows are fed unpermuted.
__device__ inline int c_row(int c, int hl) { return 8 * (c >> 2) + 4 * hl + (c & 3); }

}  // namespace mate
