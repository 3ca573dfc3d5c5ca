// Positional index that restarts at the beginning of each cell (Section 3.2: for sequences
// longer than 512 tokens the index of the positional embedding is reset per cell, so that no
// embeddings for large indices have to be learnt).  Integer work only.
//
// A cell is a maximal run of consecutive table tokens with the same (row, column).  A table
// token's index is its distance from the first token of its cell: position minus the largest
// "cell start" position at or before it, i.e. an inclusive running maximum over the sequence.
// Question tokens keep their absolute position, pads get 0.
//
// A lane takes four consecutive positions, a workgroup up to 4096 of one sequence.  Its neighbour's last position
// comes by a DPP move; the running maximum is the highest lane below with a start in a ballot, and one LDS exchange
// between wavefronts.  A workgroup that begins inside a sequence looks back for the cell it begins in: 64 positions are loaded
// with everything else, more only where a cell is longer.  Bound by latency: one round trip for the inputs and one
// barrier.  No load is behind a test of another one's value: with a position's row and column behind its flag they were two round
// trips.  By the kernel trace, before and with this form: one sequence of 512 3.2 -> 2.1 us, of 1999 3.9 -> 2.8; in a row of
// launches two of 8192 5.7 -> 3.5 and one of 16384 9.3 -> 3.4, which is the host's pace.
#include <hip/hip_runtime.h>

#include "launch.h"
#include "sequence_loads.h"

namespace mate {

constexpr int kPosEach = 4;
constexpr int kPosMaxThreads = 1024;
constexpr int kPosChunk = kPosEach * kPosMaxThreads;
constexpr int kPosMaxWaves = kPosMaxThreads / 64;

// Position i's inputs; three words, so that a neighbour's arrive by moves.
struct CellKey {
  int flag, row, col;
};
__device__ __forceinline__ bool starts_cell(const CellKey& k, const CellKey& before, bool first) {
  return (k.flag == 0) & (first | (before.flag != 0) | (before.row != k.row) | (before.col != k.col));
}
__device__ __forceinline__ int from_lane_below(int lane0, int x) {
  return __builtin_amdgcn_update_dpp(lane0, x, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}

struct PosInputs {
  const int *row, *col;
  const unsigned char* flags;
  int N;
  __device__ __forceinline__ CellKey at(int i) const {
    i = min(max(i, 0), N - 1);
    return {flags[i], row[i], col[i]};
  }
  // positions i0, i0 + 1, ... (anything past the end)
  template <int kEach>
  __device__ __forceinline__ void load(int i0, CellKey (&k)[kEach]) const {
    unsigned f = load_flags<kEach>(flags, i0, N);
    auto r = load_ids<kEach>(row, i0, N), c = load_ids<kEach>(col, i0, N);
    f = align_flags<kEach>(f, i0, N);
    r = align_ids<kEach>(r, i0, N);
    c = align_ids<kEach>(c, i0, N);
#pragma unroll
    for (int j = 0; j < kEach; ++j) k[j] = {(int)((f >> (8 * j)) & 0xffu), r[j], c[j]};
  }
};
// start[j] = the lane's latest cell start at or before its position j, -1 if it has none; `before`: the position before
// the wavefront's first
template <int kEach>
__device__ __forceinline__ void lane_starts(const CellKey (&k)[kEach], const CellKey& before, int i0, int N, int (&start)[kEach]) {
  const CellKey& last = k[kEach - 1];
  CellKey prev = {from_lane_below(before.flag, last.flag), from_lane_below(before.row, last.row), from_lane_below(before.col, last.col)};
  int latest = -1;
#pragma unroll
  for (int j = 0; j < kEach; ++j) {
    if (starts_cell(k[j], prev, i0 + j == 0) & (i0 + j < N)) latest = i0 + j;
    start[j] = latest;
    prev = k[j];
  }
}
// The latest of the lanes' `mine`s (-1: none), which ascend: wave-uniform.
__device__ __forceinline__ int latest_of(int mine) {
  const unsigned long long have = __ballot(mine >= 0);
  return have ? __builtin_amdgcn_readlane(mine, 63 - __clzll((long long)have)) : -1;
}

template <int kEach>
__global__ __launch_bounds__(kPosMaxThreads) void cell_positions_kernel(
    const int* __restrict__ row_ids, const int* __restrict__ col_ids,
    const unsigned char* __restrict__ flags, int N, int* __restrict__ out) {
  __shared__ int latest[kPosMaxWaves + 1];  // cell starts: before the workgroup's positions, then each wavefront's
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c0 = blockIdx.y * (kEach * kPosMaxThreads);
  const size_t seq = (size_t)b * N;
  const PosInputs in = {row_ids + seq, col_ids + seq, flags + seq, N};

  const int i0 = c0 + kEach * tid;
  const CellKey before = in.at(c0 + kEach * 64 * wave - 1);
  CellKey k[kEach];
  in.load(i0, k);
  int back = -1;
  bool open = false;   // the workgroup begins inside a cell whose start is not known yet
  if (c0 > 0 && wave == 0) {
    const CellKey e = in.at(c0 - 64 + lane), p = in.at(c0 - 65 + lane), first = in.at(c0);
    back = latest_of(starts_cell(e, p, false) ? c0 - 64 + lane : -1);   // (c0 is 4096 or more)
    open = back < 0 && first.flag == 0 && !starts_cell(first, in.at(c0 - 1), false);
  }
  int start[kEach];
  lane_starts(k, before, i0, N, start);
  const int mine = start[kEach - 1];
  const unsigned long long have = __ballot(mine >= 0), below = have & ((1ull << lane) - 1);
  const int from_below = __shfl(mine, below ? 63 - __clzll((long long)below) : lane, 64);
  const int wave_latest = have ? __builtin_amdgcn_readlane(mine, 63 - __clzll((long long)have)) : -1;
  if (lane == 0) {
    latest[1 + wave] = wave_latest;
    if (wave == 0) latest[0] = open ? -2 : back;
  }
  __syncthreads();
  if (c0 > 0) {
    // a cell of more than 64 positions: the whole workgroup looks, 4096 positions at a time
    for (int at = c0; at > 0 && __builtin_amdgcn_readfirstlane(latest[0]) == -2; at -= kEach * kPosMaxThreads) {
      CellKey x[kEach];
      const int j0 = at - kEach * kPosMaxThreads + kEach * tid;
      int s[kEach];
      in.load(j0, x);
      lane_starts(x, in.at(j0 - kEach * lane - 1), j0, N, s);
      const int found = latest_of(s[kEach - 1]);
      __syncthreads();
      if (lane == 0 && found >= 0) atomicMax(&latest[0], found);
      __syncthreads();
    }
  }
  // latest cell start before this wavefront's positions (later ones are later positions)
  const int earlier = latest_of(lane <= wave ? latest[lane] : -1);
  int at[kEach];
#pragma unroll
  for (int j = 0; j < kEach; ++j) {
    // a table token always has a cell start at or before it (position 0 at the latest)
    const int s = start[j] >= 0 ? start[j] : below ? from_below : earlier, i = i0 + j;
    at[j] = k[j].flag == 0 ? i - s : k[j].flag == 1 ? i : 0;
  }
  int* dst = out + seq;
  if (i0 + kEach <= N) {
    __builtin_memcpy(dst + i0, at, sizeof(at));
  } else {
#pragma unroll
    for (int j = 0; j < kEach; ++j)
      if (i0 + j < N) dst[i0 + j] = at[j];
  }
}

hipError_t launch_cell_positions(const int* row_ids, const int* col_ids, const unsigned char* flags,
                                 int B, int N, int* out, hipStream_t stream) {
  if (N < kPosEach) {
    hipLaunchKernelGGL(cell_positions_kernel<1>, dim3(B), dim3(64), 0, stream, row_ids, col_ids, flags, N, out);
    return hipGetLastError();
  }
  const int threads = N >= kPosChunk ? kPosMaxThreads : (N + kPosEach * 64 - 1) / (kPosEach * 64) * 64;
  hipLaunchKernelGGL(cell_positions_kernel<kPosEach>, dim3(B, (N + kPosChunk - 1) / kPosChunk), dim3(threads), 0, stream, row_ids,
                     col_ids, flags, N, out);
  return hipGetLastError();
}

}  // namespace mate
