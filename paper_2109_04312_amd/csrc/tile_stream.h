// The streaming loop shared by the forward, dQ and dK/dV kernels: two LDS stages, each holding one 64-row
// tile of two tensors (plus, optionally, one float per row of a third array); while one is consumed the
// other is filled by asynchronous global->LDS loads.  (More stages made the loop no faster: what a tile
// takes is its own dependent chain, and the LDS costs residency.)
//
// The token indices of a tile's 64 rows travel the same way (one word per lane into a ring
// shared by the workgroup; wavefront t mod 4 fetches the indices of tile t), a further tile ahead, so no
// load of the loop has a register destination and the only wait is the explicit one in acquire().  An
// index load is issued just before the data loads of the same iteration, so the wait for that tile's data
// also retires it, and the barrier that follows the wait publishes it to the other wavefronts -- in the very
// iteration that first reads it.
#pragma once
#include <hip/hip_runtime.h>

#include "d2l.h"
#include "stream_plan.h"

namespace mate {

constexpr int kStages = 2;
constexpr int kIdxSlots = 8;  // tiles of indices in the ring (three stages' are live at once; a power of two)

// kTiles = 2 (small launches, see small_forward in stream_plan.h): a stage holds two consecutive tiles, which the
// wavefronts meet one after the other or share, and every function below is for both.
// kQuad: tiles are read as QuadLanes says.
template <int kTileStage, int kTiles = 1, bool kQuad = false>
struct TileStream {
  static constexpr int kStageBytes = kTiles * kTileStage;
  const UnitPlan& u;
  const int* global_idx;
  char* stages;               // kStages * kStageBytes of LDS
  int (*ring)[BN];            // the workgroup's index ring [kIdxSlots][64]
  const unsigned short* X0;   // tensor staged at stage offset 0
  const unsigned short* X1;   // tensor staged at stage offset kTileBytes
  const float* row_src;       // optional: one float per streamed row -> stage offset row_off
  int row_off;
  int wave, lane;
  LoadLane ll;

  __device__ TileStream(const UnitPlan& u_, const int* gidx, char* st, int (*rg)[BN],
                        const unsigned short* x0, const unsigned short* x1, const float* rs,
                        int row_off_, int wave_, int lane_)
      : u(u_), global_idx(gidx), stages(st), ring(rg), X0(x0), X1(x1), row_src(rs), row_off(row_off_), wave(wave_),
        lane(lane_), ll(make_load_lane<kQuad>(wave_, lane_)) {}

  // (tile t of a stage that begins with tile t - j)
  __device__ char* stage(int t) { return stages + ((unsigned)(t - u.t_begin) / kTiles % kStages) * kStageBytes; }
  // 4 KB of the stage that stays empty until the first acquire(), one piece per wavefront
  __device__ char* room() { return stages + kStageBytes + wave * 4096; }
  __device__ void issue_idx(int t) {
    const int* list; int base, last;
    if (wave != (t & 3)) return;
    tile_source(u, global_idx, t, list, base, last);
    issue_row_words(list, min(base + lane, last), &ring[t & (kIdxSlots - 1)][0]);
  }
  __device__ void issue_data(int t, int j = 0) {
    const int* r = ring[t & (kIdxSlots - 1)];
    const int x0 = r[ll.row0], x1 = r[ll.row0 + 8];
    char* st = stage(t) + j * kTileStage;
    issue_tile(X0, x0, x1, ll, st, wave);
    issue_tile(X1, x0, x1, ll, st + kTileBytes, wave);
    if (row_src) issue_row_words(row_src, r[lane], st + row_off);
  }
  // Before the loop, in two steps so that the caller's own first loads (which rows it owns) can
  // travel together with the first index loads, and its row loads together with the first tile:
  // begin() issues the indices of the first two tiles; prime() waits for them and issues the
  // data of the first.
  __device__ void begin() {
#pragma unroll
    for (int s = 0; s < 2 * kTiles; ++s)
      if (u.t_begin + s < u.t_end) issue_idx(u.t_begin + s);
  }
  __device__ void prime() {
    wait_vmcnt_le(0);
    barrier_no_fence();  // every wavefront's share of the first indices is in the ring
#pragma unroll
    for (int j = 0; j < kTiles; ++j)
      if (u.t_begin + j < u.t_end) issue_data(u.t_begin + j, j);
  }
  // Top of an iteration: tile t (and t + 1) is complete in LDS for every wavefront, the stage before is
  // free; keep the pipeline full.  Returns the stage holding tile t.
  __device__ const char* acquire(int t) {
    wait_vmcnt_le<0>(0);      // my share of tile t has landed
    barrier_no_fence();       // ... everyone's has, and everyone is done with tile t - 1
#pragma unroll
    for (int j = 0; j < kTiles; ++j)
      if (t + 2 * kTiles + j < u.t_end) issue_idx(t + 2 * kTiles + j);
#pragma unroll
    for (int j = 0; j < kTiles; ++j)
      if (t + kTiles + j < u.t_end) issue_data(t + kTiles + j, j);
    return stage(t);
  }
};

}  // namespace mate
