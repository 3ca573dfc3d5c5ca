// Which tile of a product with the weights a workgroup computes.  (For the host too: a test deals all tiles of a launch.)
#pragma once
#include <hip/hip_runtime.h>

#include "division.h"

namespace mate {

// Workgroup -> tile.  A grid row is eight token tiles times all feature tiles: XCD x % 8 takes one of the token tiles, so
// the token rows that it streams stay in its L2 while the weights cycle, another one in each grid row, so that the
// padding at the end of the sequences is spread over all XCDs.  The tiles of the last token tiles, fewer than eight, are
// dealt one by one: no XCD has more than one tile more than another, where 21 whole token tiles with 12 feature tiles were 36
// tiles on some XCDs' 32 CUs, two rounds where one does (1024 -> 3072 at 5376 tokens 38 -> 32 us, at 10752 74 -> 61, gradients
// of the output projection at 7 x 577 tokens, 768 wide 31.2 -> 25.2, at 9 x 1000 40 -> 33; over 280 products of 1000 tokens and more QKV
// takes 0.91 of what it took before this deal, the tile shapes chosen for it and results through the L2, the output 0.92,
// dX 0.97, d_o 0.94).  Which tiles are padding is not known here: where sequences end in it, the XCD with the most live tiles gets its share
// of the last ones too, and one product in a hundred takes a round more by that (1024 -> 1024 at 6 x 5458 tokens, a tenth padding: one XCD has 64
// live tiles for its 32 CUs and gets another, 71 -> 88; 1024 -> 3072 at 5 x 3378, a third, 91 -> 115; 1536 -> 4608 at 12 x 1189 170 -> 198).  (Tried:
// whole token tiles wherever dealing the last ones one by one saves no round for full sequences.  These products are as before then, others
// up to 13 % slower or faster, 0.0 % in the mean over 600, and both gradients in one launch up to 1.7 times as long.  Halves and
// quarters of a token tile's features to an XCD: 0 to 4 % slower.)
constexpr int kMostGridY = 32768;  // (a grid's second dimension is at most 65536: the third continues it)
struct TileDeal {
  int tokens, features;  // tiles
  int rows;              // grid rows that are dealt as whole token tiles (or feature tiles)
  int by_feature;        // the same with the two exchanged
  __host__ __device__ int grid_x() const { return 8 * (by_feature ? tokens : features); }
  __host__ __device__ int grid_y() const { return rows + ((by_feature ? features : tokens) > 8 * rows ? 1 : 0); }
};
__host__ __device__ inline bool dealt_tile(const TileDeal& d, int x, int y, int& token_tile, int& feature_tile) {
  int major = 8 * y + ((x + 3 * y) & 7), minor = x >> 3;
  const int majors = d.by_feature ? d.features : d.tokens;
  if (y >= d.rows) major = 8 * y + uniform_div(x, d.by_feature ? d.tokens : d.features, minor);
  token_tile = d.by_feature ? minor : major;
  feature_tile = d.by_feature ? major : minor;
  return major < majors;
}
// Its sequence and its place there.  (Nothing bounds the number of sequences but memory.)
__host__ __device__ inline int sequence_of(int token_tile, int tiles_each, int& tile) { return uniform_div_any(token_tile, tiles_each, tile); }

}  // namespace mate
