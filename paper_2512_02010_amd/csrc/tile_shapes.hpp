// Host side of the tiled quantizers: how a tensor is dealt out to workgroups.  Plain C++ without HIP, so that the
// rules can be checked where there is no GPU.
#pragma once

#include <cstdint>

namespace nvfp4_46 {

constexpr int TR = 64;    // rows of a tile of k_tile    (multiple of 16)
constexpr int TC = 128;   // columns                     (multiple of 16)

// Workgroups are handed to the 8 XCDs round-robin by their index, and each XCD has its own
// L2.  A tile writes only part of every output cache line it touches: 64 of the 128 bytes of
// a row's codes, 32 bytes of a column's, 8 and 4 bytes of the scale lines.  The tiles that
// complete those lines -- horizontal neighbours for the rowwise arrays, vertical neighbours
// for the columnwise ones -- should therefore meet in one L2 while the lines are still
// there.  So the tiles are grouped into super-tiles of sx x sy tiles (8 x 16 when the tensor
// is that large: 1024 x 1024 elements), super-tile S goes to XCD S % 8, and the consecutive
// workgroups of one XCD walk through one super-tile row by row.  (One XCD per tile column,
// top to bottom, merged only the columnwise lines: 66.6 -> 58.6 us for both orientations of
// 8192 x 8192.)
struct TileMap {
  uint32_t sx, sy;      // super-tile width and height in tiles
  uint32_t last;        // the grid's last workgroup where tiles go last to first (kLastLevelBytes), or 0
};

// Super-tiles of 8 x 16 tiles (no larger than the tensor) where that gives every die about its share, or no die more
// tiles than its 32 compute units, else the largest smaller ones that do: a tensor of few tiles would otherwise be one
// super-tile, all on one die (us in a replayed graph, 8 x 16 / this: columnwise Hadamard + SR 736 x 1024 11.0 / 8.3, 1008 x
// 4096 13.2 / 9.6, 1344 x 2208 13.1 / 9.4; both orientations 336 x 1184 6.7 / 5.9, 736 x 1024 8.9 / 5.9, 1008 x 4096 11.2 / 7.9,
// 5248 x 6192 38.5 / 34.4; one tile per compute unit of one die or spread over all: 848 x 208 5.8 / 6.0).
// (Host work of every call that comes here, so counted without a division.)
inline TileMap tile_map(int64_t rows, int64_t cols) {
  const int64_t nt_r = (rows + TR - 1) / TR, nt_c = (cols + TC - 1) / TC;
  TileMap best{1u, 1u, 0u};
  int64_t best_most = INT64_MAX;
  for (int log = 7; log >= 0; --log) {                 // 8 x 16, 8 x 8, 4 x 8, 4 x 4, ... 1 x 2, 1 x 1
    const int log_wide = log >= 6 ? 3 : log / 2, log_high = log - log_wide;
    const int64_t wide = (int64_t)1 << log_wide, high = (int64_t)1 << log_high;
    const int64_t across = (nt_c + wide - 1) >> log_wide, down = (nt_r + high - 1) >> log_high;
    const TileMap map{(uint32_t)(nt_c < wide ? nt_c : wide), (uint32_t)(nt_r < high ? nt_r : high), 0u};
    if (log == 7 && across * down > 64) return map;    // more than eight turns of the largest
    // The tiles of each die: it has the super-tiles of row i and column j with (i across + j) % 8, so what counts is the
    // tiles along each axis in super-tiles of the same remainder.
    int64_t tall[8], broad[8], tiles[8] = {}, most = 0;
    for (int k = 0; k < 8; ++k) {
      tall[k] = ((down + 7 - k) >> 3 << log_high) - (((down - 1) & 7) == k ? (down << log_high) - nt_r : 0);
      broad[k] = ((across + 7 - k) >> 3 << log_wide) - (((across - 1) & 7) == k ? (across << log_wide) - nt_c : 0);
    }
    const int rows_used = down < 8 ? (int)down : 8, cols_used = across < 8 ? (int)across : 8;
    for (int i = 0; i < rows_used; ++i)
      for (int j = 0; j < cols_used; ++j) tiles[(i * (int)(across & 7) + j) & 7] += tall[i] * broad[j];
    for (int64_t t : tiles) most = t > most ? t : most;
    if (most < best_most) {
      best = map;
      best_most = most;
    }
    if (most <= 32 || most * 32 <= nt_r * nt_c * 5) break;      // within a quarter of an eighth
  }
  return best;
}

// Whole turns over the eight XCDs, each turn one super-tile per XCD.
inline int tile_grid(int64_t rows, int64_t cols, TileMap m) {
  const int64_t nt_r = (rows + TR - 1) / TR, nt_c = (cols + TC - 1) / TC;
  const int64_t supers = ((nt_c + m.sx - 1) / m.sx) * ((nt_r + m.sy - 1) / m.sy);
  return (int)(8 * ((supers + 7) / 8) * m.sx * m.sy);
}

// Both packings of 16x16 tiles (k_block2d) are made in units of 4, 8 or 16 tile rows x 4 tile columns.  A unit's steps
// of 4 x 4 tiles follow each other in its workgroup, a high unit stores longer runs.  High units pay where they fill the
// chip: what counts is how many of them there are for the four workgroups of a compute unit that run at once, a turn.
// Tensor scale and codes, us in a replayed graph, 16 / 8 / 4 tile rows:
//                       fp32                    BF16
//   512 x 512         12.5 /  9.6 /  8.0     12.1 /  9.3 /  7.8     64 units of 4
//   2048 x 2048       15.0 / 12.3 / 11.6     13.1 / 10.6 /  9.8     1024 (a turn)
//   4240 x 1024       16.1 / 14.5 / 15.4     13.5 / 11.4 / 11.6     1072; 544 units of 8
//   4096 x 2048       21.1 / 18.9 / 20.0     16.1 / 14.0 / 15.2     1024 of 8 (a turn)
//   3536 x 2496       21.9 / 22.5 / 22.3     18.2 / 18.8 / 18.4     1092; 546 units of 16
//   5216 x 2384       26.2 / 27.4 / 28.2     21.3 / 22.3 / 23.2     798 of 16
//   4096 x 4096       32.9 / 32.3 / 31.1     22.6 / 23.6 / 25.0     1024 of 16 (a turn)
//   4096 x 4112       34.6 / 33.5 / 32.9     28.3 / 25.7 / 25.3     1040: a second turn for the rest
//   5120 x 4096       39.6 / 37.8 / 36.8     29.5 / 28.6 / 29.1     1280
//   4096 x 6144       43.9 / 43.8 / 43.2     32.0 / 32.8 / 32.7     1536
//   5904 x 5344       52.4 / 53.9 / 54.5     39.3 / 40.4 / 41.2     2016
//   8192 x 8192      108.1 / 108.8 / 112.5   66.6 / 67.6 / 69.1     4096
// In fp32 the last quarter of a turn is level on average and with units of 8 sometimes far ahead (8192 x 2048 34.3 / 31.3,
// 6144 x 2064 28.5 / 26.1, but 2048 x 7792 30.2 / 31.6).
constexpr int tile_unit_rows(int64_t rows, int64_t cols, bool xf32, int64_t compute_units) {
  const int64_t across = (cols / 16 + 3) / 4, turn = 4 * compute_units;
  const int64_t of_4 = (rows / 16 + 3) / 4 * across, of_8 = (rows / 16 + 7) / 8 * across, of_16 = (rows / 16 + 15) / 16 * across;
  if (of_4 <= turn) return 4;
  if (of_8 <= turn) return 8;
  return of_16 * 4 > (xf32 ? 3 : 4) * turn && of_16 * 8 <= 11 * turn ? 8 : 16;
}

}  // namespace nvfp4_46
