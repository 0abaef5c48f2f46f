// Host side of the tiled quantizers: how a tensor is dealt out to workgroups.  Plain C++ without HIP, so that the
// rules can be checked where there is no GPU.
#pragma once

#include <cstdint>

namespace nvfp4_46 {

// Both packings of 16x16 tiles (k_block2d) are made in units of 4, 8 or 16 tile rows x 4 tile columns: the logarithm of a
// quarter of the rows.  A unit's steps of 4 x 4 tiles follow each other in its workgroup, a high unit stores longer runs.
// High units pay where they fill the chip: what counts is how many of them there are for the four workgroups of a compute
// unit that run at once, a turn.  Tensor scale and codes, us in a replayed graph, 16 / 8 / 4 tile rows:
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
constexpr uint32_t tile_unit_log(int64_t rows, int64_t cols, bool xf32, int64_t compute_units) {
  const int64_t across = (cols / 16 + 3) / 4, turn = 4 * compute_units;
  const int64_t of_4 = (rows / 16 + 3) / 4 * across, of_8 = (rows / 16 + 7) / 8 * across, of_16 = (rows / 16 + 15) / 16 * across;
  if (of_4 <= turn) return 0;
  if (of_8 <= turn) return 1;
  return of_16 * 4 > (xf32 ? 3 : 4) * turn && of_16 * 8 <= 11 * turn ? 1 : 2;
}

}  // namespace nvfp4_46
