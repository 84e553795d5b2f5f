// rules.hpp -- which of two kernels with the same bits a 2D step takes, from
// the sizes of the grid and the compute units of the chip (plain C++).
#pragma once

namespace hofks {

constexpr int STRIP_W = 60;    // cells that an Euler strip advances in x
constexpr int ET = 16;         // edge of an Euler tile

// blocks of a sub-step by strips of `rows` rows, four to a block
inline long strip_blocks(int nx, int ny, int rows) {
  return (long)((nx + STRIP_W - 1) / STRIP_W) * ((ny + 4 * rows - 1) / (4 * rows));
}

// Whether the 2D Euler sub-steps run by 16 x 16 tiles instead of strips: where
// most lanes of the strips are idle (up to 16 cells in a row, or up to two
// tiles per strip: 17 .. 32 and 61 .. 64) and there are more strips than
// compute units, so that the idle lanes cost time.  With more strips than one
// round of the tallest, the second kind is as fast by strips.  Tiles against
// strips, us per step (16^2 nodes), FP64 and FP32: 16 x 4096 380 against 410, 190
// against 226; 4 x 4096 360, 386, 167, 204; 32 x 4096 419, 431, 220, 243; 64 x
// 1024 153, 171, 121, 125; on the other side 16 x 1024 140, 122, 112, 98; 64 x 512
// 127, 113, 113, 103; 32 x 8192 805, 829, 461, 439; 40 x 1638 211, 206, 149, 133.
inline bool euler_tiles(int nx, int ny, int ncu) {
  const int nsx = (nx + STRIP_W - 1) / STRIP_W, ntx = (nx + ET - 1) / ET;
  return strip_blocks(nx, ny, 1) > ncu &&
         (ntx <= nsx || (ntx <= 2 * nsx && strip_blocks(nx, ny, 5) <= ncu));
}

}  // namespace hofks
