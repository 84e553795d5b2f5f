// rules.hpp -- which kernel or launch shape an untuned 2D step takes, from the
// sizes of the grid and the compute units of the chip (plain C++).
#pragma once

namespace hofks {

constexpr int STRIP_W = 60;    // cells that an Euler strip advances in x
constexpr int ET = 16;         // edge of an Euler tile
constexpr int W2_CELLS = 128;  // cells per block row segment of the two-cell kinetic kernel

// blocks of a sub-step by strips of `rows` rows, four to a block
inline long strip_blocks(int nx, int ny, int rows) {
  return (long)((nx + STRIP_W - 1) / STRIP_W) * ((ny + 4 * rows - 1) / (4 * rows));
}

// Rows per strip.  Short grids want many strips: with one row a sub-step alone
// takes 5.4 us on 70 x 37 cells and 6.4 on 256^2 (two rows: 6.5 and 6.3, and
// beside the kinetic kernel 17.5 -> 21.1 on 256^2, where the longer chain of a
// wavefront shows).  Alone, larger grids are bound by the FP64 issue rate,
// where more rows share more of the y fluxes and slopes, and by the last round
// of blocks (512^2 15.5 us with one row, 12.8 with three, 14.4 with four in 288
// blocks, 12.3 with five in 234).  What counts is the step, us:
// - beside FP64 pieces one row pays up to 2.5 blocks per compute unit, and up to
//   3.25 where more than a quarter of the lanes are idle, since blocks that end
//   soon keep fewer kinetic blocks out (256 x 512 x 32^2 543, 608 with three,
//   638 with five; 320 x 343 x 24^2 330, 365; 72 x 1527 x 32^2 615, 686; but 400^2
//   x 32^2, 2.7, 824, 770), except with 32 nodes and more in more than five
//   kinetic blocks per unit (398 x 332 x 32^2 699, 669; 396 x 336 x 32^2 701, 689;
//   with 24^2 and fewer one row stays ahead); then the fewest rows that give
//   each unit at most one block (364 x 467 x 32^2 776 with four, 791 with five),
//   and five;
// - beside FP32 pieces three rows where those do (256 x 512 x 16^2 166, 180 with
//   one), else two up to two blocks per unit (128 x 1024 x 32^2 428, 462 with
//   five; 364 x 467 x 32^2 520, 598), and five.
inline int strip_rows(int nx, int ny, int nv, bool fp32, int ncu) {
  const long b1 = strip_blocks(nx, ny, 1);
  const bool idle = 4L * nx < 3L * STRIP_W * ((nx + STRIP_W - 1) / STRIP_W);
  const bool kinetic = nv >= 32 && (long)((nx + W2_CELLS - 1) / W2_CELLS) * ny > 5L * ncu;
  if (4 * b1 <= (fp32 ? 8L : idle ? 13L : kinetic ? 8L : 10L) * ncu) return 1;
  if (strip_blocks(nx, ny, 3) <= ncu) return 3;
  if (fp32) return strip_blocks(nx, ny, 2) <= 2L * ncu ? 2 : 5;
  return strip_blocks(nx, ny, 4) <= ncu ? 4 : 5;
}

// Whether the 2D Euler sub-steps run by 16 x 16 tiles instead of strips: where
// most lanes of the strips are idle (up to 16 cells in a row, or up to two
// tiles per strip: 17 .. 32 and 61 .. 64) and there are more strips than
// compute units, so that the idle lanes cost time.  In more than two rounds of
// the tallest strips the second kind is as fast by them.  Tiles against strips,
// us per step with 16^2 nodes, FP64 and FP32: 16 x 4096 380 against 410, 166, 224;
// 4 x 4096 360, 386, 151, 208; 24 x 5461 544, 560, 250, 298; 32 x 8192 805, 829,
// 353, 380; 64 x 1024 153, 171, 122, 126; on the other side 16 x 1024 140, 122,
// 113, 98; 64 x 512 127, 113, 113, 102; 20 x 13107 1266, 1266, 563, 548; 40 x 1638
// 211, 206, 149, 134.
inline bool euler_tiles(int nx, int ny, int ncu) {
  const int nsx = (nx + STRIP_W - 1) / STRIP_W, ntx = (nx + ET - 1) / ET;
  return strip_blocks(nx, ny, 1) > ncu &&
         (ntx <= nsx || (ntx <= 2 * nsx && strip_blocks(nx, ny, 5) <= 2L * ncu));
}

// Wavefronts per block of a 2D FP32 kinetic launch of nb blocks, by blocks per
// compute unit.  Between two and five the launch is little more than a round
// and two wavefronts leave the Euler blocks room beside them (256^2 x 32^2, 1024
// blocks: 0.183 ms per step with two, 0.212 with four, 0.247 with eight; 300 x
// 256 x 32^2 0.263, 0.267, 0.299).  In many rounds a block of eight ends sooner
// and frees room for a whole Euler block at once (400^2 x 32^2, 2800 blocks:
// 0.436, 0.453 with four, 0.457 with two; 512^2 x 32^2 0.711, 0.762, 0.774), if
// its wavefronts have work enough for that: not on rows short of a segment (16
// x 5120, eight against four: 16^2 0.233, 0.189, 32^2 0.583, 0.492, 64^2 1.925,
// 1.409), not with 8^2 nodes (200 x 1280 0.164, 0.147), and with 16^2 and 24^2
// only up to about 1.25 blocks per unit and node (512 x 960 x 16^2, 30 per
// unit, 0.492, 0.465; 128 x 5120 x 24^2, 40, 1.138, 1.054; 512 x 2048 x 32^2,
// 64, 2.72, 2.90).  Else four are as good or better (330 x 300 x 32^2, 1800
// blocks: 0.385, 0.404 with eight, 0.439 with two; 200 x 120 x 32^2, 480
// blocks: 0.139, 0.152, 0.142).
inline int fp32_wavefronts(int nx, int nv, long nb, int ncu) {
  if (nb > 2L * ncu && nb <= 5L * ncu) return 2;
  const bool busy = nx >= 64 && nv >= 16 && (nv >= 32 || 4 * nb <= 5L * nv * ncu);
  return nb > 10L * ncu && busy ? 8 : 4;
}

// Whether an off-lattice 2D FP64 step runs in the two-cell kinetic kernel (128
// cells of a row to a block) instead of the general one (64), from the blocks
// per compute unit of either, rounded up.  A lane's second cell doubles its
// chain, which shows while a unit holds one block, and is wasted on ragged
// rows; three two-cell blocks run on a unit at a time, so three are one round
// where five general ones are more, and a fourth starts another.  General
// against two-cell kernel, us per step with (general, two-cell) blocks per unit:
// 256^2 x 32^2 (4, 2) 273, 242; 370 x 198 x 32^2 (5, 3) 382, 355; 347 x 222 x 32^2
// (6, 3) 455, 374; 332 x 371 x 32^2 (9, 5) 633, 583; 360 x 400 x 32^2 (10, 5) 614,
// 563; on the other side 64^2 x 64^2 (1, 1) 313, 558; 450 x 64 x 32^2 (2, 1) 148,
// 187; 150^2 x 16^2 (2, 2) 57, 78; 300 x 128 x 32^2 (3, 2) 196, 217; 295 x 197 x 32^2
// (4, 3) 313, 354; 256 x 400 x 32^2 (7, 4) 430, 467; 296 x 393 x 24^2 (8, 5) 291,
// 322; and 131 x 375 x 16^2 (5, 3) 106, 127, where a quarter of the lanes is
// idle.
inline bool offlattice_pairs(int nx, int ny, int ncu) {
  const long b2 = (long)((nx + W2_CELLS - 1) / W2_CELLS) * ny, b1 = (long)((nx + 63) / 64) * ny;
  const long two = (b2 + ncu - 1) / ncu, one = (b1 + ncu - 1) / ncu;
  if (two == 1 || 5 * b1 < 8 * b2) return false;
  return two == 3 ? one >= 5 : 5 * one >= 9 * two;
}

}  // namespace hofks
