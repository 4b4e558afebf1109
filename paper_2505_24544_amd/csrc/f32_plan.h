// Which tiles a launch of the float GEMM takes, and how many launches a long grid is.  No HIP in here: the tests compile it for the host.
#pragma once
#include <stdint.h>

namespace beagle {

constexpr int GEMM_F32_COLS = 64;         // columns of a tile; rows are 16 or 32
struct F32Problem { int64_t M, N, chunks; };                            // chunks of 32 k, of both segments
inline int64_t gemm_f32_tiles(const F32Problem& p, int rows) {
  return ((p.M + rows - 1) / rows) * ((p.N + GEMM_F32_COLS - 1) / GEMM_F32_COLS);
}

// What a launch takes, us: rounds of the 256 CUs at the tiles' mean depth, or the eighth of the deepest tile that a wave works through,
// whichever is longer, and a start.  Fitted to the launches of steps of 16 - 3000 rows at hidden 256 - 5120.  Some of them, us on tiles
// of 16 rows / of 32: 128 rows through Wo at hidden 512 8.7 / 11.9, at 2048 20 / 30, at 4096 68 / 56; 1040 rows into Q, K and V at hidden
// 512 31.8 / 33.4, at 1024 98 / 94, 1000 at 5120 2531 / 1666; the last gradients at 4096 of 24 rows, one chunk deep, 254 / 302, of 128 486 /
// 433, of 2048 3250 / 2480.
inline double gemm_f32_price(const F32Problem* p, int count, int rows) {
  int64_t tiles = 0, chunks = 0, deepest = 0;
  for (int i = 0; i < count; ++i) {
    const int64_t t = gemm_f32_tiles(p[i], rows);
    tiles += t; chunks += t * p[i].chunks;
    if (t > 0 && p[i].chunks > deepest) deepest = p[i].chunks;
  }
  if (tiles == 0) return 0.0;
  const bool two = rows == 32;
  const double depth = (double)chunks / (double)tiles, rounds = (double)((tiles + 255) / 256), turns = (double)((deepest + 7) / 8);
  const double work = rounds * (two ? 2.5 + 0.36 * depth : 1.1 + 0.235 * depth), chain = turns * (two ? 3.3 : 2.4);
  return (two ? 4.0 : 2.0) + (work > chain ? work : chain);
}
inline int gemm_f32_rows(const F32Problem* p, int count) {
  return gemm_f32_price(p, count, 32) < gemm_f32_price(p, count, 16) ? 32 : 16;
}
// Tiles of 16 rows request a chunk ahead up to two workgroups per CU; beyond, workgroups go in pairs.  Steps, us, ahead / in pairs: 128
// rows at 4 x 128 channels 57.8 / 60.5 (59.0 by this rule: its last launch has 896 tiles), 200 at 4 x 128 77.4 / 77.0 (75.5).
inline bool gemm_f32_ahead(int64_t tiles) { return tiles <= 512; }

// A launch holds fewer than 2^32 threads in a dimension; what the entry points accept can be more (a million rows of 3 x 4096 columns
// are 12 million tiles of 512 threads): launch(first block, blocks) for each part.
template <class F>
inline void for_launches(int64_t blocks, int threads, F&& launch) {
  const int64_t most = (int64_t)UINT32_MAX / threads;
  for (int64_t at = 0; at < blocks; at += most) launch(at, blocks - at < most ? blocks - at : most);
}

// Where part [at, at + blocks) of a grid stands that is `rows` runs of n0 blocks, then runs of n1: how many of its blocks are of the first
// kind, and the run and the place in it at which each kind goes on.
struct GridPart { uint32_t n_first, row0, blk0, row1, blk1; };
inline GridPart grid_part(int64_t at, int64_t blocks, int64_t rows, int64_t n0, int64_t n1) {
  const int64_t first = rows * n0, left = at < first ? first - at : 0, past = at > first ? at - first : 0;
  return {(uint32_t)(left < blocks ? left : blocks), (uint32_t)(at / n0), (uint32_t)(at % n0), (uint32_t)(past / n1), (uint32_t)(past % n1)};
}

}  // namespace beagle
