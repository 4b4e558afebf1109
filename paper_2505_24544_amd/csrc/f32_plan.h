// Which tiles a launch of the float GEMM takes, and how many launches a long grid is.  No HIP in here: the tests compile it for the host.
#pragma once
#include <stdint.h>

namespace beagle {

struct F32Problem { int64_t M, N, chunks; };                            // chunks of 32 k, of both segments
inline int64_t gemm_f32_tiles(const F32Problem& p, int rows, int cols) { return ((p.M + rows - 1) / rows) * ((p.N + cols - 1) / cols); }
// ahead: a wave requests a chunk ahead; alone: one workgroup to a CU
struct F32Plan { int rows, cols; bool ahead, alone; int64_t tiles; };

// What a launch takes on tiles of 16 x 64 or 32 x 64, us: rounds of the 256 CUs at the tiles' mean depth, or the eighth of the deepest tile
// that a wave works through, whichever is longer, and a start.  Fitted to the launches of steps of 16 - 3000 rows at hidden 256 - 5120.
// Some of them, us on 16 x 64 / 32 x 64: 128 rows through Wo at hidden 512 8.6 / 11.9, at 4096 68 / 56; 1040 rows into Q, K and V at
// hidden 512 32 / 33, at 1024 98 / 94, 1000 at 5120 2420 / 1730; the last gradients of 128 rows at 4096 464 / 348, of 2048 3300 / 2320.
inline double gemm_f32_price(const F32Problem* p, int count, int rows, F32Plan* out) {
  int64_t chunks = 0, deepest = 0;
  *out = {rows, 64, false, false, 0};
  for (int i = 0; i < count; ++i) {
    const int64_t t = gemm_f32_tiles(p[i], rows, 64);
    out->tiles += t; chunks += t * p[i].chunks;
    if (t > 0 && p[i].chunks > deepest) deepest = p[i].chunks;
  }
  if (out->tiles == 0) return 0.0;
  const double depth = (double)chunks / (double)out->tiles, rounds = (double)((out->tiles + 255) / 256), turns = (double)((deepest + 7) / 8);
  double start = 2.0, each, turn;
  if (rows == 32) {
    // Deep tiles of 32 rows are the faster ones alone on their CU (two fetch each other's operands out of L1): 2048 rows into Q, K and V at
    // hidden 2048 587 against 765 us, the output gradients of 512 111 / 130; and those of the first two rounds: last gradients of 300 rows
    // at 512 19.2 / 21.5.  Shallow ones in pairs, which hide each other's start: last gradients of 128 rows at 2048 94 against 108, of 24
    // at 4096 187 / 302; at a mean depth of 18 chunks 299 / 288, of 16 441 / 443.
    out->alone = depth >= 16.0 || out->tiles <= 512;
    start = out->alone ? 3.5 : 4.0;
    each = out->alone ? 2.5 + 0.36 * depth : 1.7 + 0.42 * depth;
    turn = out->alone ? 3.3 : 4.4;
  } else {
    // Tiles of 16 rows request a chunk ahead up to two workgroups per CU; beyond, workgroups go in pairs.  Steps, us, ahead / in pairs:
    // 128 rows at 4 x 128 channels 57.8 / 60.5 (59.0 by this rule: its last launch has 896 tiles), 200 at 4 x 128 77.4 / 77.0 (75.5).
    out->ahead = out->tiles <= 512;
    each = 1.1 + 0.235 * depth;
    turn = 2.4;
  }
  return start + (rounds * each > turns * turn ? rounds * each : turns * turn);
}
// 16 x 32 where those are no more than the CUs: a few rows through wide weights are bound by what a CU can fetch, and twice the CUs share
// it.  Projections of one query, us, on 16 x 64 / 16 x 32 (32 x 32 by four waves, as it was before either): hidden 3072 25 / 16 (26), 4096 32 /
// 20 (30), 5120 38 / 25 (38), 8192 72 / 45 (66).  Past a round: 16 rows into Q, K and V at 4096 53 / 58, 20 through Wo at 5120 43 / 48.
inline F32Plan gemm_f32_plan(const F32Problem* p, int count) {
  F32Plan narrow = {16, 32, false, false, 0}, a, b;
  for (int i = 0; i < count; ++i) narrow.tiles += gemm_f32_tiles(p[i], 16, 32);
  if (narrow.tiles <= 256) return narrow;
  return gemm_f32_price(p, count, 32, &b) < gemm_f32_price(p, count, 16, &a) ? b : a;
}

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
