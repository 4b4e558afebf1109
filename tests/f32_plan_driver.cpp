// Host build of csrc/f32_plan.h.  Input, one per line:
//   a launch of the float GEMM: count, then M N chunks of each problem    -> its plan: rows and columns of a tile, tiles, ahead, alone
//   0 rows n0 n1: a backward's grid, rows runs of n0 blocks, then 2 rows of n1 -> its launches, first block and blocks of each, and
//     whether every launch's first and last block of either kind come out as the block they are
#include <cstdio>
#include "../paper_2505_24544_amd/csrc/f32_plan.h"

static void grid(int64_t rows, int64_t n0, int64_t n1) {
  const int64_t first = rows * n0;
  beagle::for_launches(first + 2 * rows * n1, 512, [&](int64_t at, int64_t n) {
    const beagle::GridPart p = beagle::grid_part(at, n, rows, n0, n1);
    bool ok = true;
    auto check = [&](int64_t b) {                       // block b of this launch, as the kernel takes it apart
      if (b < 0 || b >= n) return;
      const int64_t want = at + b;
      const uint32_t x = b < p.n_first ? p.blk0 + (uint32_t)b : p.blk1 + ((uint32_t)b - p.n_first);
      if (b < p.n_first) ok = ok && want < first && p.row0 + x / n0 == want / n0 && x % n0 == want % n0;
      else ok = ok && want >= first && p.row1 + x / n1 == (want - first) / n1 && x % n1 == (want - first) % n1;
    };
    check(0); check((int64_t)p.n_first - 1); check(p.n_first); check(n / 2); check(n - 1);
    printf("%lld %lld %d ", (long long)at, (long long)n, ok ? 1 : 0);
  });
  printf("\n");
}

int main() {
  int n;
  while (scanf("%d", &n) == 1) {
    beagle::F32Problem p[6];
    long long m, c, k;
    if (n < 0 || n > 6) return 1;
    for (int i = 0; i < (n ? n : 1); ++i) {
      if (scanf("%lld %lld %lld", &m, &c, &k) != 3) return 1;
      p[i] = {m, c, k};
    }
    if (n == 0) { grid(m, c, k); continue; }
    const beagle::F32Plan q = beagle::gemm_f32_plan(p, n);
    printf("%d %d %lld %d %d\n", q.rows, q.cols, (long long)q.tiles, q.ahead ? 1 : 0, q.alone ? 1 : 0);
  }
}
