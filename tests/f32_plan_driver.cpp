// Host build of csrc/f32_plan.h.  Input, a launch per line: count, then M N chunks of each problem.  Output: rows of a tile, tiles,
// whether a chunk is requested ahead.
#include <cstdio>
#include "../paper_2505_24544_amd/csrc/f32_plan.h"

int main() {
  int n;
  while (scanf("%d", &n) == 1) {
    beagle::F32Problem p[6];
    long long m, c, k;
    if (n < 1 || n > 6) return 1;
    for (int i = 0; i < n; ++i) {
      if (scanf("%lld %lld %lld", &m, &c, &k) != 3) return 1;
      p[i] = {m, c, k};
    }
    const int rows = beagle::gemm_f32_rows(p, n);
    long long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += beagle::gemm_f32_tiles(p[i], rows);
    printf("%d %lld %d\n", rows, tiles, rows == 16 && beagle::gemm_f32_ahead(tiles) ? 1 : 0);
  }
}
