// CPU replay of the matrix-core kernel's geometry: windows and segments own
// every first pixel exactly once, a pair of an owned pixel lies in its window
// or outside the image, loads stay inside the image, and segments walk a
// multiple of the kernel's stride.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "glcm_onehot.h"

using namespace glcm;

static int fails = 0;
#define CHECK(c)                                                                \
  do {                                                                          \
    if (!(c) && ++fails < 20) std::printf("FAIL %s (line %d) W=%d H=%d y=[%d,%d) R=%d h=%d\n", #c, __LINE__, W, H, y0, y1, R, h); \
  } while (0)

static void replay(int W, int H, int y0, int y1, int R, int h) {
  const int U = onehot_stride(R), rows = y1 - y0, nwin = onehot_windows(W, R);
  CHECK((h + R) % U == 0 && h >= 1);
  CHECK(onehot_block_rows(R) % U == 0 && U % (R + 1) == 0);
  CHECK(h <= rows || y1 == H);
  std::vector<int> seen((size_t)W * (size_t)(y1 - y0), 0);
  const int segs = (rows + h - 1) / h;
  for (int s = 0; s < segs; ++s) {
    const OnehotSegment g = onehot_segment(s, h, y0, y1);
    CHECK(g.ya >= y0 && g.own >= g.ya && g.own < y1);
    for (int c = 0; c < nwin; ++c) {
      const OnehotWindow w = onehot_window(c, nwin, W, R);
      const int n = W < kOnehotWindow ? W : kOnehotWindow;
      CHECK(w.x >= 0 && w.x + n <= W && w.lo >= 0 && w.lo < w.hi && w.hi <= n);
      // pairs to the right and left of an owned pixel: in the window or outside the image
      CHECK(w.lo >= R || w.x == 0);
      CHECK(w.hi + R <= n || w.x + n == W);
      for (int y = g.ya; y < g.ya + h; ++y) {
        if (y < g.own || y >= H) continue;  // no level there
        CHECK(y < y1);
        if (y >= y1) continue;
        for (int p = w.lo; p < w.hi; ++p) ++seen[(size_t)(y - y0) * W + w.x + p];
      }
    }
  }
  for (int v : seen) CHECK(v == 1);
}

int main() {
  for (int R : {1, 2, 4}) {
    const int U = onehot_stride(R);
    for (int W = 1; W <= 200; ++W)
      for (int rows : {1, 2, 3, 5, 14, 15, 16, 31, 40})
        for (int below : {0, 3})  // rows of the image below the band
          for (int n = 1; n <= 9; ++n) {
            const int h = U * n - R;
            if (h > rows && (below || h > U * ((rows + R + U - 1) / U) - R)) continue;
            replay(W, 2 + rows + below, 2, 2 + rows, R, h);
          }
    for (int W : {33, 64, 65, 120, 257, 300, 512, 1031})
      for (int rows : {1, 2, 7, 32, 33, 100, 511, 512})
        for (int waves : {1, 4}) {
          int best = 1;
          uint32_t cost = ~0u;
          for (int n = 1; n <= kOnehotCandidates; ++n) {
            const uint32_t c = onehot_cost(n, onehot_windows(W, R), rows, R, waves);
            if (c < cost) cost = c, best = n;
          }
          const int h = onehot_candidate(best, R);
          replay(W, rows, 0, rows, R, h);
          if (rows >= 8) replay(W, rows + 9, 4, 4 + rows, R, h);
        }
  }
  std::printf(fails ? "%d failures\n" : "ok\n", fails);
  return fails ? 1 : 0;
}
