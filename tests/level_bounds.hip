// CPU replay of the level-slice kernel's geometry: for every width, height,
// offset and band count tried, the chunks of the bands cover each valid pair
// exactly once, every 16-pixel load stays inside its row, and the mixed-radix
// walk of a lane equals the division it stands for.
#include <cstdio>
#include <vector>

#include "glcm_levels.h"

using namespace glcm;

static int fails = 0;
#define CHECK(c)                                              \
  do {                                                        \
    if (!(c) && ++fails < 20) std::printf("FAIL %s (line %d)\n", #c, __LINE__); \
  } while (0)

static void replay(int W, int H, int yb, int ye, int dx, int dy, int bands) {
  const LevelRect r = level_rect(W, H, yb, ye, dx, dy);
  const int w = r.x1 - r.x0, h = r.y1 - r.y0;
  std::vector<int> seen((size_t)W * H, 0);
  const uint32_t cpr = (uint32_t)(w + kLevelChunk - 1) / kLevelChunk;
  const uint64_t chunks = (uint64_t)cpr * (uint64_t)h;
  for (int b = 0; b < bands; ++b) {
    const uint64_t c0 = chunks * (uint64_t)b / (uint64_t)bands, c1 = chunks * (uint64_t)(b + 1) / (uint64_t)bands;
    for (uint32_t lane = 0; lane < (uint32_t)kLevelThreads && c0 + lane < c1; ++lane) {
      uint64_t at = c0 + lane;
      int y = r.y0 + (int)(at / cpr);
      uint32_t c = (uint32_t)(at % cpr);
      for (; at < c1; at += kLevelThreads) {
        CHECK(y == r.y0 + (int)(at / cpr) && c == (uint32_t)(at % cpr));
        const LevelChunk ch = level_chunk(r, (int)c);
        const int n = w < kLevelChunk ? ch.n : kLevelChunk;  // pixels loaded
        CHECK(ch.x >= 0 && ch.x + n <= W && ch.x + dx >= 0 && ch.x + dx + n <= W);
        CHECK(y >= yb && y < ye && y + dy >= 0 && y + dy < H);
        for (int t = ch.skip; t < ch.n; ++t) ++seen[(size_t)y * W + ch.x + t];
        y += (int)(kLevelThreads / cpr);
        c += kLevelThreads % cpr;
        if (c >= cpr) {
          c -= cpr;
          ++y;
        }
      }
    }
  }
  for (int y = 0; y < H; ++y)
    for (int x = 0; x < W; ++x) {
      const bool valid = y >= yb && y < ye && x + dx >= 0 && x + dx < W && y + dy >= 0 && y + dy < H;
      CHECK(seen[(size_t)y * W + x] == (valid ? 1 : 0));
    }
}

int main() {
  for (int W = 1; W <= 70; ++W)
    for (int dx = -40; dx <= 40; dx += (dx > -5 && dx < 5) ? 1 : 5)
      for (int dy : {-7, -1, 0, 2, 30})
        for (int bands : {1, 3}) replay(W, 9, 0, 9, dx, dy, bands);
  for (int W : {1000, 1023, 1024, 1040, 4099})
    for (int dx : {-17, -1, 0, 4}) {
      replay(W, 40, 0, 40, dx, 1, 2);
      replay(W, 40, 3, 31, dx, -4, 5);
    }
  replay(17, 3000, 0, 3000, 1, 1, 7);
  std::printf(fails ? "%d failures\n" : "ok\n", fails);
  return fails ? 1 : 0;
}
