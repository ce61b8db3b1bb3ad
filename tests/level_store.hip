// CPU checks of the level-slice kernel's partials: the store a plan makes holds
// every call the plan can get (by level and by value, fewer offsets, smaller
// images) without dropping a band, and is neither moved nor asked for again.
#include <cstdio>
#include <cstdlib>

#include "glcm_levels.h"

using namespace glcm;

static int fails = 0;
#define CHECK(c)                                              \
  do {                                                        \
    if (!(c) && ++fails < 20) std::printf("FAIL %s (line %d)\n", #c, __LINE__); \
  } while (0)

static constexpr int kLds = 40704, kCus = 256;  // 160 KiB less 1 KiB, in dwords

static void calls_fit(int N, int K, int W, int H) {
  const uint64_t room = level_reserve(N, K, W, H, kLds, kCus);
  for (int k : {1, 2, 3, 5, 7, K - 1, K}) {
    if (k < 1 || k > K) continue;
    for (int w : {1, 17, W / 3, W}) {
      for (int h : {1, H / 7, H - 1, H}) {
        if (w < 1 || h < 1) continue;
        for (int levels = N; levels >= 1; levels -= levels > 330 ? 7 : 1) {
          LevelLayout L = level_layout(levels, k, w, h, kLds, kCus);
          if (levels < N && L.slices != 1) continue;
          const int bands = L.bands;
          CHECK(L.bytes() <= room);
          CHECK(L.fit(room) && L.bands == bands);
        }
      }
    }
  }
}

int main() {
  for (int N : {65, 128, 200, 256, 285, 300, 362, 403, 444, 512, 574, 1024})
    for (int K : {1, 4, 12})
      for (int side : {64, 1000, 4096, 65535}) calls_fit(N, K, side, side == 65535 ? side : side + 13);
  calls_fit(256, 48, 4096, 4096);

  // a layout clamped to little room: fewer bands, still inside
  for (uint64_t room = 1u << 17; room < (64u << 20); room += room / 3) {
    LevelLayout L = level_layout(256, 12, 4096, 4096, kLds, kCus);
    const uint64_t one = L.units * ((uint64_t)L.slice_dwords + 2) * 4u;
    if (L.fit(room)) CHECK(L.bands >= 1 && L.bytes() <= room);
    else CHECK(room < 2 * one);
  }

  // the store: not beyond its limit, not during a capture, no failure when there is no memory
  static uint32_t memory[4];
  int asked = 0;
  bool none = true;
  auto make = [&](size_t) -> void* {
    ++asked;
    return none ? nullptr : memory;
  };
  LevelStore s;
  CHECK(!s.hold(100, 99, true, make) && asked == 0);
  CHECK(!s.hold(100, 1000, false, make) && asked == 0);
  CHECK(!s.hold(100, 1000, true, make) && asked == 1 && s.mem == nullptr && s.bytes == 0);
  none = false;
  CHECK(s.hold(100, 1000, true, make) && asked == 2 && s.mem == memory && s.bytes == 100);
  // whatever comes later, the same memory
  CHECK(s.hold(5000, 10, true, make) && s.hold(5000, 1u << 20, false, make) && asked == 2);
  CHECK(s.mem == memory && s.bytes == 100);

  std::printf(fails ? "%d failures\n" : "ok\n", fails);
  return fails ? 1 : 0;
}
