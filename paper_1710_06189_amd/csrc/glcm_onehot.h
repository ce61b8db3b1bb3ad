// Counting N <= 16 levels on the matrix cores: geometry shared with the host.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "glcm_internal.h"

namespace glcm {

constexpr int kOnehotMaxN = 16;
// Pixels of a row a 16-lane group takes at once (the 32 K slots of one lane),
// and rows a wavefront converts at once, a lane each for four groups.
constexpr int kOnehotWindow = 32;
constexpr int onehot_block_rows(int reach) { return reach == 1 ? 16 : 15; }
// Rows counted between two tests of a segment's end (a multiple of the ring's
// reach + 1 rows, dividing a block); a segment walks h + reach rows, a
// multiple of it.
constexpr int onehot_stride(int reach) { return reach == 1 ? 4 : reach + 1; }

// Offsets counted at a reach of 1, 2 or 4: the four directions of Eq. (2) at
// d = 1; 1 and 2; 1, 2 and 4.  Slot 4 i + q is direction q (0, 45, 90, 135
// degrees) at distance 2^i.
constexpr int onehot_slots(int reach) { return reach == 1 ? 4 : (reach == 2 ? 8 : 12); }

// Slot of a canonical offset (dy > 0, or dy = 0 and dx > 0), -1 for others.
__host__ __device__ inline int onehot_slot(int dx, int dy) {
  const int ax = dx < 0 ? -dx : dx, d = ax > dy ? ax : dy;
  if (d != 1 && d != 2 && d != 4) return -1;
  const int base = d == 1 ? 0 : (d == 2 ? 4 : 8);
  if (dy == 0) return base;
  if (dy != d) return -1;
  if (dx == -d) return base + 1;
  if (dx == 0) return base + 2;
  return dx == d ? base + 3 : -1;
}

// Windows of a row of width W at a reach of R: window c covers the pixels
// [x, x + 32) (clipped to W) and owns, as first pixels, its pixels [lo, hi);
// every pixel is owned once and every pair of an owned pixel within reach lies
// in the window or outside the row.
struct OnehotWindow {
  int x, lo, hi;
};
__host__ __device__ inline int onehot_windows(int W, int R) {
  const int step = kOnehotWindow - 2 * R;
  return W <= kOnehotWindow ? 1 : 1 + (W - kOnehotWindow + step - 1) / step;
}
__host__ __device__ inline OnehotWindow onehot_window(int c, int nwin, int W, int R) {
  const int step = kOnehotWindow - 2 * R;
  const int x = W <= kOnehotWindow ? 0 : (step * c < W - kOnehotWindow ? step * c : W - kOnehotWindow);
  const int lo = c == 0 ? 0 : step * c + R - x;
  const int hi = c == nwin - 1 ? (W < kOnehotWindow ? W : kOnehotWindow) : step * (c + 1) + R - x;
  return {x, lo, hi};
}

// Row segments: the first-pixel rows [y0, y1) are cut into segs segments of h
// rows; the last starts early enough to end at y1 and leaves the rows before
// its own start (y0 + s h) uncounted.  (Fewer rows than h only where y1 = H:
// the rows below the image count nothing.)
struct OnehotSegment {
  int ya, own;  // first row walked, first row counted
};
__host__ __device__ inline OnehotSegment onehot_segment(int s, int h, int y0, int y1) {
  const int own = y0 + s * h;
  const int up = y1 - h > y0 ? y1 - h : y0;
  return {own + h > y1 ? up : own, own};
}

// Rows per segment of an image that `waves` wavefronts count by themselves:
// candidate n (1, 2, ...) walks U n rows a segment.  Its cost counts, for the
// wavefront with the most units, the vector instructions of the walked rows,
// of the blocks converted for them and of starting a unit; ~0 for a candidate
// longer than the image.
constexpr int kOnehotCandidates = 64;
__host__ __device__ inline int onehot_candidate(int n, int R) { return onehot_stride(R) * n - R; }
__host__ __device__ inline uint32_t onehot_cost(int n, int windows, int rows, int R, int waves) {
  const int h = onehot_candidate(n, R);
  if (n > 1 && h > rows) return ~0u;
  const uint32_t segs = (uint32_t)(rows + h - 1) / (uint32_t)h;
  const uint32_t units = ((uint32_t)windows * segs + 3u) / 4u, rounds = (units + (uint32_t)waves - 1u) / (uint32_t)waves;
  const uint32_t walked = (uint32_t)(h + R), blocks = (walked + (uint32_t)onehot_block_rows(R) - 1u) / (uint32_t)onehot_block_rows(R);
  return rounds * (walked * 20u + blocks * 100u + 100u);
}

struct OnehotArgs {
  const void* img;            // any alignment
  int64_t stride;
  int W, H;
  int y_begin, y_end;
  Quant q;
  int qfast;
  uint32_t qfast_shift, qfast_mask;
  int K;
  int8_t slot[kMaxK];         // slot of offset k's canonical form
  unsigned long long tmask;   // bit k: offset k is the opposite of its slot (stored transposed)
  int windows, h;             // windows per row, rows per segment
  int tasks;                  // windows * segments
  uint32_t words_total;       // K N N
  uint32_t* xbuf;             // per-XCD slices, or null: one workgroup stores to out
  uint32_t* out;
};
// Threads per workgroup and workgroups a CU holds (registers: 128 a lane, 168
// at a reach of 4).
constexpr int onehot_threads(int reach) { return reach == 4 ? 256 : 512; }
constexpr int onehot_per_cu(int reach) { return reach == 4 ? 3 : 2; }

// `groups` workgroups; dist: bit i set = offsets of distance 2^i (the reach is
// the largest).
hipError_t launch_vote_onehot(const OnehotArgs& a, int dtype_bytes, int dist, int groups, hipStream_t stream,
                              const LaunchTiming& tm = {});

}  // namespace glcm
