// Interface between the host runtime and the level-slice kernel (large N).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "glcm_internal.h"

namespace glcm {

// Counts the K GLCMs of a large N slice by slice: a workgroup owns one offset,
// one slice of first-pixel levels (whole rows of the GLCM, 16-bit bins in LDS)
// and one band of the pairs, and stores its bins packed to its own row of
// `partials`; k_sum_levels adds the bands up.
struct LevelArgs {
  const void* img;   // any alignment (a multiple of the pixel size)
  int64_t stride;    // elements
  int W, H;
  int y_begin, y_end;  // first-pixel rows
  // the levels counted: q.nlev of them.  A range of fewer values than levels
  // (hi - lo + 1 < N and hi the type's largest, e.g. 8-bit images at N > 256)
  // is counted by value, and the sum spreads the bins: value v is level
  // (v - lo) N / q.nlev.
  Quant q;
  int qfast;
  uint32_t qfast_shift, qfast_mask;
  uint32_t N;                 // levels of out
  Quant div_n, div_values;    // magic/shift for dividing by N and by q.nlev
  int K;
  int32_t dx[kMaxK], dy[kMaxK];  // as given
  int slices;                 // S: level slices per GLCM
  uint32_t slice_rows;        // levels per slice (the last may have fewer)
  uint32_t pitch;             // dwords of a GLCM row in a slice (two bins each), odd
  uint32_t slice_dwords;      // slice_rows * pitch, rounded up to a multiple of 4
  Quant div_pitch;            // magic/shift for dividing by pitch
  int bands;                  // B: workgroups per (offset, slice)
  uint32_t* partials;         // [B][K S][slice_dwords] packed counts
  uint32_t* spill_count;      // [B][K S] entries in the spill list
  uint32_t* spills;           // [B][K S][spill_cap] bins of which 2^15 counts were taken out
  uint32_t spill_cap;
  uint32_t* out;              // [K][N][N]
  int accumulate;
};

constexpr int kLevelThreads = 1024;
constexpr int kLevelChunk = 16;  // pixels of a row a lane takes at once
// A lane's 16 pairs of a step may all fall into one bin: a step of the
// workgroup adds at most this many to a 16-bit bin.
constexpr uint32_t kLevelStep = (uint32_t)kLevelThreads * kLevelChunk;

// Valid first pixels of offset (dx, dy): columns [x0, x1), rows [y0, y1).
struct LevelRect {
  int x0, x1, y0, y1;
};
__host__ __device__ inline LevelRect level_rect(int W, int H, int y_begin, int y_end, int dx, int dy) {
  LevelRect r;
  r.x0 = dx < 0 ? -dx : 0;
  r.x1 = dx > 0 ? W - dx : W;
  r.y0 = y_begin > -dy ? y_begin : -dy;
  r.y1 = y_end < H - dy ? y_end : H - dy;
  if (r.x1 <= r.x0 || r.y1 <= r.y0) r.x0 = r.x1 = r.y0 = r.y1 = 0;
  return r;
}

// Chunk c of a row of the rectangle: 16 pixels from x, of which [skip, n) are
// its own.  The last chunk of a row starts 16 pixels before the rectangle's
// end, so every 16-pixel load of first or second pixels stays inside the row;
// a rectangle narrower than 16 pixels is one chunk of n < 16, read pixel by
// pixel.
struct LevelChunk {
  int x, skip, n;
};
__host__ __device__ inline LevelChunk level_chunk(const LevelRect& r, int c) {
  const int at = r.x0 + c * kLevelChunk, w = r.x1 - r.x0;
  if (w < kLevelChunk) return {r.x0, 0, w};
  const int x = at + kLevelChunk <= r.x1 ? at : r.x1 - kLevelChunk;
  return {x, at - x, kLevelChunk};
}

// An odd pitch: neighbouring levels of smooth images (b near a) then fall on
// banks that move with a as well as with b.
constexpr uint32_t level_pitch(uint32_t N) { return ((N + 1u) / 2u) | 1u; }

hipError_t launch_vote_levels(const LevelArgs& a, int dtype_bytes, hipStream_t stream, const LaunchTiming& tm = {});

}  // namespace glcm
