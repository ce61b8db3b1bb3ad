// Interface between the host runtime and the level-slice kernel (large N).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
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

// Most bands worth their sums: two steps of pairs each, or the one step of small
// images (up to 8 bands).  Measured on MI355X, us a call, two steps; one: 300^2 N =
// 200, two offsets 22.2; 18.3, N = 256, four 17.6; 16.0; 1024^2 N = 256, four 24.5;
// 31.1.
inline uint64_t level_most_bands(uint64_t chunks) {
  return std::max<uint64_t>({1, chunks / (2 * kLevelThreads), std::min<uint64_t>(8, chunks / kLevelThreads)});
}

// Layout for `rows` first-pixel rows of width W of an image of `levels` levels
// and K offsets: slices of whole rows of a GLCM that fit the LDS (lds_words), and
// bands so that the workgroups fill the CUs once.
struct LevelLayout {
  int slices = 1, bands = 1;
  uint32_t slice_rows = 0, slice_dwords = 0, spill_cap = 0;
  uint64_t chunks = 0;
  uint64_t units = 0, row_words = 0;  // (offset, slice) pairs; words of partials a workgroup owns
  uint64_t bytes() const { return units * (uint64_t)bands * row_words * 4u; }
  // workgroups a CU holds
  uint64_t per_cu(uint64_t lds_words) const {
    return std::max<uint64_t>(1, std::min<uint64_t>(2, lds_words / slice_dwords));
  }
  void set_bands(int b) {
    bands = b;
    // a spill takes 2^15 of a workgroup's pairs (at most 16 per chunk)
    spill_cap = (uint32_t)((chunks / (uint64_t)b + 1) * 16 / 32768 + 1);
    row_words = (uint64_t)slice_dwords + 1 + spill_cap;
  }
  // As many of the bands as `room` bytes hold; false if not even one does.
  bool fit(uint64_t room) {
    int b = bands;
    if (bytes() > room) b = (int)std::max<uint64_t>(1, room / (bytes() / (uint64_t)b));
    for (; b >= 1; --b) {  // (fewer bands have longer spill lists)
      set_bands(b);
      if (bytes() <= room) return true;
    }
    return false;
  }
};

inline LevelLayout level_layout(int levels, int K, int W, int rows, int lds_words, int cus) {
  LevelLayout L;
  const uint64_t N = (uint64_t)levels, pitch = level_pitch((uint32_t)levels);
  const uint64_t most = (uint64_t)lds_words / pitch;  // levels per slice
  const uint64_t S0 = (N + most - 1) / most;
  L.slice_rows = (uint32_t)((N + S0 - 1) / S0);
  L.slices = (int)((N + L.slice_rows - 1) / L.slice_rows);
  L.slice_dwords = (uint32_t)(((uint64_t)L.slice_rows * pitch + 3) & ~3ull);
  L.units = (uint64_t)K * (uint64_t)L.slices;
  L.chunks = (((uint64_t)W + 15) / 16) * (uint64_t)rows;
  const uint64_t fill = std::max<uint64_t>(1, (uint64_t)std::max(1, cus) * L.per_cu((uint64_t)lds_words) / L.units);
  L.set_bands((int)std::min(fill, level_most_bands(L.chunks)));
  return L;
}

// Bytes of partials that hold every call of a plan of N levels, at most K
// offsets and images up to W x H: counted by level, and by value for every
// number of values below N whose GLCM is one slice (a workgroup fewer or more a
// CU, so often more bytes than by level: N = 300, one offset, 4096^2: 33.8
// against 23.2 MB).
inline uint64_t level_reserve(int N, int K, int W, int H, int lds_words, int cus) {
  uint64_t most = 0;
  for (int levels = N; levels >= 1; --levels) {
    const LevelLayout L = level_layout(levels, K, W, H, lds_words, cus);
    if (levels < N && L.slices != 1) continue;
    // workgroups and entries of their spill lists, whatever the offsets and rows of a call
    const uint64_t groups = std::min(std::max(L.units, (uint64_t)std::max(1, cus) * L.per_cu((uint64_t)lds_words)),
                                     L.units * level_most_bands(L.chunks));
    const uint64_t spills = L.units * (L.chunks / 2048 + 1) + 2 * groups;
    most = std::max(most, (groups * ((uint64_t)L.slice_dwords + 1) + spills) * 4u);
  }
  return most;
}

// A plan's partials of the level-slice kernel.  Made once, for every call the
// plan can get, and neither moved nor freed before the plan is: a captured
// graph keeps the pointer.  Without it (not allowed, no memory left) the plan
// counts with ranges of 32-bit bins, which need none.
struct LevelStore {
  uint32_t* mem = nullptr;
  size_t bytes = 0;
  // true when the store exists, or `make` (bytes -> pointer or null) could be
  // asked for it and gave it
  template <class Make>
  bool hold(uint64_t want, uint64_t most, bool may_allocate, Make make) {
    if (mem) return true;
    if (!may_allocate || want > most) return false;
    mem = (uint32_t*)make((size_t)want);
    if (mem) bytes = (size_t)want;
    return mem != nullptr;
  }
};

hipError_t launch_vote_levels(const LevelArgs& a, int dtype_bytes, hipStream_t stream, const LaunchTiming& tm = {});

}  // namespace glcm
