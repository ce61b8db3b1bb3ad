// Co-occurrence counts of N <= 16 levels as a contraction: with a(p, i) = 1
// where pixel p has level i, P(i, j) = sum_p a(p, i) a(p + d, j), a product of
// one-hot matrices for v_mfma_f32_16x16x128 on 4-bit floats (128 pixels, 16 x
// 16 levels an instruction).  Included by the .hip files only.
//
// Lane l = 16 g + m of a wavefront holds, for its group's window of 32 pixels
// (its 32 K slots), the indicator of level m: a 4-bit 0.5 where the pixel has
// it, 0 elsewhere, so a product of two is 1/4 and the fp32 sum of a quarter
// per pair is exact below 2^24 pairs.  The indicator is made 32 pixels at a
// time as one bit mask e and spread with four masked shifts: dword j of the
// operand takes pixels 4 i + j in its nibbles i, so moving the pixels by one
// renames dwords and shifts one of them by a nibble.  Pixels outside the image
// have no level, hence an empty indicator: borders need no test.
//
// e comes from the wavefront's LDS: one lane converts a 32-pixel row of one
// group (quantize, transpose to four bit planes) and stores the four
// products of planes 0 and 1 and of planes 2 and 3, of which level m selects
// one each (q01[m & 3] & q23[m >> 2]).  60 or 64 rows of the four groups are
// converted at once by the wavefront's lanes, then walked one by one, a ring
// of the last reach + 1 rows staying in registers.  Nothing depends on the
// pixels' values: noise, smooth and constant images take the same time.
// Bound by the vector instructions of a row (spreading the mask, some 20) next
// to its products (16 cycles each).  Measured on MI355X against counting in
// LDS, N = 16, u8 noise: 64^2 15.3 + 4.2 (merge) to 5.0 us, 300^2 d = 1 19 to
// 8, 2937 x 3015 d = 1, 2, 4 34 to 25, 8192^2 d = 1, 2 76 to 61.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "glcm_device.h"
#include "glcm_onehot.h"
#include "glcm_wave.h"

namespace glcm {
namespace {

typedef int i4 __attribute__((ext_vector_type(4)));
typedef int i8v __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 onehot_mfma(i4 a, i4 b, f4 c) {
  const i8v A = __builtin_shufflevector(a, a, 0, 1, 2, 3, -1, -1, -1, -1);
  const i8v B = __builtin_shufflevector(b, b, 0, 1, 2, 3, -1, -1, -1, -1);
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A, B, c, 4, 4, 0, 0, 0, 0);  // 4: E2M1, no scales
}

constexpr uint32_t kNibbles = 0x11111111u;
constexpr uint32_t kOnehotRowDwords = 8;  // q01[4], q23[4]
// LDS dwords of a wavefront: 16 rows of four windows.
constexpr uint32_t kOnehotWaveDwords = 16u * 4u * kOnehotRowDwords;

// The indicator of a row, spread over the operand's dwords.  Slots (dwords) of
// an operand are the pixel classes (mod 4) 0, 2, 1, 3: with
//   v = [O3 << 4, O1, O0, O2, O1, O3, O2, O0 >> 4]
// the operands moved by -1, 0 and +1 pixels are v[0..3], v[2..5] and v[4..7],
// all on even registers, so they need no copies.
struct OnehotRow {
  i8v v;
  __device__ __forceinline__ void set(uint32_t e) {
    const uint32_t o0 = e & kNibbles, o1 = (e >> 1) & kNibbles, o2 = (e >> 2) & kNibbles, o3 = (e >> 3) & kNibbles;
    v[0] = (int)(o3 << 4);
    v[1] = (int)o1;
    v[2] = (int)o0;
    v[3] = (int)o2;
    v[4] = (int)o1;
    v[5] = (int)o3;
    v[6] = (int)o2;
    v[7] = (int)(o0 >> 4);
    asm volatile("" : "+v"(v));  // keeps the eight in one register tuple
  }
  // pixel p + DX in the place of pixel p
  template <int DX>
  __device__ __forceinline__ i4 moved() const {
    if constexpr (DX == 0) return __builtin_shufflevector(v, v, 2, 3, 4, 5);
    else if constexpr (DX == 1) return __builtin_shufflevector(v, v, 4, 5, 6, 7);
    else if constexpr (DX == -1) return __builtin_shufflevector(v, v, 0, 1, 2, 3);
    else {
      const uint32_t o0 = (uint32_t)v[2], o2 = (uint32_t)v[3], o1 = (uint32_t)v[4], o3 = (uint32_t)v[5];
      if constexpr (DX == 2) return i4{(int)o2, (int)(o0 >> 4), (int)o3, (int)(o1 >> 4)};
      else if constexpr (DX == -2) return i4{(int)(o2 << 4), (int)o0, (int)(o3 << 4), (int)o1};
      else if constexpr (DX == 4) return i4{(int)(o0 >> 4), (int)(o2 >> 4), (int)(o1 >> 4), (int)(o3 >> 4)};
      else return i4{(int)(o0 << 4), (int)(o2 << 4), (int)(o1 << 4), (int)(o3 << 4)};
    }
  }
};

// The raw 32 pixels of a window row, as loaded.
template <typename Pix>
struct OnehotRaw {
  uint32_t w[8 * sizeof(Pix)];
};

// 32 pixels from any address; n < 32 (rows narrower than a window): from the
// aligned dwords that hold the row's bytes, the last one standing in for those
// past the row (their pixels count nothing).
template <typename Pix>
__device__ __forceinline__ void onehot_load(OnehotRaw<Pix>& r, const Pix* p, int n) {
  if (n >= kOnehotWindow) {
    __builtin_memcpy(&r, p, sizeof(r));
  } else {
    constexpr int D = 8 * (int)sizeof(Pix);
    const uint32_t sh = (uint32_t)(uintptr_t)p & 3u;
    const uint32_t* a0 = (const uint32_t*)((uintptr_t)p & ~(uintptr_t)3);
    const int last = (n * (int)sizeof(Pix) + (int)sh - 1) >> 2;
    uint32_t d[D + 1];
#pragma unroll
    for (int k = 0; k <= D; ++k) d[k] = a0[k < last ? k : last];
#pragma unroll
    for (int k = 0; k < D; ++k) r.w[k] = __builtin_amdgcn_alignbyte(d[k + 1], d[k], sh);
  }
}

// The masks of a window row: valid = bits of the pixels inside the image.
template <typename Pix, class QA>
__device__ __forceinline__ void onehot_store(uint32_t* row, const OnehotRaw<Pix>& r, const QA& a, uint32_t valid) {
  uint32_t u[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {  // pixels 8 k + j in the low, 8 k + 4 + j in the high nibble of byte j
    uint32_t lo, hi;
    if constexpr (sizeof(Pix) == 1) {
      lo = quant4_u8(r.w[2 * k], a);
      hi = quant4_u8(r.w[2 * k + 1], a);
    } else {
      lo = quant4_u16(r.w[(4 * k) % (8 * sizeof(Pix))], r.w[(4 * k + 1) % (8 * sizeof(Pix))], a);
      hi = quant4_u16(r.w[(4 * k + 2) % (8 * sizeof(Pix))], r.w[(4 * k + 3) % (8 * sizeof(Pix))], a);
    }
    u[k] = lo | (hi << 4);
  }
  // 4 x 4 bytes transposed: x[j] holds pixel 4 i + j in its nibble i
  const uint32_t a0 = __builtin_amdgcn_perm(u[1], u[0], 0x05010400u), a1 = __builtin_amdgcn_perm(u[1], u[0], 0x07030602u);
  const uint32_t b0 = __builtin_amdgcn_perm(u[3], u[2], 0x05010400u), b1 = __builtin_amdgcn_perm(u[3], u[2], 0x07030602u);
  uint32_t x0 = __builtin_amdgcn_perm(b0, a0, 0x05040100u), x1 = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
  uint32_t x2 = __builtin_amdgcn_perm(b1, a1, 0x05040100u), x3 = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
  // 4 x 4 bits of every nibble transposed: plane t has pixel 4 i + j at bit 4 i + j
  auto swap = [](uint32_t& p, uint32_t& q, uint32_t mask, int s) {
    const uint32_t np = (p & mask) | ((q << s) & ~mask), nq = ((p >> s) & mask) | (q & ~mask);
    p = np;
    q = nq;
  };
  swap(x0, x2, 0x33333333u, 2);
  swap(x1, x3, 0x33333333u, 2);
  swap(x0, x1, 0x55555555u, 1);
  swap(x2, x3, 0x55555555u, 1);
  uint4 lo, hi;
  lo.x = ~x0 & ~x1 & valid;
  lo.y = x0 & ~x1 & valid;
  lo.z = ~x0 & x1 & valid;
  lo.w = x0 & x1 & valid;
  hi.x = ~x2 & ~x3;
  hi.y = x2 & ~x3;
  hi.z = ~x2 & x3;
  hi.w = x2 & x3;
  ((uint4*)row)[0] = lo;
  ((uint4*)row)[1] = hi;
}

template <int S>
struct OnehotOffset {  // slot S's offset
  static constexpr int d = S < 4 ? 1 : (S < 8 ? 2 : 4);
  static constexpr int dx = S % 4 == 0 ? d : (S % 4 == 1 ? -d : (S % 4 == 2 ? 0 : d)), dy = S % 4 == 0 ? 0 : d;
};

// Adds the products for the first-pixel row in ring slot F: every slot of the
// distances in DIST (bit i: 2^i), wanted or not.  (Tests of the single slots
// in every step cost what they saved at 7 slots of 12; one test a slot and
// stride made chains of products on one sum, 1.6 times slower.)
template <int R, int DIST, int F, int S>
__device__ __forceinline__ void onehot_products(const i4& first, const OnehotRow (&ring)[R + 1],
                                                f4 (&acc)[onehot_slots(R)]) {
  if constexpr (S < onehot_slots(R)) {
    constexpr int dx = OnehotOffset<S>::dx, dy = OnehotOffset<S>::dy;
    if constexpr ((DIST >> (S / 4)) & 1)
      acc[S] = onehot_mfma(first, ring[(F + dy) % (R + 1)].template moved<dx>(), acc[S]);
    onehot_products<R, DIST, F, S + 1>(first, ring, acc);
  }
}

// Steps I .. of a stride of onehot_stride(R) rows: the row enters the ring, the
// row R above it is the first-pixel row.
template <int R, int DIST, int I>
__device__ __forceinline__ void onehot_steps(const uint32_t (&e)[onehot_stride(R)], OnehotRow (&ring)[R + 1],
                                             f4 (&acc)[onehot_slots(R)], const uint32_t (&own)[4]) {
  if constexpr (I < onehot_stride(R)) {
    ring[I % (R + 1)].set(e[I]);
    constexpr int F = (I + 1) % (R + 1);  // R rows above
    const i8v& v = ring[F].v;
    const i4 first = {v[2] & (int)own[0], v[3] & (int)own[2], v[4] & (int)own[1], v[5] & (int)own[3]};
    onehot_products<R, DIST, F, 0>(first, ring, acc);
    onehot_steps<R, DIST, I + 1>(e, ring, acc, own);
  }
}

// The cheapest candidate for an image of `rows` first-pixel rows (a lane each),
// the same on every lane.
template <int R>
__device__ __forceinline__ int onehot_best_rows(int windows, int rows, int waves) {
  const int n = (int)(threadIdx.x & 63u) + 1;
  // the cost above the candidate's number, so that the smallest is the cheapest
  uint32_t c = min(onehot_cost(n, windows, rows, R, waves), 0x3fffffeu) << 6 | (uint32_t)(n - 1);
#pragma unroll
  for (int o = 32; o; o >>= 1) c = min(c, (uint32_t)__shfl_xor((int)c, o));
  return onehot_candidate(__builtin_amdgcn_readfirstlane((int)(c & 63u)) + 1, R);
}

// One wavefront's share of an image's first-pixel rows [y0, y1): units unit,
// unit + stride, ... of four (window, segment) tasks each.  lds: the
// wavefront's own kOnehotWaveDwords.
template <typename Pix, int R, int DIST, class QA>
__device__ __forceinline__ void onehot_walk(const QA& a, const void* img, int64_t stride, int W, int H, int y0, int y1,
                                            int windows, int h, int tasks, int unit, int step,
                                            uint32_t* lds, f4 (&acc)[onehot_slots(R)]) {
  constexpr int BR = onehot_block_rows(R), U = onehot_stride(R);
  constexpr uint32_t kRow = 4u * kOnehotRowDwords;
  const int lane = threadIdx.x & 63;
  const int pg = lane & 3, prow = lane >> 2;  // converting: a row of group pg
  const int g = lane >> 4, m = lane & 15;     // counting: level m of group g
  uint32_t* mine = lds + (uint32_t)(prow * 4 + pg) * kOnehotRowDwords;
  const uint32_t* q01 = lds + (uint32_t)g * kOnehotRowDwords + (uint32_t)(m & 3);
  const uint32_t* q23 = lds + (uint32_t)g * kOnehotRowDwords + 4u + (uint32_t)(m >> 2);
  const int n = W < kOnehotWindow ? W : kOnehotWindow;
  const uint32_t inside = n == 32 ? ~0u : (1u << n) - 1u;
  // the rows being fetched: this lane's task (pg) of a unit
  const Pix* base = (const Pix*)img;
  OnehotSegment seg = {0, 0};
  bool live = false;
  OnehotRaw<Pix> raw;
  auto aim = [&](int u) {
    const int tp = 4 * u + pg, sp = tp / windows;
    live = tp < tasks && prow < BR;
    seg = onehot_segment(sp, h, y0, y1);
    base = (const Pix*)img + onehot_window(tp - sp * windows, windows, W, R).x;
  };
  auto fetch = [&](int b) {
    const int y = seg.ya + b + prow;
    if (live) onehot_load<Pix>(raw, base + (int64_t)(y < H ? y : H - 1) * stride, n);
  };
  aim(unit);
  fetch(0);
  const int rows = h + R;
  for (int u = unit; 4 * u < tasks; u += step) {
    const int tc = 4 * u + g, sc = tc / windows;
    const OnehotWindow wc = onehot_window(tc - sc * windows, windows, W, R);
    const uint32_t owned = tc < tasks ? (wc.hi >= 32 ? ~0u : (1u << wc.hi) - 1u) & ~((1u << wc.lo) - 1u) : 0u;
    uint32_t own[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) own[j] = (owned >> j) & kNibbles;
    OnehotRow ring[R + 1];
#pragma unroll
    for (int r = 0; r <= R; ++r) ring[r].set(0u);
    for (int b = 0; b < rows; b += BR) {
      if (live) {
        const int y = seg.ya + b + prow;
        onehot_store<Pix>(mine, raw, a, y >= seg.own && y < H ? inside : 0u);
      } else if (prow < BR) {
        ((uint4*)mine)[0] = make_uint4(0u, 0u, 0u, 0u);
      }
      // the next block, of this unit or the next one, is on its way while this
      // one is counted
      int next = b + BR;
      if (next >= rows) {
        next = 0;
        aim(u + step);  // (no live lane past the last unit)
      }
      fetch(next);
      wave_sync_lds();
      const int end = min(BR, rows - b);  // a multiple of U
      uint32_t e[U];
#pragma unroll
      for (int i = 0; i < U; ++i) e[i] = q01[(uint32_t)i * kRow] & q23[(uint32_t)i * kRow];
#pragma unroll 1
      for (int i0 = 0; i0 < end; i0 += U) {
        // the next stride's masks are read while this one is counted (the
        // last stride reads the first again)
        const uint32_t at = i0 + U < end ? (uint32_t)(i0 + U) * kRow : 0u;
        uint32_t lo[U], hi[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
          lo[i] = q01[at + (uint32_t)i * kRow];
          hi[i] = q23[at + (uint32_t)i * kRow];
        }
        onehot_steps<R, DIST, 0>(e, ring, acc, own);
#pragma unroll
        for (int i = 0; i < U; ++i) e[i] = lo[i] & hi[i];
      }
      wave_sync_lds();
    }
  }
}

// Adds a wavefront's products to hist[slot][16 i + j] (LDS): lane 16 g + j
// holds rows i = 4 g + v of column j, a quarter per pair.
template <int R, int DIST>
__device__ __forceinline__ void onehot_collect(uint32_t* hist, const f4 (&acc)[onehot_slots(R)]) {
  const uint32_t lane = threadIdx.x & 63u, at = (lane >> 4) * 64u + (lane & 15u);
#pragma unroll
  for (int s = 0; s < onehot_slots(R); ++s)
    if ((DIST >> (s / 4)) & 1) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        __hip_atomic_fetch_add(&hist[256u * (uint32_t)s + at + 16u * (uint32_t)v], (uint32_t)(acc[s][v] * 4.0f),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

}  // namespace
}  // namespace glcm
