// Counting kernel for whole rows: any of the offsets with |dx|, |dy| <= 4, N <= 255.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "glcm_device.h"
#include "glcm_internal.h"
#include "glcm_merge.h"

namespace glcm {
namespace {

// ---------------------------------------------------------------------------
// Row kernel: the fast path for offsets with |dx| <= 4 and 0 <= dy <= MAXDY <=
// 4 after canonicalisation (an offset with dy < 0 is counted as its opposite and
// voted transposed), N <= 255.  Each lane owns a 16-pixel column chunk; a
// wavefront covers 64 chunks (a span of 1024 pixels) and walks down a run of
// first-pixel rows, RPW at a time.  The MAXDY rows below a band are the first
// rows of the next one and stay in registers, and the rows after them are on
// their way while the band is counted, so each pixel is read and quantized once
// a run (and MAXDY rows of the next run).  The horizontal neighbours come from
// the adjacent lanes through DPP wave shifts.
//
// Pixels outside the image (x < 0, x >= W, or rows >= H) get the sentinel
// level N.  The LDS copy of each GLCM is (N+1) x (N+1); votes touching a
// sentinel land in row or column N and are dropped by the merge, so the vote
// loop carries no bounds checks at all.
//
// Bound by the LDS: an atomic of 64 lanes takes 4.5 cycles and, on bins as they
// come, 5 more of bank conflicts, whatever the vector instructions next to it
// (4.1 a vote; with 4.8 and 5.8 the 8192^2 image took the same time).  Measured
// on MI355X (slabs of four rows read with their halo, before, and this walk):
// 8192^2 u16 band, N = 64, 12 offsets 236 to 224 us; u8 crops, 7 offsets: 2937 x
// 3015 noise, N = 16, 24.8 to 21.9, 1531 x 1489 smooth, N = 64, 29.8 and 29.8.
// Four rows at a time instead of two: 259, 23.0, 33.8 (registers).
// ---------------------------------------------------------------------------
struct Ring {
  uint32_t w[6];  // [left halo (4 px) | 16 px chunk | right halo (4 px)], one level per byte
};

// UNAL: a row of an image whose base or pitch is not 16-byte aligned, read in
// place as the dwords that hold it (load_row_unaligned; only the wave-boundary
// lanes read halo dwords, the only ones finish_row uses).
template <typename Pix, bool UNAL>
__device__ __forceinline__ void issue_row(RawChunk<Pix>& rc, const VoteArgs& a, int y, int x0, int lane) {
#pragma unroll
  for (int h = 0; h < (int)sizeof(Pix); ++h) {
    rc.v[h] = make_uint4(0u, 0u, 0u, 0u);
    rc.lh[h] = 0u;
    rc.rh[h] = 0u;
  }
  if (y >= a.H) return;
  if constexpr (UNAL) {
    load_row_unaligned<Pix, false>(rc, Geom{a.img, a.stride, a.W, a.H}, y, x0);
    return;
  }
  const Pix* row = (const Pix*)a.img + (int64_t)y * a.stride;
  if (x0 < a.W) rc.v[0] = *(const uint4*)(row + x0);
  if (sizeof(Pix) == 2 && x0 + 8 < a.W) rc.v[sizeof(Pix) - 1] = *(const uint4*)(row + x0 + 8);
  if (lane == 0 && x0 >= 16 && x0 - 4 < a.W) {
    if (sizeof(Pix) == 1) rc.lh[0] = *(const uint32_t*)(row + x0 - 4);
    else { const uint2 t = *(const uint2*)(row + x0 - 4); rc.lh[0] = t.x; rc.lh[sizeof(Pix) - 1] = t.y; }
  }
  if (lane == 63 && x0 + 16 < a.W) {
    if (sizeof(Pix) == 1) rc.rh[0] = *(const uint32_t*)(row + x0 + 16);
    else { const uint2 t = *(const uint2*)(row + x0 + 16); rc.rh[0] = t.x; rc.rh[sizeof(Pix) - 1] = t.y; }
  }
}

template <typename Pix>
__device__ __forceinline__ void finish_row(Ring& rg, const RawChunk<Pix>& rc, const VoteArgs& a, int y, int x0,
                                           int lane, bool edge, uint32_t sent4) {
  if (y >= a.H) {  // (the same on every lane)
#pragma unroll
    for (int m = 0; m < 6; ++m) rg.w[m] = sent4;
    return;
  }
  uint32_t c[4], lh, rh;
  if (sizeof(Pix) == 1) {
    c[0] = quant4_u8(rc.v[0].x, a); c[1] = quant4_u8(rc.v[0].y, a);
    c[2] = quant4_u8(rc.v[0].z, a); c[3] = quant4_u8(rc.v[0].w, a);
    lh = quant4_u8(rc.lh[0], a);
    rh = quant4_u8(rc.rh[0], a);
  } else {
    c[0] = quant4_u16(rc.v[0].x, rc.v[0].y, a); c[1] = quant4_u16(rc.v[0].z, rc.v[0].w, a);
    c[2] = quant4_u16(rc.v[sizeof(Pix) - 1].x, rc.v[sizeof(Pix) - 1].y, a);
    c[3] = quant4_u16(rc.v[sizeof(Pix) - 1].z, rc.v[sizeof(Pix) - 1].w, a);
    lh = quant4_u16(rc.lh[0], rc.lh[sizeof(Pix) - 1], a);
    rh = quant4_u16(rc.rh[0], rc.rh[sizeof(Pix) - 1], a);
  }
  if (edge) {  // (the same on every lane)
#pragma unroll
    for (int m = 0; m < 4; ++m) c[m] = clip_dword(c[m], x0 + 4 * m, a.W, sent4);
    rh = clip_dword(rh, x0 + 16, a.W, sent4);
  }
  const uint32_t from_left = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c[3], kDppWaveShr1, 0xf, 0xf, false);
  const uint32_t from_right = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c[0], kDppWaveShl1, 0xf, 0xf, false);
  // wave-boundary lanes take the halo they loaded themselves (sentinel outside the image)
  if (x0 < 16) lh = sent4;
  rg.w[0] = lane == 0 ? lh : from_left;
  rg.w[1] = c[0]; rg.w[2] = c[1]; rg.w[3] = c[2]; rg.w[4] = c[3];
  rg.w[5] = lane == 63 ? rh : from_right;
}

// Second-pixel levels of the 16 chunk pixels for horizontal shift dx in [-4, 4]:
// bytes 4+dx .. 19+dx of the 24-byte ring row.  (dx is the same on every lane:
// a branch on its dwords and byte shifts of register pairs; shifts of 64-bit
// values take four times the cycles.)
__device__ __forceinline__ void window(const Ring& rg, int dx, uint32_t out[4]) {
  const uint32_t sh = (uint32_t)(4 + dx), r = sh & 3u;  // 0 .. 8
  if (sh < 4u) {
#pragma unroll
    for (int m = 0; m < 4; ++m) out[m] = __builtin_amdgcn_alignbyte(rg.w[m + 1], rg.w[m], r);
  } else if (sh < 8u) {
#pragma unroll
    for (int m = 0; m < 4; ++m) out[m] = __builtin_amdgcn_alignbyte(rg.w[m + 2], rg.w[m + 1], r);
  } else {
#pragma unroll
    for (int m = 0; m < 4; ++m) out[m] = rg.w[m + 2];
  }
}

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) uint32_t* lds_ptr;

// Four levels as two pairs of 16-bit numbers.
__device__ __forceinline__ us2 level_pair(uint32_t bytes, int half) {
  return __builtin_bit_cast(us2, __builtin_amdgcn_perm(0u, bytes, half ? 0x0c030c02u : 0x0c010c00u));
}

// base + 4 * (a half of x), one instruction
template <int HALF>
__device__ __forceinline__ uint32_t dword_at(us2 x, uint32_t base) {
  uint32_t r;
  if (HALF)
    asm("v_mad_u32_u16 %0, %1, 4, %2 op_sel:[1,0,0,0]" : "=v"(r) : "v"(x), "v"(base));
  else
    asm("v_mad_u32_u16 %0, %1, 4, %2" : "=v"(r) : "v"(x), "v"(base));
  return r;
}

// Votes of one offset whose canonical dy is S, for the RPW first-pixel rows of
// the band: dword (a * n1 + b) * D of the GLCM at LDS address C.  `first` holds
// the rows' a * n1 * D, 16 bits each (a GLCM in LDS has fewer dwords than that);
// two second pixels' dwords are one packed multiply-add, and an address one more
// instruction.  (Products of bytes and their sum took three a vote.)
template <int S, int RPW, int NROWS>
__device__ __forceinline__ void vote_offset(const Ring (&rows)[NROWS], const us2 (&first)[RPW][8], int nrows_first,
                                            int dx, uint32_t C, us2 D, uint32_t inc) {
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    if (i < nrows_first) {
      uint32_t b[4];
      window(rows[i + S], dx, b);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const us2 w = level_pair(b[t >> 1], t & 1) * D + first[i][t];
        __hip_atomic_fetch_add((lds_ptr)dword_at<0>(w, C), inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_add((lds_ptr)dword_at<1>(w, C), inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  }
}

// Sum of a bin's D dwords of copies.
__device__ __forceinline__ uint32_t bin_sum(const uint32_t* c, uint32_t D, bool c16) {
  uint32_t s = 0;
  if (D == 1 || D == 2) {  // (one load)
    const uint2 v = D == 1 ? make_uint2(c[0], 0u) : *(const uint2*)c;
    s = c16 ? (v.x & 0xffffu) + (v.x >> 16) + (v.y & 0xffffu) + (v.y >> 16) : v.x + v.y;
  } else {  // a multiple of 4
    for (uint32_t d = 0; d < D; d += 4) {
      const uint4 v = *(const uint4*)(c + d);
      s += c16 ? (v.x & 0xffffu) + (v.x >> 16) + (v.y & 0xffffu) + (v.y >> 16) + (v.z & 0xffffu) + (v.z >> 16) +
                     (v.w & 0xffffu) + (v.w >> 16)
               : (v.x + v.y) + (v.z + v.w);
    }
  }
  return s;
}

// Merge: word (k, i, j) of the partition, k counted from its first GLCM, is the
// sum of bin k * n1 * n1 + i * n1 + j (i and j exchanged where bit k of tmask is
// set).  A thread steps from word to word with carries instead of divisions.
__device__ __forceinline__ void store_rows(const VoteArgs& a, const uint32_t* lds, uint32_t pbase, uint32_t pwords,
                                           int region, uint32_t D, unsigned long long tmask) {
  __syncthreads();
  const uint32_t N = a.q.nlev, n1 = a.pitch, NN = N * N, nn1 = n1 * n1, step = blockDim.x;
  uint32_t* dst = a.xbuf ? xcd_slice(a) + pbase : a.partials + (size_t)region * a.words_total + pbase;
  const uint32_t sk = step / NN, si = (step - sk * NN) / N, sj = step - sk * NN - si * N;
  uint32_t k = threadIdx.x / NN, i = (threadIdx.x - k * NN) / N, j = threadIdx.x - k * NN - i * N;
  for (uint32_t w = threadIdx.x; w < pwords; w += step) {
    const uint32_t s = bin_sum(lds + (k * nn1 + ((tmask >> k) & 1ull ? j * n1 + i : i * n1 + j)) * D, D, a.c16 != 0);
    if (!a.xbuf) dst[w] = s;
    else if (s) __hip_atomic_fetch_add(dst + w, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    j += sj;
    const uint32_t cj = j >= N;
    j -= cj ? N : 0u;
    i += si + cj;
    const uint32_t ci = i >= N;
    i -= ci ? N : 0u;
    k += sk + ci;
  }
}

template <typename Pix, int MAXDY, int RPW, bool UNAL>
__global__ __launch_bounds__(rows_max_threads(sizeof(Pix), MAXDY, UNAL)) void k_vote_rows(VoteArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  const int2 rp = band_of_block(blockIdx.x, a.P, a.nregions);
  const int region = rp.x, part = rp.y;
  const uint32_t N = a.q.nlev, N1 = a.pitch, NN = N * N, NN1 = N1 * N1;
  // Partitions of the row kernel are groups of whole GLCMs (offsets).
  const uint32_t pbase = (uint32_t)part * a.part_words;
  const uint32_t pwords = min(a.part_words, a.words_total - pbase);
  const int kp0 = (int)(pbase / NN), kp1 = (int)((pbase + pwords) / NN);
  // Counters: R copies per bin, 32 bits each, or 16 bits each (copies 2m and
  // 2m+1 share a dword) when the host has bounded every count below 2^16.
  const uint32_t R = 1u << a.log2R;
  const uint32_t dwords_per_bin = a.c16 ? R / 2u : R;
  zero_lds(lds, (uint32_t)(kp1 - kp0) * NN1 * dwords_per_bin);
  __syncthreads();

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
  // This thread's dword of a bin is lane mod D (D = dwords per bin): lanes
  // sharing a dword are D chunks (16 D pixels) apart, so on smooth images they
  // rarely vote the same bin; with 16-bit counters the half is bit log2(D).
  const uint32_t D = dwords_per_bin;
  const uint32_t g = threadIdx.x & (D - 1u);
  const uint32_t h = (threadIdx.x / D) & 1u;
  const uint32_t B = D * 4u;  // bytes per bin (all copies)
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)lds + g * 4u;  // this thread's dword of the first bin
  const us2 D2 = {(unsigned short)D, (unsigned short)D}, N1D = {(unsigned short)(N1 * D), (unsigned short)(N1 * D)};
  const uint32_t inc = a.c16 ? (1u << (h * 16u)) : 1u;
  const uint32_t sent4 = N * 0x01010101u;
  const int y0 = a.y_begin + region * a.region_rows;
  const int y1 = min(a.y_end, y0 + a.region_rows);
  const int spans = (a.W + 1023) >> 10, rows_here = y1 - y0;
  // runs of a span: as many as there are wavefronts for it, of whole rows (with
  // three spans for sixteen wavefronts one is left over).  With three GLCMs or
  // fewer a run is not shorter than the MAXDY rows below it, which it reads and
  // quantizes too: its votes take no longer than that.  Measured on MI355X, us a
  // call, any length; MAXDY rows at least: N = 100, twelve offsets (three a
  // partition) 1000^2 46.8; 43.7; but N = 32, twelve (six) 300^2 19.3; 21.3, N = 64
  // 1000^2 33.5; 37.2.
  const int per_span = max(1, nwaves / spans);
  const int run_rows = max(kp1 - kp0 <= 3 ? MAXDY : 1, (rows_here + per_span - 1) / per_span);
  const int runs = (rows_here + run_rows - 1) / run_rows;  // (none where rows_here <= 0)
  constexpr int NROWS = RPW + MAXDY;

  for (int task = wave; task < spans * runs; task += nwaves) {
    const int run = task / spans, span = task - run * spans;
    const int x0 = ((span << 6) + lane) << 4;
    const bool edge = ((span + 1) << 10) + 4 > a.W;  // some pixel of the rows is past the right edge
    const int ya = y0 + run * run_rows, yb = min(y1, ya + run_rows);
    const int last = yb - 1 + MAXDY;  // the last row a pair of the run reaches
    Ring rows[NROWS];
    RawChunk<Pix> raw[RPW];
    {
      RawChunk<Pix> top[MAXDY];
#pragma unroll
      for (int i = 0; i < MAXDY; ++i) issue_row<Pix, UNAL>(top[i], a, ya + i, x0, lane);
#pragma unroll
      for (int i = 0; i < RPW; ++i)
        if (ya + MAXDY + i <= last) issue_row<Pix, UNAL>(raw[i], a, ya + MAXDY + i, x0, lane);
#pragma unroll
      for (int i = 0; i < MAXDY; ++i) finish_row<Pix>(rows[i], top[i], a, ya + i, x0, lane, edge, sent4);
    }
    for (int ys = ya; ys < yb; ys += RPW) {
      const int nfirst = min(RPW, yb - ys);
#pragma unroll
      for (int i = 0; i < RPW; ++i)
        if (i < nfirst) finish_row<Pix>(rows[MAXDY + i], raw[i], a, ys + MAXDY + i, x0, lane, edge, sent4);
#pragma unroll
      for (int i = 0; i < RPW; ++i)
        if (ys + RPW + MAXDY + i <= last) issue_row<Pix, UNAL>(raw[i], a, ys + RPW + MAXDY + i, x0, lane);
      us2 first[RPW][8];
#pragma unroll
      for (int i = 0; i < RPW; ++i)
#pragma unroll
        for (int t = 0; t < 8; ++t) first[i][t] = level_pair(rows[i].w[1 + (t >> 1)], t & 1) * N1D;
      for (int k = kp0; k < kp1; ++k) {
        const int dy = a.dy[k], dx = a.dx[k];
        const uint32_t C = lds0 + (uint32_t)(k - kp0) * NN1 * B;
        switch (dy) {
          case 0: vote_offset<0, RPW>(rows, first, nfirst, dx, C, D2, inc); break;
          case 1: if (MAXDY >= 1) vote_offset<(MAXDY >= 1 ? 1 : 0), RPW>(rows, first, nfirst, dx, C, D2, inc); break;
          case 2: if (MAXDY >= 2) vote_offset<(MAXDY >= 2 ? 2 : 0), RPW>(rows, first, nfirst, dx, C, D2, inc); break;
          case 3: if (MAXDY >= 3) vote_offset<(MAXDY >= 3 ? 3 : 0), RPW>(rows, first, nfirst, dx, C, D2, inc); break;
          case 4: if (MAXDY >= 4) vote_offset<(MAXDY >= 4 ? 4 : 0), RPW>(rows, first, nfirst, dx, C, D2, inc); break;
          default: break;  // the host never launches an offset with dy > MAXDY
        }
      }
      // the rows below the band are the first of the next one
#pragma unroll
      for (int i = 0; i < MAXDY; ++i) rows[i] = rows[RPW + i];
    }
  }
  store_rows(a, lds, pbase, pwords, region, D, a.tmask >> kp0);
}

}  // namespace

template <typename Pix, bool UNAL>
static hipError_t launch_rows_u(const VoteArgs& a, int maxdy, int wg, size_t lds_bytes, hipStream_t stream,
                                const LaunchTiming& tm) {
  const dim3 grid(a.nregions * a.P), block(wg);
  switch (maxdy) {
    case 1: return launch(k_vote_rows<Pix, 1, 2, UNAL>, a, grid, block, lds_bytes, stream, tm);
    case 2: return launch(k_vote_rows<Pix, 2, 2, UNAL>, a, grid, block, lds_bytes, stream, tm);
    case 4: return launch(k_vote_rows<Pix, 4, 2, UNAL>, a, grid, block, lds_bytes, stream, tm);
    default: return hipErrorInvalidValue;
  }
}

template <typename Pix>
static hipError_t launch_rows_t(const VoteArgs& a, int maxdy, int wg, size_t lds_bytes, hipStream_t stream,
                               const LaunchTiming& tm) {
  return a.unaligned ? launch_rows_u<Pix, true>(a, maxdy, wg, lds_bytes, stream, tm)
                     : launch_rows_u<Pix, false>(a, maxdy, wg, lds_bytes, stream, tm);
}

hipError_t launch_vote_rows(const VoteArgs& a, int dtype_bytes, int maxdy, int wg, size_t lds_bytes,
                            hipStream_t stream, const LaunchTiming& tm) {
  return dtype_bytes == 1 ? launch_rows_t<uint8_t>(a, maxdy, wg, lds_bytes, stream, tm)
                          : launch_rows_t<uint16_t>(a, maxdy, wg, lds_bytes, stream, tm);
}

}  // namespace glcm
