// Level-slice kernel: co-occurrence counts for N too large for LDS copies of
// the K GLCMs (the shared-memory bound of Section II.A, Eq. (4)-(6)).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdint>

#include "glcm_device.h"
#include "glcm_levels.h"

namespace glcm {
namespace {

constexpr int kXcds = 8;

// Workgroup -> (band, unit); the units (offset, slice) of one band run on one
// XCD (workgroup b on XCD b mod 8), whose L2 then serves the band's rows to
// all of them.
__device__ __forceinline__ int2 band_and_unit(int b, int units, int bands) {
  const int full = bands / kXcds * kXcds;
  if (b < full * units) {
    const int x = b % kXcds, s = b / kXcds;
    return make_int2(s / units * kXcds + x, s % units);
  }
  const int r = b - full * units;
  return make_int2(full + r / units, r % units);
}

// 16 pixels of a row from any address (dwords: 4 or 8).
template <typename Pix>
struct Pixels {
  uint32_t w[4 * sizeof(Pix)];
};
template <typename Pix>
__device__ __forceinline__ Pixels<Pix> load_pixels(const Pix* p) {
  Pixels<Pix> r;
  __builtin_memcpy(&r, p, sizeof(r));
  return r;
}
template <typename Pix>
__device__ __forceinline__ Pixels<Pix> load_pixels_upto(const Pix* p, int n) {
  Pixels<Pix> r;
  constexpr int per = 4 / (int)sizeof(Pix);
#pragma unroll
  for (int d = 0; d < 4 * (int)sizeof(Pix); ++d) r.w[d] = 0u;
#pragma unroll
  for (int t = 0; t < kLevelChunk; ++t)
    if (t < n) r.w[t / per] |= (uint32_t)p[t] << (8 * (int)sizeof(Pix) * (t % per));
  return r;
}

// Levels of the 16 pixels.  BYTE (N <= 256): packed, four to a dword.
template <typename Pix, bool BYTE>
struct Levels {
  uint32_t w[BYTE ? 4 : 16];
  __device__ __forceinline__ uint32_t get(int t) const {
    return BYTE ? (w[t >> 2] >> ((t & 3) * 8)) & 0xffu : w[t];
  }
};
template <typename Pix, bool BYTE>
__device__ __forceinline__ Levels<Pix, BYTE> levels_of(const Pixels<Pix>& p, const LevelArgs& a) {
  Levels<Pix, BYTE> r;
  if constexpr (BYTE) {
#pragma unroll
    for (int d = 0; d < 4; ++d)
      r.w[d] = sizeof(Pix) == 1 ? quant4_u8(p.w[d], a) : quant4_u16(p.w[2 * d], p.w[(2 * d + 1) % (4 * sizeof(Pix))], a);
  } else {
    constexpr int per = 4 / (int)sizeof(Pix);
#pragma unroll
    for (int t = 0; t < kLevelChunk; ++t) {
      const uint32_t v = (p.w[t / per] >> (8 * (int)sizeof(Pix) * (t % per))) & (sizeof(Pix) == 1 ? 0xffu : 0xffffu);
      r.w[t] = a.qfast ? v >> a.qfast_shift : quantize(v, a.q);
    }
  }
  return r;
}

// Non-zero unless the dwords all hold one value of SIZE bytes.
template <int SIZE, int D>
__device__ __forceinline__ uint32_t varies(const uint32_t (&w)[D]) {
  uint32_t d = w[0] ^ __builtin_amdgcn_alignbyte(w[0], w[0], SIZE);
#pragma unroll
  for (int i = 1; i < D; ++i) d |= w[i] ^ w[0];
  return d;
}

// Each lane takes 16 consecutive pairs at a time (two 16-byte loads at any
// alignment; lanes 16 pixels apart seldom vote the same bin on smooth images),
// the workgroup 1024 lanes a step.  Bin (a, b) of the slice is half b & 1 of
// dword (a - a0) pitch + b / 2: with w = base + 4 pitch (a - a0) + 2 b in hand a
// vote is the address w & ~3 and the increment 1 << (w << 3) (shifts take the
// low five bits, here 16 (b & 1)), five VALU instructions and one LDS atomic a
// pair.
//
// A lane whose 16 first pixels have one level, and its 16 second pixels too,
// adds its pairs at once; when that holds for every lane of the wavefront (flat
// regions, where all lanes vote one bin and each atomic takes 128 cycles), a
// step is one atomic instead of 16, also where a row ends in the wavefront (a
// lane then has fewer than 16 pairs): that is every step of rows up to 1024
// pixels.  Constant images, us a call, without and with the shortcut at row ends:
// 300^2 N = 256, one offset 49; 16, 1024^2 42; 17, 4096^2 with 12 offsets 310; 150
// (other images 114; 118).
//
// A 16-bit bin must stay below 2^16: with every bin below m, m + 2^14 s bounds
// it after s steps.  Every two steps (three while no bin has reached 2^14) the
// workgroup looks at all its bins and takes 2^15 out of those that reached it,
// one entry in the workgroup's spill list each; there are at most (pairs of
// the workgroup) / 2^15 of them.
//
// Bound: the vector instructions of a vote (71 % of the SIMDs' cycles), then LDS
// atomics on random banks (one copy of the bins; active 43 % of the time, two
// thirds of it conflicts).  Measured on MI355X, 4096^2 u8 smooth, N = 256, 12
// offsets (2.0e8 pairs): 111 us with the looks at the bins and the ends; 4 us more
// with an even row pitch.  The kernel before it, ten ranges of the 12 GLCMs' bins
// over the whole image each, took 449 us.
template <typename Pix, bool BYTE, bool SLICED>
__global__ __launch_bounds__(kLevelThreads) void k_vote_levels(LevelArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  __shared__ uint32_t s_high[2], s_spills;
  const int units = a.K * a.slices;
  const int2 bu = band_and_unit(blockIdx.x, units, a.bands);
  const int band = bu.x, unit = bu.y, k = unit / a.slices, slice = unit - k * a.slices;
  const uint32_t N = a.q.nlev;
  const uint32_t a0 = (uint32_t)slice * a.slice_rows, rows = min(a.slice_rows, N - min(N, a0));
  const int dx = __builtin_amdgcn_readfirstlane(a.dx[k]), dy = __builtin_amdgcn_readfirstlane(a.dy[k]);
  const LevelRect rc = level_rect(a.W, a.H, a.y_begin, a.y_end, dx, dy);
  const bool narrow = rc.x1 - rc.x0 < kLevelChunk;
  const uint32_t cpr = (uint32_t)(rc.x1 - rc.x0 + kLevelChunk - 1) / kLevelChunk;
  const uint64_t chunks = (uint64_t)cpr * (uint64_t)(rc.y1 - rc.y0);
  const uint64_t c0 = chunks * (uint64_t)band / (uint64_t)a.bands, c1 = chunks * (uint64_t)(band + 1) / (uint64_t)a.bands;
  const Pix* img = (const Pix*)a.img;
  const int64_t second = (int64_t)dy * a.stride + dx;

  // this lane's chunk of the next step: row y, chunk c of the row
  uint64_t at = c0 + threadIdx.x;
  int y = 0;
  uint32_t c = 0, sy = 0, sc = 0;
  if (cpr) {
    y = rc.y0 + (int)(at / cpr);
    c = (uint32_t)(at % cpr);
    sy = kLevelThreads / cpr;
    sc = kLevelThreads % cpr;
  }
  Pixels<Pix> p1 = {}, p2 = {};
  LevelChunk ch = {0, 0, 0};
  auto fetch = [&]() {
    ch = LevelChunk{0, 0, 0};
    if (at < c1) {
      ch = level_chunk(rc, (int)c);
      const Pix* p = img + (int64_t)y * a.stride + ch.x;
      if (narrow) {
        p1 = load_pixels_upto<Pix>(p, ch.n);
        p2 = load_pixels_upto<Pix>(p + second, ch.n);
      } else {
        p1 = load_pixels<Pix>(p);
        p2 = load_pixels<Pix>(p + second);
      }
    }
    at += kLevelThreads;
    y += (int)sy;
    c += sc;
    if (c >= cpr) {
      c -= cpr;
      ++y;
    }
  };
  fetch();
  zero_lds(lds, a.slice_dwords);
  if (threadIdx.x < 2) s_high[threadIdx.x] = 0u;
  if (threadIdx.x == 2) s_spills = 0u;
  const uint32_t base = lds_address(lds), pitch = 4u * a.pitch;
  const size_t row = (size_t)band * (size_t)units + (size_t)unit;
  uint32_t* list = a.spills + row * a.spill_cap;
  __syncthreads();

  int steps = 3, look = 0;
  for (uint64_t done = c0; done < c1;) {
    for (int s = 0; s < steps && done < c1; ++s, done += kLevelThreads) {
      const Levels<Pix, BYTE> f = levels_of<Pix, BYTE>(p1, a), g = levels_of<Pix, BYTE>(p2, a);
      const LevelChunk me = ch;
      uint32_t mixed;
      if constexpr (BYTE)
        mixed = varies<1>(f.w) | varies<1>(g.w);
      else
        mixed = varies<(int)sizeof(Pix)>(p1.w) | varies<(int)sizeof(Pix)>(p2.w);
      fetch();
      if (__any(me.skip != 0 || me.n != kLevelChunk)) {
        if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)mixed) == 0 && !__any(mixed != 0u && me.n != 0), 0)) {
          const uint32_t av = f.get(0) - a0, w2 = base + av * pitch + 2u * g.get(0);
          if (me.n > me.skip && (!SLICED || av < rows))
            __hip_atomic_fetch_add((lds_word_t*)(size_t)(w2 & ~3u), (uint32_t)(me.n - me.skip) << ((w2 << 3) & 31u),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          continue;
        }
#pragma unroll
        for (int t = 0; t < kLevelChunk; ++t) {
          const uint32_t av = f.get(t) - a0, w2 = base + av * pitch + 2u * g.get(t);
          if (t >= me.skip && t < me.n && (!SLICED || av < rows))
            __hip_atomic_fetch_add((lds_word_t*)(size_t)(w2 & ~3u), 1u << ((w2 << 3) & 31u), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      } else if (!__any(mixed != 0u)) {
        const uint32_t av = f.get(0) - a0, w2 = base + __umul24(av, pitch) + 2u * g.get(0);
        if (!SLICED || av < rows)
          __hip_atomic_fetch_add((lds_word_t*)(size_t)(w2 & ~3u), (uint32_t)kLevelChunk << ((w2 << 3) & 31u),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      } else {
#pragma unroll
        for (int t = 0; t < kLevelChunk; ++t) {
          const uint32_t av = SLICED ? f.get(t) - a0 : f.get(t);
          const uint32_t w2 = base + __umul24(av, pitch) + 2u * g.get(t);
          if (!SLICED || av < rows)
            __hip_atomic_fetch_add((lds_word_t*)(size_t)(w2 & ~3u), 1u << ((w2 << 3) & 31u), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    }
    if (done >= c1) break;
    __syncthreads();
    uint32_t any = 0u;  // or of all dwords: bit 15 of a half set in it, some bin has reached 2^15, ...
    for (uint32_t m = 4u * threadIdx.x; m < a.slice_dwords; m += 4u * kLevelThreads) {
      const uint4 v = *(const uint4*)(lds + m);
      any |= (v.x | v.y) | (v.z | v.w);
    }
    if (any & 0x80008000u) {
      for (uint32_t m = 4u * threadIdx.x; m < a.slice_dwords; m += 4u * kLevelThreads) {
#pragma unroll 1
        for (uint32_t e = 0; e < 4; ++e) {
          uint32_t v = lds[m + e];
          if ((v & 0x80008000u) == 0u) continue;
          for (uint32_t h = 0; h < 2; ++h) {
            if ((v >> (16u * h + 15u)) & 1u) {
              v -= 0x8000u << (16u * h);
              const uint32_t i = __hip_atomic_fetch_add(&s_spills, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              if (i < a.spill_cap) list[i] = 2u * (m + e) + h;
            }
          }
          lds[m + e] = v;
        }
      }
    }
    // (bins below 2^14 have neither bit 14 nor bit 15 set)
    if (__any((any & 0xc000c000u) != 0u) && (threadIdx.x & 63) == 0) s_high[look] = 1u;
    __syncthreads();
    steps = s_high[look] ? 2 : 3;
    // the other flag is clear for the next look, which is two barriers away
    look ^= 1;
    if (threadIdx.x == 0) s_high[look] = 0u;
  }
  __syncthreads();
  uint4* dst = (uint4*)(a.partials + row * a.slice_dwords);
  for (uint32_t m = threadIdx.x; m < a.slice_dwords / 4u; m += kLevelThreads) dst[m] = ((const uint4*)lds)[m];
  if (threadIdx.x == 0) a.spill_count[row] = s_spills;
}

// out[k][i][j] (+)= the bands' packed counts of the bin, plus 2^15 for each of
// its spills.
constexpr int kSumThreads = 256;

// The two bins of dword m of a unit, summed over the bands: x even, y odd bin.
__device__ __forceinline__ uint2 sum_bands(const LevelArgs& a, uint32_t unit, uint32_t m) {
  const size_t step = (size_t)(a.K * a.slices) * a.slice_dwords;
  const uint32_t* p = a.partials + (size_t)unit * a.slice_dwords + m;
  uint2 s = make_uint2(0u, 0u);
  int b = 0;
  for (; b + 8 <= a.bands; b += 8) {
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(size_t)(b + u) * step];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      s.x += v[u] & 0xffffu;
      s.y += v[u] >> 16;
    }
  }
  for (; b < a.bands; ++b) {
    const uint32_t v = p[(size_t)b * step];
    s.x += v & 0xffffu;
    s.y += v >> 16;
  }
  return s;
}

// A thread owns one dword (two bins) of a slice.
__global__ __launch_bounds__(kSumThreads) void k_sum_levels(LevelArgs a, uint32_t blocks_per_unit) {
  __shared__ uint32_t extra[2 * kSumThreads];
  const uint32_t unit = blockIdx.x / blocks_per_unit, b0 = (blockIdx.x - unit * blocks_per_unit) * kSumThreads;
  const uint32_t units = (uint32_t)(a.K * a.slices), N = a.N;
  const uint32_t k = unit / (uint32_t)a.slices, slice = unit - k * (uint32_t)a.slices;
  const uint32_t m = b0 + threadIdx.x;
  extra[threadIdx.x] = extra[threadIdx.x + kSumThreads] = 0u;
  uint32_t spilled = 0u;
  for (int b = (int)threadIdx.x; b < a.bands; b += kSumThreads) spilled |= a.spill_count[(size_t)b * units + unit];
  uint2 s = make_uint2(0u, 0u);
  if (m < a.slice_dwords) s = sum_bands(a, unit, m);
  if (__syncthreads_or((int)spilled)) {
    for (int b = 0; b < a.bands; ++b) {
      const size_t row = (size_t)b * units + unit;
      const uint32_t n = min(a.spill_count[row], a.spill_cap);
      for (uint32_t e = threadIdx.x; e < n; e += kSumThreads) {
        const uint32_t w = a.spills[row * a.spill_cap + e] - 2u * b0;
        if (w < 2u * kSumThreads)
          __hip_atomic_fetch_add(&extra[w], 0x8000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    __syncthreads();
    s.x += extra[2u * threadIdx.x];
    s.y += extra[2u * threadIdx.x + 1u];
  }
  // dword m holds bins (a0 + m / pitch, 2 (m mod pitch) and the next)
  const uint32_t a0 = slice * a.slice_rows, rows = min(a.slice_rows, N - min(N, a0));
  const uint32_t i = divide(m, a.div_pitch.magic, a.div_pitch.shift), j = 2u * (m - i * a.pitch);
  if (i >= rows) return;
  uint32_t* o = a.out + ((size_t)k * N + a0 + i) * N + j;
  if (j < N) o[0] = (a.accumulate ? o[0] : 0u) + s.x;
  if (j + 1u < N) o[1] = (a.accumulate ? o[1] : 0u) + s.y;
}

// The value counted for level i of N, V of them (V < N): ceil(i V / N) when
// that value's level is i, else V (no value has it).
__device__ __forceinline__ uint32_t value_of(const LevelArgs& a, uint32_t i) {
  const uint32_t V = a.q.nlev, v = divide(i * V + a.N - 1u, a.div_n.magic, a.div_n.shift);
  return v < V && divide(v * a.N, a.div_values.magic, a.div_values.shift) == i ? v : V;
}

// Fewer values than levels (one slice): a workgroup owns one row of out, level
// i of offset k.
constexpr uint32_t kSpreadValues = 320;  // more than one slice holds

__global__ __launch_bounds__(kSumThreads) void k_spread_levels(LevelArgs a) {
  __shared__ uint32_t extra[kSpreadValues];  // spilled counts of row vi, by second value
  const uint32_t N = a.N, V = a.q.nlev, k = blockIdx.x / N, i = blockIdx.x - k * N;
  const uint32_t vi = value_of(a, i), units = (uint32_t)a.K;
  for (uint32_t v = threadIdx.x; v < kSpreadValues; v += kSumThreads) extra[v] = 0u;
  uint32_t spilled = 0u;
  if (vi < V)
    for (int b = (int)threadIdx.x; b < a.bands; b += kSumThreads) spilled |= a.spill_count[(size_t)b * units + k];
  if (__syncthreads_or((int)spilled)) {
    for (int b = 0; b < a.bands; ++b) {
      const size_t row = (size_t)b * units + k;
      const uint32_t n = min(a.spill_count[row], a.spill_cap);
      for (uint32_t e = threadIdx.x; e < n; e += kSumThreads) {
        const uint32_t vj = a.spills[row * a.spill_cap + e] - 2u * vi * a.pitch;
        if (vj < V)
          __hip_atomic_fetch_add(&extra[vj], 0x8000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    __syncthreads();
  }
  uint32_t* o = a.out + ((size_t)k * N + i) * N;
  for (uint32_t j = threadIdx.x; j < N; j += kSumThreads) {
    const uint32_t vj = value_of(a, j);
    uint32_t s = 0u;
    if (vi < V && vj < V) {
      const uint2 t = sum_bands(a, k, vi * a.pitch + (vj >> 1));
      s = (vj & 1u ? t.y : t.x) + extra[vj];
    }
    o[j] = (a.accumulate ? o[j] : 0u) + s;
  }
}

template <typename K>
hipError_t launch(K kernel, const LevelArgs& a, hipStream_t stream, const LaunchTiming& tm) {
  const dim3 grid((unsigned)(a.bands * a.K * a.slices)), block(kLevelThreads);
  hipExtLaunchKernelGGL(kernel, grid, block, a.slice_dwords * 4u, stream, tm.start, tm.stop, 0u, a);
  return hipGetLastError();
}

template <typename Pix>
hipError_t launch_t(const LevelArgs& a, hipStream_t stream, const LaunchTiming& tm) {
  const bool sliced = a.slices > 1;
  if (a.q.nlev <= 256u)
    return sliced ? launch(k_vote_levels<Pix, true, true>, a, stream, tm)
                  : launch(k_vote_levels<Pix, true, false>, a, stream, tm);
  return sliced ? launch(k_vote_levels<Pix, false, true>, a, stream, tm)
                : launch(k_vote_levels<Pix, false, false>, a, stream, tm);
}

}  // namespace

hipError_t launch_vote_levels(const LevelArgs& a, int dtype_bytes, hipStream_t stream, const LaunchTiming& tm) {
  const hipError_t e = dtype_bytes == 1 ? launch_t<uint8_t>(a, stream, tm) : launch_t<uint16_t>(a, stream, tm);
  if (e != hipSuccess) return e;
  if (a.q.nlev != a.N) {
    hipLaunchKernelGGL(k_spread_levels, dim3((unsigned)a.K * a.N), dim3(kSumThreads), 0, stream, a);
    return hipGetLastError();
  }
  const uint32_t per_unit = (a.slice_dwords + kSumThreads - 1) / kSumThreads;
  hipLaunchKernelGGL(k_sum_levels, dim3(per_unit * (unsigned)(a.K * a.slices)), dim3(kSumThreads), 0, stream, a, per_unit);
  return hipGetLastError();
}

}  // namespace glcm
