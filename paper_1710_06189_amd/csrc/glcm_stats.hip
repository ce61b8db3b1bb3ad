// Post-processing of K co-occurrence matrices (N x N uint32 counts, the layout
// glcm_compute writes): the symmetric matrix P + P^T (a reading of the pair
// increment of Section I.B), the normalised matrix P / sum P, the mean of the
// normalised matrices over groups of directions, and Haralick's statistics
// f1..f13 (cited in the introduction).  Everything is computed in fp64 and
// stored as fp32, in a fixed order of operations: the same input always gives
// the same bits.
//
// N <= 32: one wavefront holds a matrix in its registers (many matrices, the
// output of a batch).  Above: workgroups per matrix (few matrices, the output
// of an image), split over the chip where the result allows it.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "glcm_device.h"
#include "glcm_stats.h"
#include "glcm_wave.h"

namespace glcm {
namespace {

constexpr int kStatsThreads = 256;
constexpr int kStatsWaves = kStatsThreads / 64;
constexpr int kWaveMaxN = 32;

// c / T correctly rounded, with r = 1 / T correctly rounded (Markstein 1990:
// each step adds the exactly known remainder times the reciprocal; the first
// leaves a faithful quotient, the second the nearest).  c and T are integers
// below 2^53, so nothing under- or overflows; c = T gives exactly 1.
__device__ __forceinline__ double quotient(double c, double T, double r) {
  double q = c * r;
  q = fma(fma(-q, T, c), r, q);
  return fma(fma(-q, T, c), r, q);
}

// ---------------------------------------------------------------------------
// A matrix of N <= 32 in a wavefront's registers: lane l holds the words
// word(v), v < kWords<L> (L = 16 for N <= 16, else 32), those below N^2 only.
// VEC: consecutive quads (16-byte loads; base 16-byte aligned, N^2 a multiple
// of 4), else every 64th word.
// ---------------------------------------------------------------------------
template <int L>
constexpr int kWords = L * L / 64;

template <bool VEC>
__device__ __forceinline__ uint32_t word_of(int lane, int v) {
  return VEC ? 4u * (uint32_t)lane + 256u * (uint32_t)(v >> 2) + (uint32_t)(v & 3) : (uint32_t)lane + 64u * (uint32_t)v;
}

// Whether any lane has a word v (the same on every lane: N = 17 needs 5 of 16).
template <bool VEC>
__device__ __forceinline__ bool has_word(uint32_t NN, int v) {
  return (VEC ? 256u * (uint32_t)(v >> 2) : 64u * (uint32_t)v) < NN;
}

template <int L, bool VEC>
__device__ __forceinline__ void load_matrix(uint32_t (&c)[kWords<L>], const uint32_t* P, uint32_t NN, int lane) {
  if constexpr (VEC) {
#pragma unroll
    for (int w = 0; w < kWords<L> / 4; ++w) {
      const uint32_t r = word_of<true>(lane, 4 * w);
      uint4 t = make_uint4(0u, 0u, 0u, 0u);
      if (r < NN) t = *(const uint4*)(P + r);
      c[4 * w] = t.x; c[4 * w + 1] = t.y; c[4 * w + 2] = t.z; c[4 * w + 3] = t.w;
    }
  } else {
#pragma unroll
    for (int v = 0; v < kWords<L>; ++v) {
      const uint32_t r = word_of<false>(lane, v);
      c[v] = 0u;
      if (has_word<false>(NN, v) && r < NN) c[v] = P[r];
    }
  }
}

template <int L, bool VEC, typename T>
__device__ __forceinline__ void store_matrix(T* out, const T (&s)[kWords<L>], uint32_t NN, int lane) {
  if constexpr (VEC) {
#pragma unroll
    for (int w = 0; w < kWords<L> / 4; ++w) {
      const uint32_t r = word_of<true>(lane, 4 * w);
      struct alignas(16) Quad { T e[4]; };
      if (r < NN) *(Quad*)(out + r) = Quad{{s[4 * w], s[4 * w + 1], s[4 * w + 2], s[4 * w + 3]}};
    }
  } else {
#pragma unroll
    for (int v = 0; v < kWords<L>; ++v) {
      const uint32_t r = word_of<false>(lane, v);
      if (has_word<false>(NN, v) && r < NN) out[r] = s[v];
    }
  }
}

// Row pitch of a matrix in LDS: odd, so that rows, columns and both diagonals
// spread over the banks.
__device__ __forceinline__ uint32_t lds_pitch(uint32_t N) { return N | 1u; }

// S = P + P^T modulo 2^32.  The wavefront holds the whole matrix before it
// writes, so in == out is safe.
// Bound: HBM (read and write K N^2 words).  Measured on MI355X, 16384 matrices
// of N = 16: 7.0 us, 4.8 TB/s (11.2 us with a workgroup per matrix reading the
// transposed words from memory).
template <int L, bool VEC>
__global__ __launch_bounds__(kStatsThreads) void k_symmetrize_wave(StatsArgs a) {
  __shared__ uint32_t tiles[kStatsWaves][L * (L + 1)];
  const uint32_t N = (uint32_t)a.N, NN = N * N, p = lds_pitch(N);
  const int lane = threadIdx.x & 63;
  uint32_t* M = tiles[threadIdx.x >> 6];
  const int nwaves = (int)gridDim.x * kStatsWaves;
  for (int k = (int)blockIdx.x * kStatsWaves + (int)(threadIdx.x >> 6); k < a.K; k += nwaves) {
    uint32_t c[kWords<L>];
    load_matrix<L, VEC>(c, a.in + (size_t)k * NN, NN, lane);
    wave_sync_lds();  // the previous matrix's reads of M are done
#pragma unroll
    for (int v = 0; v < kWords<L>; ++v) {
      if (!has_word<VEC>(NN, v)) break;
      const uint32_t r = word_of<VEC>(lane, v), i = divide(r, a.nmagic, a.nshift);
      if (r < NN) M[i * p + (r - i * N)] = c[v];
    }
    wave_sync_lds();
#pragma unroll
    for (int v = 0; v < kWords<L>; ++v) {
      if (!has_word<VEC>(NN, v)) break;
      const uint32_t r = word_of<VEC>(lane, v), i = divide(r, a.nmagic, a.nshift);
      if (r < NN) c[v] += M[(r - i * N) * p + i];
    }
    store_matrix<L, VEC>(a.out_u + (size_t)k * NN, c, NN, lane);
  }
}

// 32 < N <= 48: a workgroup per matrix, staged whole (an odd pitch, so the
// transposed reads spread over the banks); in == out is safe.  By tiles N = 33
// wastes most of two of its three pairs: 4096 matrices 14.0 us, staged 11.7, N = 48
// 17.4 and 14.7; 16384 of N = 33 42.8 and 24.7.
constexpr int kStagedMaxN = 48;
__global__ __launch_bounds__(kStatsThreads) void k_symmetrize_staged(StatsArgs a) {
  __shared__ uint32_t M[kStagedMaxN * (kStagedMaxN + 1)];
  const uint32_t N = (uint32_t)a.N, NN = N * N, p = lds_pitch(N);
  constexpr int kMost = (kStagedMaxN * kStagedMaxN + kStatsThreads - 1) / kStatsThreads;
  for (int k = blockIdx.x; k < a.K; k += gridDim.x) {
    const uint32_t* P = a.in + (size_t)k * NN;
    uint32_t* S = a.out_u + (size_t)k * NN;
    uint32_t c[kMost];
#pragma unroll
    for (int v = 0; v < kMost; ++v) {
      const uint32_t r = threadIdx.x + (uint32_t)(v * kStatsThreads);
      c[v] = r < NN ? P[r] : 0u;
    }
    __syncthreads();  // the previous matrix's reads are done
#pragma unroll
    for (int v = 0; v < kMost; ++v) {
      const uint32_t r = threadIdx.x + (uint32_t)(v * kStatsThreads), i = divide(r, a.nmagic, a.nshift);
      if (r < NN) M[i * p + (r - i * N)] = c[v];
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < kMost; ++v) {
      const uint32_t r = threadIdx.x + (uint32_t)(v * kStatsThreads), i = divide(r, a.nmagic, a.nshift);
      if (r < NN) S[r] = c[v] + M[(r - i * N) * p + i];
    }
  }
}

// N > 48: one workgroup per pair of 32 x 32 tiles (I, J), I <= J, of a matrix.
// Both tiles are read before either is written, and no other workgroup
// touches them, so in == out is safe.  12 matrices of N = 256 on MI355X: 4.4
// us (63 us with one workgroup a matrix).
constexpr uint32_t kTile = 32;

__global__ __launch_bounds__(kStatsThreads) void k_symmetrize_tiles(StatsArgs a, uint32_t pairs, uint64_t units) {
  __shared__ uint32_t A[kTile][kTile + 1], B[kTile][kTile + 1];
  const uint32_t N = (uint32_t)a.N;
  const uint32_t x = threadIdx.x % kTile, y = threadIdx.x / kTile;
  constexpr uint32_t kRows = kStatsThreads / kTile, kSteps = kTile / kRows;
  for (uint64_t u = blockIdx.x; u < units; u += gridDim.x) {
    const uint64_t k = u / pairs;
    uint32_t J = 0, t = (uint32_t)(u - k * pairs);
    while (t > J) t -= ++J;  // t = pair index J (J + 1) / 2 + I, I <= J
    const uint32_t I = t;
    const uint32_t* P = a.in + (size_t)k * N * N;
    uint32_t* S = a.out_u + (size_t)k * N * N;
    uint32_t va[kSteps], vb[kSteps];
#pragma unroll
    for (uint32_t s = 0; s < kSteps; ++s) {
      const uint32_t r = y + s * kRows;
      const uint32_t ia = I * kTile + r, ja = J * kTile + x, ib = J * kTile + r, jb = I * kTile + x;
      va[s] = ia < N && ja < N ? P[(size_t)ia * N + ja] : 0u;
      vb[s] = ib < N && jb < N ? P[(size_t)ib * N + jb] : 0u;
    }
    __syncthreads();  // the previous pair's reads are done
#pragma unroll
    for (uint32_t s = 0; s < kSteps; ++s) {
      A[y + s * kRows][x] = va[s];
      B[y + s * kRows][x] = vb[s];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t s = 0; s < kSteps; ++s) {
      const uint32_t r = y + s * kRows;
      const uint32_t ia = I * kTile + r, ja = J * kTile + x, ib = J * kTile + r, jb = I * kTile + x;
      if (ia < N && ja < N) S[(size_t)ia * N + ja] = va[s] + B[x][r];
      if (I != J && ib < N && jb < N) S[(size_t)ib * N + jb] = vb[s] + A[x][r];
    }
  }
}

// p = P / T, the quotient correctly rounded in fp64 and then to fp32 (an
// empty matrix: r = T = 1).  Group means: out[g] = (sum over the m matrices of
// group g, in order, of P_k / T_k) / m; an empty matrix adds nothing.
// AVG false: m = 1 and no division by m.  4096 groups of four matrices of N =
// 16 on MI355X: 6.6 us (16.0 us with a workgroup a group and fp64 divisions).
template <int L, bool VEC, bool AVG>
__global__ __launch_bounds__(kStatsThreads) void k_probability_wave(StatsArgs a) {
  const uint32_t NN = (uint32_t)a.N * (uint32_t)a.N;
  const int lane = threadIdx.x & 63;
  const int G = a.K / a.m, nwaves = (int)gridDim.x * kStatsWaves;
  for (int g = (int)blockIdx.x * kStatsWaves + (int)(threadIdx.x >> 6); g < G; g += nwaves) {
    const uint32_t* P = a.in + (size_t)g * (size_t)a.m * NN;
    uint32_t c[kWords<L>];
    double acc[kWords<L>];
    float o[kWords<L>];
    load_matrix<L, VEC>(c, P, NN, lane);
#pragma unroll
    for (int v = 0; v < kWords<L>; ++v) acc[v] = 0.0;
    for (int q = 0; q < a.m; ++q) {
      uint32_t next[kWords<L>];
      if (AVG && q + 1 < a.m) load_matrix<L, VEC>(next, P + (size_t)(q + 1) * NN, NN, lane);
      double t = 0.0;
#pragma unroll
      for (int v = 0; v < kWords<L>; ++v) t += (double)c[v];  // exact: below 2^53
      t = wave_sum(t);
      if (t == 0.0) t = 1.0;
      const double r = 1.0 / t;
#pragma unroll
      for (int v = 0; v < kWords<L>; ++v) acc[v] += quotient((double)c[v], t, r);
      if (AVG) {
#pragma unroll
        for (int v = 0; v < kWords<L>; ++v) c[v] = next[v];
      }
    }
#pragma unroll
    for (int v = 0; v < kWords<L>; ++v) o[v] = (float)(AVG ? acc[v] / (double)a.m : acc[v]);
    store_matrix<L, VEC>(a.out_f + (size_t)g * NN, o, NN, lane);
  }
}

// Sum of n doubles-exact counts over a workgroup of W wavefronts, to every
// thread (integers below 2^53: exact in any order).
template <int W>
__device__ __forceinline__ double total_wg(const uint32_t* P, uint32_t n, bool vec, double* part) {
  constexpr int kUnroll = W == 4 ? 4 : 8;
  double t = 0.0;
  if (vec) {
#pragma unroll kUnroll
    for (uint32_t r = 4u * threadIdx.x; r < n; r += 4u * 64u * W) {
      const uint4 v = *(const uint4*)(P + r);
      t += ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
    }
  } else {
#pragma unroll kUnroll
    for (uint32_t r = threadIdx.x; r < n; r += 64u * W) t += (double)P[r];
  }
  t = wave_sum(t);
  __syncthreads();  // the previous call's readers are done with part
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = t;
  __syncthreads();
  t = 0.0;
#pragma unroll
  for (int w = 0; w < W; ++w) t += part[w];
  return t;
}

// N > 32: every matrix (group) is written by a.parts workgroups, a.share words
// each.  Every one of them takes the totals it needs itself (the other
// workgroups' reads make them L2 hits), which costs less than a second
// launch: 12 matrices of N = 256 on MI355X normalised in 6.4 us, averaged by
// four in 15.5 us (82 and 326 us with one workgroup of 256 threads each).
constexpr int kWideWaves = 16;

template <bool AVG, int W>
__global__ __launch_bounds__(64 * W) void k_probability_wg(StatsArgs a) {
  __shared__ double part[W];
  __shared__ double totals[AVG ? kAverageMaxGroup : 1][2];
  const uint32_t NN = (uint32_t)a.N * (uint32_t)a.N;
  const uint64_t units = (uint64_t)(a.K / a.m) * a.parts;
  for (uint64_t u = blockIdx.x; u < units; u += gridDim.x) {
    const uint64_t g = u / a.parts;
    const uint32_t w0 = (uint32_t)(u - g * a.parts) * a.share;
    const uint32_t w1 = min(NN, w0 + a.share);
    const uint32_t* P = a.in + (size_t)g * (size_t)a.m * NN;
    float* o = a.out_f + (size_t)g * NN;
    if (AVG) {
      __syncthreads();  // the previous unit's readers are done with totals
      for (int q = 0; q < a.m; ++q) {
        const double t = total_wg<W>(P + (size_t)q * NN, NN, a.vec != 0, part);
        if (threadIdx.x == 0) {
          totals[q][0] = t == 0.0 ? 1.0 : t;
          totals[q][1] = t == 0.0 ? 1.0 : 1.0 / t;
        }
      }
      __syncthreads();
      for (uint32_t w = w0 + threadIdx.x; w < w1; w += blockDim.x) {
        double acc = 0.0;
        for (int q = 0; q < a.m; ++q) acc += quotient((double)P[(size_t)q * NN + w], totals[q][0], totals[q][1]);
        o[w] = (float)(acc / (double)a.m);
      }
    } else {
      double t = total_wg<W>(P, NN, a.vec != 0, part);
      if (t == 0.0) t = 1.0;
      const double r = 1.0 / t;
#pragma unroll 4
      for (uint32_t w = w0 + threadIdx.x; w < w1; w += blockDim.x) o[w] = (float)quotient((double)P[w], t, r);
    }
  }
}

// ---------------------------------------------------------------------------
// Natural logarithm of a positive normal double by table (Tang 1990): with x =
// 2^e m, 1 <= m < 2, and c = 1 + k / 128 the point nearest to m,
//     ln x = e ln 2 - ln(1/c) + ln(1 + r),  r = m (1/c) - 1,  |r| <= 2^-8,
// the last by its series to r^6 (the next term is up to r^7 / 7, below 2^-50 |r|).  c = 1 has
// 1/c = 1 and ln c = 0, and c = 2 has ln c = ln 2, so values next to 1 keep
// their relative accuracy from both sides and ln 1 is 0.  17 instructions and
// one LDS read, against about 60 of log().
// ---------------------------------------------------------------------------
constexpr int kLogPoints = 129;
constexpr double kLn2 = 0x1.62e42fefa39efp-1;
struct alignas(16) LogPoint {
  double inv, ln;  // 1/c rounded, -ln of that value
};

__device__ __forceinline__ void log_table(LogPoint* t) {
  for (int k = (int)threadIdx.x; k < kLogPoints; k += (int)blockDim.x) {
    const double inv = 1.0 / (1.0 + (double)k * (1.0 / 128.0));
    t[k] = LogPoint{inv, k == 0 ? 0.0 : (k == kLogPoints - 1 ? kLn2 : -log(inv))};
  }
}

__device__ __forceinline__ double log_tab(double x, const LogPoint* t) {
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  const uint32_t hi = (uint32_t)(b >> 32);
  const int e = (int)(hi >> 20) - 1023;
  const uint32_t k = ((hi & 0xfffffu) + 0x1000u) >> 13;
  const double m = __longlong_as_double((long long)((b & 0xfffffffffffffull) | 0x3ff0000000000000ull));
  const LogPoint p = t[k];
  const double r = fma(m, p.inv, -1.0);
  double s = fma(r, -1.0 / 6.0, 1.0 / 5.0);
  s = fma(r, s, -1.0 / 4.0);
  s = fma(r, s, 1.0 / 3.0);
  s = fma(r, s, -0.5);
  s = fma(r * r, s, r);
  return fma((double)e, kLn2, p.ln) + s;
}

__device__ __forceinline__ double neg_plogp(double p, const LogPoint* t) { return p > 0.0 ? -p * log_tab(p, t) : 0.0; }

// ---------------------------------------------------------------------------
// Haralick's f1..f13 (levels numbered from 0): f1 angular second moment, f2
// contrast, f3 correlation, f4 variance of the row marginal, f5 inverse
// difference moment, f6 sum average, f7 sum variance, f8 sum entropy, f9
// entropy, f10 difference variance, f11 difference entropy, f12 and f13 the
// information measures of correlation.
//
// Only f1 and f9 need the bins one by one.  The others follow from the exact
// integer marginals px, py and the distributions pd of |i - j| and ps of i + j:
// f2 = sum d^2 pd, f5 = sum pd / (1 + d^2), and since sum_j p(i, j) = px(i),
//     HXY1 = -sum p ln(px py) = HX + HY,  HXY2 = -sum px py ln(px py) = HX + HY.
// With a marginal on a single level p = px py, so f12 and f13 are 0 (and f3 is
// 1 by definition).
// The covariance is a difference of whole numbers below 2^53, or summed about the
// means, never a difference of rounded second moments: where the two marginals lie apart those are near N^2 and cancel (4e9
// counts in a corner left f3 at 0.20 instead of 0.289).
// ---------------------------------------------------------------------------
struct Moments {
  double asm_, ent;            // over the bins
  double cov, vx, hx, vy, hy;  // all three of cov, vx, vy times the same factor, or none
  double contrast, idm, vd, hd;  // of |i - j|
  double sa, vs, hs;           // of i + j
  bool one;                    // a marginal occupies a single level
};

__device__ __forceinline__ void haralick_store(const Moments& s, double var_x, float* f) {
  const double hxy = s.hx + s.hy, hmax = s.hx > s.hy ? s.hx : s.hy;
  const double x = 1.0 - exp(-2.0 * (hxy - s.ent));
  f[0] = (float)s.asm_;
  f[1] = (float)s.contrast;
  f[2] = (float)(s.one ? 1.0 : s.cov / sqrt(s.vx * s.vy));
  f[3] = (float)var_x;
  f[4] = (float)s.idm;
  f[5] = (float)s.sa;
  f[6] = (float)s.vs;
  f[7] = (float)s.hs;
  f[8] = (float)s.ent;
  f[9] = (float)s.vd;
  f[10] = (float)s.hd;
  f[11] = (float)(s.one ? 0.0 : (s.ent - hxy) / hmax);
  f[12] = (float)sqrt(!s.one && x > 0.0 ? x : 0.0);
}

// What a wavefront keeps of a matrix of N <= 32: sums over the counts (not the
// probabilities) of i, i^2, j, ... are whole numbers below 2^53 (T < 2^42), so
// they are exact, and so is sum i j c = (sum i^2 c + sum j^2 c - sum (i - j)^2 c)
// / 2; T^2 times a variance or the covariance then has one rounding.
struct WholeMoments {
  double T, asm_, ent;
  double x1, x2, hx, y1, y2, hy;  // rows, columns: first and second sum, entropy
  double d1, d2, hd, idm;         // |i - j|
  double s1, s2, hs;              // i + j - (N - 1): below N in magnitude
  double one;
};

__device__ __forceinline__ void haralick_store(const WholeMoments& w, double N, float* f) {
  const double T = w.T, inv2 = 1.0 / (T * T);
  Moments s;
  s.asm_ = w.asm_;
  s.ent = w.ent;
  s.vx = difference_of_products(T, w.x2, w.x1, w.x1);
  s.vy = difference_of_products(T, w.y2, w.y1, w.y1);
  s.cov = difference_of_products(T, 0.5 * (w.x2 + w.y2 - w.d2), w.x1, w.y1);
  s.hx = w.hx;
  s.hy = w.hy;
  s.contrast = w.d2 / T;
  s.idm = w.idm;
  s.vd = difference_of_products(T, w.d2, w.d1, w.d1) * inv2;
  s.hd = w.hd;
  s.sa = (w.s1 + (N - 1.0) * T) / T;
  s.vs = difference_of_products(T, w.s2, w.s1, w.s1) * inv2;
  s.hs = w.hs;
  s.one = w.one != 0.0;
  haralick_store(s, s.vx * inv2, f);
}

// Sum over a group of L lanes (16 or 32), on all of them.
template <int L>
__device__ __forceinline__ double group_sum(double v) {
  v = row16_sum(v);
  return L == 16 ? v : sum_xor16(v);
}

// One matrix of N <= L per wavefront.  The matrix is staged once in the
// wavefront's LDS; groups of L lanes then walk one distribution each (rows,
// columns, |i - j|, i + j: all four at once with L = 16, two and two with
// L = 32).  Lane l of a group adds N entries: row l, column l, or the
// (anti-)diagonal i - j = l (i + j = l) modulo N, which wraps once from
// i - j = l to l - N (from i + j = l to l + N).  Sums are taken within the
// group for all its distributions together.  The closing arithmetic (a
// square root, an exponential, divisions) runs for up to kPark matrices at
// once, a lane each.
// Bound: VALU issue (fp64).  Measured on MI355X, 16384 matrices of N = 16:
// 23.4 us; 83.8 us when lane l walked row, column and diagonals one after the
// other, every statistic was summed bin by bin over the whole wavefront and
// the logarithms were log()'s.
constexpr int kPark = 4;

template <int L, bool VEC>
__global__ __launch_bounds__(kStatsThreads, L == 16 ? 4 : 3) void k_haralick_wave(StatsArgs a) {
  __shared__ LogPoint table[kLogPoints];
  __shared__ uint32_t tiles[kStatsWaves][L * (L + 1)];
  __shared__ WholeMoments parked[kStatsWaves][kPark];
  const uint32_t N = (uint32_t)a.N, NN = N * N, pitch = lds_pitch(N);
  const int lane = threadIdx.x & 63;
  const uint32_t l = (uint32_t)lane & (L - 1u);
  uint32_t* M = tiles[threadIdx.x >> 6];
  WholeMoments* park = parked[threadIdx.x >> 6];
  const double dl = (double)l, idm_w = 1.0 / (1.0 + dl * dl);
  log_table(table);
  __syncthreads();
  const int nwaves = (int)gridDim.x * kStatsWaves;
  int held = 0, k_first = 0;
  for (int k = (int)blockIdx.x * kStatsWaves + (int)(threadIdx.x >> 6); k < a.K; k += nwaves) {
    uint32_t c[kWords<L>];
    load_matrix<L, VEC>(c, a.in + (size_t)k * NN, NN, lane);
    wave_sync_lds();  // the previous matrix's reads of M are done
    double T = 0.0;
#pragma unroll
    for (int v = 0; v < kWords<L>; ++v) {
      const uint32_t r = word_of<VEC>(lane, v), i = divide(r, a.nmagic, a.nshift);
      if (r < NN) M[i * pitch + (r - i * N)] = c[v];
      T += (double)c[v];
    }
    T = wave_sum(T);
    if (held == 0) k_first = k;
    WholeMoments* st = park + held;
    if (T == 0.0) {
      if (lane == 0) st->asm_ = -1.0;  // empty: zeros
    } else {
      const double inv = 1.0 / T;
      wave_sync_lds();
#pragma unroll
      for (int pass = 0; pass < (L == 16 ? 1 : 2); ++pass) {
        // 0 rows, 1 columns, 2 |i - j|, 3 i + j
        const int task = L == 16 ? lane >> 4 : 2 * pass + (lane >> 5);
        uint32_t idx = task == 1 ? l : l * pitch;
        const uint32_t step = task == 0 ? 1u : (task == 1 ? pitch : (task == 2 ? pitch + 1u : 1u - pitch));
        const uint32_t wrap_at = task < 2 ? N : (task == 2 ? N - l : l + 1u);
        const uint32_t wrap_by = task == 2 ? 0u - N * pitch : N * pitch;
        uint64_t sum = 0, before = 0;
        if (l < N) {
#pragma unroll 4
          for (uint32_t j = 0; j < N; ++j) {
            if (j == wrap_at) {
              idx += wrap_by;
              before = sum;
            }
            sum += M[idx];
            idx += step;
          }
        }
        if (wrap_at >= N) before = sum;
        // c0: the count of value l; c1: that of value l + N (i + j only).  The
        // wrapped part of |i - j| class d counts for N - d.
        const uint64_t after = sum - before;
        double c0 = (double)before;
        const double c1 = task == 3 ? (double)after : 0.0;
        const int from = (int)(((uint32_t)lane & ~(L - 1u)) + (l ? N - l : 0u));  // lane of class N - l
        const double folded = __shfl((double)after, from & 63);
        if (task == 2 && l != 0 && l < N) c0 += folded;
        const double v0 = task == 3 ? dl - (double)(N - 1u) : dl, v1 = dl + 1.0;
        const double a0 = v0 * c0, a1 = v1 * c1;
        const double m1 = group_sum<L>(a0 + a1), m2 = group_sum<L>(fma(v0, a0, v1 * a1));
        const double x0 = quotient(c0, T, inv), x1 = quotient(c1, T, inv);
        const double ent = group_sum<L>(neg_plogp(x0, table) + neg_plogp(x1, table));
        const uint64_t live = __ballot(c0 > 0.0);
        if (L == 16 || pass == 1) {
          const double idm = group_sum<L>(idm_w * x0);
          if (l == 0 && task == 2) {
            st->d1 = m1; st->d2 = m2; st->hd = ent; st->idm = idm;
          }
          if (l == 0 && task == 3) {
            st->s1 = m1; st->s2 = m2; st->hs = ent;
          }
        }
        if (L == 16 || pass == 0) {
          const uint32_t rows = (uint32_t)(L == 16 ? live & 0xffffu : live & 0xffffffffu);
          const uint32_t cols = (uint32_t)(L == 16 ? (live >> 16) & 0xffffu : live >> 32);
          if (l == 0 && task == 0) {
            st->x1 = m1; st->x2 = m2; st->hx = ent;
            st->one = __popc(rows) == 1 || __popc(cols) == 1 ? 1.0 : 0.0;
          }
          if (l == 0 && task == 1) {
            st->y1 = m1; st->y2 = m2; st->hy = ent;
          }
        }
      }
      double sq = 0.0, ent = 0.0;
#pragma unroll
      for (int v = 0; v < kWords<L>; ++v) {
        double p = (double)c[v] * inv;
        p = fma(fma(-p, T, (double)c[v]), inv, p);
        sq += p * p;
        ent += neg_plogp(p, table);
      }
      sq = wave_sum(sq);
      ent = wave_sum(ent);
      if (lane == 0) {
        st->T = T;
        st->asm_ = sq;
        st->ent = ent;
      }
    }
    if (++held == kPark || k + nwaves >= a.K) {
      wave_sync_lds();
      if (lane < held) {
        float* f = a.out_f + (size_t)(k_first + lane * nwaves) * kHaralickStats;
        const WholeMoments s = park[lane];
        if (s.asm_ < 0.0) {
          for (int q = 0; q < kHaralickStats; ++q) f[q] = 0.0f;
        } else {
          haralick_store(s, (double)N, f);
        }
      }
      wave_sync_lds();
      held = 0;
    }
  }
}

// N > 32: one workgroup of W wavefronts per matrix.  A first walk, a
// wavefront per row, takes the row sums, the column sums (a lane keeps its
// columns) and the total; a second takes the bins' own sums and adds each bin
// to its (anti-)diagonal with LDS atomics, where a wavefront's lanes hit
// consecutive words (32 bits wide where the total fits, else 64).  A quarter
// of the wavefronts then reduces each distribution.
// Bound: VALU issue and the LDS of the one CU that holds the matrix.
// Measured on MI355X, 12 matrices of N = 256: 55 us (282 us with 256 threads,
// a thread per diagonal and three logarithm terms a bin).
template <int W>
__device__ __forceinline__ void haralick_bins(const uint32_t* P, int N, double T, double inv, uint32_t* ps, uint32_t* pd,
                                              const LogPoint* table, double& sq, double& ent) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int j0 = 0; j0 < N; j0 += 256) {
    uint32_t next[4];
    auto load = [&](int i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + 64 * e + lane;
        next[e] = i < N && j < N ? P[(size_t)i * N + j] : 0u;
      }
    };
    load(wave);
#pragma unroll 1
    for (int i = wave; i < N; i += W) {
      uint32_t c[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) c[e] = next[e];
      load(i + W);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + 64 * e + lane;
        if (c[e] != 0u) {
          __hip_atomic_fetch_add(&ps[i + j], c[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          __hip_atomic_fetch_add(&pd[i > j ? i - j : j - i], c[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          double p = (double)c[e] * inv;
          p = fma(fma(-p, T, (double)c[e]), inv, p);
          sq += p * p;
          ent -= p * log_tab(p, table);
        }
      }
    }
  }
}

// The same for 2^32 counts and more, where sum i j c is no longer a whole number
// below 2^53: the covariance is summed about the means.  (Rare, so a bin at a time
// with few registers.)
template <int W>
__device__ __forceinline__ void haralick_bins_wide(const uint32_t* P, int N, double T, double inv, unsigned long long* ps,
                                                   unsigned long long* pd, const LogPoint* table, double mux, double muy,
                                                   double& sq, double& ent, double& cov) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll 1
  for (int i = wave; i < N; i += W) {
    double along = 0.0;
#pragma unroll 1
    for (int j = lane; j < N; j += 64) {
      const uint32_t c = P[(size_t)i * N + j];
      if (c == 0u) continue;
      __hip_atomic_fetch_add(&ps[i + j], (unsigned long long)c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_fetch_add(&pd[i > j ? i - j : j - i], (unsigned long long)c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      const double p = quotient((double)c, T, inv);
      sq += p * p;
      ent -= p * log_tab(p, table);
      along = fma(p, (double)j - muy, along);
    }
    cov = fma((double)i - mux, along, cov);
  }
}

template <int W>
__global__ __launch_bounds__(64 * W) void k_haralick(StatsArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ LogPoint table[kLogPoints];
  __shared__ double part[W], part2[W], part3[W], sums[W][5];
  __shared__ int occupied[W];
  const int N = a.N, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // row[N] col[N] as doubles, then ps[2N - 1] pd[N] as 64- or 32-bit counts
  double* row = (double*)dyn;
  double* col = row + N;
  unsigned long long* ps = (unsigned long long*)(col + N);
  unsigned long long* pd = ps + (2 * N - 1);
  uint32_t* ps32 = (uint32_t*)ps;
  uint32_t* pd32 = ps32 + (2 * N - 1);
  log_table(table);
  for (int k = blockIdx.x; k < a.K; k += gridDim.x) {
    const uint32_t* P = a.in + (size_t)k * (size_t)N * (size_t)N;
    float* f = a.out_f + (size_t)k * kHaralickStats;
    __syncthreads();  // the previous matrix is done with the LDS (and the table is written)
    for (int t = threadIdx.x; t < N; t += 64 * W) row[t] = col[t] = 0.0;
    for (int t = threadIdx.x; t < 3 * N - 1; t += 64 * W) ps[t] = 0;
    __syncthreads();
    double T = 0.0, cov = 0.0;  // cov: sum i j c (whole numbers below 2^53 for fewer than 2^32 counts)
    for (int j0 = 0; j0 < N; j0 += 256) {
      double cs[4] = {0.0, 0.0, 0.0, 0.0}, is[4] = {0.0, 0.0, 0.0, 0.0};
      for (int i = wave; i < N; i += W) {
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int j = j0 + 64 * e + lane;
          const double c = j < N ? (double)P[(size_t)i * N + j] : 0.0;
          cs[e] += c;
          is[e] = fma((double)i, c, is[e]);
          s += c;
        }
        s = wave_sum(s);
        T += s;
        if (lane == 0) row[i] += s;  // (row i is this wavefront's alone)
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + 64 * e + lane;
        cov = fma((double)j, is[e], cov);
        if (j < N && cs[e] != 0.0) __hip_atomic_fetch_add(&col[j], cs[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    if (lane == 0) part[wave] = T;
    __syncthreads();
    T = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) T += part[w];
    if (T == 0.0) {
      if (threadIdx.x < kHaralickStats) f[threadIdx.x] = 0.0f;
      continue;
    }
    const double inv = 1.0 / T;
    const bool narrow = T <= 4294967295.0;
    double sq = 0.0, ent = 0.0;
    if (narrow) {
      haralick_bins<W>(P, N, T, inv, ps32, pd32, table, sq, ent);
    } else {
      double mux = 0.0, muy = 0.0;  // by every wavefront
      for (int t = lane; t < N; t += 64) {
        mux = fma((double)t, row[t], mux);
        muy = fma((double)t, col[t], muy);
      }
      cov = 0.0;
      haralick_bins_wide<W>(P, N, T, inv, ps, pd, table, wave_sum(mux) * inv, wave_sum(muy) * inv, sq, ent, cov);
    }
    sq = wave_sum(sq);
    ent = wave_sum(ent);
    cov = wave_sum(cov);
    __syncthreads();
    if (lane == 0) {
      part[wave] = sq;
      part2[wave] = ent;
      part3[wave] = cov;
    }
    // distribution `task` (0 rows, 1 columns, 2 |i - j|, 3 i + j) by W / 4 wavefronts
    constexpr int G = W / 4;
    const int task = wave / G, first = (wave % G) * 64 + lane, n = task == 3 ? 2 * N - 1 : N;
    auto count = [&](int t) {
      return task == 0 ? row[t] : (task == 1 ? col[t]
                       : (task == 2 ? (narrow ? (double)pd32[t] : (double)pd[t]) : (narrow ? (double)ps32[t] : (double)ps[t])));
    };
    double mean = 0.0, h = 0.0, con = 0.0, idm = 0.0;
    int occ = 0;
    for (int t = first; t < n; t += 64 * G) {
      const double c = count(t), x = quotient(c, T, inv), d = (double)t;
      mean = fma(d, narrow ? c : x, mean);
      con += d * d * x;
      idm += x / (1.0 + d * d);
      h += neg_plogp(x, table);
      occ += x > 0.0 ? 1 : 0;
    }
    mean = wave_sum(mean);
    con = wave_sum(con);
    idm = wave_sum(idm);
    h = wave_sum(h);
    const int live = (int)wave_sum((uint32_t)occ);
    if (lane == 0) {
      sums[wave][0] = mean; sums[wave][1] = h; sums[wave][2] = con; sums[wave][3] = idm;
      occupied[wave] = live;
    }
    __syncthreads();
    mean = 0.0;
#pragma unroll
    for (int w = 0; w < G; ++w) mean += sums[task * G + w][0];
    if (narrow) mean = quotient(mean, T, inv);  // (of whole numbers: exact for a single level)
    double var = 0.0;
    for (int t = first; t < n; t += 64 * G) {
      const double d = (double)t - mean;
      var += d * d * quotient(count(t), T, inv);
    }
    var = wave_sum(var);
    if (lane == 0) sums[wave][4] = var;
    __syncthreads();
    if (threadIdx.x == 0) {
      auto over = [&](int tk, int q) {
        double v = 0.0;
        for (int w = 0; w < G; ++w) v += sums[tk * G + w][q];
        return v;
      };
      int ox = 0, oy = 0;
      Moments s;
      s.asm_ = s.ent = s.cov = 0.0;
      for (int w = 0; w < W; ++w) {
        s.asm_ += part[w];
        s.ent += part2[w];
        s.cov += part3[w];
      }
      for (int w = 0; w < G; ++w) {
        ox += occupied[w];
        oy += occupied[G + w];
      }
      s.hx = over(0, 1); s.vx = over(0, 4);
      s.hy = over(1, 1); s.vy = over(1, 4);
      s.hd = over(2, 1); s.vd = over(2, 4);
      s.contrast = over(2, 2); s.idm = over(2, 3);
      if (narrow) s.cov = difference_of_products(T, s.cov, over(0, 0), over(1, 0)) * inv * inv;
      s.sa = narrow ? over(3, 0) / T : over(3, 0); s.hs = over(3, 1); s.vs = over(3, 4);
      s.one = ox == 1 || oy == 1;
      haralick_store(s, s.vx, f);
    }
  }
}

unsigned grid_for(uint64_t units, unsigned most) { return (unsigned)(units < most ? (units > 0 ? units : 1) : most); }

// 16-byte loads and stores of whole matrices: every matrix starts on a
// 16-byte boundary.
bool vec_ok(const StatsArgs& a, const void* out) {
  return (a.N * a.N) % 4 == 0 && (uintptr_t)a.in % 16 == 0 && (uintptr_t)out % 16 == 0;
}

#define GLCM_WAVE_LAUNCH(K, UNITS, OUT, ...)                                                                     \
  do {                                                                                                           \
    const dim3 grid(grid_for(((uint64_t)(UNITS) + kStatsWaves - 1) / kStatsWaves, 8192)), block(kStatsThreads);  \
    const bool vec = vec_ok(a, OUT);                                                                             \
    if (a.N <= 16 && vec) hipLaunchKernelGGL((K<16, true __VA_ARGS__>), grid, block, 0, stream, a);              \
    else if (a.N <= 16) hipLaunchKernelGGL((K<16, false __VA_ARGS__>), grid, block, 0, stream, a);               \
    else if (vec) hipLaunchKernelGGL((K<32, true __VA_ARGS__>), grid, block, 0, stream, a);                      \
    else hipLaunchKernelGGL((K<32, false __VA_ARGS__>), grid, block, 0, stream, a);                              \
  } while (0)
#define GLCM_COMMA ,

// Workgroups per matrix (group of m) for N > 32: enough to fill the chip, at
// least 4096 words each, and few enough that the totals every one of them
// takes stay small beside the cache: parts * N^2 <= 2^26 words.
void split(StatsArgs* a, uint64_t groups) {
  const uint64_t NN = (uint64_t)a->N * (uint64_t)a->N;
  const uint64_t fill = std::max<uint64_t>(1, 1024 / std::max<uint64_t>(1, groups));
  const uint64_t parts = std::max<uint64_t>(1, std::min<uint64_t>({(NN + 4095) / 4096, fill, (uint64_t)(1u << 26) / NN}));
  a->share = (uint32_t)((((NN + parts - 1) / parts) + 3) & ~3ull);
  a->parts = (uint32_t)((NN + a->share - 1) / a->share);
}

// Small matrices leave four wavefronts enough to do, and more workgroups fit.
// Measured on MI355X, us a call, sixteen; four wavefronts: 4096 matrices normalised
// N = 33 23.8; 13.0, N = 64 33.3; 29.8, 4096 averaged by four N = 33 15.4; 12.8, N = 44
// 17.0; 18.1 (16384: 59.6; 55.0), N = 48 18.2; 20.9; few matrices the same.
template <bool AVG>
void launch_probability(const StatsArgs& a, uint64_t groups, hipStream_t stream) {
  const dim3 grid(grid_for(groups * a.parts, 8192));
  if (a.N <= (AVG ? 44 : 64))
    hipLaunchKernelGGL((k_probability_wg<AVG, 4>), grid, dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL((k_probability_wg<AVG, kWideWaves>), grid, dim3(64 * kWideWaves), 0, stream, a);
}

}  // namespace

hipError_t launch_symmetrize(const StatsArgs& a, hipStream_t stream) {
  if (a.N <= kWaveMaxN) {
    GLCM_WAVE_LAUNCH(k_symmetrize_wave, a.K, a.out_u, );
    return hipGetLastError();
  }
  if (a.N <= kStagedMaxN) {
    hipLaunchKernelGGL(k_symmetrize_staged, dim3(grid_for((uint64_t)a.K, 8192)), dim3(kStatsThreads), 0, stream, a);
    return hipGetLastError();
  }
  const uint64_t nt = ((uint64_t)a.N + kTile - 1) / kTile, pairs = nt * (nt + 1) / 2, units = pairs * (uint64_t)a.K;
  hipLaunchKernelGGL(k_symmetrize_tiles, dim3(grid_for(units, 16384)), dim3(kStatsThreads), 0, stream, a,
                     (uint32_t)pairs, units);
  return hipGetLastError();
}

hipError_t launch_normalize(const StatsArgs& a0, hipStream_t stream) {
  StatsArgs a = a0;
  a.m = 1;
  if (a.N <= kWaveMaxN) {
    GLCM_WAVE_LAUNCH(k_probability_wave, a.K, a.out_f, GLCM_COMMA false);
    return hipGetLastError();
  }
  a.vec = vec_ok(a, a.in) ? 1 : 0;
  split(&a, (uint64_t)a.K);
  launch_probability<false>(a, (uint64_t)a.K, stream);
  return hipGetLastError();
}

hipError_t launch_average(const StatsArgs& a0, hipStream_t stream) {
  StatsArgs a = a0;
  if (a.N <= kWaveMaxN) {
    GLCM_WAVE_LAUNCH(k_probability_wave, a.K / a.m, a.out_f, GLCM_COMMA true);
    return hipGetLastError();
  }
  a.vec = vec_ok(a, a.in) ? 1 : 0;
  const uint64_t groups = (uint64_t)(a.K / a.m);
  split(&a, groups);
  launch_probability<true>(a, groups, stream);
  return hipGetLastError();
}

hipError_t launch_haralick(const StatsArgs& a, hipStream_t stream) {
  if (a.N <= kWaveMaxN) {
    // as many wavefronts as the chip holds at 4 per SIMD: a wavefront then has
    // several matrices of a batch, whose closing arithmetic runs together
    const dim3 grid(grid_for(((uint64_t)a.K + kStatsWaves - 1) / kStatsWaves, 1024)), block(kStatsThreads);
    const bool vec = vec_ok(a, a.in);
    if (a.N <= 16 && vec) hipLaunchKernelGGL((k_haralick_wave<16, true>), grid, block, 0, stream, a);
    else if (a.N <= 16) hipLaunchKernelGGL((k_haralick_wave<16, false>), grid, block, 0, stream, a);
    else if (vec) hipLaunchKernelGGL((k_haralick_wave<32, true>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((k_haralick_wave<32, false>), grid, block, 0, stream, a);
    return hipGetLastError();
  }
  // Workgroups of four wavefronts once the matrices outnumber the CUs (a second
  // one waits for the first then, with sixteen), up to the N where the walk of a
  // matrix by four is a good deal longer.  Measured on MI355X, us a call, four; sixteen wavefronts:
  // K = 256 N = 33 11.6; 19.4, 64 16.3; 21.2, 96 27.1; 26.0, 128 34.7; 28.8.  K = 257
  // N = 33 11.9; 30.4, 96 27.8; 44.5, 128 35.1; 49.2, 160 53.4; 66.4.  K = 1024 N = 64
  // 21.0; 75.2, 96 44.4; 95.1, 128 57.2; 106, 160 90.3; 140; K = 512 N = 160 77.6; 71.3.
  // So the line lies low in N above 256 matrices, and at N <= 64 below them.
  const size_t lds = (size_t)(5 * a.N - 1) * sizeof(double);
  if (a.N <= 96 && a.K > 256)
    hipLaunchKernelGGL(k_haralick<4>, dim3(grid_for((uint64_t)a.K, 8192)), dim3(256), (uint32_t)lds, stream, a);
  else
    hipLaunchKernelGGL(k_haralick<16>, dim3(grid_for((uint64_t)a.K, 8192)), dim3(1024), (uint32_t)lds, stream, a);
  return hipGetLastError();
}

}  // namespace glcm
