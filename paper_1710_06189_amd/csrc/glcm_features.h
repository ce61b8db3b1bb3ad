// Five Haralick statistics of one GLCM by a wavefront or a workgroup: shared by
// the features kernel and the batch kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "glcm_wave.h"

namespace glcm {
namespace {

// ---------------------------------------------------------------------------
// Five Haralick statistics of one GLCM.  The contrast, the energy and the
// correlation come from exact sums of the counts; entropy and homogeneity are
// fp32 logarithms and quotients of the exact counts, added in fp64 and divided
// by T once, so no rounding is common to the terms: the largest relative error
// of 100 matrices of N = 16 is 5.4e-8, the final store's own.  (Terms of p = c (1 /
// T) in fp32, added in fp64: energy and entropy 1.2e-7, homogeneity 9.0e-8; added
// in fp32 2.0e-7.)
//
// N <= 160: the bins are walked 64 at a time, a segment of consecutive bins a
// step, every lane at work whatever N is.  (A lane that keeps a column idles where
// N is no divisor of 64: 4096 matrices of N = 33 22.9 us a call, 14.6 by segments.)
// The moments are whole numbers below 2^53, added in fp64.  Segment s belongs to class s mod W, W =
// features_waves(N); a lane's fp64 sums of a class are added in the order of its
// segments, the W classes in order, and the lanes then meet by exchanges.  So the
// result depends on W alone, not on which wavefronts did the work: W wavefronts
// with a class each (glcm_features_wg: few GLCMs), one with all classes in its
// registers (glcm_features_many: many) and one that takes them one after the
// other (glcm_features_wave: GLCMs in LDS) give the same bits.
//
// N > 160: a workgroup of 16 wavefronts; a lane keeps its column, so sum c,
// sum i c and sum i^2 c per column are all the integers a bin adds to.  (1024
// matrices of N = 129 66 us by columns, 57 by segments; N = 160 86 and 80; by
// columns N = 200 and above lose at most a quarter of the lanes and need fewer
// sums a bin.)
// ---------------------------------------------------------------------------
constexpr int kFeatures16 = 16;        // a lane per column up to here
constexpr int kFeaturesLinear = 160;   // segments of 64 bins up to here
constexpr int features_waves(int N) { return N <= 32 ? 1 : (N <= 48 ? 4 : 16); }

constexpr double kLn2 = 0x1.62e42fefa39efp-1, kLog2e = 0x1.71547652b82fep+0;

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63u; }

// c / (1 + d^2), rounded like the division (the quotient by the reciprocal,
// corrected by its exact remainder; no operand is denormal).  Half the
// instructions of a division: 12 matrices of N = 256 35.8 to 32.5 us.
__device__ __forceinline__ float homog_term(float c, float d) {
  const float y = fmaf(d, d, 1.0f), r = __builtin_amdgcn_rcpf(y), q = c * r;
  return fmaf(fmaf(-q, y, c), r, q);
}

// What a lane adds up over its bins for entropy and homogeneity (T below 2^32).
// The one bin with more than half of the counts waits in `most` (its term is
// left out of ent until features_most adds it), so that a step has no branch.
struct FeatureTerms {
  double ent, homog;  // -sum c log2 p, sum c / (1 + (i - j)^2)
};
__device__ __forceinline__ void features_term(uint32_t c, double dc, float d, uint32_t half, double invT, FeatureTerms& f) {
  const float p = c != 0u && c <= half ? (float)(dc * invT) : 1.0f;  // (log2 1 = 0)
  // of the significand alone (1/2 to 1), the exponent being exact: the
  // instruction's error, some 4e-8 of its result and of one sign, is then small
  // beside log2 p
  const double l = (double)__builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(p)) + (double)__builtin_amdgcn_frexp_expf(p);
  f.ent = fma(-dc, l, f.ent);
  f.homog += (double)homog_term((float)c, d);
}
// -c log2 p of the count above T / 2: log2 of u = 1 - x rounded, x the exact
// complement, times x / (1 - u), which keeps the relative accuracy next to p = 1
// (the rounding of u cancels).
__device__ __forceinline__ double features_most(uint32_t c, uint32_t T, double invT) {
  const double x = (double)(T - c) * invT;
  const float u = (float)(1.0 - x);
  const double y = 1.0 - (double)u, r = __builtin_amdgcn_rcp(y);
  const double lp = u == 1.0f ? -x * kLog2e : (double)__builtin_amdgcn_logf(u) * x * fma(fma(-y, r, 1.0), r, r);
  return -(double)c * lp;
}

// Total of the matrix over one wavefront's share of the words (w of W).
__device__ __forceinline__ unsigned long long features_total(const uint32_t* P, uint32_t NN, uint32_t w, uint32_t W,
                                                             uint32_t lane) {
  unsigned long long T = 0;
#pragma unroll 8
  for (uint32_t r = 64u * w + lane; r < NN; r += 64u * W) T += P[r];
  return wave_sum(T);
}

// Statistics of a matrix with no counts, or with 2^32 or more.
__device__ __forceinline__ float features_none(unsigned long long T) { return T == 0 ? 0.0f : __builtin_nanf(""); }

// ---------------------------------------------------------------------------
// N <= 160
// ---------------------------------------------------------------------------
struct FeatureMoments {
  double si, sii, sij, sj, sjj;  // of the counts: i, i^2, i j, j, j^2
  unsigned long long sq;         // sum c^2 (up to 2^64)
  __device__ __forceinline__ void add(double di, double dj, double dc, uint32_t c) {
    const double ic = di * dc, jc = dj * dc;
    si += ic;
    sj += jc;
    sii = fma(di, ic, sii);
    sij = fma(di, jc, sij);
    sjj = fma(dj, jc, sjj);
    sq += (unsigned long long)c * c;
  }
  __device__ __forceinline__ void reduce() {
    si = wave_sum(si);
    sii = wave_sum(sii);
    sij = wave_sum(sij);
    sj = wave_sum(sj);
    sjj = wave_sum(sjj);
    sq = wave_sum(sq);
  }
};

__device__ __forceinline__ void features_store(double T, const FeatureMoments& m, double ent, double homog, float* o) {
  const double inv = 1.0 / T;
  const double vi = difference_of_products(T, m.sii, m.si, m.si);  // T^2 var_i
  const double vj = difference_of_products(T, m.sjj, m.sj, m.sj);
  const double cv = difference_of_products(T, m.sij, m.si, m.sj);
  o[0] = (float)((m.sii + m.sjj - 2.0 * m.sij) / T);
  o[1] = (float)((double)m.sq * inv * inv);
  o[2] = (float)(ent * kLn2 * inv);
  o[3] = (float)(homog * inv);
  o[4] = (float)(vi != 0.0 && vj != 0.0 ? cv / sqrt(vi * vj) : 1.0);
}

// A lane's bins of segments first, first + step, ...; U of them in flight, in one
// class (C = 1) or segment u of a round in class u (C = U).
template <int U, int C>
__device__ __forceinline__ void features_segments(const uint32_t* P, uint32_t N, uint32_t T, double invT, uint32_t first,
                                                  uint32_t step, uint32_t lane, FeatureMoments& m,
                                                  FeatureTerms (&f)[C]) {
  static_assert(C == 1 || C == U, "");
  const uint32_t NN = N * N, half = T >> 1, hop = 64u * step;
  const uint32_t hi = hop / N, hj = hop - hi * N;
  uint32_t t = 64u * first + lane, i = t / N, j = t - i * N;
  uint32_t most = 0u;
  int at = 0;
#pragma unroll 1
  for (uint32_t s = 64u * first; s < NN; s += U * hop) {
    uint32_t c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      c[u] = t < NN ? P[t] : 0u;
      t += hop;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double dc = (double)c[u], di = (double)i, dj = (double)j;
      m.add(di, dj, dc, c[u]);
      features_term(c[u], dc, (float)(di - dj), half, invT, f[C == 1 ? 0 : u]);
      if (c[u] > half) {
        most = c[u];
        at = u;
      }
      i += hi;
      j += hj;
      const uint32_t carry = j >= N;
      j -= carry ? N : 0u;
      i += carry;
    }
  }
  if (most != 0u) {
    const double e = features_most(most, T, invT);
#pragma unroll
    for (int k = 0; k < C; ++k) f[k].ent += C == 1 || k == at ? e : 0.0;
  }
}

struct FeatureShare {  // scratch of a workgroup of W wavefronts
  unsigned long long total;
  FeatureMoments moments;
  double ent[64], homog[64];  // a lane's
};

// By a workgroup of W = features_waves(N) wavefronts, two barriers.  Every
// thread of the workgroup must call it.
template <int W>
__device__ __forceinline__ void glcm_features_wg(const uint32_t* P, uint32_t N, float* o, FeatureShare* share) {
  const uint32_t w = threadIdx.x >> 6, lane = lane_id();
  unsigned long long T = features_total(P, N * N, w, W, lane);
  if (lane == 0) share[w].total = T;
  __syncthreads();
  T = 0;
#pragma unroll
  for (int x = 0; x < W; ++x) T += share[x].total;
  if (T == 0 || T > 0xffffffffull) {
    if (threadIdx.x < 5) o[threadIdx.x] = features_none(T);
    return;
  }
  FeatureMoments m = {};
  FeatureTerms f[1] = {{0.0, 0.0}};
  features_segments<4, 1>(P, N, (uint32_t)T, 1.0 / (double)T, w, W, lane, m, f);
  m.reduce();
  if (lane == 0) share[w].moments = m;
  share[w].ent[lane] = f[0].ent;
  share[w].homog[lane] = f[0].homog;
  __syncthreads();
  if (w != 0) return;
  double ent = 0.0, homog = 0.0;
#pragma unroll
  for (int x = 0; x < W; ++x) {
    ent += share[x].ent[lane];
    homog += share[x].homog[lane];
  }
  m = {};
  if (lane < (uint32_t)W) m = share[lane].moments;
  m.reduce();
  ent = wave_sum(ent);
  homog = wave_sum(homog);
  if (lane == 0) features_store((double)T, m, ent, homog, o);
}

// By one wavefront with the W classes in its registers.  Every lane must call
// it; lane 0 writes o.
template <int W>
__device__ __forceinline__ void glcm_features_many(const uint32_t* P, uint32_t N, float* o, uint32_t lane) {
  const unsigned long long T = features_total(P, N * N, 0, 1, lane);
  if (T == 0 || T > 0xffffffffull) {
    if (lane < 5) o[lane] = features_none(T);
    return;
  }
  FeatureMoments m = {};
  FeatureTerms f[W] = {};
  features_segments<W == 1 ? 4 : W, W>(P, N, (uint32_t)T, 1.0 / (double)T, 0, 1, lane, m, f);
  double ent = 0.0, homog = 0.0;
#pragma unroll
  for (int x = 0; x < W; ++x) {
    ent += f[x].ent;
    homog += f[x].homog;
  }
  m.reduce();
  ent = wave_sum(ent);
  homog = wave_sum(homog);
  if (lane == 0) features_store((double)T, m, ent, homog, o);
}

// By one wavefront, class after class, with few registers and little code.
__device__ __forceinline__ void glcm_features_wave(const uint32_t* P, uint32_t N, float* o, uint32_t lane) {
  const unsigned long long T = features_total(P, N * N, 0, 1, lane);
  if (T == 0 || T > 0xffffffffull) {
    if (lane < 5) o[lane] = features_none(T);
    return;
  }
  const double invT = 1.0 / (double)T;
  const uint32_t W = (uint32_t)features_waves((int)N);
  FeatureMoments m = {};
  double ent = 0.0, homog = 0.0;
#pragma unroll 1
  for (uint32_t w = 0; w < W; ++w) {
    FeatureTerms f[1] = {{0.0, 0.0}};
    features_segments<1, 1>(P, N, (uint32_t)T, invT, w, W, lane, m, f);
    ent += f[0].ent;
    homog += f[0].homog;
  }
  m.reduce();
  ent = wave_sum(ent);
  homog = wave_sum(homog);
  if (lane == 0) features_store((double)T, m, ent, homog, o);
}

// N <= 16, by one wavefront: each group of 16 lanes keeps a column a lane.
// wide: the GLCM at P, a fourth of the rows per group; else up to four GLCMs,
// P's and the ones that follow (count in all), a group each.  o: the statistics,
// likewise.  The sums of four rows are added in the same order either way, so
// both give the same bits.  ROLLED: a row at a time (short code).  Every lane
// must call it.
template <bool ROLLED>
__device__ __forceinline__ void glcm_features_16(const uint32_t* P, uint32_t N, int count, bool wide, float* o,
                                                 uint32_t lane) {
  constexpr uint32_t U = kFeatures16 / 4;  // rows of a fourth
  const uint32_t q = lane >> 4, j = lane & 15u;
  const uint32_t mine = wide ? 0u : q;  // this lane's GLCM
  const bool live = (int)mine < count && j < N;
  const uint32_t begin = wide ? U * q : 0u, end = wide ? begin + U : (N + U - 1u) / U * U;
  P += mine * N * N;
  unsigned long long T = 0;
  for (uint32_t i = begin; i < end; i += U) {
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) T += live && i + u < N ? P[(i + u) * N + j] : 0u;
  }
  if (wide) T = sum_xor32(sum_xor16((uint64_t)T));
  T = row16_sum(T);
  const bool empty = T == 0 || T > 0xffffffffull;
  const double invT = 1.0 / (double)T, dj = (double)j;
  const uint32_t half = (uint32_t)T >> 1;
  double col = 0.0, ci = 0.0, cii = 0.0;
  unsigned long long sq = 0;
  FeatureTerms lower = {0.0, 0.0}, upper = {0.0, 0.0};  // rows 0 .. 7 (or the lane's fourth), 8 .. 15
  for (uint32_t i = begin; i < end; i += U) {
    uint32_t c[U], most = 0u;
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) c[u] = live && !empty && i + u < N ? P[(i + u) * N + j] : 0u;
    FeatureTerms f = {0.0, 0.0};
    auto row = [&](uint32_t cr, uint32_t r) {
      const double dc = (double)cr, di = (double)r, ic = di * dc;
      col += dc;
      ci += ic;
      cii = fma(di, ic, cii);
      sq += (unsigned long long)cr * cr;
      features_term(cr, dc, (float)(di - dj), half, invT, f);
      most = cr > half ? cr : most;
    };
    if constexpr (ROLLED) {
#pragma unroll 1
      for (uint32_t r = i; r < i + U; ++r) {
        row(c[0], r);
        c[0] = c[1];
        c[1] = c[2];
        c[2] = c[3];
      }
    } else {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) row(c[u], i + u);
    }
    if (most != 0u) f.ent += features_most(most, (uint32_t)T, invT);
    const bool up = !wide && i >= 2u * U;
    lower.ent += up ? 0.0 : f.ent;
    lower.homog += up ? 0.0 : f.homog;
    upper.ent += up ? f.ent : 0.0;
    upper.homog += up ? f.homog : 0.0;
  }
  if (wide) {  // the four fourths
    lower.ent = sum_xor16(lower.ent);
    lower.homog = sum_xor16(lower.homog);
    upper.ent = __shfl_xor(lower.ent, 32);
    upper.homog = __shfl_xor(lower.homog, 32);
    col = sum_xor32(sum_xor16(col));
    ci = sum_xor32(sum_xor16(ci));
    cii = sum_xor32(sum_xor16(cii));
    sq = sum_xor32(sum_xor16((uint64_t)sq));
  }
  const double ent = row16_sum(lower.ent + upper.ent), homog = row16_sum(lower.homog + upper.homog);
  FeatureMoments m;
  m.si = row16_sum(ci);
  m.sii = row16_sum(cii);
  m.sij = row16_sum(dj * ci);
  m.sj = row16_sum(dj * col);
  m.sjj = row16_sum(dj * dj * col);
  m.sq = row16_sum(sq);
  if ((int)mine >= count || (wide && q != 0u)) return;
  if (empty) {
    if (j < 5) o[5u * mine + j] = features_none(T);
  } else if (j == 0) {
    features_store((double)T, m, ent, homog, o + 5u * mine);
  }
}

// One GLCM's statistics by one wavefront, its counts in LDS.
__device__ __forceinline__ void glcm_features_any(const uint32_t* P, uint32_t N, float* o, uint32_t lane) {
  if (N <= kFeatures16)
    glcm_features_16<true>(P, N, 1, true, o, lane);
  else
    glcm_features_wave(P, N, o, lane);
}

// ---------------------------------------------------------------------------
// N > 160: whole-number sums of any N.
// ---------------------------------------------------------------------------
struct FeatureInts {
  unsigned long long si, sii, sij, sj, sjj, sq;
};

__device__ __forceinline__ void features_store(unsigned long long T, const FeatureInts& s, double ent, double homog, float* o) {
  using i128 = __int128;
  const i128 tT = (i128)T;
  const i128 vi = (i128)s.sii * tT - (i128)s.si * (i128)s.si;  // T^2 var_i
  const i128 vj = (i128)s.sjj * tT - (i128)s.sj * (i128)s.sj;  // T^2 var_j
  const i128 cv = (i128)s.sij * tT - (i128)s.si * (i128)s.sj;  // T^2 cov
  const unsigned long long sc = s.sii + s.sjj - 2ull * s.sij;
  const double dT = (double)T, inv = 1.0 / dT;
  o[0] = (float)((double)sc / dT);
  o[1] = (float)((double)s.sq * inv * inv);
  o[2] = (float)(ent * kLn2 * inv);
  o[3] = (float)(homog * inv);
  o[4] = (float)(vi != 0 && vj != 0 ? (double)cv / sqrt((double)vi * (double)vj) : 1.0);
}

struct FeatureLargeShare {
  unsigned long long total, ints[6];
  double ent[64], homog[64];
};

// By a workgroup of W wavefronts, a row of 64 columns at a time; two barriers.
// Bound: the logarithms of the one CU that holds the matrix.
template <int W>
__device__ __forceinline__ void glcm_features_large(const uint32_t* P, uint32_t N, float* o, FeatureLargeShare* share) {
  const uint32_t w = threadIdx.x >> 6, lane = lane_id();
  unsigned long long T = features_total(P, N * N, w, W, lane);
  if (lane == 0) share[w].total = T;
  __syncthreads();
  T = 0;
#pragma unroll
  for (int x = 0; x < W; ++x) T += share[x].total;
  if (T == 0 || T > 0xffffffffull) {
    if (threadIdx.x < 5) o[threadIdx.x] = features_none(T);
    return;
  }
  const double invT = 1.0 / (double)T;
  const uint32_t half = (uint32_t)T >> 1;
  FeatureInts s = {0, 0, 0, 0, 0, 0};
  FeatureTerms f = {0.0, 0.0};
  uint32_t most = 0u;
  constexpr uint32_t U = 4;  // rows in flight
  for (uint32_t j = lane; j - lane < N; j += 64u) {  // (the same trip count on every lane)
    const float fj = (float)j;
    uint32_t col = 0;  // (sums of a column stay below T)
    unsigned long long ci = 0, cii = 0;
    for (uint32_t t = w; t < N; t += U * W) {
      uint32_t c[U], any = 0u;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t i = t + u * W;
        c[u] = j < N && i < N ? P[(size_t)i * N + j] : 0u;
        any |= c[u];
      }
      if (__ballot(any != 0u) == 0ull) continue;  // (away from the diagonal of a smooth image)
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t i = t + u * W;
        col += c[u];
        ci += (unsigned long long)i * c[u];
        cii += (unsigned long long)(i * i) * c[u];
        s.sq += (unsigned long long)c[u] * c[u];
        features_term(c[u], (double)c[u], (float)i - fj, half, invT, f);
        most = c[u] > half ? c[u] : most;
      }
    }
    s.si += ci;
    s.sii += cii;
    s.sij += (unsigned long long)j * ci;
    s.sj += (unsigned long long)j * col;
    s.sjj += (unsigned long long)(j * j) * col;
  }
  if (most != 0u) f.ent += features_most(most, (uint32_t)T, invT);
  const unsigned long long ints[6] = {wave_sum(s.si), wave_sum(s.sii), wave_sum(s.sij),
                                      wave_sum(s.sj), wave_sum(s.sjj), wave_sum(s.sq)};
  if (lane == 0) {
#pragma unroll
    for (int q = 0; q < 6; ++q) share[w].ints[q] = ints[q];
  }
  share[w].ent[lane] = f.ent;
  share[w].homog[lane] = f.homog;
  __syncthreads();
  if (w != 0) return;
  double ent = 0.0, homog = 0.0;
#pragma unroll
  for (int x = 0; x < W; ++x) {
    ent += share[x].ent[lane];
    homog += share[x].homog[lane];
  }
  s = {0, 0, 0, 0, 0, 0};
  if (lane < (uint32_t)W) {
    const unsigned long long* v = share[lane].ints;
    s = {v[0], v[1], v[2], v[3], v[4], v[5]};
  }
  s = {wave_sum(s.si), wave_sum(s.sii), wave_sum(s.sij), wave_sum(s.sj), wave_sum(s.sjj), wave_sum(s.sq)};
  ent = wave_sum(ent);
  homog = wave_sum(homog);
  if (lane == 0) features_store(T, s, ent, homog, o);
}

}  // namespace
}  // namespace glcm
