// Five Haralick statistics of one GLCM by a wavefront or a workgroup: shared by
// the features kernel and the batch kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "glcm_wave.h"

namespace glcm {
namespace {

// ---------------------------------------------------------------------------
// Five Haralick statistics of one GLCM.  Exact integer sums for the contrast
// and the correlation moments; fp32 terms, added in fp64, for energy, entropy
// and homogeneity; fp64 (from exact 128-bit integers) for the correlation.
//
// The bins are walked by W wavefronts.  A wavefront takes R = 64 / N whole rows
// at a time (64 columns of one row when N > 64) and a lane keeps its column, so
// sum c, sum i c and sum i^2 c per column are all the integers a bin adds to;
// the rest follows once at the end (sum j c = j sum c and so on, and
// sum (i - j)^2 c = sum i^2 c + sum j^2 c - 2 sum i j c).  A lane's fp64 sums of
// the W wavefronts are added in order and the lanes then meet by exchanges, so
// the result depends on W, not on which wavefronts did the work: one wavefront
// that plays all W (glcm_features_wave) gives the same bits as W of them
// (glcm_features_wg).  Bound: latency of the loads and of the one reduction up
// to N = 128, the logarithms of the one CU that holds the matrix above.
// Measured on MI355X, 7 matrices of N = 64: 11.5 us with 4 wavefronts that each
// reduce their own sums, 7.1 with 16 and one reduction; 12 of N = 256: 36.8 and
// 35.8 (32.5 with the quotients below).  Up to N = 48 four wavefronts leave a lane at most 12 bins.
// ---------------------------------------------------------------------------
constexpr int features_waves(int N) { return N <= 32 ? 1 : (N <= 48 ? 4 : 16); }

struct FeatureSums {
  unsigned long long si, sii, sij, sj, sjj;
  double energy, ent, homog;
};

// The five statistics from the exact integer sums and the fp32 sums.
__device__ __forceinline__ void features_store(unsigned long long T, const FeatureSums& s, float* o) {
  using i128 = __int128;
  const i128 tT = (i128)T;
  const i128 vi = (i128)s.sii * tT - (i128)s.si * (i128)s.si;  // T^2 var_i
  const i128 vj = (i128)s.sjj * tT - (i128)s.sj * (i128)s.sj;  // T^2 var_j
  const i128 cv = (i128)s.sij * tT - (i128)s.si * (i128)s.sj;  // T^2 cov
  const unsigned long long sc = s.sii + s.sjj - 2ull * s.sij;
  double corr = 1.0;
  if (vi != 0 && vj != 0) corr = (double)cv / sqrt((double)vi * (double)vj);
  o[0] = (float)((double)sc / (double)T);
  o[1] = (float)s.energy;
  o[2] = (float)s.ent;
  o[3] = (float)s.homog;
  o[4] = (float)corr;
}

// p / (1 + d^2), rounded like the division (the quotient by the reciprocal,
// corrected by its exact remainder; no operand is denormal).  Half the
// instructions of a division: 12 matrices of N = 256 35.8 to 32.5 us.
__device__ __forceinline__ float homog_term(float p, uint32_t d) {
  const float df = (float)d, y = fmaf(df, df, 1.0f), r = __builtin_amdgcn_rcpf(y), q = p * r;
  return fmaf(fmaf(-q, y, p), r, q);
}

// Total of the matrix over one wavefront's share of the words (w of W).
__device__ __forceinline__ unsigned long long features_total(const uint32_t* P, uint32_t NN, uint32_t w, uint32_t W) {
  unsigned long long T = 0;
#pragma unroll 8
  for (uint32_t r = 64u * w + (threadIdx.x & 63u); r < NN; r += 64u * W) T += P[r];
  return wave_sum(T);
}

// This lane's share of the sums of wavefront w of W (T below 2^32).
__device__ __forceinline__ FeatureSums features_sums(const uint32_t* P, uint32_t N, unsigned long long T, float invT,
                                                     uint32_t w, uint32_t W) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t R = N <= 64u ? 64u / N : 1u;
  const uint32_t i0 = N <= 64u ? lane / N : 0u, jl = N <= 64u ? lane - i0 * N : lane;
  FeatureSums s = {0, 0, 0, 0, 0, 0.0, 0.0, 0.0};
  constexpr uint32_t U = 4;  // loads in flight
  const uint32_t half = (uint32_t)(T >> 1);
  for (uint32_t j = jl; j - jl < N; j += 64u) {  // (the same trip count on every lane)
    const bool live = i0 < R && j < N;
    uint32_t col = 0;  // (sums of a column stay below T)
    unsigned long long ci = 0, cii = 0;
    for (uint32_t t = w * R; t < N; t += U * W * R) {
      uint32_t c[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t i = t + u * W * R + i0;
        c[u] = live && i < N ? P[(size_t)i * N + j] : 0u;
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        if (c[u] == 0u) continue;
        const uint32_t i = t + u * W * R + i0;
        col += c[u];
        ci += (unsigned long long)i * c[u];
        cii += (unsigned long long)(i * i) * c[u];
        const float p = (float)c[u] * invT;
        s.energy += (double)(p * p);
        // -p ln p; for p > 1/2 use log1p of the exact complement to keep accuracy
        const float lp = (c[u] > half) ? log1pf(-(float)(T - c[u]) * invT) : logf(p);
        s.ent -= (double)(p * lp);
        const uint32_t d = i > j ? i - j : j - i;
        s.homog += (double)homog_term(p, d);
      }
    }
    s.si += ci;
    s.sii += cii;
    s.sij += (unsigned long long)j * ci;
    s.sj += (unsigned long long)j * col;
    s.sjj += (unsigned long long)(j * j) * col;
  }
  return s;
}

// The lanes' shares, on every lane.
__device__ __forceinline__ FeatureSums features_reduce(const FeatureSums& s) {
  return {wave_sum(s.si), wave_sum(s.sii), wave_sum(s.sij), wave_sum(s.sj), wave_sum(s.sjj),
          wave_sum(s.energy), wave_sum(s.ent), wave_sum(s.homog)};
}

struct FeatureShare {  // scratch of a workgroup of W wavefronts
  unsigned long long total, ints[5];
  double energy[64], ent[64], homog[64];  // a lane's
};

// By a workgroup of W wavefronts (W = features_waves(N)): two barriers.  Every
// thread of the workgroup must call it.
template <int W>
__device__ __forceinline__ void glcm_features_wg(const uint32_t* P, uint32_t N, float* o, FeatureShare* share) {
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  unsigned long long T = features_total(P, N * N, w, W);
  if (lane == 0) share[w].total = T;
  __syncthreads();
  T = 0;
#pragma unroll
  for (int x = 0; x < W; ++x) T += share[x].total;
  if (T == 0 || T > 0xffffffffull) {
    if (threadIdx.x < 5) o[threadIdx.x] = T == 0 ? 0.0f : __builtin_nanf("");
    return;
  }
  FeatureSums s = features_sums(P, N, T, 1.0f / (float)T, w, W);
  const unsigned long long ints[5] = {wave_sum(s.si), wave_sum(s.sii), wave_sum(s.sij), wave_sum(s.sj), wave_sum(s.sjj)};
  if (lane == 0) {
#pragma unroll
    for (int q = 0; q < 5; ++q) share[w].ints[q] = ints[q];
  }
  share[w].energy[lane] = s.energy;
  share[w].ent[lane] = s.ent;
  share[w].homog[lane] = s.homog;
  __syncthreads();
  if (w != 0) return;
  s = {0, 0, 0, 0, 0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int x = 0; x < W; ++x) {
    s.energy += share[x].energy[lane];
    s.ent += share[x].ent[lane];
    s.homog += share[x].homog[lane];
  }
  if (lane < (uint32_t)W) {
    s.si = share[lane].ints[0];
    s.sii = share[lane].ints[1];
    s.sij = share[lane].ints[2];
    s.sj = share[lane].ints[3];
    s.sjj = share[lane].ints[4];
  }
  s = features_reduce(s);
  if (lane == 0) features_store(T, s, o);
}

// N <= 16, by one wavefront: each group of 16 lanes keeps a column a lane.
// wide: the GLCM at P, a fourth of the rows per group; else up to four GLCMs,
// P's and the ones that follow (count in all), a group each.  o: the statistics,
// likewise.  The sums of four rows are added in the same order either way, so
// both give the same bits.  Every lane must call it.
constexpr int kFeatures16 = 16;
__device__ __forceinline__ void glcm_features_16(const uint32_t* P, uint32_t N, int count, bool wide, float* o) {
  constexpr uint32_t U = kFeatures16 / 4;  // rows of a fourth
  const uint32_t lane = threadIdx.x & 63u, q = lane >> 4, j = lane & 15u;
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
  const float invT = 1.0f / (float)T;
  const uint32_t half = (uint32_t)(T >> 1);
  uint32_t col = 0;
  unsigned long long ci = 0, cii = 0;
  double energy = 0.0, ent = 0.0, homog = 0.0;     // rows 0 .. 7 (or the lane's fourth)
  double energy1 = 0.0, ent1 = 0.0, homog1 = 0.0;  // rows 8 .. 15
  for (uint32_t i = begin; i < end; i += U) {
    uint32_t c[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) c[u] = live && !empty && i + u < N ? P[(i + u) * N + j] : 0u;
    double fe = 0.0, fn = 0.0, fh = 0.0;
    uint32_t r = i;
#pragma unroll 1
    for (; r < i + U; ++r) {  // (not unrolled: short code, for the instruction cache)
      const uint32_t cr = c[0];
      c[0] = c[1];
      c[1] = c[2];
      c[2] = c[3];
      if (cr == 0u) continue;
      col += cr;
      ci += (unsigned long long)r * cr;
      cii += (unsigned long long)(r * r) * cr;
      const float p = (float)cr * invT;
      fe += (double)(p * p);
      const float lp = (cr > half) ? log1pf(-(float)(T - cr) * invT) : logf(p);
      fn -= (double)(p * lp);
      const uint32_t d = r > j ? r - j : j - r;
      fh += (double)homog_term(p, d);
    }
    const bool upper = !wide && i >= 2u * U;
    energy += upper ? 0.0 : fe;
    ent += upper ? 0.0 : fn;
    homog += upper ? 0.0 : fh;
    energy1 += upper ? fe : 0.0;
    ent1 += upper ? fn : 0.0;
    homog1 += upper ? fh : 0.0;
  }
  FeatureSums s;
  if (wide) {  // the four fourths
    energy = sum_xor16(energy);
    ent = sum_xor16(ent);
    homog = sum_xor16(homog);
    energy1 = __shfl_xor(energy, 32);
    ent1 = __shfl_xor(ent, 32);
    homog1 = __shfl_xor(homog, 32);
    col = (uint32_t)__shfl_xor((int)col, 16) + col;
    col = (uint32_t)__shfl_xor((int)col, 32) + col;
    ci = sum_xor32(sum_xor16((uint64_t)ci));
    cii = sum_xor32(sum_xor16((uint64_t)cii));
  }
  s.energy = row16_sum(energy + energy1);
  s.ent = row16_sum(ent + ent1);
  s.homog = row16_sum(homog + homog1);
  s.si = row16_sum(ci);
  s.sii = row16_sum(cii);
  s.sij = row16_sum((unsigned long long)j * ci);
  s.sj = row16_sum((unsigned long long)j * col);
  s.sjj = row16_sum((unsigned long long)(j * j) * col);
  if ((int)mine >= count || (wide && q != 0u)) return;
  if (empty) {
    if (j < 5) o[5u * mine + j] = T == 0 ? 0.0f : __builtin_nanf("");
  } else if (j == 0) {
    features_store(T, s, o + 5u * mine);
  }
}

// N > 16: by one wavefront that plays all of features_waves(N), with no LDS and
// no barrier.  Every lane must call it; lane 0 writes o.
__device__ __forceinline__ void glcm_features_wave(const uint32_t* P, uint32_t N, float* o) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t W = (uint32_t)features_waves((int)N);
  const unsigned long long T = features_total(P, N * N, 0, 1);
  if (T == 0 || T > 0xffffffffull) {
    if (lane < 5) o[lane] = T == 0 ? 0.0f : __builtin_nanf("");
    return;
  }
  const float invT = 1.0f / (float)T;
  FeatureSums a = {0, 0, 0, 0, 0, 0.0, 0.0, 0.0};
  for (uint32_t w = 0; w < W; ++w) {
    const FeatureSums s = features_sums(P, N, T, invT, w, W);
    a = {a.si + s.si, a.sii + s.sii, a.sij + s.sij, a.sj + s.sj, a.sjj + s.sjj,
         a.energy + s.energy, a.ent + s.ent, a.homog + s.homog};
  }
  a = features_reduce(a);
  if (lane == 0) features_store(T, a, o);
}

// One GLCM's statistics by one wavefront.
__device__ __forceinline__ void glcm_features_any(const uint32_t* P, uint32_t N, float* o) {
  if (N <= kFeatures16)
    glcm_features_16(P, N, 1, true, o);
  else
    glcm_features_wave(P, N, o);
}

}  // namespace
}  // namespace glcm
