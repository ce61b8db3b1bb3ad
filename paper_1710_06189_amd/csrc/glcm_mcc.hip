// Haralick's maximal correlation coefficient (the fourteenth statistic) of K
// co-occurrence matrices, fp64 on the matrix cores.

#include <hip/hip_runtime.h>

#include "glcm_device.h"
#include "glcm_stats.h"
#include "glcm_wave.h"

namespace glcm {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kMccThreads = 256;
constexpr int kMccWaves = kMccThreads / 64;
// Squarings at most: a spectrum whose largest eigenvalue repeats never becomes
// rank one, and then the estimate's relative error is below ln(N) / 2^34.
constexpr int kMccSquarings = 34;
constexpr double kMccTol = 1e-5;

// Haralick's fourteenth statistic, the maximal correlation coefficient: the
// square root of the second largest eigenvalue of
// Q(i, j) = sum_c p(i, c) p(j, c) / (px(i) py(c)).  Q is similar to B B^T with
// B(i, c) = p(i, c) / sqrt(px(i) py(c)), whose largest singular triple is
// known: 1, sqrt(px), sqrt(py).  The kernel subtracts it,
//     D(i, c) = (p(i, c) - px(i) py(c)) / sqrt(px(i) py(c)),
// the numerator as c T - row(i) col(c) in exact integers held in doubles (one
// rounding each, no cancellation), and needs the largest eigenvalue of
// S = D D^T.  Squaring M_0 = S / tr S again and again,
//     f_j = tr(M_j^2) = |M_j|_F^2,   M_{j+1} = M_j^2 / f_j,
// gives it as tr S * prod_j f_j^(1 / 2^(j+1)); a rounding error of squaring j
// enters divided by 2^j.  With M_j's other eigenvalues summing to
// s <= (1 - f_j) the product's next factors are 1 within s^2 / 2^j, so it ends
// once 1 - f_j < 1e-5.  (M_j^2 is scaled by an approximate 1 / f_j, s_j, whose
// exact value goes into the product.)
//
// One wavefront per matrix (TB x TB tiles of 16 x 16, zero padded): lane l =
// 16 g + i holds D(16 a + i, 16 c + 4 g + v), v < 4, of every tile (a, c),
// which is both operands of S's v_mfma_f64_16x16x4; and since S is symmetric
// a result tile, lane l holding rows r(g, v) of column i, is both operands of
// the next squaring whatever r is, so no value ever moves between lanes.
//
// Bound: vector instructions (650 a matrix, 59 % of the SIMDs' cycles), then the
// products (22 of 64 cycles, 32 %), which overlap little with two wavefronts a SIMD
// that each wait for a wavefront sum between two squarings.
// Measured on MI355X, 16384 matrices of N = 16: 36 us a call (57 us
// with one logarithm per squaring and a tolerance of 1e-10); cyclic Jacobi
// rotations of S in LDS, the form before this one, took 2750 us (three
// barriers for each of fifteen rounds of five or so sweeps).
template <int TB>
__global__ __launch_bounds__(kMccThreads, TB <= 2 ? 2 : 1) void k_haralick_mcc(StatsArgs a) {
  const int N = a.N, lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int nwaves = (int)gridDim.x * kMccWaves;
  for (int k = (int)blockIdx.x * kMccWaves + (int)(threadIdx.x >> 6); k < a.K; k += nwaves) {
    const uint32_t* P = a.in + (size_t)k * (size_t)N * (size_t)N;
    d4 D[TB][TB];
    double rs[TB], cs[TB][4];  // row sums (of row 16 a + i) and column sums (of column 16 c + 4 g + v)
#pragma unroll
    for (int c = 0; c < TB; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) cs[c][v] = 0.0;
#pragma unroll
    for (int r = 0; r < TB; ++r) {
      double s = 0.0;
#pragma unroll
      for (int c = 0; c < TB; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int y = 16 * r + i, x = 16 * c + 4 * g + v;
          const double p = (y < N && x < N) ? (double)P[y * N + x] : 0.0;
          D[r][c][v] = p;
          s += p;
          cs[c][v] += p;
        }
      rs[r] = sum_xor32(sum_xor16(s));
    }
    double T = 0.0;
#pragma unroll
    for (int r = 0; r < TB; ++r) T += rs[r];
    T = row16_sum(T);
    if (T == 0.0) {  // (uniform; N = 1 has D = 0 below)
      if (lane == 0) a.out_f[k] = 0.0f;
      continue;
    }
    const double invT = 1.0 / T;
    double wr[TB], wc[TB][4];  // 1 / sqrt of the marginals, 0 where a marginal is 0
#pragma unroll
    for (int r = 0; r < TB; ++r) wr[r] = rs[r] > 0.0 ? rsqrt(rs[r]) * invT : 0.0;
#pragma unroll
    for (int c = 0; c < TB; ++c) {
#pragma unroll
      for (int v = 0; v < 4; ++v) cs[c][v] = row16_sum(cs[c][v]);
      // lane q of a quad takes column 4 g + q's square root for its group
      const int q = i & 3;
      const double c0 = cs[c][0], c1 = cs[c][1], c2 = cs[c][2], c3 = cs[c][3];
      const double own = q == 0 ? c0 : (q == 1 ? c1 : (q == 2 ? c2 : c3));
      const double w = own > 0.0 ? rsqrt(own) : 0.0;
      wc[c][0] = quad_bcast<0>(w);
      wc[c][1] = quad_bcast<1>(w);
      wc[c][2] = quad_bcast<2>(w);
      wc[c][3] = quad_bcast<3>(w);
    }
    double t0 = 0.0;
#pragma unroll
    for (int r = 0; r < TB; ++r)
#pragma unroll
      for (int c = 0; c < TB; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double prod = rs[r] * cs[c][v], perr = fma(rs[r], cs[c][v], -prod);
          const double d = (fma(D[r][c][v], T, -prod) - perr) * wr[r] * wc[c][v];
          D[r][c][v] = d;
          t0 += d * d;
        }
    t0 = wave_sum(t0);  // tr S
    if (!(t0 > 0.0)) {
      if (lane == 0) a.out_f[k] = 0.0f;
      continue;
    }
    d4 M[TB][TB];
    {
      const double scale = 1.0 / t0;
#pragma unroll
      for (int r = 0; r < TB; ++r)
#pragma unroll
        for (int c = 0; c < TB; ++c) {
          d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int m = 0; m < TB; ++m)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              acc = __builtin_amdgcn_mfma_f64_16x16x4f64(D[r][m][v], D[c][m][v], acc, 0, 0, 0);
          M[r][c] = acc * scale;
        }
    }
    double fac = 1.0;  // lane j: s_j, of the last squaring f_j
    int j = 0;
    for (;; ++j) {
      double f = 0.0;
#pragma unroll
      for (int r = 0; r < TB; ++r)
#pragma unroll
        for (int c = 0; c < TB; ++c)
#pragma unroll
          for (int v = 0; v < 4; ++v) f = fma(M[r][c][v], M[r][c][v], f);
      f = wave_sum(f);
      if (!(1.0 - f > kMccTol) || j + 1 == kMccSquarings) {  // (the same value on every lane)
        fac = lane == j ? f : fac;
        break;
      }
      const double scale = __builtin_amdgcn_rcp(f);
      fac = lane == j ? scale : fac;
      d4 Q[TB][TB];
#pragma unroll
      for (int r = 0; r < TB; ++r)
#pragma unroll
        for (int c = 0; c < TB; ++c) {
          d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int m = 0; m < TB; ++m)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              acc = __builtin_amdgcn_mfma_f64_16x16x4f64(M[m][r][v], M[m][c][v], acc, 0, 0, 0);
          Q[r][c] = acc;
        }
#pragma unroll
      for (int r = 0; r < TB; ++r)
#pragma unroll
        for (int c = 0; c < TB; ++c) M[r][c] = Q[r][c] * scale;
    }
    // ln of the product, a factor per lane (one logarithm for all of them)
    const double ln = wave_sum(ldexp(log(fac), -1 - lane) * (lane == j ? 1.0 : -1.0));
    if (lane == 0) a.out_f[k] = (float)(sqrt(t0) * exp(0.5 * ln));
  }
}

}  // namespace

hipError_t launch_haralick_mcc(const StatsArgs& a, hipStream_t stream) {
  const int want = (a.K + kMccWaves - 1) / kMccWaves;
  const dim3 grid((unsigned)(want < 4096 ? want : 4096)), block(kMccThreads);
  switch ((a.N + 15) / 16) {
    case 1: hipLaunchKernelGGL(k_haralick_mcc<1>, grid, block, 0, stream, a); break;
    case 2: hipLaunchKernelGGL(k_haralick_mcc<2>, grid, block, 0, stream, a); break;
    case 3: hipLaunchKernelGGL(k_haralick_mcc<3>, grid, block, 0, stream, a); break;
    case 4: hipLaunchKernelGGL(k_haralick_mcc<4>, grid, block, 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace glcm
