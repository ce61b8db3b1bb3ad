// Haralick statistics kernels: a wavefront or a workgroup per GLCM (Section I;
// the five statistics and their precision are described in glcm_features.h).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "glcm_features.h"
#include "glcm_internal.h"

namespace glcm {
namespace {

// 33 <= N <= 160, few GLCMs: a workgroup of W wavefronts each.
template <int W>
__global__ __launch_bounds__(64 * W) void k_features(const uint32_t* glcm, int N, float* out) {
  __shared__ FeatureShare share[W];
  glcm_features_wg<W>(glcm + (size_t)blockIdx.x * (uint32_t)N * (uint32_t)N, (uint32_t)N,
                      out + (size_t)blockIdx.x * 5, share);
}

// N > 160.
__global__ __launch_bounds__(1024) void k_features_large(const uint32_t* glcm, int N, float* out) {
  __shared__ FeatureLargeShare share[16];
  glcm_features_large<16>(glcm + (size_t)blockIdx.x * (uint32_t)N * (uint32_t)N, (uint32_t)N,
                          out + (size_t)blockIdx.x * 5, share);
}

// One wavefront per GLCM of 16 < N <= 160, four per workgroup.
template <int W>
__global__ __launch_bounds__(256) void k_features_many(const uint32_t* glcm, int K, int N, float* out) {
  const int k = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (k < K)
    glcm_features_many<W>(glcm + (size_t)k * (uint32_t)N * (uint32_t)N, (uint32_t)N, out + (size_t)k * 5, lane_id());
}

// N <= 16: a wavefront per GLCM, or (FOUR) per four of them.
template <bool FOUR>
__global__ __launch_bounds__(256) void k_features_16(const uint32_t* glcm, int K, int N, float* out) {
  const int k = (blockIdx.x * 4 + (int)(threadIdx.x >> 6)) * (FOUR ? 4 : 1);
  if (k < K)
    glcm_features_16<false>(glcm + (size_t)k * (uint32_t)N * (uint32_t)N, (uint32_t)N, FOUR ? min(K - k, 4) : 1, !FOUR,
                            out + (size_t)k * 5, lane_id());
}

}  // namespace

// A workgroup of W wavefronts shortens one GLCM's statistics, a wavefront each
// keeps more GLCMs going; the lines lie where the chip is full.  Measured on
// MI355X, us a call, workgroups; wavefronts: N = 33 K = 1024 8.5; 9.0, 2048 12.1;
// 10.2, 16384 66; 46.  N = 48 K = 2048 16.2; 15.6.  N = 49 K = 512 11.2; 13.2, 1024
// 19.4; 13.4.  N = 64 K = 512 11.6; 18.0, 1024 20.3; 19.2, 8192 154; 83.  N = 128 K =
// 2048 103; 120.  N = 16, a GLCM; four a wavefront: K = 4096 8.5; 8.9, 16384 14.0;
// 10.6.
hipError_t launch_features(const uint32_t* glcm, int K, int N, float* out, hipStream_t stream) {
  const dim3 four((K + 3) / 4), block(256);
  const int W = features_waves(N);
  if (N > kFeaturesLinear) {
    hipLaunchKernelGGL(k_features_large, dim3(K), dim3(1024), 0, stream, glcm, N, out);
  } else if (N <= kFeatures16) {
    if (K >= 8192)
      hipLaunchKernelGGL(k_features_16<true>, dim3((K + 15) / 16), block, 0, stream, glcm, K, N, out);
    else
      hipLaunchKernelGGL(k_features_16<false>, four, block, 0, stream, glcm, K, N, out);
  } else if (W == 1) {
    hipLaunchKernelGGL(k_features_many<1>, four, block, 0, stream, glcm, K, N, out);
  } else if (W == 4) {
    if (K >= 2048)
      hipLaunchKernelGGL(k_features_many<4>, four, block, 0, stream, glcm, K, N, out);
    else
      hipLaunchKernelGGL(k_features<4>, dim3(K), dim3(256), 0, stream, glcm, N, out);
  } else {
    if (K >= N * N / 4)
      hipLaunchKernelGGL(k_features_many<16>, four, block, 0, stream, glcm, K, N, out);
    else
      hipLaunchKernelGGL(k_features<16>, dim3(K), dim3(1024), 0, stream, glcm, N, out);
  }
  return hipGetLastError();
}

}  // namespace glcm
