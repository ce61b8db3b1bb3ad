// Haralick statistics kernels: a wavefront or a workgroup per GLCM (Section I;
// the five statistics and their precision are described in glcm_features.h).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "glcm_features.h"
#include "glcm_internal.h"

namespace glcm {
namespace {

// N > 32: one workgroup of W wavefronts per GLCM.
template <int W>
__global__ __launch_bounds__(64 * W) void k_features(const uint32_t* glcm, int N, float* out) {
  __shared__ FeatureShare share[W];
  glcm_features_wg<W>(glcm + (size_t)blockIdx.x * (uint32_t)N * (uint32_t)N, (uint32_t)N,
                      out + (size_t)blockIdx.x * 5, share);
}

// N <= 32: one wavefront per GLCM, four per workgroup.
__global__ __launch_bounds__(256) void k_features_wave(const uint32_t* glcm, int K, int N, float* out) {
  const int k = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (k < K) glcm_features_any(glcm + (size_t)k * (uint32_t)N * (uint32_t)N, (uint32_t)N, out + (size_t)k * 5);
}

}  // namespace

hipError_t launch_features(const uint32_t* glcm, int K, int N, float* out, hipStream_t stream) {
  switch (features_waves(N)) {
    case 1: hipLaunchKernelGGL(k_features_wave, dim3((K + 3) / 4), dim3(256), 0, stream, glcm, K, N, out); break;
    case 4: hipLaunchKernelGGL(k_features<4>, dim3(K), dim3(256), 0, stream, glcm, N, out); break;
    default: hipLaunchKernelGGL(k_features<16>, dim3(K), dim3(1024), 0, stream, glcm, N, out); break;
  }
  return hipGetLastError();
}

}  // namespace glcm
