// One image of N <= 16 levels on the matrix cores (glcm_onehot_device.h).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdint>

#include "glcm_onehot_device.h"

namespace glcm {
namespace {

template <typename Pix, int R, int DIST>
__global__ __launch_bounds__(onehot_threads(R), R == 4 ? 3 : 4) void k_vote_onehot(OnehotArgs a) {
  constexpr int kThreads = onehot_threads(R), kWaves = kThreads / 64, S = onehot_slots(R);
  __shared__ __attribute__((aligned(16))) uint32_t tiles[kWaves][kOnehotWaveDwords];
  __shared__ uint32_t hist[S * 256];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (uint32_t w = threadIdx.x; w < (uint32_t)S * 256u; w += kThreads) hist[w] = 0u;
  f4 acc[S];
#pragma unroll
  for (int s = 0; s < S; ++s) acc[s] = f4{0.f, 0.f, 0.f, 0.f};
  onehot_walk<Pix, R, DIST>(a, a.img, a.stride, a.W, a.H, a.y_begin, a.y_end, a.windows, a.h, a.tasks,
                            (int)blockIdx.x * kWaves + wave, (int)gridDim.x * kWaves, tiles[wave], acc);
  __syncthreads();
  onehot_collect<R, DIST>(hist, acc);
  __syncthreads();
  const uint32_t N = a.q.nlev, NN = N * N;
  uint32_t xcc = 0;
  if (a.xbuf) asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(xcc));
  uint32_t* xs = a.xbuf + (size_t)(xcc & (kXcdSlots - 1u)) * a.words_total;
  for (int k = 0; k < a.K; ++k) {
    const uint32_t* P = hist + 256u * (uint32_t)a.slot[k];
    const bool tr = (a.tmask >> k) & 1ull;
    const uint32_t w = threadIdx.x & 255u, i = w >> 4, j = w & 15u;
    if (threadIdx.x < 256u && i < N && j < N) {
      const uint32_t c = tr ? P[16u * j + i] : P[w];
      if (a.xbuf) {
        if (c) __hip_atomic_fetch_add(xs + (uint32_t)k * NN + i * N + j, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      } else {
        a.out[(uint32_t)k * NN + i * N + j] = c;
      }
    }
  }
}

template <typename Pix, int R, int DIST>
hipError_t launch_r(const OnehotArgs& a, int groups, hipStream_t stream, const LaunchTiming& tm) {
  hipExtLaunchKernelGGL((k_vote_onehot<Pix, R, DIST>), dim3((unsigned)groups), dim3(onehot_threads(R)), 0, stream,
                        tm.start, tm.stop, 0u, a);
  return hipGetLastError();
}

template <typename Pix>
hipError_t launch_t(const OnehotArgs& a, int dist, int groups, hipStream_t stream, const LaunchTiming& tm) {
  switch (dist) {
    case 1: return launch_r<Pix, 1, 1>(a, groups, stream, tm);
    case 2: return launch_r<Pix, 2, 2>(a, groups, stream, tm);
    case 3: return launch_r<Pix, 2, 3>(a, groups, stream, tm);
    case 4: return launch_r<Pix, 4, 4>(a, groups, stream, tm);
    case 5: return launch_r<Pix, 4, 5>(a, groups, stream, tm);
    case 6: return launch_r<Pix, 4, 6>(a, groups, stream, tm);
    case 7: return launch_r<Pix, 4, 7>(a, groups, stream, tm);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_vote_onehot(const OnehotArgs& a, int dtype_bytes, int dist, int groups, hipStream_t stream,
                              const LaunchTiming& tm) {
  return dtype_bytes == 1 ? launch_t<uint8_t>(a, dist, groups, stream, tm)
                          : launch_t<uint16_t>(a, dist, groups, stream, tm);
}

}  // namespace glcm
