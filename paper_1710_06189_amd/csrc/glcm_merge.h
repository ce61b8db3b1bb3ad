// Shared by the LDS counting kernels: the merge of their copies, the order of
// their workgroups and their launch.  Included by the .hip files only.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdint>

#include "glcm_device.h"
#include "glcm_internal.h"

namespace glcm {
namespace {

// ---------------------------------------------------------------------------
// Merge of the LDS copies (the final sum of Section II.A), in two steps that
// need no synchronisation between workgroups inside a kernel:
//
//  * merge = per-XCD accumulation: every workgroup adds its non-zero counts to
//    the accumulation slice of the XCD it runs on (hardware register XCC_ID),
//    with workgroup-scope atomics, which execute in that XCD's L2 (all CUs of
//    an XCD share it, and no other XCD touches the slice).  The kernel
//    boundary writes the L2s back; k_finish sums the slices into `out` and
//    clears them for the next launch.
//  * merge = band partials: every workgroup stores its counts to its own row
//    of a partial buffer and k_reduce sums the rows.
//
// Word w of the partition sits at dword w * R of the LDS (R copies).
// ---------------------------------------------------------------------------
// The accumulation slice of the XCD this wavefront runs on.
__device__ __forceinline__ uint32_t* xcd_slice(const VoteArgs& a) {
  uint32_t xcc;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(xcc));
  return a.xbuf + (size_t)(xcc & (kXcdSlots - 1u)) * a.words_total;
}

__device__ void store_partial(const VoteArgs& a, const uint32_t* lds, uint32_t pbase, uint32_t pwords, int region) {
  __syncthreads();
  const uint32_t R = 1u << a.log2R;
  uint32_t* dst = a.xbuf ? xcd_slice(a) + pbase : a.partials + (size_t)region * a.words_total + pbase;
  for (uint32_t w = threadIdx.x; w < pwords; w += blockDim.x) {
    const uint32_t* c = lds + (w << a.log2R);
    uint32_t s = 0;
    if (R >= 4) {
      for (uint32_t d = 0; d < R; d += 4) {
        const uint4 v = *(const uint4*)(c + d);
        s += (v.x + v.y) + (v.z + v.w);
      }
    } else {
      for (uint32_t d = 0; d < R; ++d) s += c[d];
    }
    if (!a.xbuf) dst[w] = s;
    else if (s) __hip_atomic_fetch_add(dst + w, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// Workgroup -> (band, partition).  Workgroups go to the XCDs round-robin
// (workgroup b runs on XCD b mod 8), and every partition of a band reads the
// band's rows: keeping the partitions of one band on one XCD lets its L2
// serve the second read instead of HBM.  Workgroup b = 8 s + x takes
// partition s mod P of band 8 (s / P) + x for the first 8 floor(nregions / 8)
// bands; the remaining bands take the plain order (a bijection either way).
constexpr int kXcds = 8;
__device__ __forceinline__ int2 band_of_block(int b, int P, int nregions) {
  const int full = nregions / kXcds * kXcds;
  if (P > 1 && b < full * P) {
    const int x = b % kXcds, s = b / kXcds;
    return make_int2(s / P * kXcds + x, s % P);
  }
  const int r = b - full * P;
  return make_int2(full + r / P, r % P);
}

template <typename K>
hipError_t launch(K kernel, const VoteArgs& a, dim3 grid, dim3 block, size_t lds_bytes, hipStream_t stream,
                         const LaunchTiming& tm) {
  // with events, the dispatch itself stamps the kernel's start and end
  hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds_bytes, stream, tm.start, tm.stop, 0u, a);
  return hipGetLastError();
}

}  // namespace
}  // namespace glcm
