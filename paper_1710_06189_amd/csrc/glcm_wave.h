// Sums over the lanes of a wavefront by DPP lane moves and half exchanges (no
// LDS round trips).  Included by the .hip files only.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace glcm {
namespace {

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_move(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, true);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_move(unsigned long long v) {
  return (unsigned long long)dpp_move<CTRL, ROWS>((uint32_t)v) |
         ((unsigned long long)dpp_move<CTRL, ROWS>((uint32_t)(v >> 32)) << 32);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_move(float v) {
  return __uint_as_float(dpp_move<CTRL, ROWS>(__float_as_uint(v)));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double v) {
  return __longlong_as_double((long long)dpp_move<CTRL, ROWS>((unsigned long long)__double_as_longlong(v)));
}
__device__ __forceinline__ uint32_t lane63(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }
__device__ __forceinline__ unsigned long long lane63(unsigned long long v) {
  return (unsigned long long)lane63((uint32_t)v) | ((unsigned long long)lane63((uint32_t)(v >> 32)) << 32);
}
__device__ __forceinline__ float lane63(float v) { return __uint_as_float(lane63(__float_as_uint(v))); }
__device__ __forceinline__ double lane63(double v) {
  return __longlong_as_double((long long)lane63((unsigned long long)__double_as_longlong(v)));
}

// Wavefront sum: prefix sums within each row of 16 lanes (row_shr 1, 2, 4, 8),
// then lane 15 of rows 0 and 2 is added into rows 1 and 3 (row_bcast:15) and
// lane 31 into rows 2 and 3 (row_bcast:31), leaving the total in lane 63,
// which is returned to all (a scalar: the same bits on every lane).
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
  v += dpp_move<0x111, 0xf>(v);  // row_shr:1
  v += dpp_move<0x112, 0xf>(v);  // row_shr:2
  v += dpp_move<0x114, 0xf>(v);  // row_shr:4
  v += dpp_move<0x118, 0xf>(v);  // row_shr:8
  v += dpp_move<0x142, 0xa>(v);  // row_bcast:15 into rows 1, 3
  v += dpp_move<0x143, 0xc>(v);  // row_bcast:31 into rows 2, 3
  return lane63(v);
}

// Sum over the 16 lanes of a DPP row, on all of them (rotations by 8, 4, 2, 1).
template <typename T>
__device__ __forceinline__ T row16_sum(T v) {
  v += dpp_move<0x128, 0xf>(v);
  v += dpp_move<0x124, 0xf>(v);
  v += dpp_move<0x122, 0xf>(v);
  v += dpp_move<0x121, 0xf>(v);
  return v;
}

// v + (lane ^ 16)'s v, v + (lane ^ 32)'s v.
__device__ __forceinline__ double sum_xor16(double v) { return v + __shfl_xor(v, 16); }
__device__ __forceinline__ double sum_xor32(double v) { return v + __shfl_xor(v, 32); }
__device__ __forceinline__ uint64_t sum_xor16(uint64_t v) { return v + (uint64_t)__shfl_xor((unsigned long long)v, 16); }
__device__ __forceinline__ uint64_t sum_xor32(uint64_t v) { return v + (uint64_t)__shfl_xor((unsigned long long)v, 32); }

// Orders a wavefront's LDS writes before its lanes read each other's words
// (and its reads before later writes).
__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Lane Q of each group of four, on all four (quad_perm:[Q,Q,Q,Q]).
template <int Q>
__device__ __forceinline__ double quad_bcast(double v) {
  return dpp_move<Q * 0x55, 0xf>(v);
}

// a b - c d with about one rounding (Kahan): the products' rounding errors are
// taken back exactly.  (Not contracted: p - q has to be the rounded products'.)
__device__ __forceinline__ double difference_of_products(double a, double b, double c, double d) {
#pragma clang fp contract(off)
  const double p = a * b, q = c * d;
  return (p - q) + (fma(a, b, -p) - fma(c, d, -q));
}

}  // namespace
}  // namespace glcm
