// The library on the CPU over stand-ins for the HIP calls it makes here: memory
// is the host's, launches do nothing, and allocations above a limit fail.  A
// plan whose level-slice partials cannot be had is created all the same and
// counts with the kernel that needs none.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "glcm.h"

static size_t limit = SIZE_MAX;
static int refused, mallocs, launches;
static hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
static struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} config;

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024 : (a == hipDeviceAttributeMultiprocessorCount ? 256 : 0);
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (n > limit) return ++refused, hipErrorOutOfMemory;
  ++mallocs;
  *p = std::calloc(1, n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { return *s = capture, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = (hipEvent_t)&limit, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* t, const void* p) {
  *t = hipPointerAttribute_t{};
  t->type = hipMemoryTypeDevice;
  t->devicePointer = const_cast<void*>(p);
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return ++launches, hipSuccess; }
hipError_t hipExtLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t, hipEvent_t, hipEvent_t, int) {
  return ++launches, hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) {
  config = {g, b, l, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, hipStream_t* s) {
  *g = config.grid, *b = config.block, *l = config.lds, *s = config.stream;
  return hipSuccess;
}
}

static int fails = 0;
#define CHECK(c)                                              \
  do {                                                        \
    if (!(c) && ++fails < 20) std::printf("FAIL %s (line %d)\n", #c, __LINE__); \
  } while (0)

int main() {
  const glcm_offset_t offs[2] = {{1, 0}, {-1, 1}};
  constexpr int W = 700, H = 500, N = 256;
  std::vector<uint8_t> img(W * H);
  std::vector<uint32_t> out(2 * N * N);
  glcm_plan_t plan = nullptr;
  auto count = [&](int lo) {
    return glcm_compute(plan, img.data(), W, H, W, GLCM_U8, N, (uint32_t)lo, 255, offs, 2, out.data(), nullptr);
  };

  // no memory for the partials: the plan exists, its calls work
  limit = 20u << 20;  // the accumulation slices take 8 MiB, the partials twice as much as this
  CHECK(glcm_plan_create(&plan, GLCM_U8, N, 2, offs, 4096, 4096, 0) == GLCM_OK && plan);
  if (plan) {
    size_t bare = 0, held = 0;
    CHECK(refused == 1 && mallocs > 0);
    CHECK(glcm_plan_workspace(plan, &bare) == GLCM_OK && bare <= limit);
    launches = 0;
    CHECK(count(0) == GLCM_OK && launches == 2);
    // not asked for while the stream is captured
    limit = SIZE_MAX;
    capture = hipStreamCaptureStatusActive;
    mallocs = launches = 0;
    CHECK(count(0) == GLCM_OK && mallocs == 0 && launches == 2);
    // had as soon as there is memory, and not again
    capture = hipStreamCaptureStatusNone;
    for (int lo = 0; lo < 256; lo += 15) CHECK(count(lo) == GLCM_OK && mallocs == 1);
    CHECK(glcm_plan_workspace(plan, &held) == GLCM_OK && held > bare);
    CHECK(glcm_plan_destroy(plan) == GLCM_OK);
  }
  std::printf(fails ? "%d failures\n" : "ok\n", fails);
  return fails != 0;
}
