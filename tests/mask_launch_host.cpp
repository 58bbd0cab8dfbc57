// The mask kernel's launches as the library asks for them, without a GPU: stands in for the few HIP calls on the way and
// prints what reaches hipLaunchKernel (tests/test_mask_launch_host.py links it with the library's objects).
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "rf2.h"

static size_t limit_set = 0;

extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind) { std::memcpy(to, from, n); return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int value) { limit_set = (size_t)value; return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3 block, void**, size_t lds, hipStream_t) {
  std::printf("%u %zu %zu\n", block.x, lds, limit_set);
  return hipSuccess;
}
}

int main() {
  float means = 0;
  int32_t lists = 0;
  for (int d : {64, 128})
    for (int heads : {1, 300})            // at most one workgroup per compute unit, and more
      for (int columns = 16; columns <= 2048; columns += 16)
        for (int mode : {RF2_SELECT_TOPN, RF2_SELECT_CDF}) {
          rf2_config c = {};
          c.batch = 1, c.heads = heads, c.head_dim = d, c.T = c.H = 1, c.W = columns * 64, c.block = 64, c.sparsity = 0.5f;
          c.select_mode = mode, c.cdf_threshold = 0.9f;
          rf2_plan* plan = nullptr;
          limit_set = 0;
          std::printf("%d %d %d %d ", d, heads, columns, mode);
          if (rf2_plan_create(&c, &plan) != RF2_OK) return 1;
          if (rf2_predict_mask(plan, &means, &means, &lists, &lists, nullptr, nullptr, nullptr, nullptr) != RF2_OK) return 2;
          rf2_plan_destroy(plan);
        }
  return 0;
}
