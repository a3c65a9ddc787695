// Stands in front of the library's HIP calls and training launches, so that
// xtm_mlp_train runs without a device: memory is the host's, and the launch of
// step FAIL_AT (from the environment, counted from 0) reports an error.
#include <hip/hip_runtime_api.h>
#include <hip/hip_vector_types.h>

#include <cstdlib>
#include <cstring>

extern "C" {
size_t stub_allocated = 0;  // bytes in all
hipError_t hipMalloc(void** p, size_t n) {
  stub_allocated += n;
  *p = std::malloc(n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind) {
  std::memcpy(to, from, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(to, from, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
}

namespace xtm {
hipError_t launch_adam_bias(double2* bias, int32_t first_step, int64_t n, hipStream_t) {
  for (int64_t i = 0; i < n; ++i) bias[i].x = (double)(first_step + i);
  return hipSuccess;
}
hipError_t launch_mlp_train_step(float*, float*, float*, const float*, const float*, const float*,
                                 const int32_t*, int64_t, float, const double2* bias, float,
                                 float*, float*, hipStream_t) {
  static int made = 0;
  if (bias->x != (double)(8 + made)) return hipErrorInvalidValue;  // step 8 is the first
  return made++ == std::atoi(std::getenv("FAIL_AT")) ? hipErrorUnknown : hipSuccess;
}
}  // namespace xtm
