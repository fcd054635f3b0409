// Kernel launches that can be made to fail, over hip_stub.cpp (test infrastructure). The status is that of the last launch,
// as HIP reported it before an error outlived the next success: a caller that reads it after several launches sees the last one's.
#include <hip/hip_runtime_api.h>

namespace {
int g_count = 0, g_fail_at = 0;
hipError_t g_last = hipSuccess;
}  // namespace

extern "C" {
void shim_reset(int fail_at) {  // the fail_at-th launch from here on fails (0: none)
  g_count = 0;
  g_fail_at = fail_at;
  g_last = hipSuccess;
}
int shim_launches(void) { return g_count; }

hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
  g_last = ++g_count == g_fail_at ? hipErrorLaunchFailure : hipSuccess;
  return g_last;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
}
