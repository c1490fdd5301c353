// ems_math_probe.hip -- a test hook: the step's elementary functions
// evaluated on the device, element by element (the host build of ems_math.hpp
// starts from other reciprocal estimates and takes the library's roots and
// quotients, so it cannot stand for them).
#include <hip/hip_runtime.h>

#include "ems_runtime.hpp"

namespace ems {

namespace {

constexpr int kBlock = 256;

__global__ __launch_bounds__(kBlock) void k_math(uint32_t function, uint64_t n, const double* a, const double* b,
                                                 double* out) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
    const double x = a[i], y = b ? b[i] : 0.0;
    double s, c, v = 0.0;
    switch (function) {
      case EMS_MATH_LOG: v = xlog(x); break;
      case EMS_MATH_EXP: v = xexp(x); break;
      case EMS_MATH_SIN_TURN: xsincos_turn(x, &s, &c); v = s; break;
      case EMS_MATH_COS_TURN: xsincos_turn(x, &s, &c); v = c; break;
      case EMS_MATH_SQRT: v = xsqrt(x); break;
      case EMS_MATH_QUOTIENT: v = quot(x, y); break;
      case EMS_MATH_QUOTIENT_F32: v = (double)quot((float)x, (float)y); break;
    }
    out[i] = v;
  }
}

}  // namespace

hipError_t launch_math(uint32_t function, uint64_t n, const double* a, const double* b, double* out, hipStream_t s) {
  const uint64_t want = (n + kBlock - 1) / kBlock;
  const uint32_t blocks = (uint32_t)(want < 8192 ? want : 8192);
  hipLaunchKernelGGL(k_math, dim3(blocks), dim3(kBlock), 0, s, function, n, a, b, out);
  return hipGetLastError();
}

}  // namespace ems
