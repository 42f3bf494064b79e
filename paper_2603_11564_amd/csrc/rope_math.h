// Device code of the rotation shared by the kernels that rotate.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace dapq {
namespace {

__device__ __forceinline__ double bf16_to_f64(uint16_t b) { return (double)__uint_as_float((uint32_t)b << 16); }

// fp64 -> bf16, round to nearest even, as if in one step: the value is first brought to fp32 with rounding to odd
// (truncate toward zero, then set the last bit if anything was cut off: the cut-off part can then neither make nor
// break a tie 16 bits further up), and the 16 low bits are rounded by the hardware conversion.  The truncation is
// the ordinary (nearest) conversion stepped back by one unit when it went away from zero.
__device__ __forceinline__ uint16_t f64_to_bf16(double x) {
  const float f = (float)x;
  const double back = (double)f;
  uint32_t u = __float_as_uint(f);
  if (back != x) {  // inexact (also true for NaN, which stays NaN)
    if (fabs(back) > fabs(x)) u -= 1u;
    u |= 1u;
  }
  return __builtin_bit_cast(uint16_t, (__bf16)__uint_as_float(u));
}

// Sine and cosine of pos * theta^(-2c/d); neg_log2_theta_2_over_d = -2 log2(theta) / d.
__device__ __forceinline__ void rope_angle(int pos, int c, double neg_log2_theta_2_over_d, double* sn, double* cs) {
  const double omega = exp2((double)c * neg_log2_theta_2_over_d);  // theta^(-2c/d)
  sincos((double)pos * omega, sn, cs);
}
inline double rope_exponent(double theta, int head_dim) { return -2.0 * log2(theta) / (double)head_dim; }

}  // namespace
}  // namespace dapq
