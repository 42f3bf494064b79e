// What a kernel of a few microseconds does before it can ask for its first data: its arguments, and which part of the work it has.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dapq {
namespace {

// The arguments of a kernel lie in memory that the first load of each 64-byte line reaches in about a microsecond, and the
// compiler loads them where they are used, one wait after the other.
// Brings the lines of a kernel's first BYTES of arguments into the scalar cache with one wait, before anything is asked of them.
// To be called first in a kernel that lasts a few microseconds.
template <int BYTES>
__device__ __forceinline__ void touch_args() {
  const __attribute__((address_space(4))) uint32_t* args =
      (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int kLines = (BYTES + 63) / 64;
  static_assert(kLines >= 1 && kLines <= 6, "arguments of the kernels here");
  const uint32_t a = args[0], b = args[kLines > 1 ? 16 : 0], c = args[kLines > 2 ? 32 : 0], d = args[kLines > 3 ? 48 : 0],
                 e = args[kLines > 4 ? 64 : 0], f = args[kLines > 5 ? 80 : 0];
  asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d), "s"(e), "s"(f));
}

// a / b for inv = 1.0f / b (rounded to nearest), 0 <= a < kQuotientMax, b >= 1: the product is off by less than 2^-2 / b, and
// (a + 1/2) / b lies at least half of 1 / b away from a whole number.  A division by a value that the compiler does not know is
// some thirty instructions in a row, one of 64 bits a hundred or more; this is four.
constexpr int kQuotientMax = 1 << 21;
__device__ __forceinline__ int quotient(int a, float inv) { return (int)(((float)a + 0.5f) * inv); }
// The same for values that are the same in all lanes, of any size.
__device__ __forceinline__ int uniform_quotient(int a, int b, float inv) {
  return __builtin_amdgcn_readfirstlane(a < kQuotientMax ? quotient(a, inv) : a / b);
}

}  // namespace
}  // namespace dapq
