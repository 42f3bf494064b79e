// Device code shared by the kernels: scans and reductions over the lanes of a wave.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dapq {
namespace {

// Scans and reductions over the 64 lanes of a wave with data-parallel-primitive moves (a register-to-register
// move between lanes costs a few clocks; a shuffle goes through the LDS crossbar and takes over a hundred, and a
// scan is six of them in a chain).  A wave is four rows of 16 lanes: shifts by 1, 2, 4, 8 scan inside the rows
// (lanes without a source take the identity), then lane 15 of a row is handed to the whole next row (rows 1 and 3),
// then lane 31 to rows 2 and 3.
enum : int {
  kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118,
  kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143
};
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_take(uint32_t identity, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, CTRL, ROW_MASK, 0xf, false);
}
struct OpAdd {
  static constexpr uint32_t identity = 0u;
  __device__ __forceinline__ static uint32_t apply(uint32_t a, uint32_t b) { return a + b; }
};
struct OpMin {
  static constexpr uint32_t identity = 0xFFFFFFFFu;
  __device__ __forceinline__ static uint32_t apply(uint32_t a, uint32_t b) { return a < b ? a : b; }
};
struct OpMax {
  static constexpr uint32_t identity = 0u;
  __device__ __forceinline__ static uint32_t apply(uint32_t a, uint32_t b) { return a > b ? a : b; }
};
// inclusive scan in lane order: lane l gets op(v[0], ..., v[l])
template <class Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v = Op::apply(v, dpp_take<kDppRowShr1, 0xf>(Op::identity, v));
  v = Op::apply(v, dpp_take<kDppRowShr2, 0xf>(Op::identity, v));
  v = Op::apply(v, dpp_take<kDppRowShr4, 0xf>(Op::identity, v));
  v = Op::apply(v, dpp_take<kDppRowShr8, 0xf>(Op::identity, v));
  v = Op::apply(v, dpp_take<kDppRowBcast15, 0xa>(Op::identity, v));
  v = Op::apply(v, dpp_take<kDppRowBcast31, 0xc>(Op::identity, v));
  return v;
}
// the reduction over all lanes, in every lane
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan<Op>(v), 63);
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return wave_reduce<OpAdd>(v); }

}  // namespace
}  // namespace dapq
