// Position assignment (Sec. 4.1): rotary embedding of bf16 vectors at given absolute positions.
// The pseudo queries get positions L_p .. L_p+N-1, the positions of the first N decode steps.
//
// One thread owns one (row, channel pair) and a run of heads: it evaluates the angle
// pos * theta^(-2c/d) and its sine / cosine once in fp64 and then walks its heads, so the
// transcendental work (more than ten times the work of one rotation) is shared by the heads of a
// run; runs are 8 heads long, longer (up to 64) while the launch still has thousands of waves, shorter while it has fewer
// than a thousand.
// fp64 keeps the angle exact enough at positions beyond 10^5 (an fp32 product pos * omega would be
// off by ~1e-2 rad there); the rotation is done in fp64 as well and rounded to bf16 once, which is
// what makes the result equal to a float64 evaluation bit for bit, and what the kernel's time goes
// into (fp64 multiplies and the two conversions per rotated pair).
#include <math.h>

#include "dapq_internal.h"
#include "kernel_args.h"
#include "rope_math.h"

namespace dapq {
namespace {

// half_shift: log2(head_dim / 2), or -1 if that is no power of two.  HEADS > 0: the length of the runs of a small call, whose loads are
// all in flight before the angle is evaluated (64 rows, 32 heads, 2 to a thread: 3.0 -> 2.8 us; with runs of sixteen heads that
// would cost more registers than it gives).
// STREAM: the results are stored with the non-temporal hint, so that they leave the caches while the kernel runs and are not written back in the
// midst of the key stream of the score pass that follows.  Rotation and both passes of 16 prompts of 200..2500 keys, 32 layers, 128 rows (134 MB of
// queries) 674 -> 661 us; 32 prompts of 700 keys 627 -> 619; 32 layers, 2000 keys (8.4 MB) 64.5 -> 62.2; 16 (4.2 MB) 45.0 -> 45.2; 8 (2.1 MB)
// 28.3 -> 28.6.  The rotation alone: 8.4 MB 6.2 -> 5.5 us, 67 MB 32.0 -> 27.4, 268 MB 100 -> 98.  (Loads with the hint: 95.5, but 665 for 656.)
template <int HEADS, bool STREAM>
__global__ __launch_bounds__(256) void rope_kernel(const uint16_t* x_in, uint16_t* x_out, const int32_t* __restrict__ pos,
                                                   int64_t rows, int heads, int head_dim, int64_t stride_row, int64_t stride_head,
                                                   double neg_log2_theta_2_over_d, int pairing, int heads_per_thread, int half_shift) {
  touch_args<88>();
  const int half = head_dim >> 1;
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (gid >= rows * half) return;
  const int64_t row = half_shift >= 0 ? gid >> half_shift : gid / half;
  const int c = (int)(gid - row * half);
  const int ia = pairing == 0 ? c : 2 * c;
  const int ib = pairing == 0 ? c + half : 2 * c + 1;
  const uint16_t* src = x_in + row * stride_row;
  uint16_t* dst = x_out + row * stride_row;
  double sn, cs;
  if constexpr (HEADS > 0) {
    const int hd0 = blockIdx.y * HEADS;
    const int p = pos[row];
    uint16_t ra[HEADS], rb[HEADS];
#pragma unroll
    for (int u = 0; u < HEADS; ++u) {
      const int64_t at = (int64_t)(hd0 + u < heads ? hd0 + u : heads - 1) * stride_head;
      ra[u] = src[at + ia];
      rb[u] = src[at + ib];
    }
    __builtin_amdgcn_sched_barrier(0);
    rope_angle(p, c, neg_log2_theta_2_over_d, &sn, &cs);
#pragma unroll
    for (int u = 0; u < HEADS; ++u) {
      if (hd0 + u >= heads) break;
      const double a = bf16_to_f64(ra[u]), b = bf16_to_f64(rb[u]);
      dst[(int64_t)(hd0 + u) * stride_head + ia] = f64_to_bf16(a * cs - b * sn);
      dst[(int64_t)(hd0 + u) * stride_head + ib] = f64_to_bf16(b * cs + a * sn);
    }
    return;
  }
  rope_angle(pos[row], c, neg_log2_theta_2_over_d, &sn, &cs);
  auto put = [&](int64_t at, uint16_t v) {
    if constexpr (STREAM) __builtin_nontemporal_store(v, dst + at);
    else dst[at] = v;
  };
  const int hd0 = blockIdx.y * heads_per_thread;
  const int hd1 = hd0 + heads_per_thread < heads ? hd0 + heads_per_thread : heads;
  int hd = hd0;
  for (; hd + 4 <= hd1; hd += 4) {  // four heads per trip: eight loads in flight before the first rotation
    uint16_t ra[4], rb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      ra[u] = src[(int64_t)(hd + u) * stride_head + ia];
      rb[u] = src[(int64_t)(hd + u) * stride_head + ib];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double a = bf16_to_f64(ra[u]), b = bf16_to_f64(rb[u]);
      put((int64_t)(hd + u) * stride_head + ia, f64_to_bf16(a * cs - b * sn));
      put((int64_t)(hd + u) * stride_head + ib, f64_to_bf16(b * cs + a * sn));
    }
  }
  for (; hd < hd1; ++hd) {
    const double a = bf16_to_f64(src[(int64_t)hd * stride_head + ia]);
    const double b = bf16_to_f64(src[(int64_t)hd * stride_head + ib]);
    put((int64_t)hd * stride_head + ia, f64_to_bf16(a * cs - b * sn));
    put((int64_t)hd * stride_head + ib, f64_to_bf16(b * cs + a * sn));
  }
}

// Sec. 4.1 / Sec. 5.1: which prompt token each pseudo token copies (first m, last n) and the position
// it is given (L_p + i), for every sequence of a possibly ragged batch, without a host round trip
// for the sequence lengths.
__global__ void pseudo_tokens_kernel(const int32_t* cu_seqlens, int64_t total_tokens, int batch, int first_m, int last_n,
                                     int32_t* token_idx, int32_t* positions) {
  const int n = first_m + last_n;
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= batch * n) return;
  const int b = gid / n, i = gid - b * n;
  int64_t start;
  int L;
  if (cu_seqlens == nullptr) {
    L = (int)(total_tokens / batch);
    start = (int64_t)b * L;
  } else {
    start = cu_seqlens[b];
    L = cu_seqlens[b + 1] - (int)start;
  }
  int src;
  if (i < first_m) src = i < L - 1 ? i : L - 1;
  else src = L > 0 ? (L - last_n + (i - first_m) > 0 ? L - last_n + (i - first_m) : 0) : -1;
  token_idx[gid] = src >= 0 ? (int32_t)(start + src) : -1;
  positions[gid] = L + i;
}

}  // namespace
}  // namespace dapq

using namespace dapq;

extern "C" DAPQ_API int dapq_pseudo_tokens(const dapq_shape* shape, int32_t first_m, int32_t last_n, int32_t* token_idx,
                                           int32_t* positions, void* stream) {
  int rc = check_shape(shape, false, false, false);
  if (rc != DAPQ_OK) return rc;
  DAPQ_REQUIRE(token_idx != nullptr && positions != nullptr, DAPQ_ERR_INVALID_ARG, "token_idx and positions must not be NULL");
  DAPQ_REQUIRE(first_m >= 0 && last_n >= 0 && (int64_t)first_m + last_n == shape->n_pseudo, DAPQ_ERR_INVALID_ARG,
               "first_m (%d) + last_n (%d) must equal n_pseudo (%d)", first_m, last_n, shape->n_pseudo);
  const int64_t work = (int64_t)shape->batch * shape->n_pseudo;
  DAPQ_REQUIRE(work < ((int64_t)1 << 31), DAPQ_ERR_UNSUPPORTED, "batch * n_pseudo is too large");
  hipLaunchKernelGGL(pseudo_tokens_kernel, dim3((unsigned)((work + 255) / 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), shape->cu_seqlens, shape->total_tokens, shape->batch, first_m, last_n,
                     token_idx, positions);
  DAPQ_HIP_LAUNCH_CHECK("pseudo_tokens_kernel");
  return DAPQ_OK;
}


extern "C" DAPQ_API int dapq_rope_apply(const void* x_in, void* x_out, const int32_t* pos, int64_t rows, int32_t heads,
                               int32_t head_dim, int64_t stride_row, int64_t stride_head, double theta,
                               int32_t pairing, void* stream) {
  DAPQ_REQUIRE(x_in != nullptr && x_out != nullptr && pos != nullptr, DAPQ_ERR_INVALID_ARG,
               "x_in, x_out and pos must not be NULL");
  DAPQ_REQUIRE(rows >= 0 && heads >= 1, DAPQ_ERR_INVALID_ARG, "rows (%lld) must be >= 0 and heads (%d) >= 1",
               (long long)rows, heads);
  DAPQ_REQUIRE(head_dim >= 2 && head_dim % 2 == 0, DAPQ_ERR_INVALID_ARG, "head_dim (%d) must be even and >= 2",
               head_dim);
  DAPQ_REQUIRE(pairing == 0 || pairing == 1, DAPQ_ERR_INVALID_ARG, "pairing must be 0 (half) or 1 (interleaved)");
  DAPQ_REQUIRE(theta > 0.0 && isfinite(theta), DAPQ_ERR_INVALID_ARG, "theta must be finite and > 0");
  DAPQ_REQUIRE(stride_head >= head_dim && stride_row >= 0, DAPQ_ERR_INVALID_ARG,
               "stride_head (%lld) must cover head_dim and stride_row (%lld) must be >= 0", (long long)stride_head,
               (long long)stride_row);
  const int64_t work = rows * (head_dim / 2);
  DAPQ_REQUIRE(work / 256 < ((int64_t)1 << 31), DAPQ_ERR_UNSUPPORTED, "too many rows");
  if (work == 0) return DAPQ_OK;
  int hpt = 8;
  while (hpt < 64 && hpt * 2 <= heads && (work / 64) * ((heads + 2 * hpt - 1) / (2 * hpt)) >= 4096) hpt *= 2;
  // small calls: shorter runs until there is a wave per SIMD (64 rows x 32 heads as part of a score call: 0.5 to 1 us of 3.5)
  // (the waves of a run of heads are rounded up: fewer than 64 channel pairs are one wave, and many heads of them keep their runs)
  while (hpt > 1 && hpt <= 8 && (work + 63) / 64 * (((int64_t)heads + hpt - 1) / hpt) < 1024) hpt /= 2;
  const int64_t head_runs = ((int64_t)heads + hpt - 1) / hpt;
  DAPQ_REQUIRE(head_runs <= 65535, DAPQ_ERR_UNSUPPORTED, "heads (%d) exceeds %d", heads, 65535 * hpt);
  const double e = rope_exponent(theta, head_dim);
  const int half = head_dim / 2, half_shift = (half & (half - 1)) == 0 ? __builtin_ctz((unsigned)half) : -1;
  auto kernel = hpt == 1 ? rope_kernel<1, false> : (hpt == 2 ? rope_kernel<2, false> : (hpt == 4 ? rope_kernel<4, false> : rope_kernel<0, false>));
  if (hpt >= 8 && work >= ((int64_t)1 << 20) / heads) kernel = rope_kernel<0, true>;  // from 4 MB of results on (a pair: four bytes)
  hipLaunchKernelGGL(kernel, dim3((unsigned)((work + 255) / 256), (unsigned)head_runs), dim3(256), 0,
                     static_cast<hipStream_t>(stream),
                     static_cast<const uint16_t*>(x_in), static_cast<uint16_t*>(x_out), pos, rows, heads, head_dim,
                     stride_row, stride_head, e, pairing, hpt, half_shift);
  DAPQ_HIP_LAUNCH_CHECK("rope_kernel");
  return DAPQ_OK;
}
