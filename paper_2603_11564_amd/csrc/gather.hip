// Cache pruning (Sec. 4.2): only the key-value pairs in M_retain are kept; the pseudo segment is
// discarded.  Copies the retained K and V rows, bit for bit, into the compact cache
// [layer][sequence][KV head][slot][d].
//
// Pure copy, bound by memory: 16 lanes move one 256-byte row with one 16-byte load and store each, so every row is
// read and written in full cache lines; a workgroup of 256 threads moves 32 rows of K or of V, two per 16-lane group.
// Two rows to a group are enough in flight with eight workgroups to a compute unit, and leave the last workgroups of a launch less to do (four and
// one: below).  From 8 MB on the stores carry the non-temporal hint: nobody reads the compact cache before the rest of it is
// written (a model's weights pass through the caches in between), and lines that are not kept leave room for reads.  From 192 MB on, where the rows read can't still lie in the 256 MB
// memory-side cache for a second call either, the loads do too; smaller calls find rows there that the score passes or the caller brought in.
// Us, four rows to a group without hints -> two without, two with hinted stores, two with both (one with both), MB read and written:
//   2 MB    2.37 -> 1.94, 1.94, 1.94 (1.98)       8   2.90 -> 2.54, 2.42, 2.75 (3.25)      32    6.6 -> 6.4, 5.9, 7.3 (7.7)
//   129    27.9 -> 26.4, 21.3, 22.7 (23.2)      258  52.5 -> 51.1, 44.8, 42.5 (43.4)      515  104.9 -> 102.9, 92.8, 84.2 (87.3; 6.1 TB/s)
// Those are calls again and again.  Four rows without hints -> these, with a selection and over three sets of buffers in turn: 16 MB 10.8 -> 9.9, 64 23.5 ->
// 21.9, 134 43.0 -> 37.2, 258 67.4 -> 57.4, 515 115.4 -> 99.2.  Behind score passes a call gains nothing: what it writes goes out during the next
// kernels without the hint (258 MB 48.0 -> 49.2, 64 16.7 -> 17.2; with the decode steps of all layers after it, each behind 200 MB of weights, 2275 -> 2271
// and 578 -> 577).  Decode steps with nothing between read the compact cache from memory and take 10 to 24 % longer (8 layers of 64 MB 62 -> 77, 32 of
// 134 190 -> 211, 32 of 258 253 -> 303): with stores that only write through L2 they do not (62, 190, 242; the call behind score passes 43.3 at 258 MB),
// but the calls in turn lose half their gain and more (64 MB 23.3, 134 41.8; 258 64.1 for 60.5).
#include "dapq_internal.h"
#include "kernel_args.h"

namespace dapq {
namespace {

struct GatherParams {
  const uint16_t* k;
  const uint16_t* v;
  const int32_t* idx;
  const int32_t* count;
  const int32_t* cu_seqlens;
  uint16_t* k_out;
  uint16_t* v_out;
  int64_t k_stride_layer, k_stride_seq, k_stride_head, k_stride_token;
  int64_t v_stride_layer, v_stride_seq, v_stride_head, v_stride_token;
  int32_t batch, n_kv_heads, budget, seq_len;  // seq_len: dense batches
  float inv_kv_heads, inv_batch;
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ROWS: rows in flight per 16-lane group.  STREAM_IN, STREAM_OUT: loads and stores of rows carry the non-temporal hint.
template <int ROWS, bool STREAM_IN, bool STREAM_OUT>
__global__ __launch_bounds__(256) void gather_kernel(GatherParams p) {
  touch_args<sizeof(GatherParams)>();
  const int ch = threadIdx.x & 15;
  const int slot0 = blockIdx.x * (16 * ROWS) + (threadIdx.x >> 4);  // this group's slots: slot0 + 16*r
  const int head = (int)blockIdx.y;  // (layer * batch + seq) * Hkv + kv
  const bool is_v = blockIdx.z == 1;
  const int n = p.count[head];
  // (a launch has at most 65535 heads)
  const int rest = __builtin_amdgcn_readfirstlane(quotient(head, p.inv_kv_heads)), kv = head - rest * p.n_kv_heads;
  const int layer = __builtin_amdgcn_readfirstlane(quotient(rest, p.inv_batch)), seq = rest - layer * p.batch;
  int64_t start;
  int L;
  if (p.cu_seqlens == nullptr) {
    L = p.seq_len;
    start = (int64_t)seq * L;
  } else {
    start = p.cu_seqlens[seq];
    L = p.cu_seqlens[seq + 1] - (int)start;
  }
  if (slot0 >= n) return;
  const uint16_t* base = is_v ? p.v + layer * p.v_stride_layer + seq * p.v_stride_seq + kv * p.v_stride_head
                              : p.k + layer * p.k_stride_layer + seq * p.k_stride_seq + kv * p.k_stride_head;
  const int64_t stride_token = is_v ? p.v_stride_token : p.k_stride_token;
  uint16_t* dst = (is_v ? p.v_out : p.k_out) + (int64_t)head * p.budget * kHeadDim;
  const int32_t* idx = p.idx + (int64_t)head * p.budget;
  // all index loads first, then all row loads, then the stores
  int j[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const int slot = slot0 + 16 * r;
    j[r] = slot < n ? idx[slot] : -1;
  }
  u32x4 row[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    row[r] = u32x4{0, 0, 0, 0};
    if (j[r] >= 0 && j[r] < L) {  // never follow an index outside the sequence
      const u32x4* src = reinterpret_cast<const u32x4*>(base + (start + j[r]) * stride_token) + ch;
      row[r] = STREAM_IN ? __builtin_nontemporal_load(src) : *src;
    }
  }
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const int slot = slot0 + 16 * r;
    if (j[r] >= 0 && j[r] < L) {
      u32x4* out = reinterpret_cast<u32x4*>(dst + (int64_t)slot * kHeadDim) + ch;
      if (STREAM_OUT) __builtin_nontemporal_store(row[r], out);
      else *out = row[r];
    }
  }
}

}  // namespace
}  // namespace dapq

using namespace dapq;

extern "C" DAPQ_API int dapq_gather(const dapq_shape* shape, const void* k, const void* v, const int32_t* idx,
                           const int32_t* count, int32_t budget, void* k_out, void* v_out, void* stream) {
  int rc = check_shape(shape, false, true, true);
  if (rc != DAPQ_OK) return rc;
  DAPQ_REQUIRE(k != nullptr && v != nullptr && idx != nullptr && count != nullptr && k_out != nullptr &&
                   v_out != nullptr,
               DAPQ_ERR_INVALID_ARG, "k, v, idx, count, k_out and v_out must not be NULL");
  DAPQ_REQUIRE(budget >= 1, DAPQ_ERR_INVALID_ARG, "budget (%d) must be >= 1", budget);
  DAPQ_REQUIRE(((reinterpret_cast<uintptr_t>(k) | reinterpret_cast<uintptr_t>(v) | reinterpret_cast<uintptr_t>(k_out) |
                 reinterpret_cast<uintptr_t>(v_out)) & 15) == 0,
               DAPQ_ERR_UNSUPPORTED, "k, v, k_out and v_out must be 16-byte aligned");
  const int64_t heads = (int64_t)shape->n_layers * shape->batch * shape->n_kv_heads;
  DAPQ_REQUIRE(heads <= 65535, DAPQ_ERR_UNSUPPORTED, "n_layers * batch * n_kv_heads (%lld) exceeds 65535",
               (long long)heads);
  GatherParams p;
  p.k = static_cast<const uint16_t*>(k);
  p.v = static_cast<const uint16_t*>(v);
  p.idx = idx;
  p.count = count;
  p.cu_seqlens = shape->cu_seqlens;
  p.k_out = static_cast<uint16_t*>(k_out);
  p.v_out = static_cast<uint16_t*>(v_out);
  p.k_stride_layer = shape->k_stride_layer; p.k_stride_seq = shape->k_stride_seq;
  p.k_stride_head = shape->k_stride_head; p.k_stride_token = shape->k_stride_token;
  p.v_stride_layer = shape->v_stride_layer; p.v_stride_seq = shape->v_stride_seq;
  p.v_stride_head = shape->v_stride_head; p.v_stride_token = shape->v_stride_token;
  p.seq_len = (int32_t)(shape->total_tokens / shape->batch);
  p.inv_kv_heads = 1.0f / (float)shape->n_kv_heads;
  p.inv_batch = 1.0f / (float)shape->batch;
  p.batch = shape->batch;
  p.n_kv_heads = shape->n_kv_heads;
  p.budget = budget;
  // bytes read and written where every head keeps its whole budget (figures: above)
  const int64_t moved = 2 * 2 * heads * budget * kHeadDim * (int64_t)sizeof(uint16_t);
  auto kernel = moved >= ((int64_t)192 << 20) ? gather_kernel<2, true, true>
                                              : (moved >= ((int64_t)8 << 20) ? gather_kernel<2, false, true> : gather_kernel<2, false, false>);
  int rows = 32;  // of a workgroup
  if (budget > 1 << 28) {  // (a launch holds fewer than 2^32 threads along an axis)
    rows = 64;
    kernel = gather_kernel<4, true, true>;
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)(((int64_t)budget + rows - 1) / rows), (unsigned)heads, 2), dim3(256), 0,
                     static_cast<hipStream_t>(stream), p);
  DAPQ_HIP_LAUNCH_CHECK("gather_kernel");
  return DAPQ_OK;
}
