// Importance scoring (Sec. 4.2, S(j) = sum_i Attention(q_i, k_j); Attention = softmax over the
// prompt keys, App. C.1) as two streaming passes over K for gfx950.
//
//   pass 1  (score_wave_pass1_kernel + score_combine_kernel): lse2[row] = log2 sum_j 2^(c * q_row.k_j)
//   pass 2  (score_wave_pass2_kernel [+ score_group_sum_kernel]): S(j) = sum_rows 2^(c * q_row.k_j - lse2[row])
// with c = scale * log2(e).  "rows" are the R = g*N pseudo-query rows of the g query heads that
// share one KV head.  Nothing of size N x L_p is ever stored.  Where a (layer, sequence, KV head) fits one
// workgroup -- one row group, at most 4 chunks per sequence of a dense batch -- dapq_score runs both passes in
// one launch (score_fused_kernel: the same two walks, the merge in between through LDS).
// Prompts of up to 512 keys, at most 256 rows, are the waves of one workgroup: score_short_kernel, one launch for both passes or for either.
// Calls too small to fill the chip that way go through score_tile_pass1_kernel and score_tile_pass2_kernel instead: a
// workgroup per 32 to 256 keys whose waves share out the query rows (make_score_plan draws the line).  Ragged batches go through the
// wave kernels in segments of the packed key axis (Segments).
//
// Work split.  The unit of work is ONE wave (four independent ones are launched as a workgroup).  It keeps a group of up to 256 Q rows of one KV head in
// registers as MFMA operand fragments (up to eight 32-row blocks = 256 registers, from five on pinned to the
// accumulation half of the register file; one wave per SIMD owns the whole 512-register file) and
// walks its own chunk of keys of one (layer, sequence, KV head).  There are kernels for two to eight row blocks, and the row groups
// of a head hold as many each: a padded row block is a sixth to an eighth of the arithmetic, which bounds the passes from five on (both
// passes, 32 layers, 8 KV heads, us, with two, four and eight only -> these: 148 rows, 32768 keys 1106 -> 829; 192, 20000 keys 690 ->
// 576; 224, 32768 keys 1143 -> 1055; 296 (twice five), 8 layers, 40000 keys 606 -> 450; 96, 32768 keys 776 -> 750; 74, 4 KV heads, 5
// prompts of 3926 keys 254 -> 231).  Nothing is shared between waves:
// no barrier anywhere in the separate-pass kernels (the one-launch form has two, between its passes),
// no cross-wave reduction.  Heads with more than 256 rows are split into row
// groups (grid.y): pass 1 needs nothing more (its sums are per row), pass 2 writes one plane of
// column sums per group (group 0 into the result) and a small kernel adds the planes in group order.
// Keys arrive through a per-wave ring of 32-key sub-blocks in LDS (buffer_load_dwordx4 ... lds, five
// slots of 8 KB: four sub-blocks = 32 KB in flight per wave, 128 KB per compute unit; 16-byte
// chunks XOR-swizzled so that the MFMA operand reads are bank-conflict free), and every fragment is
// read from LDS exactly once per wave.  v_mfma_f32_32x32x16_bf16 runs on every (sub-block, row
// block) unit:
//   pass 1 uses D[key][query] (K as the A operand): a lane owns one query column, the reduction
//           over keys stays inside the lane;
//   pass 2 uses D[query][key] (Q as the A operand): a lane owns one key column, the reduction over
//           query rows stays inside the lane, and -lse2 of the lane's 16 rows per row block sits in
//           registers (128 of them).
// Pass 1 does not track a running maximum: it exponentiates against a per-row reference logit taken
// from the first sub-block (2^x has 127 binades of headroom above it) and only if a sum overflows
// redoes the chunk with a conventional online maximum.
//
// With one wave per SIMD every instruction costs issue time, so the kernels are built around the
// instruction count per MFMA ("slice"): one MFMA, and for two logits of the previous unit one FMA,
// one exponential and one add each; the rest (transfer issue, ring wait, fragment reads, loop
// control) is about one more instruction per slice.

#include <float.h>
#include <math.h>

#include <mutex>

#include "dapq_internal.h"
#include "kernel_args.h"
#include "wave_scan.h"

namespace dapq {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));  // 16 bytes; native vector, stays in registers

struct ScoreParams {
  const uint16_t* q;
  const uint16_t* k;
  const int32_t* cu_seqlens;  // NULL = dense
  int32_t* cu_chunks;         // [batch+1] prefix of per-sequence chunk counts (ragged batches of more than 64 sequences)
  float2* parts;              // [layer*Hkv][max_chunks][rows_pad] (reference, sum) in the log2 domain; a ragged batch: of
                              // sequence b in segment i at index b + i
  float* tile_parts;          // tile form: their log2 in one value, reference + log2(sum), -inf for no sum (parts is NULL)
  float* lse2;                // [layer][batch][Hq][N]
  float* scores;              // [layer][Hkv][total_tokens]
  float* partial;             // [n_groups-1][layer][Hkv][total_tokens] column sums of row groups 1.. (n_groups > 1)
  int64_t k_stride_layer, k_stride_seq, k_stride_head, k_stride_token;
  int64_t q_stride_layer, q_stride_seq, q_stride_head, q_stride_row;
  int64_t total_tokens;
  int32_t n_layers, batch, n_q_heads, n_kv_heads, group, n_pseudo;
  int32_t rows, rows_pad, n_groups, chunk_keys, max_chunks;
  int32_t segments;           // ragged batches in the wave form: segments a head is cut into (chunk_keys is a sub-block then)
  int32_t wg_groups;          // row groups that sit side by side in a workgroup (dense launches; 1, 2 or 4)
  float c;  // scale * log2(e)
  // What every workgroup would divide for before it can ask for its first key:
  int32_t seq_len, chunks_per_seq;  // dense batches
  int32_t chunk_shift;              // ragged batches and the tile form: log2(chunk_keys)
  int32_t stage_q;                  // tile form: the queries go through LDS too
  float inv_n_pseudo, inv_kv_heads, inv_rows_pad;
  float stream_share;               // see KeyStream
};


constexpr int kSubBytes = 32 * kHeadDim * 2;          // one 32-key sub-block
// The least that a running maximum is.  Not -inf: the logits of a whole sub-block may be that (masked keys, say), and then add nothing.
constexpr float kLowest = -FLT_MAX;

// Which (sequence, chunk) a workgroup works on.
struct Work {
  int seq;
  int64_t tok0;  // packed token index of the first key of the chunk
  int key0;      // first key of the chunk inside the sequence
  int nkeys;     // keys in the chunk (<= chunk_keys), 0 = nothing to do
  int seq_len;
};

// Wave-uniform values pinned to scalar registers.
__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ unsigned uniform_u32(unsigned v) { return (unsigned)__builtin_amdgcn_readfirstlane((int)v); }
template <typename T>
__device__ __forceinline__ const T* uniform_ptr(const T* ptr) {
  const unsigned long long v = (unsigned long long)(uintptr_t)ptr;
  const unsigned lo = (unsigned)uniform_i32((int)(unsigned)(v & 0xFFFFFFFFull));
  const unsigned hi = (unsigned)uniform_i32((int)(unsigned)(v >> 32));
  return reinterpret_cast<const T*>((uintptr_t)(((unsigned long long)hi << 32) | lo));
}
// Chunks of a sequence of L keys (of a ragged batch: chunk_keys is a power of two).
__device__ __forceinline__ int chunks_of_length(const ScoreParams& p, int L) {
  return L > 0 ? (L + p.chunk_keys - 1) >> p.chunk_shift : 0;
}
// The lane number, formed where it is asked for: neither it nor what follows from it is kept in registers from before.
__device__ __forceinline__ int fresh_lane() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  return lane;
}

// A ragged batch of at most 64 sequences, one to a lane: the sequence's start, length and the chunks up to its end.
// Every wave forms this itself out of two loads and a scan: looking a chunk up in the prefix in device memory is a
// chain of log2(batch) + 3 dependent loads, and the kernel that writes the prefix a launch of its own.
struct LaneSequence {
  int start, len, chunks, chunks_end;
};
__device__ __forceinline__ LaneSequence lane_sequence(const ScoreParams& p) {
  const int lane = fresh_lane();
  LaneSequence q;
  q.start = p.cu_seqlens[lane < p.batch ? lane : p.batch];
  q.len = p.cu_seqlens[lane < p.batch ? lane + 1 : p.batch] - q.start;
  q.chunks = chunks_of_length(p, q.len);
  q.chunks_end = (int)wave_scan<OpAdd>((uint32_t)q.chunks);
  return q;
}

// The same for a wave-uniform chunk index, with the result pinned to scalar registers: everything
// derived from it (key base pointer, buffer descriptors, trip counts) then stays scalar too.  Called by whole waves.
__device__ __forceinline__ Work locate(const ScoreParams& p, int gchunk);
__device__ __forceinline__ Work locate_uniform(const ScoreParams& p, int gchunk) {
  Work w = locate(p, gchunk);
  w.seq = uniform_i32(w.seq);
  w.key0 = uniform_i32(w.key0);
  w.nkeys = uniform_i32(w.nkeys);
  w.seq_len = uniform_i32(w.seq_len);
  const unsigned lo = (unsigned)uniform_i32((int)(unsigned)(w.tok0 & 0xFFFFFFFFll));
  const unsigned hi = (unsigned)uniform_i32((int)(unsigned)((unsigned long long)w.tok0 >> 32));
  w.tok0 = (int64_t)(((unsigned long long)hi << 32) | lo);
  return w;
}

__device__ __forceinline__ Work locate(const ScoreParams& p, int gchunk) {
  Work w;
  w.nkeys = 0;
  if (p.cu_seqlens == nullptr) {
    if (p.chunks_per_seq == 0) return w;
    w.seq = 0;
    if (p.batch > 1) w.seq = gchunk / p.chunks_per_seq;
    if (w.seq >= p.batch) return w;
    w.key0 = (gchunk - w.seq * p.chunks_per_seq) * p.chunk_keys;
    w.tok0 = (int64_t)w.seq * p.seq_len + w.key0;
    w.seq_len = p.seq_len;
  } else if (p.batch <= 64) {
    const LaneSequence q = lane_sequence(p);
    w.seq = __popcll(__ballot(q.chunks_end <= gchunk));  // (lanes past the batch repeat the last end)
    if (w.seq >= p.batch) return w;
    w.key0 = (gchunk - __builtin_amdgcn_readlane(q.chunks_end - q.chunks, w.seq)) * p.chunk_keys;
    w.tok0 = (int64_t)__builtin_amdgcn_readlane(q.start, w.seq) + w.key0;
    w.seq_len = __builtin_amdgcn_readlane(q.len, w.seq);
  } else {
    if (gchunk >= p.cu_chunks[p.batch]) return w;
    int lo = 0, hi = p.batch;  // largest b with cu_chunks[b] <= gchunk
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (p.cu_chunks[mid] <= gchunk) lo = mid; else hi = mid;
    }
    w.seq = lo;
    const int start = p.cu_seqlens[lo];
    w.seq_len = p.cu_seqlens[lo + 1] - start;
    w.key0 = (gchunk - p.cu_chunks[lo]) * p.chunk_keys;
    w.tok0 = (int64_t)start + w.key0;
  }
  const int left = w.seq_len - w.key0;
  w.nkeys = left < p.chunk_keys ? left : p.chunk_keys;
  if (w.nkeys < 0) w.nkeys = 0;
  return w;
}

// A ragged batch in the wave form: the packed key axis of a head -- the 32-key sub-blocks of its sequences one after the other,
// `total` of them -- is cut into segments of equal length, the same for all heads, and a wave (per row group) takes one.
// Segment i holds sub-blocks total * i / n up to total * (i + 1) / n of n segments; none is empty.  (Handed out chunk by chunk from
// work lists, each chunk with a ring fill of its own, the waves kept too few keys in flight -- with at most 128 rows the passes are
// bound by the key stream -- and the last items of a launch ran alone.  dapq_score, 32 layers: 16 prompts of 200..2500 keys, 128 rows
// 742 -> 611 us; 2 of 11520, 128 rows 640 -> 557; 64 of 100..500, 256 rows 1167 -> 1020; 8 of 4096..16384, 512 rows 5326 -> 5259.  Two
// waves to a SIMD with a ring of two slots each, on the lists, were slower than either.)
struct Segments {
  int total, n;
  __device__ __forceinline__ int start(int i) const { return (int)((int64_t)total * i / n); }
  // the segment of sub-block g: the last one that starts at or before it
  __device__ __forceinline__ int of(int g) const { return (int)((((int64_t)g + 1) * n - 1) / total); }
};
__device__ __forceinline__ Segments segments_of(const ScoreParams& p, int total) {
  return {total, p.segments < total ? p.segments : total};
}
// The sub-blocks of a segment: `left` of them, from number `sub` of sequence `seq` on (`last`: down from there, the segment's last).
struct Segment {
  int seq, sub, left;
};
__device__ __forceinline__ Segment segment_of_wave(const ScoreParams& p, int i, bool last) {
  Segment r = {0, 0, 0};
  LaneSequence q;
  const bool by_lanes = p.batch <= 64;
  if (by_lanes) q = lane_sequence(p);
  const Segments segs = segments_of(p, by_lanes ? __builtin_amdgcn_readlane(q.chunks_end, 63) : p.cu_chunks[p.batch]);
  if (i >= segs.n) return r;
  const int first = segs.start(i), end = segs.start(i + 1), g = last ? end - 1 : first;
  if (by_lanes) {
    r.seq = __popcll(__ballot(q.chunks_end <= g));
    r.sub = g - __builtin_amdgcn_readlane(q.chunks_end - q.chunks, r.seq);
  } else {
    int lo = 0, hi = p.batch;  // largest b with cu_chunks[b] <= g (no empty sequence: those end where they start)
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (p.cu_chunks[mid] <= g) lo = mid; else hi = mid;
    }
    r.seq = lo;
    r.sub = g - p.cu_chunks[lo];
  }
  r.seq = uniform_i32(r.seq);
  r.sub = uniform_i32(r.sub);
  r.left = uniform_i32(end - first);
  return r;
}
// Start and length of a sequence, through the scalar cache: a vector load's answer would be waited for behind the key ring.
struct SeqRange {
  int start, len;
};
__device__ __forceinline__ SeqRange seq_range(const ScoreParams& p, int seq) {
  const __attribute__((address_space(4))) int32_t* cu =
      (const __attribute__((address_space(4))) int32_t*)(uintptr_t)p.cu_seqlens + seq;
  const int start = cu[0], end = cu[1];
  return {start, end - start};
}

// LDS position of 16-byte chunk `ch` of sub-block row `key`: rows are 256 B apart, chunks XOR-swizzled by
// the row so that 16 consecutive rows reading the same logical chunk hit 16 different bank groups.
__device__ __forceinline__ int lds_chunk_index(int key, int ch) { return key * 16 + (ch ^ (key & 15)); }

// Fragment s of lane (n, h) of an MFMA operand is the 8 channels [(2s+h)*8, +8) of row n: the same
// for a 32-row block of Q read straight from global memory.
__device__ __forceinline__ void frag_from_q(bf16x8 (&f)[8], const ScoreParams& p, const uint16_t* qbase, int row,
                                            int h) {
  const int rc = row < p.rows ? row : p.rows - 1;  // padding rows repeat the last row; their results are dropped
  const int head = quotient(rc, p.inv_n_pseudo), i = rc - head * p.n_pseudo;
  const uint16_t* src = qbase + (int64_t)head * p.q_stride_head + (int64_t)i * p.q_stride_row;
#pragma unroll
  for (int s = 0; s < 8; ++s) f[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(src + (2 * s + h) * 8));
}

__device__ __forceinline__ float xhalf(float v) { return __shfl_xor(v, 32, 64); }

// v + (v of the lane 32 away), in every lane, on the vector ALU alone (v_permlane32_swap exchanges the upper half of
// its first operand with the lower half of its second): no trip through LDS, hence no wait on the LDS counter, which
// with a single wave per SIMD would be dead time.  The wait states around the swap are the ones the hazard rules
// of gfx950 ask for between a vector write and a lane swap of the same register, and between the swap and its use.
__device__ __forceinline__ float sum_halves(float v) {
  float a = v, b = v;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return a + b;  // a = (v.lo, v.lo), b = (v.hi, v.hi)
}
__device__ __forceinline__ float max_halves(float v) {
  float a = v, b = v;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return fmaxf(a, b);
}

// Column sums of one sub-block go out through a buffer store whose range check drops what must not be written:
// lanes of the upper half carry an offset far past the end, and keys at or past nkeys fall outside num_records.
struct ColumnStore {
  __amdgpu_buffer_rsrc_t rsrc;
  unsigned lane_off;  // byte offset of this lane's key inside a sub-block; out of range for the upper half
};
__device__ __forceinline__ ColumnStore make_column_store(float* out, int nkeys, int n, int h) {
  ColumnStore cs;
  cs.rsrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, nkeys * 4, 0x00020000);
  cs.lane_off = h == 0 ? (unsigned)n * 4u : 0xC0000000u;
  return cs;
}
__device__ __forceinline__ void store_columns(const ColumnStore& cs, int first_key, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), cs.rsrc,
                                            (int)(cs.lane_off + (unsigned)first_key * 4u), 0, 0);
}

// Row of the 32x32 MFMA result held in accumulator register v of a lane in half h.
__device__ __forceinline__ int acc_row(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }

typedef const u32x4 __attribute__((address_space(3))) * lds_vec_ptr;

// 16-byte LDS read at a per-lane byte address plus a compile-time offset (folds into the instruction).
__device__ __forceinline__ bf16x8 lds_read16(unsigned lane_addr, int const_off) {
  return __builtin_bit_cast(bf16x8, *(lds_vec_ptr)(uintptr_t)(lane_addr + const_off));
}

// Per-sequence prefix of chunk counts for ragged batches: one wave, 64 sequences per trip (a scan by shuffles
// inside the wave, the running total carried from trip to trip).
__global__ void score_chunk_prefix_kernel(const int32_t* cu_seqlens, int32_t* cu_chunks, int batch, int chunk_keys) {
  const int lane = threadIdx.x;  // launched with exactly 64 threads
  if (lane == 0) cu_chunks[0] = 0;
  int carry = 0;
  for (int b0 = 0; b0 < batch; b0 += 64) {
    const int b = b0 + lane;
    int mine = 0;
    if (b < batch) {
      const int L = cu_seqlens[b + 1] - cu_seqlens[b];
      mine = L > 0 ? (L + chunk_keys - 1) / chunk_keys : 0;
    }
    int inc = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int o = __shfl_up(inc, d, 64);
      if (lane >= d) inc += o;
    }
    if (b < batch) cu_chunks[b + 1] = carry + inc;
    carry += __shfl(inc, 63, 64);
  }
}

// Merge the per-chunk (reference, sum) pairs of a row: lse2 = log2 sum_c z_c 2^(ref_c).
//
// A workgroup takes 64 rows of one (layer, sequence, KV head), a lane per row, and its waves share out the chunks in
// runs of kCombineRun, whose loads are all in flight together.  What bounds it is latency: one thread walking a row's
// chunks alone, twice, was a chain of 2 x chunks loads (one layer, 8 heads, 128 rows, 8191 keys = 64 chunks: 37 us next
// to two score passes of 13 us; the whole dapq_score call 60 us then, 26 us now).
// The sum does not depend on how many waves share the work: run r belongs to class r % kCombineClasses, a class is
// summed in run order, chunk by chunk, and the classes are added in class order (up to kCombineRun chunks: plain chunk
// order, which is what score_fused_kernel does).
constexpr int kCombineRun = 8, kCombineClasses = 16;
__global__ __launch_bounds__(64 * kCombineClasses) void score_combine_kernel(ScoreParams p, int row_tiles, float inv_row_tiles, int first_seq) {
  __shared__ float lds_max[kCombineClasses][64], lds_sum[kCombineClasses][64];
  const int lane = threadIdx.x & 63, wave = uniform_i32((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
  touch_args<sizeof(ScoreParams) + 12>();
  const int seq = uniform_i32(quotient((int)blockIdx.x, inv_row_tiles)), row = (int)(blockIdx.x - seq * row_tiles) * 64 + lane;
  const int b = first_seq + seq;
  const int layer = uniform_i32(quotient((int)blockIdx.y, p.inv_kv_heads)), kv = (int)blockIdx.y - layer * p.n_kv_heads;
  int c0, c1, total = 0;
  if (p.cu_seqlens == nullptr) {
    c0 = b * p.chunks_per_seq;
    c1 = c0 + p.chunks_per_seq;
  } else if (p.batch <= 64) {
    const LaneSequence q = lane_sequence(p);
    c1 = __builtin_amdgcn_readlane(q.chunks_end, b);
    c0 = c1 - __builtin_amdgcn_readlane(q.chunks, b);
    total = __builtin_amdgcn_readlane(q.chunks_end, 63);
  } else {
    c0 = p.cu_chunks[b];
    c1 = p.cu_chunks[b + 1];
    total = p.cu_chunks[p.batch];
  }
  if (p.segments > 0 && c1 > c0) {  // the wave form of a ragged batch: one sum per segment that holds some of the sequence
    const Segments segs = segments_of(p, total);
    c0 = b + segs.of(c0);
    c1 = b + segs.of(c1 - 1) + 1;
  }
  const int n = c1 - c0, runs = (n + kCombineRun - 1) / kCombineRun;
  const int64_t src = ((int64_t)blockIdx.y * p.max_chunks + c0) * p.rows_pad + (row < p.rows ? row : p.rows - 1);
  // t[i] = log2 of the sum of chunk run * kCombineRun + i, -inf for chunks without one
  auto load_run = [&](int run, float (&t)[kCombineRun]) {
    if (p.tile_parts != nullptr) {
#pragma unroll
      for (int i = 0; i < kCombineRun; ++i) {
        const int c = run * kCombineRun + i;
        const float v = p.tile_parts[src + (int64_t)(c < n ? c : n - 1) * p.rows_pad];
        t[i] = c < n ? v : -INFINITY;
      }
      return;
    }
    float2 v[kCombineRun];
#pragma unroll
    for (int i = 0; i < kCombineRun; ++i) {
      const int c = run * kCombineRun + i;
      v[i] = p.parts[src + (int64_t)(c < n ? c : n - 1) * p.rows_pad];
    }
#pragma unroll
    for (int i = 0; i < kCombineRun; ++i)
      t[i] = run * kCombineRun + i < n && v[i].y > 0.0f ? v[i].x + log2f(v[i].y) : -INFINITY;
  };
  float t[kCombineRun], m = -INFINITY;
  for (int run = wave; run < runs; run += waves) {
    load_run(run, t);
#pragma unroll
    for (int i = 0; i < kCombineRun; ++i) m = fmaxf(m, t[i]);
  }
  if (waves > 1) {
    lds_max[wave][lane] = m;
    __syncthreads();
    for (int w = 0; w < waves; ++w) m = fmaxf(m, lds_max[w][lane]);
  }
  const bool one_run = wave + waves >= runs;  // its run is still in t
  float s = 0.0f;
  for (int k = wave; k < kCombineClasses && k < runs; k += waves) {
    float sum = 0.0f;
    for (int run = k; run < runs; run += kCombineClasses) {
      if (!one_run) load_run(run, t);
#pragma unroll
      for (int i = 0; i < kCombineRun; ++i) sum += exp2f(t[i] - m);
    }
    if (waves > 1) lds_sum[k][lane] = sum;
    else s += sum;
  }
  if (waves > 1) {
    __syncthreads();
    if (wave != 0) return;
    for (int k = 0; k < kCombineClasses && k < runs; ++k) s += lds_sum[k][lane];
  }
  if (row >= p.rows) return;
  // (m is -inf, and s not a number, only where no chunk has a sum)
  const int64_t first = (((int64_t)layer * p.batch + b) * p.n_q_heads + (int64_t)kv * p.group) * p.n_pseudo;
  p.lse2[first + row] = (s > 0.0f) ? m + log2f(s) : 0.0f;
}

// ---------------------------------------------------------------------------------------------
// The score kernels: one wave = a group of query rows x its own key stream.
// ---------------------------------------------------------------------------------------------
constexpr int kWaveStages = 5;            // ring slots (40 KB per wave, 160 KB per compute unit)
constexpr int kSubVec = kSubBytes / 16;   // 512 16-byte chunks per sub-block
// Dense launches start their waves up to four to a workgroup, one per SIMD of a compute unit, each with its own ring:
// they never meet at a barrier.  The waves of a workgroup are the row groups of a chunk side by side (a KV head with
// more than 256 query rows: they read the same keys at the same time, and the second reader finds them in the compute
// unit's L2 instead of fetching them through the fabric again: 6 % at 512 and 1024 rows) and then consecutive chunks
// (the dispatcher places fewer workgroups and the waves of a compute unit read one head's queries once: 2-3 % for the
// stream-bound shapes).  Every workgroup must be full -- waves of a half-empty one would idle their SIMDs for the whole
// launch -- so the number of consecutive chunks is the largest of 4, 2, 1 (divided by the row groups) that divides
// the chunk count.  (Ragged batches: the same, with segments of the packed key axis for chunks.)
constexpr int kWavesPerGroup = 4;
constexpr int wave_lds(int nst) { return nst * kSubBytes; }

// Per-lane byte offsets of the four distinct 16-byte chunks a lane fetches in sub_dma: transfer i
// moves key rows 4i..4i+3, lane (row0 = lane / 16, pos = lane % 16) fills LDS position pos of row
// 4i + row0 with the logical chunk pos ^ ((4i + row0) & 15) = (pos ^ row0) ^ (4 * (i & 3)).
__device__ __forceinline__ void sub_dma_lane_offsets(unsigned (&voff)[4], int64_t stride_token, int lane) {
  const unsigned row0 = (unsigned)lane >> 4, pos = (unsigned)lane & 15u;
#pragma unroll
  for (int j = 0; j < 4; ++j) voff[j] = row0 * (unsigned)stride_token * 2u + ((pos ^ row0) ^ (4u * j)) * 16u;
}

// One wave moves the 32-key sub-block that starts at key0 into an LDS slot: 8 transfers of 1 KB
// (buffer_load_dwordx4 ... lds).  The buffer descriptor spans from the first row of the sub-block to
// the end of the last key row of the chunk, so rows past the end of the chunk read as zeros; the
// uniform part of every address lives in scalar registers (descriptor base, scalar offset per
// transfer) and the lane part is one of the four precomputed offsets.  A sub-block that is not `live` (it starts before
// the chunk or at or past its end) gets an empty descriptor: the eight transfers still count as vector
// memory operations (the waits rely on a fixed number per sub-block) but fetch nothing and fill the
// slot with zeros.
// AUX: the transfers' cache policy.
constexpr int kNonTemporal = 2;
template <int AUX = 0>
__device__ __forceinline__ void sub_dma(u32x4* slot, const uint16_t* kbase, int64_t stride_token, int key0, int nkeys, bool live,
                                        const unsigned (&voff)[4]) {
  const int64_t stride_b = stride_token * 2;
  const char* base = reinterpret_cast<const char*>(kbase) + (live ? (int64_t)key0 * stride_b : (int64_t)0);
  const int64_t span = (int64_t)(nkeys - key0 - 1) * stride_b + kHeadDim * 2;
  const unsigned records = !live ? 0u : (span > (int64_t)0xFFFFFFFFll ? 0xFFFFFFFFu : (unsigned)span);
  const __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, (int)records, 0x00020000);
#pragma unroll
  for (int i = 0; i < 8; ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(slot + i * 64), 16,
                                             (int)voff[i & 3], (int)((unsigned)(4 * i) * (unsigned)stride_b), 0, AUX);
}

// Waits until the sub-block after the current one has landed: at most the transfers (8 operations each) of the NST - 1 newer
// ones are in flight.
template <int NST>
__device__ __forceinline__ void wait_ring_full() {
  static_assert(NST >= 2 && NST <= 5, "ring sizes the kernels use");
  if (NST == 5) asm volatile("s_waitcnt vmcnt(32)" ::: "memory");
  else if (NST == 4) asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
  else if (NST == 3) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
}

// The instruction order is pinned with empty asm statements that take values as read-write operands:
// what produces an operand must come before the statement, what uses it after.  One sits right
// after the MFMA of a slice (it "redefines" the K fragment the MFMA read and the two pending
// exponents, so the MFMA leads the slice and the vector work follows), one at the end of the slice.
// Neither names a transcendental's result or the accumulator in flight: both would cost wait states.
// (Naming the K fragment of the next MFMA at the slice end as well keeps that MFMA from starting
// early, but measures 1-2 % slower per pass over a few hundred back-to-back launches.)
#define DAPQ_WAVE_SLICE_MID(kfrag, x0, x1) asm volatile("" : "+v"(kfrag), "+v"(x0), "+v"(x1))
#define DAPQ_WAVE_SLICE_END(prev, x0, x1, t0, t1, addr) \
  asm volatile("" : "+v"(prev), "+v"(x0), "+v"(x1), "+v"(t0), "+v"(t1), "+v"(addr))

// One step of the four-stage vector pipeline over pairs of logits: the exponentials started two
// steps ago (p0, p1: two sets of registers take turns) are added to the sums they belong to (t0,
// t1), the exponents formed in the previous step are exponentiated into the registers just freed,
// and the exponents of a new pair are formed (x = a*c + o).  Every result is first read a full step
// after the instruction that produces it, whatever order the compiler picks inside a step.
// (first: t0 starts with this pair)
#define DAPQ_VALU_STEP(first, a0, a1, o0, o1, t0, t1, p0, p1) \
  do {                                                 \
    if (first) {                                       \
      t0 = p0 + p1;                                    \
    } else {                                           \
      t0 += p0;                                        \
      t1 += p1;                                        \
    }                                                  \
    p0 = __builtin_amdgcn_exp2f(x0);                   \
    p1 = __builtin_amdgcn_exp2f(x1);                   \
    x0 = fmaf((a0), c, (o0));                          \
    x1 = fmaf((a1), c, (o1));                          \
  } while (0)
// step k of a unit: even steps use the first set of pending exponentials, odd steps the second
#define DAPQ_VALU_STEP_K(k, first, a0, a1, o0, o1, t0, t1)                     \
  do {                                                                         \
    if ((k) % 2 == 0) DAPQ_VALU_STEP(first, a0, a1, o0, o1, t0, t1, ea0, ea1); \
    else DAPQ_VALU_STEP(first, a0, a1, o0, o1, t0, t1, eb0, eb1);              \
  } while (0)

// Pipelined walk of one wave over `count` sub-blocks of its stream of keys, all of one sequence: numbers first_sub,
// first_sub + 1, ... of it (a reversed stream: first_sub, first_sub - 1, ...).
//   on entry  kf = fragments of the first one, which lies in ring slot `slot`; the transfers of the NST - 1 sub-blocks
//             after it are under way (they lie in the slots after that one, in turn)
//   on exit   kf = fragments of the sub-block after the last one, in slot `slot` (zeros if it does not exist)
// Every iteration issues the transfer of the sub-block NST ahead into the slot of the current sub-block
// once its fragments are in registers, and waits for the next sub-block before its last unit; as every
// sub-block is 8 operations, existing or not, that wait is a fixed count.
// A unit is one sub-block against one 32-row block of Q: 8 MFMAs, one per slice.  While the MFMAs
// of a unit issue, the 16 logits per lane of the unit before it enter the vector pipeline, one pair
// per slice (the MFMA leads its slice, so the last MFMA of a unit is a full slice old when its
// first result is read).  The sum a step adds to belongs to the pair three steps back: steps 0..2
// of a unit still feed the unit two back.
// PASS 1: off1[rb] = -(reference logit * c) of row block rb; acc[rb] receives the row sums.  In segments
// and long chunks a unit's 16 terms of a lane are added up first (su): the same number of additions, and small
// terms meet a large sum once a unit instead of one by one (8 prompts of 4096..16384 keys, 512 rows: 6e-7 off float64).
// PASS 2: off2[rb][v] = -lse2 of the row that accumulator register v of this lane holds in row
//         block rb (-inf for padding rows, which then add 0).  S of every key goes to out.
// NST = slots of the sub-block ring.
template <int NRB, int PASS, int NST, class Stream>
__device__ __forceinline__ void wave_walk(u32x4* ring, int& slot, Stream& keys, int first_sub, int count, int nkeys,
                                          bf16x8 (&kf)[8], const bf16x8 (&qf)[NRB][8], float c,
                                          const float (&off1)[NRB], const float (&off2)[PASS == 2 ? NRB : 1][16],
                                          float (&acc)[NRB], float* out, const unsigned (&voff)[4], int n, int h) {
  constexpr bool kUnitSums = PASS == 1 && Stream::kUnitSums;
  auto first_key = [&](int sub) { return (Stream::kReversed ? first_sub - sub : first_sub + sub) * 32; };
  const unsigned ring_base = (unsigned)(uintptr_t)(lds_vec_ptr)ring;
  unsigned fa[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) fa[s] = ring_base + (unsigned)(n * 16 + ((2 * s + h) ^ (n & 15))) * 16u;
  const ColumnStore cols = make_column_store(PASS == 2 ? out : nullptr, PASS == 2 ? nkeys : 0, n, h);
  f32x16 prev;
#pragma unroll
  for (int v = 0; v < 16; ++v) prev[v] = -INFINITY;  // 2^(-inf) = 0: the first steps add nothing
  float x0 = -INFINITY, x1 = -INFINITY, ea0 = 0.0f, ea1 = 0.0f, eb0 = 0.0f, eb1 = 0.0f, sa = 0.0f, sb = 0.0f, su = 0.0f;
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) acc[rb] = 0.0f;

  int read_slot = slot + 1 == NST ? 0 : slot + 1;  // ring slot of the sub-block after the current one
  for (int sub = 0; sub < count; ++sub) {
    const unsigned next_slot = (unsigned)read_slot * (unsigned)kSubBytes;
    read_slot = read_slot + 1 == NST ? 0 : read_slot + 1;
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      constexpr int kLast = NRB - 1;
      const int rb1 = (rb + NRB - 1) % NRB;  // row block of the previous unit (prev)
      const int rb2 = (rb + NRB - 2) % NRB;  // row block of the unit before it
      if (rb == 1) {
        // the slot of this sub-block is free (its fragments are in registers and have been used)
        keys.fetch(ring + slot * kSubVec, voff, first_key(sub + NST));
        slot = slot + 1 == NST ? 0 : slot + 1;
      }
      if (rb == kLast) wait_ring_full<NST>();  // sub-block sub+1 has landed: NST-1 newer ones are in flight
      f32x16 cur = {0};
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        if (PASS == 1) cur = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[rb][s], cur, 0, 0, 0);
        else cur = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[rb][s], kf[s], cur, 0, 0, 0);
        DAPQ_WAVE_SLICE_MID(kf[s], x0, x1);
        if (rb == kLast) kf[s] = lds_read16(fa[s] + next_slot, 0);  // last use: fetch the next sub-block's
        if (PASS == 2) {
          DAPQ_VALU_STEP_K(s, false, prev[2 * s], prev[2 * s + 1], off2[PASS == 2 ? rb1 : 0][2 * s],
                           off2[PASS == 2 ? rb1 : 0][2 * s + 1], sa, sb);
          if (s == 2 && rb == 1) {
            // the adds above took in the last logits of the previous sub-block: its column sums are complete
            if (sub > 0) store_columns(cols, first_key(sub - 1), sum_halves(sa + sb));
            sa = sb = 0.0f;
          }
          DAPQ_WAVE_SLICE_END(prev, x0, x1, sa, sb, fa[(s + 1) & 7]);
        } else {
          if constexpr (kUnitSums) {
            DAPQ_VALU_STEP_K(s, s == 3, prev[2 * s], prev[2 * s + 1], off1[rb1], off1[rb1], su, su);
            if (s == 2) acc[rb2] += su;  // the unit two back is complete
            DAPQ_WAVE_SLICE_END(prev, x0, x1, su, acc[rb2], fa[(s + 1) & 7]);
          } else {
            if (s < 3) DAPQ_VALU_STEP_K(s, false, prev[2 * s], prev[2 * s + 1], off1[rb1], off1[rb1], acc[rb2], acc[rb2]);
            else DAPQ_VALU_STEP_K(s, false, prev[2 * s], prev[2 * s + 1], off1[rb1], off1[rb1], acc[rb1], acc[rb1]);
            DAPQ_WAVE_SLICE_END(prev, x0, x1, acc[rb1], acc[rb2], fa[(s + 1) & 7]);
          }
        }
      }
      prev = cur;
    }
  }

  // drain: prev = last unit (row block NRB-1); three more steps on -inf flush the pipeline
  {
    constexpr int rbl = NRB - 1, rbl1 = NRB - 2;
#pragma unroll
    for (int k = 0; k < 11; ++k) {
      const float a0 = k < 8 ? prev[(2 * k) & 15] : -INFINITY, a1 = k < 8 ? prev[(2 * k + 1) & 15] : -INFINITY;
      if (PASS == 1) {
        if constexpr (kUnitSums) {
          DAPQ_VALU_STEP_K(k, k == 3, a0, a1, off1[rbl], off1[rbl], su, su);
          if (k == 2) acc[rbl1] += su;
          if (k == 10) acc[rbl] += su;
        } else {
          if (k < 3) DAPQ_VALU_STEP_K(k, false, a0, a1, off1[rbl], off1[rbl], acc[rbl1], acc[rbl1]);
          else DAPQ_VALU_STEP_K(k, false, a0, a1, off1[rbl], off1[rbl], acc[rbl], acc[rbl]);
        }
      } else {
        DAPQ_VALU_STEP_K(k, false, a0, a1, off2[PASS == 2 ? rbl : 0][(2 * k) & 15], off2[PASS == 2 ? rbl : 0][(2 * k + 1) & 15], sa,
                         sb);
      }
    }
    if (PASS == 2 && count > 0) store_columns(cols, first_key(count - 1), sum_halves(sa + sb));
  }
}

// One sub-block the plain way (pass 1): masks keys >= nkeys (or, CAUSAL, the keys after each query's
// own position), fixes the reference logits (FIRST) or tracks a running maximum (SAFE).
template <int NRB, bool SAFE, bool FIRST, bool CAUSAL = false>
__device__ __forceinline__ void wave_sub_simple(const bf16x8 (&kf)[8], const bf16x8 (&qf)[NRB][8], float c,
                                                float (&ref)[NRB], float (&z)[NRB], int key0, int nkeys, int h,
                                                const int* last_key = nullptr) {
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    f32x16 a = {0};
#pragma unroll
    for (int s = 0; s < 8; ++s) a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[rb][s], a, 0, 0, 0);
    if (CAUSAL) {
      // last_key[rb]: the last key this lane's query of row block rb may see
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (key0 + acc_row(v, h) > last_key[rb]) a[v] = -INFINITY;
    } else if (key0 + 32 > nkeys) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (key0 + acc_row(v, h) >= nkeys) a[v] = -INFINITY;
    }
    if (SAFE || FIRST) {
      float m = a[0];
#pragma unroll
      for (int v = 1; v < 16; ++v) m = fmaxf(m, a[v]);
      m = fmaxf(m, xhalf(m)) * c;
      if (SAFE) {
        const float mnew = fmaxf(fmaxf(ref[rb], m), kLowest);
        z[rb] *= __builtin_amdgcn_exp2f(ref[rb] - mnew);
        ref[rb] = mnew;
      } else {
        ref[rb] = m;
      }
    }
    const float nref = -ref[rb];
    float sum = 0.0f;
#pragma unroll
    for (int v = 0; v < 16; ++v) sum += __builtin_amdgcn_exp2f(fmaf(a[v], c, nref));
    z[rb] += sum;
  }
}

// The Q fragments only ever feed MFMAs, which can read their A/B operands from the accumulation
// half of the register file: pin them there so that the vector half stays free for everything the
// vector ALU touches (accumulators, exponentials, offsets).
template <int NRB>
__device__ __forceinline__ void pin_q_in_agprs(bf16x8 (&qf)[NRB][8]) {
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int s = 0; s < 8; ++s) asm volatile("" : "+a"(qf[rb][s]));
}

template <int NRB>
__device__ __forceinline__ void wave_load_frags(bf16x8 (&kf)[8], const u32x4* slot, int n, int h) {
#pragma unroll
  for (int s = 0; s < 8; ++s) kf[s] = lds_read16((unsigned)(uintptr_t)(lds_vec_ptr)slot + (unsigned)lds_chunk_index(n, 2 * s + h) * 16u, 0);
}

// Two waves fit a SIMD as soon as their registers are half of it or less, as up to four row blocks' are, and then the waves of workgroups of one,
// two or three are put two to a SIMD while others have none.  Naming a register keeps a SIMD for every wave.
template <int NRB>
__device__ __forceinline__ void one_wave_per_simd() {
  if (NRB <= 4) asm volatile("" ::: "a127");
}

// The keys a wave goes through, in the order in which they enter its ring: the sub-blocks of one chunk of a dense batch, or
// (SEG) of a segment of a ragged one, sequence after sequence.  REV: from the last sub-block down.  The ring is filled ahead
// across the sequences of a segment: while the wave changes to the queries of the next one, that one's first NST - 1
// sub-blocks are on their way.
// STREAM (see key_hints): the transfers carry the non-temporal hint, but for the last keys of a dense chunk in pass 1 (from `stream_to` on,
// 128 MB of all chunks in flight), which the memory-side cache then still has when pass 2 starts there.
template <bool REV, bool SEG, bool UNIT, bool STREAM>
struct KeyStream {
  static constexpr bool kReversed = REV, kSegment = SEG, kUnitSums = UNIT;
  const ScoreParams& p;
  const uint16_t* head;  // SEG: the KV head's keys
  const uint16_t* base;  // first key of the sequence (dense: of the chunk) that is being fetched
  int nkeys;             // its keys
  int sub, seq, left;    // SEG: the sub-block that is fetched next, of which sequence, and how many of the segment are to come
  int stream_to;         // (STREAM, pass 1 of a chunk)
  __device__ __forceinline__ void enter(SeqRange r) {
    nkeys = uniform_i32(r.len);
    base = uniform_ptr(head + (int64_t)seq * p.k_stride_seq + (int64_t)r.start * p.k_stride_token);
  }
  // key0: the first key of the sub-block in its chunk (a segment counts them itself)
  __device__ __forceinline__ void fetch(u32x4* slot, const unsigned (&voff)[4], int key0) {
    const int first = SEG ? sub * 32 : key0;
    const bool live = SEG ? left > 0 : (REV ? key0 >= 0 : key0 < nkeys);
    if constexpr (STREAM && (REV || SEG)) {
      sub_dma<kNonTemporal>(slot, base, p.k_stride_token, first, nkeys, live, voff);
    } else if constexpr (STREAM) {
      if (key0 < stream_to) sub_dma<kNonTemporal>(slot, base, p.k_stride_token, first, nkeys, live, voff);
      else sub_dma(slot, base, p.k_stride_token, first, nkeys, live, voff);
    } else {
      sub_dma(slot, base, p.k_stride_token, first, nkeys, live, voff);
    }
    if constexpr (SEG) {
      sub += REV ? -1 : 1;
      left -= 1;
      if (left > 0 && (REV ? sub < 0 : sub > (nkeys - 1) / 32)) {
        SeqRange r;
        do {  // (a segment that goes on has another sequence with keys)
          seq += REV ? -1 : 1;
          r = seq_range(p, seq);
        } while (r.len <= 0);
        enter(r);
        sub = REV ? (nkeys - 1) / 32 : 0;
      }
    }
  }
};
// The ring is filled whether the sub-blocks exist or not (sub_dma): the waits count operations.
template <int NST, class Stream>
__device__ __forceinline__ void fill_ring(u32x4* ring, Stream& keys, const unsigned (&voff)[4], int first_sub) {
#pragma unroll
  for (int i = 0; i < NST; ++i) keys.fetch(ring + i * kSubVec, voff, (Stream::kReversed ? first_sub - i : first_sub + i) * 32);
}

// One row block of the queries into a ring slot, laid out like a sub-block of keys: row `row0` of the head and the 31 after it (rows past
// the last one repeat it; their results are dropped).
__device__ __forceinline__ void queries_dma(u32x4* slot, const ScoreParams& p, const uint16_t* qbase, int row0) {
  const int lane = fresh_lane();
  if ((p.n_pseudo & 31) == 0 && row0 + 32 <= p.rows && p.q_stride_row < ((int64_t)1 << 26)) {  // all of one query head
    const int head = uniform_i32(quotient(row0, p.inv_n_pseudo)), at = row0 - head * p.n_pseudo;
    unsigned voff[4];
    sub_dma_lane_offsets(voff, p.q_stride_row, lane);
    sub_dma(slot, uniform_ptr(qbase + (int64_t)head * p.q_stride_head + (int64_t)at * p.q_stride_row), p.q_stride_row, 0, 32, true, voff);
    return;
  }
  const int r = lane >> 4;
  const unsigned piece = (unsigned)(lane & 15) ^ (unsigned)r;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = row0 + 4 * i + r, rc = row < p.rows ? row : p.rows - 1;
    const int head = quotient(rc, p.inv_n_pseudo), at = rc - head * p.n_pseudo;
    const uint16_t* src = qbase + (int64_t)head * p.q_stride_head + (int64_t)at * p.q_stride_row + (piece ^ (4u * (i & 3))) * 8u;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)(slot + i * 64), 16, 0, 0);
  }
}
// The start of a wave of a dense launch: its queries come through the ring in front of its keys.  On exit the first sub-block lies, or
// will, in ring slot `slot`, and the NST - 1 after it are under way.  Loaded as fragments, 32 bytes of each of 32 rows at a time, the queries
// of the four waves of a compute unit kept its address unit busy for some 7 us at the start of every chunk.  Both passes with the
// rotation, us: 8 layers, 256 rows, 4096 keys 68.2 -> 58.8; 32 layers of 4 KV heads, 256 rows, 1104 keys 50.0 -> 44.4; one layer, 256
// rows, 2 prompts of 24498 keys, extended 87.4 -> 81.4; 64 prompts of 512 keys 1602 -> 1579; C2's one chunk to a wave 1.000.  (The sequences of a
// segment, whose ring is running: no faster so, 757 -> 764 for 16 prompts of 200..2500 keys, 128 rows; nor two row blocks: 16 rows, 8
// prompts of 9783 keys 55.1 -> 56.8, 64 rows, 8 of 5000 as fast; nor short chunks, see few_keys.  Those load them as fragments.)
template <int NRB, int NST, class Stream>
__device__ __forceinline__ void start_with_queries(const ScoreParams& p, u32x4* ring, int& slot, Stream& keys, bf16x8 (&qf)[NRB][8],
                                                   const uint16_t* qbase, int gbase, const unsigned (&voff)[4], int first_sub, int n,
                                                   int h) {
  auto item = [&](int i) {  // number i of what goes through the ring
    if (i < NRB) queries_dma(ring + i % NST * kSubVec, p, qbase, gbase + i * 32);
    else keys.fetch(ring + i % NST * kSubVec, voff, (Stream::kReversed ? first_sub - (i - NRB) : first_sub + (i - NRB)) * 32);
  };
#pragma unroll
  for (int i = 0; i < NST; ++i) item(i);
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    wait_ring_full<NST>();
    wave_load_frags<NRB>(qf[rb], ring + rb % NST * kSubVec, n, h);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // they are out of their slot
    item(rb + NST);
  }
  if (NRB > 4) pin_q_in_agprs<NRB>(qf);
  slot = NRB % NST;
}

// Pass 1 of `count` sub-blocks of one sequence (or chunk), from number first_sub on, against row group `group` of `head` =
// layer * n_kv_heads + KV head.  kbase: its first key, nkeys: its keys; `start`: the first of this wave.  kf, slot and keys: as
// in wave_walk.  FRAGS: the queries come as fragments, beside a ring that the caller has filled (else through it, see
// start_with_queries).  The (reference, sum) pairs go to outp.
template <int NRB, int NST, bool FRAGS, class Stream>
__device__ __forceinline__ void pass1_piece(const ScoreParams& p, u32x4* ring, int& slot, Stream& keys, bf16x8 (&kf)[8],
                                            bf16x8 (&qf)[NRB][8], const uint16_t* qbase, const uint16_t* kbase, int first_sub,
                                            int count, int nkeys, int gbase, const unsigned (&voff)[4], bool start,
                                            float2* outp) {
  const int lane = fresh_lane(), n = lane & 31, h = lane >> 5;
  if constexpr (FRAGS) {
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) frag_from_q(qf[rb], p, qbase, gbase + rb * 32 + n, h);
    if (NRB > 4) pin_q_in_agprs<NRB>(qf);
  } else {
    start_with_queries<NRB, NST>(p, ring, slot, keys, qf, qbase, gbase, voff, first_sub, n, h);
  }
  if (start) {
    wait_ring_full<NST>();
    wave_load_frags<NRB>(kf, ring + slot * kSubVec, n, h);
  }
  // the fragments in kf have been used: their slot takes the sub-block NST ahead, and the next one's fragments follow
  auto advance = [&](int sub) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (they are out of their slot)
    keys.fetch(ring + slot * kSubVec, voff, (sub + NST) * 32);
    slot = slot + 1 == NST ? 0 : slot + 1;
    wait_ring_full<NST>();
    wave_load_frags<NRB>(kf, ring + slot * kSubVec, n, h);
  };
  float ref[NRB], z[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    ref[rb] = -INFINITY;
    z[rb] = 0.0f;
  }
  // the first sub-block the plain way: it fixes the reference logits
  wave_sub_simple<NRB, false, true>(kf, qf, p.c, ref, z, first_sub * 32, nkeys, h);
  advance(first_sub);
  const int last_sub = first_sub + count - 1, full = nkeys / 32 - first_sub - 1;  // sub-blocks of 32 keys after the first one
  const int walk = full < count - 1 ? full : count - 1;
  if (walk > 0) {
    float off[NRB], zs[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) off[rb] = -ref[rb];
    const float no_off2[1][16] = {};
    wave_walk<NRB, 1, NST>(ring, slot, keys, first_sub + 1, walk, nkeys, kf, qf, p.c, off, no_off2, zs, nullptr, voff, n, h);
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) z[rb] += zs[rb];
  }
  if (count > 1 && walk < count - 1) {  // the partial last sub-block
    wave_sub_simple<NRB, false, false>(kf, qf, p.c, ref, z, last_sub * 32, nkeys, h);
    advance(last_sub);
  }

  // a sum that is not finite means a logit sat more than ~127 binades above the reference, or that those of the first sub-block are all -inf: redo
  // the piece with a running maximum, one sub-block at a time, straight from memory
  bool bad = false;
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) bad = bad || !(z[rb] < INFINITY);
  if (__any(bad ? 1 : 0)) {
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      ref[rb] = -INFINITY;
      z[rb] = 0.0f;
    }
    for (int sub = first_sub; sub <= last_sub; ++sub) {
      const int key = sub * 32 + n < nkeys ? sub * 32 + n : nkeys - 1;  // (repeated keys are masked)
      const uint16_t* src = kbase + (int64_t)key * p.k_stride_token + 8 * h;
#pragma unroll
      for (int s = 0; s < 8; ++s) kf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(src + 16 * s));
      wave_sub_simple<NRB, true, false>(kf, qf, p.c, ref, z, sub * 32, nkeys, h);
    }
    wave_load_frags<NRB>(kf, ring + slot * kSubVec, n, h);  // (what was in kf before)
  }

  if (!Stream::kSegment) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (outp may be in the ring)
  // the two lane halves hold different keys of the same query
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    const float zz = z[rb] + xhalf(z[rb]);
    if (h == 0) outp[rb * 32 + n] = make_float2(ref[rb], zz);
  }
}

__device__ __forceinline__ const uint16_t* wave_q_base(const ScoreParams& p, int layer, int kv, int seq) {
  return p.q + (int64_t)layer * p.q_stride_layer + (int64_t)seq * p.q_stride_seq + (int64_t)kv * p.group * p.q_stride_head;
}

// Pass 1 of one chunk of a dense batch: `group` = row group, `chunk_id` = chunk along the packed key axis.  The chunk must have
// keys.  FUSED (score_fused_kernel): the chunk's (reference, sum) pairs go to the start of the wave's own ring, which is
// drained by then, instead of to global memory.  SHORT: the queries as fragments.
template <int NRB, int NST, bool UNIT, bool STREAM, bool FUSED = false, bool SHORT = false>
__device__ __forceinline__ void pass1_chunk(const ScoreParams& p, u32x4* ring, const Work& w, int chunk_id, int group, int head,
                                            bf16x8 (&qf)[NRB][8], int lane) {
  unsigned voff[4];
  sub_dma_lane_offsets(voff, p.k_stride_token, lane);
  const int layer = uniform_i32(quotient(head, p.inv_kv_heads)), kv = head - layer * p.n_kv_heads;
  const uint16_t* kbase = uniform_ptr(p.k + (int64_t)layer * p.k_stride_layer + (int64_t)w.seq * p.k_stride_seq +
                                      (int64_t)kv * p.k_stride_head + w.tok0 * p.k_stride_token);
  const int gbase = group * (NRB * 32);  // first row of this wave's row group
  KeyStream<false, false, UNIT, STREAM> keys = {p, nullptr, kbase, w.nkeys, 0, 0, 0,
                                                STREAM ? uniform_i32((int)(p.stream_share * (float)w.nkeys)) : 0};
  constexpr bool kFrags = NRB == 2 || SHORT;
  if (kFrags) fill_ring<NST>(ring, keys, voff, 0);
  bf16x8 kf[8];
  int slot = 0;
  float2* outp = FUSED ? reinterpret_cast<float2*>(ring) : p.parts + ((int64_t)head * p.max_chunks + chunk_id) * p.rows_pad + gbase;
  pass1_piece<NRB, NST, kFrags>(p, ring, slot, keys, kf, qf, wave_q_base(p, layer, kv, w.seq), kbase, 0, (w.nkeys + 31) / 32, w.nkeys,
                        gbase, voff, true, outp);
}

// Pass 1 of one segment of a ragged batch.
template <int NRB, int NST, bool STREAM>
__device__ __forceinline__ void pass1_segment(const ScoreParams& p, u32x4* ring, int segment, int group, int head,
                                              bf16x8 (&qf)[NRB][8], int lane) {
  Segment at = segment_of_wave(p, segment, false);
  if (at.left == 0) return;
  unsigned voff[4];
  sub_dma_lane_offsets(voff, p.k_stride_token, lane);
  const int layer = uniform_i32(quotient(head, p.inv_kv_heads)), kv = head - layer * p.n_kv_heads;
  const int gbase = group * (NRB * 32);
  KeyStream<false, true, true, STREAM> keys = {
      p, uniform_ptr(p.k + (int64_t)layer * p.k_stride_layer + (int64_t)kv * p.k_stride_head), nullptr, 0, at.sub, at.seq, at.left, 0};
  keys.enter(seq_range(p, at.seq));
  fill_ring<NST>(ring, keys, voff, 0);
  bf16x8 kf[8];
  int slot = 0;
  for (bool start = true;; start = false) {
    const SeqRange r = seq_range(p, at.seq);
    if (r.len > 0) {
      const int nkeys = uniform_i32(r.len), rest = (nkeys - 1) / 32 + 1 - at.sub, count = at.left < rest ? at.left : rest;
      const uint16_t* kbase = uniform_ptr(keys.head + (int64_t)at.seq * p.k_stride_seq + (int64_t)r.start * p.k_stride_token);
      pass1_piece<NRB, NST, true>(p, ring, slot, keys, kf, qf, wave_q_base(p, layer, kv, at.seq), kbase, at.sub, count, nkeys, gbase,
                            voff, start,
                            p.parts + ((int64_t)head * p.max_chunks + at.seq + segment) * p.rows_pad + gbase);
      at.left -= count;
      if (at.left == 0) break;
    }
    at.seq += 1;
    at.sub = 0;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Which (chunk, row group) a wave of a dense launch works on.  The waves of a workgroup take p.wg_groups row groups of
// the same chunk side by side, then the next chunk: the row groups of a chunk read the same keys at the same time, and
// in one compute unit the second reader finds them in L2 instead of fetching them through the fabric again.
struct WaveSlot {
  int chunk, group;
};
__device__ __forceinline__ WaveSlot wave_slot(const ScoreParams& p, int wave_id) {
  const int waves = (int)(blockDim.x >> 6), gpw = p.wg_groups, cpw = waves / gpw;
  WaveSlot s;
  s.chunk = uniform_i32((int)blockIdx.x * cpw + wave_id / gpw);
  s.group = uniform_i32((int)blockIdx.y * gpw + wave_id % gpw);
  return s;
}

// The grid names the items, one per wave: (chunk, row group, layer x KV head).  SEG (ragged batches, whose lengths
// the host does not know): a segment of the packed key axis in the place of the chunk.  SHORT: see few_keys.
template <int NRB, bool SEG, bool UNIT, bool SHORT, bool STREAM, int NST>
__global__ __launch_bounds__(64 * kWavesPerGroup, 1) void score_wave_pass1_kernel(ScoreParams p) {
  extern __shared__ u32x4 rings[];
  one_wave_per_simd<NRB>();
  const int wave_id = uniform_i32((int)(threadIdx.x >> 6));
  u32x4* ring = rings + wave_id * (wave_lds(NST) / 16);
  const int lane = threadIdx.x & 63;
  bf16x8 qf[NRB][8];
  const WaveSlot slot = wave_slot(p, wave_id);
  if constexpr (SEG) {
    pass1_segment<NRB, NST, STREAM>(p, ring, slot.chunk, slot.group, (int)blockIdx.z, qf, lane);
  } else {
    const Work w = locate_uniform(p, slot.chunk);
    if (w.nkeys == 0) return;
    pass1_chunk<NRB, NST, UNIT, STREAM, false, SHORT>(p, ring, w, slot.chunk, slot.group, (int)blockIdx.z, qf, lane);
  }
}

// Pass 2 of `count` sub-blocks of one sequence (or chunk), from number first_sub down (arguments as pass1_piece).  lse: of the
// sequence's first row, out: where the sums of its first key go.  LOADED: the query fragments are in registers and off2 is
// filled.
template <int NRB, int NST, bool LOADED, bool FRAGS, class Stream>
__device__ __forceinline__ void pass2_piece(const ScoreParams& p, u32x4* ring, int& slot, Stream& keys, bf16x8 (&kf)[8],
                                            bf16x8 (&qf)[NRB][8], float (&off2)[NRB][16], const uint16_t* qbase,
                                            const float* lse, int first_sub, int count, int nkeys, int gbase,
                                            const unsigned (&voff)[4], bool start, float* out) {
  const int lane = fresh_lane(), n = lane & 31, h = lane >> 5;
  if constexpr (!LOADED) {
    if constexpr (FRAGS) {
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) frag_from_q(qf[rb], p, qbase, gbase + rb * 32 + n, h);
      if (NRB > 4) pin_q_in_agprs<NRB>(qf);
    } else {
      start_with_queries<NRB, NST>(p, ring, slot, keys, qf, qbase, gbase, voff, first_sub, n, h);
    }
    // -lse2 of the rows this lane's accumulator registers hold; -inf for padding rows, which then add 0
    if ((reinterpret_cast<uintptr_t>(lse) & 15) == 0 && (p.rows & 3) == 0) {
      // the four rows of an accumulator quad are consecutive: one 16-byte load each
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int row = gbase + rb * 32 + acc_row(4 * b, h);
          const float4 v = row < p.rows ? *reinterpret_cast<const float4*>(lse + row) : make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
          off2[rb][4 * b] = -v.x;
          off2[rb][4 * b + 1] = -v.y;
          off2[rb][4 * b + 2] = -v.z;
          off2[rb][4 * b + 3] = -v.w;
        }
    } else {
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = gbase + rb * 32 + acc_row(v, h);
          off2[rb][v] = row < p.rows ? -lse[row] : -INFINITY;
        }
    }
  }
  if (start) {
    wait_ring_full<NST>();
    wave_load_frags<NRB>(kf, ring + slot * kSubVec, n, h);
  }
  float unused_off[NRB], unused_acc[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) unused_off[rb] = 0.0f;
  wave_walk<NRB, 2, NST>(ring, slot, keys, first_sub, count, nkeys, kf, qf, p.c, unused_off, off2, unused_acc, out, voff, n, h);
}
__device__ __forceinline__ const float* wave_lse(const ScoreParams& p, int layer, int kv, int seq) {
  return p.lse2 + (((int64_t)layer * p.batch + seq) * p.n_q_heads + (int64_t)kv * p.group) * p.n_pseudo;
}
// The column sums of a row group of a head.  With several row groups each writes its own plane (group 0 straight into the
// result); a small kernel adds the others onto it.
__device__ __forceinline__ float* wave_plane(const ScoreParams& p, int head, int group) {
  float* plane = group == 0 ? p.scores : p.partial + (int64_t)(group - 1) * p.n_layers * p.n_kv_heads * p.total_tokens;
  return plane + (int64_t)head * p.total_tokens;
}

// Pass 2 of one chunk of a dense batch (arguments as pass1_chunk).  FUSED (score_fused_kernel): the query fragments are still in
// registers from pass 1 and the caller has filled off2.
template <int NRB, int NST, bool SHORT, bool STREAM, bool FUSED = false>
__device__ __forceinline__ void pass2_chunk(const ScoreParams& p, u32x4* ring, const Work& w, int group, int head,
                                            bf16x8 (&qf)[NRB][8], float (&off2)[NRB][16], int lane) {
  unsigned voff[4];
  sub_dma_lane_offsets(voff, p.k_stride_token, lane);
  const int layer = uniform_i32(quotient(head, p.inv_kv_heads)), kv = head - layer * p.n_kv_heads;
  const uint16_t* kbase = uniform_ptr(p.k + (int64_t)layer * p.k_stride_layer + (int64_t)w.seq * p.k_stride_seq +
                                      (int64_t)kv * p.k_stride_head + w.tok0 * p.k_stride_token);
  float* out = const_cast<float*>(uniform_ptr(wave_plane(p, head, group) + w.tok0));
  const int nsubs = (w.nkeys + 31) / 32;
  KeyStream<true, false, false, STREAM> keys = {p, nullptr, kbase, w.nkeys, 0, 0, 0, 0};
  constexpr bool kFrags = NRB == 2 || SHORT;
  if (FUSED || kFrags) fill_ring<NST>(ring, keys, voff, nsubs - 1);
  bf16x8 kf[8];
  int slot = 0;
  pass2_piece<NRB, NST, FUSED, kFrags>(p, ring, slot, keys, kf, qf, off2, wave_q_base(p, layer, kv, w.seq), wave_lse(p, layer, kv, w.seq),
                               nsubs - 1, nsubs, w.nkeys, group * (NRB * 32), voff, true, out);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Pass 2 of one segment of a ragged batch, from its last sub-block to its first.
template <int NRB, int NST, bool STREAM>
__device__ __forceinline__ void pass2_segment(const ScoreParams& p, u32x4* ring, int segment, int group, int head,
                                              bf16x8 (&qf)[NRB][8], float (&off2)[NRB][16], int lane) {
  Segment at = segment_of_wave(p, segment, true);
  if (at.left == 0) return;
  unsigned voff[4];
  sub_dma_lane_offsets(voff, p.k_stride_token, lane);
  const int layer = uniform_i32(quotient(head, p.inv_kv_heads)), kv = head - layer * p.n_kv_heads;
  KeyStream<true, true, true, STREAM> keys = {
      p, uniform_ptr(p.k + (int64_t)layer * p.k_stride_layer + (int64_t)kv * p.k_stride_head), nullptr, 0, at.sub, at.seq, at.left, 0};
  keys.enter(seq_range(p, at.seq));
  fill_ring<NST>(ring, keys, voff, 0);
  bf16x8 kf[8];
  int slot = 0;
  for (bool start = true;; start = false) {
    const SeqRange r = seq_range(p, at.seq);
    if (r.len > 0) {
      const int nkeys = uniform_i32(r.len);
      if (!start) at.sub = (nkeys - 1) / 32;
      const int count = at.left < at.sub + 1 ? at.left : at.sub + 1;
      // (the sums of a piece go out relative to its first key: their offsets are 32 bits wide)
      const int key0 = (at.sub + 1 - count) * 32, keys_here = nkeys - key0 < count * 32 ? nkeys - key0 : count * 32;
      float* out = const_cast<float*>(uniform_ptr(wave_plane(p, head, group) + r.start + key0));
      pass2_piece<NRB, NST, false, true>(p, ring, slot, keys, kf, qf, off2, wave_q_base(p, layer, kv, at.seq),
                                   wave_lse(p, layer, kv, at.seq), count - 1, count, keys_here, group * (NRB * 32), voff, start, out);
      at.left -= count;
      if (at.left == 0) break;
    }
    at.seq -= 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// (SEG as in pass 1.)  Heads and, inside a chunk or segment, the keys are walked in the opposite order to pass 1: what pass 1
// read last (the ends of the chunks in flight, the heads of the last round) is still in the 256 MB memory-side cache
// when pass 2 starts.
template <int NRB, bool SEG, bool SHORT, bool STREAM, int NST>
__global__ __launch_bounds__(64 * kWavesPerGroup, 1) void score_wave_pass2_kernel(ScoreParams p) {
  extern __shared__ u32x4 rings[];
  one_wave_per_simd<NRB>();
  const int wave_id = uniform_i32((int)(threadIdx.x >> 6));
  u32x4* ring = rings + wave_id * (wave_lds(NST) / 16);
  const int lane = threadIdx.x & 63;
  bf16x8 qf[NRB][8];
  float off2[NRB][16];
  const WaveSlot slot = wave_slot(p, wave_id);
  const int head = (int)(gridDim.z - 1 - blockIdx.z);
  if constexpr (SEG) {
    pass2_segment<NRB, NST, STREAM>(p, ring, slot.chunk, slot.group, head, qf, off2, lane);
  } else {
    const Work w = locate_uniform(p, slot.chunk);
    if (w.nkeys == 0) return;
    pass2_chunk<NRB, NST, SHORT, STREAM>(p, ring, w, slot.group, head, qf, off2, lane);
  }
}

// Both passes in one launch, for dense batches whose (layer, sequence, KV head) problems are one workgroup each: at
// most 256 query rows (one row group) and as many chunks per sequence as the workgroup has waves (1 to 4).  A wave walks its
// chunk forward for pass 1, the waves of the workgroup exchange their (reference, sum) pairs through LDS (their rings
// are drained then) and each merges them -- the arithmetic of score_combine_kernel, chunk by chunk in the same order,
// so lse2 and with it the scores have the bits of the three-kernel path -- and walks its chunk backward for pass 2 with
// the query fragments still in registers.  What this saves is everything between the passes: a kernel boundary at
// which every wave of the chip waits for the slowest, the combine kernel, the second placement of the workgroups and
// the second read of the queries.  lse2 is not written anywhere.
// SHORT: see few_keys.
template <int NRB, bool UNIT, bool SHORT, bool STREAM, int NST>
__global__ __launch_bounds__(64 * kWavesPerGroup, 1) void score_fused_kernel(ScoreParams p) {
  extern __shared__ u32x4 rings[];
  one_wave_per_simd<NRB>();
  const int wave_id = uniform_i32((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
  u32x4* ring = rings + wave_id * (wave_lds(NST) / 16);
  const int lane = threadIdx.x & 63, h = lane >> 5;
  bf16x8 qf[NRB][8];
  const int chunk = uniform_i32((int)blockIdx.x * waves + wave_id);  // blockIdx.x is the sequence
  const int head = (int)blockIdx.z;
  const Work work = locate_uniform(p, chunk);
  pass1_chunk<NRB, NST, UNIT, STREAM, true, SHORT>(p, ring, work, chunk, 0, head, qf, lane);
  __syncthreads();
  // lse2 of rows lane, lane + 64, ...: every wave merges all chunks itself
  constexpr int kRowsPerLane = (NRB * 32 + 63) / 64;  // (an odd number of row blocks: the last rows are no one's)
  float lse[kRowsPerLane];
#pragma unroll
  for (int r = 0; r < kRowsPerLane; ++r) {
    const int row = r * 64 + lane;
    float m = -INFINITY;
    for (int w = 0; w < waves; ++w) {
      const float2 v = reinterpret_cast<const float2*>(rings + w * (wave_lds(NST) / 16))[row];
      if (v.y > 0.0f) m = fmaxf(m, v.x + log2f(v.y));
    }
    float sum = 0.0f;
    for (int w = 0; w < waves; ++w) {
      const float2 v = reinterpret_cast<const float2*>(rings + w * (wave_lds(NST) / 16))[row];
      if (v.y > 0.0f) sum += exp2f(v.x + log2f(v.y) - m);
    }
    lse[r] = (sum > 0.0f) ? m + log2f(sum) : 0.0f;
  }
  __syncthreads();  // everybody has read everybody's pairs: the rings may be overwritten
  // -lse2 of the rows this lane's accumulator registers hold, through the wave's own ring (rows beyond the head's: -inf,
  // they then add 0)
  float* mine = reinterpret_cast<float*>(ring);
#pragma unroll
  for (int r = 0; r < kRowsPerLane; ++r) mine[r * 64 + lane] = (r * 64 + lane) < p.rows ? -lse[r] : -INFINITY;
  asm volatile("" ::: "memory");  // (the reads below are of another type than the writes above)
  float off2[NRB][16];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const float4 v = *reinterpret_cast<const float4*>(mine + rb * 32 + acc_row(4 * b, h));
      off2[rb][4 * b] = v.x;
      off2[rb][4 * b + 1] = v.y;
      off2[rb][4 * b + 2] = v.z;
      off2[rb][4 * b + 3] = v.w;
    }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // off2 is out of the ring before pass 2 refills it
  pass2_chunk<NRB, NST, false, STREAM, true>(p, ring, work, 0, head, qf, off2, lane);
}

// The causal block of the pseudo tokens' own keys (Sec. 4.1: they are prefilled in-sequence): a wave scores one block of 32 query rows
// against the n_pseudo pseudo keys, row i = row % n_pseudo seeing keys 0..i, and folds the result into lse2 in place.  The four waves of a workgroup have row blocks of the same (sequence,
// layer, KV head) and share its keys, which come into LDS in whole rows, a sub-block to a wave; the queries too, or, FRAGS, straight
// from memory: up to two row blocks, whose loads keep no one waiting and whose LDS would keep other workgroups out.  Up to sixteen waves of
// a compute unit hide each other's trips to memory.  One launch, us, one wave for up to eight row blocks -> this: 4096 sequences x heads of 128
// rows 34.9 -> 30.9, of 256 89.1 -> 59.0; 256 of 128 rows 6.4 -> 4.9; of 64 rows 5.7 -> 5.1 (queries through LDS 5.0), 4096 of them 27.0 ->
// 25.3 (25.6); 8 of one row 3.6 -> 3.4 (3.8), 4096 of them 7.0 -> 5.4 (8.0).
struct PseudoParams {
  const uint16_t* kp;
  int64_t stride_layer, stride_seq, stride_head, stride_row;
};

constexpr int kPseudoWaves = 4, kPseudoSubs = 4;  // most row blocks of a workgroup, sub-blocks of keys that lie in LDS at a time
template <bool FRAGS>
__global__ __launch_bounds__(64 * kPseudoWaves, 4) void score_pseudo_kernel(ScoreParams p, PseudoParams pp) {
  extern __shared__ u32x4 pseudo_area[];  // the queries' row blocks (not FRAGS), then the keys
  const int seq = blockIdx.x;
  const int layer = uniform_i32(quotient((int)blockIdx.z, p.inv_kv_heads)), kv = (int)blockIdx.z - layer * p.n_kv_heads;
  const int wave = uniform_i32((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const uint16_t* qbase = p.q + (int64_t)layer * p.q_stride_layer + (int64_t)seq * p.q_stride_seq +
                          (int64_t)kv * p.group * p.q_stride_head;
  const uint16_t* kbase = uniform_ptr(pp.kp + (int64_t)layer * pp.stride_layer + (int64_t)seq * pp.stride_seq +
                                      (int64_t)kv * pp.stride_head);
  float* lse = p.lse2 + (((int64_t)layer * p.batch + seq) * p.n_q_heads + (int64_t)kv * p.group) * p.n_pseudo;
  const int row0 = ((int)blockIdx.y * waves + wave) * 32, row = row0 + n, rc = row < p.rows ? row : p.rows - 1;
  const bool mine = row0 < p.rows;  // (a wave without rows brings in keys)
  u32x4 *queries = pseudo_area + wave * kSubVec, *keys = pseudo_area + (FRAGS ? 0 : waves * kSubVec);
  bf16x8 qf[1][8];
  if (mine) {
    if constexpr (FRAGS) frag_from_q(qf[0], p, qbase, row, h);
    else queries_dma(queries, p, qbase, row0);
  }
  const int last_key[1] = {rc - quotient(rc, p.inv_n_pseudo) * p.n_pseudo};
  const float old = lse[rc];
  float ref[1] = {-INFINITY}, z[1] = {0.0f};
  unsigned voff[4];
  sub_dma_lane_offsets(voff, pp.stride_row, lane);
  const int nsubs = (p.n_pseudo + 31) / 32;
  for (int sub0 = 0; sub0 < nsubs; sub0 += kPseudoSubs) {
    const int subs = nsubs - sub0 < kPseudoSubs ? nsubs - sub0 : kPseudoSubs;
    if (sub0 != 0) __syncthreads();  // everybody is done with the keys before these
    for (int sub = wave; sub < subs; sub += waves)  // (rows past the last one arrive as zeros)
      sub_dma(keys + sub * kSubVec, kbase, pp.stride_row, (sub0 + sub) * 32, p.n_pseudo, true, voff);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (!mine) continue;
    if (!FRAGS && sub0 == 0) wave_load_frags<1>(qf[0], queries, n, h);
    for (int sub = 0; sub < subs; ++sub) {
      const int key0 = (sub0 + sub) * 32;
      if (!__any(last_key[0] >= key0)) continue;
      bf16x8 kf[8];
      wave_load_frags<1>(kf, keys + sub * kSubVec, n, h);
      wave_sub_simple<1, true, false, true>(kf, qf, p.c, ref, z, key0, p.n_pseudo, h, last_key);
    }
  }
  const float zz = z[0] + xhalf(z[0]);
  if (mine && h == 0 && row < p.rows) {
    const float block = ref[0] + log2f(zz);  // log2 of the block's sum; zz >= 1, or 0: the logits that the row sees are all -inf
    const float m = fmaxf(old, block);
    lse[row] = m + log2f(__builtin_amdgcn_exp2f(old - m) + __builtin_amdgcn_exp2f(block - m));
  }
}

// ---------------------------------------------------------------------------------------------
// The tile form of the passes: one workgroup = a tile of p.chunk_keys (32 to 256) keys of one (layer, sequence, KV head) x all its
// query rows.  For calls that are bound by latency (make_score_plan says which, and how many keys a tile has): keys and queries are
// brought into LDS once, in whole rows, by all waves together, and a wave works on one row block and its share of the
// sub-blocks, so that a call of a few thousand keys still has a workgroup for every compute unit and each wave a chain of one to four
// (sub-block, row block) units.  Operands loaded straight from memory into the layout of the matrix instructions (32 bytes of
// each of 32 rows per load) cost the queries more than everything else in the kernel.
// ---------------------------------------------------------------------------------------------
constexpr int kTileWaves = 8;
constexpr int kTileThreads = 64 * kTileWaves;
// `sums`: and the column sums of its row blocks, in pass 2
constexpr int tile_lds(int chunk_keys, int row_blocks, bool stage_q, bool sums) {
  return chunk_keys * kHeadDim * 2 +
         (row_blocks < kTileWaves ? row_blocks : kTileWaves) * ((stage_q ? kSubBytes : 0) + (sums ? chunk_keys * (int)sizeof(float) : 0));
}

// Which tile a workgroup works on: the KV heads of a chunk are neighbours in the grid (in the packed layout they share
// the rows of K), then the chunks, then the layers; pass 2 (`reversed`) walks layers and chunks from the far end.
struct Tile {
  int layer, kv, chunk;
};
__device__ __forceinline__ Tile tile_of_workgroup(const ScoreParams& p, bool reversed) {
  Tile t;
  const int c = uniform_i32(quotient((int)blockIdx.x, p.inv_kv_heads));
  t.kv = (int)blockIdx.x - c * p.n_kv_heads;
  t.chunk = reversed ? p.max_chunks - 1 - c : c;
  t.layer = (int)(reversed ? gridDim.z - 1 - blockIdx.z : blockIdx.z);
  return t;
}

// How the waves of a workgroup share out the row blocks and sub-blocks: wave = part * rbs + row block, a part being every
// parts-th sub-block.  (Waves past the last part only bring in keys and queries.)  Where the queries do not go through LDS (STAGED
// is false; tiles of kTileKeys) a wave takes all sub-blocks: it would load its row block for fewer of them.
struct TileShare {
  int subs, rbs, parts, rb, part;
};
// The most parts that the eight waves make of rbs row blocks (staged).
__host__ __device__ constexpr int tile_most_parts(int rbs) { return rbs > 4 ? 1 : (rbs > 2 ? 2 : (rbs == 2 ? 4 : 8)); }
template <bool STAGED>
__device__ __forceinline__ TileShare tile_share(const ScoreParams& p, int wave, int waves) {
  TileShare s;
  const int row_blocks = p.rows_pad >> 5;
  s.subs = STAGED ? p.chunk_keys >> 5 : kTileKeys / 32;
  s.rbs = row_blocks < waves ? row_blocks : waves;
  s.rb = wave;
  s.part = 0;
  s.parts = 1;
  if (!STAGED) {
    if (wave >= s.rbs) s.part = 1;
    return s;
  }
  s.parts = tile_most_parts(s.rbs);
  s.parts = s.parts < s.subs ? s.parts : s.subs;
  while (s.rb >= s.rbs) {
    s.rb -= s.rbs;
    s.part += 1;
  }
  return s;
}

// The waves share out the transfers, 1 KB (four rows) each: first the row blocks of the queries (rows past the last one repeat
// it; their results are dropped), then the tile's keys (rows past the end of the chunk arrive as zeros, see sub_dma); with eight
// waves one transfer per wave and row block or sub-block.
template <bool STAGED>
__device__ __forceinline__ void tile_dma(u32x4* keys, u32x4* queries, const ScoreParams& p, const uint16_t* kbase,
                                         const uint16_t* qbase, int nkeys, const TileShare& s, int wave, int waves, int lane) {
  const int r = lane >> 4;
  const unsigned piece = (unsigned)(lane & 15) ^ (unsigned)r;
  for (int i = 0; STAGED && i < s.rbs; ++i) {
    const int row = i * 32 + 4 * wave + r, rc = row < p.rows ? row : p.rows - 1;
    const int head = quotient(rc, p.inv_n_pseudo), at = rc - head * p.n_pseudo;
    const uint16_t* src = qbase + (int64_t)head * p.q_stride_head + (int64_t)at * p.q_stride_row + (piece ^ (4u * (unsigned)(wave & 3))) * 8u;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)(queries + i * kSubVec + wave * 64), 16, 0, 0);
  }
  const int64_t stride_b = p.k_stride_token * 2;
  for (int x = wave; x < s.subs * 8; x += waves) {
    const int row = 4 * x;
    const bool live = row < nkeys;
    const char* base = reinterpret_cast<const char*>(kbase) + (live ? (int64_t)row * stride_b : (int64_t)0);
    const int64_t span = (int64_t)(nkeys - row - 1) * stride_b + kHeadDim * 2;
    const unsigned records = !live ? 0u : (span > (int64_t)0xFFFFFFFFll ? 0xFFFFFFFFu : (unsigned)span);
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, (int)records, 0x00020000);
    const unsigned voff = (unsigned)r * (unsigned)stride_b + (piece ^ (4u * ((unsigned)x & 3u))) * 16u;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(keys + x * 64), 16, (int)voff, 0, 0, 0);
  }
}
// Until all but the last `newer` sub-blocks of the tile have landed, for the whole workgroup.
__device__ __forceinline__ void tile_wait(int newer) {
  switch (newer) {
    case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    case 1: asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); break;
    case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
    case 3: asm volatile("s_waitcnt vmcnt(3)" ::: "memory"); break;
    case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
    case 5: asm volatile("s_waitcnt vmcnt(5)" ::: "memory"); break;
    case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(7)" ::: "memory"); break;
  }
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ const uint16_t* tile_q_base(const ScoreParams& p, const Tile& t, int seq) {
  return p.q + (int64_t)t.layer * p.q_stride_layer + (int64_t)seq * p.q_stride_seq +
         (int64_t)t.kv * p.group * p.q_stride_head;
}
__device__ __forceinline__ const uint16_t* tile_k_base(const ScoreParams& p, const Tile& t, const Work& w) {
  return uniform_ptr(p.k + (int64_t)t.layer * p.k_stride_layer + (int64_t)w.seq * p.k_stride_seq +
                     (int64_t)t.kv * p.k_stride_head + w.tok0 * p.k_stride_token);
}

// Pass 1 with a running maximum.  STAGED: U sub-blocks of a wave at a time, parts apart, as they arrive (two_at_a_time); else 64 keys at a
// time, a wave's next row block loaded while it finishes the one before.
template <bool STAGED, int U>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(!STAGED ? 5 : (U == 1 ? 4 : 2)))) void score_tile_pass1_kernel(ScoreParams p) {
  extern __shared__ u32x4 tile_area[];
  __shared__ float2 sums[STAGED ? kTileWaves : 1][32];
  touch_args<sizeof(ScoreParams)>();
  const Tile t = tile_of_workgroup(p, false);
  const Work w = locate_uniform(p, t.chunk);
  if (w.nkeys == 0) return;  // (the same for the whole workgroup)
  const int wave = uniform_i32((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const TileShare s = tile_share<STAGED>(p, wave, waves);
  u32x4 *keys = tile_area, *queries = tile_area + s.subs * kSubVec;
  const uint16_t* qbase = tile_q_base(p, t, w.seq);
  tile_dma<STAGED>(keys, queries, p, tile_k_base(p, t, w), qbase, w.nkeys, s, wave, waves, lane);
  const int row_blocks = p.rows_pad / 32;
  float* outp = p.tile_parts + (((int64_t)t.layer * p.n_kv_heads + t.kv) * p.max_chunks + t.chunk) * p.rows_pad;
  bf16x8 qf[8];
  if constexpr (!STAGED) {
    frag_from_q(qf, p, qbase, wave * 32 + n, h);
    tile_wait(0);
    for (int rb = wave; rb < row_blocks; rb += waves) {
      float ref = kLowest, z[2] = {0.0f, 0.0f};
#pragma unroll 1
      for (int half = 0; half < kTileKeys / 64; ++half) {
        f32x16 a[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          bf16x8 kf[8];
          if (u == 1) __builtin_amdgcn_sched_barrier(0);
          wave_load_frags<1>(kf, keys + (2 * half + u) * kSubVec, n, h);
          a[u] = f32x16{0};
#pragma unroll
          for (int e = 0; e < 8; ++e) a[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[e], qf[e], a[u], 0, 0, 0);
        }
        const int first = half * 64;
        if (w.nkeys < first + 64) {
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v)
              if (u * 32 + acc_row(v, 0) >= w.nkeys - first - 4 * h) a[u][v] = -INFINITY;
        }
        float m = a[0][0];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int v = 0; v < 16; ++v) m = fmaxf(m, a[u][v]);
        const float mnew = fmaxf(ref, max_halves(m) * p.c);
        const float scale = __builtin_amdgcn_exp2f(ref - mnew);
        z[0] *= scale;
        z[1] *= scale;
        ref = mnew;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int v = 0; v < 16; ++v) z[v & 1] += __builtin_amdgcn_exp2f(fmaf(a[u][v], p.c, -mnew));
      }
      if (rb + waves < row_blocks) frag_from_q(qf, p, qbase, (rb + waves) * 32 + n, h);
      const float both = sum_halves(z[0] + z[1]);
      if (h == 0) outp[rb * 32 + n] = both > 0.0f ? ref + log2f(both) : -INFINITY;
    }
    return;
  }
  for (int rb0 = 0; rb0 < row_blocks; rb0 += s.rbs) {  // (one trip up to eight row blocks)
    const int rb = rb0 + s.rb;
    const bool mine = s.part < s.parts && rb < row_blocks;
    if (rb0 != 0 && mine) frag_from_q(qf, p, qbase, rb * 32 + n, h);
    float ref = kLowest, z[2] = {0.0f, 0.0f};
    const int step = U * s.parts;
#pragma unroll 1
    for (int sub0 = 0; sub0 < s.subs; sub0 += step) {
      if (rb0 == 0) tile_wait(s.subs - sub0 - step);
      if (rb0 == 0 && sub0 == 0 && mine) wave_load_frags<1>(qf, queries + s.rb * kSubVec, n, h);
      const int first = (sub0 + s.part) * 32;
      if (!mine || first >= w.nkeys) continue;
      bf16x8 kf[U][8];
      f32x16 a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        wave_load_frags<1>(kf[u], keys + (sub0 + s.part + u * s.parts) * kSubVec, n, h);
        a[u] = f32x16{0};
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u][e], qf[e], a[u], 0, 0, 0);
      if (w.nkeys < first + (U - 1) * s.parts * 32 + 32) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (acc_row(v, 0) >= w.nkeys - first - u * s.parts * 32 - 4 * h) a[u][v] = -INFINITY;
      }
      float m = a[0][0];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < 16; ++v) m = fmaxf(m, a[u][v]);
      const float mnew = fmaxf(ref, max_halves(m) * p.c);
      const float scale = __builtin_amdgcn_exp2f(ref - mnew);
      z[0] *= scale;
      z[1] *= scale;
      ref = mnew;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < 16; ++v) z[v & 1] += __builtin_amdgcn_exp2f(fmaf(a[u][v], p.c, -mnew));
    }
    const float both = sum_halves(z[0] + z[1]);
    if (s.parts == 1) {
      if (h == 0 && mine) outp[rb * 32 + n] = both > 0.0f ? ref + log2f(both) : -INFINITY;
      continue;
    }
    // the parts of a row block in order (a part without keys has no sum); at most four row blocks: one trip
    if (h == 0 && mine) sums[wave][n] = make_float2(ref, both);
    __syncthreads();
    if (threadIdx.x < s.rbs * 32) {
      const int block = (int)threadIdx.x >> 5;
      float m = -INFINITY, sum = 0.0f;
      for (int i = 0; i < s.parts; ++i) m = fmaxf(m, sums[i * s.rbs + block][n].x);
      for (int i = 0; i < s.parts; ++i) {
        const float2 v = sums[i * s.rbs + block][n];
        sum = fmaf(v.y, __builtin_amdgcn_exp2f(v.x - m), sum);
      }
      outp[threadIdx.x] = sum > 0.0f ? m + log2f(sum) : -INFINITY;
    }
  }
}

// Pass 2: a lane's column sums over the rows of its wave, then over the row blocks in order through LDS.
// MERGE: lse2 is not read but formed from the partials of pass 1, by every workgroup for itself, with the arithmetic of
// score_combine_kernel in its order (same bits), instead of a launch of 3 to 4 us.
// Not STAGED: calls of several workgroups to a compute unit; four fit (the column sums lie behind the keys, as large as the launch needs
// them; 96 registers for workgroups of five waves), and queries and lse2 are asked for with the keys.  Pass 2, ragged, us: 16 layers, 64
// rows, 12355 keys 105.2 -> 101.6; 2 layers, 32 rows, 74770 keys 70.5 -> 68.8.
constexpr int kMergeRuns = 4;                                    // runs of kCombineRun chunks a thread holds
constexpr int kMergeMaxRows = kTileThreads;
// How many chunks per sequence the threads of a workgroup can merge (0: more rows than threads).
__host__ __device__ constexpr int tile_merge_chunks(int rows_pad) {
  return rows_pad > kTileThreads ? 0 : kTileThreads / rows_pad * kMergeRuns * kCombineRun < kCombineClasses * kCombineRun
                                           ? kTileThreads / rows_pad * kMergeRuns * kCombineRun
                                           : kCombineClasses * kCombineRun;
}
template <bool MERGE, bool STAGED, int U>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(!STAGED ? 5 : (U == 1 ? 4 : 2)))) void score_tile_pass2_kernel(ScoreParams p) {
  extern __shared__ u32x4 tile_area[];
  __shared__ __align__(16) float neg_lse[MERGE ? kMergeMaxRows : 4];
  __shared__ float merge_max[MERGE ? kMergeMaxRows : 1], merge_sum[MERGE ? kMergeMaxRows * kMergeRuns : 1];
  touch_args<sizeof(ScoreParams)>();
  const Tile t = tile_of_workgroup(p, true);
  const Work w = locate_uniform(p, t.chunk);
  if (w.nkeys == 0) return;  // (the same for the whole workgroup)
  const int wave = uniform_i32((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const int waves = (int)(blockDim.x >> 6);
  const TileShare s = tile_share<STAGED>(p, wave, waves);
  u32x4 *keys = tile_area, *queries = tile_area + s.subs * kSubVec;
  const int tile_keys = s.subs * 32;
  float* cols = reinterpret_cast<float*>(queries + (STAGED ? s.rbs * kSubVec : 0));  // [row block][key]
  const uint16_t* qbase = tile_q_base(p, t, w.seq);
  const float* lse =
      p.lse2 + (((int64_t)t.layer * p.batch + w.seq) * p.n_q_heads + (int64_t)t.kv * p.group) * p.n_pseudo;
  const int row_blocks = p.rows_pad / 32;
  // thread = (row, share): runs share, share + shares, ... of the sequence's chunks
  const int share = MERGE ? quotient((int)threadIdx.x, p.inv_rows_pad) : 0, row = MERGE ? (int)threadIdx.x - share * p.rows_pad : 0;
  const int shares = quotient(kTileThreads, p.inv_rows_pad);
  const int chunks = chunks_of_length(p, w.seq_len), runs = (chunks + kCombineRun - 1) / kCombineRun;
  float part[kMergeRuns][kCombineRun];
  if (MERGE) {
    const int first = t.chunk - (w.key0 >> p.chunk_shift);  // the sequence's first chunk
    const float* src = uniform_ptr(p.tile_parts + (((int64_t)t.layer * p.n_kv_heads + t.kv) * p.max_chunks + first) * p.rows_pad);
#pragma unroll
    for (int k = 0; k < kMergeRuns; ++k) {
      if (k * shares < runs) {
#pragma unroll
        for (int i = 0; i < kCombineRun; ++i) {
          const int c = (share + k * shares) * kCombineRun + i;
          part[k][i] = src[(unsigned)((c < chunks ? c : chunks - 1) * p.rows_pad + row)];
        }
      }
    }
  }
  tile_dma<STAGED>(keys, queries, p, tile_k_base(p, t, w), qbase, w.nkeys, s, wave, waves, lane);
  if (MERGE) {
    float m = -INFINITY;
#pragma unroll
    for (int k = 0; k < kMergeRuns; ++k) {
      if (k * shares < runs) {
#pragma unroll
        for (int i = 0; i < kCombineRun; ++i) {
          part[k][i] = (share + k * shares) * kCombineRun + i < chunks ? part[k][i] : -INFINITY;
          m = fmaxf(m, part[k][i]);
        }
      }
    }
    merge_max[threadIdx.x] = m;
    __syncthreads();
    if (share < shares) {
      for (int i = 0; i < shares; ++i) m = fmaxf(m, merge_max[i * p.rows_pad + row]);
#pragma unroll
      for (int k = 0; k < kMergeRuns; ++k) {
        const int run = share + k * shares;
        if (run < runs) {
          float sum = 0.0f;
#pragma unroll
          for (int i = 0; i < kCombineRun; ++i) sum += exp2f(part[k][i] - m);
          merge_sum[run * p.rows_pad + row] = sum;
        }
      }
    }
    __syncthreads();
    if (share == 0) {
      float sum = 0.0f;
      for (int k = 0; k < runs; ++k) sum += merge_sum[k * p.rows_pad + row];
      neg_lse[row] = row < p.rows ? (sum > 0.0f ? -(m + log2f(sum)) : -0.0f) : -INFINITY;
    }
    // (visible to all after the barrier below)
  }
  const bool quads = (reinterpret_cast<uintptr_t>(lse) & 15) == 0 && (p.rows & 3) == 0;
  bf16x8 qf[8];
  float off[16];
  // -lse2 of the rows this lane's accumulator registers hold; -inf for padding rows, which then add 0
  auto load_off = [&](int rb) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int row = rb * 32 + acc_row(4 * b, h);
      if (MERGE) {
        const float4 v = *reinterpret_cast<const float4*>(&neg_lse[row]);
        off[4 * b] = v.x;
        off[4 * b + 1] = v.y;
        off[4 * b + 2] = v.z;
        off[4 * b + 3] = v.w;
      } else if (quads) {  // the four rows of an accumulator quad are consecutive: one 16-byte load
        const float4 v = row < p.rows ? *reinterpret_cast<const float4*>(lse + row)
                                      : make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
        off[4 * b] = -v.x;
        off[4 * b + 1] = -v.y;
        off[4 * b + 2] = -v.z;
        off[4 * b + 3] = -v.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) off[4 * b + e] = row + e < p.rows ? -lse[row + e] : -INFINITY;
      }
    }
  };
  if (!STAGED && s.part == 0) {  // (what comes straight from memory is asked for with the tile)
    frag_from_q(qf, p, qbase, s.rb * 32 + n, h);
    load_off(s.rb);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  for (int rb0 = 0; rb0 < row_blocks; rb0 += s.rbs) {  // (one trip up to eight row blocks)
    const int rb = rb0 + s.rb;
    if (s.part >= s.parts || rb >= row_blocks) continue;
    if (rb0 != 0) frag_from_q(qf, p, qbase, rb * 32 + n, h);
    else if (STAGED) wave_load_frags<1>(qf, queries + s.rb * kSubVec, n, h);
    if (STAGED || rb0 != 0) load_off(rb);
#pragma unroll 1
    for (int sub = s.part; sub < s.subs; sub += U * s.parts) {
      bf16x8 kf[U][8];
      f32x16 a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        wave_load_frags<1>(kf[u], keys + (sub + u * s.parts) * kSubVec, n, h);
        a[u] = f32x16{0};
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[e], kf[u][e], a[u], 0, 0, 0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float z[2] = {0.0f, 0.0f};
#pragma unroll
        for (int v = 0; v < 16; ++v) z[v & 1] += __builtin_amdgcn_exp2f(fmaf(a[u][v], p.c, off[v]));
        float* col = cols + s.rb * tile_keys + (sub + u * s.parts) * 32 + n;
        const float both = sum_halves(z[0] + z[1]);
        if (h == 0) *col = rb0 == 0 ? both : *col + both;
      }
    }
  }
  __syncthreads();
  float* out = p.scores + ((int64_t)t.layer * p.n_kv_heads + t.kv) * p.total_tokens + w.tok0;
  for (int key = threadIdx.x; key < w.nkeys; key += (int)blockDim.x) {
    float sum = cols[key];
    for (int i = 1; i < s.rbs; ++i) sum += cols[i * tile_keys + key];
    out[key] = sum;
  }
}

// ---------------------------------------------------------------------------------------------
// Short prompts of dense batches: one workgroup has all keys (up to 512) and query rows (up to 256) of a (layer, sequence, KV head), which come into
// LDS once, in whole rows; both passes run out of it in one launch.  A wave works on one row block and its share of the sub-blocks, as in the
// tile form.  The waves of score_fused_kernel, one to 128 keys, each take in all the queries, and a head of 200 keys has two of them: what bounds
// calls of up to a few heads to a compute unit is that start and a wave's 32 units in a row (short_call has figures).
// MODE: both passes, or the first (lse2 out) or the second (lse2 in) alone, with the same bits.  STAGED: the queries through LDS too, which holds
// them beside all 512 keys up to two row blocks, 480 with three, 448 with four, 416, 384 and 352 with five to seven and 320 with eight.
// ---------------------------------------------------------------------------------------------
constexpr int kShortKeys = 512, kShortRows = 256;
enum { kShortBoth = 0, kShortStats = 1, kShortAccumulate = 2 };
constexpr int short_lds(int subs, int row_blocks, bool stage_q) {
  return subs * kSubBytes + row_blocks * ((stage_q ? kSubBytes : 0) + subs * 32 * (int)sizeof(float));
}
constexpr int kShortStaticLds = kTileWaves * 32 * (int)sizeof(float2) + kShortRows * (int)sizeof(float);
constexpr int kShortMostLds = 160 * 1024 - kShortStaticLds;
template <int MODE, bool STAGED>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(4))) void score_short_kernel(ScoreParams p) {
  extern __shared__ u32x4 tile_area[];
  __shared__ float2 sums[kTileWaves][32];
  __shared__ __align__(16) float neg_lse[kShortRows];
  touch_args<sizeof(ScoreParams)>();
  const int seq = (int)blockIdx.x, nkeys = p.seq_len, wave = uniform_i32((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  Tile t;
  t.layer = uniform_i32(quotient((int)blockIdx.z, p.inv_kv_heads));
  t.kv = (int)blockIdx.z - t.layer * p.n_kv_heads;
  t.chunk = 0;
  TileShare s;
  s.subs = (nkeys + 31) / 32;
  s.rbs = (p.rows + 31) / 32;
  s.parts = tile_most_parts(s.rbs);
  s.parts = s.parts < s.subs ? s.parts : s.subs;
  s.rb = wave;
  s.part = 0;
  while (s.rb >= s.rbs) {
    s.rb -= s.rbs;
    s.part += 1;
  }
  const bool mine = s.part < s.parts;  // (the other waves bring in keys and queries)
  u32x4 *keys = tile_area, *queries = tile_area + s.subs * kSubVec;
  float* cols = reinterpret_cast<float*>(queries + (STAGED ? s.rbs * kSubVec : 0));  // [row block][key]
  const int64_t tok0 = (int64_t)seq * p.seq_len;
  const uint16_t* qbase = tile_q_base(p, t, seq);
  const uint16_t* kbase = uniform_ptr(p.k + (int64_t)t.layer * p.k_stride_layer + (int64_t)seq * p.k_stride_seq +
                                      (int64_t)t.kv * p.k_stride_head + tok0 * p.k_stride_token);
  float* lse = p.lse2 + (((int64_t)t.layer * p.batch + seq) * p.n_q_heads + (int64_t)t.kv * p.group) * p.n_pseudo;
  const int row = (int)threadIdx.x;  // of the threads that look after a row
  float old = 0.0f;
  if (MODE == kShortAccumulate && row < p.rows) old = lse[row];
  bf16x8 qf[8];
  if (!STAGED && mine) frag_from_q(qf, p, qbase, s.rb * 32 + n, h);
  tile_dma<STAGED>(keys, queries, p, kbase, qbase, nkeys, s, wave, kTileWaves, lane);

  if constexpr (MODE == kShortAccumulate) {
    if (row < s.rbs * 32) neg_lse[row] = row < p.rows ? -old : -INFINITY;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  } else {
    float ref = kLowest, z[2] = {0.0f, 0.0f};
#pragma unroll 1
    for (int sub0 = 0; sub0 < s.subs; sub0 += s.parts) {
      tile_wait(s.subs - sub0 - s.parts > 0 ? s.subs - sub0 - s.parts : 0);
      if (STAGED && sub0 == 0 && mine) wave_load_frags<1>(qf, queries + s.rb * kSubVec, n, h);
      const int sub = sub0 + s.part;
      if (!mine || sub >= s.subs) continue;
      bf16x8 kf[8];
      wave_load_frags<1>(kf, keys + sub * kSubVec, n, h);
      f32x16 a = {0};
#pragma unroll
      for (int e = 0; e < 8; ++e) a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[e], qf[e], a, 0, 0, 0);
      if (nkeys < sub * 32 + 32) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (acc_row(v, 0) >= nkeys - sub * 32 - 4 * h) a[v] = -INFINITY;
      }
      float m = a[0];
#pragma unroll
      for (int v = 1; v < 16; ++v) m = fmaxf(m, a[v]);
      const float mnew = fmaxf(ref, max_halves(m) * p.c);
      const float scale = __builtin_amdgcn_exp2f(ref - mnew);
      z[0] *= scale;
      z[1] *= scale;
      ref = mnew;
#pragma unroll
      for (int v = 0; v < 16; ++v) z[v & 1] += __builtin_amdgcn_exp2f(fmaf(a[v], p.c, -mnew));
    }
    const float both = sum_halves(z[0] + z[1]);
    // (parts whose sum is no number are left out, as score_combine_kernel does; here, since a branch in the merge costs 1 us of 6; waves that are no
    // one's are not read)
    if (h == 0) sums[wave][n] = both > 0.0f ? make_float2(ref, both) : make_float2(-INFINITY, 0.0f);
    __syncthreads();
    if (row < s.rbs * 32) {
      const int block = row >> 5;
      float m = -INFINITY, sum = 0.0f;
      for (int i = 0; i < s.parts; ++i) m = fmaxf(m, sums[i * s.rbs + block][n].x);
      for (int i = 0; i < s.parts; ++i) {
        const float2 v = sums[i * s.rbs + block][n];
        sum = fmaf(v.y, __builtin_amdgcn_exp2f(v.x - m), sum);
      }
      const float l = sum > 0.0f ? m + log2f(sum) : 0.0f;
      if (MODE == kShortStats && row < p.rows) lse[row] = l;
      neg_lse[row] = row < p.rows ? -l : -INFINITY;
    }
    if constexpr (MODE == kShortStats) return;
    __syncthreads();
  }

  if (mine) {
    if (STAGED && MODE == kShortAccumulate) wave_load_frags<1>(qf, queries + s.rb * kSubVec, n, h);
    float off[16];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const float4 v = *reinterpret_cast<const float4*>(&neg_lse[s.rb * 32 + acc_row(4 * b, h)]);
      off[4 * b] = v.x;
      off[4 * b + 1] = v.y;
      off[4 * b + 2] = v.z;
      off[4 * b + 3] = v.w;
    }
#pragma unroll 1
    for (int sub = s.part; sub < s.subs; sub += s.parts) {
      bf16x8 kf[8];
      wave_load_frags<1>(kf, keys + sub * kSubVec, n, h);
      f32x16 a = {0};
#pragma unroll
      for (int e = 0; e < 8; ++e) a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[e], kf[e], a, 0, 0, 0);
      float z[2] = {0.0f, 0.0f};
#pragma unroll
      for (int v = 0; v < 16; ++v) z[v & 1] += __builtin_amdgcn_exp2f(fmaf(a[v], p.c, off[v]));
      const float both = sum_halves(z[0] + z[1]);
      if (h == 0) cols[s.rb * s.subs * 32 + sub * 32 + n] = both;
    }
  }
  __syncthreads();
  float* out = p.scores + ((int64_t)t.layer * p.n_kv_heads + t.kv) * p.total_tokens + tok0;
  if (row < nkeys) {  // (at most a key to a thread)
    float sum = cols[row];
    for (int i = 1; i < s.rbs; ++i) sum += cols[i * s.subs * 32 + row];
    out[row] = sum;
  }
}

// S = sum over row groups of their planes of column sums, in group order; group 0's plane is the
// result array itself.
__global__ void score_group_sum_kernel(const float* partial, float* scores, int64_t count, int n_groups) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count; e += stride) {
    float s = scores[e];
    for (int g = 1; g < n_groups; ++g) s += partial[(int64_t)(g - 1) * count + e];
    scores[e] = s;
  }
}

template <typename F>
int set_lds(F kernel, int bytes) { return set_max_dynamic_lds(reinterpret_cast<const void*>(kernel), bytes); }

// SIMDs of the current device (4 per compute unit); 4 if the device cannot be asked.
int simd_count() {
  static std::mutex mu;
  static int simds[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 4;
  std::lock_guard<std::mutex> lock(mu);
  if (simds[dev] == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 1;
    simds[dev] = 4 * cus;
  }
  return simds[dev];
}

// The waves of a launch per head and row group: chunks of a dense batch, segments of a ragged one.
int64_t wave_chunks(const ScorePlan& plan) { return plan.segments > 0 ? plan.segments : plan.max_chunks; }

// A launch holds fewer than 2^32 threads along an axis; with more its grid comes out short, without an error.  The sequences of a dense batch go
// through in as many launches as that takes, `threads` along the axis to each: launch(parameters of those from one on, how many).  All but the
// last launch have a multiple of four sequences, so that workgroups stay full (see group_shape).
template <typename F>
int for_sequences(const dapq_shape* s, const ScoreParams& p, int64_t threads, F launch) {
  const int64_t most = (((int64_t)1 << 32) - 1) / threads / 4 * 4;
  if (s->cu_seqlens != nullptr || s->batch <= most || p.seq_len == 0) return launch(p, (int64_t)s->batch);
  for (int64_t first = 0; first < s->batch; first += most) {
    ScoreParams part = p;
    part.q += first * p.q_stride_seq;
    part.k += first * (p.k_stride_seq + p.seq_len * p.k_stride_token);
    if (p.parts != nullptr) part.parts += first * p.chunks_per_seq * p.rows_pad;
    if (p.lse2 != nullptr) part.lse2 += first * p.n_q_heads * p.n_pseudo;
    if (p.scores != nullptr) part.scores += first * p.seq_len;
    if (p.partial != nullptr) part.partial += first * p.seq_len;
    const int rc = launch(part, s->batch - first < most ? s->batch - first : most);
    if (rc != DAPQ_OK) return rc;
  }
  return DAPQ_OK;
}

// How a launch packs its waves into workgroups: `waves` to a workgroup (kWavesPerGroup or 1), of which `groups`
// are the row groups of one chunk side by side (see wave_slot) and waves / groups consecutive chunks.
struct GroupShape {
  int waves, groups;
  dim3 grid(const ScorePlan& plan, const dapq_shape* s, int64_t seqs) const {  // `seqs` of the batch's sequences
    const int cpw = waves / groups;
    const int64_t chunks = seqs < s->batch ? wave_chunks(plan) / s->batch * seqs : wave_chunks(plan);
    return dim3((unsigned)((chunks + cpw - 1) / cpw), (unsigned)(plan.n_groups / groups), (unsigned)(s->n_layers * s->n_kv_heads));
  }
  // threads of a launch along the axis of the sequences, to each (see for_sequences)
  int64_t threads(const ScorePlan& plan, const dapq_shape* s) const { return 64 * groups * ((wave_chunks(plan) + s->batch - 1) / s->batch); }
};
GroupShape group_shape(const dapq_shape* s, const ScorePlan& plan) {
  const int groups = plan.n_groups % 4 == 0 ? 4 : (plan.n_groups % 2 == 0 ? 2 : 1);
  int chunks = kWavesPerGroup / groups;  // consecutive chunks in a workgroup: every workgroup must be full
  while (chunks > 1 && wave_chunks(plan) % chunks != 0) chunks /= 2;
  return {groups * chunks, groups};
}

// Whether the keys of a call stream: the transfers of the wave kernels carry the non-temporal hint.  Keys that the caches cannot hold until pass
// 2 reads them again are kept there to no one's use, and what they push out costs the stream more than the hint does: up to 128 rows, where the
// stream sets the pace, the passes gain a tenth, and the power that the caches do not take is worth 1 to 2 % to the others.  `reuse`: bytes of
// keys between a key's two reads (one kernel: those of the workgroups that run at a time; else all).  Without hints -> with, us, dapq_score
// of 8 KV heads a layer:
//   64 rows, MB of keys   134 64.4 -> 63.7    268 98.5 -> 98.6    403 144.9 -> 139.2    537 177.9 -> 162.9    786 274 -> 244    2147 730 -> 664
//   128 rows              134 64.6 -> 65.0    268 108.5 -> 110.8  403 161.2 -> 158.4    537 191.9 -> 183.8    786 282 -> 268    2147 767 -> 735
//   192 and 256 rows      403 to 1074 0.98 to 1.02 of the time; 2147 931 -> 932 and 1139 -> 1118
//   ragged, 128 rows      374 158.9 -> 158.0  572 234.7 -> 216.6  791 335.6 -> 303.2    2998 1161 -> 1054 (256 rows 374 1.01, 791 0.96, 2998 1.00)
//   one kernel, 32 layers, 64 rows: 64 prompts of 512 keys (134 MB at a time) 620 -> 714, 32 of 1024 (268 MB) 637 -> 700, 8 of 2048 (537 MB)
//   363 -> 342; 128 rows 757 -> 840, 763 -> 806, 378 -> 371
// Not so several row groups, whose waves find each other's keys in L2: 512 rows, 8 prompts of 4096..16384 keys 5321 -> 5625.
struct KeyHints {
  bool on;
  float share;  // of a chunk that streams in pass 1 (see KeyStream)
};
KeyHints key_hints(const dapq_shape* s, const ScorePlan& plan, bool one_kernel) {
  if (plan.tile || plan.n_groups > 1) return {false, 0.0f};
  const double all = (double)s->n_layers * s->n_kv_heads * (double)s->total_tokens * (kHeadDim * 2);
  const int64_t mean = s->total_tokens / s->batch, wave_keys = mean < plan.chunk_keys ? mean : plan.chunk_keys;
  const double at_once = (double)simd_count() * (double)wave_keys * (kHeadDim * 2), reuse = one_kernel && at_once < all ? at_once : all;
  const bool on = reuse >= (plan.row_blocks <= 4 ? 384e6 : (plan.segments > 0 ? 768e6 : 1536e6));
  constexpr double kKept = 128e6;  // half the memory-side cache
  return {on, reuse > kKept ? (float)(1.0 - kKept / reuse) : 0.0f};
}

int fill_params(const dapq_shape* s, const ScorePlan& plan, ScoreParams* p) {
  p->cu_seqlens = s->cu_seqlens;
  p->k_stride_layer = s->k_stride_layer; p->k_stride_seq = s->k_stride_seq;
  p->k_stride_head = s->k_stride_head; p->k_stride_token = s->k_stride_token;
  p->q_stride_layer = s->q_stride_layer; p->q_stride_seq = s->q_stride_seq;
  p->q_stride_head = s->q_stride_head; p->q_stride_row = s->q_stride_row;
  p->total_tokens = s->total_tokens;
  p->n_layers = s->n_layers; p->batch = s->batch; p->n_q_heads = s->n_q_heads; p->n_kv_heads = s->n_kv_heads;
  p->group = s->n_q_heads / s->n_kv_heads; p->n_pseudo = s->n_pseudo;
  p->rows = plan.rows; p->rows_pad = plan.rows_pad; p->n_groups = plan.n_groups;
  p->chunk_keys = plan.chunk_keys; p->max_chunks = (int32_t)plan.max_chunks;
  p->segments = plan.segments;
  p->wg_groups = 1;
  p->tile_parts = nullptr;
  p->c = s->scale * 1.4426950408889634f;
  p->seq_len = (int32_t)(s->total_tokens / s->batch);
  p->chunks_per_seq = (p->seq_len + plan.chunk_keys - 1) / plan.chunk_keys;
  p->chunk_shift = __builtin_ctz((unsigned)plan.chunk_keys);
  p->stage_q = plan.tile && plan.stage_q;
  p->inv_n_pseudo = 1.0f / (float)s->n_pseudo;
  p->inv_kv_heads = 1.0f / (float)s->n_kv_heads;
  p->inv_rows_pad = 1.0f / (float)plan.rows_pad;
  p->stream_share = 0.0f;
  return DAPQ_OK;
}

void set_parts(const ScorePlan& plan, char* workspace, ScoreParams* p) {
  p->parts = plan.tile ? nullptr : reinterpret_cast<float2*>(workspace + plan.off_parts);
  p->tile_parts = plan.tile ? reinterpret_cast<float*>(workspace + plan.off_parts) : nullptr;
}

int aligned16(const void* ptr, const char* name) {
  DAPQ_REQUIRE(ptr != nullptr, DAPQ_ERR_INVALID_ARG, "%s is NULL", name);
  DAPQ_REQUIRE((reinterpret_cast<uintptr_t>(ptr) & 15) == 0, DAPQ_ERR_UNSUPPORTED, "%s is not 16-byte aligned", name);
  return DAPQ_OK;
}

// The prefix of the chunk counts in device memory, for the passes of a shape that need it.
int launch_chunk_prefix(const dapq_shape* s, const ScorePlan& plan, const ScoreParams& p, hipStream_t stream) {
  if (s->cu_seqlens == nullptr || s->batch <= 64) return DAPQ_OK;
  hipLaunchKernelGGL(score_chunk_prefix_kernel, dim3(1), dim3(64), 0, stream, s->cu_seqlens, p.cu_chunks, s->batch,
                     plan.chunk_keys);
  DAPQ_HIP_LAUNCH_CHECK("score_chunk_prefix_kernel");
  return DAPQ_OK;
}

dim3 tile_grid(const dapq_shape* s, const ScorePlan& plan) {
  return dim3((unsigned)(plan.max_chunks * s->n_kv_heads), 1u, (unsigned)s->n_layers);
}
// Eight waves where the queries are staged; else one per row block, at most eight, at least four (with fewer than four row
// blocks the others only bring in keys: a lone wave issues the 32 transfers of a tile one by one).
dim3 tile_threads(const ScorePlan& plan) {
  const int waves = plan.stage_q || plan.row_blocks > kTileWaves ? kTileWaves : (plan.row_blocks < 4 ? 4 : plan.row_blocks);
  return dim3(64u * (unsigned)waves);
}
// Whether a wave of a staged call takes two of its sub-blocks at a time: where it has several (both numbers are powers of two).  Two waves to a
// SIMD do not hide each other's waits, two interleaved sub-blocks do; dapq_score of one layer of 8 KV heads, us, one -> two: 4096 keys, 256
// rows 14.2 -> 14.0, 296 18.9 -> 17.8, 512 22.2 -> 21.0; 8192 keys, 128 rows 14.4 -> 14.1, 256 20.4 -> 19.5, 384 29.5 -> 27.0.  A kernel
// with both forms in it is slower by 0.3 us, a first trip through more code: 1024 keys, 256 rows 10.2 -> 10.6, 8192 keys, 16 rows 10.5 -> 10.8.
bool two_at_a_time(const ScorePlan& plan) {
  return plan.stage_q && plan.chunk_keys / 32 > tile_most_parts(plan.row_blocks < kTileWaves ? plan.row_blocks : kTileWaves);
}
// (the whole dynamic limit once: see set_max_dynamic_lds)
#define DAPQ_LAUNCH_TILE(kernel, sums)                                                                           \
  do {                                                                                                           \
    if ((rc = set_lds(kernel, tile_lds(kTileMaxKeys, kTileWaves, true, sums))) != DAPQ_OK) return rc;            \
    hipLaunchKernelGGL(kernel, tile_grid(s, plan), tile_threads(plan),                                           \
                       tile_lds(plan.chunk_keys, plan.row_blocks, plan.stage_q, sums), stream, p);               \
    DAPQ_HIP_LAUNCH_CHECK(#kernel);                                                                              \
  } while (0)

// launch(row blocks of a wave) for the numbers that wave_row_split gives.
#define DAPQ_BY_ROW_BLOCKS(row_blocks, launch) \
  do {                                         \
    switch (row_blocks) {                      \
      case 2: launch(2); break;                \
      case 3: launch(3); break;                \
      case 4: launch(4); break;                \
      case 5: launch(5); break;                \
      case 6: launch(6); break;                \
      case 7: launch(7); break;                \
      default: launch(8);                      \
    }                                          \
  } while (0)

// Whether the waves of a dense launch start with the queries as fragments (SHORT) although they are six row blocks or more.  All keys of
// a chunk of a few sub-blocks fit the ring at once; they and fragments arrive in one trip to memory, and behind queries that go through the
// ring they wait for two or three.  It is the shorter start where the waves of a compute unit are workgroups of their own (side by side in
// one, their many loads set the pace: 32 prompts x heads of 512 keys, 256 rows 30.2 us through the ring, 36.7), in one kernel up to some
// eight rounds of waves.  (Three to five row blocks with as few keys are all score_short_kernel's, as are up to 512 heads.)  Ring -> fragments, us,
// dapq_score with inputs in the caches / out of memory, by workgroups:
//                       600                    1024                   4096                    8192                    12288                   32768
//   192 rows, 128 keys  22.6/22.5 -> 21.7/23.5  27.9/28.9 -> 24.6/28.9  100.7/101.1 -> 95.7/99.3  190.5/184.6 -> 189.1/183.3  277.7/265.9 -> 285.1/269.8  677/670 -> 712/704
//   256 rows, 64 keys   19.5/21.1 -> 18.8/21.7  26.7/30.7 -> 24.0/27.5  92.6/93.5 -> 85.7/87.3    169.0/162.1 -> 167.2/156.8  238.3/230.1 -> 247.9/239.7  570/553 -> 639/622
// (224 rows, 70 and 128 keys, and 256 rows, 96 and 128 keys, alike.)  Stats and accumulate alone, an odd number of chunks: from a wave per SIMD on 0.87
// to 1.01 of the time (2056 of 256 rows, 64 keys 46.9 -> 40.9, 42.8 -> 41.0; 2056 of 768 rows, 128 keys 138.9 -> 129.4, 145.7 -> 136.4; 16392 of 192 rows,
// 128 keys 295 -> 286, 290 -> 281), with fewer (513 to 1023 of up to 256 rows) 1.02 to 1.11 (600 of 256 rows, 128 keys 21.3 -> 22.9, 17.4 -> 19.1).
bool few_keys(const dapq_shape* s, const ScorePlan& plan, const GroupShape& gs) {
  return plan.segments == 0 && gs.waves == 1 && s->total_tokens / s->batch <= kMinChunkKeys;
}

int launch_wave_pass1(const dapq_shape* s, const ScorePlan& plan, ScoreParams all, hipStream_t stream) {
  const GroupShape gs = group_shape(s, plan);
  all.wg_groups = gs.groups;
  const bool few = few_keys(s, plan, gs);
  const KeyHints key = key_hints(s, plan, false);
  const bool hints = key.on;
  all.stream_share = key.share;
  return for_sequences(s, all, gs.threads(plan, s), [&](const ScoreParams& p, int64_t seqs) -> int {
    int rc = DAPQ_OK;
#define DAPQ_LAUNCH_W1(NRBV, SEGV, UNITV, SHORTV, STREAMV)                                                                 \
  do {                                                                                                                     \
    if ((rc = set_lds(score_wave_pass1_kernel<NRBV, SEGV, UNITV, SHORTV, STREAMV, kWaveStages>,                            \
                      kWavesPerGroup * wave_lds(kWaveStages))) != DAPQ_OK)                                                 \
      return rc;                                                                                                           \
    hipLaunchKernelGGL((score_wave_pass1_kernel<NRBV, SEGV, UNITV, SHORTV, STREAMV, kWaveStages>), gs.grid(plan, s, seqs), \
                       dim3(64 * gs.waves), gs.waves * wave_lds(kWaveStages), stream, p);                                  \
  } while (0)
#define DAPQ_LAUNCH_W1_KEYS(NRBV)                                                      \
  do {                                                                                 \
    if (plan.segments > 0 && hints) DAPQ_LAUNCH_W1(NRBV, true, true, false, true);     \
    else if (plan.segments > 0) DAPQ_LAUNCH_W1(NRBV, true, true, false, false);        \
    else if (plan.unit_sums && hints) DAPQ_LAUNCH_W1(NRBV, false, true, false, true);  \
    else if (plan.unit_sums) DAPQ_LAUNCH_W1(NRBV, false, true, false, false);          \
    else if (few && NRBV > 5) DAPQ_LAUNCH_W1(NRBV, false, false, (NRBV > 5), false);   \
    else if (hints) DAPQ_LAUNCH_W1(NRBV, false, false, false, true);                   \
    else DAPQ_LAUNCH_W1(NRBV, false, false, false, false);                             \
  } while (0)
    DAPQ_BY_ROW_BLOCKS(plan.row_blocks, DAPQ_LAUNCH_W1_KEYS);
#undef DAPQ_LAUNCH_W1_KEYS
#undef DAPQ_LAUNCH_W1
    DAPQ_HIP_LAUNCH_CHECK("score_wave_pass1_kernel");
    return DAPQ_OK;
  });
}

int launch_stats(const dapq_shape* s, const ScorePlan& plan, ScoreParams p, hipStream_t stream) {
  int rc = launch_chunk_prefix(s, plan, p, stream);
  if (rc != DAPQ_OK) return rc;
  if (plan.tile) {
    if (two_at_a_time(plan)) DAPQ_LAUNCH_TILE((score_tile_pass1_kernel<true, 2>), false);
    else if (plan.stage_q) DAPQ_LAUNCH_TILE((score_tile_pass1_kernel<true, 1>), false);
    else DAPQ_LAUNCH_TILE((score_tile_pass1_kernel<false, 1>), false);
    if (p.lse2 == nullptr) return DAPQ_OK;  // pass 2 merges the partials itself
  } else {
    if ((rc = launch_wave_pass1(s, plan, p, stream)) != DAPQ_OK) return rc;
  }
  // as many waves per 64 rows as the (mean) sequence has runs of chunks
  const int64_t chunks_per_seq = (plan.max_chunks + s->batch - 1) / s->batch, row_tiles = (plan.rows + 63) / 64;
  int64_t combine_waves = (chunks_per_seq + kCombineRun - 1) / kCombineRun;
  combine_waves = combine_waves < 1 ? 1 : (combine_waves > kCombineClasses ? kCombineClasses : combine_waves);
  // (a launch holds fewer than 2^32 threads along an axis)
  const int64_t seqs_per_launch = (kQuotientMax - 1) / row_tiles;
  for (int64_t first = 0; first < s->batch; first += seqs_per_launch) {
    const int64_t seqs = s->batch - first < seqs_per_launch ? s->batch - first : seqs_per_launch;
    hipLaunchKernelGGL(score_combine_kernel, dim3((unsigned)(row_tiles * seqs), (unsigned)(s->n_layers * s->n_kv_heads)),
                       dim3((unsigned)(64 * combine_waves)), 0, stream, p, (int)row_tiles, 1.0f / (float)row_tiles,
                       (int)first);
    DAPQ_HIP_LAUNCH_CHECK("score_combine_kernel");
  }
  return DAPQ_OK;
}

int launch_wave_pass2(const dapq_shape* s, const ScorePlan& plan, ScoreParams all, hipStream_t stream) {
  const GroupShape gs = group_shape(s, plan);
  all.wg_groups = gs.groups;
  const bool few = few_keys(s, plan, gs), hints = key_hints(s, plan, false).on;
  return for_sequences(s, all, gs.threads(plan, s), [&](const ScoreParams& p, int64_t seqs) -> int {
    int rc = DAPQ_OK;
#define DAPQ_LAUNCH_W2(NRBV, SEGV, SHORTV, STREAMV)                                                                       \
  do {                                                                                                                    \
    if ((rc = set_lds(score_wave_pass2_kernel<NRBV, SEGV, SHORTV, STREAMV, kWaveStages>,                                  \
                      kWavesPerGroup * wave_lds(kWaveStages))) != DAPQ_OK)                                                \
      return rc;                                                                                                          \
    hipLaunchKernelGGL((score_wave_pass2_kernel<NRBV, SEGV, SHORTV, STREAMV, kWaveStages>), gs.grid(plan, s, seqs),       \
                       dim3(64 * gs.waves), gs.waves * wave_lds(kWaveStages), stream, p);                                 \
  } while (0)
#define DAPQ_LAUNCH_W2_KEYS(NRBV)                                               \
  do {                                                                          \
    if (plan.segments > 0 && hints) DAPQ_LAUNCH_W2(NRBV, true, false, true);    \
    else if (plan.segments > 0) DAPQ_LAUNCH_W2(NRBV, true, false, false);       \
    else if (few && NRBV > 5) DAPQ_LAUNCH_W2(NRBV, false, (NRBV > 5), false);   \
    else if (hints) DAPQ_LAUNCH_W2(NRBV, false, false, true);                   \
    else DAPQ_LAUNCH_W2(NRBV, false, false, false);                             \
  } while (0)
    DAPQ_BY_ROW_BLOCKS(plan.row_blocks, DAPQ_LAUNCH_W2_KEYS);
#undef DAPQ_LAUNCH_W2_KEYS
#undef DAPQ_LAUNCH_W2
    DAPQ_HIP_LAUNCH_CHECK("score_wave_pass2_kernel");
    return DAPQ_OK;
  });
}

int launch_accumulate(const dapq_shape* s, const ScorePlan& plan, ScoreParams p, hipStream_t stream) {
  int rc = launch_chunk_prefix(s, plan, p, stream);  // (pass 2 can be called on its own: it rebuilds the prefix it walks)
  if (rc != DAPQ_OK) return rc;
  if (plan.tile) {
    const bool two = two_at_a_time(plan);
    if (p.lse2 == nullptr && two) DAPQ_LAUNCH_TILE((score_tile_pass2_kernel<true, true, 2>), true);
    else if (p.lse2 == nullptr) DAPQ_LAUNCH_TILE((score_tile_pass2_kernel<true, true, 1>), true);
    else if (two) DAPQ_LAUNCH_TILE((score_tile_pass2_kernel<false, true, 2>), true);
    else if (plan.stage_q) DAPQ_LAUNCH_TILE((score_tile_pass2_kernel<false, true, 1>), true);
    else DAPQ_LAUNCH_TILE((score_tile_pass2_kernel<false, false, 1>), true);
    return DAPQ_OK;
  }
  if ((rc = launch_wave_pass2(s, plan, p, stream)) != DAPQ_OK) return rc;
  if (plan.n_groups > 1) {
    const int64_t count = (int64_t)s->n_layers * s->n_kv_heads * s->total_tokens;
    const int64_t want = (count + 255) / 256;
    const unsigned blocks = (unsigned)(want < 1 ? 1 : (want > 16384 ? 16384 : want));
    hipLaunchKernelGGL(score_group_sum_kernel, dim3(blocks), dim3(256), 0, stream, p.partial, p.scores, count,
                       plan.n_groups);
    DAPQ_HIP_LAUNCH_CHECK("score_group_sum_kernel");
  }
  return DAPQ_OK;
}

// Whether one launch of score_fused_kernel can do both passes: a dense batch, one row group, and the chunks of a
// sequence exactly the waves of a workgroup.
// Returns the waves of such a workgroup (1 to 4), or 0 if the passes have to be separate launches.
int fused_waves(const dapq_shape* s, const ScorePlan& plan) {
  if (plan.tile || s->cu_seqlens != nullptr || plan.n_groups != 1 || s->total_tokens == 0) return 0;
  const int64_t chunks_per_seq = plan.max_chunks / s->batch;  // dense: max_chunks = batch * chunks per sequence
  if (chunks_per_seq * s->batch != plan.max_chunks) return 0;
  return chunks_per_seq >= 1 && chunks_per_seq <= kWavesPerGroup ? (int)chunks_per_seq : 0;
}
bool fused_applies(const dapq_shape* s, const ScorePlan& plan) { return fused_waves(s, plan) != 0; }

int launch_fused(const dapq_shape* s, const ScorePlan& plan, ScoreParams all, hipStream_t stream) {
  const GroupShape gs = {fused_waves(s, plan), 1};
  all.wg_groups = 1;
  const int64_t heads = (int64_t)s->n_layers * s->n_kv_heads;
  const bool few = few_keys(s, plan, gs) && s->batch * heads <= 8192;
  const KeyHints key = key_hints(s, plan, true);
  const bool hints = key.on;
  all.stream_share = key.share;
  return for_sequences(s, all, 64 * gs.waves, [&](const ScoreParams& p, int64_t seqs) -> int {
    const dim3 grid((unsigned)seqs, 1u, (unsigned)heads);
    int rc = DAPQ_OK;
#define DAPQ_LAUNCH_F(NRBV, UNITV, SHORTV, STREAMV)                                                                         \
  do {                                                                                                                      \
    if ((rc = set_lds(score_fused_kernel<NRBV, UNITV, SHORTV, STREAMV, kWaveStages>,                                        \
                      kWavesPerGroup * wave_lds(kWaveStages))) != DAPQ_OK)                                                  \
      return rc;                                                                                                            \
    hipLaunchKernelGGL((score_fused_kernel<NRBV, UNITV, SHORTV, STREAMV, kWaveStages>), grid, dim3(64 * gs.waves),          \
                       gs.waves * wave_lds(kWaveStages), stream, p);                                                        \
  } while (0)
#define DAPQ_LAUNCH_F_FORM(NRBV)                                              \
  do {                                                                        \
    if (plan.unit_sums && hints) DAPQ_LAUNCH_F(NRBV, true, false, true);      \
    else if (plan.unit_sums) DAPQ_LAUNCH_F(NRBV, true, false, false);         \
    else if (few && NRBV > 5) DAPQ_LAUNCH_F(NRBV, false, (NRBV > 5), false);  \
    else if (hints) DAPQ_LAUNCH_F(NRBV, false, false, true);                  \
    else DAPQ_LAUNCH_F(NRBV, false, false, false);                            \
  } while (0)
    DAPQ_BY_ROW_BLOCKS(plan.row_blocks, DAPQ_LAUNCH_F_FORM);
#undef DAPQ_LAUNCH_F_FORM
#undef DAPQ_LAUNCH_F
    DAPQ_HIP_LAUNCH_CHECK("score_fused_kernel");
    return DAPQ_OK;
  });
}

// Whether the calls of a shape run in score_short_kernel (the same line for the call of both passes and for the separate ones, whose bits agree).
// Its workgroup has a compute unit's LDS nearly to itself from 64 rows and 256 keys on, so it loses where a unit gets several heads in turn
// that the waves of score_fused_kernel take four at a time.  8 KV heads a layer, us, waves -> this, dapq_score (stats, accumulate):
//   up to 256 heads    256 rows, 128 keys, 8 heads 19.5 -> 8.3 (14.4 -> 6.2, 11.5 -> 5.5), 256 heads 20.8 -> 10.9; 384 keys, 256 heads 26.0 -> 22.6
//                      128 rows, 256 keys, 8 heads 13.4 -> 8.5, 256 heads 15.3 -> 10.7; 64 rows, 512 keys, 256 heads 17.1 -> 12.8; 32 rows 16.0 -> 9.7;
//                      left to the waves, a wave with sixteen sub-blocks: 256 rows, 512 keys, 256 heads 28.4 -> 27.9 (19.9 -> 19.9, 17.4 -> 18.7),
//                      192 rows 24.7 -> 26.6; and row blocks that leave waves idle over long prompts (at most twice as many sub-blocks in a row):
//                      160 rows, 384 keys 16.4 -> 17.9, 96 rows, 448 keys 14.8 -> 12.3 (accumulate 7.2 -> 7.7)
//   512 heads          256 rows, 128 keys 25.1 -> 20.3 (19.6 -> 15.6, 16.4 -> 15.0); 64 rows, 384 keys 19.8 -> 18.7 (16.7 -> 15.0, 14.1 -> 14.4: the one
//                      call of the three that loses at all); left to the waves: 256 rows, 200 keys 27.9 -> 28.1, 128 rows, 256 keys 20.3 -> 19.5 (16.7 -> 15.1,
//                      14.1 -> 14.8)
//   more, two to a unit     128 rows, 128 keys, 1024 heads 22.4 -> 17.2, 4096 77.3 -> 61.1; 64 rows, 200 keys 22.6 -> 17.8 and 78.7 -> 63.3; 32 rows, 256
//                      keys 23.6 -> 15.1 and 85.5 -> 56.2; left to the waves, one to a unit: 64 rows, 256 keys, 1024 heads 24.6 -> 26.7, 256 rows, 64 keys
//                      25.4 -> 27.1
// 300 drawn calls of 8 to 8192 heads that it takes: 0.65 of the time in the geometric mean, 1.01 at most (stats 0.55, 1.00; accumulate 0.66, 1.02).
bool short_call(const dapq_shape* s, const ScorePlan& plan) {
  if (plan.tile || s->cu_seqlens != nullptr || plan.rows > kShortRows || s->total_tokens < s->batch || s->total_tokens / s->batch > kShortKeys) return false;
  const int subs = (int)((s->total_tokens / s->batch + 31) / 32), row_blocks = (plan.rows + 31) / 32;
  const int parts = tile_most_parts(row_blocks) < subs ? tile_most_parts(row_blocks) : subs, in_a_row = (subs + parts - 1) / parts;
  const int staged = short_lds(subs, row_blocks, true);
  const int64_t heads = (int64_t)s->n_layers * s->n_kv_heads * s->batch;
  if (heads <= 256) return in_a_row <= 12 && in_a_row <= 2 * row_blocks && (staged <= kShortMostLds || subs <= 12);
  if (heads <= 512 && staged <= kShortMostLds && (subs <= 4 || in_a_row <= 3)) return true;
  return staged + kShortStaticLds <= 80 * 1024 && subs * row_blocks > 1;
}
int launch_short(const dapq_shape* s, const ScorePlan& plan, const ScoreParams& all, int mode, hipStream_t stream) {
  const int subs = (int)((s->total_tokens / s->batch + 31) / 32), row_blocks = (plan.rows + 31) / 32;
  const bool stage_q = short_lds(subs, row_blocks, true) <= kShortMostLds;
  return for_sequences(s, all, kTileThreads, [&](const ScoreParams& p, int64_t seqs) -> int {
    const dim3 grid((unsigned)seqs, 1u, (unsigned)(s->n_layers * s->n_kv_heads));
    int rc = DAPQ_OK;
#define DAPQ_LAUNCH_SHORT(MODEV, STAGEDV)                                                                                              \
  do {                                                                                                                                 \
    if ((rc = set_lds(score_short_kernel<MODEV, STAGEDV>, kShortMostLds)) != DAPQ_OK) return rc;                                       \
    hipLaunchKernelGGL((score_short_kernel<MODEV, STAGEDV>), grid, dim3(kTileThreads), short_lds(subs, row_blocks, STAGEDV), stream, p); \
  } while (0)
    if (mode == kShortBoth && stage_q) DAPQ_LAUNCH_SHORT(kShortBoth, true);
    else if (mode == kShortBoth) DAPQ_LAUNCH_SHORT(kShortBoth, false);
    else if (mode == kShortStats && stage_q) DAPQ_LAUNCH_SHORT(kShortStats, true);
    else if (mode == kShortStats) DAPQ_LAUNCH_SHORT(kShortStats, false);
    else if (stage_q) DAPQ_LAUNCH_SHORT(kShortAccumulate, true);
    else DAPQ_LAUNCH_SHORT(kShortAccumulate, false);
#undef DAPQ_LAUNCH_SHORT
    DAPQ_HIP_LAUNCH_CHECK("score_short_kernel");
    return DAPQ_OK;
  });
}

// Whether pass 2 of the tile form merges the partials itself: the threads of a workgroup can hold every sequence's, and
// there is a compute unit for every workgroup (tiles of 128 keys, one layer: 4096 keys 18.7 -> 17.6 us; 8191, two workgroups to a
// compute unit: 25.5 -> 27.2).
bool tile_merges(const dapq_shape* s, const ScorePlan& plan) {
  if (!plan.tile || !plan.stage_q || plan.max_chunks * s->n_kv_heads * s->n_layers > simd_count() / 4) return false;
  const int64_t longest = s->cu_seqlens == nullptr ? s->total_tokens / s->batch : s->total_tokens;
  return (longest + plan.chunk_keys - 1) / plan.chunk_keys <= tile_merge_chunks(plan.rows_pad);
}

int check_workspace(void* workspace, size_t workspace_bytes, const ScorePlan& plan) {
  DAPQ_REQUIRE(workspace != nullptr, DAPQ_ERR_INVALID_ARG, "workspace is NULL");
  DAPQ_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255) == 0, DAPQ_ERR_UNSUPPORTED,
               "workspace is not 256-byte aligned");
  DAPQ_REQUIRE(workspace_bytes >= plan.total_bytes, DAPQ_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed",
               workspace_bytes, plan.total_bytes);
  return DAPQ_OK;
}

}  // namespace
}  // namespace dapq

using namespace dapq;

extern "C" DAPQ_API int dapq_score_stats(const dapq_shape* shape, const void* q, const void* k, float* lse2,
                                         void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_shape(shape, true, true, false);
  if (rc != DAPQ_OK) return rc;
  ScorePlan plan;
  if ((rc = make_score_plan(shape, workspace_bytes, &plan)) != DAPQ_OK) return rc;
  if ((rc = aligned16(q, "q")) != DAPQ_OK) return rc;
  if ((rc = aligned16(k, "k")) != DAPQ_OK) return rc;
  DAPQ_REQUIRE(lse2 != nullptr, DAPQ_ERR_INVALID_ARG, "lse2 is NULL");
  if ((rc = check_workspace(workspace, workspace_bytes, plan)) != DAPQ_OK) return rc;
  ScoreParams p;
  fill_params(shape, plan, &p);
  char* ws = static_cast<char*>(workspace);
  p.q = static_cast<const uint16_t*>(q);
  p.k = static_cast<const uint16_t*>(k);
  p.cu_chunks = reinterpret_cast<int32_t*>(ws + plan.off_cu_chunks);
  set_parts(plan, ws, &p);
  p.lse2 = lse2;
  p.scores = nullptr;
  p.partial = nullptr;
  if (short_call(shape, plan)) return launch_short(shape, plan, p, kShortStats, static_cast<hipStream_t>(stream));
  return launch_stats(shape, plan, p, static_cast<hipStream_t>(stream));
}

extern "C" DAPQ_API int dapq_score_accumulate(const dapq_shape* shape, const void* q, const void* k,
                                              const float* lse2, float* scores, void* workspace,
                                              size_t workspace_bytes, void* stream) {
  int rc = check_shape(shape, true, true, false);
  if (rc != DAPQ_OK) return rc;
  ScorePlan plan;
  if ((rc = make_score_plan(shape, workspace_bytes, &plan)) != DAPQ_OK) return rc;
  if ((rc = aligned16(q, "q")) != DAPQ_OK) return rc;
  if ((rc = aligned16(k, "k")) != DAPQ_OK) return rc;
  DAPQ_REQUIRE(lse2 != nullptr, DAPQ_ERR_INVALID_ARG, "lse2 is NULL");
  DAPQ_REQUIRE(scores != nullptr, DAPQ_ERR_INVALID_ARG, "scores is NULL");
  if ((rc = check_workspace(workspace, workspace_bytes, plan)) != DAPQ_OK) return rc;
  ScoreParams p;
  fill_params(shape, plan, &p);
  p.q = static_cast<const uint16_t*>(q);
  p.k = static_cast<const uint16_t*>(k);
  p.cu_chunks = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + plan.off_cu_chunks);
  p.parts = nullptr;
  p.partial = reinterpret_cast<float*>(static_cast<char*>(workspace) + plan.off_partial);
  p.lse2 = const_cast<float*>(lse2);
  p.scores = scores;
  if (short_call(shape, plan)) return launch_short(shape, plan, p, kShortAccumulate, static_cast<hipStream_t>(stream));
  return launch_accumulate(shape, plan, p, static_cast<hipStream_t>(stream));
}

extern "C" DAPQ_API int dapq_score_single_launch(const dapq_shape* shape) {
  int rc = check_shape(shape, true, true, false);
  if (rc != DAPQ_OK) return rc;
  ScorePlan plan;
  if ((rc = make_score_plan(shape, SIZE_MAX, &plan)) != DAPQ_OK) return rc;
  return fused_applies(shape, plan) ? 1 : 0;
}

extern "C" DAPQ_API int dapq_score(const dapq_shape* shape, const void* q, const void* k, float* scores,
                                   void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_shape(shape, true, true, false);
  if (rc != DAPQ_OK) return rc;
  ScorePlan plan;
  if ((rc = make_score_plan(shape, workspace_bytes, &plan)) != DAPQ_OK) return rc;
  DAPQ_REQUIRE(scores != nullptr, DAPQ_ERR_INVALID_ARG, "scores is NULL");
  if ((rc = check_workspace(workspace, workspace_bytes, plan)) != DAPQ_OK) return rc;
  if (fused_applies(shape, plan)) {
    if ((rc = aligned16(q, "q")) != DAPQ_OK) return rc;
    if ((rc = aligned16(k, "k")) != DAPQ_OK) return rc;
    ScoreParams p;
    fill_params(shape, plan, &p);
    p.q = static_cast<const uint16_t*>(q);
    p.k = static_cast<const uint16_t*>(k);
    p.cu_chunks = nullptr;
    p.parts = nullptr;
    p.partial = nullptr;
    p.lse2 = nullptr;
    p.scores = scores;
    if (short_call(shape, plan)) return launch_short(shape, plan, p, kShortBoth, static_cast<hipStream_t>(stream));
    return launch_fused(shape, plan, p, static_cast<hipStream_t>(stream));
  }
  if (tile_merges(shape, plan)) {
    if ((rc = aligned16(q, "q")) != DAPQ_OK) return rc;
    if ((rc = aligned16(k, "k")) != DAPQ_OK) return rc;
    ScoreParams p;
    fill_params(shape, plan, &p);
    char* ws = static_cast<char*>(workspace);
    p.q = static_cast<const uint16_t*>(q);
    p.k = static_cast<const uint16_t*>(k);
    p.cu_chunks = reinterpret_cast<int32_t*>(ws + plan.off_cu_chunks);
    set_parts(plan, ws, &p);
    p.partial = nullptr;
    p.lse2 = nullptr;
    p.scores = scores;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if ((rc = launch_stats(shape, plan, p, st)) != DAPQ_OK) return rc;
    return launch_accumulate(shape, plan, p, st);
  }
  float* lse2 = reinterpret_cast<float*>(static_cast<char*>(workspace) + plan.off_lse2);
  if ((rc = dapq_score_stats(shape, q, k, lse2, workspace, workspace_bytes, stream)) != DAPQ_OK) return rc;
  return dapq_score_accumulate(shape, q, k, lse2, scores, workspace, workspace_bytes, stream);
}


extern "C" DAPQ_API int dapq_score_stats_extend(const dapq_shape* shape, const void* q, const void* k_pseudo,
                                                int64_t kp_stride_layer, int64_t kp_stride_seq, int64_t kp_stride_head,
                                                int64_t kp_stride_row, float* lse2, void* stream) {
  int rc = check_shape(shape, true, false, false);
  if (rc != DAPQ_OK) return rc;
  ScorePlan plan;
  if ((rc = make_score_plan(shape, SIZE_MAX, &plan)) != DAPQ_OK) return rc;
  if ((rc = aligned16(q, "q")) != DAPQ_OK) return rc;
  if ((rc = aligned16(k_pseudo, "k_pseudo")) != DAPQ_OK) return rc;
  DAPQ_REQUIRE(lse2 != nullptr, DAPQ_ERR_INVALID_ARG, "lse2 is NULL");
  DAPQ_REQUIRE(kp_stride_layer >= 0 && kp_stride_seq >= 0 && kp_stride_head >= 0, DAPQ_ERR_INVALID_ARG,
               "k_pseudo strides must be >= 0");
  DAPQ_REQUIRE(kp_stride_row >= shape->head_dim && kp_stride_row < ((int64_t)1 << 26), DAPQ_ERR_INVALID_ARG,
               "kp_stride_row (%lld) must be in [head_dim, 2^26)", (long long)kp_stride_row);
  DAPQ_REQUIRE(kp_stride_layer % 8 == 0 && kp_stride_seq % 8 == 0 && kp_stride_head % 8 == 0 && kp_stride_row % 8 == 0,
               DAPQ_ERR_UNSUPPORTED, "k_pseudo strides must be multiples of 8 elements (16-byte rows)");
  DAPQ_REQUIRE(shape->batch <= 65535, DAPQ_ERR_UNSUPPORTED, "batch must be <= 65535");
  ScoreParams p;
  fill_params(shape, plan, &p);
  p.q = static_cast<const uint16_t*>(q);
  p.k = nullptr;
  p.cu_chunks = nullptr;
  p.parts = nullptr;
  p.partial = nullptr;
  p.scores = nullptr;
  p.lse2 = lse2;
  PseudoParams pp;
  pp.kp = static_cast<const uint16_t*>(k_pseudo);
  pp.stride_layer = kp_stride_layer; pp.stride_seq = kp_stride_seq;
  pp.stride_head = kp_stride_head; pp.stride_row = kp_stride_row;
  const int row_blocks = (plan.rows + 31) / 32, nsubs = (shape->n_pseudo + 31) / 32;
  const int waves = row_blocks < kPseudoWaves ? row_blocks : kPseudoWaves;
  const dim3 grid((unsigned)shape->batch, (unsigned)((row_blocks + waves - 1) / waves), (unsigned)(shape->n_layers * shape->n_kv_heads));
  const int key_subs = nsubs < kPseudoSubs ? nsubs : kPseudoSubs;
  const dim3 threads(64u * (unsigned)waves);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (row_blocks <= 2) hipLaunchKernelGGL(score_pseudo_kernel<true>, grid, threads, key_subs * kSubBytes, st, p, pp);
  else hipLaunchKernelGGL(score_pseudo_kernel<false>, grid, threads, (waves + key_subs) * kSubBytes, st, p, pp);
  DAPQ_HIP_LAUNCH_CHECK("score_pseudo_kernel");
  return DAPQ_OK;
}

// ---------------------------------------------------------------------------------------------
// dapq_score for callers that cannot allocate device memory (code under HIP graph capture, tight serving loops):
// the workspace of the two passes lives in a file-scope device array instead of a caller buffer.
// ---------------------------------------------------------------------------------------------
namespace {

constexpr size_t kStaticScratchBytes = DAPQ_STATIC_SCRATCH_BYTES;
// One copy per GPU the library runs on, held until the process ends.  In host code this name is only a handle
// for hipGetSymbolAddress: the device address it stands for is looked up once per device and kept below.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

int scratch_of_current_device(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(DAPQ_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
  DAPQ_REQUIRE(dev >= 0 && dev < kMaxDevices, DAPQ_ERR_UNSUPPORTED, "device index %d is beyond the %d this library tracks",
               dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || ptr == nullptr)
      return fail(DAPQ_ERR_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return DAPQ_OK;
}

}  // namespace

extern "C" DAPQ_API size_t dapq_score_static_capacity(void) { return kStaticScratchBytes; }

extern "C" DAPQ_API int dapq_score_static(const dapq_shape* shape, const void* q, const void* k, float* scores,
                                          void* stream) {
  int rc = check_shape(shape, true, true, false);
  if (rc != DAPQ_OK) return rc;
  ScorePlan plan;
  if ((rc = make_score_plan(shape, SIZE_MAX, &plan)) != DAPQ_OK) return rc;
  DAPQ_REQUIRE(plan.total_bytes <= kStaticScratchBytes, DAPQ_ERR_WORKSPACE,
               "this shape needs %zu bytes of workspace, the built-in scratch array holds %zu: use dapq_score with a "
               "caller workspace", plan.total_bytes, kStaticScratchBytes);
  void* ptr = nullptr;
  if ((rc = scratch_of_current_device(&ptr)) != DAPQ_OK) return rc;
  // nothing in the workspace has to start at zero: pass 1 writes every partial that the combine step reads, and
  // the combine step writes every lse2 that pass 2 reads
  return dapq_score(shape, q, k, scores, ptr, kStaticScratchBytes, stream);
}
