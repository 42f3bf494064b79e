// One decode step over the compact cache (Sec. 4.2, last paragraph: decoding starts at position L_p and
// uses only the compressed cache): out = softmax(q K_c^T / sqrt(d_k)) V_c per query head, over the first
// count rows of the KV head's compact cache as dapq_gather wrote it.
//
// One workgroup per (layer, sequence, KV head); its waves take tiles of 32 cache rows in turn and meet once, at the end.
// What bounds a call is how fast the compute units in use can take in bytes and how little stands before and after: a
// call of one layer has only a few heads, each 0.5 MB, and one compute unit takes about 20 bytes a clock from beyond its
// L2 and 54 from L2.  So there is one sweep over K_c and V_c together, the loads of a tile are issued as soon as the
// registers or the LDS slot of an earlier one are spent (the first ones before the row count is known), every load
// instruction covers whole rows (K_c goes through LDS for that: loading the operand layout straight from memory,
// consecutive lanes in consecutive rows, runs at 15 bytes a clock), both products run on v_mfma_f32_16x16x32_bf16,
// and where the heads alone would leave most of the chip idle the value channels of a head are dealt to 2 or 4
// workgroups ("slices"): each reads all of K_c (they start a slice of the tiles apart) but only its share of V_c.
//   logits   D[key][column] = K_c tile (A operand, 16 keys x 32 channels per instruction) x q (B operand).  The columns
//            are 4 query heads x 4 parts: column 4 * part + head.
//   weights  2^(c * logit - ref) in fp32.  ref is the largest logit of the wave's first tile with a finite one; it only
//            moves (and the sums are rescaled) if a later logit lies more than kDecodeHeadroom binades above it.  Weights of
//            up to 2^4 over 2^13 rows keep the sums of values below 2^110 in the range of fp32.  (Headroom 0 moves too often: 983
//            rows, 1 sequence 6.9 -> 7.6 us; 60 and 4 take the same time.  A check of the sums and a second sweep where they left the
//            range: 0.25 us.)
//   output   D[column][channel] += weights (A) x V_c (B).  A weight enters as three bf16 numbers whose sum it is, bit
//            for bit (8 + 8 + 8 bits of its significand): part 0 carries the first, part 1 the second, part 2 the third,
//            so one instruction multiplies all three with V_c and nothing is lost against fp32 weights (part 3 is not
//            used).  A lane's four logits of a tile are four keys of one column, which is how the A operand wants
//            them once the keys of an instruction are counted tile by tile; V_c follows: a lane loads the same
//            piece (CPL channels) of 8 rows and transposes the 8 x CPL block in its own registers, and instruction
//            j of a tile gives the channels CPL * n + j.
// Measured (32 query / 8 KV heads, one layer): 983 rows, 1 sequence 24.9 -> 6.7 us; 64..256 rows, 50 sequences
// 38.9 -> 9.8 us (3.4 TB/s); 983 rows, 64 sequences 74.9 -> 40.5 us (6.3 TB/s); 8 query heads per KV head, 4096 rows, 1 sequence 140.7 -> 19.9 us.  (Before: vector products, sixteen
// waves per head, logits and weights through LDS, the cache read twice for more than 4 query heads.)
#include <math.h>

#include <type_traits>

#include "dapq_internal.h"

namespace dapq {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kDecodeMaxRows = 8192;
constexpr int kDecodeTile = 32;           // cache rows a wave takes at a time
constexpr int kDecodeParts = 3;           // bf16 numbers that make up a weight
constexpr float kDecodeHeadroom = 4.0f;   // binades a logit may lie above the reference
constexpr float kDecodeLowest = -3.4028234663852886e38f;  // where the reference starts: finite, a logit of -inf then weighs 0

struct DecodeParams {
  const uint16_t* q;        // [layer][seq][Hq][d]
  const uint16_t* k_cache;  // [layer][seq][Hkv][budget][d]
  const uint16_t* v_cache;
  const int32_t* count;     // [layer][seq][Hkv]
  float* out;               // [layer][seq][Hq][d]
  int32_t group, budget;    // group: query heads per KV head
  float c;                  // scale * log2(e)
};

constexpr int kDecodeSlotBytes = kDecodeTile * kHeadDim * 2;  // one tile of K_c
constexpr int kDecodeSlots = 2;                               // per wave
constexpr int decode_wave_bytes(int ht) { return kDecodeSlots * kDecodeSlotBytes + ht * 4 * kHeadDim * 2; }  // and its queries

// K_c and V_c of a head through buffer descriptors whose range check returns zeros for rows past the budget.
struct DecodeSource {
  __amdgpu_buffer_rsrc_t k, v;
  unsigned k_off[4], v_off;
};
// AUX: cache policy of the loads.
constexpr int kNonTemporal = 2;
// One wave moves a tile of K_c into an LDS slot, 1 KB (4 rows) per transfer, rows 256 B apart, the 16-byte chunks of a row
// XOR-swizzled by the row so that the operand reads are free of bank conflicts.
template <int AUX>
__device__ __forceinline__ void load_k(char* slot, const DecodeSource& src, int row0) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const unsigned off = src.k_off[i & 3] + (unsigned)(row0 + 16 * (i >> 2)) * kHeadDim * 2;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src.k, (__attribute__((address_space(3))) void*)(slot + i * 1024), 16, (int)off, 0,
                                             0, AUX);
  }
}
// A tile of a slice of V_c as it sits in the registers of lane 16 * kg + n: v[e] = channels CPL * n .. + CPL of the slice of
// row 16 * (e / 4) + 4 * kg + e % 4.
template <int CPL, int AUX>
__device__ __forceinline__ void load_v(unsigned (&v)[8][CPL / 2], const DecodeSource& src, int row0) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const unsigned off = src.v_off + (unsigned)(row0 + 16 * (e >> 2)) * kHeadDim * 2 + (e & 3) * kHeadDim * 2;
    if constexpr (CPL == 8) {
      const u32x4 u = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(src.v, (int)off, 0, AUX));
#pragma unroll
      for (int i = 0; i < 4; ++i) v[e][i] = u[i];
    } else if constexpr (CPL == 4) {
      const u32x2 u = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(src.v, (int)off, 0, AUX));
      v[e][0] = u[0];
      v[e][1] = u[1];
    } else {
      v[e][0] = __builtin_bit_cast(unsigned, __builtin_amdgcn_raw_buffer_load_b32(src.v, (int)off, 0, AUX));
    }
  }
}

// Keeps the loads before it before the loads after it: the waits count loads in the order they were issued.
__device__ __forceinline__ void keep_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// HT tiles of 4 query heads per sweep over the cache, CPL channels per lane (16 * CPL of the 128 per workgroup).
// STREAM: the caches of all heads are more than the chip's caches keep until the next step, and their loads carry the non-temporal hint.
template <int HT, int CPL, int WAVES, bool STREAM>
__global__ __launch_bounds__(64 * WAVES, 2) void decode_attention_kernel(DecodeParams p) {
  extern __shared__ char lds[];  // [waves]: kDecodeSlots tiles of K_c, the queries; at the end weighted sums, references, sums of weights
  constexpr int kAux = STREAM ? kNonTemporal : 0;
  constexpr bool kEarly = kHeadDim / (16 * CPL) > 1;  // (see first_loads)
  constexpr bool kTail = HT == 1 || CPL < 8;         // a wave's last tile has code of its own (two head tiles and all channels: no registers for it)
  constexpr int kHeads = 4 * HT, kChannels = 16 * CPL, kSlices = kHeadDim / kChannels, kThreads = 64 * WAVES;
  static_assert((kDecodeParts * kHeads * kChannels + 2 * kHeads) * 4 <= kDecodeSlots * kDecodeSlotBytes,
                "what a wave leaves at the end fits where its tiles were");
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int kWaveBytes = decode_wave_bytes(HT);
  char* ring = lds + wave * kWaveBytes;
  const int slice = blockIdx.y;
  const int g = p.group;
  const int64_t head = blockIdx.x;  // (layer * batch + seq) * Hkv + kv
  DecodeSource src;
  src.k = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.k_cache + head * p.budget * kHeadDim), 0,
                                            p.budget * kHeadDim * 2, 0x00020000);
  src.v = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.v_cache + head * p.budget * kHeadDim), 0,
                                            p.budget * kHeadDim * 2, 0x00020000);
#pragma unroll
  for (int j = 0; j < 4; ++j) src.k_off[j] = (unsigned)((4 * j + kg) * kHeadDim * 2 + ((n ^ kg) ^ (4 * j)) * 16);
  src.v_off = (unsigned)(4 * kg * kHeadDim * 2 + (slice * kChannels + n * CPL) * 2);
  // the part of a weight that this lane's column stands for: what is left once the leading 8 bits were taken off n / 4 times
  const unsigned mask1 = n >= 4 ? 0xFFFF0000u : 0u, mask2 = n >= 8 ? 0xFFFF0000u : 0u;
  // tile number i of this workgroup: the slices of a head start a slice apart
  int tiles = (p.budget + kDecodeTile - 1) / kDecodeTile;
  auto row_of = [&](int i) {
    int t = i + slice * tiles / kSlices;
    t = t < tiles ? t : t - tiles;
    return t * kDecodeTile;
  };
  auto row_or_none = [&](int i) { return kEarly || i < tiles ? row_of(i) : kDecodeMaxRows; };
  int rows = p.count[head];
  auto clamp_rows = [&]() {
    rows = __builtin_amdgcn_readfirstlane(rows);
    rows = rows < 0 ? 0 : (rows > p.budget ? p.budget : rows);
    return (rows + kDecodeTile - 1) / kDecodeTile;
  };

  for (int h0 = 0; h0 < g; h0 += kHeads) {
    const int nh = g - h0 < kHeads ? g - h0 : kHeads;  // query heads of this sweep
    const int64_t qrow0 = head * g + h0;
    // the queries come in whole rows too: lane l has piece l % 16 of query head l / 16 of a head tile
    u32x4 qrow[HT];
#pragma unroll
    for (int t = 0; t < HT; ++t) {
      const int h = 4 * t + kg;
      __builtin_memcpy(&qrow[t], p.q + (qrow0 + (h < nh ? h : nh - 1)) * kHeadDim + 8 * n, 16);  // (q_decode may be unaligned)
    }
    keep_order();
    // The slices of a few heads have the first tiles on their way before the row count is known (rows past the count are inside the cache all the
    // same).  Where heads fill the chip, bytes count: only a wave's first rows of K_c, and not of heads so short that a wave may have none.  Us, all
    // tiles early and four waves' worth of loads past the end -> first tile early -> none early, one slice: 50 sequences of 64..256 rows
    // 10.9 -> 9.8 -> 9.8; 64 of 32..130, 1 query head 8.6 -> 7.9 -> 7.5; 20 of 256 6.8 -> 6.7 -> 6.9; 16 of 983 12.2 -> 12.2 -> 12.3.
    unsigned vt[8][CPL / 2];
    auto first_loads = [&]() {
      const bool short_head = tiles < 2 * WAVES;
      if (!kEarly && h0 == 0 && short_head) tiles = clamp_rows();
      load_k<kAux>(ring, src, row_or_none(wave));
      if (!kEarly && h0 == 0 && !short_head) tiles = clamp_rows();
      if (kEarly || !kTail || wave + WAVES < tiles) load_k<kAux>(ring + kDecodeSlotBytes, src, row_or_none(wave + WAVES));
      keep_order();
      load_v<CPL, kAux>(vt, src, row_or_none(wave));
      keep_order();
    };
    first_loads();
    u32x4* qs = reinterpret_cast<u32x4*>(ring + kDecodeSlots * kDecodeSlotBytes);
#pragma unroll
    for (int t = 0; t < HT; ++t) qs[t * 64 + kg * 16 + (n ^ kg)] = qrow[t];  // (swizzled like the tiles, by the head)
    bf16x8 qf[HT][4];
#pragma unroll
    for (int t = 0; t < HT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        qf[t][s] = __builtin_bit_cast(bf16x8, qs[t * 64 + (n & 3) * 16 + ((4 * s + kg) ^ (n & 3))]);
    if (kEarly && h0 == 0) {
      const int filled = clamp_rows();
      if (filled != tiles) {  // the slices start elsewhere
        tiles = filled;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        first_loads();
      }
    }
    if (rows == 0) {  // an empty cache attends to nothing
      for (int e = tid; e < nh * kChannels; e += kThreads)
        p.out[(qrow0 + e / kChannels) * kHeadDim + slice * kChannels + e % kChannels] = 0.0f;
      continue;
    }
    f32x4 acc[HT][CPL];
    float ref[HT], sum[HT];
#pragma unroll
    for (int t = 0; t < HT; ++t) {
#pragma unroll
      for (int j = 0; j < CPL; ++j) acc[t][j] = {0.0f, 0.0f, 0.0f, 0.0f};
      ref[t] = kDecodeLowest;
      sum[t] = 0.0f;
    }

    int slot = 0;
    // Tile i; MORE: the wave has another one, whose loads go out.  (Loads past the end of the cache fetch nothing, but keep the compute unit's
    // address unit busy as long as any others: with three tiles' worth of them at a wave's end 983 rows, 1 sequence 7.05 us, now 6.7; 256 rows
    // 4.9, now 4.2; 32 layers, 4 sequences of 75..300 rows 24.7, now 21.7.)
    auto step = [&](int i, auto more) {
      constexpr bool MORE = decltype(more)::value;
      const int row0 = row_of(i);
      const bool partial = row0 + kDecodeTile > rows;
      // in flight, oldest first: K_c of this tile, (MORE) K_c of the next one, V_c of this tile (8 loads each)
      if constexpr (MORE) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      const u32x4* kt = reinterpret_cast<const u32x4*>(ring + slot * kDecodeSlotBytes);
      bf16x8 kf[2][4];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int s = 0; s < 4; ++s) kf[hf][s] = __builtin_bit_cast(bf16x8, kt[(16 * hf + n) * 16 + ((4 * s + kg) ^ n)]);
      float xs[HT][8];
#pragma unroll
      for (int t = 0; t < HT; ++t) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          f32x4 d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int s = 0; s < 4; ++s) d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[hf][s], qf[t][s], d, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 4; ++v) xs[t][4 * hf + v] = d[v];
        }
      }
      if constexpr (MORE) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the tile is out of its slot before that is refilled
        load_k<kAux>(ring + slot * kDecodeSlotBytes, src, i + 2 * WAVES < tiles ? row_of(i + 2 * WAVES) : kDecodeMaxRows);
        slot ^= 1;
        keep_order();
      }
      u32x4 pa[HT];  // the weights as A operand
#pragma unroll
      for (int t = 0; t < HT; ++t) {
        float(&x)[8] = xs[t];
        if (partial) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (row0 + 16 * (e >> 2) + 4 * kg + (e & 3) >= rows) x[e] = -INFINITY;
        }
        float m = x[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) m = fmaxf(m, x[e]);
        m *= p.c;
        if (__any(m > ref[t] + kDecodeHeadroom)) {  // (always for the first tile that has a logit)
          m = fmaxf(m, __shfl_xor(m, 16, 64));
          m = fmaxf(m, __shfl_xor(m, 32, 64));
          const float moved = fmaxf(ref[t], m);
          const float f = __builtin_amdgcn_exp2f(ref[t] - moved);
          ref[t] = moved;
          sum[t] *= f;
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            const float fh = __shfl(f, h, 64);  // column h belongs to head h; row h of every part does too
#pragma unroll
            for (int j = 0; j < CPL; ++j) acc[t][j][h] *= fh;
          }
        }
        unsigned w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float y = __builtin_amdgcn_exp2f(fmaf(x[e], p.c, -ref[t]));
          sum[t] += y;
          const float y1 = y - __uint_as_float(__float_as_uint(y) & mask1);
          const float y2 = y1 - __uint_as_float(__float_as_uint(y1) & mask2);
          w[e] = __float_as_uint(y2);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) pa[t][e] = __builtin_amdgcn_perm(w[2 * e + 1], w[2 * e], 0x07060302u);
      }
      if (partial) {  // what lies past the count may be anything: 0 times it must be 0
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (row0 + 16 * (e >> 2) + 4 * kg + (e & 3) >= rows) {
#pragma unroll
            for (int j = 0; j < CPL / 2; ++j) vt[e][j] = 0u;
          }
      }
#pragma unroll
      for (int j = 0; j < CPL; ++j) {  // channels CPL * n + j of the slice
        u32x4 vb;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          vb[e] = __builtin_amdgcn_perm(vt[2 * e + 1][j >> 1], vt[2 * e][j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
        for (int t = 0; t < HT; ++t)
          acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pa[t]), __builtin_bit_cast(bf16x8, vb),
                                                             acc[t][j], 0, 0, 0);
      }
      if constexpr (MORE) {
        load_v<CPL, kAux>(vt, src, kTail || i + WAVES < tiles ? row_of(i + WAVES) : kDecodeMaxRows);
        keep_order();
      }
    };
    int i = wave;
    for (; i + (kTail ? WAVES : 0) < tiles; i += WAVES) step(i, std::true_type{});
    if (kTail && i < tiles) step(i, std::false_type{});

    // What the wave leaves goes where its tiles were (none is in flight any more).  (A wave without a tile is not read below.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    float* mine = reinterpret_cast<float*>(ring);
    constexpr int kSums = kDecodeParts * kHeads * kChannels;  // floats in front of the references and the sums of weights
#pragma unroll
    for (int t = 0; t < HT; ++t) {
      float s = sum[t];
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      if (lane < 4) {
        mine[kSums + 4 * t + lane] = ref[t];
        mine[kSums + kHeads + 4 * t + lane] = s;
      }
      if (kg < kDecodeParts) {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          float* dst = mine + (kg * kHeads + 4 * t + h) * kChannels + CPL * n;
#pragma unroll
          for (int j = 0; j < CPL; ++j) dst[j] = acc[t][j][h];
        }
      }
    }
    __syncthreads();
    const int waves = tiles < WAVES ? tiles : WAVES;
    for (int e = tid; e < nh * kChannels; e += kThreads) {
      const int h = e / kChannels;
      auto left = [&](int w, int at) { return reinterpret_cast<const float*>(lds + w * kWaveBytes)[at]; };
      float m = left(0, kSums + h);
      for (int w = 1; w < waves; ++w) m = fmaxf(m, left(w, kSums + h));
      float o = 0.0f, first = 0.0f, s = 0.0f;  // first: the sums over the weights' first parts alone
      for (int w = 0; w < waves; ++w) {  // fixed order
        const float f = __builtin_amdgcn_exp2f(left(w, kSums + h) - m);
        o = fmaf(f, left(w, e) + (left(w, kHeads * kChannels + e) + left(w, 2 * kHeads * kChannels + e)), o);
        first = fmaf(f, left(w, e), first);
        s = fmaf(f, left(w, kSums + kHeads + h), s);
      }
      // (an infinite value times the second or third part of a weight, which may be 0, is no number: the first part, which is not 0
      // where the weight is not, then has the say)
      p.out[(qrow0 + h) * kHeadDim + slice * kChannels + e % kChannels] = (o == o ? o : first) / s;
    }
    if (h0 + kHeads < g) __syncthreads();  // everything has been read before the next sweep's tiles arrive
  }
}

template <int HT, int CPL, int WAVES, bool STREAM>
int launch_decode(int64_t heads, const DecodeParams& p, hipStream_t stream) {
  constexpr int kBytes = WAVES * decode_wave_bytes(HT);
  const int rc = set_max_dynamic_lds(reinterpret_cast<const void*>(decode_attention_kernel<HT, CPL, WAVES, STREAM>), kBytes);
  if (rc != DAPQ_OK) return rc;
  // a launch holds fewer than 2^32 threads along an axis: 2^24 heads and more go in several
  constexpr int64_t kMostHeads = (int64_t)1 << 22;
  const int64_t q_step = (int64_t)p.group * kHeadDim, cache_step = (int64_t)p.budget * kHeadDim;
  for (int64_t first = 0; first < heads; first += kMostHeads) {
    DecodeParams part = p;
    part.q += first * q_step;
    part.k_cache += first * cache_step;
    part.v_cache += first * cache_step;
    part.count += first;
    part.out += first * q_step;
    hipLaunchKernelGGL((decode_attention_kernel<HT, CPL, WAVES, STREAM>),
                       dim3((unsigned)(heads - first < kMostHeads ? heads - first : kMostHeads), kHeadDim / (16 * CPL)),
                       dim3(64 * WAVES), kBytes, stream, part);
    DAPQ_HIP_LAUNCH_CHECK("decode_attention_kernel");
  }
  return DAPQ_OK;
}

// Slices per head: every slice reads all of K_c, so they pay only while their workgroups have a compute unit each (four slices up to
// 64 heads, two up to 128) and the caches of all heads together are not so large that the second and further readers of K_c
// find it gone.  One layer, us with four / two / one slice:
//   4 query heads per KV head, 256 rows    32 heads 5.0 / 5.6 / 5.9   64: 5.3 / 5.8 / 5.7     80: 8.7 / 6.0 / 5.9    160: 12.9 / 10.1 / 6.2
//                              983         32: 7.4 / 7.9 / 8.9        64: 8.2 / 8.7 / 9.2     96: 15.5 / 10.6 / 10.5 128: 19.3 / 13.6 / 12.5
//                              2048        40: 12.5 / 12.8 / 14.5     48: 15.1 / 13.1 / 14.9  56: 18.4 / 14.1 / 14.8 64: 22.0 / 15.4 / 15.0
//                              4096        24: 20.5 / 21.0 / 23.7     32: 25.6 / 21.5 / 24.1  48: 39.5 / 24.2 / 25.0 56: 47.2 / 26.6 / 25.1
//   8, 983                                 64: 9.5 / 10.1 / 12.5      96: 17.1 / 11.5 / 12.9  128: 21.3 / 15.2 / 14.2
//   8, 4096                                24: 22.5 / 22.9 / 30.8     32: 27.9 / 23.6 / 30.9  64: 58.2 / 30.6 / 31.0 80: 74.8 / 37.1 / 31.2
// From 5 query heads per KV head on, two slices against one are even at 128 heads of 800 rows, 112 of 950, 96 of 1200 and 80 of 1750 or
// so: a line by heads x heads x rows (two / one, 8 heads: 128 of 1088 16.2 / 15.0, 112 of 1243 16.2 / 15.3, 96 of 1100 12.9 / 13.5, 80 of
// 1600 15.6 / 15.9, 66 of 2110 18.4 / 19.0).
template <int HT>
int launch_decode_slices(int64_t heads, const DecodeParams& p, hipStream_t stream) {
  const int64_t rows = heads * p.budget;
  if (heads <= 64 && (rows <= 88 * 1024 || heads <= 24)) return launch_decode<HT, 2, 8, false>(heads, p, stream);
  if (heads <= 128 && (HT == 1 ? rows <= 112 * 1024 || heads <= 48 : heads * rows <= 11 << 20 || heads <= 64)) return launch_decode<HT, 4, 8, false>(heads, p, stream);
  // From 128 MB of caches on their rows stream, if one sweep reads them: us without -> with hints, 8 KV heads, 983 rows, the same caches again / those
  // of several layers in turn, as in a model, sequences: 16 (64 MB) 12.4 -> 14.6 / 16.7 -> 15.5, 24 (97 MB) 16.7 -> 16.6 / 20.2 -> 18.5, 32
  // 21.5 -> 21.3 / 25.4 -> 23.0, 64 40.6 -> 40.9 / 47.4 -> 42.2 (6.1 TB/s).  (Smaller ones that come round at once are found in the memory-side cache.)
  if (p.group <= 4 * HT && rows >= (int64_t)128 * 1000 * 1000 / (2 * kHeadDim * 2)) return launch_decode<HT, 8, 4, true>(heads, p, stream);
  return launch_decode<HT, 8, 4, false>(heads, p, stream);
}

}  // namespace
}  // namespace dapq

using namespace dapq;

extern "C" DAPQ_API int dapq_decode_attention(const dapq_shape* shape, const void* q_decode, const void* k_cache,
                                              const void* v_cache, const int32_t* count, int32_t budget, float* out,
                                              void* stream) {
  int rc = check_shape(shape, false, false, false);
  if (rc != DAPQ_OK) return rc;
  DAPQ_REQUIRE(q_decode != nullptr && k_cache != nullptr && v_cache != nullptr && count != nullptr && out != nullptr,
               DAPQ_ERR_INVALID_ARG, "q_decode, k_cache, v_cache, count and out must not be NULL");
  DAPQ_REQUIRE(budget >= 1 && budget <= kDecodeMaxRows, DAPQ_ERR_UNSUPPORTED, "budget (%d) must be in [1, %d]", budget,
               kDecodeMaxRows);
  DAPQ_REQUIRE(isfinite(shape->scale) && shape->scale > 0.0f, DAPQ_ERR_INVALID_ARG, "scale must be finite and > 0");
  DAPQ_REQUIRE(((reinterpret_cast<uintptr_t>(k_cache) | reinterpret_cast<uintptr_t>(v_cache)) & 15) == 0,
               DAPQ_ERR_UNSUPPORTED, "k_cache and v_cache must be 16-byte aligned");
  DAPQ_REQUIRE(shape->batch <= 65535 && shape->n_layers <= 65535, DAPQ_ERR_UNSUPPORTED,
               "batch and n_layers must be <= 65535");
  DecodeParams p;
  p.q = static_cast<const uint16_t*>(q_decode);
  p.k_cache = static_cast<const uint16_t*>(k_cache);
  p.v_cache = static_cast<const uint16_t*>(v_cache);
  p.count = count;
  p.out = out;
  p.group = shape->n_q_heads / shape->n_kv_heads;
  p.budget = budget;
  p.c = shape->scale * 1.4426950408889634f;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t heads = (int64_t)shape->n_layers * shape->batch * shape->n_kv_heads;
  return p.group <= 4 ? launch_decode_slices<1>(heads, p, st) : launch_decode_slices<2>(heads, p, st);
}
