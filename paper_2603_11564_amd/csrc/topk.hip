// M_retain = TopK_j S(j) (Sec. 4.2): per (layer, sequence, KV head) the budget positions with the
// largest pooled score, equal scores lowest position first, written in ascending position.
//
// One workgroup per head (256 to 1024 threads of 8 to 64 keys, reg_kernel_for).  Selection is exact, on the
// order-preserving integer image of the fp32 score: it finds the threshold T (the budget-th largest key) and how many keys
// equal to T are still needed (topk_select; the streaming kernel takes T digit by digit with 256-bin histograms).  The
// last step is an ordered compaction: key j is kept if score > T, or score == T and fewer than `need` equal keys precede it;
// prefix counts of (greater, equal) give both the decision and the output slot, so the result is ascending and
// deterministic (no atomic decides an order).  Max-pooling makes runs of bit-equal scores, so the tie rule is on
// the main path.
//
// Heads of up to 65536 keys (topk_reg_kernel) are read from HBM once into registers, thread t
// owning the consecutive keys [t*KPT, (t+1)*KPT): every pass runs out of registers and the
// compaction needs a single workgroup scan.  Because a thread holds a run of consecutive scores, the
// same kernel can apply the max-pool that precedes selection (Sec. 1 / Sec. 5.1) on the way in
// (dapq_pool_topk): three halo scores per side for the window of 7, no pooled array in HBM.
// Longer heads go through the same kernel in pieces of 32768 keys, each leaving its survivors in candidate lists
// (caller's workspace), and topk_merge_kernel selects among the candidates of a head; without the workspace
// topk_stream_kernel stages what fits in LDS (36864 keys) or re-reads the scores on every pass.
#include "dapq_internal.h"
#include "kernel_args.h"
#include "wave_scan.h"

namespace dapq {
namespace {

constexpr int kTopkThreads = 1024;
constexpr int kTopkWaves = kTopkThreads / 64;
constexpr int kTopkLdsKeys = 36864;
constexpr int kStreamTiles = 4;                            // tiles of 4096 keys the streaming kernel has in flight
constexpr int kStreamLdsHead = 260 + kStreamTiles * 16 + 60;  // words of LDS in front of its staged keys (16-byte aligned)

// A value that is the same in all lanes, as a scalar.
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

struct TopkParams {
  const float* pooled;        // the scores selection runs on (the register variant can pool them itself)
  float* pooled_out;          // register variant with a pooling radius: where to write the pooled scores, or NULL
  const int32_t* cu_seqlens;
  const int32_t* budget_per_seq;
  int32_t* idx;
  int32_t* count;
  int64_t total_tokens;
  int32_t batch, n_kv_heads, budget;
  int32_t seq_len;            // dense batches: total_tokens / batch
  float inv_segs, inv_budget;
  int32_t min_len, max_len;  // this launch handles the heads with min_len <= L <= max_len
  // Long heads in pieces (cand_idx != NULL): workgroup (kv * n_segs + seg) selects among keys [seg * seg_len,
  // (seg + 1) * seg_len) of its head and leaves its survivors (order keys and positions in the head, ascending) and
  // their number in the candidate lists; topk_merge_kernel then selects among the candidates of a head.
  int32_t n_segs, seg_len;
  uint32_t* cand_key;   // [head][n_segs][budget]
  int32_t* cand_idx;    // [head][n_segs][budget]
  int32_t* cand_count;  // [head][n_segs]
};

// fp32 -> uint32 with the same order for all non-NaN values.
__device__ __forceinline__ uint32_t order_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// What every variant needs to know about its head; heads of another launch (length outside
// [min_len, max_len]), keep == 0 and keep == L are finished here.
struct TopkHead {
  const float* src;   // first score of the piece this workgroup selects from (the whole head, or a segment of it)
  int32_t* out;
  uint32_t* out_key;  // segments: where the survivors' keys go (else NULL)
  int L, keep;        // length of the piece, how many of it survive
  int base, head_len; // where the piece starts in its head, and the head's length (pooling windows cross pieces)
  bool done;          // nothing left to select
  bool foreign;       // the head belongs to another launch
};

// PIECES: the workgroup takes a piece of a long head.
template <bool PIECES>
__device__ __forceinline__ TopkHead topk_head(const TopkParams& p) {
  TopkHead hd;
  const int tid = threadIdx.x;
  const int nseg = PIECES ? p.n_segs : 1;
  const int kv = PIECES ? uniform_quotient((int)blockIdx.x, nseg, p.inv_segs) : (int)blockIdx.x, seg = (int)blockIdx.x - kv * nseg;
  const int b = blockIdx.y, layer = blockIdx.z;
  int64_t start;
  if (p.cu_seqlens == nullptr) {
    hd.head_len = p.seq_len;
    start = (int64_t)b * hd.head_len;
  } else {
    start = p.cu_seqlens[b];
    hd.head_len = p.cu_seqlens[b + 1] - (int)start;
  }
  hd.base = 0;
  hd.out_key = nullptr;
  hd.foreign = hd.head_len < p.min_len || hd.head_len > p.max_len;
  if (hd.foreign) {
    hd.done = true;
    hd.keep = 0;
    hd.L = 0;
    hd.out = nullptr;
    hd.src = nullptr;
    return hd;
  }
  int want = p.budget_per_seq ? p.budget_per_seq[b] : p.budget;
  want = want < 0 ? 0 : (want > p.budget ? p.budget : want);
  const int64_t head = ((int64_t)layer * p.batch + b) * p.n_kv_heads + kv;
  const float* head_src = p.pooled + ((int64_t)layer * p.n_kv_heads + kv) * p.total_tokens + start;
  if (PIECES) {
    hd.base = seg * p.seg_len;
    const int left = hd.head_len - hd.base;
    hd.L = left < 0 ? 0 : (left > p.seg_len ? p.seg_len : left);
    hd.keep = want < hd.L ? want : hd.L;
    const int64_t slot = head * nseg + seg;
    hd.out = p.cand_idx + slot * p.budget;
    hd.out_key = p.cand_key + slot * p.budget;
    hd.src = head_src + hd.base;
    if (tid == 0) p.cand_count[slot] = hd.keep;
    hd.done = hd.keep == 0;  // (a piece that survives whole still goes through the selection: its keys are wanted)
    return hd;
  }
  hd.L = hd.head_len;
  hd.keep = want < hd.L ? want : hd.L;
  hd.out = p.idx + head * p.budget;
  hd.src = head_src;
  if (tid == 0) p.count[head] = hd.keep;
  hd.done = hd.keep == 0;
  if (!hd.done && hd.keep == hd.L) {  // everything survives
    for (int j = tid; j < hd.L; j += (int)blockDim.x) hd.out[j] = j;
    hd.done = true;
  }
  return hd;
}

// After a histogram pass: wave 0 finds the digit d of T, the one with greater(d) < need <= greater(d)
// + hist[d], and publishes (d, need - greater(d), hist[d]) in bcast.
__device__ __forceinline__ void topk_pick_digit(const uint32_t* hist, uint32_t* bcast, int need, int lane) {
  // lane l owns digits 4l..4l+3; suffix sums over the lanes above, then inside the lane
  const uint32_t h0 = hist[4 * lane], h1 = hist[4 * lane + 1], h2 = hist[4 * lane + 2], h3 = hist[4 * lane + 3];
  const uint32_t mine = h0 + h1 + h2 + h3;
  const uint32_t upto = wave_scan<OpAdd>(mine);  // keys whose digit is <= 4l+3
  const uint32_t above = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63) - upto;  // keys whose digit is > 4l+3
  const uint32_t g3 = above, g2 = g3 + h3, g1 = g2 + h2, g0 = g1 + h1;  // keys with a larger digit
  const uint32_t un = (uint32_t)need;
  if (g3 < un && un <= g3 + h3) { bcast[0] = 4 * lane + 3; bcast[1] = un - g3; bcast[2] = h3; }
  if (g2 < un && un <= g2 + h2) { bcast[0] = 4 * lane + 2; bcast[1] = un - g2; bcast[2] = h2; }
  if (g1 < un && un <= g1 + h1) { bcast[0] = 4 * lane + 1; bcast[1] = un - g1; bcast[2] = h1; }
  if (g0 < un && un <= g0 + h0) { bcast[0] = 4 * lane + 0; bcast[1] = un - g0; bcast[2] = h0; }
}

// STAGED: the register variants of up to 32 keys per thread bring their head in through LDS (reg_kernel_for): the staging area of a wave is its
// threads' runs, KPT words each, and eight more words for the scores before and after them.  (64 keys per thread times 1024 threads do not fit.)
constexpr int reg_variant_wave_words(int kpt) { return 64 * kpt + 8; }
constexpr int reg_variant_rows_bytes(int threads, int kpt) { return threads / 64 * reg_variant_wave_words(kpt) * (int)sizeof(float); }
// (then the bins, which have a place of their own: a wave need not wait for the others until it counts)
constexpr int reg_variant_stage_bytes(int threads, int kpt) { return reg_variant_rows_bytes(threads, kpt) + threads * (int)sizeof(uint4); }
// Where the 16-byte piece `piece` of row `row` lies (in words), rows of KPT words: pieces XOR-swizzled so that sixteen threads next to
// each other find the same piece of their rows in sixteen different groups of banks.
template <int KPT>
__device__ __forceinline__ int stage_piece(int row, int piece) {
  constexpr int kPieces = KPT / 4, kShift = __builtin_ctz(16 / kPieces);
  static_assert(kPieces >= 1 && kPieces <= 16 && (kPieces & (kPieces - 1)) == 0, "whole rows of 16 pieces");
  return (row * kPieces + (piece ^ ((row >> kShift) & (kPieces - 1)))) * 4;
}

// bits = 16 * bits + the flags key > t of four keys, the first one on top: a compare and an add with carry per key.
// A carry may be read two wait states after the compare that made it, and neither the hardware nor the compiler sees to that
// inside inline assembly: the flags of four keys lie in four register pairs, three instructions stand between each compare and
// its add.  (t in a vector register: that one is free to read whenever it was written.)  As fast as compare and add in turn
// through one pair, without the waits: selection + gather of 8 and of 256 heads of 32768 keys 19.6 and 76.4 us either way.
__device__ __forceinline__ void push_greater(uint32_t& bits, const uint32_t* key, uint32_t t) {
  uint64_t c0, c1, c2, c3;
  asm("v_cmp_lt_u32 %1, %5, %6\n\tv_cmp_lt_u32 %2, %5, %7\n\tv_cmp_lt_u32 %3, %5, %8\n\tv_cmp_lt_u32 %4, %5, %9\n\t"
      "v_addc_co_u32 %0, %1, %0, %0, %1\n\tv_addc_co_u32 %0, %2, %0, %0, %2\n\t"
      "v_addc_co_u32 %0, %3, %0, %0, %3\n\tv_addc_co_u32 %0, %4, %0, %0, %4"
      : "+&v"(bits), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
      : "v"(t), "v"(key[0]), "v"(key[1]), "v"(key[2]), "v"(key[3]));
}

// ---- selection among the keys a workgroup holds in registers (KPT per thread, thread t's before thread t+1's):
// the `keep` largest, ties to the lowest position, handed to place(i, slot) in ascending position order (register
// i of the calling thread is survivor number `slot`; BY_REGISTER: i is known to the compiler, so that place can look into registers, and
// many survivors cost no more than few).  All threads have passed a barrier between their last use of `bins` and the first
// place().  A register without a key holds 0 (a key is at least 1); the workgroup has n_keys; `whole`: all registers of this wave hold keys.  keep >= 1 and at most n_keys.
// bins: LDS of THREADS uint4 that nobody else reads any more; thread t looks after bins 4t .. 4t+3.
//
// The threshold T (the keep-th largest key) is closed in on: [lo, lo + range] starts as the span of the keys and becomes,
// per pass, the one of 4 * THREADS equal bins that T lies in; when at most 64 candidates are left they are ranked by
// comparing all with all.  With sixteen waves to a compute unit the time is the vector instructions of a thread (16
// clocks each), and a pass is four per key: keys of scores span a few octaves, a bin is then a few thousandths of an
// octave, and one pass leaves a few dozen.  (Digits of the key instead -- sign and exponent, then 8 bits at a time --
// took 11 900 clocks for the first, whose bins are two octaves wide and are counted in packed fields, and 12 600 for the
// others.)  Keys in the lowest bin are not counted one by one: they are what the other bins leave over, so that a head full of
// zeros does not queue up at one address.  Nor are those of a bin above it that a wave's keys crowd into: the wave counts them in
// registers and adds the sum (heads of one value with one key below it: 8 of 32768 keys 94 us without, 17 with; 256 of 8192
// 27 and 10).  Kept positions are bits of a word per 32 keys, and the survivors are walked bit by bit.  Selection with pooling, by
// digits -> by bins: 8 heads of 32768 keys, 983 kept, 21.5 -> 15.9 us; 256 heads 28.8 -> 18.7; 64 heads of 131072 keys, 3932
// kept, in pieces 65 -> 43; 256 heads of 2000 keys, 128 kept, 14.9 -> 11.8.
// Of 27 000 clocks of one workgroup over 32768 keys (33 000 with a test per register for whether it holds a key, candidates looked
// for register by register and ranked by one wave) 24 000 are left: arguments 800, loading 4100 (11 400 with 256 heads), dealing out
// and pooling 2000, keys and their span 3000, bins 6800 (a wave's LDS addition takes 12 clocks however many of its lanes add,
// and whether or not the loop masks them), bits and ranks 3800, compaction 3000.  With the gather: 8 heads 19.1 -> 15.9 us, 64 heads
// of 131072 keys in pieces 88.2 -> 82.9.  (Two and four times the bins, which leave fewer candidates: 17.1 -> 17.2 and 18.3 us.)
constexpr int kRankMax = 64;  // candidates that are ranked
constexpr int kCrowd = 3;     // neighbouring lanes of 60 with keys of one bin: a bin that holds a fifth of them (in a spread of keys, 0.1)
template <int THREADS, int KPT, bool BY_REGISTER, class Place>
__device__ __forceinline__ void topk_select(const uint32_t (&key)[KPT], int n_keys, int keep, uint4* bins, bool whole,
                                            Place place) {
  constexpr int kWaves = THREADS / 64, kWords = (KPT + 31) / 32, kBins = 4 * THREADS;
  static_assert(KPT % 4 == 0 && (KPT < 32 || KPT % 32 == 0), "whole quads and whole words of position bits");
  static_assert((kBins & (kBins - 1)) == 0 && kWaves <= 64, "bins and waves");
  __shared__ uint32_t wave_min[kWaves], wave_max[kWaves], wave_count[kWaves];
  __shared__ uint32_t found[3];  // bin, need, population of the bin
  __shared__ uint32_t last[kRankMax], ranks[kRankMax];
  __shared__ uint32_t last_n;
  __shared__ uint32_t wave_gt[kWaves], wave_eq[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  uint32_t lo, range, left = (uint32_t)n_keys;  // candidates: the `left` keys with key - lo <= range
  int need = keep;
  {
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
    if (whole) {
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        kmin = key[i] < kmin ? key[i] : kmin;
        kmax = key[i] > kmax ? key[i] : kmax;
      }
      kmin -= 1u;
    } else {  // (a register without a key holds 0: key - 1 wraps to the largest value and never is the minimum)
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        kmin = key[i] - 1u < kmin ? key[i] - 1u : kmin;
        kmax = key[i] > kmax ? key[i] : kmax;
      }
    }
    kmin = wave_scan<OpMin>(kmin);
    kmax = wave_scan<OpMax>(kmax);
    if (lane == 63) {
      wave_min[wave] = kmin;
      wave_max[wave] = kmax;
    }
    bins[tid] = make_uint4(0, 0, 0, 0);
    if (tid == 0) last_n = 0;
    if (tid < kRankMax) ranks[tid] = 0;
    __syncthreads();
    kmin = wave_scan<OpMin>(lane < kWaves ? wave_min[lane] : 0xFFFFFFFFu);  // (lane 63 has all of them)
    kmax = wave_scan<OpMax>(lane < kWaves ? wave_max[lane] : 0u);
    kmin = (uint32_t)__builtin_amdgcn_readlane((int)kmin, 63);
    kmax = (uint32_t)__builtin_amdgcn_readlane((int)kmax, 63);
    lo = uniform(kmin) + 1u;
    range = uniform(kmax) - lo;
  }
  while (range != 0u && left > (uint32_t)kRankMax) {
    const int bits = 32 - __builtin_clz(range), shift = bits > __builtin_ctz(kBins) ? bits - __builtin_ctz(kBins) : 0;
    // from the second bin on (range >= 1 << shift); keys that are no candidates and empty registers are not in it
    const uint32_t lo1 = lo + (1u << shift), range1 = range - (1u << shift);
    uint32_t* count = reinterpret_cast<uint32_t*>(bins) + 1;
    // Whether the wave's keys crowd into a bin: one register of all lanes, compared with the neighbouring lane's
    const uint32_t sample = key[KPT / 2] - lo1 <= range1 ? (key[KPT / 2] - lo1) >> shift : 0xFFFFFFFFu;
    const uint64_t equal = __ballot(sample != 0xFFFFFFFFu && sample == dpp_take<kDppRowShr1, 0xf>(0xFFFFFFFFu, sample));
    if (__popcll(equal) < kCrowd) {
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        if (key[i] - lo1 <= range1) atomicAdd(&count[(key[i] - lo1) >> shift], 1u);
      }
    } else {
      const uint32_t crowded = (uint32_t)__builtin_amdgcn_readlane((int)sample, __ffsll((long long)equal) - 1);
      const uint32_t crowd_at = crowded << shift;  // above lo1
      const uint32_t crowd_range = range1 - crowd_at < (1u << shift) - 1u ? range1 - crowd_at : (1u << shift) - 1u;
      uint32_t same = 0;
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        const uint32_t at = key[i] - lo1;
        if (at - crowd_at <= crowd_range) ++same;
        else if (at <= range1) atomicAdd(&count[at >> shift], 1u);
      }
      same = wave_sum(same);
      if (lane == 0) atomicAdd(&count[crowded], same);
    }
    __syncthreads();
    uint4 c = bins[tid];
    bins[tid] = make_uint4(0, 0, 0, 0);
    const uint32_t upto = wave_scan<OpAdd>(c.x + c.y + c.z + c.w);
    if (lane == 63) wave_count[wave] = upto;
    __syncthreads();
    // candidates in this wave's bins and below / in all bins but the lowest
    uint32_t below = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint32_t n = wave_count[w];
      below += w < wave ? n : 0u;
      all += n;
    }
    if (tid == 0) c.x = left - all;
    // g3 .. g0: candidates in a higher bin than 4t+3 .. 4t
    const uint32_t g3 = all - (below + upto), g2 = g3 + c.w, g1 = g2 + c.z, g0 = g1 + c.y, un = (uint32_t)need;
    if (g3 < un && un <= g0 + c.x) {
      const int k = un <= g2 ? 3 : (un <= g1 ? 2 : (un <= g0 ? 1 : 0));
      found[0] = (uint32_t)(4 * tid + k);
      found[1] = un - (k == 3 ? g3 : (k == 2 ? g2 : (k == 1 ? g1 : g0)));
      found[2] = k == 3 ? c.w : (k == 2 ? c.z : (k == 1 ? c.y : c.x));
    }
    __syncthreads();
    const uint32_t bin = uniform(found[0]), width = (1u << shift) - 1u, rest = range - (bin << shift);
    lo += bin << shift;
    range = rest < width ? rest : width;
    need = (int)uniform(found[1]);
    left = uniform(found[2]);
    // (found is written again only behind the next pass's barriers)
  }
  // ---- which keys are above the span and which are in it, a bit each (lo >= 1: registers without a key are neither)
  uint32_t gt[kWords], eq[kWords], my_gt = 0, my_eq = 0;
#pragma unroll
  for (int w = 0; w < kWords; ++w) {
    gt[w] = eq[w] = 0;
#pragma unroll
    for (int i = 32 * w; i < KPT && i < 32 * w + 32; i += 4) {
      push_greater(gt[w], &key[i], lo + range);
      push_greater(eq[w], &key[i], lo - 1u);
    }
    eq[w] &= ~gt[w];
  }
  if (range != 0u) {
    // the candidates of a thread go to the list one after the other; registers that no thread of the wave has one in are
    // passed over four at a time
    uint32_t mine = 0;
#pragma unroll
    for (int w = 0; w < kWords; ++w) mine += (uint32_t)__popc(eq[w]);
    uint32_t at = 0;
    if (mine != 0) at = atomicAdd(&last_n, mine);
    const uint32_t first_at = at;
#pragma unroll
    for (int i = 0; i < KPT; i += 4) {
      const int top = KPT - i / 32 * 32 < 32 ? KPT - i / 32 * 32 - 1 : 31;
      const uint32_t four = (eq[i / 32] >> (top - i % 32 - 3)) & 15u;
      if (__any((int)four)) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (four & (8u >> u)) last[at++] = key[i + u];
      }
    }
    __syncthreads();
    // all with all: lane = candidate, every wave compares it with its share of them (one wave alone: up to 3000 clocks while the
    // others wait)
    const uint32_t v = (uint32_t)lane < left ? last[lane] : 0u;
    uint32_t rank = 0;  // candidates above this one, and (<< 16) the same as this one
    for (int e = wave; e < (int)left; e += kWaves) {
      const uint32_t o = last[e];
      rank += o > v ? 1u : (o == v ? 0x10000u : 0u);
    }
    if (wave < (int)left) atomicAdd(&ranks[lane], rank);
    __syncthreads();
    rank = ranks[lane];
    const int above = (int)(rank & 0xFFFFu), same = (int)(rank >> 16);
    const uint64_t hit = __ballot((uint32_t)lane < left && above < need && need <= above + same);  // (equal keys hit together)
    const int first = __ffsll((long long)hit) - 1;
    const uint32_t T = (uint32_t)__builtin_amdgcn_readlane((int)v, first);
    need -= __builtin_amdgcn_readlane(above, first);
    at = first_at;
#pragma unroll
    for (int w = 0; w < kWords; ++w) {
      uint32_t rest = eq[w];
      while (rest != 0) {  // (first register on top)
        const uint32_t bit = 0x80000000u >> __clz((int)rest);
        const uint32_t k = last[at++];
        rest ^= bit;
        if (k > T) gt[w] |= bit;
        if (k != T) eq[w] ^= bit;
      }
    }
  }

  // ---- ordered compaction: one exclusive scan of the per-thread (greater, equal) counts
#pragma unroll
  for (int w = 0; w < kWords; ++w) {
    my_gt += (uint32_t)__popc(gt[w]);
    my_eq += (uint32_t)__popc(eq[w]);
  }
  const uint32_t inc_gt = wave_scan<OpAdd>(my_gt), inc_eq = wave_scan<OpAdd>(my_eq);  // inclusive, inside the wave
  if (lane == 63) {
    wave_gt[wave] = inc_gt;
    wave_eq[wave] = inc_eq;
  }
  __syncthreads();
  uint32_t pre_gt = inc_gt - my_gt, pre_eq = inc_eq - my_eq;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) {
      pre_gt += wave_gt[w];
      pre_eq += wave_eq[w];
    }
  }
  const uint32_t un = (uint32_t)need;
  uint32_t pos = pre_gt + (pre_eq < un ? pre_eq : un);
  uint32_t room = pre_eq < un ? un - pre_eq : 0u;  // equal keys of this thread that are still taken
#pragma unroll
  for (int w = 0; w < kWords; ++w) {
    const int top = KPT - 32 * w < 32 ? KPT - 32 * w - 1 : 31;
    uint32_t e = room != 0 ? eq[w] : 0u;
    while ((uint32_t)__popc(e) > room) e &= e - 1;  // the last ones go: the lowest bits are the last registers
    room -= (uint32_t)__popc(e);
    uint32_t take = gt[w] | e;
    if constexpr (BY_REGISTER) {
#pragma unroll
      for (int i = 32 * w; i < KPT && i < 32 * w + 32; ++i) {
        if ((take >> (top - i % 32)) & 1u) place(i, pos++);
      }
    } else {
      while (take != 0) {
        const int bit = 31 - __clz((int)take);
        take ^= 1u << bit;
        place(32 * w + top - bit, pos++);
      }
    }
  }
}

// The largest of the 2R + 1 scores from ext[i] on (R == 3: of the maxima of three that ext holds by then).
template <int R, int N>
__device__ __forceinline__ float window_max(const float (&ext)[N], int i) {
  if constexpr (R == 3) return fmaxf(fmaxf(ext[i], ext[i + 2]), ext[i + 4]);
  float m = ext[i];
#pragma unroll
  for (int t = 1; t <= 2 * R; ++t) m = fmaxf(m, ext[i + t]);
  return m;
}

// ---- heads that fit in registers.  R > 0: the input is the un-pooled score and the kernel applies
// the max-pool of radius R itself (window clipped at the ends of the sequence) before selecting.
template <int THREADS, int KPT, int R, bool PIECES, bool STAGED>
__global__ __launch_bounds__(THREADS) void topk_reg_kernel(TopkParams p) {
  static_assert(!PIECES || STAGED, "the keys of a piece's survivors go through the staging area");
  touch_args<sizeof(TopkParams)>();
  const int tid = threadIdx.x;
  const TopkHead hd = topk_head<PIECES>(p);
  if (hd.foreign || (hd.done && p.pooled_out == nullptr)) return;  // a finished head may still owe its pooled scores
  const int L = hd.L;
  // position j of this piece is a position of its head (the pooling window does not stop at the end of a piece)
  auto in_head = [&](int j) { return (unsigned)(hd.base + j) < (unsigned)hd.head_len; };

  // thread t owns keys [t*KPT, t*KPT + KPT): registers i < nvalid hold a key.  (A layout with
  // contiguous rows per wave makes the compaction twice as long.)
  const int j0 = tid * KPT;
  const int nvalid = L - j0 < 0 ? 0 : (L - j0 > KPT ? KPT : L - j0);
  // (a wave whose threads all have KPT keys is spared the tests)
  const bool whole = __all(nvalid == KPT);
  float ext[KPT + 2 * R];  // scores j0-R .. j0+KPT+R-1; -inf outside the sequence
  if constexpr (STAGED) {
    // A wave brings in its own keys with coalesced loads (a thread reading its run straight from memory makes every load instruction
    // touch 64 cache lines) and deals them out to its threads through its part of the staging area; the scores before and
    // after them, of which the windows at its ends take some, come along.  Nothing is shared with the other waves: those whose keys
    // arrive first pool them while the others wait.  Pooling, selection and gather of 8 heads of 32768 keys 15.7 -> 14.9 us, 256 heads
    // 72.9 -> 71.5; 32 of 8757 keys, straight from memory before, 20.2 -> 16.7.
    extern __shared__ float stage_area[];
    static_assert(R <= 4, "the halo of a run is read as one 16-byte piece of each neighbouring row");
    const int lane = tid & 63, first = (tid - lane) * KPT;
    float* rows = stage_area + (tid >> 6) * reg_variant_wave_words(KPT);
    if (first < L) {
      float halo = -INFINITY;
      if (R > 0 && lane < 8) {
        const int j = lane < 4 ? first - 4 + lane : first + 64 * KPT + (lane - 4);
        if (in_head(j)) halo = hd.src[j];
      }
      if ((reinterpret_cast<uintptr_t>(hd.src) & 15) == 0) {
        float4 v[KPT / 4];
#pragma unroll
        for (int it = 0; it < KPT / 4; ++it) {
          const int g = first + (it * 64 + lane) * 4;
          if (g + 4 <= L) {
            v[it] = *reinterpret_cast<const float4*>(hd.src + g);
          } else {
            v[it] = make_float4(g < L ? hd.src[g] : 0.0f, g + 1 < L ? hd.src[g + 1] : 0.0f, g + 2 < L ? hd.src[g + 2] : 0.0f, 0.0f);
          }
        }
#pragma unroll
        for (int it = 0; it < KPT / 4; ++it) {
          const int at = it * 64 + lane;
          *reinterpret_cast<float4*>(rows + stage_piece<KPT>(at / (KPT / 4), at % (KPT / 4))) = v[it];
        }
      } else {
        // Heads of an odd length follow each other: words instead of quads, all of them in flight (one by one: with the gather 128 heads
        // of 53063 keys 75.3 us, now 64.8; 32 of 60001 39.1, now 29.2).
        float v[KPT];
#pragma unroll
        for (int it = 0; it < KPT; ++it) {
          const int j = first + it * 64 + lane;
          v[it] = hd.src[j < L ? j : L - 1];
        }
#pragma unroll
        for (int it = 0; it < KPT; ++it) {
          const int at = it * 64 + lane;
          rows[stage_piece<KPT>(at / KPT, at % KPT / 4) + at % 4] = v[it];
        }
      }
      if (R > 0 && lane < 8) rows[64 * KPT + lane] = halo;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // (words that no key of the head was written to are never selected below)
#pragma unroll
    for (int i = 0; i < KPT; i += 4) {
      const float4 v = *reinterpret_cast<const float4*>(rows + stage_piece<KPT>(lane, i / 4));
      ext[R + i] = v.x;
      ext[R + i + 1] = v.y;
      ext[R + i + 2] = v.z;
      ext[R + i + 3] = v.w;
    }
    if (!whole) {
#pragma unroll
      for (int i = 0; i < KPT; ++i) ext[R + i] = i < nvalid ? ext[R + i] : -INFINITY;
    }
    if (R > 0) {
      const float4 lv = *reinterpret_cast<const float4*>(rows + (lane > 0 ? stage_piece<KPT>(lane - 1, KPT / 4 - 1) : 64 * KPT));
      const float4 rv = *reinterpret_cast<const float4*>(rows + (lane < 63 ? stage_piece<KPT>(lane + 1, 0) : 64 * KPT + 4));
      const float left[4] = {lv.x, lv.y, lv.z, lv.w}, right[4] = {rv.x, rv.y, rv.z, rv.w};
#pragma unroll
      for (int r = 0; r < R; ++r) {  // (words of the area nobody wrote lie outside the head)
        ext[r] = in_head(j0 - R + r) ? left[4 - R + r] : -INFINITY;
        ext[R + KPT + r] = in_head(j0 + KPT + r) ? right[r] : -INFINITY;
      }
    }
  } else {
    if (nvalid == KPT && (reinterpret_cast<uintptr_t>(hd.src + j0) & 15) == 0) {
#pragma unroll
      for (int i = 0; i < KPT; i += 4) {
        const float4 v = *reinterpret_cast<const float4*>(hd.src + j0 + i);
        ext[R + i] = v.x;
        ext[R + i + 1] = v.y;
        ext[R + i + 2] = v.z;
        ext[R + i + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < KPT; ++i) ext[R + i] = i < nvalid ? hd.src[j0 + i] : -INFINITY;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int jl = j0 - R + r, jr = j0 + KPT + r;
      ext[r] = in_head(jl) ? hd.src[jl] : -INFINITY;
      ext[R + KPT + r] = in_head(jr) ? hd.src[jr] : -INFINITY;
    }
  }
  if constexpr (R == 3) {
    // the window of 7 in two steps: ext[j] becomes the largest of three, and three of those cover the window
#pragma unroll
    for (int j = 0; j < KPT + 4; ++j) ext[j] = fmaxf(fmaxf(ext[j], ext[j + 1]), ext[j + 2]);
  }
  uint32_t key[KPT];
  uint32_t signs = 0;
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    key[i] = __float_as_uint(window_max<R>(ext, i));
    signs |= key[i];
  }
  if (KPT > 32 || __any((int)signs < 0)) {
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      const uint32_t k = order_key(__uint_as_float(key[i]));
      key[i] = k > 1u ? k : 1u;
    }
  } else {  // no negative score in this wave, as in sums of weights: one operation per key instead of four
#pragma unroll
    for (int i = 0; i < KPT; ++i) key[i] |= 0x80000000u;
  }
  if (p.pooled_out != nullptr) {
#pragma unroll
    for (int i = 0; i < KPT; ++i)
      if (i < nvalid) p.pooled_out[(hd.src - p.pooled) + j0 + i] = window_max<R>(ext, i);
  }
  // registers past the end of the head hold 0, which no key is (a key is at least 1): everything below can then
  // tell them by value, and no per-register validity mask has to stay alive through the kernel
  if (!whole) {
#pragma unroll
    for (int i = 0; i < KPT; ++i) key[i] = i < nvalid ? key[i] : 0u;
  }
  if (hd.done) return;

  // The survivors go out through LDS where there is room (the staging area, which everybody has read by then): whole cache lines
  // instead of a few words of many.  64 heads of 131072 keys, 3932 kept: pieces 24.6 -> 18.3 us, and the merge, whose lists came in 64 bytes
  // to a thread and whose positions were fetched one by one, 14.1 -> 12.2.
  if constexpr (STAGED) {
    extern __shared__ float stage_area[];
    uint4* bins = reinterpret_cast<uint4*>(stage_area + reg_variant_rows_bytes(THREADS, KPT) / (int)sizeof(float));
    if constexpr (PIECES) {
      constexpr int kRoom = reg_variant_rows_bytes(THREADS, KPT) / (int)sizeof(uint2);
      uint2* kept = reinterpret_cast<uint2*>(stage_area);
      const bool room = hd.keep <= kRoom;
      topk_select<THREADS, KPT, true>(key, L, hd.keep, bins, whole, [&](int i, uint32_t slot) {
        if (room) {
          kept[slot] = make_uint2(key[i], (uint32_t)(hd.base + j0 + i));
        } else {
          hd.out_key[slot] = key[i];
          hd.out[slot] = hd.base + j0 + i;
        }
      });
      if (!room) return;
      __syncthreads();
      for (int s = tid; s < hd.keep; s += THREADS) {
        const uint2 v = kept[s];
        hd.out_key[s] = v.x;
        hd.out[s] = (int32_t)v.y;
      }
    } else {
      int32_t* kept = reinterpret_cast<int32_t*>(stage_area);
      topk_select<THREADS, KPT, false>(key, L, hd.keep, bins, whole, [&](int i, uint32_t slot) { kept[slot] = j0 + i; });
      __syncthreads();
      for (int s = tid; s < hd.keep; s += THREADS) hd.out[s] = kept[s];
    }
  } else {
    __shared__ uint4 bins[THREADS];
    topk_select<THREADS, KPT, false>(key, L, hd.keep, bins, whole, [&](int i, uint32_t slot) { hd.out[slot] = j0 + i; });
  }
}

// ---- a long head whose pieces have been through topk_reg_kernel: the `keep` largest of the candidates they left.
// A thread owns KPT consecutive slots of the head's [n_segs][budget] candidate lists; the slots a piece did not fill
// are empty.  Candidates are in ascending position inside a list and the lists in piece order, so ties still go to
// the lowest position and the result is ascending.
constexpr int kTopkMaxSegs = 64;
// Up to 32 slots to a thread, a wave's part of the candidate lists comes in with coalesced loads and is dealt out to its threads through
// rows of LDS, as in topk_reg_kernel (a thread reading its own run straight from memory makes every load touch 64 cache lines); the
// area is then the bins', and in the end the survivors'.
constexpr bool merge_variant_is_staged(int kpt) { return kpt <= 32; }
constexpr int merge_variant_bytes(int threads, int kpt) {
  return merge_variant_is_staged(kpt) ? threads * (kpt + 4) * (int)sizeof(int32_t) : 0;
}
template <int THREADS, int KPT>
__global__ __launch_bounds__(THREADS) void topk_merge_kernel(TopkParams p) {
  __shared__ int32_t seg_count[kTopkMaxSegs];
  touch_args<sizeof(TopkParams)>();
  const int tid = threadIdx.x;
  const int kv = blockIdx.x, b = blockIdx.y, layer = blockIdx.z;
  int L;
  if (p.cu_seqlens == nullptr) L = p.seq_len;
  else L = p.cu_seqlens[b + 1] - p.cu_seqlens[b];
  if (L < p.min_len || L > p.max_len) return;
  int want = p.budget_per_seq ? p.budget_per_seq[b] : p.budget;
  want = want < 0 ? 0 : (want > p.budget ? p.budget : want);
  const int keep = want < L ? want : L;
  const int64_t head = ((int64_t)layer * p.batch + b) * p.n_kv_heads + kv;
  if (tid == 0) p.count[head] = keep;
  if (keep == 0) return;
  const int nseg = p.n_segs, slots = nseg * p.budget;
  int32_t of_seg = 0;
  if (tid < nseg) of_seg = p.cand_count[head * nseg + tid];
  const uint32_t* ck = p.cand_key + head * slots;
  const int32_t* ci = p.cand_idx + head * slots;
  int32_t* out = p.idx + head * p.budget;
  const int s0 = tid * KPT;
  int seg = quotient(s0, p.inv_budget), r = s0 - seg * p.budget;  // (at most 65536 slots)
  // (slots that hold no candidate are read too: the workspace's old contents, which are dropped)
  const bool quads = (slots & 3) == 0 && (reinterpret_cast<uintptr_t>(ck) & 15) == 0;
  constexpr bool kStaged = merge_variant_is_staged(KPT);
  constexpr int kRow = KPT + 4;
  extern __shared__ float stage_area[];
  uint32_t* rows = reinterpret_cast<uint32_t*>(stage_area);
  uint32_t key[KPT], at[KPT];
  // val[i] = list[s0 + i], for the slots there are
  auto load_run = [&](const uint32_t* list, uint32_t (&val)[KPT]) {
    if constexpr (kStaged) {
      const int lane = tid & 63, first = (tid - lane) * KPT;  // a wave's own slots: nothing is shared with the others
      if (quads) {
#pragma unroll
        for (int i = 0; i < KPT; i += 4) {
          const int g = first + i * 64 + lane * 4;
          if (g < slots) *reinterpret_cast<uint4*>(&rows[g / KPT * kRow + g % KPT]) = *reinterpret_cast<const uint4*>(list + g);
        }
      } else {
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
          const int g = first + i * 64 + lane;
          if (g < slots) rows[g / KPT * kRow + g % KPT] = list[g];
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int i = 0; i < KPT; i += 4) {
        const uint4 v = *reinterpret_cast<const uint4*>(&rows[tid * kRow + i]);
        val[i] = v.x;
        val[i + 1] = v.y;
        val[i + 2] = v.z;
        val[i + 3] = v.w;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (the next list goes through the same rows)
    } else {
#pragma unroll
      for (int i = 0; i < KPT; i += 4) {
        if (quads && s0 + i < slots) {
          const uint4 v = *reinterpret_cast<const uint4*>(list + s0 + i);
          val[i] = v.x;
          val[i + 1] = v.y;
          val[i + 2] = v.z;
          val[i + 3] = v.w;
        } else if (!quads) {
#pragma unroll
          for (int u = 0; u < 4; ++u) val[i + u] = s0 + i + u < slots ? list[s0 + i + u] : 0u;
        }
      }
    }
  };
  load_run(ck, key);
  if constexpr (kStaged) load_run(reinterpret_cast<const uint32_t*>(ci), at);
  if (tid < nseg) seg_count[tid] = of_seg;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const bool valid = s0 + i < slots && r < seg_count[seg < nseg ? seg : 0];
    key[i] = valid ? key[i] : 0u;
    if (++r == p.budget) {
      r = 0;
      ++seg;
    }
  }
  int n_keys = 0;
  for (int i = 0; i < nseg; ++i) n_keys += seg_count[i];
  if constexpr (kStaged) {
    // (all rows have been read: there was a barrier)
    int32_t* kept = reinterpret_cast<int32_t*>(stage_area);
    topk_select<THREADS, KPT, true>(key, n_keys, keep, reinterpret_cast<uint4*>(stage_area), false,
                                    [&](int i, uint32_t slot) { kept[slot] = (int32_t)at[i]; });
    __syncthreads();
    for (int s = tid; s < keep; s += THREADS) out[s] = kept[s];
  } else {
    __shared__ uint4 bins[THREADS];
    topk_select<THREADS, KPT, false>(key, n_keys, keep, bins, false, [&](int i, uint32_t slot) { out[slot] = ci[s0 + i]; });
  }
}

// ---- longer heads
__global__ __launch_bounds__(kTopkThreads) void topk_stream_kernel(TopkParams p) {
  extern __shared__ uint32_t smem[];
  uint32_t* hist = smem;             // [256]
  uint32_t* bcast = smem + 256;      // [3]: digit, need, population of the digit
  uint32_t* wave_tot = smem + 260;   // [kStreamTiles][16]
  uint32_t* keys = smem + kStreamLdsHead;  // [kTopkLdsKeys] staged order keys (if they fit)

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const TopkHead hd = topk_head<false>(p);
  if (hd.done) return;
  const int L = hd.L;
  const float* src = hd.src;
  int32_t* out = hd.out;
  const bool staged = L <= kTopkLdsKeys;
  if (staged) {
    for (int j = tid; j < L; j += kTopkThreads) keys[j] = order_key(src[j]);
  }
  __syncthreads();
  // a thread takes four consecutive keys per trip (one 16-byte load when the head is 16-byte aligned): a trip is a
  // tile of 4096 keys, thread t owning keys [4t, 4t + 4) of it.  Keys past the end read as 0 and are never candidates.
  const bool aligned = (reinterpret_cast<uintptr_t>(src) & 15) == 0;
  auto keys_at = [&](int j, uint32_t (&k)[4]) {
    if (staged) {
      if (j + 3 < L) {
        const uint4 v = *reinterpret_cast<const uint4*>(keys + j);  // keys is 16-byte aligned, j a multiple of 4
        k[0] = v.x; k[1] = v.y; k[2] = v.z; k[3] = v.w;
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) k[u] = j + u < L ? keys[j + u] : 0u;
      }
    } else if (aligned && j + 3 < L) {
      const float4 v = *reinterpret_cast<const float4*>(src + j);
      k[0] = order_key(v.x); k[1] = order_key(v.y); k[2] = order_key(v.z); k[3] = order_key(v.w);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) k[u] = j + u < L ? order_key(src[j + u]) : 0u;
    }
  };
  constexpr int kTile = 4 * kTopkThreads;
  // kStreamTiles tiles per trip, all their loads issued before the first key is looked at: with one workgroup per
  // head a pass is a chain of load latencies, and this is how many of them overlap

  // ---- radix select: threshold T = the keep-th largest key, need = how many keys == T to take
  uint32_t prefix = 0, mask = 0;
  int need = hd.keep;
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (int jb = 0; jb < L; jb += kStreamTiles * kTile) {  // the trip count is the same for every thread
      uint32_t k[kStreamTiles][4];
#pragma unroll
      for (int t = 0; t < kStreamTiles; ++t) keys_at(jb + t * kTile + 4 * tid, k[t]);
#pragma unroll
      for (int t = 0; t < kStreamTiles; ++t) {
        const int j = jb + t * kTile + 4 * tid;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bool cand = j + u < L && (k[t][u] & mask) == prefix;
          const uint32_t d = (k[t][u] >> shift) & 255u;
          const uint64_t have = __ballot(cand);
          if (have != 0) {
            const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, __ffsll((long long)have) - 1);
            const uint64_t same = __ballot(cand && d == d0);
            if (cand && d != d0) atomicAdd(&hist[d], 1u);
            if (lane == 0) atomicAdd(&hist[d0], (uint32_t)__popcll(same));
          }
        }
      }
    }
    __syncthreads();
    if (wave == 0) topk_pick_digit(hist, bcast, need, lane);
    __syncthreads();
    prefix |= bcast[0] << shift;
    mask |= 255u << shift;
    need = (int)bcast[1];
    __syncthreads();
  }
  const uint32_t T = prefix;

  // ---- ordered compaction, kStreamTiles tiles of 4096 keys at a time: per-thread counts of (greater, equal) in
  // each tile, an inclusive scan inside the wave, wave totals through LDS, then every thread writes its survivors
  // in key order (all keys of a tile come before those of the next)
  uint32_t base_gt = 0, base_eq = 0;  // keys > T / == T before the current tile (same in all threads)
  const uint32_t un = (uint32_t)need;
  for (int jb = 0; jb < L; jb += kStreamTiles * kTile) {
    uint32_t k[kStreamTiles][4], my[kStreamTiles], inc[kStreamTiles];
#pragma unroll
    for (int t = 0; t < kStreamTiles; ++t) keys_at(jb + t * kTile + 4 * tid, k[t]);
#pragma unroll
    for (int t = 0; t < kStreamTiles; ++t) {
      const int j = jb + t * kTile + 4 * tid;
      my[t] = 0;  // (greater << 16) | equal over this thread's four keys of the tile
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (j + u < L) my[t] += (k[t][u] > T ? 0x10000u : 0u) + (k[t][u] == T ? 1u : 0u);
      }
      inc[t] = wave_scan<OpAdd>(my[t]);
      if (lane == 63) wave_tot[t * kTopkWaves + wave] = inc[t];
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kStreamTiles; ++t) {
      const int j = jb + t * kTile + 4 * tid;
      uint32_t pre = inc[t] - my[t], blk = 0;  // packed counts before this thread inside the tile / of the whole tile
#pragma unroll
      for (int w = 0; w < kTopkWaves; ++w) {
        const uint32_t tot = wave_tot[t * kTopkWaves + w];
        if (w < wave) pre += tot;
        blk += tot;
      }
      uint32_t pre_gt = base_gt + (pre >> 16), pre_eq = base_eq + (pre & 0xFFFFu);
      if (my[t] != 0) {
        uint32_t pos = pre_gt + (pre_eq < un ? pre_eq : un);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (j + u < L) {
            if (k[t][u] > T) {
              out[pos++] = j + u;
            } else if (k[t][u] == T) {
              if (pre_eq < un) out[pos++] = j + u;
              ++pre_eq;
            }
          }
        }
      }
      base_gt += blk >> 16;
      base_eq += blk & 0xFFFFu;
    }
    __syncthreads();
  }
}

}  // namespace
}  // namespace dapq

using namespace dapq;

namespace dapq {
namespace {

// Register-variant shapes: (threads, keys per thread).  Short heads use small workgroups so that
// several of them share a compute unit.
struct RegVariant {
  int threads, kpt;
  bool staged;  // the scores through LDS
  int64_t max_len() const { return (int64_t)threads * kpt; }
};

RegVariant reg_variant_for(int64_t len) {
  if (len <= 256 * 32) return {256, 32, true};
  if (len <= 512 * 32) return {512, 32, true};  // (32 keys per thread is the lean code: 64 per thread spills scalar registers)
  if (len <= 1024 * 32) return {1024, 32, true};
  return {1024, 64, false};
}

// The kernel for a launch of `heads` heads of at most `longest` keys, and `mean` on average, that variant v holds.  Eight keys to a thread instead of 32 make
// four times the waves, which hide each other's waits, of as many instructions; up to 4096 keys they are also the faster ones where
// several workgroups share a compute unit, beyond that only while there is one for every head.  Pooling and selection, us, 8 / 256 /
// 512 / 1024 heads: 1000 keys 256 x 32 8.3 / 9.0 / 9.8 / 12.5, 256 x 8 5.7 / 6.2 / 6.6 / 7.6; 4000 keys 256 x 32 8.6 / 9.1 / 10.2 / 13.1,
// 512 x 8 6.2 / 6.7 / 8.1 / 11.0; 8000 keys 256 x 32 8.8 / 9.5 / 10.6 / 14.6, 1024 x 8 7.8 / 8.6 / 11.9 / 20.9.  (16000 keys: 512 x 32 10.0 /
// 10.6 / 15.0, 1024 x 16 9.8 / 10.6 / 20.3.)
RegVariant reg_kernel_for(RegVariant v, int64_t longest, int64_t mean, int64_t heads) {
  if (longest <= 256 * 8) return {256, 8, true};
  if (longest <= 512 * 8) return {512, 8, true};
  if (longest <= 1024 * 8 && heads <= 256) return {1024, 8, true};
  // Many heads of a ragged batch that are much shorter than the workgroup could hold: the staging area, of which they use the start, lets four
  // workgroups of 256 threads (two of 512) share a compute unit, registers would let seven.  Us, through LDS -> straight from memory: 1280
  // heads of 1083 keys on average 17.5 -> 14.9, 4096 of 783 47.2 -> 41.7 (without a workspace, 512 threads, 69.4 -> 56.6), 4096 of 1872
  // 49.8 -> 45.3; 1024 of 822 10.3, 2048 of 2557 29.1 and longer ones stay as they are (straight from memory 13.4 and 31.7).
  if (v.threads < 1024 && mean * 4 <= v.max_len() && heads * v.threads > 256 * 1024) v.staged = false;
  return v;
}

template <int THREADS, int KPT, int R, bool PIECES, bool STAGED>
int launch_reg_kernel(dim3 grid, hipStream_t st, const TopkParams& p) {
  constexpr int kBytes = STAGED ? reg_variant_stage_bytes(THREADS, KPT) : 0;
  if (kBytes > 0) {
    const int rc = set_max_dynamic_lds(reinterpret_cast<const void*>(topk_reg_kernel<THREADS, KPT, R, PIECES, STAGED>), kBytes);
    if (rc != DAPQ_OK) return rc;
  }
  hipLaunchKernelGGL((topk_reg_kernel<THREADS, KPT, R, PIECES, STAGED>), grid, dim3(THREADS), kBytes, st, p);
  return DAPQ_OK;
}

template <int R>
int launch_reg(RegVariant v, bool pieces, dim3 grid, hipStream_t st, const TopkParams& p) {
  if (pieces) return launch_reg_kernel<1024, 32, R, true, true>(grid, st, p);
  if (v.kpt == 8) {
    if (v.threads == 256) return launch_reg_kernel<256, 8, R, false, true>(grid, st, p);
    if (v.threads == 512) return launch_reg_kernel<512, 8, R, false, true>(grid, st, p);
    return launch_reg_kernel<1024, 8, R, false, true>(grid, st, p);
  }
  if (v.threads == 256) return v.staged ? launch_reg_kernel<256, 32, R, false, true>(grid, st, p) : launch_reg_kernel<256, 32, R, false, false>(grid, st, p);
  if (v.threads == 512) return v.staged ? launch_reg_kernel<512, 32, R, false, true>(grid, st, p) : launch_reg_kernel<512, 32, R, false, false>(grid, st, p);
  if (v.kpt == 32) return launch_reg_kernel<1024, 32, R, false, true>(grid, st, p);
  return launch_reg_kernel<1024, 64, R, false, false>(grid, st, p);
}

int launch_reg_radius(int radius, RegVariant v, bool pieces, dim3 grid, hipStream_t st, const TopkParams& p) {
  switch (radius) {
    case 0: return launch_reg<0>(v, pieces, grid, st, p);
    case 1: return launch_reg<1>(v, pieces, grid, st, p);
    case 2: return launch_reg<2>(v, pieces, grid, st, p);
    case 3: return launch_reg<3>(v, pieces, grid, st, p);
    default: return launch_reg<4>(v, pieces, grid, st, p);
  }
}

template <int THREADS, int KPT>
int launch_merge_kernel(dim3 grid, hipStream_t st, const TopkParams& p) {
  constexpr int kBytes = merge_variant_bytes(THREADS, KPT);
  if (kBytes > 0) {
    const int rc = set_max_dynamic_lds(reinterpret_cast<const void*>(topk_merge_kernel<THREADS, KPT>), kBytes);
    if (rc != DAPQ_OK) return rc;
  }
  hipLaunchKernelGGL((topk_merge_kernel<THREADS, KPT>), grid, dim3(THREADS), kBytes, st, p);
  return DAPQ_OK;
}
int launch_merge(RegVariant v, dim3 grid, hipStream_t st, const TopkParams& p) {
  if (v.threads == 256) return launch_merge_kernel<256, 32>(grid, st, p);
  if (v.kpt == 16) return launch_merge_kernel<1024, 16>(grid, st, p);
  if (v.kpt == 32) return launch_merge_kernel<1024, 32>(grid, st, p);
  return launch_merge_kernel<1024, 64>(grid, st, p);
}

int topk_common_checks(const dapq_shape* shape, const float* in, int32_t budget, const int32_t* idx, const int32_t* count) {
  int rc = check_shape(shape, false, false, false);
  if (rc != DAPQ_OK) return rc;
  DAPQ_REQUIRE(in != nullptr && idx != nullptr && count != nullptr, DAPQ_ERR_INVALID_ARG,
               "scores, idx and count must not be NULL");
  DAPQ_REQUIRE(budget >= 1, DAPQ_ERR_INVALID_ARG, "budget (%d) must be >= 1", budget);
  DAPQ_REQUIRE(shape->batch <= 65535 && shape->n_layers <= 65535, DAPQ_ERR_UNSUPPORTED,
               "batch and n_layers must be <= 65535");
  return DAPQ_OK;
}

// Which kernels a batch goes to.  Heads that fit the chosen register variant go there; longer ones go in pieces of
// kTopkPieceLen keys through the variant for 32768 keys and a merge (if the caller brought the workspace for the
// candidate lists), else to the streaming kernel.  A dense batch knows its length; a ragged one launches both kinds,
// each skipping the heads of the other.
constexpr int kTopkPieceLen = 1024 * 32;
struct TopkRoute {
  RegVariant variant, kernel;  // what the short heads' kernel has to hold, and the kernel
  int64_t reg_max;     // heads up to this length: the register variant
  bool any_short, any_long;
  // the long heads in pieces
  bool pieces_possible;
  int n_segs;
  size_t off_key, off_idx, off_count, pieces_bytes;
};

// with_pieces: the caller brought the workspace, so heads of more than one piece's length (32768 keys) need not go
// to the variant with 64 keys per thread (slower per key than two pieces and a merge) or to the streaming kernel.
TopkRoute topk_route(const dapq_shape* shape, int32_t budget, bool with_pieces) {
  TopkRoute r;
  const bool ragged = shape->cu_seqlens != nullptr;
  const int64_t mean = shape->total_tokens / shape->batch;
  const int64_t longest = ragged ? shape->total_tokens : mean;
  // a ragged batch sizes the variant for 1.5 x its mean length (or everything, if that is less)
  int64_t sized_for = !ragged ? mean : (mean + mean / 2 < longest ? mean + mean / 2 : longest);
  if (with_pieces && sized_for > kTopkPieceLen) sized_for = kTopkPieceLen;
  r.variant = reg_variant_for(sized_for);
  r.reg_max = r.variant.max_len();
  const int64_t heads = (int64_t)shape->n_layers * shape->batch * shape->n_kv_heads;
  r.kernel = reg_kernel_for(r.variant, longest < r.reg_max ? longest : r.reg_max, mean, heads);
  r.any_short = ragged || mean <= r.reg_max;  // (a dense batch of longer heads has nothing for the register variant)
  r.any_long = longest > r.reg_max;
  const int64_t n_segs = (longest + kTopkPieceLen - 1) / kTopkPieceLen;
  r.pieces_possible = r.any_long && n_segs <= kTopkMaxSegs && n_segs * budget <= 65536 &&
                      (int64_t)shape->n_kv_heads * n_segs <= 0x7FFFFFFF;
  r.n_segs = (int)n_segs;
  r.off_key = r.off_idx = r.off_count = r.pieces_bytes = 0;
  if (r.pieces_possible) {
    const size_t list = align_up((size_t)heads * (size_t)n_segs * (size_t)budget * 4, 256);
    r.off_key = 0;
    r.off_idx = list;
    r.off_count = 2 * list;
    r.pieces_bytes = 2 * list + align_up((size_t)heads * (size_t)n_segs * 4, 256);
  }
  return r;
}

// The kernels for the long heads of a launch whose TopkParams are filled except for the long-head fields.
// radius > 0: the kernels of the pieces pool the scores themselves.
int launch_long_heads(const dapq_shape* shape, const TopkRoute& r, TopkParams p, int radius, void* workspace,
                      size_t workspace_bytes, hipStream_t st) {
  p.min_len = (int32_t)r.reg_max + 1;
  p.max_len = INT32_MAX;
  const dim3 grid((unsigned)shape->n_kv_heads, (unsigned)shape->batch, (unsigned)shape->n_layers);
  if (r.pieces_possible && workspace != nullptr && workspace_bytes >= r.pieces_bytes) {
    char* ws = static_cast<char*>(workspace);
    p.n_segs = r.n_segs;
    p.inv_segs = 1.0f / (float)r.n_segs;
    p.seg_len = kTopkPieceLen;
    p.cand_key = reinterpret_cast<uint32_t*>(ws + r.off_key);
    p.cand_idx = reinterpret_cast<int32_t*>(ws + r.off_idx);
    p.cand_count = reinterpret_cast<int32_t*>(ws + r.off_count);
    const dim3 piece_grid((unsigned)(shape->n_kv_heads * r.n_segs), (unsigned)shape->batch, (unsigned)shape->n_layers);
    int rc = launch_reg_radius(radius, RegVariant{1024, 32, true}, true, piece_grid, st, p);
    if (rc != DAPQ_OK) return rc;
    DAPQ_HIP_LAUNCH_CHECK("topk_reg_kernel (pieces)");
    // (one workgroup per long head: from 8193 candidate slots on, the large workgroup's sixteen waves)
    const int64_t slots = (int64_t)r.n_segs * p.budget;
    rc = launch_merge(slots <= 256 * 32    ? RegVariant{256, 32, true}
                      : slots <= 1024 * 16 ? RegVariant{1024, 16, true}
                      : slots <= 1024 * 32 ? RegVariant{1024, 32, true}
                                           : RegVariant{1024, 64, false},
                      grid, st, p);
    if (rc != DAPQ_OK) return rc;
    DAPQ_HIP_LAUNCH_CHECK("topk_merge_kernel");
    return DAPQ_OK;
  }
  DAPQ_REQUIRE(radius == 0, DAPQ_ERR_INVALID_ARG, "internal: the streaming kernel does not pool");
  // heads of up to kTopkLdsKeys keys are staged in LDS; if none of this launch can be that short the staging
  // area is left out
  const int lds_bytes = (kStreamLdsHead + (p.min_len <= kTopkLdsKeys ? kTopkLdsKeys : 0)) * (int)sizeof(uint32_t);
  // the limit is raised once, to the size with the staging area
  const int rc_lds = set_max_dynamic_lds(reinterpret_cast<const void*>(topk_stream_kernel),
                                         (kStreamLdsHead + kTopkLdsKeys) * (int)sizeof(uint32_t));
  if (rc_lds != DAPQ_OK) return rc_lds;
  hipLaunchKernelGGL(topk_stream_kernel, grid, dim3(kTopkThreads), lds_bytes, st, p);
  DAPQ_HIP_LAUNCH_CHECK("topk_stream_kernel");
  return DAPQ_OK;
}

TopkParams topk_params(const dapq_shape* shape, const float* in, float* pooled_out, int32_t budget,
                       const int32_t* budget_per_seq, int32_t* idx, int32_t* count) {
  TopkParams p;
  p.pooled = in;
  p.pooled_out = pooled_out;
  p.cu_seqlens = shape->cu_seqlens;
  p.budget_per_seq = budget_per_seq;
  p.idx = idx;
  p.count = count;
  p.total_tokens = shape->total_tokens;
  p.batch = shape->batch;
  p.n_kv_heads = shape->n_kv_heads;
  p.budget = budget;
  p.seq_len = (int32_t)(shape->total_tokens / shape->batch);
  p.inv_segs = 1.0f;
  p.inv_budget = 1.0f / (float)budget;
  p.min_len = 0;
  p.max_len = INT32_MAX;
  p.n_segs = 1;
  p.seg_len = 0;
  p.cand_key = nullptr;
  p.cand_idx = nullptr;
  p.cand_count = nullptr;
  return p;
}

}  // namespace
}  // namespace dapq

extern "C" DAPQ_API size_t dapq_topk_workspace_bytes(const dapq_shape* shape, int32_t budget) {
  if (check_shape(shape, false, false, false) != DAPQ_OK || budget < 1) return 0;
  return topk_route(shape, budget, true).pieces_bytes;
}

namespace dapq {
namespace {
// The route of a call: with the pieces if the caller's workspace holds their candidate lists.
TopkRoute topk_route_for(const dapq_shape* shape, int32_t budget, const void* workspace, size_t workspace_bytes) {
  const TopkRoute with = topk_route(shape, budget, true);
  if (with.pieces_possible && workspace != nullptr && workspace_bytes >= with.pieces_bytes) return with;
  return topk_route(shape, budget, false);
}
}  // namespace
}  // namespace dapq

extern "C" DAPQ_API int dapq_topk(const dapq_shape* shape, const float* pooled, int32_t budget, const int32_t* budget_per_seq,
                         int32_t* idx, int32_t* count, void* workspace, size_t workspace_bytes, void* stream) {
  int rc = topk_common_checks(shape, pooled, budget, idx, count);
  if (rc != DAPQ_OK) return rc;
  TopkParams p = topk_params(shape, pooled, nullptr, budget, budget_per_seq, idx, count);
  const TopkRoute route = topk_route_for(shape, budget, workspace, workspace_bytes);
  const dim3 grid((unsigned)shape->n_kv_heads, (unsigned)shape->batch, (unsigned)shape->n_layers);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (route.any_short) {
    p.max_len = (int32_t)route.reg_max;
    if ((rc = launch_reg<0>(route.kernel, false, grid, st, p)) != DAPQ_OK) return rc;
    DAPQ_HIP_LAUNCH_CHECK("topk_reg_kernel");
  }
  if (route.any_long) return launch_long_heads(shape, route, p, 0, workspace, workspace_bytes, st);
  return DAPQ_OK;
}

extern "C" DAPQ_API int dapq_pool_topk(const dapq_shape* shape, const float* scores, int32_t width, int32_t budget,
                                       const int32_t* budget_per_seq, int32_t* idx, int32_t* count, float* pooled,
                                       void* workspace, size_t workspace_bytes, void* stream) {
  int rc = topk_common_checks(shape, scores, budget, idx, count);
  if (rc != DAPQ_OK) return rc;
  DAPQ_REQUIRE(width >= 1 && width <= 63 && (width & 1) == 1, DAPQ_ERR_INVALID_ARG,
               "width (%d) must be odd and in [1, 63]", width);
  DAPQ_REQUIRE(pooled != scores, DAPQ_ERR_INVALID_ARG, "pooled must not alias scores");
  const int64_t longest = shape->cu_seqlens == nullptr ? shape->total_tokens / shape->batch : shape->total_tokens;
  const dim3 grid((unsigned)shape->n_kv_heads, (unsigned)shape->batch, (unsigned)shape->n_layers);
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t heads = (int64_t)shape->n_layers * shape->batch * shape->n_kv_heads;
  TopkParams p = topk_params(shape, scores, pooled, budget, budget_per_seq, idx, count);
  const TopkRoute route = topk_route_for(shape, budget, workspace, workspace_bytes);
  if (width <= 9 && route.any_long && route.pieces_possible && workspace != nullptr &&
      workspace_bytes >= route.pieces_bytes) {
    // heads of more than 32768 keys in pieces, whose kernels pool across the piece boundaries; the others in one
    // workgroup each
    if (route.any_short) {
      p.max_len = (int32_t)route.reg_max;
      if ((rc = launch_reg_radius(width / 2, route.kernel, false, grid, st, p)) != DAPQ_OK) return rc;
      DAPQ_HIP_LAUNCH_CHECK("topk_reg_kernel");
    }
    return launch_long_heads(shape, route, p, width / 2, workspace, workspace_bytes, st);
  }
  if (width <= 9 && longest <= 64 * kTopkThreads) {
    // one kernel: every head fits a register variant, which pools on the way in
    const RegVariant v = reg_kernel_for(reg_variant_for(longest), longest, shape->total_tokens / shape->batch, heads);
    if ((rc = launch_reg_radius(width / 2, v, false, grid, st, p)) != DAPQ_OK) return rc;
    DAPQ_HIP_LAUNCH_CHECK("topk_reg_kernel");
    return DAPQ_OK;
  }
  DAPQ_REQUIRE(pooled != nullptr, DAPQ_ERR_UNSUPPORTED,
               "width %d / head length %lld need the two-kernel path: pass a pooled buffer (or, for width <= 9, a "
               "workspace of dapq_topk_workspace_bytes())", width, (long long)longest);
  if ((rc = dapq_pool(shape, scores, pooled, width, stream)) != DAPQ_OK) return rc;
  return dapq_topk(shape, pooled, budget, budget_per_seq, idx, count, workspace, workspace_bytes, stream);
}
