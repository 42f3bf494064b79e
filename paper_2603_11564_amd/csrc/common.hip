// Error reporting, shape validation and the launch plan of libdapq (host code only).
#include <math.h>
#include <string.h>

#include <mutex>
#include <vector>

#include "dapq_internal.h"

namespace dapq {

char* error_buffer() {
  static thread_local char buf[512] = {0};
  return buf;
}

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(error_buffer(), 512, fmt, ap);
  va_end(ap);
  return code;
}

int set_max_dynamic_lds(const void* kernel, int bytes) {
  struct Entry { const void* kernel; int device; };
  static std::mutex mu;
  static std::vector<Entry> done;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(DAPQ_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
  std::lock_guard<std::mutex> lock(mu);
  for (const Entry& it : done)
    if (it.kernel == kernel && it.device == dev) return DAPQ_OK;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return fail(DAPQ_ERR_HIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
  done.push_back({kernel, dev});
  return DAPQ_OK;
}

static bool stride_ok(int64_t s) { return s >= 0 && (s % 8) == 0; }

int check_shape(const dapq_shape* s, bool need_q, bool need_k, bool need_v) {
  DAPQ_REQUIRE(s != nullptr, DAPQ_ERR_INVALID_ARG, "shape is NULL");
  DAPQ_REQUIRE(s->n_layers >= 1 && s->batch >= 1, DAPQ_ERR_INVALID_ARG,
               "n_layers (%d) and batch (%d) must be >= 1", s->n_layers, s->batch);
  DAPQ_REQUIRE(s->n_kv_heads >= 1 && s->n_q_heads >= 1 && s->n_q_heads % s->n_kv_heads == 0,
               DAPQ_ERR_INVALID_ARG, "n_q_heads (%d) must be a positive multiple of n_kv_heads (%d)",
               s->n_q_heads, s->n_kv_heads);
  DAPQ_REQUIRE(s->n_pseudo >= 1, DAPQ_ERR_INVALID_ARG, "n_pseudo (%d) must be >= 1", s->n_pseudo);
  DAPQ_REQUIRE(s->total_tokens >= 0, DAPQ_ERR_INVALID_ARG, "total_tokens is negative");
  DAPQ_REQUIRE(s->head_dim == kHeadDim, DAPQ_ERR_UNSUPPORTED, "head_dim %d is not supported (128 only)",
               s->head_dim);
  DAPQ_REQUIRE(s->total_tokens < (int64_t)1 << 31, DAPQ_ERR_UNSUPPORTED,
               "total_tokens %lld does not fit the int32 token offsets", (long long)s->total_tokens);
  DAPQ_REQUIRE((int64_t)s->n_layers * s->n_kv_heads <= 65535, DAPQ_ERR_UNSUPPORTED,
               "n_layers * n_kv_heads (%lld) exceeds the grid limit 65535",
               (long long)s->n_layers * s->n_kv_heads);
  if (s->cu_seqlens == nullptr) {
    DAPQ_REQUIRE(s->total_tokens % s->batch == 0, DAPQ_ERR_INVALID_ARG,
                 "dense batch: total_tokens (%lld) is not a multiple of batch (%d)",
                 (long long)s->total_tokens, s->batch);
  }
  if (need_q) {
    DAPQ_REQUIRE(stride_ok(s->q_stride_layer) && stride_ok(s->q_stride_seq) && stride_ok(s->q_stride_head) &&
                     stride_ok(s->q_stride_row) && s->q_stride_row >= kHeadDim,
                 DAPQ_ERR_UNSUPPORTED, "q strides must be non-negative multiples of 8 elements (row >= 128)");
    DAPQ_REQUIRE(isfinite(s->scale) && s->scale > 0.0f, DAPQ_ERR_INVALID_ARG, "scale must be finite and > 0");
  }
  if (need_k) {
    DAPQ_REQUIRE(stride_ok(s->k_stride_layer) && stride_ok(s->k_stride_seq) && stride_ok(s->k_stride_head) &&
                     stride_ok(s->k_stride_token) && s->k_stride_token >= kHeadDim,
                 DAPQ_ERR_UNSUPPORTED, "k strides must be non-negative multiples of 8 elements (token >= 128)");
    DAPQ_REQUIRE(s->k_stride_token < ((int64_t)1 << 26), DAPQ_ERR_UNSUPPORTED,
                 "k_stride_token (%lld) must be below 2^26 elements", (long long)s->k_stride_token);
  }
  if (need_v) {
    DAPQ_REQUIRE(stride_ok(s->v_stride_layer) && stride_ok(s->v_stride_seq) && stride_ok(s->v_stride_head) &&
                     stride_ok(s->v_stride_token) && s->v_stride_token >= kHeadDim,
                 DAPQ_ERR_UNSUPPORTED, "v strides must be non-negative multiples of 8 elements (token >= 128)");
  }
  return DAPQ_OK;
}

// Lays out the workspace of a plan whose rows are split and whose partial sums are counted.
static void carve_workspace(const dapq_shape* s, int64_t heads, ScorePlan* p) {
  size_t off = 0;
  p->off_cu_chunks = off;
  off = align_up(off + sizeof(int32_t) * ((size_t)s->batch + 1), 256);
  off += 256;  // (nothing lies here: workspaces have always had it)
  p->off_parts = off;
  off = align_up(off + sizeof(float) * (p->tile ? 1 : 2) * (size_t)heads * (size_t)p->max_chunks * p->room_rows, 256);
  p->off_lse2 = off;
  off = align_up(off + sizeof(float) * (size_t)s->n_layers * s->batch * s->n_q_heads * s->n_pseudo, 256);
  p->off_partial = off;
  if (p->n_groups > 1) off = align_up(off + sizeof(float) * (size_t)(p->n_groups - 1) * (size_t)heads * (size_t)s->total_tokens, 256);
  p->total_bytes = off;
}
// How many partial sums of a row a workspace of `room` bytes holds in the wave form (negative: it does not even hold the rest).
static int64_t partials_that_fit(const dapq_shape* s, int64_t heads, ScorePlan p, size_t room) {
  p.max_chunks = 0;
  carve_workspace(s, heads, &p);
  if (room < p.total_bytes) return -1;
  // (a row block's partials are whole multiples of 256 bytes)
  const uint64_t most = (room - p.total_bytes) / (sizeof(float) * 2 * (size_t)heads * p.room_rows);
  return most < ((uint64_t)1 << 31) ? (int64_t)most : ((int64_t)1 << 31);
}

// The plan's chunks along the key axis and its workspace, once the rows are split and the chunk is chosen.
static int finish_score_plan(const dapq_shape* s, int64_t heads, int chunk, ScorePlan* p) {
  p->chunk_keys = chunk;
  if (p->segments > 0) {
    p->max_chunks = (int64_t)s->batch + p->segments;
  } else if (s->cu_seqlens == nullptr) {
    const int64_t L = s->total_tokens / s->batch;
    p->max_chunks = (int64_t)s->batch * ((L + chunk - 1) / chunk);
  } else {
    p->max_chunks = (s->total_tokens + chunk - 1) / chunk + s->batch;
  }
  if (p->max_chunks < 1) p->max_chunks = 1;
  DAPQ_REQUIRE(p->max_chunks < ((int64_t)1 << 31), DAPQ_ERR_UNSUPPORTED, "too many key chunks");
  DAPQ_REQUIRE(p->n_groups <= 65535, DAPQ_ERR_UNSUPPORTED, "too many query rows per KV head");
  carve_workspace(s, heads, p);
  return DAPQ_OK;
}

// The power of two with the shortest rounds x (chunk + a start-up of 160 keys), which bounds what a chunk may do to accuracy and
// workspace (see make_score_plan).
static int dense_chunk_of_two(const dapq_shape* s, int64_t heads, const ScorePlan& p, int64_t wave_slots) {
  const int64_t L = s->total_tokens / s->batch;
  int64_t best = INT64_MAX;
  int chunk = kMinChunkKeys;
  for (int c = kMaxChunkKeys; c >= kMinChunkKeys; c /= 2) {
    const int64_t units = heads * p.n_groups * s->batch * ((L + c - 1) / c);
    const int64_t cost = (units + wave_slots - 1) / wave_slots * ((L < c ? L : c) + 160);
    if (cost < best) {
      best = cost;
      chunk = c;
    }
  }
  return chunk;
}

// Time of both passes of a dense batch in chunks of c keys, in nanoseconds, as far as c decides it.  The machine runs wave_slots waves
// at a time, each for as long as its chunk, and a round of waves pays a start-up (queries, ring fill).  Up to four chunks of a
// sequence with one row group are the waves of one workgroup, which does both passes (dapq_score in one kernel): one start-up for both and
// no merge between them, but a compute unit holds four such waves only if their number divides four.  Otherwise there are three
// launches, the merge reads a row of partials per chunk, and with few rows workgroups of two waves, which an even number of chunks makes
// that four does not divide, are placed badly (64 rows, 32 chunk streams: 20 chunks 48 us, 22 chunks 57, 23 chunks 48).
// The constants lose least over 732 dense shapes (1 to 32 layers, 1 to 16 prompts of 130 to 131072 keys, 16 to 1024 rows), each timed in
// some 20 chunk lengths: against the best power of two 0.906 of the time in the geometric mean, none above 1.09 (with a start-up of
// 160 keys for both forms, and one to four chunks only where they fill the rounds: 0.940 and 1.85; the best of the lengths: 0.896).
// (Start-ups of 7000 and 11000, as they are since the queries come through the ring, and costs of five to seven row blocks of their own are
// worth a quarter of a hundredth of the time, 70 dense shapes, and took shapes from dapq_score_static that it has served.)
static int64_t dense_cost(const ScorePlan& p, int64_t streams, int64_t batch, int64_t L, int64_t c, int64_t wave_slots) {
  const int blocks = p.room_rows / (32 * p.n_groups);
  const int64_t n = (L + c - 1) / c, walk = (L < c ? L : c) * (blocks == 8 ? 75 : (blocks == 4 ? 52 : 45));
  if (p.n_groups == 1 && n <= 4) {
    const int64_t workgroups = wave_slots / 4 * (n <= 1 ? 4 : 4 / n);
    return (streams + workgroups - 1) / workgroups * (walk + 10000);
  }
  const bool pairs = p.row_blocks <= 4 && batch * n % 4 == 2;
  return (streams * n + wave_slots - 1) / wave_slots * (walk + 15000) + 7500 + 120 * n + (pairs ? 6000 : 0);
}

struct DenseChunk {
  int keys;      // 0: none
  int64_t cost;  // see dense_cost
};
// Keys per wave of a dense batch, with at most `most` chunks per sequence (at least what the longest chunks make): the best power of
// two (`two`), unless another number of equal chunks of whole sub-blocks is better by a hundredth: as many as fill 1, 2, ... 16
// rounds of waves, or one to four.
// A lane of pass 1 adds up its half of a chunk one by one, and what that costs in accuracy grows with the chunk (2^14 keys: 1.7e-5 of a
// score): chunks longer than the power of two form their sums in two steps, which is as fast and more accurate.  (Not so the others,
// whose results stay what they were; and powers of two above 2^13 are not exceeded, since two results that are both right would be that
// far apart.)
// Best power of two -> this, us: 32 layers, 256 rows, 19748 keys 784 -> 613; 16 layers, 512 rows, 2 prompts of 2556 keys 238 -> 182; 8
// layers, 128 rows, 5 prompts of 2316 keys 122 -> 73.
static DenseChunk dense_chunk(const dapq_shape* s, int64_t heads, const ScorePlan& p, int64_t wave_slots, int two, int64_t most) {
  const int64_t L = s->total_tokens / s->batch, streams = heads * p.n_groups * s->batch;
  DenseChunk best = {0, INT64_MAX};
  if (most < 1) return best;
  int64_t bar = INT64_MAX;  // what a chunk that is not the power of two has to stay below
  const bool two_fits = (L + two - 1) / two <= most;
  if (two_fits) {
    best = {two, dense_cost(p, streams, s->batch, L, two, wave_slots)};
    bar = best.cost - best.cost / 100;
  }
  auto consider = [&](int64_t n) {
    n = n < most ? n : most;
    int64_t c = ((L + n - 1) / n + 31) / 32 * 32;
    c = c < kMinChunkKeys ? kMinChunkKeys : (c > kMaxChunkKeys ? kMaxChunkKeys : c);
    if ((L + c - 1) / c > most || (c > two && two > 8192 && two_fits)) return false;
    const int64_t cost = dense_cost(p, streams, s->batch, L, c, wave_slots);
    if (cost < bar) {
      best = {(int)c, cost};
      bar = cost;
    }
    return c == kMinChunkKeys || n == most;  // more would not be more
  };
  for (int64_t n = 1; n <= (p.n_groups == 1 ? 4 : 1); ++n) consider(n);
  for (int64_t r = 1; r <= 16; ++r)
    if (r * wave_slots >= streams && consider(r * wave_slots / streams)) break;
  return best;
}

// Segments per head of a ragged batch, `streams` heads x row groups: the waves run in whole rounds of wave_slots, each as long as
// its share of the key axis, whatever the lengths of the sequences.  Of the numbers that fill 1, 2, ... 16 rounds the one with the
// least to do: a round's start-up (ring, queries) costs about what a two-hundredth of a head's keys do.  (At most 2^26 keys to a
// segment, for the offsets in it.)  It does not fall with the tokens, so that fewer of them never need a larger workspace.
// `most`: no more of them (1 if not even one round of waves is that few).
static int ragged_segments(int64_t streams, int64_t wave_slots, int64_t total_tokens, int64_t most) {
  int64_t best = 1;
  double least = INFINITY;
  for (int64_t rounds = 1; rounds <= 16; ++rounds) {
    const int64_t n = rounds * wave_slots / streams;
    if (n < 1 || n > most) continue;
    const double cost = (double)rounds * (1.0 / (double)n + 0.005);
    if (cost < least) {
      least = cost;
      best = n;
    }
  }
  const int64_t fewest = (total_tokens >> 26) + 1;
  return (int)(best > fewest ? best : fewest);
}

// Whether a ragged shape in chunks of a power of two keys, the one with the least work per wave slot and half a chunk of tail, fits the
// array of dapq_score_static: those shapes it has always served.
static bool ragged_chunks_fit_static(const dapq_shape* s, int64_t heads, const ScorePlan& p, int64_t wave_slots) {
  const int64_t streams = heads * p.n_groups, mean = s->total_tokens / s->batch;
  int64_t best = INT64_MAX;
  int chunk = kMinChunkKeys;
  for (int c = kMaxChunkKeys; c >= kMinChunkKeys; c /= 2) {
    const int64_t units = streams * ((s->total_tokens + c - 1) / c + s->batch / 2);
    const int64_t cost = (streams * s->total_tokens + units * 256) / wave_slots + (c <= mean ? c / 2 : mean / 2 + (c - mean) / 4);
    if (cost < best) {
      best = cost;
      chunk = c;
    }
  }
  ScorePlan t = p;
  t.segments = 0;
  return finish_score_plan(s, heads, chunk, &t) == DAPQ_OK && t.total_bytes <= DAPQ_STATIC_SCRATCH_BYTES;
}

// The workspace that a shape asks for serves every shape that is no larger in layers, heads, rows, sequences and (dense) keys of a
// sequence or (ragged) keys: plans do not fall and rise with the shape, a smaller one may want more partial sums, and it then makes do
// with fewer chunks or segments.  For that no shape asks for less than kRoomWaves waves' partials (or what it has at all: of all its
// chunks of the fewest keys; a wave each), and none is refused that many: half the machine's waves, which every plan of several
// launches fills anyway.
constexpr int64_t kRoomWaves = 512;

// Fewest chunks of a sequence, of those that a shape makes do with.
static int64_t dense_fewest(int64_t L, int64_t streams) {
  const int64_t all = (L + kMinChunkKeys - 1) / kMinChunkKeys, longest = (L + kMaxChunkKeys - 1) / kMaxChunkKeys;
  const int64_t some = all < kRoomWaves / streams ? all : kRoomWaves / streams;
  return some > longest ? some : (longest > 1 ? longest : 1);
}
// What a dense shape asks for at least.
static size_t dense_least_bytes(const dapq_shape* s, int64_t heads, ScorePlan p) {
  const int64_t L = s->total_tokens / s->batch, streams = heads * p.n_groups * s->batch;
  const int64_t all = streams * ((L + kMinChunkKeys - 1) / kMinChunkKeys);
  const int64_t waves = all < kRoomWaves ? all : kRoomWaves;
  p.max_chunks = 0;
  carve_workspace(s, heads, &p);
  return p.total_bytes + sizeof(float) * 2 * (size_t)waves * (p.room_rows / p.n_groups);
}
// Fewer and longer chunks, in a workspace of `room` bytes that does not hold the plan's.
static void fit_dense(const dapq_shape* s, int64_t heads, int64_t wave_slots, int two, size_t room, ScorePlan* p) {
  const int64_t L = s->total_tokens / s->batch, streams = heads * p->n_groups * s->batch;
  const int64_t most = partials_that_fit(s, heads, *p, room) / s->batch;
  if (most < dense_fewest(L, streams)) return;
  const int chunk = dense_chunk(s, heads, *p, wave_slots, two, most).keys;
  ScorePlan t = *p;
  t.unit_sums = chunk > two;
  if (finish_score_plan(s, heads, chunk, &t) == DAPQ_OK && t.total_bytes <= room) *p = t;
}

// Fewer segments, in a workspace of `room` bytes that does not hold the plan's.  (Where all shapes that fit the array of
// dapq_score_static ask for it whole, their plans may be of fewer waves than kRoomWaves.)
static bool fit_ragged(const dapq_shape* s, int64_t heads, int64_t wave_slots, size_t room, ScorePlan* p) {
  const int64_t streams = heads * p->n_groups, chunks = (s->total_tokens + kMinChunkKeys - 1) / kMinChunkKeys;
  const int64_t most = partials_that_fit(s, heads, *p, room) - s->batch;
  int64_t fewest = (s->total_tokens >> 26) + 1;
  if (room < DAPQ_STATIC_SCRATCH_BYTES) {
    const int64_t some = chunks < kRoomWaves / streams ? chunks : kRoomWaves / streams;
    fewest = some > fewest ? some : fewest;
  }
  if (most < fewest) return false;
  ScorePlan t = *p;
  t.segments = ragged_segments(streams, wave_slots, s->total_tokens, most);
  // (not even one round of waves: as many as there is room for)
  if (wave_slots / streams > most && t.segments < most) t.segments = (int)most;
  if (finish_score_plan(s, heads, 32, &t) != DAPQ_OK || t.total_bytes > room) return false;
  *p = t;
  return true;
}

int make_score_plan(const dapq_shape* s, size_t workspace_bytes, ScorePlan* p) {
  const int g = s->n_q_heads / s->n_kv_heads;
  const int64_t rows64 = (int64_t)g * s->n_pseudo;
  DAPQ_REQUIRE(rows64 <= (1 << 20), DAPQ_ERR_UNSUPPORTED, "group * n_pseudo = %lld rows per KV head is too large",
               (long long)rows64);
  p->rows = (int)rows64;
  const int64_t heads = (int64_t)s->n_layers * s->n_kv_heads;
  // one wave per (chunk, row group): a group is up to 256 rows, all in the wave's registers
  const RowSplit split = wave_row_split(p->rows);
  p->n_groups = split.n_groups;
  p->row_blocks = split.row_blocks;
  p->rows_pad = p->n_groups * p->row_blocks * 32;
  p->room_rows = p->n_groups * split.room_blocks * 32;
  p->tile = false;
  p->stage_q = false;
  p->unit_sums = false;
  p->segments = 0;

  constexpr int64_t kWaveSlots = 1024;
  int rc;
  if (s->cu_seqlens == nullptr) {
    const int two = dense_chunk_of_two(s, heads, *p, kWaveSlots);
    const DenseChunk best = dense_chunk(s, heads, *p, kWaveSlots, two, INT64_MAX);
    p->unit_sums = best.keys > two;
    rc = finish_score_plan(s, heads, best.keys, p);
    if (rc == DAPQ_OK && p->total_bytes > DAPQ_STATIC_SCRATCH_BYTES) {
      // a shape that dapq_score_static serves with the power of two, with hardly more time than the best takes, or in one kernel (which
      // leaves the workspace alone) with a sixteenth more, is served, by the same kernels as dapq_score's: a line of room, not of time
      const int64_t most = partials_that_fit(s, heads, *p, DAPQ_STATIC_SCRATCH_BYTES) / s->batch, L = s->total_tokens / s->batch;
      const DenseChunk fits = dense_chunk(s, heads, *p, kWaveSlots, two, most);
      const bool one_kernel = p->n_groups == 1 && fits.keys != 0 && (L + fits.keys - 1) / fits.keys <= 4;
      if (fits.keys != 0 &&
          ((L + two - 1) / two <= most || fits.cost <= best.cost + best.cost / (one_kernel ? 16 : 100))) {
        p->unit_sums = fits.keys > two;
        rc = finish_score_plan(s, heads, fits.keys, p);
      }
    }
    if (rc == DAPQ_OK) {
      const size_t least = dense_least_bytes(s, heads, *p);
      if (p->total_bytes < least) p->total_bytes = least;
      if (p->total_bytes > workspace_bytes) fit_dense(s, heads, kWaveSlots, two, workspace_bytes, p);
    }
  } else {
    p->segments = ragged_segments(heads * p->n_groups, kWaveSlots, s->total_tokens, INT64_MAX);
    rc = finish_score_plan(s, heads, 32, p);
    // A line of room, not of time: a shape that dapq_score_static has always served is still served, by the same kernels as
    // dapq_score's.  All such plans ask for the whole array: fewer tokens then never need a larger workspace.
    if (rc == DAPQ_OK && p->total_bytes > DAPQ_STATIC_SCRATCH_BYTES && ragged_chunks_fit_static(s, heads, *p, kWaveSlots) &&
        fit_ragged(s, heads, kWaveSlots, DAPQ_STATIC_SCRATCH_BYTES, p))
      p->total_bytes = DAPQ_STATIC_SCRATCH_BYTES;
    if (rc == DAPQ_OK && p->total_bytes > workspace_bytes) fit_ragged(s, heads, kWaveSlots, workspace_bytes, p);
  }
  if (rc != DAPQ_OK) return rc;

  // The tile form.  It is the faster one where the wave form leaves the chip idle or pays its start-up per chunk (the queries of up
  // to 256 rows into one wave, a ring of its own).  Both passes of dapq_score, wave form -> tiles of 128 keys with the queries
  // straight from memory, 8 KV heads: one layer, 1024 keys, 256 rows 38.6 -> 14.9 us; 8191 keys, 128 rows 26.9 -> 18.6; 16384 keys,
  // 256 rows 44 -> 41, 512 rows 57 -> 61; 32768 keys, 128 rows 39 -> 45; ragged, 8 prompts of 1000 keys, one layer, 128 rows 76 ->
  // 24, 4 layers, 128 rows (10 000 units) 146 -> 59, 512 rows (40 000 units) 188 -> 174.  Where a sequence is at most four chunks of the
  // fewest keys, dapq_score runs both passes in one kernel and stays with that one.
  // Calls of at most 256 workgroups, a compute unit each, take tiles as small as that allows (ragged ones up to 128 keys: larger
  // tiles would need less workspace than a longer batch), with the queries through LDS in whole rows; larger calls live from several
  // workgroups to a compute unit, which the queries' LDS would keep out (128 rows, 16384 keys: 32 us with it, 27 without).
  // With the rotation, tiles of 128 keys -> these: 1024 keys, 256 rows 17.7 -> 13.4 us; 4096 keys 19.1 -> 17.1; 8191 keys, 128 rows
  // 21.9 -> 17.7 (no separate merge of the normalisers at 32 tiles); 5000 keys, 16 rows 17.9 -> 12.8.
  const bool ragged = s->cu_seqlens != nullptr;
  const bool one_kernel = !ragged && p->n_groups == 1 && s->total_tokens / s->batch <= 4 * kMinChunkKeys;
  const int64_t row_blocks = (p->rows + 31) / 32;
  const int64_t tiles = heads * (ragged ? s->total_tokens / kTileKeys + s->batch
                                        : s->batch * ((s->total_tokens / s->batch + kTileKeys - 1) / kTileKeys));
  if (one_kernel || tiles * row_blocks > (ragged ? 65536 : 8192) || (!ragged && tiles > 1024)) return DAPQ_OK;
  ScorePlan t = *p;
  t.tile = true;
  t.segments = 0;
  t.row_blocks = (int)row_blocks;
  t.n_groups = 1;
  t.rows_pad = t.room_rows = t.row_blocks * 32;
  int keys = kTileKeys;
  t.stage_q = false;
  for (int c = kTileMinKeys; c <= (ragged ? kTileKeys : kTileMaxKeys); c *= 2) {
    const int64_t L = s->total_tokens / s->batch;
    if (heads * (ragged ? s->total_tokens / c + s->batch : s->batch * ((L + c - 1) / c)) <= 256) {
      keys = c;
      t.stage_q = true;
      break;
    }
  }
  rc = finish_score_plan(s, heads, keys, &t);
  if (rc != DAPQ_OK) return rc;
  // The figure is no smaller than the wave form's: smaller shapes may run in that (see kRoomWaves).
  if (t.total_bytes < p->total_bytes) t.total_bytes = p->total_bytes;
  // The partials of the tile form can take more room than the wave form does (the shapes above: 4.0 MB at 29 696 tokens).  A workspace
  // that holds only the wave form gets the wave form.  And a shape that dapq_score_static serves is still served, by the same kernels
  // as dapq_score's: tiles of more than its scratch array (128 bytes per unit: about 32 000 units) are not taken where the wave form
  // fits it.  That line is one of room, not of time.
  if (t.total_bytes > DAPQ_STATIC_SCRATCH_BYTES && p->total_bytes <= DAPQ_STATIC_SCRATCH_BYTES) return DAPQ_OK;
  if (t.total_bytes <= workspace_bytes) *p = t;
  return DAPQ_OK;
}

}  // namespace dapq

extern "C" DAPQ_API size_t dapq_workspace_bytes(const dapq_shape* shape) {
  if (dapq::check_shape(shape, false, false, false) != DAPQ_OK) return 0;
  dapq::ScorePlan plan;
  if (dapq::make_score_plan(shape, SIZE_MAX, &plan) != DAPQ_OK) return 0;
  return plan.total_bytes;
}

extern "C" DAPQ_API const char* dapq_last_error(void) { return dapq::error_buffer(); }
