// Host-side helpers shared by the libdapq translation units: error reporting, argument checks and
// the launch plan (chunking of the key axis, workspace carving).  No device code here.
#pragma once

#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>

#include "dapq.h"

namespace dapq {

// Thread-local message returned by dapq_last_error().
char* error_buffer();
int fail(int code, const char* fmt, ...);

#define DAPQ_REQUIRE(cond, code, ...)            \
  do {                                           \
    if (!(cond)) return ::dapq::fail((code), __VA_ARGS__); \
  } while (0)

#define DAPQ_HIP_LAUNCH_CHECK(what)                                                          \
  do {                                                                                       \
    hipError_t e__ = hipGetLastError();                                                      \
    if (e__ != hipSuccess) return ::dapq::fail(DAPQ_ERR_HIP, "%s: %s", (what), hipGetErrorString(e__)); \
  } while (0)

constexpr int kHeadDim = 128;
constexpr int kMinChunkKeys = 128;      // fewest keys one wave of a score pass walks over
constexpr int kMaxChunkKeys = 1 << 16;  // most
// Keys of a workgroup of the tile form of the score passes; the size of a call is counted in tiles of kTileKeys.
constexpr int kTileKeys = 128, kTileMinKeys = 32, kTileMaxKeys = 256;

// How the score passes split the work; a pure function of the shape and of the size of the workspace, so that
// dapq_workspace_bytes() and the launchers agree.
struct ScorePlan {
  bool stage_q;    // tile form: the queries go through LDS
  bool unit_sums;  // wave form, dense: pass 1 adds up a unit's terms first
  bool tile;       // the tile kernels (a workgroup per chunk, its waves share out the rows) instead of the wave kernels
  int rows;        // R = (H_q/H_kv) * N query rows scored against every key of a KV head
  int n_groups;    // row groups of row_blocks * 32 rows, one wave each per chunk (tile: 1)
  int row_blocks;  // 32-row blocks per wave (2 to 8; tile: all of them)
  int rows_pad;    // n_groups * row_blocks * 32
  int room_rows;   // rows that the workspace has partial sums for: at least rows_pad
  int chunk_keys;  // keys per wave, a multiple of 32 (tile form: keys of a tile, a power of two; in segments: those of a sub-block)
  int segments;    // ragged batches in the wave form: the waves that share a head's packed key axis (else 0)
  int64_t max_chunks;  // partial sums of a row: upper bound on sum_b ceil(L_b / chunk_keys), or batch + segments
  // workspace carving (byte offsets)
  size_t off_cu_chunks, off_parts, off_lse2, off_partial, total_bytes;
};

// Validates the fields every entry point relies on.  need_q / need_k / need_v say which stride
// groups must be usable.  Returns DAPQ_OK or sets the error and returns its code.
int check_shape(const dapq_shape* s, bool need_q, bool need_k, bool need_v);
// workspace_bytes: what the caller's workspace holds (SIZE_MAX to ask for what the shape would like).
int make_score_plan(const dapq_shape* s, size_t workspace_bytes, ScorePlan* plan);

// How the wave kernels split the rows: one wave holds a group of up to 256 in its registers, the groups of a head as many each.
// The workspace is sized as if a wave held 2, 4 or 8 row blocks, so that its figure does not fall where a row more makes a
// head two groups of fewer blocks.
struct RowSplit {
  int n_groups, row_blocks, room_blocks;
};
inline RowSplit wave_row_split(int rows) {
  const int blocks = (rows + 31) / 32, n_groups = (blocks + 7) / 8, each = (blocks + n_groups - 1) / n_groups;
  return {n_groups, each < 2 ? 2 : each, each <= 2 ? 2 : (each <= 4 ? 4 : 8)};
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Raises a kernel's dynamic-LDS limit to `bytes` (the most that kernel is ever launched with), once per kernel
// and device.  The value never changes afterwards, so launches from several host threads cannot meet a smaller
// limit than they need.
int set_max_dynamic_lds(const void* kernel, int bytes);

}  // namespace dapq
