// How a projection of pseudo queries is cut into waves (host code only; qproj.hip has the kernels).
#ifndef DAPQ_QPROJ_PLAN_H
#define DAPQ_QPROJ_PLAN_H

#include <stddef.h>
#include <stdint.h>

#include "dapq.h"

namespace dapq {

constexpr int kBlockK = 64;           // hidden channels per block: 128-byte rows in LDS
constexpr int64_t kQprojUnits = 256;  // compute units

// The numbers of planes of partial sums that a call may have: qproj_reduce_rope_kernel is built for each of them.  (There is room for sixteen
// single waves' planes, but where so many are possible fewer workgroups of four cost less.)
#define DAPQ_QPROJ_PLANES(each) each(1) each(2) each(3) each(4) each(5) each(6) each(7) each(8)
constexpr bool qproj_planes_have_a_kernel(int planes) {
#define DAPQ_ONE_OF(n) planes == n ||
  return DAPQ_QPROJ_PLANES(DAPQ_ONE_OF) false;
#undef DAPQ_ONE_OF
}

// How a call is cut into waves; a pure function of the description so that the workspace query and the
// launcher agree.
struct QprojPlan {
  int ft, mb, waves, tiles_f, sweeps, k_splits, kb_per_split;  // waves of a workgroup, workgroups along the hidden axis, blocks to a wave
  size_t workspace_bytes;
};

inline QprojPlan make_qproj_plan(const dapq_qproj& s) {
  QprojPlan pl;
  const int64_t features = (int64_t)s.n_q_heads * s.head_dim;
  // two row blocks per wave unless 32 rows are all there is
  pl.mb = s.rows > 32 ? 2 : 1;
  pl.sweeps = (int)(((int64_t)s.rows + 32 * pl.mb - 1) / (32 * pl.mb));
  // four feature tiles per wave while that still fills the chip (1024 SIMDs), two otherwise
  const int64_t waves4 = (features + 127) / 128 * pl.sweeps * s.n_layers;
  pl.ft = waves4 >= 768 ? 4 : 2;
  pl.tiles_f = (int)((features + 32 * pl.ft - 1) / (32 * pl.ft));
  // still too few waves: several waves per tile, each with a share of the hidden blocks (at least 8 per wave,
  // so that the ring's start-up is paid a few times at most), and one pass that adds their sums
  const int n_kb = s.hidden / kBlockK;
  const int64_t waves = (int64_t)pl.tiles_f * pl.sweeps * s.n_layers;
  pl.k_splits = 1;
  while (pl.k_splits < 16 && waves * pl.k_splits < 768 && n_kb / (pl.k_splits * 2) >= 8) pl.k_splits *= 2;
  pl.kb_per_split = (n_kb + pl.k_splits - 1) / pl.k_splits;
  pl.workspace_bytes = pl.k_splits == 1 ? 0
                                        : (size_t)pl.k_splits * s.n_layers * ((size_t)pl.sweeps * 32 * pl.mb) *
                                              ((size_t)pl.tiles_f * 32 * pl.ft) * sizeof(float);
  pl.waves = 1;
  // (Several sweeps of more than one round: bound by what the compute units take in of the rows, and a round's start-up is in the open.  2
  // layers, single waves -> four: 5120 wide, 128 rows 37.4 -> 44.9; 4096 wide, 148 rows 28.7 -> 33.0.)
  if (pl.k_splits == 1 || (pl.sweeps > 1 && waves > kQprojUnits)) return pl;
  // Four waves to a workgroup, which has a compute unit to itself, add up before they write: half the planes or fewer, and more of
  // the weight in flight.  Whatever costs least, in tenths of the time that one of four waves takes for a block: workgroups of four, as many
  // along the hidden axis as there is room for planes, but not more than eight, or single waves, of which a compute unit holds four or
  // five (their rings) and which take a block the faster the fewer they are.  The constants lose least over 826 calls (1 to 8 layers, 16 to
  // 256 rows, 1024 to 16384 wide, 8 to 64 heads of 128), each timed as single waves and as one to eight workgroups of four, weights out of
  // memory: against the single waves 0.942 of the time in the geometric mean and 36 calls above 1.025, none above 1.12 (with 40 for a block of
  // three single waves too, and a tenth on top of them for their planes: 0.949, 86 calls, up to 1.245; the best of all ways 0.923).  Calls,
  // us, single waves -> four: one layer 4096 wide, 256 rows 24.0 -> 20.9; 2 layers of 64 rows 22.8 -> 18.0; 8 layers 83.0 -> 66.8, of 16
  // rows 73.5 -> 55.7; 5120 wide, 64 rows 18.5 -> 16.5.  Single waves stay where three to each unit are a whole round: 3 layers of 8 heads, 5120
  // wide, 256 rows 23.9, four 29.6; 2 layers 6144 wide, 64 rows 38.8, four 44.8.
  const int per_unit = pl.mb == 2 ? 4 : 5;
  const int64_t tiles = waves, singles = tiles * pl.k_splits, units = kQprojUnits;
  const int64_t rounds = (singles + units * per_unit - 1) / (units * per_unit), shared = rounds > 1 ? per_unit : (singles + units - 1) / units;
  constexpr int kPlane = 6;
  int64_t best = kPlane * pl.k_splits;
  if (shared <= 3) best += 33 * pl.kb_per_split + 150;
  else if (shared == 4) best += rounds * (45 * pl.kb_per_split + 60);
  else best += rounds * (55 * pl.kb_per_split + 130);
  // (rows that a last sweep is short of are not fetched, which the workgroups of four gain by: one layer 4096 wide, 192 rows 23.7 us, 148 rows
  // 21.3 out of memory and 18.3 with the weights in the caches; single waves 22.1, 21.7 and 19.4)
  auto blocks_of_four = [&](int64_t each) {
    const int64_t rows = (int64_t)pl.sweeps * 32 * pl.mb;
    return 40 * each - (pl.sweeps > 1 ? 15 * each * (rows - s.rows) / rows : 0);
  };
  const int most = pl.k_splits < 8 ? pl.k_splits : 8;
  for (int splits = 1; splits <= most; ++splits) {
    const int each = (n_kb + 4 * splits - 1) / (4 * splits);
    if ((int64_t)(splits - 1) * 4 * each >= n_kb) continue;  // (a workgroup without blocks)
    const int64_t cost = (tiles * splits + units - 1) / units * (blocks_of_four(each) + (pl.mb == 2 ? 110 : 80)) + kPlane * splits;
    if (cost < best) {
      best = cost;
      pl.waves = 4;
      pl.k_splits = splits;
      pl.kb_per_split = each;
    }
  }
  return pl;
}

}  // namespace dapq

#endif  // DAPQ_QPROJ_PLAN_H
