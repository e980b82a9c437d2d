// Unit tasks of batches and the server: nests of one to three reducing segments as
// independent pieces of a wavefront's work (hp_units.hip; the partition is made by
// unit_route in hp_units.cpp).
#pragma once

#include <stdint.h>

#include "hp_internal.h"

namespace hp {

enum UnitOut : int32_t { UNIT_F64 = 0, UNIT_F32, UNIT_I64, UNIT_I32 };

// A nest as unit tasks.  The view is that of the segment kernels: out[o] = Q over q of M
// over m of L over the contiguous row (o, q, m); a single reduction has M and Q of one
// iteration.  Unit u is one of
//   a run of groups of 2^pair_bits (o, q) pairs side by side   (mparts = lparts = 1),
//   steps [per part, per (part + 1)) of pair u / mparts         (part = u % mparts),
//   elements [part_len part, ...) of row u / lparts             (part = u % lparts).
// With `partial` a unit leaves carriers of M (or, split rows, of L) in ws and a fold task
// per output ends the nest.
struct UnitDesc {
  const void* in;
  void* out;
  unsigned char* ws;
  int64_t pairs;
  int32_t eL, eM, eQ;
  int32_t opL, opM, opQ;
  int32_t vecs;       // vectors per lane of a row (0: rows shorter than a vector)
  int32_t lane_bits;  // 2^lane_bits lanes per row
  int32_t pair_bits;
  int32_t steps;      // steps of a pair
  int32_t run;        // groups per unit
  int32_t mparts, per;
  int32_t lparts, part_len;
  int32_t out_kind;   // UnitOut
  int32_t partial;
  int32_t direct;     // one segment: a row's value is an output
  int32_t fold_form;  // FoldForm
  int32_t fold_waves; // 1 or kFoldWaves
  int32_t pad[4];
};
static_assert(sizeof(UnitDesc) == 128, "one descriptor is one 128-byte line");

struct UnitRoute {
  int32_t on;        // 0: the nest runs as the plan's own tasks
  int32_t dtype;
  UnitDesc d;        // pointers unset
  int64_t units;
  int64_t folds;     // fold tasks, one per output
  uint64_t ws_bytes;
  double unit_bytes; // input bytes of the largest unit, for the order of the tasks
};

// Tasks of one launch: its threads stay below 2^32, the limit of a grid (a list of more
// goes out in several launches).
constexpr int64_t launch_tasks(int64_t threads_per_task) { return ((int64_t)1 << 31) / threads_per_task; }

// What is left of an output -- for eQ iterations of Q, `rows` groups of `parts` carriers
// (rows: the iterations of M where rows were cut) -- is folded by a wave or, where that
// would take long, by the kFoldWaves waves of a workgroup.  Each form takes so many rounds
// of memory latency, some 0.8 us each.
constexpr int kFoldWaves = 16;
enum FoldForm : int32_t {
  FOLD_LANE_Q = 0,  // a lane per iteration of Q
  FOLD_LANE_ROW,    // a wave per iteration of Q, a lane per row
  FOLD_WAVE         // a wave per iteration of Q, or per row without Q
};
struct FoldPlan {
  int32_t form;
  int64_t rounds;
};
inline FoldPlan fold_plan(bool hasQ, int64_t eQ, int64_t rows, int64_t parts, int64_t waves) {
  auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int64_t lanes = 64 * waves, some = up(parts, 4);  // four loads in flight
  const int64_t r = hasQ ? up(eQ, waves) * up(rows, 64) * some : up(rows, lanes) * some;
  const int64_t w = hasQ ? up(eQ, waves) * rows * up(parts, 256) : rows > 1 ? up(rows, waves) * up(parts, 256) : up(parts, 4 * lanes);
  if (hasQ) {
    const int64_t q = up(eQ, lanes) * rows * some;
    if (q <= r && q <= w) return FoldPlan{FOLD_LANE_Q, q};
  }
  return r < w ? FoldPlan{FOLD_LANE_ROW, r} : FoldPlan{FOLD_WAVE, w};
}

// The unit route of a batched nest whose plan is L.  tuned: L comes from the tuner cache,
// whose grid (units per output or outputs per unit) and lanes per output are kept.
UnitRoute unit_route(const hp_nest* nest, uint32_t flags, const Lowered& L, bool tuned);

}  // namespace hp
