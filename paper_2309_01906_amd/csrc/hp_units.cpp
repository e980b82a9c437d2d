// Partition of batched nests into unit tasks (host only).
#include <cstring>

#include "hp_units.h"

namespace hp {

static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline int log2u(uint64_t x) {
  int r = 0;
  while ((1ull << r) < x) ++r;
  return r;
}

// The cost of one unit, in vectors per lane (1 KiB of input each).  A wave pays some 2 us
// for its task and its descriptor before its first data, so smaller units cost more than
// the finer tail gains, and larger ones leave a few waves behind in small batches (10,000
// bf16 nests / 300 mixed ones: cost 8 111 / 51 us, 16 89 / 39, 24 82.5 / 38, 40 84 / 46).
// The end of a step of rows costs as much as a few vectors (its butterfly, and the
// carrier of M): short rows make smaller units.
static constexpr int64_t kUnitCost = 24;

// Rounds of a fold (fold_plan) from which the waves of a workgroup share an output (a
// multiple where outputs fill the chip), and up to which that is worth it: a nest of more
// stays with its plan's tasks, which split the outermost level over the chip; plan tasks that
// read single elements are slower yet.  A batch of one nest (rounds of a workgroup): 1 x
// 16384 x 8 x 64 SUM, MAX, ARGMIN (16) 180 us by one wave, 36 by sixteen, 67 as plan tasks; 4
// x 64 x 16 x 1024 (4) 81, 15 and 51; 4 x 65536 x 4 x 16 (64) 90 by sixteen, 66 as plan
// tasks; 1 x 65536 x 23 x 2 (64) 651, 75 and 926; 1 x 524288 x 4 x 5 (512) 485
// by sixteen, 301 as plan tasks.
static constexpr int64_t kLongFold = 4, kMostRounds = 40;

UnitRoute unit_route(const hp_nest* n, uint32_t flags, const Lowered& L, bool tuned) {
  UnitRoute r, off;
  memset(&r, 0, sizeof r);
  memset(&off, 0, sizeof off);
  if (n->dtype != HP_I32 && n->dtype != HP_F32 && n->dtype != HP_BF16) return off;
  const bool flt = n->dtype != HP_I32;
  const int es = n->dtype == HP_BF16 ? 2 : 4;
  const int64_t vec = 16 / es;
  const int d = n->depth;
  int p = 0;
  while (p < d && n->op[p] == HP_OP_NONE) ++p;
  if (p == d) return off;
  int64_t n_out = 1;
  for (int l = 0; l < p; ++l) n_out *= n->extent[l];
  // segments, outermost first; a SUM / MIN / MAX level of one iteration passes its value on
  int op[3], ns = 0;
  int64_t e[3];
  for (int l = p; l < d; ++l) {
    const bool arg = n->op[l] == HP_OP_ARGMIN || n->op[l] == HP_OP_ARGMAX;
    if (!arg && n->extent[l] == 1 && (ns || l + 1 < d)) continue;
    if (!arg && ns && op[ns - 1] == n->op[l]) {
      e[ns - 1] *= n->extent[l];
      continue;
    }
    if (ns == 3) return off;
    op[ns] = n->op[l];
    e[ns++] = n->extent[l];
  }
  if (!ns) return off;
  const int64_t lim = (int64_t)1 << 28;  // elements: 32-bit byte offsets inside a pair
  for (int k = 0; k < ns; ++k)
    if (e[k] > lim) return off;
  UnitDesc& D = r.d;
  D.eL = (int32_t)e[ns - 1];
  D.eM = ns >= 2 ? (int32_t)e[ns - 2] : 1;
  D.eQ = ns == 3 ? (int32_t)e[0] : 1;
  D.opL = op[ns - 1];
  D.opM = ns >= 2 ? op[ns - 2] : HP_OP_SUM;
  D.opQ = ns == 3 ? op[0] : HP_OP_NONE;
  D.direct = ns == 1 ? 1 : 0;
  if ((int64_t)D.eL * D.eM > lim || n_out > lim / D.eQ) return off;
  const int64_t pairs = n_out * D.eQ;
  D.pairs = pairs;
  D.out_kind = flt ? ((flags & HP_FLAG_OUT_F32) ? UNIT_F32 : UNIT_F64) : L.dp.out_kind == OUT_I64 ? UNIT_I64 : UNIT_I32;
  // a row's value leaves as its operator's type, unless a level of one iteration widened it
  if (!flt && (D.out_kind == UNIT_I64) != (D.opL == HP_OP_SUM)) D.direct = 0;
  D.mparts = D.lparts = 1;
  D.run = 1;
  const int64_t pair_bytes = (int64_t)D.eL * D.eM * es;
  // lanes of a row, and pairs side by side while M leaves lane groups over
  const int64_t need = cdiv(D.eL, vec);
  D.lane_bits = D.eL < vec ? 0 : need >= kWave ? 6 : log2u((uint64_t)need);
  int64_t groups = 1;
  auto shape = [&]() {
    D.vecs = D.eL < vec ? 0 : (int32_t)cdiv(need, (int64_t)1 << D.lane_bits);
    const int64_t rows = kWave >> D.lane_bits;
    D.pair_bits = 0;
    while (2 * (int64_t)D.eM <= (rows >> D.pair_bits)) ++D.pair_bits;
    D.steps = (int32_t)cdiv(D.eM, rows >> D.pair_bits);
    groups = cdiv(pairs, (int64_t)1 << D.pair_bits);
  };
  shape();
  int64_t lparts = 1, mparts = 1, run = 1;
  if (tuned && ns == 1 && L.dp.nw == 1) {
    // the cached recipe's grid: parts per output, or outputs per unit on its lanes
    lparts = L.dp.gsplit;
    if (lparts == 1) {
      int lanes = 0;
      for (int l = 0; l < L.dp.depth; ++l)
        if (l >= L.dp.p) lanes += log2u((uint64_t)L.dp.lv[l].vf);
      // (beyond 8 vectors per lane a row takes the whole wave instead)
      if (lanes < D.lane_bits && D.eL >= vec && cdiv(need, (int64_t)1 << lanes) < 8) {
        D.lane_bits = lanes;
        shape();
      }
      const int64_t units = L.dp.grid > groups ? groups : L.dp.grid;
      run = cdiv(groups, units);
    }
  } else {
    const int64_t step = (D.vecs ? D.vecs : 1) + (D.vecs >= 8 ? 2 : flt || D.direct ? 4 : 6), pair = step * D.steps;
    if (pair <= 2 * kUnitCost) {
      run = kUnitCost / pair;
    } else if (step <= 2 * kUnitCost) {
      mparts = cdiv(pair, kUnitCost);
      if (mparts > D.steps) mparts = D.steps;
    } else {
      lparts = cdiv(step, kUnitCost);
    }
  }
  if (lparts > 1 && D.eL < 4 * vec * kWave) lparts = 1;
  if (lparts > 1) {
    // parts of whole passes of the wave (64 vectors), the last not shorter than a vector
    int64_t len = cdiv(cdiv(D.eL, lparts), vec * kWave) * vec * kWave;
    lparts = cdiv(D.eL, len);
    while (lparts > 1 && D.eL - (lparts - 1) * len < vec) {
      len += vec * kWave;
      lparts = cdiv(D.eL, len);
    }
    D.lparts = (int32_t)lparts;
    D.part_len = (int32_t)len;
    D.lane_bits = 6;
  }
  if (lparts == 1 && mparts > 1) {
    D.per = (int32_t)cdiv(D.steps, mparts);
    mparts = cdiv(D.steps, D.per);
    D.mparts = (int32_t)mparts;
  }
  // 32-bit offsets inside a unit of short rows
  const int64_t group_elems = ((int64_t)D.eL * D.eM) << D.pair_bits;
  if (run > lim / group_elems) run = lim / group_elems;
  if (run < 1) run = 1;
  if (run > groups) run = groups;
  D.run = (int32_t)(run > 0x7FFFFFFF ? 0x7FFFFFFF : run);
  const int64_t most = 0x7FFFFFFF;
  int64_t carriers = 0;
  if (D.lparts > 1) {
    if (pairs * D.eM > most / D.lparts) return off;
    r.units = pairs * D.eM * D.lparts;
    carriers = r.units;
    r.unit_bytes = (double)D.part_len * es;
  } else if (D.mparts > 1) {
    if (pairs > most / D.mparts) return off;
    r.units = pairs * D.mparts;
    carriers = r.units;
    r.unit_bytes = (double)pair_bytes * D.per / D.steps;
  } else {
    r.units = cdiv(groups, D.run);
    carriers = ns == 3 ? pairs : 0;
    r.unit_bytes = (double)(pair_bytes << D.pair_bits) * D.run;
    // carriers of 16 bytes must stay well below the input they stand for, or be few
    if (carriers && pair_bytes < 32 && carriers > (1 << 18)) return off;
  }
  // Device memory that the plan's tasks do without, with the fold tasks: up to 64 MiB, or a
  // sixteenth of the input (1048576 x 64 x 4 x 2, 2 GiB, would keep another GiB).
  const int64_t kept = carriers * kSlotBytes + (carriers ? n_out * 8 : 0), some = (int64_t)(L.info.in_bytes / 16);
  if (kept > 64 << 20 && kept > some && kept > (int64_t)L.info.workspace_bytes) return off;
  D.partial = carriers ? 1 : 0;
  D.fold_waves = 1;
  if (carriers) {
    const int64_t rows = D.lparts > 1 ? D.eM : 1, parts = D.lparts > 1 ? D.lparts : D.mparts;
    FoldPlan f = fold_plan(ns == 3, D.eQ, rows, parts, 1);
    if (f.rounds > (n_out <= 256 ? kLongFold : 8 * kLongFold)) {
      D.fold_waves = kFoldWaves;
      f = fold_plan(ns == 3, D.eQ, rows, parts, kFoldWaves);
      if (f.rounds > (L.dp.chunk > 1 ? kMostRounds : 4 * kMostRounds)) return off;
    }
    D.fold_form = f.form;
  }
  r.folds = carriers ? n_out : 0;
  r.ws_bytes = (uint64_t)carriers * kSlotBytes;
  r.dtype = n->dtype;
  r.on = 1;
  return r;
}

}  // namespace hp
