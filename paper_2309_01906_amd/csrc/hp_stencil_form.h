// Which form a stencil launch takes, and the register form's strips (host only; the kernels
// are in hp_stencil.hip).
#pragma once

#include "hp_internal.h"

namespace hp {

constexpr int kRegCols = 4 * kWave;  // columns of a wave's strip in the register form
constexpr int reg_ghost(int t) { return t <= 4 ? 4 : 8; }

// Rows per wave: the waves of nb row blocks run as `used` = ceil(waves / SIMDs) shares
// of rows + 2 T steps on the fullest SIMD.  From 5 sweeps the steps are issue-bound and
// a wave alone leaves gaps, worth about 1.2 of a share, and more than three shares never
// pay for their ghost rows (8192 x 8192, 8 sweeps: 3 shares of 111 steps 148 us, 2 of 158
// 162 us; 7 sweeps: 3 shares 134 us, 4 149 us).  Below that HBM is the bound and few long
// strips stream best, but at least two waves per SIMD (8192 x 8192, 4 sweeps: 2 shares
// 122 us, 4 shares 130 us).
inline int reg_rows(long long R, long long C, int t) {
  const long long simds = 1024;  // 256 compute units x 4
  const long long w = kRegCols - 2 * reg_ghost(t);
  const long long ns = (C + w - 1) / w;
  long long best = 0, rows = R;
  for (long long k = 1; k <= (t >= 5 ? 3 : 8); ++k) {
    long long nb = k * simds / ns;
    if (nb < 1) nb = 1;
    const long long rb = (R + nb - 1) / nb;
    const long long used = (ns * ((R + rb - 1) / rb) + simds - 1) / simds;
    const long long cost = (t >= 5 ? 10 * used + 12 : 10 * (used < 2 ? 2 : used)) * (rb + 2 * t);
    if (best == 0 || cost < best) {
      best = cost;
      rows = rb;
    }
  }
  return (int)rows;
}

// Whether a launch of t sweeps takes the register form.  Measured against the best LDS
// tile: one sweep stays with LDS (8192 x 8192: 98 against 111 us, both near a copy's
// rate), two sweeps too on arrays beyond the last-level cache (8192 x 8192: 102 against
// 110 us; 4096 x 4096: 25 against 24 us) and on narrow ones that fill their strips
// badly (7000 x 300: 7.8 against 8.6 us); with 3 and 4 sweeps registers are faster
// (8192 x 8192, 4: 147 -> 122 us) but on large arrays that fill their strips badly (3000
// x 500, 4: 10.2 against 10.6 us).  One or two strips both hold an edge, whose columns are
// loaded and stored one by one: tall ones stay with LDS where that has been the faster form
// (2 sweeps: 2516 x 484 7.4 against 8.7 us, but 380 x 492 5.9 against 4.6; 3: 4096 x 380 8.6
// against 9.4; 4: 2048 x 256 8.3 against 8.9).  From 5 sweeps a wave of a small array has
// more ghost rows than rows of its own, and both forms are mostly latency: what each takes
// then is estimated, in tenths of a microsecond -- the register form by the steps of the
// fullest SIMD's waves (rows and ghost rows), the LDS form by the tiles of a compute unit,
// each with its launch -- from fits to 18 arrays of 200 x 200 to 8192 x 8192 cells (LDS
// against registers, 8 sweeps: 600 x 600 15.0 and 13.6 us, 1024 x 1024 15.7 and 16.3,
// 7000 x 300, whose two strips both hold an edge, 20.6 and 22.0, 1500 x 1500 20.5 and
// 18.5, 8192 x 8192 266 and 148).  Over 6,200 arrays of 3 x 3 to 8192 x 8192 cells ten were
// more than 4 % slower than in LDS, by at most 7 %.
inline bool reg_form(long long R, long long C, int t) {
  if (t <= 1) return false;
  const long long w = kRegCols - 2 * reg_ghost(t), ns = (C + w - 1) / w;
  const bool full = 10 * C > 9 * ns * w;
  if (t == 2 && (ns == 2 ? R > 800 : ns == 1 && R > (full ? 1024 : 4096))) return false;
  if (t == 2) return R < (1ll << 25) / C && 4 * C >= 3 * ns * w;
  const double tiles = (double)((R + 63) / 64) * (double)((C + 63) / 64) / 256;  // 64 x 64, per compute unit
  if (t == 3 && (ns == 2 ? 4 * C > 3 * ns * w && R > 2048 && R <= 4608 : ns == 1 && full && R > 1024)) return false;
  if (t == 4 && ns == 2 && R > 1024 && R <= 2048) return false;
  if (t <= 4) return 10 * C >= 7 * ns * w || tiles <= 1;
  const long long rows = reg_rows(R, C, t), used = (ns * ((R + rows - 1) / rows) + 1023) / 1024;
  const double reg = 33 + 0.78 * t * (double)(rows + 2 * t) * (double)(10 * used + 12) / 22 * (ns <= 2 ? 1.05 : 1.0);
  const double lds = 3 + 18.5 * t + (tiles > 1 ? 5.6 * t * (tiles - 1) : 0);
  return reg <= lds;
}

}  // namespace hp
