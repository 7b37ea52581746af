// Launch schedules of a plan: the shapes of the modal contractions (host rules
// on rows, modes and bases) and their form in momfbd_tuning.
//
// The gradient's and the phase's shape are either selected or open, and an open
// one is chosen here by size.  get_tuning reports an open shape under a pair of
// values that selects nothing else (4 row tiles; 8 x 8, or 2 x 4 where 8 x 8
// would not fit), and set_tuning takes these, like 0, as open: what get_tuning
// reports restores what ran, on this plan and, open or selected, on another.
#pragma once

#include "contract_mfma.h"
#include "internal.h"
#include "momfbd.h"

namespace mfbd {

constexpr int kCus = 256;
constexpr size_t kLdsPerCu = 160 * 1024;

// ---- gradient
// Few rows under an open schedule (4 waves, row tiles 0) take the kernel that
// stages nothing (k_grad_rows), whose basis reads grow with rows x mode tiles
// and which needs no block of 128 rows to be full: 11.6 against 12.4 us at 2700
// rows x 3 tiles (64 x 64), 18 against 21.5 at 1000 x 10, 29 against 73 at 441 x
// 5 (128 x 128, three bases), but 27.8 against 20 at 5400 x 6 and 26.3 against
// 25.7 at 1944 x 8.
constexpr long kFewRowTiles = 12000;
inline bool grad_few_rows(const Dims& d) {
  return d.grad_waves != 8 && d.grad_rt == 0 &&
         (long)d.P * d.J * ((d.M + 15) / 16) <= kFewRowTiles;
}

// Row tiles per wave of the staged kernel (open: 2, whose blocks of 128 rows
// were the fastest staged shape at every size measured).
inline int grad_row_tiles_of(const Dims& d) {
  return d.grad_waves == 8 || d.grad_rt == 0 ? 2 : d.grad_rt;
}

inline int grad_splits_staged(long blocks, int nchunk) {
  // a block for every CU, as long as every split keeps at least 4 chunks of
  // 32 pixels to pipeline through its LDS stages (2 row tiles x 4 waves, 5400
  // rows x 88 modes at 64 x 64: 21 us at 8 splits of 4 chunks, 22.6 at 4;
  // 11 532 x 66: 32.4 at 4 splits, 33.2 at 8)
  int s = 1;
  while (s < kMaxGradSplits && blocks * s < kCus && nchunk / (2 * s) >= 4) s *= 2;
  return s;
}

inline int grad_splits_auto(const Dims& d) {
  const int R = d.P * d.J, W = d.grad_waves == 8 ? 8 : 4;
  const int zc = d.zc > 0 ? d.zc : d.C;
  const int nchunk = zc * d.bandpix() / 32;
  const long rows = 16L * grad_row_tiles_of(d) * W, blocks = (R + rows - 1) / rows;
  if (grad_few_rows(d) || R <= 256) {
    // at least 8 chunks to a split
    int s = 1;
    while (s < kMaxGradSplits && blocks * s < 512 && nchunk / (2 * s) >= 8) s *= 2;
    return s;
  }
  return grad_splits_staged(blocks, nchunk);
}

inline int grad_splits_of(const Dims& d) {
  return d.grad_splits > 0 ? d.grad_splits : grad_splits_auto(d);
}

// ---- phase
// Open: 64 columns and 8 waves, the faster at nearly every size beyond kFewCols
// columns: 9.7 against 12.6 us (128 columns, 8 waves) at 2700 columns x 44 modes,
// 26.7 against 29.5 at 11 532 x 66 (64 x 64), 97 against 129 at 3072 x 150 (128 x
// 128, four bases); they fit for every mode count.  From 193 modes on they take
// more than half of a CU's LDS, and a launch of many blocks does better with
// three blocks of 32 columns there: 200 modes of 64 x 64, 3072 columns 22.0
// against 28.8 us (two bases 28.6 against 37.8), 3844 columns 20.3 against 26.5, 11
// 532 columns 54 against 62; two bases of 96 x 96, 4000 columns, 62 against 66, of
// 128 x 128, 1536 columns, 51 against 58 (48 columns, two blocks: 19.8, 27.3, 25.0,
// 52, 64 and 46, but 40 against 35 at 4000 columns of 96 x 96, one basis).  At
// 800 columns of 96 x 96, one basis, 19.4 against 17.7: fewer blocks keep 64.
// Up to kFewCols columns the kernel that stages nothing: 3.1 against 5.1 us at 8
// columns x 44 modes, 4.3 against 12.3 at 128 x 66 (64 x 64), 9 against 16.2 at 120
// x 150 (128 x 128), but 12.8 against 7.9 at 200 x 66 (96 x 96, three bases).
constexpr int kFewCols = 128;
struct PhaseShape {
  bool few;        // nothing staged (ct, waves unused)
  int ct, waves;   // 16-column tiles and waves per workgroup
};
inline PhaseShape phase_shape_of(const Dims& d, int Mq) {
  if (d.phase_ct > 0) return PhaseShape{false, d.phase_ct, d.phase_waves};
  const long R = (long)d.P * d.J, zc = d.zc > 0 ? d.zc : d.C;
  if (R <= kFewCols) return PhaseShape{true, 0, 0};
  const bool one_per_cu = 2 * contract::phase_lds_bytes(4, Mq) > kLdsPerCu;
  const long blocks = 4 * zc * ((R + 63) / 64);   // a quarter of the band each
  return PhaseShape{false, one_per_cu && blocks >= 3 * kCus / 4 ? 2 : 4, 8};
}

// A shape that can be selected for Mq padded modes: its staged coefficients
// must fit 128 KB of LDS.
inline bool phase_shape_fits(int ct, int waves, int Mq) {
  return ((ct == 4 && waves == 8) || (ct == 8 && waves == 16)) &&
         contract::phase_lds_bytes(ct, Mq) <= 128 * 1024;
}

// The pair that stands for the open shape.
inline void phase_open_pair(int Mq, int* ct, int* waves) {
  const bool wide = contract::phase_lds_bytes(8, Mq) <= 128 * 1024;
  *ct = wide ? 8 : 2;
  *waves = wide ? 8 : 4;
}

// ---- momfbd_tuning
inline bool schedule_values_ok(const momfbd_tuning& t) {
  return (t.xcd_forward == 0 || t.xcd_forward == 1) && (t.xcd_adjoint == 0 || t.xcd_adjoint == 1) &&
         (t.object_pairs_per_thread == 1 || t.object_pairs_per_thread == 2 ||
          t.object_pairs_per_thread == 4) &&
         (t.grad_waves == 4 || t.grad_waves == 8) &&
         (t.grad_splits == 0 || t.grad_splits == 1 || t.grad_splits == 2 || t.grad_splits == 4 ||
          t.grad_splits == 8) &&
         (t.grad_row_tiles == 0 ||
          (t.grad_waves == 4 ? t.grad_row_tiles >= 2 && t.grad_row_tiles <= 4
                             : t.grad_row_tiles == 2)) &&
         (t.object_fused == 0 || t.object_fused == 1);
}

// The schedule of `t` into `d`; false, and `d` as it was, for a value out of range.
inline bool schedule_set(const momfbd_tuning& t, int Mq, Dims& d) {
  if (!schedule_values_ok(t)) return false;
  int ct = 0, waves = 0;
  phase_open_pair(Mq, &ct, &waves);
  const bool open = (t.phase_col_tiles == 0 && t.phase_waves == 0) ||
                    (t.phase_col_tiles == ct && t.phase_waves == waves);
  if (!open && !phase_shape_fits(t.phase_col_tiles, t.phase_waves, Mq)) return false;
  d.phase_ct = open ? 0 : t.phase_col_tiles;
  d.phase_waves = open ? 0 : t.phase_waves;
  d.xcd_fwd = t.xcd_forward;
  d.xcd_adj = t.xcd_adjoint;
  d.obj_ppt = t.object_pairs_per_thread;
  d.grad_waves = t.grad_waves;
  d.grad_splits = t.grad_splits;
  d.grad_rt = t.grad_waves == 8 || t.grad_row_tiles == 4 ? 0 : t.grad_row_tiles;
  d.fuse_obj = t.object_fused;
  return true;
}

inline momfbd_tuning schedule_get(const Dims& d, int Mq) {
  momfbd_tuning t;
  t.xcd_forward = d.xcd_fwd;
  t.xcd_adjoint = d.xcd_adj;
  t.object_pairs_per_thread = d.obj_ppt;
  t.grad_waves = d.grad_waves;
  t.grad_splits = grad_splits_of(d);
  t.grad_row_tiles = d.grad_waves == 8 ? 2 : d.grad_rt == 0 ? 4 : d.grad_rt;
  t.phase_col_tiles = d.phase_ct;
  t.phase_waves = d.phase_waves;
  if (d.phase_ct == 0) phase_open_pair(Mq, &t.phase_col_tiles, &t.phase_waves);
  t.object_fused = fused_object(d) ? 1 : 0;
  return t;
}

}  // namespace mfbd
