// Internal: tile shapes of the bf16 GEMM (gemm_bf16.hip) and the choice among them for one
// product.  Pure host arithmetic, also used to size workspaces.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace ffsplit {

enum {
  GEMM_128x128 = 0,   // 4 wavefronts, wave tile 64x64, two workgroups per CU
  GEMM_128x256 = 1,   // 4 wavefronts, wave tile 128x64, two workgroups per CU
  GEMM_128x320 = 2,   // 8 wavefronts, wave tile 64x80
  GEMM_256x256 = 3,   // 8 wavefronts, wave tile 128x64 (two left operands: gemm_dual.hip)
  GEMM_256x320 = 4,   // 8 wavefronts, wave tile 128x80
  GEMM_64x64 = 5,     // 4 wavefronts, wave tile 32x32
  GEMM_64x128 = 6,    // 4 wavefronts, wave tile 32x64
  GEMM_SHAPES = 7
};

struct GemmPlan {
  int shape;
  int split;   // > 1: that many ranges of the reduction, fp32 partials, one summing launch
  int fix;     // the ranges are added inside the launch
};

// Choice by estimated time.  A launch of W workgroups puts ceil(W / 256) of them on the fullest
// CU; each walks its share of the 32-deep slabs at the shape's time per slab (t1: alone on its CU,
// t2: both of two residents) and pays a fixed part (ring filling, store).  `row`: factor of t1 and
// t2 for a row-major left operand, whose loads fetch 64 bytes of a row at a time.  Partial sums
// cost a launch, their traffic and a dependent load per range.
// The figures (us) are a least-squares fit to the DIFFERENCES between whole forward passes that run
// one product on another tile or number of ranges: 4000 such runs over 489 products of 65 to 8192
// tokens, model widths 512 to 5120.  What every choice pays alike is not in them (the power limit
// above all: 256x256 tiles of a large product take 0.66 us a slab by themselves), so they rank the
// choices and do not predict a launch's length: the traced length is up to 1.5 times the estimate.
// The chosen tile's pass is 0.24 % longer than the best one's on average, 1.6 % in the 95th
// percentile; with figures from products timed alone, one after another, it was 1.25 % and 7 %
// (too many ranges, and ranges where none was best).
// 128x320, 256x320 and 64x64 have no gated form (a wavefront's columns do not hold whole (gate, up)
// pairs); two left operands: 128x128 and 256x256 only, never split.
struct GemmShape { int bm, bn, per_cu; double t1, t2, fixed, row; };
inline const GemmShape& gemm_shape(int shape, bool dual) {
  static const GemmShape single[GEMM_SHAPES] = {{128, 128, 2, 0.177, 0.332, 2.6, 1.21}, {128, 256, 2, 0.287, 0.526, 4.4, 1.12},
                                                {128, 320, 1, 0.359, 0, 4.3, 1.11},     {256, 256, 1, 0.453, 0, 6.8, 1.08},
                                                {256, 320, 1, 0.565, 0, 8.1, 1.09},     {64, 64, 2, 0.105, 0.154, 1.5, 1.155},
                                                {64, 128, 2, 0.135, 0.239, 1.9, 1.14}};
  static const GemmShape two[GEMM_SHAPES] = {{128, 128, 2, 0.150, 0.332, 2.5, 1.0}, {}, {}, {256, 256, 1, 0.428, 0, 5.9, 1.0}, {}, {}, {}};
  return dual ? two[shape] : single[shape];
}
inline bool gemm_shape_usable(const GemmShape& c, bool glu) { return c.bm > 0 && !(glu && (c.bn == 320 || c.bn == 64)); }
constexpr int GEMM_MAX_SPLIT = 16, GEMM_MIN_SLABS = 8;   // ranges of a reduction; slabs of 32 per range
constexpr double GEMM_SUM_US = 3.4, GEMM_SUM_RANGE_US = 0.29, GEMM_SUM_BYTES_PER_US = 3.4e6;
inline size_t gemm_part_bytes(int64_t M, int N, int split) { return (size_t)split * M * ((N + 31) / 32 * 32) * 4; }

// With `fix`, ranges of 64x64 tiles are added inside the launch by the last workgroup of a tile (un-activated
// products behind the first, GemmPlan::fix), 1.7 us less than a summing launch: 300 tokens of an OPT-1.3B-sized layer
// 44.5 -> 42.8 us, of a Llama-2-7B-sized one 75.7 -> 72.9.  With larger tiles one CU's reads of all ranges
// take as long as that launch or longer (256x256, three ranges: equal; four: 36 us of 365 slower).
constexpr double GEMM_FIX_GAIN_US = 1.7;
constexpr int GEMM_FIX_MAX_SPLIT = 8;
constexpr int FIX_COUNTERS = 256;   // tiles of a product whose ranges are added inside the launch (two ranges fill its one round)
inline size_t gemm_fix_bytes(int64_t M, int N, int split) { return (size_t)((M + 63) / 64) * ((N + 63) / 64) * split * 16384; }

// A reduction is split only to fill one round of the machine (256 CUs times the residents of a CU).
inline GemmPlan gemm_plan(int64_t M, int N, int K, bool glu, bool dual, bool a_tiled, bool can_split, bool fix = false) {
  GemmPlan best = {GEMM_128x128, 1, 0};
  double best_t = 1e30;
  const int slabs = (K + 31) / 32;
  for (int s = 0; s < GEMM_SHAPES; ++s) {
    const GemmShape& c = gemm_shape(s, dual);
    if (!gemm_shape_usable(c, glu)) continue;
    const double row = a_tiled ? 1.0 : c.row;
    const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    for (int sp = 1; sp == 1 || (can_split && sp <= GEMM_MAX_SPLIT && slabs / sp >= GEMM_MIN_SLABS &&
                                 tiles * sp <= 256 * c.per_cu); ++sp) {
      const int64_t load = (tiles * sp + 255) / 256;
      const int n = (slabs + sp - 1) / sp;
      double t = c.per_cu == 1 ? load * (n * c.t1 * row + c.fixed)
                               : (load / 2) * (n * c.t2 * row + c.fixed) + (load & 1) * (n * c.t1 * row + c.fixed);
      const bool in_launch = fix && s == GEMM_64x64 && sp > 1 && sp <= GEMM_FIX_MAX_SPLIT;
      if (in_launch) t -= GEMM_FIX_GAIN_US;
      if (sp > 1) t += GEMM_SUM_US + GEMM_SUM_RANGE_US * (sp - 1) + (double)gemm_part_bytes(M, N, sp) / GEMM_SUM_BYTES_PER_US;
      if (t < best_t) { best_t = t; best.shape = s; best.split = sp; best.fix = in_launch; }
    }
  }
  return best;
}

// Bytes that hold the partial sums of any plan of at most M rows, so that a workspace sized for a batch
// serves every smaller one (the plans' own need rises and falls with M).  A plan of `sp` ranges has at
// most one round of tiles, and its summing costs less than the shape would lose without it.
inline size_t gemm_part_room(int64_t M, int N, int K, bool glu, bool a_tiled) {
  size_t room = 0;
  const int slabs = (K + 31) / 32;
  for (int s = 0; s < GEMM_SHAPES; ++s) {
    const GemmShape& c = gemm_shape(s, false);
    if (!gemm_shape_usable(c, glu)) continue;
    const int64_t tiles_n = (N + c.bn - 1) / c.bn;
    for (int sp = 2; sp <= GEMM_MAX_SPLIT && slabs / sp >= GEMM_MIN_SLABS; ++sp) {
      const int64_t rows = 256 * c.per_cu / (sp * tiles_n) * c.bm;
      const bool in_launch = a_tiled && !glu && s == GEMM_64x64 && sp <= GEMM_FIX_MAX_SPLIT;
      const double gain = (slabs - (slabs + sp - 1) / sp) * c.t1 * (a_tiled ? 1.0 : c.row) - GEMM_SUM_US -
                          GEMM_SUM_RANGE_US * (sp - 1) + (in_launch ? GEMM_FIX_GAIN_US : 0.0);
      if (rows <= 0 || gain <= 0) continue;
      const int64_t m = rows < M ? rows : M;
      const size_t fits = gemm_part_bytes(m, N, sp), pays = (size_t)(gain * GEMM_SUM_BYTES_PER_US) + 256;
      size_t b = fits < pays ? fits : pays;
      // (whole tiles where the ranges are added inside the launch)
      if (in_launch && gemm_fix_bytes(m, N, sp) > b) b = gemm_fix_bytes(m, N, sp);
      if (b > room) room = b;
    }
  }
  return room;
}
}  // namespace ffsplit
