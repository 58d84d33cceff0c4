// Internal: tile shapes of the bf16 GEMM (gemm_bf16.hip) and the choice among them for one
// product.  Pure host arithmetic, also used to size workspaces.
#pragma once
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
};

// Choice by estimated time.  A launch of W workgroups puts ceil(W / 256) of them on the fullest
// CU; each walks its share of the 32-deep slabs at the shape's measured time per slab (t1: alone
// on its CU, t2: both of two residents) and pays a fixed part (ring filling, store).  Partial sums
// cost their traffic at 4.2 TB/s and a launch.  Measured on random operands (us per slab): 128x128
// 0.21 alone, 0.40 as a pair (bound by the 61 bytes per clock a CU's vector cache delivers);
// 128x256 0.38 / 0.70; 128x320 0.50; 256x256 0.66; 256x320 1.0 (the last two are at the power
// limit: 1.5 PFLOP/s); 64x64 0.15 / 0.21 and 64x128 0.19 / 0.34 (four resp. eight MFMAs a wavefront
// between barriers: bound by the latency of a slab, so they pay where larger tiles leave CUs idle or
// need a split and its summing launch.  With them (us, before -> now): OPT-1.3B-sized layer, 65
// tokens 45 -> 37, 300 with biases 56.4 -> 49.2, 1000 61 -> 55, 2000 81.5 -> 76.8; a 768-wide one,
// 400 tokens 37 -> 27.6; Llama-2-7B-sized, 200 tokens 89.4 -> 82.5; the OPT-13B-sized one is unchanged).
// 128x320, 256x320 and 64x64 have no gated form (a wavefront's columns do not hold
// whole (gate, up) pairs); two left operands: 128x128 and 256x256 only, never split.
inline GemmPlan gemm_plan(int64_t M, int N, int K, bool glu, bool dual, bool can_split) {
  struct Shape { int bm, bn, per_cu; double t1, t2, fixed; };
  static const Shape single[GEMM_SHAPES] = {{128, 128, 2, 0.215, 0.40, 2.5}, {128, 256, 2, 0.38, 0.70, 3.0},
                                            {128, 320, 1, 0.50, 0, 4.0},     {256, 256, 1, 0.66, 0, 6.0},
                                            {256, 320, 1, 1.0, 0, 6.0},     {64, 64, 2, 0.15, 0.21, 2.5},
                                            {64, 128, 2, 0.19, 0.34, 2.5}};
  static const Shape two[GEMM_SHAPES] = {{128, 128, 2, 0.30, 0.55, 3.0}, {}, {}, {256, 256, 1, 0.85, 0, 6.0}, {}, {}, {}};
  GemmPlan best = {GEMM_128x128, 1};
  double best_t = 1e30;
  const int slabs = (K + 31) / 32;
  for (int s = 0; s < GEMM_SHAPES; ++s) {
    const Shape& c = dual ? two[s] : single[s];
    if (c.bm == 0 || (glu && (c.bn == 320 || c.bn == 64))) continue;
    const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    for (int sp = 1; sp <= (can_split ? 16 : 1) && (sp == 1 || slabs / sp >= 8); ++sp) {
      const int64_t load = (tiles * sp + 255) / 256;
      const int n = (slabs + sp - 1) / sp;
      double t = c.per_cu == 1 ? load * (n * c.t1 + c.fixed)
                               : (load / 2) * (n * c.t2 + c.fixed) + (load & 1) * (n * c.t1 + c.fixed);
      if (sp > 1) t += 4.0 + (double)sp * M * N * 4 / 4.2e6;
      if (t < best_t) { best_t = t; best.shape = s; best.split = sp; }
    }
  }
  return best;
}

}  // namespace ffsplit
