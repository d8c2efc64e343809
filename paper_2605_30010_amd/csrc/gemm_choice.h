// Which workgroup tiling each part of a GEMM runs on.  Plain C++ without HIP: launch_gemm carries out what
// plan_gemm lists, and a test on the CPU checks that list over the sizes.
//
// The rows of one matrix are summed over k in one order.  Equal rows (the tokens of a frame that stands still)
// then have equal bits wherever they lie, so the similarities of equal frames are equal and Alg. 1's strict
// comparison fuses none of them.  A launch over all rows may use any order; a launch over some of them takes only the
// tilings that add k-steps in ascending order to one accumulator.
#pragma once

namespace et {

// Workgroup tilings (tile_config of et_gemm_bf16, up to kCfgHalf):
//   0  256 x 256, 8 wavefronts, persistent, one workgroup per compute unit
//   1  128 x 128, 4 wavefronts, persistent, two workgroups per compute unit
//   2   64 x  64, k split over 4 wavefronts, two workgroups per compute unit      (gemm_small.hip)
//   3  128 x  64, k split over 2 groups of 4 wavefronts (4 of 2 where k-tiles are odd) (gemm_small.hip)
//   4  128 x 128, k split over 2 groups of 4 wavefronts                           (gemm_small.hip)
//   5  256 x 128, 8 wavefronts in two alternating halves                          (gemm_small.hip)
//   6   64 x  64, 4 wavefronts with a quadrant each, two workgroups per compute unit (gemm_small.hip): the last tile rows only
enum { kCfgBig = 0, kCfg128 = 1, kCfgWave = 2, kCfgPair64 = 3, kCfgPair128 = 4, kCfgHalf = 5, kCfgStrip = 6, kCfgCount = 7 };

// One accumulator per output element, k ascending.
inline bool in_k_order(int cfg) { return cfg == kCfgBig || cfg == kCfg128 || cfg == kCfgHalf || cfg == kCfgStrip; }

inline long gemm_tiles(int cfg, long rows, long cols) {
  static const int bm[kCfgCount] = {256, 128, 64, 128, 128, 256, 64}, bn[kCfgCount] = {256, 128, 64, 64, 128, 128, 64};
  return ((rows + bm[cfg] - 1) / bm[cfg]) * ((cols + bn[cfg] - 1) / bn[cfg]);
}

// Expected time of one launch in microseconds, launch overhead included: a fixed part (first loads,
// epilogue) plus a part per k-tile of 64 in each round of tiles.  A compute unit is slower when its
// neighbours work too (shared caches, and the clock falls with the power drawn), hence the terms in
// t / slots.  Fitted to launches on 256 compute units at widths of 768 to 4352, 64 to 13122 rows, weights
// from HBM; measured at K = 1152 / 4352:
//   wave     6.5-7 / 15-17 us for one round of 256 tiles, 10 / 28 for two, 14 / 40 for three
//   pair64   8.3 / 23 for one round, 15.4 / 43 for two; an odd number of k-tiles, one round at 5, 7, 11, 17, 69 of them, 7.2, 7.8, 9.0, 11.0,
//            26.0 where 6, 8, 12, 18, 68 take 6.8, 7.2, 8.5, 10.1, 24.4
//   pair128  11-12.5 / 30-33 for one round, 22 / 63 for two
//   half     17 / 47 (135 tiles), 18.3 / 52 (207-243), 34 / 103 for two rounds, 50 for three
//            5 to 8 k-tiles, a round of several: 8.9-10.8 (5), 10.4-11.8 (7), 12.3-13.5 (8)
//   128      half rounds of 256 tiles: 13.8, 18, 26, 33.5, 40.5, .. 56 for seven; with a residual 17.5 / 52.5, 21.3 / 62.5, 36 /
//            110, 40 / 133 (the loads of the residual rows wait for the next tile's operands)
//   256      25 / 80 (70 tiles), 26 (182), 30.5 (252), 33 / 98 (230, residual), 55 (448), 87 (728)
//   strip    7.4 (54 tiles) / 18, 8.2 (204), 10.4 (340), 18 / 45 for four and three rounds
inline double gemm_cost(int cfg, long rows, long cols, int K, bool residual = false) {
  const double kt = K / 64;
  const long t = gemm_tiles(cfg, rows, cols);
  auto rounds = [](long n, long slots) { return (double)((n + slots - 1) / slots); };
  switch (cfg) {
    case kCfgWave: return 3.2 + rounds(t, 256) * 0.195 * kt;
    case kCfgPair64:                                       // (two kernels, see above)
      return 0.5 + rounds(t, 256) * ((K / 64) % 2 ? 2.9 + 0.32 * kt : 2.7 + 0.298 * kt);
    case kCfgPair128: return t <= 256 ? 3.6 + kt * (0.36 + 0.09 * (double)t / 256.0) : 0.5 + rounds(t, 256) * (3.2 + 0.42 * kt);
    case kCfgHalf:                                         // (of several rounds each pays its own first loads and epilogue: short k-loops)
      if (t > 256) return rounds(t, 256) * (kt > 4 && kt < 11 ? 5.0 + 0.56 * kt : 2.2 + 0.82 * kt);
      return 5.5 + kt * (0.56 + 0.16 * (double)t / 256.0);
    case kCfgStrip: return 3.2 + rounds(t, 256) * 0.205 * kt;
    case kCfg128: {
      const double h = rounds(t, 256);                     // half rounds: two workgroups share a compute unit
      // (Dearer by design than 256 x 256: this formula gives 0.9 to 1.0 of what a launch takes by itself, that one 0.75 at short K, 0.8
      // to 0.9 at 12 to 24 k-tiles and 0.95 beyond, with a residual, which it has no term for, and without.  128 x 128 moves more
      // operand bytes, which costs clock in the launches beside it.  Over 130 launches of 1500 to 24000 rows what is chosen takes
      // 1.6 % longer than the fastest single tiling, with a residual at most 8 %.)
      if (!residual) return h < 2 ? 4.2 + 0.5 * kt : 4.2 + 0.8 * kt + (h - 2) * (0.9 + 0.45 * kt);
      const long pairs = (long)h / 2;
      const double single = (long)h % 2 ? 1.0 : 0.0;
      if (pairs == 0) return 3.5 + 0.72 * kt;
      return 6.5 + 0.82 * kt + (double)(pairs - 1) * (0.6 + 1.02 * kt) + single * (3.0 + 0.66 * kt);
    }
    default: {
      const long last = t % 256;
      return (double)(t / 256) * (1.5 + 1.47 * kt) + (last ? 4.0 + kt * (1.0 + 0.42 * (double)last / 256.0) : 2.5);
    }
  }
}

// Whether the persistent kernel walks one tile per workgroup on `cus` compute units (the others always do).  What it
// refuses otherwise depends on this, so the device's own count is asked for; the costs above only rank the tilings
// and keep the 256 units that they were measured on.
inline bool one_round(int cfg, long rows, long cols, int cus) {
  if (cfg == kCfgBig) return gemm_tiles(cfg, rows, cols) <= cus;
  if (cfg == kCfg128) return gemm_tiles(cfg, rows, cols) <= 2L * cus;
  return true;
}

struct GemmPart {
  int row0, rows, col0, cols, cfg;
};
struct GemmPlan {
  static constexpr int kMax = 16;
  GemmPart part[kMax];
  int n = 0;
  void add(long row0, long rows, long col0, long cols, int cfg) {
    part[n++] = GemmPart{(int)row0, (int)rows, (int)col0, (int)cols, cfg};
  }
};

// What plan_gemm may do: split rows off into launches of their own; only tilings that walk one tile per workgroup.
struct GemmRules {
  int K, cus;
  bool rows_splittable, one_tile;
  bool residual = false;                   // the launch has the residual epilogue (its cost only)
};

inline int cheapest_tiling(const GemmRules &r, long rows, long cols, bool ordered, double *cost) {
  int best = ordered ? kCfgStrip : kCfgWave;
  *cost = gemm_cost(best, rows, cols, r.K, r.residual);
  for (int cfg = 0; cfg < kCfgStrip; ++cfg) {
    if ((ordered && !in_k_order(cfg)) || (r.one_tile && !one_round(cfg, rows, cols, r.cus))) continue;
    const double c = gemm_cost(cfg, rows, cols, r.K, r.residual);
    if (c < *cost) { *cost = c; best = cfg; }
  }
  return best;
}

// Adds the launches of one part of the matrix; `ordered`: other launches share its columns.
inline void plan_gemm_part(const GemmRules &r, long row0, long rows, long col0, long cols, bool ordered, GemmPlan &out) {
  double best = 0.0;
  const int cfg = cheapest_tiling(r, rows, cols, ordered, &best);
  // Big tiles over the whole part but the rows or columns that would make a last, nearly empty round
  // (a partly filled last tile row or column, or the tile rows past a whole number of rounds): those
  // go to launches of their own with smaller tiles, if that saves at least 3 % and 4 us over the best
  // single launch.
  long best_dr = 0, best_dc = 0;
  const long tm = (rows + 255) / 256, tn = (cols + 255) / 256;
  if (!r.one_tile && tm * tn > 256 && out.n + 4 <= GemmPlan::kMax) {
    const long max_dr = r.rows_splittable ? (tm < 8 ? tm - 1 : 8) : 0, max_dc = (cols % 256 != 0 && tn > 1) ? 1 : 0;
    double split_best = best - (best * 0.03 > 4.0 ? best * 0.03 : 4.0);
    for (long dr = 0; dr <= max_dr; ++dr)
      for (long dc = 0; dc <= max_dc; ++dc) {
        if (!dr && !dc) continue;
        const long rm = dr ? (tm - dr) * 256 : rows, cm = dc ? (tn - dc) * 256 : cols;
        double right = 0.0, bottom = 0.0;
        if (dc) cheapest_tiling(r, rm, cols - cm, ordered || dr > 0, &right);      // right strip next to the main block
        if (dr) cheapest_tiling(r, rows - rm, cols, true, &bottom);                // bottom strip over the full width
        const double c = gemm_cost(kCfgBig, rm, cm, r.K, r.residual) + right + bottom;
        if (c < split_best - 1e-9) { split_best = c; best_dr = dr; best_dc = dc; }
      }
  }
  if (!best_dr && !best_dc) return out.add(row0, rows, col0, cols, cfg);
  const long rm = best_dr ? (tm - best_dr) * 256 : rows, cm = best_dc ? (tn - best_dc) * 256 : cols;
  out.add(row0, rm, col0, cm, kCfgBig);
  if (best_dc) plan_gemm_part(r, row0, rm, col0 + cm, cols - cm, ordered || best_dr > 0, out);
  if (best_dr) plan_gemm_part(r, row0 + rm, rows - rm, col0, cols, true, out);
}

inline GemmPlan plan_gemm(const GemmRules &r, long rows, long cols) {
  GemmPlan out;
  plan_gemm_part(r, 0, rows, 0, cols, false, out);
  return out;
}

}  // namespace et
