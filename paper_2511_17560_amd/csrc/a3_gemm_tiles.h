// Which tile the GEMMs of a3_gemm_pp.h run in, and which tile a workgroup takes.  Integer and cost rules only, no device
// code: constexpr functions serve the kernels and the host alike, and compile with any C++17 compiler.
#pragma once

#include <cstddef>

// Workgroup -> (weight tile, activation tile).  The tiles are laid end to end in groups of gm weight tiles, a group's weight
// tiles fastest; consecutive workgroup ids go to different XCDs, and each XCD takes an eighth of that sequence in one piece
// (to within one tile), so that the 32 workgroups it runs at a time share about gm weight tiles and 32 / gm activation tiles
// through its L2, and no XCD has more than its share.  (Every eighth weight tile to an XCD, all its activation tiles with it,
// left 36 of 216 tiles to each of two XCDs, four more than it has CUs: 82 us for 1500 rows x 4608 x 3584 against 50.)
constexpr bool gemm_tile_of(int n_wt, int n_xt, int gm, int id, int &wt, int &xt) {
  const int xcd = id & 7, q = id >> 3, total = n_wt * n_xt, each = total >> 3, extra = total & 7;
  if (q >= each + (xcd < extra ? 1 : 0)) return false;
  const int t = xcd * each + (xcd < extra ? xcd : extra) + q;
  const int g = t / (gm * n_xt), r = t - g * (gm * n_xt), left = n_wt - g * gm, cnt = gm < left ? gm : left;
  xt = r / cnt;
  wt = g * gm + r - xt * cnt;
  return true;
}
constexpr unsigned gemm_tile_grid(int n_wt, int n_xt) { return 8u * (unsigned)(((long)n_wt * n_xt + 7) / 8); }

// Weight tiles per group of gemm_tile_of.  Where all tiles of an XCD run at once their order does not matter and groups of one
// leave the fewest weight tiles to two XCDs (200 rows x 3584 x 3584: 19.4 us, 20.6 in groups of four); otherwise an XCD's
// share of the weight tiles, at most 4.
constexpr int gemm_tile_group(int n_wt, int n_xt) { return n_wt * n_xt <= 256 ? 1 : n_wt <= 24 ? (n_wt + 7) / 8 : 4; }

// ---- choice of the tile --------------------------------------------------------------------------------
enum gemm_tile_id { GEMM_256x256, GEMM_256x192, GEMM_256x128, GEMM_128x192, GEMM_128x128, GEMM_128x64, GEMM_TILES };
// What a tile costs, measured with weights that come from HBM, 332 .. 16448 rows x 4096 .. 28672 weight rows: time of a
// 64-element slab while the chip is not at its power limit (one workgroup per CU), and the rate of products that the power
// limit leaves when it is (larger tiles move fewer bytes per product).  Start and end of a workgroup: about 8 us.  The slabs
// of 256x256 and 256x128 are what they take with two thirds to three quarters of the CUs busy, between the two (with 1.03 and
// 0.68, what they take with few busy, 256x256 was chosen for 1729 .. 1917 rows x 6144 x 4096: 92 us, 256x192 takes 76).
struct gemm_tile_cost { int bm, bn; double us_slab, pflops; };
constexpr gemm_tile_cost kGemmTileCost[GEMM_TILES] = {{256, 256, 1.20, 1.38}, {256, 192, 0.84, 1.28}, {256, 128, 0.74, 1.10},
                                                      {128, 192, 0.60, 1.00}, {128, 128, 0.50, 0.85}, {128, 64, 0.37, 0.65}};
struct gemm_tile_choice { int tile, splits; };
// tuning values "proj_ntw" and "gemm_tb": -1 (no choice made) or the tile they ask for
constexpr int gemm_tile_of_knob(int v) {
  constexpr int tile[] = {GEMM_256x128, GEMM_256x192, GEMM_256x256, GEMM_128x192, GEMM_128x128, GEMM_128x64};
  return v >= 2 && v <= 7 ? tile[v - 2] : -1;
}
// n_w weight rows, n_x activation rows, `slabs` slabs; up to max_splits ways to split the reduction (each costs a pass over
// the fp32 partial results at about 3 TB/s, write and read, and a launch).
constexpr gemm_tile_choice gemm_choose_tile(int n_w, int n_x, int slabs, int max_splits) {
  gemm_tile_choice best{GEMM_256x256, 1};
  double best_us = 1e30;
  for (int t = 0; t < GEMM_TILES; ++t)
    for (int sp = 1; sp <= max_splits && sp * 4 <= slabs + 3; sp *= 2) {
      const gemm_tile_cost &c = kGemmTileCost[t];
      const long wgs = (long)((n_w + c.bm - 1) / c.bm) * ((n_x + c.bn - 1) / c.bn) * sp;
      const int s = (slabs + sp - 1) / sp;
      const double round_us = 8. + s * c.us_slab, power_us = 2. * c.bm * c.bn * 64. * s * 256. / (c.pflops * 1e9);
      const double last_us = power_us * (wgs % 256) / 256.;
      double us = (double)(wgs / 256) * (round_us > power_us ? round_us : power_us);
      if (wgs % 256) us += round_us > last_us ? round_us : last_us;
      if (sp > 1) us += 4. + 8. * sp * n_w * (double)n_x / 3e6;
      if (us < best_us) { best_us = us; best.tile = t; best.splits = sp; }
    }
  return best;
}
