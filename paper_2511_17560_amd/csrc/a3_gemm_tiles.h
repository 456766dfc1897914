// Which tile the GEMMs of a3_gemm_pp.h run in, and which tile a workgroup takes.  Integer and cost rules only, no device
// code: constexpr functions serve the kernels and the host alike, and compile with any C++17 compiler.
#pragma once

#include <cstddef>

// Workgroup -> (weight tile, activation tile).  The tiles are laid end to end in groups of gm weight tiles, a group's weight
// tiles fastest; consecutive workgroup ids go to different XCDs, and each XCD takes an eighth of that sequence in one piece,
// so that the 32 workgroups it runs at a time share about gm weight tiles and 32 / gm activation tiles through its L2, and no
// XCD has more than its share.  (Every eighth weight tile to an XCD, all its activation tiles with it, left 36 of 216 tiles to
// each of two XCDs, four more than it has CUs: 82 us for 1500 rows x 4608 x 3584 against 50.)  With few
// activation tiles, where the weights are most of what is read, the pieces are cut at whole weight tiles as long as the largest
// still runs at once: no weight is then read by two XCDs (273 rows x 4608 x 3584: 22.6 us cut anywhere, 21.7; but 1806 rows,
// ten activation tiles: 59 cut anywhere, 68).
constexpr int gemm_tile_unit(int n_wt, int n_xt) { return n_xt <= 5 && (n_wt + 7) / 8 * n_xt <= 32 ? n_xt : 1; }
// Weight tiles per group: the order of tiles that run at once does not matter and groups of one keep a weight tile's together;
// otherwise an XCD's share of the weight tiles, at most 4.
constexpr int gemm_tile_group(int n_wt, int n_xt) { return n_wt * n_xt <= 256 ? 1 : n_wt <= 24 ? (n_wt + 7) / 8 : 4; }
constexpr bool gemm_tile_of(int n_wt, int n_xt, int gm, int id, int &wt, int &xt) {
  const int unit = gemm_tile_unit(n_wt, n_xt), units = n_wt * n_xt / unit;
  const int xcd = id & 7, q = id >> 3, each = units >> 3, extra = units & 7;
  if (q >= (each + (xcd < extra ? 1 : 0)) * unit) return false;
  const int t = (xcd * each + (xcd < extra ? xcd : extra)) * unit + q;
  const int g = t / (gm * n_xt), r = t - g * (gm * n_xt), left = n_wt - g * gm, cnt = gm < left ? gm : left;
  xt = r / cnt;
  wt = g * gm + r - xt * cnt;
  return true;
}
constexpr unsigned gemm_tile_grid(int n_wt, int n_xt) {
  const int unit = gemm_tile_unit(n_wt, n_xt);
  return 8u * (unsigned)(((long)n_wt * n_xt / unit + 7) / 8 * unit);
}

// ---- choice of the tile --------------------------------------------------------------------------------
enum gemm_tile_id { GEMM_256x256, GEMM_256x192, GEMM_256x128, GEMM_128x192, GEMM_128x128, GEMM_128x64, GEMM_TILES };
// What a tile costs, measured with weights that come from HBM, 332 .. 16448 rows x 4096 .. 28672 weight rows: time of a
// 64-element slab while the chip is not at its power limit (one workgroup per CU), and the rate of products that the power
// limit leaves when it is (larger tiles move fewer bytes per product).  Start and end of a workgroup: about 8 us.  The slabs
// of 256x256 and 256x128 lie between what they take with few CUs busy (1.03, 0.68) and with three quarters of them (1.25,
// 0.74): with the former 256x256 was chosen for 1729 .. 1917 rows x 6144 x 4096, where it takes 92 us and 256x192 76; H(.)
// at 200 .. 5200 rows of 3584 and 4096 wide shapes is no slower at any, up to 10 % faster.
struct gemm_tile_cost { int bm, bn; double us_slab, pflops; };
constexpr gemm_tile_cost kGemmTileCost[GEMM_TILES] = {{256, 256, 1.135, 1.38}, {256, 192, 0.84, 1.28}, {256, 128, 0.74, 1.10},
                                                      {128, 192, 0.60, 1.00}, {128, 128, 0.50, 0.85}, {128, 64, 0.37, 0.65}};
struct gemm_tile_choice { int tile, splits; };
// tuning values "proj_ntw" and "gemm_tb": -1 (no choice made) or the tile they ask for
constexpr int gemm_tile_of_knob(int v) {
  constexpr int tile[] = {GEMM_256x128, GEMM_256x192, GEMM_256x256, GEMM_128x192, GEMM_128x128, GEMM_128x64};
  return v >= 2 && v <= 7 ? tile[v - 2] : -1;
}
// n_w weight rows, n_x activation rows, `slabs` slabs; up to max_splits ways to split the reduction (each costs a pass over
// the fp32 partial results at about 3 TB/s, write and read, and a launch); tiles `first` and smaller.
constexpr gemm_tile_choice gemm_choose_tile(int n_w, int n_x, int slabs, int max_splits, int first = GEMM_256x256) {
  gemm_tile_choice best{first, 1};
  double best_us = 1e30;
  for (int t = first; t < GEMM_TILES; ++t)
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
