// Which tile shape serves a product of the linear layers (linear.hip), and how grad W's contraction is split.
// Host code only.
#pragma once

namespace tvm {

constexpr int kBK = 64;  // contraction per LDS tile

enum { k256, k192, k128, k64, kShapes };
constexpr int kTileI[kShapes] = {256, 256, 128, 64};  // output rows
constexpr int kTileJ[kShapes] = {256, 192, 128, 64};  // output columns
inline long long tiles_of(int c, int I, int J) {
  return ((long long)I + kTileI[c] - 1) / kTileI[c] * (((long long)J + kTileJ[c] - 1) / kTileJ[c]);
}
// The 128 and 64 shapes take a workgroup per tile (a multiple of 8 of them), and a launch is limited to 2^32 - 1 threads; the
// 256-row shapes are persistent, 256 workgroups at most.  (64 x 64 tiles of 2^29 rows and 32 columns, two row sets, are 2^24
// workgroups: one too many.)
constexpr int kSmallThreads = 256;
inline long long small_workgroups(long long tiles) { return 8 * ((tiles + 7) / 8); }
inline bool grid_fits(int c, long long tiles) { return c < k128 || small_workgroups(tiles) * kSmallThreads < (1ll << 32); }

// Time of a product (ns): `tiles` output tiles of shape c over `steps` contraction tiles each are rounds of 256 workgroups, each
// its steps and a fixed part (first operands, results), behind a start-up.  The weights are fits to kernel times of all four
// shapes, R = 40 ... 65536 rows, widths 32 ... 4608 either way (so weights only: the choice matters, not the time): 1144 products
// of the forward, where the choice is 0.03 % behind the fastest shape on average and 4.8 % at most; grad x (whose second operand
// is read transposed: other weights) costs a whole backward 0.01 % on average of 551 products, 1.1 % at most.
// Some of the times, back to back (us; 256 | 192 | 128 | 64):
//   forward, 500 x 768 -> 768:       17 |  14 |  10 | 5.6     few tiles: small ones fill the chip
//   forward, 1024 x 1152 -> 1152:    24 |  20 |  14 |  14
//   forward, 2048 x 768 -> 3072:     23 |  21 |  31 |  38     the small shapes' fixed part, round after round
//   forward, 8192 x 64 -> 1152:      15 |  13 |  21 |  23     short contraction: first operands and stores
//   forward, 5000 x 96 -> 1312:      12 |  14 |  19 |  20     ... where 192 columns need one round more
//   forward, 16384 x 768 -> 3072:   126 | 130 | 244 | 295
//   forward, 8192 x 4608 -> 1152:   182 | 149 | 211 | 247     long contraction, and 1152 = 6 x 192: no padded columns
struct ShapeCost {
  int start, fixed, step;
};
constexpr ShapeCost kCostRow[kShapes] = {{2231, 7416, 929}, {638, 5645, 750}, {0, 4184, 482}, {622, 1455, 173}};
constexpr ShapeCost kCostTr[kShapes] = {{3632, 13659, 1047}, {806, 10481, 823}, {3535, 4645, 458}, {3090, 2010, 162}};
inline long long product_ns(const ShapeCost& c, long long tiles, int steps) {
  return c.start + (tiles + 255) / 256 * (c.fixed + (long long)steps * c.step);
}
// Shape of the forward (qtr false: `sets` x [I][J] with the second operand's rows along the contraction) or of grad x (qtr true).
// Every shape adds an output element's products in the same order: the choice does not show in the results.
inline int pick_shape(bool qtr, int sets, int I, int J, int C) {
  const ShapeCost* const cost = qtr ? kCostTr : kCostRow;
  const int steps = (int)(((long long)C + kBK - 1) / kBK);
  int best = k256;
  long long best_ns = product_ns(cost[k256], sets * tiles_of(k256, I, J), steps);
  for (int c = k192; c < kShapes; ++c) {
    const long long tiles = sets * tiles_of(c, I, J), ns = product_ns(cost[c], tiles, steps);
    if (ns < best_ns && grid_fits(c, tiles)) {
      best = c;
      best_ns = ns;
    }
  }
  return best;
}
inline int dw_splits(int F, int K, int R) {
  const int tiles = ((F + kTileI[k256] - 1) / kTileI[k256]) * ((K + kTileJ[k256] - 1) / kTileJ[k256]);
  const int ntot = 2 * ((R + kBK - 1) / kBK);
  // (the most splits any tile shape uses, and what the workspace is sized for)
  // The fewest rounds of workgroups over the chip's 256 CUs (one workgroup each), each round costing its share of
  // the contraction plus a fixed part (start-up, the float32 partial tile); ties go to fewer splits.
  int best = 1;
  long long best_cost = -1;
  for (int s = 1; s <= 32 && s <= ntot; ++s) {
    const long long rounds = ((long long)s * tiles + 255) / 256;
    const long long cost = rounds * ((ntot + s - 1) / s + 64);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = s;
    }
  }
  return best;
}
// grad W: time of `tiles` output tiles of shape c over `steps` contraction tiles each, in units of 1/60 us (weights of a fit: a
// contraction tile of 256 x 256 counts 1.8 us; it takes 1.2 us on an idle chip and 1.6 on a full one).
inline long long dw_cost(int c, long long tiles, int steps) {
  constexpr int kStep[kShapes] = {108, 86, 46, 27}, kFixed[kShapes] = {49, 87, 58, 54};
  return (tiles + 255) / 256 * ((long long)steps * kStep[c] + kFixed[c]);
}
// Shape and number of contraction splits of grad W: what the partial tiles cost on top is two passes over them at
// 5 TB/s and a launch (3 us).  The 128 and 64 shapes write bf16 directly when there is one split.  Never more splits
// than dw_splits: the workspace is sized for those.
// (us of grad W alone, 256 | 192 | 128 | 64: R 500 768 -> 768 19 | 17 | 16 | 7; R 4096 768 -> 3072 53 | 48 | 62 | 71; R 16384
// 1152 -> 3456 252 | 220 | 292 | 503.  At 189 layers of 288 ... 4608 and R = 64 ... 16384 the choice is 5 % behind the fastest
// shape on average: it is late to turn to 64 x 64, by up to 5 us, as rounds of 256 are counted for a shape that runs two
// workgroups per CU.)
struct DwPlan {
  int shape, splits;
};
inline DwPlan plan_dw(int F, int K, int R, int max_splits) {
  const int ntot = 2 * ((R + kBK - 1) / kBK);
  DwPlan best{k256, max_splits};
  long long best_cost = -1;
  for (int c = 0; c < kShapes; ++c)
    for (int s = 1; s <= max_splits; ++s) {
      const long long tiles = s * tiles_of(c, F, K);
      if (!grid_fits(c, tiles)) continue;
      long long cost = dw_cost(c, tiles, (ntot + s - 1) / s);
      if (s > 1 || c < k128) cost += 180 + (long long)s * F * K / 10000;  // 8 bytes per partial sum, 60 units per us
      if (best_cost < 0 || cost < best_cost) {
        best_cost = cost;
        best = DwPlan{c, s};
      }
    }
  return best;
}

}  // namespace tvm
