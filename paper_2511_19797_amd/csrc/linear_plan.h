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
// its steps and a fixed part (first operands, results), behind a start-up.  The weights are fits to times of all four shapes at
// 1177 forward shapes and 556 of grad x (whose second operand is read transposed: other weights), R = 64 ... 65536 rows, widths
// 32 ... 4608 either way: the choice is within 1 % of the 256 x 256 shape or faster at all but 9 of them (at most 4 %, one
// round's noise), and 0.1 % behind the fastest shape on average.  Some of them (us; 256 | 192 | 128 | 64):
//   forward, 256 x 4608 -> 1152:    102 |  98 |  51 |  31     few tiles: small ones fill the chip
//   forward, 1024 x 1536 -> 1152:    40 |  38 |  24 |  27
//   forward, 2048 x 768 -> 1536:     26 |  25 |  28 |  31     the small shapes' fixed part, round after round
//   forward, 2048 x 1152 -> 3456:    38 |  61 |  67 |  81     224 tiles of 256 are one round, 288 of 192 are two
//   forward, 16384 x 384 -> 1152:    46 |  48 |  79 | 102     short contraction: 192 has the larger fixed part
//   forward, 16384 x 4608 -> 1152:  395 | 384 | 455 | 636     long contraction, and 1152 = 6 x 192: no padded columns
//   forward, 16384 x 1152 -> 4608:  321 | 355 | 524 | 690
// The layers of a whole block with tangent, forward and backward (us, with 256 x 256 tiles alone / with this choice): B1 T256
// C1152 forward 232 / 198, B2 T250 C768 626 / 529 (both then bound by the host's calls), B32 T256 C1152 2727 / 2684, B16 T1024
// 5434 / 5359.
struct ShapeCost {
  int start, fixed, step;
};
constexpr ShapeCost kCostRow[kShapes] = {{4323, 4654, 1625}, {2820, 8013, 1356}, {1500, 5408, 693}, {865, 2359, 265}};
constexpr ShapeCost kCostTr[kShapes] = {{3060, 8558, 1427}, {2889, 8984, 1114}, {2938, 5155, 625}, {1628, 2537, 214}};
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
// grad W: time of `tiles` output tiles of shape c over `steps` contraction tiles each, in hundredths of a contraction tile of
// the 256 x 256 shape (1.5 us on an idle chip, 2 us on a full one).
inline long long dw_cost(int c, long long tiles, int steps) {
  constexpr int kStep[kShapes] = {100, 88, 45, 28}, kFixed[kShapes] = {150, 130, 70, 50};
  return (tiles + 255) / 256 * ((long long)steps * kStep[c] + kFixed[c]);
}
// Shape and number of contraction splits of grad W: what the partial tiles cost on top is two passes over them at
// 5 TB/s and a launch (3 us).  The 128 and 64 shapes write bf16 directly when there is one split.  Never more splits
// than dw_splits: the workspace is sized for those.
// (us of the whole backward, R 500 768 -> 768: 53 with 16 splits of 256 x 256 tiles, 35 with one of 64 x 64; R 16384
// 1152 -> 3456: 597 with 3 splits of 256 x 256, 581 with 3 of 256 x 192.  Against every shape but 64 and every number of splits,
// twelve layers of 384 ... 4608 and R = 2048 ... 65536: within 4 % of the fastest, never behind the 256 shape by more than 1.5 %.)
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
