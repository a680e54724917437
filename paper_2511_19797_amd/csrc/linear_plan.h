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

// Time of `tiles` output tiles of shape c over `steps` contraction tiles each, in units of a hundredth of a contraction
// tile of the 256 x 256 shape (1.5 us on an idle chip, 2 us on a full one): rounds of workgroups over the chip's 256
// CUs times steps and a fixed part.  The weights are fits to measured times, R = 64 ... 16384 rows, widths 384, 768,
// 1152 and their multiples by 3 and 4: they put the fastest shape first, or one within 3 % of it.  Some of both sides
// (us; 256 | 192 | 128 | 64):
//   forward, 256 x 4608 -> 1152:    104 |  99 |  52 |  32     few tiles: small ones fill the chip
//   forward, 1024 x 4608 -> 1152:   101 |  94 |  53 |  60
//   forward, 2048 x 1152 -> 3456:    40 |  58 |  63 |  75     224 tiles of 256 are one round, 288 of 192 are two
//   forward, 16384 x 4608 -> 1152:  395 | 384 | 455 | 636     1152 = 6 x 192: no padded columns
//   forward, 16384 x 1152 -> 4608:  321 | 355 | 524 | 690
// The layers of a whole block with tangent, forward and backward (us, before / with this choice): B1 T256 C1152 forward 232 /
// 198, B2 T250 C768 626 / 529 (both then bound by the host's calls), B32 T256 C1152 2727 / 2684, B16 T1024 5434 / 5359.
inline long long tile_cost(int c, long long tiles, int steps) {
  constexpr int kStep[kShapes] = {100, 88, 45, 28}, kFixed[kShapes] = {150, 130, 70, 50}, kSlots[kShapes] = {256, 256, 256, 512};
  return (tiles + kSlots[c] - 1) / kSlots[c] * ((long long)steps * kStep[c] + kFixed[c]);
}
inline int pick_shape(int sets, int I, int J, int C) {
  int best = k256;
  for (int c = k192; c < kShapes; ++c) {
    const int steps = (C + kBK - 1) / kBK;
    if (grid_fits(c, sets * tiles_of(c, I, J)) &&
        tile_cost(c, sets * tiles_of(c, I, J), steps) < tile_cost(best, sets * tiles_of(best, I, J), steps))
      best = c;
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
// Shape and number of contraction splits of grad W: what the partial tiles cost on top is two passes over them at
// 5 TB/s and a launch (3 us).  The 128 and 64 shapes write bf16 directly when there is one split.  Never more splits
// than dw_splits: the workspace is sized for those.
// (us of the whole backward, R 500 768 -> 768: 53 with 16 splits of 256 x 256 tiles, 35 with one of 64 x 64; R 16384
// 1152 -> 3456: 597 with 3 splits of 256 x 256, 581 with 3 of 256 x 192.)
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
      // (grad W's 64 x 64 tiles fit one workgroup per CU: half as many at once)
      long long cost = tile_cost(c, c == k64 ? 2 * tiles : tiles, (ntot + s - 1) / s);
      if (s > 1 || c < k128) cost += 180 + (long long)s * F * K / 10000;  // 8 bytes per partial sum, 60 units per us
      if (best_cost < 0 || cost < best_cost) {
        best_cost = cost;
        best = DwPlan{c, s};
      }
    }
  return best;
}

}  // namespace tvm
