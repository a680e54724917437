// What the kernels of the linear layers (linear.hip, linear_pipe.hip) share.
#pragma once
#include "linear_plan.h"
#include "mfma_tiles.h"

namespace tvm {

struct Divisor {
  unsigned d, m;  // m = floor((2^32 - 1) / d)
  static Divisor of(unsigned d) { return Divisor{d, 0xffffffffu / d}; }
};

// OUT[i][j] = sum_c P[i][c] Q[j][c]
struct GemmArgs {
  const bf16* P[2];   // two row sets (forward, grad x) or two contraction sets (grad W)
  const bf16* Q[2];
  long long ldP, ldQ; // row pitch in elements of the matrices as stored
  int I, J, C;        // output rows, output columns, contraction length per set
  int csets;          // contraction sets (1, or 2 for grad W)
  bf16* out[2];       // one per row set (forward, grad x); row pitch ldo
  long long ldo;
  const bf16* bias;   // added to out[0] only (the tangent has no bias), may be null
  float* part;        // grad W: float32 partial tiles [splits][I][J]
  int splits;
  int nz;             // row sets (forward, grad x: 2) or splits (grad W)
  Divisor by_set, by_group, by_rest, by_splits;  // tiles of a row set, of a group of tile rows, tile rows of the last group
};
constexpr int kGI = 8;  // tile rows per group in the order the tiles are handed out

// The 256-row tile shapes (linear_pipe.hip); shape: k256 or k192.
hipError_t launch_gemm_fwd(int shape, const GemmArgs& g, hipStream_t st);
hipError_t launch_gemm_gx(int shape, const GemmArgs& g, hipStream_t st);
hipError_t launch_gemm_gw(int shape, const GemmArgs& g, hipStream_t st);

}  // namespace tvm
