// What the kernels of the linear layers (linear.hip, linear_pipe.hip) share.
#pragma once
#include "linear_plan.h"
#include "pipe_ops.h"

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
  inline void set_divisors(int shape, bool partial);
};
constexpr int kGI = 8;  // tile rows per group in the order the tiles are handed out
inline void GemmArgs::set_divisors(int shape, bool partial) {
  const unsigned nI = (unsigned)((I + kTileI[shape] - 1) / kTileI[shape]), nJ = (unsigned)((J + kTileJ[shape] - 1) / kTileJ[shape]);
  by_set = Divisor::of(nI * nJ);
  by_group = Divisor::of(kGI * nJ);
  by_rest = Divisor::of(nI % kGI == 0 ? 1u : nI % kGI);
  by_splits = Divisor::of((unsigned)(partial ? splits : 1));
}

struct Quotient {
  unsigned q, r;
};
// n / d for n < 2^31, in scalar registers: the estimate from the reciprocal is at most one too small.
__device__ __forceinline__ Quotient divide(unsigned n, Divisor by) {
  Quotient o{__umulhi(n, by.m), 0u};
  o.r = n - o.q * by.d;
  if (o.r >= by.d) {
    o.r -= by.d;
    ++o.q;
  }
  return o;
}

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
constexpr unsigned kNowhere = 0x80000000u;  // a byte offset that every bounds check refuses

// One operand's contraction tile of 64 entries x N output rows (or columns).
//   row access: [N][64], 128 bytes a row; 16-byte chunk c of row s sits at position c ^ ((s >> 1) & 7) of its row
//   transposed: [64][N], 2 N bytes a row; 64-byte group g of row s sits at g ^ (s & 3), or g ^ ((s >> 1) & 1) where two rows
//     (N = 64) or two and a half groups (N = 192) make a turn of the banks
// Both fragment reads (16-byte reads of 16 consecutive rows, the transposing read of 4 rows x 64 bytes) then touch every
// bank once, without padding, and a wave-load fetches whole 128-byte lines.
template <bool TR, int N>
struct Operand {
  static constexpr int LOADS = N / 32;                     // wave-loads per wave and tile (four waves)
  static constexpr int NV = TR && N == 192 ? 3 : 1;        // different lane offsets among them
  static constexpr int ROWS_STEP = TR ? (N == 192 ? 32 : 2048 / N) : 32;  // rows from load x to load x + NV
  static constexpr int PITCH = TR ? 2 * N : 128;
  static constexpr int NB = N / 64;                        // blocks of 32 per wave (two waves side by side)
  static constexpr int NA = TR ? NB : 4;                   // read addresses: per block, or per contraction step
  unsigned voff[NV];
  unsigned half;                                           // row access: kNowhere for lanes of the tile's second half
  unsigned addr[NA];
  __device__ __forceinline__ static int group(int g, int s) { return N % 128 ? g ^ ((s >> 1) & 1) : g ^ (s & 3); }
  __device__ __forceinline__ void setup(unsigned lds, int w, int wave, int lane, unsigned pitch) {
    const int ic = lane & 31, hh = lane >> 5;
    half = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int pos = (wave + 4 * v) * 64 + lane;
      if (TR) {
        const int s = pos / (N / 8), c = pos - s * (N / 8);
        voff[v] = (unsigned)s * pitch + (unsigned)(group(c >> 2, s) * 4 + (c & 3)) * 16u;
      } else {
        const int s = pos >> 3, c = (pos & 7) ^ ((s >> 1) & 7);
        voff[v] = (unsigned)s * pitch + (unsigned)c * 16u;
        half = c >= 4 ? kNowhere : 0u;
      }
    }
#pragma unroll
    for (int n = 0; n < NA; ++n) {
      if (TR) {
        const int i = ic & 15, y = 2 * (ic >> 4) + ((i & 3) >> 1), r = 8 * hh + (i >> 2);
        addr[n] = lds + (unsigned)(r * PITCH + group(w * NB + n, r) * 64 + y * 16 + (i & 1) * 8);
      } else {
        addr[n] = lds + (unsigned)((w * NB * 32 + ic) * 128 + ((2 * n + hh) ^ ((ic >> 1) & 7)) * 16);
      }
    }
  }
  // fragment of block b, contraction step kk, of the tile `at` bytes behind the read addresses
  __device__ __forceinline__ bf16x8 frag(int b, int kk, unsigned at = 0) const {
    if (TR) return lds_read_tr(addr[b] + at, addr[b] + at + 4 * PITCH, kk * 16 * PITCH);
    return lds_read16(addr[kk] + at, b * 32 * 128);
  }
  __device__ __forceinline__ void move(unsigned by) {
#pragma unroll
    for (int n = 0; n < NA; ++n) addr[n] += by;
  }
};

// Bounds-checked asynchronous global->LDS load, 16 bytes per lane: lanes whose offset is not below the descriptor's size
// write zeros.  (The vector addition is also the wait state due between the scalar write of M0 and the load.)
__device__ __forceinline__ void load_lds(u32x4 srd, unsigned voff, unsigned add, unsigned lds, int imm) {
  unsigned t;
  asm volatile(
      "s_add_u32 m0, %1, %5\n\t"
      "v_add_u32 %0, %2, %3\n\t"
      "buffer_load_dwordx4 %0, %4, 0 offen lds"
      : "=&v"(t)
      : "s"(lds), "s"(add), "v"(voff), "s"(srd), "n"(imm)
      : "memory", "m0", "scc");
}
__device__ __forceinline__ u32x4 descriptor(unsigned long long base, unsigned bytes) {
  return u32x4{(unsigned)base, (unsigned)(base >> 32), bytes, 0x00027000u};
}

// The 256-row tile shapes (linear_pipe.hip); shape: k256 or k192.
hipError_t launch_gemm_fwd(int shape, const GemmArgs& g, hipStream_t st);
hipError_t launch_gemm_gx(int shape, const GemmArgs& g, hipStream_t st);
hipError_t launch_gemm_gw(int shape, const GemmArgs& g, hipStream_t st);

}  // namespace tvm
