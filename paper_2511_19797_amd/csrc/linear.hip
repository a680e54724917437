// Linear layers of the block on the bf16 matrix cores (gfx950): a token's features and their tangent through
// y = W x + b, ty = W tx (the weights carry no tangent: the network's JVP runs along its inputs), and the backward
// gx = W^T gy, gtx = W^T gty, gW = sum over tokens (gy x^T + gty tx^T), gb = sum over tokens gy.
//
// One kernel serves the three products.  It computes  OUT[i][j] = sum_c P[i][c] Q[j][c]  with either operand stored
// with its contraction index along the rows of a row-major matrix ("row" access: [i][c]) or along the columns'
// direction, i.e. as [c][i] ("transposed" access):
//     forward   OUT = y  [token][f]:  P = x  [token][k] row,         Q = W [f][k] row          (c = k)
//     grad x    OUT = gx [token][k]:  P = gy [token][f] row,         Q = W [f][k] transposed   (c = f)
//     grad W    OUT = gW [f][k]:      P = gy [token][f] transposed,  Q = x [token][k] transposed (c = token)
// The forward and grad x run once over the stacked rows [x; tx] (two row sets, one launch); grad W contracts over
// both sets.  Everything is computed transposed, D = Q-fragment x P-fragment, so that a lane owns one output ROW
// (32 per 32x32 block) and 16 of its columns: results leave through LDS as whole rows (store_tile_coalesced).
//
// Four tile shapes (chosen by pick_shape and plan_dw, linear_plan.h): 256 x 256 and 256 x 192 in linear_pipe.hip, 128 x 128 and
// 64 x 64 here (gemm_small_kernel).
//
// grad W contracts over all tokens of both sets (32K rows at DiT-XL/2 512 px) for few output tiles, so the token
// range is split over several workgroups per tile; each leaves a float32 partial tile in the workspace and a second
// small kernel adds them in a fixed order (no atomics) and rounds once.  gb is a column sum of gy: partial sums over
// row ranges, then one kernel that adds those.
#include <type_traits>

#include "linear_gemm.h"

namespace tvm {
namespace {

// All waves of the workgroup.  (Not __syncthreads, which waits for every load in flight.)
__device__ __forceinline__ void barrier() { asm volatile("s_barrier" ::: "memory"); }

// float32 partial tile of one wave (kWI x kWJ blocks from row i, column jw of split zz): lane = output row, four
// consecutive columns per register group.
template <int kWI, int kWJ>
__device__ __forceinline__ void store_partial(const GemmArgs& g, const f32x16 (&acc)[kWI][kWJ], int zz, int i_first, int jw,
                                              int ic, int hh) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  float* dst = g.part + (long long)zz * g.I * g.J;
#pragma unroll
  for (int a = 0; a < kWI; ++a) {
    const int i = i_first + a * 32 + ic;
    if (i >= g.I) continue;
#pragma unroll
    for (int b = 0; b < kWJ; ++b)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int j = jw + b * 32 + 8 * q4 + 4 * hh;
        if (j < g.J) {  // (J is a multiple of 8: four columns are in range together)
          const f32x4 v = {acc[a][b][4 * q4], acc[a][b][4 * q4 + 1], acc[a][b][4 * q4 + 2], acc[a][b][4 * q4 + 3]};
          *reinterpret_cast<f32x4*>(dst + (long long)i * g.J + j) = v;
        }
      }
  }
}

// The products for shapes with few 256-row tiles: workgroups of four waves on 64 x 64 or 128 x 128 output tiles (N), one tile
// each.  What bounds a contraction tile of 64 is LDS: at N = 64 32 KB of fragment reads and 16 KB that land there, 384 cycles at
// 128 bytes a cycle, next to 128 cycles of products per wave (N = 128: 96 KB, 768 and 512).  So a wave reads the fragments of
// the next tile between the products of this one, the loads run NST - 2 tiles ahead, in the loop counted rather than drained (at the
// start the compiler, which sees the bias load and not the assembly's, waits for all first stages in front of the bias product, with
// or without a bias; split grad W has no such wait), and their descriptors move by additions: a tile takes 430 cycles (900), against 740 (1500) with reads, then products, and descriptors
// worked out anew for every tile.  us before / now: forward 256 x 1152 -> 1152 9.6 / 7.5, 256 x 4608 -> 1152 26.8 / 18.2, 500 x 3072
// -> 768 19.1 / 13.6, 500 x 1152 -> 3456 (128) 17.8 / 15.0; grad x 256 x 1152 -> 4608 28.2 / 17.4; grad W 500 x 768 -> 3072 (128) 16.2 / 13.6.
// Operand tiles as in linear_pipe.hip (Operand: whole cache lines, no padding, zeros beyond the edges).  Contraction tiles are
// taken in the same order and every output element is the same chain of products as there: results are bit for bit the same
// (with equal splits).
template <bool PTR, bool QTR, bool PARTIAL, int N, int NST, int OCC>
__global__ __launch_bounds__(kSmallThreads, OCC) void gemm_small_kernel(GemmArgs g) {
  constexpr int W = N / 64;                              // blocks of 32 x 32 per wave, either way
  using OP = Operand<PTR, N>;
  using OQ = Operand<QTR, N>;
  constexpr unsigned HALF = N * 128u, BUF = 2 * HALF;    // a stage: P tile, Q tile
  constexpr int LOADS = OP::LOADS + OQ::LOADS;           // wave-loads per wave and tile
  constexpr unsigned OUT_REGION = 32 * (64 * W + 16);    // per wave, for store_tile_coalesced
  static_assert(NST >= 4 && (NST - 2) * LOADS < 64 && 4 * OUT_REGION <= NST * BUF && NST * BUF * OCC <= 160 * 1024, "stages");
  __shared__ __attribute__((aligned(1024))) char lds[NST * BUF];
  const int nI = (g.I + N - 1) / N, nJ = (g.J + N - 1) / N, total = g.nz * nI * nJ;
  // XCD x owns the x-th eighth of the tile list (as in linear_pipe.hip: groups of kGI tile rows, down the group first)
  const int wg = (int)(blockIdx.x & 7) * ((total + 7) >> 3) + (int)(blockIdx.x >> 3);
  if (wg >= min(total, ((int)(blockIdx.x & 7) + 1) * ((total + 7) >> 3))) return;
  const int lane = threadIdx.x & 63, ic = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wi = wave & 1, wj = wave >> 1;
  const Quotient zq = divide((unsigned)wg, g.by_set), grp = divide(zq.r, g.by_group);
  const int zz = (int)zq.q, it_first = (int)grp.q * kGI;
  const Quotient jt = nI - it_first >= kGI ? Quotient{grp.r / kGI, grp.r % kGI} : divide(grp.r, g.by_rest);
  const int i0 = (it_first + (int)jt.r) * N, j0 = (int)jt.q * N;
  const int nct = (g.C + kBK - 1) / kBK, ntot = g.csets * nct;
  const int t_begin = PARTIAL ? (int)divide((unsigned)zz * (unsigned)ntot, g.by_splits).q : 0;  // splits <= 32, ntot <= 2^26
  const int t_end = PARTIAL ? (int)divide((unsigned)(zz + 1) * (unsigned)ntot, g.by_splits).q : ntot;
  const bool two = g.csets == 2;  // grad W: contraction over both row sets
  const int clast = g.C - (nct - 1) * kBK;
  const unsigned pitchP = (unsigned)(g.ldP * 2), pitchQ = (unsigned)(g.ldQ * 2);
  const int validP = min(g.I - i0, N), validQ = min(g.J - j0, N);
  const unsigned lds0 = lds_addr_of(lds);
  OP op;
  OQ oq;
  op.setup(lds0, wi, wave, lane, pitchP);
  oq.setup(lds0 + HALF, wj, wave, lane, pitchQ);
  // accumulators start from bias x 1 as one more product, exactly the bias (row set 0 only): block b's column 32 b + ic
  f32x16 acc[W][W];
  unsigned bias_bits[W];
  {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16*>(g.bias), 0, !PARTIAL && g.bias != nullptr && zz == 0 ? g.J * 2 : 0, 0x00027000);
#pragma unroll
    for (int b = 0; b < W; ++b) {
      const unsigned off = (unsigned)(j0 + (wj * W + b) * 32 + ic) * 2u;
      bias_bits[b] = PARTIAL ? 0u : (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)(hh == 0 ? off : kNowhere), 0, 0);
    }
  }
  // The loads' cursor: descriptors (first byte, size for the bounds check) and lane offsets of contraction tile c_t.  Within a
  // set a move is three additions per operand; c_plain counts the moves left until something else is due.
  u32x4 sp, sq;
  unsigned vp = op.voff[0], vq = oq.voff[0];
  int c_t, c_plain = 0;
  auto place = [&](int t) {
    c_t = t;
    const int set = two && t >= nct ? 1 : 0, ct = t - set * nct;
    const long long c0 = (long long)ct * kBK;
    const bool last = ct == nct - 1;
    const bf16 *p = g.P[two ? set : PARTIAL ? 0 : zz], *q = g.Q[set];
    const unsigned rows = (unsigned)((last ? clast : kBK) - 1);
    if (PTR) sp = descriptor((unsigned long long)(uintptr_t)(p + c0 * g.ldP + i0), rows * pitchP + (unsigned)validP * 2u);
    else sp = descriptor((unsigned long long)(uintptr_t)(p + (long long)i0 * g.ldP + c0), (unsigned)(validP - 1) * pitchP + (unsigned)(g.C - (int)c0) * 2u);
    if (QTR) sq = descriptor((unsigned long long)(uintptr_t)(q + c0 * g.ldQ + j0), rows * pitchQ + (unsigned)validQ * 2u);
    else sq = descriptor((unsigned long long)(uintptr_t)(q + (long long)j0 * g.ldQ + c0), (unsigned)(validQ - 1) * pitchQ + (unsigned)(g.C - (int)c0) * 2u);
    const unsigned cut = last && clast <= 32 ? kNowhere : 0u;  // row access: the second half of a set's last tile is absent
    if (!PTR) vp = op.voff[0] | (op.half & cut);
    if (!QTR) vq = oq.voff[0] | (oq.half & cut);
    if (t >= t_end) sp[2] = sq[2] = 0;  // beyond the end: loads that fetch nothing, so that the count of loads in flight stays the same
    // plain moves: up to the tile before the set's last one, and before the end
    c_plain = min(nct - 2 - ct, t_end - 1 - t);
  };
  auto move = [&]() {
    if (c_plain > 0) {
      --c_plain;
      ++c_t;
      sp = descriptor(((unsigned long long)sp[1] << 32 | sp[0]) + (PTR ? 64ull * pitchP : 128ull), PTR ? sp[2] : sp[2] - 128u);
      sq = descriptor(((unsigned long long)sq[1] << 32 | sq[0]) + (QTR ? 64ull * pitchQ : 128ull), QTR ? sq[2] : sq[2] - 128u);
    } else if (c_t < t_end) {
      place(c_t + 1);
    }
  };
  // wave-load x of the cursor's tile into the stage at `to`
  auto issue = [&](unsigned to, int x) __attribute__((always_inline)) {
    const unsigned l = lds0 + to + (unsigned)wave * 1024u;
    if (x < OP::LOADS) load_lds(sp, vp, (unsigned)(x * OP::ROWS_STEP) * pitchP, l, x * 4096);
    else load_lds(sq, vq, (unsigned)((x - OP::LOADS) * OQ::ROWS_STEP) * pitchQ, l, (int)HALF + (x - OP::LOADS) * 4096);
  };
  bf16x8 pf[2][kBK / 16][W], qf[2][kBK / 16][W];
  auto fetch = [&](int set, int kk, unsigned at) {
#pragma unroll
    for (int a = 0; a < W; ++a) pf[set][kk][a] = op.frag(a, kk, at);
#pragma unroll
    for (int b = 0; b < W; ++b) qf[set][kk][b] = oq.frag(b, kk, at);
  };
  place(t_begin);
  for (unsigned x = 0; x < NST - 1; ++x) {
#pragma unroll
    for (int y = 0; y < LOADS; ++y) issue(x * BUF, y);
    move();
  }
  {
    const bf16x8 one = __builtin_bit_cast(bf16x8, u32x4{hh == 0 ? 0x3f80u : 0u, 0u, 0u, 0u});
#pragma unroll
    for (int b = 0; b < W; ++b) {
      const bf16x8 bv = __builtin_bit_cast(bf16x8, u32x4{bias_bits[b], 0u, 0u, 0u});
#pragma unroll
      for (int a = 0; a < W; ++a) acc[a][b] = mfma(bv, one, zero16());
    }
  }
  dma_wait_keep<(NST - 2) * LOADS>();
  barrier();
#pragma unroll
  for (int kk = 0; kk < kBK / 16; ++kk) fetch(0, kk, 0);
  unsigned at = 0;  // tile t's stage
  auto turn = [&](int t, int set) {
    const unsigned next = at + BUF == NST * BUF ? 0 : at + BUF, before = at == 0 ? (NST - 1) * BUF : at - BUF;
    dma_wait_keep<(NST - 3) * LOADS>();
    barrier();  // tile t + 1 is there for everyone, and everyone has tile t - 1 in registers: its stage is refilled now
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      fetch(set ^ 1, kk, next);
#pragma unroll
      for (int x = kk * LOADS / 4; x < (kk + 1) * LOADS / 4; ++x) issue(before, x);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b) acc[a][b] = mfma(qf[set][kk][b], pf[set][kk][a], acc[a][b]);
      __builtin_amdgcn_sched_barrier(0);
    }
    move();
    at = next;
  };
  for (int t = t_begin; t < t_end; t += 2) {
    turn(t, 0);
    if (t + 1 < t_end) turn(t + 1, 1);
  }
  const int jw = j0 + wj * (W * 32);
  if (PARTIAL) {
    store_partial<W, W>(g, acc, zz, i0 + wi * W * 32, jw, ic, hh);
    dma_wait();  // (no load may land in LDS that the next workgroup owns)
    return;
  }
  dma_wait();  // the loads past the end land in stages that the results are about to go through
  __syncthreads();
  if (jw < g.J) {
    const unsigned lw = lds0 + (unsigned)wave * OUT_REGION;
#pragma unroll
    for (int a = 0; a < W; ++a)
      store_tile_coalesced<W>(lw, g.out[zz] + jw, g.ldo, i0 + (wi * W + a) * 32, g.I, g.J - jw, acc[a], 1.f, lane);
  }
}

// Adds `splits` float32 partial matrices of n elements in order and rounds once to bf16.  8 elements per thread.
__global__ __launch_bounds__(256) void sum_partials_kernel(const float* __restrict__ part, int splits, long long n,
                                                           bf16* __restrict__ out) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  const long long e = ((long long)blockIdx.x * 256 + threadIdx.x) * 8;
  if (e >= n) return;
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
  for (int s = 0; s < splits; ++s) {
    const f32x4* p = reinterpret_cast<const f32x4*>(part + (long long)s * n + e);
    s0 += p[0];
    s1 += p[1];
  }
  bf16x8 o;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    o[t] = (bf16)s0[t];
    o[4 + t] = (bf16)s1[t];
  }
  *reinterpret_cast<bf16x8*>(out + e) = o;
}

// Column sums of gy [R][F] over `chunks` row ranges: part[chunk][f] (float32).  A lane takes 8 columns (16-byte
// loads, a wave 512 columns of a row), the four waves of a workgroup every fourth row of the chunk each; their sums
// meet in LDS, in a fixed order.
__global__ __launch_bounds__(256) void colsum_kernel(const bf16* __restrict__ gy, int R, int F, long long ld, int chunks,
                                                     float* __restrict__ part) {
  __shared__ float red[4][64][8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ch = blockIdx.y;
  const int f = (blockIdx.x * 64 + lane) * 8;  // (F is a multiple of 8: eight columns are in range together)
  const int r0 = (int)((long long)ch * R / chunks), r1 = (int)((long long)(ch + 1) * R / chunks);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (f < F) {
    const bf16* col = gy + f;
    int r = r0 + wave;
    for (; r + 12 < r1; r += 16) {  // four rows in flight
      bf16x8 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const bf16x8*>(col + (long long)(r + 4 * u) * ld);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += (float)v[u][e];
    }
    for (; r < r1; r += 4) {
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(col + (long long)r * ld);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += (float)v[e];
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[wave][lane][e] = acc[e];
  __syncthreads();
  if (wave == 0 && f < F) {
#pragma unroll
    for (int e = 0; e < 8; ++e) part[(long long)ch * F + f + e] = (red[0][lane][e] + red[1][lane][e]) + (red[2][lane][e] + red[3][lane][e]);
  }
}

// Adds the `chunks` partial rows of the column sums, part[chunk][f], and rounds once to bf16.  A workgroup of 16
// waves takes 64 columns: wave w adds rows w, w + 16, ... (16 loads in flight), and the 16 sums meet in LDS, in a
// fixed order.  (Few output elements and many rows: with a thread per column walking all rows in turn, one or two
// workgroups spent 70 us on 256 rows of dependent latencies.)
__global__ __launch_bounds__(1024) void bias_sum_kernel(const float* __restrict__ part, int chunks, int F,
                                                        bf16* __restrict__ out) {
  __shared__ float red[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int f = blockIdx.x * 64 + lane;
  float acc = 0.f;
  if (f < F) {
    for (int c0 = wave; c0 < chunks; c0 += 256) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int c = c0 + 16 * u;
        v[u] = c < chunks ? part[(long long)c * F + f] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) acc += v[u];
    }
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && f < F) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += red[w][lane];
    out[f] = (bf16)t;
  }
}

// Both of these in one launch, for few rows: workgroup = 64 columns (8 lanes of 16 bytes per row), 128 rows at a time;
// a wave's eight rows meet by lane exchanges, the sixteen waves in LDS, in a fixed order.  Bound by its launch and one
// memory latency or two: 500 x 768 ... 3072 in 4 us, against 4.6 + 3 ... 4 us and a
// launch more.
__global__ __launch_bounds__(1024) void colsum_direct_kernel(const bf16* __restrict__ gy, int R, int F, long long ld,
                                                             bf16* __restrict__ out) {
  __shared__ float red[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int f = blockIdx.x * 64 + (lane & 7) * 8;  // (F is a multiple of 8: eight columns are in range together)
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (f < F) {
    const bf16* col = gy + f;
    int r = threadIdx.x >> 3;
    for (; r + 384 < R; r += 512) {  // four rows in flight
      bf16x8 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const bf16x8*>(col + (long long)(r + 128 * u) * ld);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += (float)v[u][e];
    }
    for (; r < R; r += 128) {
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(col + (long long)r * ld);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += (float)v[e];
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    acc[e] += __shfl_xor(acc[e], 8);
    acc[e] += __shfl_xor(acc[e], 16);
    acc[e] += __shfl_xor(acc[e], 32);
  }
  if (lane < 8)
#pragma unroll
    for (int e = 0; e < 8; ++e) red[wave][lane * 8 + e] = acc[e];
  __syncthreads();
  const int c = blockIdx.x * 64 + threadIdx.x;
  if (threadIdx.x < 64 && c < F) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += red[w][threadIdx.x];
    out[c] = (bf16)t;
  }
}
constexpr int kDirectRows = 2048;  // up to this many rows the column sums take one launch

static_assert(kTileI[k128] == 128 && kTileJ[k128] == 128 && kTileI[k64] == 64 && kTileJ[k64] == 64 && kBK == 64, "the plan's tiles");

int bias_chunks(int R) {
  const int c = (R + 63) / 64;
  return c > 256 ? 256 : c;
}

// Launches a product with tile shape c (128 or 64).  Stages: more of them (10 at 64 x 64 with one workgroup per CU, 5 at 128 x 128)
// gain nothing, the loads are there in time, and cost 0.5 - 1 us of start-up; 4 at 64 x 64 lose 10 % on long contractions.
template <bool PTR, bool QTR, bool PARTIAL>
hipError_t launch_small(int c, GemmArgs g, hipStream_t st) {
  const dim3 grid((unsigned)small_workgroups(g.nz * tiles_of(c, g.I, g.J))), block(kSmallThreads);
  g.set_divisors(c, PARTIAL);
  if (c == k128) hipLaunchKernelGGL((gemm_small_kernel<PTR, QTR, PARTIAL, 128, 4, 1>), grid, block, 0, st, g);
  else hipLaunchKernelGGL((gemm_small_kernel<PTR, QTR, PARTIAL, 64, 5, 2>), grid, block, 0, st, g);
  return hipGetLastError();
}

}  // namespace

// Row pitches (elements) up to 2^20: a tile's per-lane byte offsets (row within the tile x pitch) stay inside 32 bits.
bool linear_supported(int R, int K, int F, long long ldx, long long ldy, int dtype) {
  return dtype == 1 && R >= 1 && K >= 32 && F >= 32 && K % 32 == 0 && F % 32 == 0 && ldx >= K && ldy >= F &&
         ldx % 8 == 0 && ldy % 8 == 0 && ldx <= (1ll << 20) && ldy <= (1ll << 20) && K <= (1 << 20) && F <= (1 << 20);
}

size_t linear_bwd_workspace_bytes(int R, int K, int F) {
  const size_t dw = (size_t)dw_splits(F, K, R) * F * K * sizeof(float);
  const size_t db = (size_t)bias_chunks(R) * F * sizeof(float);
  return ((dw + 255) & ~(size_t)255) + ((db + 255) & ~(size_t)255);
}

hipError_t launch_linear_fwd(int R, int K, int F, long long ldx, long long ldy, const void* x, const void* tx,
                             const void* w, const void* bias, void* y, void* ty, hipStream_t st) {
  GemmArgs g{};
  g.P[0] = (const bf16*)x;
  g.P[1] = (const bf16*)tx;
  g.Q[0] = g.Q[1] = (const bf16*)w;
  g.ldP = ldx;
  g.ldQ = K;
  g.I = R;
  g.J = F;
  g.C = K;
  g.csets = 1;
  g.out[0] = (bf16*)y;
  g.out[1] = (bf16*)ty;
  g.ldo = ldy;
  g.bias = (const bf16*)bias;
  g.nz = 2;
  const int shape = pick_shape(false, 2, R, F, K);
  return shape < k128 ? launch_gemm_fwd(shape, g, st) : launch_small<false, false, false>(shape, g, st);
}

hipError_t launch_linear_bwd(int R, int K, int F, long long ldx, long long ldy, const void* x, const void* tx,
                             const void* w, const void* gy, const void* gty, void* gx, void* gtx, void* gw, void* gbias,
                             void* workspace, hipStream_t st) {
  {  // gx = gy W, gtx = gty W: rows = tokens, contraction over f, W read transposed
    GemmArgs g{};
    g.P[0] = (const bf16*)gy;
    g.P[1] = (const bf16*)gty;
    g.Q[0] = g.Q[1] = (const bf16*)w;
    g.ldP = ldy;
    g.ldQ = K;
    g.I = R;
    g.J = K;
    g.C = F;
    g.csets = 1;
    g.out[0] = (bf16*)gx;
    g.out[1] = (bf16*)gtx;
    g.ldo = ldx;
    g.nz = 2;
    const int shape = pick_shape(true, 2, R, K, F);
    const hipError_t e = shape < k128 ? launch_gemm_gx(shape, g, st) : launch_small<false, true, false>(shape, g, st);
    if (e != hipSuccess) return e;
  }
  const int max_splits = dw_splits(F, K, R);
  const DwPlan plan = plan_dw(F, K, R, max_splits);
  const int splits = plan.splits;
  float* part = static_cast<float*>(workspace);
  {  // gW = gy^T x + gty^T tx: contraction over the tokens of both sets, both operands read transposed
    GemmArgs g{};
    g.P[0] = (const bf16*)gy;
    g.P[1] = (const bf16*)gty;
    g.Q[0] = (const bf16*)x;
    g.Q[1] = (const bf16*)tx;
    g.ldP = ldy;
    g.ldQ = ldx;
    g.I = F;
    g.J = K;
    g.C = R;
    g.csets = 2;
    g.part = part;
    g.splits = splits;
    g.nz = splits;
    g.out[0] = (bf16*)gw;
    g.ldo = K;
    if (splits == 1 && plan.shape >= k128) {
      const hipError_t e = launch_small<true, true, false>(plan.shape, g, st);
      if (e != hipSuccess) return e;
    } else {
      hipError_t e = plan.shape < k128 ? launch_gemm_gw(plan.shape, g, st) : launch_small<true, true, true>(plan.shape, g, st);
      if (e != hipSuccess) return e;
      const long long n = (long long)F * K;
      hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)((n / 8 + 255) / 256)), dim3(256), 0, st, part, splits, n,
                         (bf16*)gw);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  if (gbias != nullptr && R <= kDirectRows) {
    hipLaunchKernelGGL(colsum_direct_kernel, dim3((unsigned)((F + 63) / 64)), dim3(1024), 0, st, (const bf16*)gy, R, F, ldy,
                       (bf16*)gbias);
    return hipGetLastError();
  }
  if (gbias != nullptr) {
    const size_t dw = ((size_t)max_splits * F * K * sizeof(float) + 255) & ~(size_t)255;
    float* bp = reinterpret_cast<float*>(static_cast<char*>(workspace) + dw);
    const int chunks = bias_chunks(R);
    hipLaunchKernelGGL(colsum_kernel, dim3((F + 511) / 512, chunks), dim3(256), 0, st, (const bf16*)gy, R, F, ldy, chunks, bp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bias_sum_kernel, dim3((unsigned)((F + 63) / 64)), dim3(1024), 0, st, bp, chunks, F, (bf16*)gbias);
    return hipGetLastError();
  }
  return hipSuccess;
}

}  // namespace tvm
