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

// Shape of a workgroup: NWI x NWJ waves, each with WI x WJ blocks of 32 x 32; NST LDS stages; OCC workgroups per CU.
template <int NWI_, int NWJ_, int WI_, int WJ_, int NST_, int OCC_>
struct Cfg {
  static constexpr int NWI = NWI_, NWJ = NWJ_, WI = WI_, WJ = WJ_, NST = NST_, OCC = OCC_;
  static constexpr int NW = NWI_ * NWJ_, NT = 64 * NW;
  static constexpr int TI = NWI_ * WI_ * 32;  // output rows per workgroup
  static constexpr int TJ = NWJ_ * WJ_ * 32;  // output columns per workgroup
};

// Transposed fragment with the contraction index in natural order: lane (ic, hh) gets, of column 32*db + ic of the
// tile, rows 16*cc + 8*hh + 0..7 (the first transposing read takes rows 8hh..8hh+3, the second 8hh+4..8hh+7;
// four consecutive rows share one swizzle term, as in Tile::taddr).
template <class T>
struct TrNat {
  int lo, hi;
  __device__ __forceinline__ static TrNat make(int ic, int hh) {
    const int i = ic & 15, bq = ic >> 4;
    const int y = 2 * bq + ((i & 3) >> 1);
    const int r0 = 8 * hh + (i >> 2), r1 = r0 + 4;
    const int sub = (i & 1) * 8;
    return TrNat{(r0 * T::PCH + (y ^ ((r0 >> 2) & 3))) * 16 + sub, (r1 * T::PCH + (y ^ ((r1 >> 2) & 3))) * 16 + sub};
  }
  __device__ __forceinline__ bf16x8 frag(const char* p, int cc, int db) const {
    typedef bf16x4 __attribute__((address_space(3))) * lp;
    const int imm = cc * 16 * T::PCH * 16 + db * 64;
    const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lp)(p + lo + imm));
    const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lp)(p + hi + imm));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};

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

// The same product for shapes with few 256-row tiles: workgroups of four waves on 64 x 64 or 128 x 128 output tiles, one
// tile each, many workgroups in flight.  What bounds it is latency (a contraction tile is 128 or 512 cycles of matrix
// work per wave against some 2000 from L2), so the contraction runs NST - 1 tiles ahead through NST LDS stages, with one
// barrier per tile and the loads in flight counted rather than drained.  Tiles are filled and read as in the attention kernels
// (mfma_tiles.h: swizzled row-major tiles; "row" fragments are 16-byte reads, "transposed" ones the transposing LDS read, here
// with the contraction index in natural order so that both kinds pair up).  Contraction tiles are taken in the same order and
// every output element is the same chain of products as in linear_pipe.hip: results are bit for bit the same (with equal
// splits).
template <bool PTR, bool QTR, bool PARTIAL, class C>
__global__ __launch_bounds__(C::NT, C::OCC) void gemm_small_kernel(GemmArgs g) {
  constexpr int kNW = C::NW, kWI = C::WI, kWJ = C::WJ, kTI = C::TI, kTJ = C::TJ, NST = C::NST;
  using TP = typename std::conditional<PTR, Tile<kBK, kTI / 8, kNW>, Tile<kTI, 4, kNW>>::type;
  using TQ = typename std::conditional<QTR, Tile<kBK, kTJ / 8, kNW>, Tile<kTJ, 4, kNW>>::type;
  constexpr int P_BYTES = PTR ? TP::BYTES : 2 * TP::BYTES, Q_BYTES = QTR ? TQ::BYTES : 2 * TQ::BYTES;
  constexpr int BUF = P_BYTES + Q_BYTES;
  constexpr int LOADS = (PTR ? 1 : 2) * TP::IPW + (QTR ? 1 : 2) * TQ::IPW;
  constexpr int OUT_REGION = 32 * (64 * kWJ + 16);
  static_assert(NST >= 3 && (NST - 2) * LOADS < 64 && kNW * OUT_REGION <= NST * BUF, "stages");
  __shared__ __attribute__((aligned(16))) char lds[NST * BUF];
  const int nI = (g.I + kTI - 1) / kTI, nJ = (g.J + kTJ - 1) / kTJ, total = g.nz * nI * nJ;
  // XCD x owns the x-th eighth of the tile list (as in linear_pipe.hip: groups of kGI tile rows, down the group first)
  const int wg = (int)(blockIdx.x & 7) * ((total + 7) >> 3) + (int)(blockIdx.x >> 3);
  if (wg >= min(total, ((int)(blockIdx.x & 7) + 1) * ((total + 7) >> 3))) return;
  const int tid = threadIdx.x, lane = tid & 63, ic = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi = wave % C::NWI, wj = wave / C::NWI;
  const int zz = wg / (nI * nJ), id = wg - zz * (nI * nJ);
  const int grp = id / (kGI * nJ), it_first = grp * kGI, gs = min(nI - it_first, kGI);
  const int rem = id - grp * (kGI * nJ), jt = rem / gs, it = it_first + (rem - jt * gs);
  const int i0 = it * kTI, j0 = jt * kTJ;
  const int nct = (g.C + kBK - 1) / kBK, ntot = g.csets * nct;
  const int t_begin = PARTIAL ? (int)((long long)zz * ntot / g.splits) : 0;
  const int t_end = PARTIAL ? (int)((long long)(zz + 1) * ntot / g.splits) : ntot;
  const bool two = g.csets == 2;  // grad W: contraction over both row sets
  const int clast = g.C - (nct - 1) * kBK;
  const unsigned lds0 = lds_addr_of(lds);
  const unsigned pitchP = (unsigned)(g.ldP * 2), pitchQ = (unsigned)(g.ldQ * 2);
  typename TP::Offs op_full, op_last;
  typename TQ::Offs oq_full, oq_last;
  if (PTR) {
    const typename TP::Lane l = TP::lane_setup(min(g.I - i0, kTI), wave, lane);
    op_full = TP::offsets(l, pitchP, kBK);
    op_last = TP::offsets(l, pitchP, clast);
  } else {
    op_full = op_last = TP::offsets(TP::lane_setup(32, wave, lane), pitchP, min(g.I - i0, kTI));
  }
  if (QTR) {
    const typename TQ::Lane l = TQ::lane_setup(min(g.J - j0, kTJ), wave, lane);
    oq_full = TQ::offsets(l, pitchQ, kBK);
    oq_last = TQ::offsets(l, pitchQ, clast);
  } else {
    oq_full = oq_last = TQ::offsets(TQ::lane_setup(32, wave, lane), pitchQ, min(g.J - j0, kTJ));
  }
  const typename TP::RAddr rp = TP::raddr(ic, hh);
  const typename TQ::RAddr rq = TQ::raddr(ic, hh);
  const TrNat<TP> tp = TrNat<TP>::make(ic, hh);
  const TrNat<TQ> tq = TrNat<TQ>::make(ic, hh);
  f32x16 acc[kWI][kWJ];
  {
    const bool with_bias = !PARTIAL && g.bias != nullptr && zz == 0;
    const int jw = j0 + wj * (kWJ * 32);
#pragma unroll
    for (int b = 0; b < kWJ; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int j = jw + b * 32 + drow(r, hh);
        const float v = with_bias && j < g.J ? (float)g.bias[j] : 0.f;
#pragma unroll
        for (int a = 0; a < kWI; ++a) acc[a][b][r] = v;
      }
  }
  // all wave-loads of contraction tile t (beyond the end: the last one again, never used) into the stage at `buf`
  auto issue = [&](int t, unsigned buf) {
    t = min(t, t_end - 1);
    const int set = two && t >= nct ? 1 : 0, ct = t - set * nct;
    const long long c0 = (long long)ct * kBK;
    const bool last = ct == nct - 1;
    const bf16* pb = g.P[two ? set : PARTIAL ? 0 : zz] + (PTR ? c0 * g.ldP + i0 : (long long)i0 * g.ldP + c0);
    const bf16* qb = g.Q[set] + (QTR ? c0 * g.ldQ + j0 : (long long)j0 * g.ldQ + c0);
    const int half2 = (last && clast <= 32) ? 0 : 32;
#pragma unroll
    for (int x = 0; x < TP::IPW; ++x) {
      TP::issue_at(PTR && last ? op_last.o[x] : op_full.o[x], x, pb, buf, wave);
      if (!PTR) TP::issue_at(op_full.o[x], x, pb + half2, buf + TP::BYTES, wave);
    }
#pragma unroll
    for (int x = 0; x < TQ::IPW; ++x) {
      TQ::issue_at(QTR && last ? oq_last.o[x] : oq_full.o[x], x, qb, buf + P_BYTES, wave);
      if (!QTR) TQ::issue_at(oq_full.o[x], x, qb + half2, buf + P_BYTES + TQ::BYTES, wave);
    }
  };
#pragma unroll
  for (int x = 0; x < NST - 1; ++x) issue(t_begin + x, lds0 + x * BUF);
  int n = 0;
  for (int t = t_begin; t < t_end; ++t) {
    dma_wait_keep<(NST - 2) * LOADS>();  // this wave's share of tile t has landed
    const int ct = two && t >= nct ? t - nct : t;
    if (ct == nct - 1 && clast < kBK) {  // entries beyond the set's end were fetched as copies: zeros instead
      char* pt = lds + n * BUF;
#pragma unroll
      for (int x = 0; x < TP::IPW; ++x) {
        const int pos = (wave + x * kNW) * 64 + lane;
        if (PTR) {
          if (pos / TP::PCH >= clast) *reinterpret_cast<uint4*>(pt + pos * 16) = make_uint4(0u, 0u, 0u, 0u);
        } else if (clast <= 32) {
          *reinterpret_cast<uint4*>(pt + TP::BYTES + pos * 16) = make_uint4(0u, 0u, 0u, 0u);
        }
      }
    }
    __syncthreads();  // it is there for everyone, and everyone is done with tile t-1, whose stage is refilled now
    const int nf = n == 0 ? NST - 1 : n - 1;
    issue(t + NST - 1, lds0 + nf * BUF);
    const char* sp = lds + n * BUF;
    const char* sq = sp + P_BYTES;
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      bf16x8 pf[kWI], qf[kWJ];
#pragma unroll
      for (int a = 0; a < kWI; ++a)
        pf[a] = PTR ? tp.frag(sp, kk, wi * kWI + a) : TP::frag_row(sp + (kk >> 1) * TP::BYTES, rp, wi * kWI + a, kk & 1);
#pragma unroll
      for (int b = 0; b < kWJ; ++b)
        qf[b] = QTR ? tq.frag(sq, kk, wj * kWJ + b) : TQ::frag_row(sq + (kk >> 1) * TQ::BYTES, rq, wj * kWJ + b, kk & 1);
#pragma unroll
      for (int a = 0; a < kWI; ++a)
#pragma unroll
        for (int b = 0; b < kWJ; ++b) acc[a][b] = mfma(qf[b], pf[a], acc[a][b]);
    }
    n = n + 1 == NST ? 0 : n + 1;
  }
  const int jw = j0 + wj * (kWJ * 32);
  if (PARTIAL) {
    store_partial<kWI, kWJ>(g, acc, zz, i0 + wi * kWI * 32, jw, ic, hh);
    dma_wait();  // (no load may land in LDS that the next workgroup owns)
    return;
  }
  dma_wait();  // the loads past the end land in stages that the results are about to go through
  __syncthreads();
  if (jw < g.J) {
    const unsigned lw = lds0 + (unsigned)wave * OUT_REGION;
#pragma unroll
    for (int a = 0; a < kWI; ++a)
      store_tile_coalesced<kWJ>(lw, g.out[zz] + jw, g.ldo, i0 + (wi * kWI + a) * 32, g.I, g.J - jw, acc[a], 1.f, lane);
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

// The tile shapes in use
using Cfg128 = Cfg<2, 2, 2, 2, 3, 1>;  // 128 x 128, four waves
using Cfg64 = Cfg<2, 2, 1, 1, 4, 2>;   // 64 x 64, four waves
template <class C>
constexpr bool shape_is(int c) { return C::TI == kTileI[c] && C::TJ == kTileJ[c]; }
static_assert(shape_is<Cfg128>(k128) && shape_is<Cfg64>(k64), "the plan's tiles");
static_assert(Cfg128::NT == kSmallThreads && Cfg64::NT == kSmallThreads, "the plan's limit");

int bias_chunks(int R) {
  const int c = (R + 63) / 64;
  return c > 256 ? 256 : c;
}

// Launches a product with tile shape c (128 or 64).
template <bool PTR, bool QTR, bool PARTIAL>
hipError_t launch_small(int c, const GemmArgs& g, hipStream_t st) {
  const dim3 grid((unsigned)small_workgroups(g.nz * tiles_of(c, g.I, g.J)));
  if (c == k64) hipLaunchKernelGGL((gemm_small_kernel<PTR, QTR, PARTIAL, Cfg64>), grid, dim3(Cfg64::NT), 0, st, g);
  else hipLaunchKernelGGL((gemm_small_kernel<PTR, QTR, PARTIAL, Cfg128>), grid, dim3(Cfg128::NT), 0, st, g);
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
