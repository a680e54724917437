// float32 attention with tangent on the float32 matrix cores (v_mfma_f32_16x16x4_f32: full float32 operands, products
// and sums).  Head dims that are multiples of 4 up to 128, but for calls of a handful of rows (f32_mfma.h says which); what it
// does not take runs on the plain-ALU kernels (generic_kernels.hip), whose formulas these kernels share.
//
// What bounds it: the float32 matrix rate (157 TFLOP/s, a sixteenth of the bf16 one), so operand traffic is cheap by
// comparison and nothing of the streamed side goes through LDS.  A workgroup owns 16 rows of the fixed side (queries
// in the forward and the query-side backward, keys in the key-side backward); its four waves deal the streamed side's
// tiles of 16 rows out among themselves, each with accumulators of its own that are added through LDS at the end.  With
// 16 rows per workgroup and four waves on each, 256-token sequences of 48 heads are 3072 waves, three per SIMD.
//
//   * Scores are computed transposed, D[streamed row][fixed row], lane (i = lane & 15, g = lane >> 4) holding column i
//     (its fixed row) and rows 4g..4g+3.  The contraction over the head dim is walked in an order that suits 16-byte
//     loads: step (t, c) has lane group g at column 16t + 4g + c, on both operands, so that lane (i, g) reads four steps
//     of row i with one load of columns 16t+4g..+3.
//   * A score tile is the B operand of the output products as it stands: step r contracts over streamed rows 4g + r.
//     The A operand is then column-wise, X[row 4g+r][column]: lane (i, g) loads columns 64ch + 4i..+3 of its row, and the
//     four entries go to four output blocks, i.e. row i of block (ch, e) is column 64ch + 4i + e (a last half chunk of 32
//     columns: 64ch + 2i + e).
//   * Fixed-side operands sit in LDS in the order the lanes read them (one 16-byte read per four contraction steps).
//   * Streamed rows are read with bounds-checked buffer loads: rows beyond the end and columns beyond the head dim
//     read as zero.
// A float32 training step at B4 H12 N256 d64 (8.5 GFLOP): 105 us (130 before the backward's loads were put in stages), 81
// TFLOP/s by the algorithmic count and 104 by the executed one (the backward's two kernels both form the score tiles), against
// 3590 us on the plain-ALU kernels, whose lanes each walked a row of their own with 4-byte loads.  The smallest call (B1 H2
// N64 d32), where launches and latency count: 23 us.
#include "f32_mfma.h"
#include "mfma_tiles.h"

namespace tvm {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;

constexpr int kR = 16;   // rows per tile, either side
constexpr int kNW = 4;   // waves per workgroup, each on its own streamed tiles
constexpr unsigned kOut = 0x80000000u;  // offset of a column beyond the head dim: out of range whatever row is added

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// One head of one tensor: `rows` rows of D floats, `pitch` bytes apart (rows * pitch < 2^31).
struct Head {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ static Head make(const float* p, int rows, unsigned pitch, int D) {
    return Head{__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)((unsigned)(rows - 1) * pitch + (unsigned)D * 4u),
                                                  0x00027000)};
  }
  __device__ __forceinline__ f32x4 ld4(unsigned off) const {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
  }
  __device__ __forceinline__ float ld1(unsigned off) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
  }
  __device__ __forceinline__ f32x2 ld2(unsigned off) const {
    return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
  }
};

// Everything that depends on the padded head dim DP (a multiple of 32) and the lane.
template <int DP>
struct Geo {
  static constexpr int NT = DP / 16;               // 16-byte loads of a row-wise fragment set; output blocks
  static constexpr int NCH = DP / 64;              // whole column chunks
  static constexpr bool HALF = DP % 64 != 0;       // and a half one
  static constexpr int LDR = DP + 4;               // row pitch (floats) of the reduction buffer: 16-byte rows, four banks apart
  static constexpr int FIX = NT * 64;              // float4 of one fixed tensor in LDS
  struct Rows { f32x4 t[NT]; };                    // row-wise fragments of one streamed tile
  struct Cols { f32x4 c[4][NCH ? NCH : 1]; f32x2 h[4]; };  // column-wise fragments
  struct Acc { f32x4 b[NT]; };                     // 16 fixed rows x DP columns

  unsigned row_off[NT], col_off[NCH ? NCH : 1], half_off;
  int i, g;
  __device__ __forceinline__ void init(int lane, int D, unsigned pitch) {
    i = lane & 15;
    g = lane >> 4;
#pragma unroll
    for (int t = 0; t < NT; ++t) row_off[t] = 16 * t + 4 * g < D ? (unsigned)i * pitch + (16 * t + 4 * g) * 4u : kOut;
    const unsigned r4 = 4u * g * pitch;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) col_off[ch] = 64 * ch + 4 * i < D ? r4 + (64 * ch + 4 * i) * 4u : kOut;
    half_off = 64 * NCH + 2 * i < D ? r4 + (64 * NCH + 2 * i) * 4u : kOut;
  }
  __device__ __forceinline__ Rows rows(const Head& h, unsigned tile) const {
    Rows x;
#pragma unroll
    for (int t = 0; t < NT; ++t) x.t[t] = h.ld4(row_off[t] + tile);
    return x;
  }
  __device__ __forceinline__ Cols cols(const Head& h, unsigned tile, unsigned pitch) const {
    Cols x;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) x.c[r][ch] = h.ld4(col_off[ch] + tile + r * pitch);
      if constexpr (HALF) x.h[r] = h.ld2(half_off + tile + r * pitch);
    }
    return x;
  }
  // acc += X^T w, contraction over the tile's 16 rows
  __device__ __forceinline__ static void out(Acc& acc, const Cols& x, const f32x4& w) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc.b[4 * ch + e] = mfma4(x.c[r][ch][e], w[r], acc.b[4 * ch + e]);
      if constexpr (HALF) {
        acc.b[4 * NCH] = mfma4(x.h[r][0], w[r], acc.b[4 * NCH]);
        acc.b[4 * NCH + 1] = mfma4(x.h[r][1], w[r], acc.b[4 * NCH + 1]);
      }
    }
  }
  __device__ __forceinline__ static Acc zero() {
    Acc a;
#pragma unroll
    for (int t = 0; t < NT; ++t) a.b[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    return a;
  }
  // Fixed rows row0.. of one tensor into LDS, in the order the lanes read them; rows and columns beyond the end are zero.
  __device__ __forceinline__ static void fix(f32x4* dst, const float* head, long long pitch, int row0, int rows, int D) {
    for (int x = threadIdx.x; x < FIX; x += 64 * kNW) {
      const int row = row0 + (x & 15), col = 16 * (x >> 6) + 4 * ((x >> 4) & 3);
      dst[x] = row < rows && col < D ? *reinterpret_cast<const f32x4*>(head + row * pitch + col) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  // The four waves' accumulators added in order and multiplied by f: thread (row = tid >> 4, x = tid & 15) gets columns
  // 64ch + 4x..+3 and the half chunk's 64 NCH + 2x..+1 of its row.
  struct Row { f32x4 c[NCH ? NCH : 1]; f32x2 h; };
  __device__ __forceinline__ static Row gather(float* red, const Acc& a, int wave, int i, int g) {
    __syncthreads();  // the buffer's previous readers are done
    float* mine = red + (wave * kR + i) * LDR;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
        *reinterpret_cast<f32x4*>(mine + 64 * ch + 16 * g + 4 * r) =
            f32x4{a.b[4 * ch][r], a.b[4 * ch + 1][r], a.b[4 * ch + 2][r], a.b[4 * ch + 3][r]};
      if constexpr (HALF)
        *reinterpret_cast<f32x2*>(mine + 64 * NCH + 8 * g + 2 * r) = f32x2{a.b[4 * NCH][r], a.b[4 * NCH + 1][r]};
    }
    __syncthreads();
    const float* src = red + (threadIdx.x >> 4) * LDR;
    const int x = threadIdx.x & 15;
    Row o{};
#pragma unroll
    for (int w = 0; w < kNW; ++w) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) o.c[ch] += *reinterpret_cast<const f32x4*>(src + w * kR * LDR + 64 * ch + 4 * x);
      if constexpr (HALF) o.h += *reinterpret_cast<const f32x2*>(src + w * kR * LDR + 64 * NCH + 2 * x);
    }
    return o;
  }
  __device__ __forceinline__ static void store(float* row, const Row& o, float f, int D) {
    const int x = threadIdx.x & 15;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch)
      if (64 * ch + 4 * x < D) *reinterpret_cast<f32x4*>(row + 64 * ch + 4 * x) = o.c[ch] * f;
    if constexpr (HALF)
      if (64 * NCH + 2 * x < D) *reinterpret_cast<f32x2*>(row + 64 * NCH + 2 * x) = o.h * f;
  }
};

// c += X F over the head dim: streamed fragments x, fixed fragments f (in LDS)
#define TVM_F32_STEP(acc, x, f)                                               \
  _Pragma("unroll") for (int c_ = 0; c_ < 4; ++c_) acc = mfma4((x)[c_], (f)[c_], acc)

template <int DP>
__global__ __launch_bounds__(256, 2) void fwd_f32_kernel(Shape s, const float* __restrict__ q, const float* __restrict__ k,
                                                         const float* __restrict__ v, const float* __restrict__ tq,
                                                         const float* __restrict__ tk, const float* __restrict__ tv,
                                                         float* __restrict__ o, float* __restrict__ to,
                                                         float* __restrict__ lse, float* __restrict__ stats) {
  using G = Geo<DP>;
  __shared__ f32x4 fixed[2 * G::FIX];
  __shared__ __attribute__((aligned(16))) float red[kNW * kR * G::LDR];
  __shared__ float wm[kNW][kR], wl[kNW][kR], wc[kNW][kR], wref[kR];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nblk = (s.M + kR - 1) / kR, wg = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = wg / nblk, b = bh / s.H, h = bh % s.H, i0 = (wg - bh * nblk) * kR;
  const long long base = b * s.sb + h * s.sh, qbase = b * s.qsb + h * s.qsh;
  const unsigned pitch = (unsigned)(s.sn * 4);
  G::fix(fixed, q + qbase, s.qsn, i0, s.M, s.D);
  G::fix(fixed + G::FIX, tq + qbase, s.qsn, i0, s.M, s.D);
  const Head hk = Head::make(k + base, s.N, pitch, s.D), htk = Head::make(tk + base, s.N, pitch, s.D);
  const Head hv = Head::make(v + base, s.N, pitch, s.D), htv = Head::make(tv + base, s.N, pitch, s.D);
  G geo;
  geo.init(lane, s.D, pitch);
  const int i = geo.i, g = geo.g;
  typename G::Acc ao = G::zero(), at = G::zero();
  float m = -INFINITY, l = 0.f, cs = 0.f;
  __syncthreads();
  for (int j0 = wave * kR; j0 < s.N; j0 += kNW * kR) {
    const unsigned tile = (unsigned)j0 * pitch;
    const typename G::Rows kf = geo.rows(hk, tile), tkf = geo.rows(htk, tile);
    const typename G::Cols vf = geo.cols(hv, tile, pitch), tvf = geo.cols(htv, tile, pitch);
    f32x4 z = {0.f, 0.f, 0.f, 0.f}, za = z, zb = z;
#pragma unroll
    for (int t = 0; t < G::NT; ++t) {
      const f32x4 fq = fixed[t * 64 + lane], ftq = fixed[G::FIX + t * 64 + lane];
      TVM_F32_STEP(z, kf.t[t], fq);
      TVM_F32_STEP(za, kf.t[t], ftq);
      TVM_F32_STEP(zb, tkf.t[t], fq);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      z[r] = j0 + 4 * g + r < s.N ? z[r] * s.alpha : -INFINITY;
      mx = fmaxf(mx, z[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float mn = fmaxf(m, mx);
    const float ref = mn == -INFINITY ? 0.f : mn;  // a wave whose keys so far all have probability 0
    const float f = __expf(m - ref);
    f32x4 p, pz;
    float sp = 0.f, sz = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __expf(z[r] - ref);
      pz[r] = p[r] * ((za[r] + zb[r]) * s.alpha);
      sp += p[r];
      sz += pz[r];
    }
    l = l * f + sp;
    cs = cs * f + sz;
    m = mn;
#pragma unroll
    for (int t = 0; t < G::NT; ++t) {
      ao.b[t] *= f;
      at.b[t] *= f;
    }
    G::out(ao, vf, p);
    G::out(at, vf, pz);
    G::out(at, tvf, p);
  }
  // the four waves' sums over their keys, brought to one reference maximum
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  cs += __shfl_xor(cs, 16);
  cs += __shfl_xor(cs, 32);
  if (lane < kR) wm[wave][i] = m;
  __syncthreads();
  float mall = wm[0][i];
#pragma unroll
  for (int w = 1; w < kNW; ++w) mall = fmaxf(mall, wm[w][i]);
  const float ref = mall == -INFINITY ? 0.f : mall;
  const float f = __expf(m - ref);
  if (lane < kR) {
    wl[wave][i] = l * f;
    wc[wave][i] = cs * f;
    if (wave == 0) wref[i] = ref;
  }
#pragma unroll
  for (int t = 0; t < G::NT; ++t) {
    ao.b[t] *= f;
    at.b[t] *= f;
  }
  const typename G::Row ro = G::gather(red, ao, wave, i, g);
  typename G::Row rt = G::gather(red, at, wave, i, g);
  const int row = threadIdx.x >> 4;
  if (i0 + row >= s.M) return;
  float ls = 0.f, c = 0.f;
#pragma unroll
  for (int w = 0; w < kNW; ++w) {
    ls += wl[w][row];
    c += wc[w][row];
  }
  const float inv = 1.f / ls, mubar = c * inv;
#pragma unroll
  for (int ch = 0; ch < G::NCH; ++ch) rt.c[ch] -= ro.c[ch] * mubar;  // (scaled by inv below)
  if constexpr (G::HALF) rt.h -= ro.h * mubar;
  const long long a = qbase + (long long)(i0 + row) * s.qsn;
  G::store(o + a, ro, inv, s.D);
  G::store(to + a, rt, inv, s.D);
  if ((threadIdx.x & 15) == 0) {
    const long long r = (long long)bh * s.M + i0 + row;
    if (lse) lse[r] = wref[row] + __logf(ls);
    if (stats) stats[r] = mubar;
  }
}

// Query side of the backward: dq, dtq of 16 queries, and Step 1's row scalars for the key side behind it.
// The loads are put in stages, each sent off a group of products before it is used (the scheduling barriers hold the
// compiler to that), so that few fragments live at once: 253 registers instead of 280 at DP = 128, two waves per SIMD
// instead of one.  With a tangent there are products enough behind the next tile's first rows to load them one tile ahead
// (a wave without one asks for an offset out of range, and for the head's first bytes, unused, in lanes beyond the head dim, where
// kOut + kOut is 0: reading its own tile once more cost 7 % of a backward of 64 x 64 at DP = 128, and a branch around the loads
// spills).  DP = 32 has the registers to take the second stage's loads with the first.
// Both upstream gradients, B2 H16 N256 d128: 62 us before, 48 now; B2 H8 N1024 d64: 185 before, 167 now.  Without
// the tangent there is little to put behind a stage's loads: B4 H12 N256 d64 18.4 us with all loads first, 18.8 in stages
// and 20.2 with the next tile's rows ahead, so there all loads come first.
// MODE as in BwdArgs: 0 both upstream gradients, 1 gO only, 2 gTO only.
template <int DP, int MODE>
__global__ __launch_bounds__(256, MODE == 1 ? (DP <= 64 ? 2 : 1) : DP <= 32 ? 4 : DP <= 64 ? 3 : 2) void bwd_row_f32_kernel(
    Shape s, const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const float* __restrict__ tq, const float* __restrict__ tk, const float* __restrict__ tv, const float* __restrict__ o,
    const float* __restrict__ to, const float* __restrict__ lse, const float* __restrict__ stats,
    const float* __restrict__ gO, const float* __restrict__ gTO, float* __restrict__ dsig, float* __restrict__ sig1,
    float* __restrict__ dq, float* __restrict__ dtq) {
  using G = Geo<DP>;
  constexpr bool TAN = MODE != 1, GO = MODE != 2;
  __shared__ f32x4 fixed[4 * G::FIX];  // q, tq, gO, gTO
  __shared__ __attribute__((aligned(16))) float red[kNW * kR * G::LDR];
  __shared__ float rows[2][kR];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nblk = (s.M + kR - 1) / kR, wg = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = wg / nblk, b = bh / s.H, h = bh % s.H, i0 = (wg - bh * nblk) * kR;
  const long long base = b * s.sb + h * s.sh, qbase = b * s.qsb + h * s.qsh;
  const unsigned pitch = (unsigned)(s.sn * 4);
  G::fix(fixed, q + qbase, s.qsn, i0, s.M, s.D);
  if constexpr (TAN) G::fix(fixed + G::FIX, tq + qbase, s.qsn, i0, s.M, s.D);
  if constexpr (GO) G::fix(fixed + 2 * G::FIX, gO + qbase, s.qsn, i0, s.M, s.D);
  if constexpr (TAN) G::fix(fixed + 3 * G::FIX, gTO + qbase, s.qsn, i0, s.M, s.D);
  {  // Step 1: dsig = gO.O + gTO.tO, sig1 = gTO.O; sixteen threads per row
    const int row = threadIdx.x >> 4, x = threadIdx.x & 15;
    float a = 0.f, c1 = 0.f;
    if (i0 + row < s.M) {
      const long long ro = qbase + (long long)(i0 + row) * s.qsn;
      for (int c = 4 * x; c < s.D; c += 64) {
        const f32x4 oc = *reinterpret_cast<const f32x4*>(o + ro + c);
        if constexpr (GO) {
          const f32x4 gc = *reinterpret_cast<const f32x4*>(gO + ro + c);
#pragma unroll
          for (int e = 0; e < 4; ++e) a = fmaf(gc[e], oc[e], a);
        }
        if constexpr (TAN) {
          const f32x4 tg = *reinterpret_cast<const f32x4*>(gTO + ro + c), toc = *reinterpret_cast<const f32x4*>(to + ro + c);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            a = fmaf(tg[e], toc[e], a);
            c1 = fmaf(tg[e], oc[e], c1);
          }
        }
      }
    }
#pragma unroll
    for (int d = 8; d > 0; d >>= 1) {
      a += __shfl_xor(a, d);
      c1 += __shfl_xor(c1, d);
    }
    if (x == 0) {
      rows[0][row] = a;
      rows[1][row] = c1;
      if (i0 + row < s.M) {
        const long long r = (long long)bh * s.M + i0 + row;
        dsig[r] = a;
        sig1[r] = c1;
      }
    }
  }
  const Head hk = Head::make(k + base, s.N, pitch, s.D), hv = Head::make(v + base, s.N, pitch, s.D);
  const Head htk = TAN ? Head::make(tk + base, s.N, pitch, s.D) : hk, htv = TAN ? Head::make(tv + base, s.N, pitch, s.D) : hv;
  G geo;
  geo.init(lane, s.D, pitch);
  const int i = geo.i, g = geo.g;
  const long long r_i = (long long)bh * s.M + min(i0 + i, s.M - 1);
  const float lse_i = lse[r_i], mubar_i = TAN ? stats[r_i] : 0.f;
  typename G::Acc aq = G::zero(), atq = G::zero();
  __syncthreads();
  const float dsig_i = rows[0][i], sig1_i = rows[1][i];
  typename G::Rows kf, vf, tkf, tvf;
  if constexpr (TAN) {
    const unsigned first = wave * kR < s.N ? (unsigned)(wave * kR) * pitch : kOut;
    kf = geo.rows(hk, first);
    tkf = geo.rows(htk, first);
  }
  for (int j0 = wave * kR; j0 < s.N; j0 += kNW * kR) {
    const unsigned tile = (unsigned)j0 * pitch;
    const unsigned next = j0 + kNW * kR < s.N ? tile + (unsigned)(kNW * kR) * pitch : kOut;
    if constexpr (!TAN) kf = geo.rows(hk, tile);
    vf = geo.rows(hv, tile);
    typename G::Cols kc, tkc;
    if constexpr (!TAN) kc = geo.cols(hk, tile, pitch);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 z = zero, za = zero, zb = zero, da = zero, db = zero, e = zero;
    if constexpr (TAN) {
      if constexpr (DP <= 32) {
        tvf = geo.rows(htv, tile);
        kc = geo.cols(hk, tile, pitch);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < G::NT; ++t) {
        const f32x4 fq = fixed[t * 64 + lane], ftq = fixed[G::FIX + t * 64 + lane];
        TVM_F32_STEP(z, kf.t[t], fq);
        TVM_F32_STEP(za, kf.t[t], ftq);
        TVM_F32_STEP(zb, tkf.t[t], fq);
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (DP > 32) {
        tvf = geo.rows(htv, tile);
        kc = geo.cols(hk, tile, pitch);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int t = 0; t < G::NT; ++t) {
        const f32x4 ftg = fixed[3 * G::FIX + t * 64 + lane];
        if constexpr (GO) {
          const f32x4 fg = fixed[2 * G::FIX + t * 64 + lane];
          TVM_F32_STEP(da, vf.t[t], fg);
        }
        TVM_F32_STEP(e, vf.t[t], ftg);
      }
      __builtin_amdgcn_sched_barrier(0);
      tkc = geo.cols(htk, tile, pitch);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < G::NT; ++t) {
        const f32x4 ftg = fixed[3 * G::FIX + t * 64 + lane];
        TVM_F32_STEP(db, tvf.t[t], ftg);
      }
      __builtin_amdgcn_sched_barrier(0);
      kf = geo.rows(hk, next);
      tkf = geo.rows(htk, next);
      __builtin_amdgcn_sched_barrier(0);
    } else {
#pragma unroll
      for (int t = 0; t < G::NT; ++t) {
        const f32x4 fq = fixed[t * 64 + lane], fg = fixed[2 * G::FIX + t * 64 + lane];
        TVM_F32_STEP(z, kf.t[t], fq);
        TVM_F32_STEP(da, vf.t[t], fg);
      }
    }
    f32x4 gz, gzt;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool ok = j0 + 4 * g + r < s.N;
      const float p = __expf(z[r] * s.alpha - lse_i);
      float x = p * ((da[r] + db[r]) - dsig_i);
      if constexpr (TAN) {
        const float n = (za[r] + zb[r]) * s.alpha - mubar_i, xt = p * (e[r] - sig1_i);
        x = fmaf(xt, n, x);
        gzt[r] = ok ? xt : 0.f;
      }
      gz[r] = ok ? x : 0.f;
    }
    G::out(aq, kc, gz);
    if constexpr (TAN) {
      G::out(atq, kc, gzt);
      G::out(aq, tkc, gzt);
    }
  }
  const int row = threadIdx.x >> 4;
  const long long a = qbase + (long long)(i0 + row) * s.qsn;
  const typename G::Row rq = G::gather(red, aq, wave, i, g);
  if (i0 + row < s.M) G::store(dq + a, rq, s.alpha, s.D);
  if constexpr (TAN) {
    const typename G::Row rt = G::gather(red, atq, wave, i, g);
    if (i0 + row < s.M) G::store(dtq + a, rt, s.alpha, s.D);
  }
}

// Key side: dk, dtk, dv, dtv of 16 keys, the queries streamed.
// The loads are put in stages here too: the products of q and tq run while the rows of gO and gTO come in, and so on.  With
// all rows of a tile loaded at once and 64-bit addresses for its row scalars the kernel took 200 registers at DP = 64, two
// waves per SIMD: a short sequence's 768 workgroups were a full round and a half-empty one.  It takes 168 now (DP = 96: 241,
// was 304), one wave more.  Both upstream gradients: B4 H12 N256 d64 75.6 us before, 51 now (its products alone: 31); B2 H8
// N1024 d64 278 and 224; B2 H16 N256 d96 66 and 48, d128 82 and 69.  At DP = 128 two waves would spill 24
// registers and cost 73 us.  DP = 32 loads the second stage with the first: 128 registers, four waves (backward of 16384 heads
// of 6 x 6, d 32: 225 us before, 203 with 136 registers, 182 now).
template <int DP, int MODE>
__global__ __launch_bounds__(256, DP <= 32 ? 4 : DP <= 64 ? 3 : DP <= 96 ? 2 : 1) void bwd_col_f32_kernel(
    Shape s, const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const float* __restrict__ tq, const float* __restrict__ tk, const float* __restrict__ tv, const float* __restrict__ lse,
    const float* __restrict__ stats, const float* __restrict__ gO, const float* __restrict__ gTO,
    const float* __restrict__ dsig, const float* __restrict__ sig1, float* __restrict__ dk, float* __restrict__ dtk,
    float* __restrict__ dv, float* __restrict__ dtv) {
  using G = Geo<DP>;
  constexpr bool TAN = MODE != 1, GO = MODE != 2;
  __shared__ f32x4 fixed[4 * G::FIX];  // k, tk, v, tv
  __shared__ __attribute__((aligned(16))) float red[kNW * kR * G::LDR];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nblk = (s.N + kR - 1) / kR, wg = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = wg / nblk, b = bh / s.H, h = bh % s.H, j0 = (wg - bh * nblk) * kR;
  const long long base = b * s.sb + h * s.sh, qbase = b * s.qsb + h * s.qsh;
  const unsigned pitch = (unsigned)(s.qsn * 4);
  G::fix(fixed, k + base, s.sn, j0, s.N, s.D);
  if constexpr (TAN) G::fix(fixed + G::FIX, tk + base, s.sn, j0, s.N, s.D);
  G::fix(fixed + 2 * G::FIX, v + base, s.sn, j0, s.N, s.D);
  if constexpr (TAN) G::fix(fixed + 3 * G::FIX, tv + base, s.sn, j0, s.N, s.D);
  const Head hq = Head::make(q + qbase, s.M, pitch, s.D);
  const Head htq = TAN ? Head::make(tq + qbase, s.M, pitch, s.D) : hq;
  const Head hg = GO ? Head::make(gO + qbase, s.M, pitch, s.D) : hq, htg = TAN ? Head::make(gTO + qbase, s.M, pitch, s.D) : hq;
  const long long rbase = (long long)bh * s.M;
  const Head hl = Head::make(lse + rbase, s.M, 4, 1), hd = Head::make(dsig + rbase, s.M, 4, 1);
  const Head hs = TAN ? Head::make(stats + rbase, s.M, 4, 1) : hl, h1 = TAN ? Head::make(sig1 + rbase, s.M, 4, 1) : hl;
  G geo;
  geo.init(lane, s.D, pitch);
  const int i = geo.i, g = geo.g;
  typename G::Acc ak = G::zero(), atk = G::zero(), av = G::zero(), atv = G::zero();
  __syncthreads();
  for (int i0 = wave * kR; i0 < s.M; i0 += kNW * kR) {
    const unsigned tile = (unsigned)i0 * pitch;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 z = zero, za = zero, zb = zero, da = zero, db = zero, e = zero;
    typename G::Rows qf = geo.rows(hq, tile), tqf, gf, tgf;
    if constexpr (TAN) tqf = geo.rows(htq, tile);
    if constexpr (GO) gf = geo.rows(hg, tile);
    f32x4 vl, vs, vd, v1;  // row scalars of queries i0 + 4g + r
    const auto second = [&] {  // what the second group of products and the pointwise part need
      if constexpr (TAN) tgf = geo.rows(htg, tile);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const unsigned x = (unsigned)(i0 + 4 * g + r) * 4u;
        vl[r] = hl.ld1(x);
        vd[r] = hd.ld1(x);
        if constexpr (TAN) {
          vs[r] = hs.ld1(x);
          v1[r] = h1.ld1(x);
        }
      }
    };
    if constexpr (DP <= 32) second();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < G::NT; ++t) {
      const f32x4 fk = fixed[t * 64 + lane];
      TVM_F32_STEP(z, qf.t[t], fk);
      if constexpr (TAN) {
        const f32x4 ftk = fixed[G::FIX + t * 64 + lane];
        TVM_F32_STEP(zb, qf.t[t], ftk);
        TVM_F32_STEP(za, tqf.t[t], fk);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (DP > 32) second();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < G::NT; ++t) {
      const f32x4 fv = fixed[2 * G::FIX + t * 64 + lane];
      if constexpr (GO) TVM_F32_STEP(da, gf.t[t], fv);
    }
    const typename G::Cols qc = geo.cols(hq, tile, pitch);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < G::NT; ++t) {
      if constexpr (TAN) {
        const f32x4 fv = fixed[2 * G::FIX + t * 64 + lane], ftv = fixed[3 * G::FIX + t * 64 + lane];
        TVM_F32_STEP(db, tgf.t[t], ftv);
        TVM_F32_STEP(e, tgf.t[t], fv);
      }
    }
    typename G::Cols tqc;
    if constexpr (TAN) tqc = geo.cols(htq, tile, pitch);
    __builtin_amdgcn_sched_barrier(0);
    f32x4 p, pd, gz, gzt;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool ok = i0 + 4 * g + r < s.M;
      p[r] = ok ? __expf(z[r] * s.alpha - vl[r]) : 0.f;
      float x = p[r] * ((da[r] + db[r]) - vd[r]);
      if constexpr (TAN) {
        const float n = (za[r] + zb[r]) * s.alpha - vs[r], xt = p[r] * (e[r] - v1[r]);
        x = fmaf(xt, n, x);
        pd[r] = ok ? p[r] * n : 0.f;
        gzt[r] = ok ? xt : 0.f;
      }
      gz[r] = ok ? x : 0.f;
    }
    typename G::Cols gc, tgc;
    if constexpr (GO) gc = geo.cols(hg, tile, pitch);
    __builtin_amdgcn_sched_barrier(0);
    G::out(ak, qc, gz);
    if constexpr (TAN) {
      G::out(atk, qc, gzt);
      tgc = geo.cols(htg, tile, pitch);
      __builtin_amdgcn_sched_barrier(0);
      G::out(ak, tqc, gzt);
    }
    if constexpr (GO) G::out(av, gc, p);
    if constexpr (TAN) {
      G::out(atv, tgc, p);
      G::out(av, tgc, pd);
    }
  }
  const int row = threadIdx.x >> 4;
  const bool rowok = j0 + row < s.N;
  const long long a = base + (long long)(j0 + row) * s.sn;
  auto leave = [&](const typename G::Acc& acc, float* dst, float f) {
    const typename G::Row x = G::gather(red, acc, wave, i, g);
    if (rowok) G::store(dst + a, x, f, s.D);
  };
  leave(ak, dk, s.alpha);
  leave(av, dv, 1.f);
  if constexpr (TAN) {
    leave(atk, dtk, s.alpha);
    leave(atv, dtv, 1.f);
  }
}

template <int DP>
hipError_t fwd_f32_t(const Shape& s, const FwdArgs& a, hipStream_t st) {
  const int grid = (s.M + kR - 1) / kR * s.B * s.H;
  hipLaunchKernelGGL(fwd_f32_kernel<DP>, dim3(grid), dim3(64 * kNW), 0, st, s, (const float*)a.q, (const float*)a.k,
                     (const float*)a.v, (const float*)a.tq, (const float*)a.tk, (const float*)a.tv, (float*)a.o, (float*)a.to,
                     a.lse, a.stats);
  return hipGetLastError();
}
template <int DP, int MODE>
hipError_t bwd_row_f32_t(const Shape& s, const BwdArgs& a, hipStream_t st) {
  const int grid = (s.M + kR - 1) / kR * s.B * s.H;
  hipLaunchKernelGGL((bwd_row_f32_kernel<DP, MODE>), dim3(grid), dim3(64 * kNW), 0, st, s, (const float*)a.q,
                     (const float*)a.k, (const float*)a.v, (const float*)a.tq, (const float*)a.tk, (const float*)a.tv,
                     (const float*)a.o, (const float*)a.to, a.lse, a.stats, (const float*)a.gO, (const float*)a.gTO, a.dsig,
                     a.sig1, (float*)a.dq, (float*)a.dtq);
  return hipGetLastError();
}
template <int DP, int MODE>
hipError_t bwd_col_f32_t(const Shape& s, const BwdArgs& a, hipStream_t st) {
  const int grid = (s.N + kR - 1) / kR * s.B * s.H;
  hipLaunchKernelGGL((bwd_col_f32_kernel<DP, MODE>), dim3(grid), dim3(64 * kNW), 0, st, s, (const float*)a.q,
                     (const float*)a.k, (const float*)a.v, (const float*)a.tq, (const float*)a.tk, (const float*)a.tv, a.lse,
                     a.stats, (const float*)a.gO, (const float*)a.gTO, a.dsig, a.sig1, (float*)a.dk, (float*)a.dtk,
                     (float*)a.dv, (float*)a.dtv);
  return hipGetLastError();
}
template <int DP>
hipError_t bwd_row_f32_m(const Shape& s, const BwdArgs& a, hipStream_t st) {
  return a.mode == 0 ? bwd_row_f32_t<DP, 0>(s, a, st) : a.mode == 1 ? bwd_row_f32_t<DP, 1>(s, a, st) : bwd_row_f32_t<DP, 2>(s, a, st);
}
template <int DP>
hipError_t bwd_col_f32_m(const Shape& s, const BwdArgs& a, hipStream_t st) {
  return a.mode == 0 ? bwd_col_f32_t<DP, 0>(s, a, st) : a.mode == 1 ? bwd_col_f32_t<DP, 1>(s, a, st) : bwd_col_f32_t<DP, 2>(s, a, st);
}

}  // namespace

hipError_t launch_fwd_f32(const Shape& s, const FwdArgs& a, hipStream_t st) {
  return s.D <= 32 ? fwd_f32_t<32>(s, a, st) : s.D <= 64 ? fwd_f32_t<64>(s, a, st) : s.D <= 96 ? fwd_f32_t<96>(s, a, st) : fwd_f32_t<128>(s, a, st);
}
hipError_t launch_bwd_row_f32(const Shape& s, const BwdArgs& a, hipStream_t st) {
  return s.D <= 32 ? bwd_row_f32_m<32>(s, a, st) : s.D <= 64 ? bwd_row_f32_m<64>(s, a, st) : s.D <= 96 ? bwd_row_f32_m<96>(s, a, st) : bwd_row_f32_m<128>(s, a, st);
}
hipError_t launch_bwd_col_f32(const Shape& s, const BwdArgs& a, hipStream_t st) {
  return s.D <= 32 ? bwd_col_f32_m<32>(s, a, st) : s.D <= 64 ? bwd_col_f32_m<64>(s, a, st) : s.D <= 96 ? bwd_col_f32_m<96>(s, a, st) : bwd_col_f32_m<128>(s, a, st);
}

}  // namespace tvm
