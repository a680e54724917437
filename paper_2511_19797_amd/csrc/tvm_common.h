// Shared device-side types for the tvmattn kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tvm {

typedef __bf16 bf16;

// Logical problem: M queries and N keys per (batch, head), head dim D.  Key-side tensors (k, v, tk, tv and their
// gradients) are [B,H,N,D] with element strides sb, sh, sn; query-side tensors (q, tq, o, to, gO, gTO, dq,
// dtq) are [B,H,M,D] with qsb, qsh, qsn; lse, stats and the workspace row vectors are [B,H,M] contiguous.
struct Shape {
  int B, H, N, D;
  float alpha;          // softmax scale actually used (already resolved from desc.scale)
  long long sb, sh, sn; // element strides, key side
  int M;                // queries (= N for self-attention)
  long long qsb, qsh, qsn;  // element strides, query side
};

__device__ __forceinline__ float ldf(const float* p) { return *p; }
__device__ __forceinline__ float ldf(const bf16* p) { return (float)*p; }
__device__ __forceinline__ void stf(float* p, float x) { *p = x; }
__device__ __forceinline__ void stf(bf16* p, float x) { *p = (bf16)x; }  // round-to-nearest-even

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
  return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

// Host-side launchers (defined in the kernel translation units; all return hipGetLastError()).
struct FwdArgs {
  const void *q, *k, *v, *tq, *tk, *tv;
  void *o, *to;
  float *lse, *stats;
  // forward with the query side's normalisation folded in (launch_fwd_mfma_qnorm only): q, tq are the rows before the
  // norm; the gain, eps, and where the normalised rows go
  const float* ngq = nullptr;
  float neps = 0.f;
  void *qn = nullptr, *tqn = nullptr;
};
struct BwdArgs {
  const void *q, *k, *v, *tq, *tk, *tv, *o, *to;
  const float *lse, *stats;
  const void *gO, *gTO;
  void *dq, *dk, *dv, *dtq, *dtk, *dtv;
  float *dsig;  // workspace: delta + Sigma_2 per row
  float *sig1;  // workspace: Sigma_1 per row
  float *lse2;  // workspace: lse in log2 units per row (written and read by the hand-scheduled kernels only)
  int mode;     // upstream gradients that exist: 0 both, 1 gO only (gTO null), 2 gTO only (gO null)
  // backward through the QK-norm in the epilogues (launch_bwd_*_pipe_qknorm only): the rows before the
  // normalisation, the gains, eps, and one partial gain-gradient row per workgroup of the two kernels
  const void *nq = nullptr, *ntq = nullptr, *nk = nullptr, *ntk = nullptr;
  const float *ngq = nullptr, *ngk = nullptr;
  float neps = 0.f;
  float *npart_q = nullptr, *npart_k = nullptr;
  // streamed side in several parts (bwd_splits): float32 partial gradients [parts][tensors][B*H*rows][D], null: one part
  float* part = nullptr;
};
// Parts that the streamed side of a backward kernel is cut into, so that few rows occupy the chip all the same: `fixed` rows
// per (batch, head) in workgroups of 128, `streamed` rows per (batch, head).  Every part is a workgroup of its own per 128
// rows and leaves float32 sums of its tensors, which bwd_part_sum.hip adds in order.  Only where the workgroups of all
// parts fit the 256 CUs at once (one each: a workgroup's LDS stages fill a CU), and at least four tiles of 64 rows to a
// part.  Of those the fewest tiles one after the other, what the sum costs counted in tiles (1.5 - 2 us each): a launch
// and the first tiles' latency are worth four, the partial sums of 256 workgroups two for each tensor (both ways at 5 TB/s).
// Below 1024 streamed rows there is less than that to be had.  Whole backward (us, whole / in parts): one head of 1024, d = 64
// 62 / 38; one head of 4096 207 / 71; one of 8192 402 / 172; four of 4096 210 / 169; 16 heads of 1024, d = 72 in two parts 77 / 79
// (whole by this rule).  Calls with gO alone take the parts of the call with both gradients, by whose tensors the rule weighs
// the sum and the workspace is sized: twice what they leave, so they are cut in fewer parts than would pay (eight heads of
// 1024, d = 64: 46 / 45).
constexpr int kBwdCUs = 256, kBwdFix = 128;
inline int bwd_splits(long long heads, int fixed, int streamed, int tensors) {
  const long long wgs = heads * (((long long)fixed + kBwdFix - 1) / kBwdFix);
  const int tiles = (int)(((long long)streamed + 63) / 64);
  if (tiles < 16 || 2 * wgs > kBwdCUs) return 1;
  int best = 1, best_cost = tiles;
  for (int p = 2; p <= tiles / 4 && p * wgs <= kBwdCUs; ++p) {
    const int cost = (tiles + p - 1) / p + 4 + (int)(2 * tensors * p * wgs / kBwdCUs);
    if (cost < best_cost) {
      best_cost = cost;
      best = p;
    }
  }
  return best;
}
// Rows first .. end-1 of part z of `rows` rows cut into `parts` parts: whole tiles of 64, floor(z tiles / parts) of them
// before part z.  The product z tiles does not fit 32 bits from 2^29 rows on, so the quotient is taken apart first.
struct PartRows {
  int first, end;
};
__host__ __device__ inline PartRows part_rows(int rows, int z, int parts) {
  const unsigned tiles = ((unsigned)rows + 63u) >> 6, n = (unsigned)parts, q = tiles / n, r = tiles - q * n;
  const unsigned t0 = (unsigned)z * q + (unsigned)z * r / n, t1 = ((unsigned)z + 1u) * q + ((unsigned)z + 1u) * r / n;
  return PartRows{(int)(t0 * 64u), t1 == tiles ? rows : (int)(t1 * 64u)};
}
// The generic-order kernels of the backward: whether one of `wgs` workgroups on `rows` fixed rows per head stores its results as
// whole rows through LDS rather than straight from the accumulators, 8 bytes per lane and row.  Whole rows halve the store
// instructions' cost, but every wave stages all its padded columns, also for rows and columns that do not exist: they pay where
// the chip is full or nothing is padded (whole backward, us, straight / whole rows; one workgroup per 128 rows of a head):
//   64 rows:   64 heads d = 72 10.0 / 10.8, d = 64 10.3 / 10.2;  1024 heads d = 72 31.9 / 32.8, d = 64 28.0 / 26.7, d = 128 49.8 / 46.4
//   96 rows:   192 heads d = 56 12.4 / 12.0, d = 80 14.2 / 13.7;  256 heads d = 48 12.2 / 11.9;  64 heads d = 112 the same
//   128 rows:  16 heads d = 40 +7 %, d = 72 12.8 / 13.1, d = 64 14.5 / 13.1;  256 heads d = 40 -3 %, d = 72 18.3 / 16.8;
//              2048 heads d = 72 103 / 90, d = 64 87 / 74, d = 8 26.4 / 28.0
//   512 rows:  1 head d = 48 +7 %, d = 72 27.3 / 27.5;  192 heads d = 48 -10 %;  512 heads d = 16 +2 %
// With the tangent (head dims above 96, 64 rows or fewer on the other side) from 96 rows on: one other-side row, d = 104, 256
// heads of 96 rows -6 %, of 65 the same; 64 other-side rows, d = 128, any number of heads of 128 rows -7 %.
inline bool leave_as_rows(bool tangent, long long wgs, int rows, int D) {
  if (rows < (tangent ? 96 : 64) || D <= 24) return false;
  if (D > 120) return true;
  if (rows < 96) return wgs >= (D >= 112 ? 256 : 512) && (D == 64 || D >= 80);
  if (D % 32 == 0 || D >= 112) return rows >= 128 || wgs >= 192;
  return wgs >= (D < 56 ? 256 : rows < 128 ? 192 : 128);
}
// Bytes of the partial gradients of the larger of the two backward kernels (0: neither is cut).  At most
// 256 workgroups x 128 rows x 96 columns x 4 tensors of float32 = 48 MiB (128 columns x 2 tensors: 32 MiB).
inline size_t bwd_part_bytes(const Shape& s, int dtype) {
  if (dtype != 1 || s.D > 128 || s.D % 8 != 0) return 0;
  const long long heads = (long long)s.B * s.H;
  const int ct = s.D > 96 ? 2 : 4;  // tensors of a key-side kernel: above 96 it runs as two passes, one after the other
  const int rs = bwd_splits(heads, s.M, s.N, 2), cs = bwd_splits(heads, s.N, s.M, ct);
  const size_t row = rs > 1 ? (size_t)rs * 2 * heads * s.M * s.D * sizeof(float) : 0;
  const size_t col = cs > 1 ? (size_t)cs * ct * heads * s.N * s.D * sizeof(float) : 0;
  return row > col ? row : col;
}
constexpr size_t kBwdPartMax = (size_t)kBwdCUs * kBwdFix * 96 * 4 * sizeof(float);

hipError_t launch_fwd_generic(const Shape& s, int dtype, const FwdArgs& a, hipStream_t st);
hipError_t launch_bwd_pre(const Shape& s, int dtype, const BwdArgs& a, hipStream_t st);
hipError_t launch_bwd_col_generic(const Shape& s, int dtype, const BwdArgs& a, hipStream_t st);
hipError_t launch_bwd_row_generic(const Shape& s, int dtype, const BwdArgs& a, hipStream_t st);

// bf16 matrix-core paths; `supported` says whether the shape is one they take.
bool mfma_supported(const Shape& s, int dtype);
hipError_t launch_fwd_mfma(const Shape& s, const FwdArgs& a, hipStream_t st);
hipError_t launch_fwd_mfma_qnorm(const Shape& s, const FwdArgs& a, hipStream_t st);
hipError_t launch_bwd_col_mfma(const Shape& s, const BwdArgs& a, hipStream_t st);
hipError_t launch_bwd_row_mfma(const Shape& s, const BwdArgs& a, hipStream_t st);
hipError_t launch_bwd_col_onesided(const Shape& s, const BwdArgs& a, hipStream_t st);  // a.mode 1 or 2, any head dim
hipError_t launch_bwd_row_onesided(const Shape& s, const BwdArgs& a, hipStream_t st);
hipError_t launch_bwd_row_pipe(const Shape& s, const BwdArgs& a, hipStream_t st);  // head dims up to 96
hipError_t launch_bwd_col_pipe(const Shape& s, const BwdArgs& a, hipStream_t st);  // head dims up to 96, after the former
hipError_t launch_bwd_row_pipe_qknorm(const Shape& s, const BwdArgs& a, hipStream_t st);  // the same two with the QK-norm's
hipError_t launch_bwd_col_pipe_qknorm(const Shape& s, const BwdArgs& a, hipStream_t st);  // backward in their epilogues
// Adds the partial gradients of `parts` parts in order, scales and rounds them: `tensors` outputs [B,H,rows,D] (query-side or
// key-side strides), the first `scaled` of them times alpha (bwd_part_sum.hip).
hipError_t launch_bwd_part_sum(const Shape& s, bool query_side, const float* part, int parts, int tensors, int scaled,
                               void* const* out, hipStream_t st);
hipError_t launch_gain_grad_sum(const float* part_q, int rows_q, float* gg_q, const float* part_k, int rows_k, float* gg_k,
                                int D, hipStream_t st);  // adds partial gain-gradient rows in order (qknorm.hip)


// RMSNorm with gain as QK-norm, with tangent (qknorm.hip).  One side = the rows of q (and tq) or of k (and tk).
struct NormSide {
  const void *x, *tx;      // inputs [B,H,n,D]
  const float* g;          // gain [D]
  const void *gy, *gty;    // backward: upstream gradients of the normalised tensor and of its tangent
  void *y, *ty;            // forward: outputs; backward: gradients of x and tx
  float* part;             // backward: per-workgroup partial sums of the gain gradient [nwg][D]
  float* gg;               // backward: gain gradient [D]
  int n;                   // rows per (batch, head)
  long long sb, sh, sn;    // element strides
  int nwg;                 // workgroups that work on this side
};
struct NormArgs {
  NormSide side[2];
  int B, H, D;
  float eps;
};
constexpr int kNormRowsPerWg = 16;   // rows a workgroup works on at a time (16 lanes each)
constexpr int kNormMaxWg = 1024;     // workgroups per side at most (they stride over the rows; two sides fill the chip)
hipError_t launch_qknorm_fwd(const NormArgs& a, int dtype, hipStream_t st);
hipError_t launch_qknorm_bwd(const NormArgs& a, int dtype, hipStream_t st);


// Normalised adaptive-layer-norm modulation with tangent (adaln.hip).
struct AdalnArgs {
  const void *x, *tx, *gy, *gty;    // [B,T,C] dtype, contiguous (gy, gty: backward only)
  const void *gres = nullptr, *gtres = nullptr;  // backward, optional (both or neither): added to the gradients of x, tx
  const float *a, *ta, *b, *tb;     // [B,C] float32
  void *y, *ty;                     // forward: outputs; backward: gradients of x and tx
  float* part;                      // backward workspace [B][nwg][4][C]: per-workgroup sums over tokens
  float *ga, *gta, *gb, *gtb;       // backward: gradients of a, ta, b, tb
  int B, T, C, nwg;                 // nwg: workgroups per batch element
  float eps;
};
// Normalised gate of a residual branch: z = x + RMSNorm^-(c) o h with tangent, and its backward.
struct GateArgs {
  const void *x, *tx, *h, *th;      // [B,T,C] dtype, contiguous (x, tx: forward only)
  const void *gz, *gtz;             // backward: upstream gradients, [B,T,C] dtype
  const float *c, *tc;              // [B,C] float32
  void *z, *tz;                     // forward: outputs; backward: gradients of h and th
  float* part;                      // backward workspace [B][nwg][2][C]: per-workgroup sums over tokens
  float *gc, *gtc;                  // backward: gradients of c, tc
  int B, T, C, nwg;
  float eps;
};
hipError_t launch_gate_fwd(const GateArgs& a, int dtype, hipStream_t st);
hipError_t launch_gate_bwd(const GateArgs& a, int dtype, hipStream_t st);
bool adaln_supported(int C, int dtype);
// The MLP's activation with tangent (n elements per tensor, a whole number of 16-byte chunks).
hipError_t launch_gelu_fwd(long long n, int dtype, const void* u, const void* tu, void* a, void* ta, hipStream_t st);
hipError_t launch_gelu_bwd(long long n, int dtype, const void* u, const void* tu, const void* ga, const void* gta,
                           void* gu, void* gtu, hipStream_t st);
// Linear layer on a token and its tangent (linear.hip): bf16 only, K and F multiples of 32.
// ldx, ldy: row pitch in elements of the [R,K] tensors (x, tx, gx, gtx) and of the [R,F] tensors (y, ty, gy, gty).
bool linear_supported(int R, int K, int F, long long ldx, long long ldy, int dtype);
size_t linear_bwd_workspace_bytes(int R, int K, int F);
hipError_t launch_linear_fwd(int R, int K, int F, long long ldx, long long ldy, const void* x, const void* tx,
                             const void* w, const void* bias, void* y, void* ty, hipStream_t st);
hipError_t launch_linear_bwd(int R, int K, int F, long long ldx, long long ldy, const void* x, const void* tx,
                             const void* w, const void* gy, const void* gty, void* gx, void* gtx, void* gw, void* gbias,
                             void* workspace, hipStream_t st);
int adaln_wgs(int B, int T, bool backward, bool gate);  // workgroups per batch element of a token kernel
hipError_t launch_adaln_fwd(const AdalnArgs& a, int dtype, hipStream_t st);
hipError_t launch_adaln_bwd(const AdalnArgs& a, int dtype, hipStream_t st);

}  // namespace tvm
