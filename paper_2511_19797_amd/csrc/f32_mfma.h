// Launchers of the float32 matrix-core kernels (f32_mfma.hip) and which calls they take; chosen inside launch_*_generic.
#pragma once
#include "tvm_common.h"

namespace tvm {

// OR-ed into the dtype of a launch_*_generic call: plain-ALU kernels whatever the shape (TVMATTN_FLAG_PLAIN_ALU).
constexpr int kPlainAlu = 0x100;

// What these kernels can read: rows are addressed by 32-bit byte offsets within a head (a ragged last tile of 16 included), and
// 16-byte loads take whole groups of four columns (pitches and bases are 16-byte multiples for every call).
inline bool f32_mfma_reads(const Shape& s, int dtype) {  // false for a dtype with kPlainAlu
  constexpr long long kMax = (1ll << 31) - 1;
  const auto fits = [](int rows, long long pitch) { return pitch <= kMax / 4 / ((long long)rows + 16); };
  return dtype == 0 && s.D % 4 == 0 && s.D <= 128 && fits(s.N, s.sn) && fits(s.M, s.qsn);
}
// Of those calls the plain-ALU kernels keep the ones with a handful of rows: a tile here is 16 rows whatever there is of them, and
// a workgroup sets up and adds four waves' accumulators for it, where a plain-ALU workgroup is four rows.  Measured, heads = B * H
// (us, plain / here, graphs of calls back to back; d = head dim):
//   forward, 1 x 1:    1 head, d 16 3.5 / 3.9;  16384 heads: d 16 29 / 43, d 64 65 / 88, d 128 126 / 297
//            4 x 4:    2048 heads: d 16 8.4 / 8.3, d 32 10.8 / 8.7, d 64 15.4 / 12.8, d 128 28 / 34;  16384: d 64 88 / 98
//            16 x 1:   1 head, d 128 7.3 / 7.6
//            1 x 16:   2048 heads, d 128 53 / 43
//   backward, both gradients, 1 x 1:  1 head: d 4 8.4 / 9.0, d 64 21 / 12;  16384 heads: d 16 104 / 148, d 64 303 / 326
//            4 x 4:    1 head: d 4 9.4 / 9.0, d 16 12.0 / 9.1;  16384 heads: d 16 181 / 167, d 32 272 / 170, d 64 469 / 332,
//                      d 128 1023 / 1224      6 x 6: here (d 4 on one head 10.5 / 8.8)
//   backward, gO alone: here at every size (1 x 1: 16384 heads, d 128 458 / 385)
// The backward's lines are on the plain kernels' side of where the times meet (4 x 4: d 96 on 1024 heads 57 / 38, d 16 on 16384
// above; 4 x 1, d 64 on 4096 heads 106 / 86): with so few rows the plain kernels' sums are the more exact ones.  Relative error of
// dv against 64 bits, plain / here: 4 x 4, d 96 2.1e-7 / 3.3e-7; 4 x 1 0.7e-7 / 3.8e-7 (dq, dk: 5e-7 on both).
inline bool f32_mfma_fwd(const Shape& s, int dtype) {
  if (!f32_mfma_reads(s, dtype)) return false;
  const long long heads = (long long)s.B * s.H;
  if (s.M <= 4 && s.N <= 4) return !(s.D <= 16 || s.D > 64 || s.N == 1 || heads >= 4096 || (s.N == 2 && s.D > 32));
  if (s.N <= 2 && heads * s.M <= 1024) return s.D > 16 && s.D <= 32;
  return !(s.D > 96 && heads >= 4096 && ((s.M <= 4 && s.N <= 16) || (s.M <= 8 && s.N <= 8)));
}
inline bool f32_mfma_bwd(const Shape& s, int dtype, int mode) {
  if (!f32_mfma_reads(s, dtype)) return false;
  if (mode == 1 || s.M > 4 || s.N > 4) return true;
  const long long heads = (long long)s.B * s.H;
  const bool one = s.M == 1 && s.N == 1;
  if (heads >= 4096) return !(s.D <= 16 || s.D > 64 || one || (s.D > 32 && (s.M == 1 || s.N == 1)));
  return !(s.D <= 4 || (s.D <= 8 && one) || (s.D <= 16 && one && heads >= 2048) || (s.D > 64 && heads >= 1024) ||
           (s.D > 96 && heads >= 512));
}
hipError_t launch_fwd_f32(const Shape& s, const FwdArgs& a, hipStream_t st);
hipError_t launch_bwd_row_f32(const Shape& s, const BwdArgs& a, hipStream_t st);  // forms the row scalars itself (no launch_bwd_pre)
hipError_t launch_bwd_col_f32(const Shape& s, const BwdArgs& a, hipStream_t st);  // after the former

}  // namespace tvm
