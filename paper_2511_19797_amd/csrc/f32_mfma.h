// Launchers of the float32 matrix-core kernels (f32_mfma.hip), chosen inside launch_*_generic.
#pragma once
#include "tvm_common.h"

namespace tvm {

// OR-ed into the dtype of a launch_*_generic call: plain-ALU kernels whatever the shape (TVMATTN_FLAG_PLAIN_ALU).
constexpr int kPlainAlu = 0x100;

bool f32_mfma_supported(const Shape& s, int dtype);  // false for a dtype with kPlainAlu
hipError_t launch_fwd_f32(const Shape& s, const FwdArgs& a, hipStream_t st);
hipError_t launch_bwd_row_f32(const Shape& s, const BwdArgs& a, hipStream_t st);  // forms the row scalars itself (no launch_bwd_pre)
hipError_t launch_bwd_col_f32(const Shape& s, const BwdArgs& a, hipStream_t st);  // after the former

}  // namespace tvm
