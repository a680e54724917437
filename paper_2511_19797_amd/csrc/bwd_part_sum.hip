// Second half of a backward whose streamed side was cut into parts (bwd_splits in tvm_common.h): adds the parts'
// float32 sums in order, scales, rounds once to bf16 and writes the gradients with the caller's strides.
//
// Bound by its bytes, which were written a moment before and mostly come from the caches: 8 columns per thread, the
// loads of eight parts in flight.  One head of 4096, d = 64: 5 us for two tensors of 8 parts, 7 us for four.  With it the query
// side of that call takes 28 + 5 us (94 whole) and the key side 33 + 7 us (115 whole).
#include "mfma_tiles.h"

namespace tvm {
namespace {

struct PartSumArgs {
  const float* part;  // [parts][tensors][heads * rows][D]
  bf16* out[4];
  long long one;      // heads * rows * D
  int parts, tensors, scaled, H, rows, D;  // scaled: how many of the tensors, from the first on, are scaled by alpha
  long long sb, sh, sn;
  float alpha;
};

__global__ __launch_bounds__(256) void bwd_part_sum_kernel(PartSumArgs g) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  const long long e = ((long long)blockIdx.x * 256 + threadIdx.x) * 8;
  if (e >= g.one) return;
  const int t = blockIdx.y;  // tensor
  const float* src = g.part + t * g.one + e;
  const long long pitch = g.tensors * g.one;
  f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
  int p = 0;
  for (; p + 8 <= g.parts; p += 8) {
    f32x4 u[8], v[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      u[x] = *reinterpret_cast<const f32x4*>(src + (p + x) * pitch);
      v[x] = *reinterpret_cast<const f32x4*>(src + (p + x) * pitch + 4);
    }
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      a += u[x];
      b += v[x];
    }
  }
  for (; p < g.parts; ++p) {
    a += *reinterpret_cast<const f32x4*>(src + p * pitch);
    b += *reinterpret_cast<const f32x4*>(src + p * pitch + 4);
  }
  const float f = t < g.scaled ? g.alpha : 1.f;
  bf16x8 o;
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    o[x] = (bf16)(a[x] * f);
    o[4 + x] = (bf16)(b[x] * f);
  }
  const long long r = e / g.D;  // (D is a multiple of 8: the eight columns belong to one row)
  const int c = (int)(e - r * g.D), bh = (int)(r / g.rows), i = (int)(r - (long long)bh * g.rows);
  const int bb = bh / g.H, h = bh - bb * g.H;
  bf16* const dst = t == 0 ? g.out[0] : t == 1 ? g.out[1] : t == 2 ? g.out[2] : g.out[3];
  *reinterpret_cast<bf16x8*>(dst + bb * g.sb + h * g.sh + i * g.sn + c) = o;
}

}  // namespace

hipError_t launch_bwd_part_sum(const Shape& s, bool query_side, const float* part, int parts, int tensors, int scaled,
                               void* const* out, hipStream_t st) {
  PartSumArgs g{};
  g.part = part;
  for (int t = 0; t < tensors; ++t) g.out[t] = (bf16*)out[t];
  g.H = s.H;
  g.rows = query_side ? s.M : s.N;
  g.D = s.D;
  g.one = (long long)s.B * s.H * g.rows * s.D;
  g.parts = parts;
  g.tensors = tensors;
  g.scaled = scaled;
  g.sb = query_side ? s.qsb : s.sb;
  g.sh = query_side ? s.qsh : s.sh;
  g.sn = query_side ? s.qsn : s.sn;
  g.alpha = s.alpha;
  hipLaunchKernelGGL(bwd_part_sum_kernel, dim3((unsigned)((g.one / 8 + 255) / 256), (unsigned)tensors), dim3(256), 0, st, g);
  return hipGetLastError();
}

}  // namespace tvm
