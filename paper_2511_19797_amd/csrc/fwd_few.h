// Forward for few query rows (fwd_few.hip): which calls it takes.
#pragma once
#include "tvm_common.h"

namespace tvm {

// A workgroup there is 32 query rows, one to a CU (up to d = 32 three fit its LDS): its time goes up with every 256 of them, while
// fwd_mfma.hip takes the same time until its workgroups of 128 or 256 rows fill the chip (2048 such blocks of 32).  The lines
// lie at the last whole 256 blocks where this one is ahead by more than 5 % (us at d = 64, blocks of 32 rows: fwd_mfma.hip /
// here):
//    256 keys:   256: 12 / 12 (both the host's time)    512: 12 / 14
//   1024 keys:   128: 38 / 12    256: 39 / 13    512: 40 / 24    768: 40 / 38    (d = 128: 768: 52 / 57)
//   4096 keys:   128: 136 / 32   256: 137 / 36   512: 137 / 69   768: 138 / 101  1024: 138 / 132  (d = 128: 768: 179 / 170)
inline bool fwd_few_rows(const Shape& s) {
  if (s.N < 128) return false;
  const long long blocks = (long long)s.B * s.H * (((long long)s.M + 31) / 32);
  return blocks <= (s.N < 512 ? 256 : s.N < 2048 || s.D > 96 ? 512 : 768);
}
hipError_t launch_fwd_few(const Shape& s, const FwdArgs& a, hipStream_t st);

}  // namespace tvm
