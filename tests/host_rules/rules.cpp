// The host-side rules that choose kernels and cut work, for the tests: one query per input line, one answer per output line.
#include <cstdio>
#include <cstring>

#include "../../paper_2511_19797_amd/csrc/f32_mfma.h"
#include "../../paper_2511_19797_amd/csrc/fwd_few.h"
#include "../../paper_2511_19797_amd/csrc/linear_plan.h"
#include "../../paper_2511_19797_amd/csrc/tvm_common.h"

using namespace tvm;

int main() {
  char what[32];
  long long a[8];
  char line[256];
  while (std::fgets(line, sizeof line, stdin)) {
    const int n = std::sscanf(line, "%31s %lld %lld %lld %lld %lld %lld %lld %lld", what, a, a + 1, a + 2, a + 3, a + 4, a + 5, a + 6,
                              a + 7) - 1;
    if (!std::strcmp(what, "part_rows") && n == 3) {  // rows z parts
      const PartRows p = part_rows((int)a[0], (int)a[1], (int)a[2]);
      std::printf("%d %d\n", p.first, p.end);
    } else if (!std::strcmp(what, "bwd_splits") && n == 4) {  // heads fixed streamed tensors
      std::printf("%d\n", bwd_splits(a[0], (int)a[1], (int)a[2], (int)a[3]));
    } else if (!std::strcmp(what, "fwd_few") && n == 4) {  // heads M N D
      Shape s{};
      s.B = 1;
      s.H = (int)a[0];
      s.M = (int)a[1];
      s.N = (int)a[2];
      s.D = (int)a[3];
      std::printf("%d\n", fwd_few_rows(s) ? 1 : 0);
    } else if (!std::strcmp(what, "linear") && n == 3) {  // R K F: tile shapes of y, grad x, grad W (0 .. 3), splits of grad W
      const int R = (int)a[0], K = (int)a[1], F = (int)a[2];
      const DwPlan w = plan_dw(F, K, R, dw_splits(F, K, R));
      std::printf("%d %d %d %d\n", pick_shape(false, 2, R, F, K), pick_shape(true, 2, R, K, F), w.shape, w.splits);
    } else if (!std::strcmp(what, "f32") && n == 4) {  // heads M N D: matrix cores in the forward, the backward, with gO alone
      Shape s{};
      s.B = 1;
      s.H = (int)a[0];
      s.M = (int)a[1];
      s.N = (int)a[2];
      s.D = (int)a[3];
      s.sn = s.qsn = s.D;
      std::printf("%d %d %d\n", f32_mfma_fwd(s, 0) ? 1 : 0, f32_mfma_bwd(s, 0, 0) ? 1 : 0, f32_mfma_bwd(s, 0, 1) ? 1 : 0);
    } else if (!std::strcmp(what, "rows") && n == 4) {  // tangent heads rows D
      std::printf("%d\n", leave_as_rows(a[0] != 0, a[1] * ((a[2] + 127) / 128), (int)a[2], (int)a[3]) ? 1 : 0);
    } else {
      std::printf("? %s", line);
    }
  }
}
