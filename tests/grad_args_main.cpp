// The gradient GEMM stores rows by eights: an output that ends elsewhere is refused before anything is launched.
#include <cstdio>

#include "fused_shared.h"

int main() {
  for (int rows = 1; rows < 24; ++rows) {
    if (rows % 8 == 0) continue;
    adwin::GradArgs a{};
    a.H = 64; a.k_rows = 64; a.nk_total = 1; a.row_tiles = a.h_tiles = a.ksplit = a.half_tiles = 1;
    a.out_rows = rows;
    if (adwin::launch_grad_gemm(a, nullptr) != hipErrorInvalidValue) {
      std::printf("%d rows accepted\n", rows);
      return 1;
    }
  }
  std::puts("refused");
  return 0;
}
