// Host harness for polar_rot (the rigid update's Kabsch rotation of a
// well-conditioned matrix): reads matrices (9 values, row-major) from stdin,
// prints its status (1/0) and the rotation (9, row-major; zeros when 0).
#include <cstdio>

#include "../../paper_1902_01061_amd/csrc/common.h"

int main() {
  double A[9];
  for (;;) {
    for (double& x : A)
      if (std::scanf("%lf", &x) != 1) return 0;
    double R[9] = {0};
    const bool ok = sgr::polar_rot(A, R);
    std::printf("%d", ok ? 1 : 0);
    for (double x : R) std::printf(" %.17g", x);
    std::printf("\n");
  }
}
