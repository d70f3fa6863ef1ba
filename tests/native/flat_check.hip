// Check of the polynomial for 2^x on [-1, 0] (gfc::kFlat): prints its largest
// relative error and its mean error in double precision.
#include <cmath>
#include <cstdio>

#include "gfc_device.hpp"

int main() {
  constexpr int N = 1 << 20;
  double worst = 0, mean = 0;
  for (int i = 0; i <= N; ++i) {
    const double x = -(double)i / N;
    double p = gfc::kFlat[gfc::kFlatDeg];
    for (int j = gfc::kFlatDeg - 1; j >= 0; --j) p = p * x + gfc::kFlat[j];
    const double e = p / std::exp2(x) - 1.0;
    worst = std::fmax(worst, std::fabs(e));
    mean += e / (N + 1);
  }
  std::printf("%.6e %.6e\n", worst, mean);
  return 0;
}
