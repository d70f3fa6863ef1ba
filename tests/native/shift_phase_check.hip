// Check of the phase of a shift (gfc::shift_phase) and of its argument
// (gfc::shift_arg).  As a host program: per W the largest error of hi + lo / pi
// against -2 (n + f) k / W, in half turns, and of the phase against double
// precision.  The kernel below is compiled for the device only, to look at the
// operations that the argument takes there.
#include <cmath>
#include <cstdint>
#include <cstdio>

#include "gfc_device.hpp"

template <int W>
static void check() {
  double arg = 0, phase = 0;
  uint32_t x = 12345u + W;
  for (int i = 0; i < 400; ++i) {
    x = x * 1664525u + 1013904223u;
    const float f = i == 0 ? 0.f : i == 1 ? 1.f : (float)(x >> 8) * (1.f / 16777216.f);
    x = x * 1664525u + 1013904223u;
    const int n = (int)(x >> 20) & (W - 1);
    for (int k = -W / 2; k <= W / 2; ++k) {
      float hi, lo, s, c;
      gfc::shift_arg<W>(f, n, k, &hi, &lo);
      gfc::shift_phase<W>(f, n, k, &s, &c);
      // exact in double: 24 + 8 bits times at most 8 bits, over a power of two
      const double half = -2.0 * ((double)n + (double)f) * k / W;
      const double d = half - hi, turns = 2.0 * std::rint(0.5 * d);
      arg = std::fmax(arg, std::fabs((d - turns) - lo / M_PI));
      const double a = M_PI * (half - 2.0 * std::rint(0.5 * half));
      phase = std::fmax(phase, std::fmax(std::fabs(s - std::sin(a)), std::fabs(c - std::cos(a))));
    }
  }
  std::printf("%d %.6e %.6e\n", W, arg, phase);
}

__global__ void shift_arg_kernel(const float* f, const int* n, float* hi, float* lo) {
  const int i = threadIdx.x;
  gfc::shift_arg<64>(f[i], n[i], i - 32, hi + i, lo + i);
}

int main() {
  check<16>();
  check<32>();
  check<64>();
  check<128>();
  check<256>();
  return 0;
}
