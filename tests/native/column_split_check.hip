// Host-side check of the adjoint's column split (gfc::ColumnSplit): per W the
// rms over galaxy positions near the middle and low columns of the phase error
// that 64 rows of a smooth image have in common, and the largest error of the
// packed column 0.
#include <cmath>
#include <complex>
#include <cstdint>
#include <cstdio>

#include "gfc_device.hpp"
#include "bwd_common.hpp"

using C = std::complex<double>;

static uint32_t state = 12345u;
static double uniform() {
  state = state * 1664525u + 1013904223u;
  return (state >> 8) * (1.0 / 16777216.0);
}
static C at(gfc::ColumnSplit s, C z, C zr, float2* zf, float2* zrf) {
  *zf = make_float2((float)z.real(), (float)z.imag());
  *zrf = make_float2((float)zr.real(), (float)zr.imag());
  const float2 r = s.at(*zf, *zrf);
  return C(r.x, r.y);
}

template <int W>
static void check() {
  double sq = 0, worst0 = 0;
  long count = 0;
  for (int it = 0; it < 400; ++it) {
    const float x = (float)(W / 2 + uniform());
    const int n = (int)std::floor(x);
    const float f = x - (float)n;
    for (int c = 0; c <= W / 8; c += c < 8 ? 1 : W / 64) {
      const int t = c * (GFC_TW_N / W);
      const gfc::ColumnSplit s = gfc::column_split<W>(f, n & (W - 1), c, make_float2(gfc::kTwCos[t], -gfc::kTwSin[t]));
      const double turns = std::fmod((double)x * c / W, 1.0);
      const C tw = C(0, -1) * std::exp(C(0, -2 * M_PI * c / W)), phase = std::exp(C(0, 2 * M_PI * turns)) / ((double)W * W);
      double mean = 0;
      for (int row = 0; row < 64; ++row) {
        const C e = std::polar(0.5 + uniform(), 2 * M_PI * uniform());
        float2 z, zr;
        if (c == 0) {  // Z[0] = (even sum, odd sum); both columns of a row with these sums
          const C got = at(s, e, e, &z, &zr);
          const C want = C(z.x + (double)z.y, z.x - (double)z.y) / ((double)W * W);
          worst0 = std::fmax(worst0, std::abs(got - want) / std::abs(want));
          continue;
        }
        // even and odd pixels of a smooth row: tw (Z - conj Z') = Z + conj Z'
        const C got = at(s, e * (1.0 + std::conj(tw)), std::conj(e * (1.0 - std::conj(tw))), &z, &zr);
        const C a(z.x, z.y), b(zr.x, -(double)zr.y);
        mean += std::arg(got / (phase * (a + b + tw * (a - b)))) / 64;
      }
      if (c) sq += mean * mean, ++count;
    }
  }
  std::printf("%d %.6e %.6e\n", W, std::sqrt(sq / count), worst0);
}

int main() {
  check<64>();
  check<128>();
  check<256>();
  return 0;
}
