// Largest error of the factors of passes 1 and 2 (geo_factors) against the
// same numbers in long double, in units of the type's half spacing at one
// (2^-24, 2^-53): one line per radix and precision, over the ratios
// s = exp(2 pi i num / den) of stages of up to 262144 samples.
#include <algorithm>
#include <cmath>
#include <cstdio>

#include "fft_core.hpp"

using namespace fcas;

template <int R, typename T>
static void check(const char* prec) {
  const long double tp = 6.283185307179586476925286766559L, unit = sizeof(T) == 4 ? 0x1p-24L : 0x1p-53L;
  long double worst = 0;
  for (int n : {64, 512, 768, 1024 * 48, 1024 * 192, 512 * 384, 512 * 512})
    for (int num = 0, den = n; num < den / R; num += 1 + num / 61) {
      cplx<T> w[geo_count(R)];
      geo_factors<R>(w, num, den);
      for (int f = 0; f < geo_count(R); ++f) {
        const long double a = tp * ((long double)(geo_mul(R, f) * num) / den + geo_off(R, f) / 16.0L);
        worst = std::max({worst, fabsl(w[f].x - cosl(a)), fabsl(w[f].y - sinl(a))});
      }
    }
  std::printf("%d %s %.3Lf\n", R, prec, worst / unit);
}

int main() {
#define BOTH(R)         \
  check<R, float>("f32"); \
  check<R, double>("f64");
  BOTH(2) BOTH(3) BOTH(4) BOTH(8) BOTH(16)
  return 0;
}
