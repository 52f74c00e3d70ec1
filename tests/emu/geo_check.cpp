// Runs the stages of one transform with in-register factors (GeoSet,
// geo_stage), thread by thread with the kernels' write / read order, and
// prints the largest error against the direct sum in long double, relative to
// the largest output: one line per shape.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "fitness_tiles.hpp"

using namespace fcas;

template <typename Real, int L, int E, class Rad, int I, bool SHIFT, bool HALF>
static void stages(std::vector<std::vector<cplx<Real>>>& v, std::vector<cplx<Real>>& buf,
                   const std::vector<GeoSet<Real, L, E, Rad, SHIFT>>& g) {
  if constexpr (I < Rad::count) {
    for (size_t t = 0; t < v.size(); ++t)
      geo_stage<Real, L, E, Rad, I, SHIFT, HALF && I == 0, 4>(v[t].data(), buf.data(), g[t], (int)t);
    if constexpr (I < Rad::count - 1)
      for (size_t t = 0; t < v.size(); ++t) stage_gather<Real, L, E, 4>(v[t].data(), buf.data(), (int)t);
    stages<Real, L, E, Rad, I + 1, SHIFT, HALF>(v, buf, g);
  }
}

template <typename Real, int L, int E, class Rad, bool SHIFT, bool HALF>
static void check(const char* name) {
  static_assert(Rad::product() == L, "radices");
  constexpr int P = L / E, n1 = 48;
  const int j1 = SHIFT ? 37 : 0;
  std::vector<cplx<Real>> x(L), buf(lds_padded_len<4>(L));
  unsigned s = 12345;
  auto rnd = [&]() { s = s * 1664525u + 1013904223u; return (Real)((double)(s >> 8) / 8388608.0 - 1.0); };
  for (int k = 0; k < (HALF ? L / 2 : L); ++k) x[k] = mk<Real>(rnd(), rnd());
  std::vector<std::vector<cplx<Real>>> v(P, std::vector<cplx<Real>>(E));
  std::vector<GeoSet<Real, L, E, Rad, SHIFT>> g(P);
  for (int t = 0; t < P; ++t) {
    for (int q = 0; q < E; ++q) v[t][q] = x[t + q * P];
    g[t].init(t, j1, SHIFT ? n1 : 1);
  }
  stages<Real, L, E, Rad, 0, SHIFT, HALF>(v, buf, g);
  long double worst = 0, top = 0;
  const long double tp = 6.283185307179586476925286766559L;
  for (int j = 0; j < L; ++j) {
    long double re = 0, im = 0;
    for (int k = 0; k < (HALF ? L / 2 : L); ++k) {
      // exp(2 pi i k (j + j1 / n1) / L), the angle reduced exactly
      const long long num = (long long)k * ((long long)j * n1 + j1) % ((long long)L * n1);
      const long double a = tp * num / ((long double)L * n1);
      const long double c = cosl(a), d = sinl(a);
      re += x[k].x * c - x[k].y * d;
      im += x[k].x * d + x[k].y * c;
    }
    const cplx<Real> y = v[j % P][j / P];
    worst = std::max({worst, fabsl(y.x - re), fabsl(y.y - im)});
    top = std::max({top, fabsl(re), fabsl(im)});
  }
  std::printf("%s %s %.3Le\n", name, sizeof(Real) == 4 ? "f32" : "f64", worst / top);
}

#define BOTH(L, E, SHIFT, HALF, ...)                                                    \
  check<float, L, E, Radices<__VA_ARGS__>, SHIFT, HALF>(#L ":" #E ":" #__VA_ARGS__);    \
  check<double, L, E, Radices<__VA_ARGS__>, SHIFT, HALF>(#L ":" #E ":" #__VA_ARGS__);

int main() {
  // pass-1 columns: half-zero inputs, no shift
  BOTH(16, 8, false, true, 8, 2)
  BOTH(32, 8, false, true, 8, 4)
  BOTH(64, 8, false, true, 8, 8)
  BOTH(128, 8, false, true, 8, 8, 2)
  BOTH(256, 8, false, true, 8, 8, 4)
  BOTH(512, 8, false, true, 8, 8, 8)
  BOTH(256, 16, false, true, 16, 16)
  BOTH(512, 16, false, true, 16, 16, 2)
  BOTH(48, 12, false, true, 12, 4)
  BOTH(96, 12, false, true, 12, 4, 2)
  BOTH(192, 12, false, true, 12, 4, 4)
  BOTH(384, 12, false, true, 12, 4, 4, 2)
  // rows: shifted by a fraction of a sample, or not (after a middle pass)
  BOTH(64, 8, true, false, 8, 8)
  BOTH(64, 8, false, false, 8, 8)
  BOTH(128, 8, true, false, 8, 4, 4)
  BOTH(512, 8, true, false, 8, 8, 8)
  BOTH(512, 8, false, false, 8, 8, 8)
  BOTH(768, 12, true, false, 4, 4, 4, 4, 3)
  BOTH(1024, 16, true, false, 16, 8, 8)
  BOTH(1024, 16, true, false, 16, 16, 4)
  BOTH(1024, 8, true, false, 8, 8, 8, 2)
  return 0;
}
