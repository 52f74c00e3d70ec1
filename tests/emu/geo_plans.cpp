// Runs the two main transforms of every plan (FCAS_PLAN_LIST), thread by thread
// with the kernels' write / read order, against the direct sum in long double:
// the half-zero columns of pass 1, and the rows of pass 2, shifted by j1 / N1 of
// a sample for the first, second, middle and last row j1 of the plan's own N1
// (not shifted after a middle pass).  Prints one line per plan, precision,
// transform and row: the largest error relative to the largest output.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "plans.hpp"

using namespace fcas;

template <typename Real, int L, int E, class Rad, int I, bool SHIFT, bool HALF, int PAD>
static void stages(std::vector<std::vector<cplx<Real>>>& v, std::vector<cplx<Real>>& buf,
                   const std::vector<GeoSet<Real, L, E, Rad, SHIFT>>& g) {
  if constexpr (I < Rad::count) {
    for (size_t t = 0; t < v.size(); ++t)
      geo_stage<Real, L, E, Rad, I, SHIFT, HALF && I == 0, PAD>(v[t].data(), buf.data(), g[t], (int)t);
    if constexpr (I < Rad::count - 1)
      for (size_t t = 0; t < v.size(); ++t) stage_gather<Real, L, E, PAD>(v[t].data(), buf.data(), (int)t);
    stages<Real, L, E, Rad, I + 1, SHIFT, HALF, PAD>(v, buf, g);
  }
}

// exp(2 pi i m / n) for m < n
struct Roots {
  std::vector<long double> c, s;
  void make(int n) {
    if ((int)c.size() == n) return;
    c.resize(n);
    s.resize(n);
    for (int m = 0; m < n; ++m) {
      const long double a = 6.283185307179586476925286766559L * m / n;
      c[m] = cosl(a);
      s[m] = sinl(a);
    }
  }
};

template <typename Real, int L, int E, class Rad, bool SHIFT, bool HALF, int PAD>
static void check(int plan, const char* what, int j1, int n1) {
  constexpr int P = L / E, K = HALF ? L / 2 : L;
  static Roots roots;
  roots.make(L * n1);
  std::vector<cplx<Real>> x(L), buf(lds_padded_len<PAD>(L));
  unsigned seed = 12345 + plan;
  auto rnd = [&]() { seed = seed * 1664525u + 1013904223u; return (Real)((double)(seed >> 8) / 8388608.0 - 1.0); };
  for (int k = 0; k < K; ++k) x[k] = mk<Real>(rnd(), rnd());
  std::vector<std::vector<cplx<Real>>> v(P, std::vector<cplx<Real>>(E));
  std::vector<GeoSet<Real, L, E, Rad, SHIFT>> g(P);
  for (int t = 0; t < P; ++t) {
    for (int q = 0; q < E; ++q) v[t][q] = x[t + q * P];
    g[t].init(t, j1, n1);
  }
  stages<Real, L, E, Rad, 0, SHIFT, HALF, PAD>(v, buf, g);
  long double worst = 0, top = 0;
  for (int j = 0; j < L; ++j) {
    long double re = 0, im = 0;
    const long long step = ((long long)j * n1 + j1) % ((long long)L * n1);
    long long m = 0;
    for (int k = 0; k < K; ++k) {
      re += x[k].x * roots.c[m] - x[k].y * roots.s[m];
      im += x[k].x * roots.s[m] + x[k].y * roots.c[m];
      m += step;
      if (m >= (long long)L * n1) m -= (long long)L * n1;
    }
    const cplx<Real> y = v[j % P][j / P];
    worst = std::max({worst, fabsl(y.x - re), fabsl(y.y - im)});
    top = std::max({top, fabsl(re), fabsl(im)});
  }
  std::printf("%d %s %s %d %.3Le\n", plan, sizeof(Real) == 4 ? "f32" : "f64", what, j1, worst / top);
}

template <typename Real, class PL>
static void plan_checks(int id) {
  check<Real, PL::N1, PL::E1, typename PL::Rad1, false, true, kPad1>(id, "columns", 0, 1);
  if constexpr (PL::THREE)
    check<Real, PL::N2, PL::E2, typename PL::Rad2, false, false, kPad2>(id, "rows", 0, 1);
  else
    for (int j1 : {0, 1, PL::N1 / 2, PL::N1 - 1})
      check<Real, PL::N2, PL::E2, typename PL::Rad2, true, false, kPad2>(id, "rows", j1, PL::N1);
}

int main() {
#define FCAS_GEO_PLAN(id, ...)       \
  plan_checks<float, PlanF##id>(id); \
  plan_checks<double, PlanD##id>(id);
  FCAS_PLAN_LIST(FCAS_GEO_PLAN)
  return 0;
}
