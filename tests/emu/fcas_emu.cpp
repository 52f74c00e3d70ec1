// CPU emulator of one fitness evaluation through the library's own tile and
// stage functions (paper_2002_02150_amd/csrc/fitness_tiles.hpp), thread by
// thread, with a separate LDS buffer per transform and the kernel's
// write / barrier / read order.  Built with the host address sanitizer by the
// tests, so any out-of-range index in the pass logic aborts on the CPU.
//
// usage: fcas_emu <precision 0|1> <plan> <n_det> <k_lo> <k_hi> <df> <f_star> <in_prefix> <out_file>
//   inputs  <in_prefix>.{pos,ten,sigma,b,theta} float64, <in_prefix>.y complex64 or complex128 [K][n_det]
//   output  N float64 Gamma^2_j, then best value, best sample (float64)
//   FCAS_EMU_ROW=d in the environment plants a mistake: pass 2 takes the
//   factors of row j1 + d (mod N1) for row j1
#include <algorithm>
#include <array>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "plans.hpp"

using namespace fcas;

template <typename T>
static std::vector<T> read_all(const std::string& path) {
  FILE* f = std::fopen(path.c_str(), "rb");
  if (!f) { std::perror(path.c_str()); std::exit(2); }
  std::fseek(f, 0, SEEK_END);
  long bytes = std::ftell(f);
  std::fseek(f, 0, SEEK_SET);
  std::vector<T> v(bytes / sizeof(T));
  if (std::fread(v.data(), sizeof(T), v.size(), f) != v.size()) std::exit(3);
  std::fclose(f);
  return v;
}

template <typename Real, int E>
struct Regs {
  cplx<Real> v[2][E];
};

// All stages of a length-L transform for the threads of a work-group sharing
// one LDS buffer per transform: buffer of thread `tid` is bufs[owner(tid)],
// index t = pos(tid).  Passes 1 and 2: factors in registers (one GeoSet per
// thread); the middle pass: a table of twiddles.
template <typename Real, int L, int E, class Rad, int I, bool SHIFT, bool HALF, int PAD, class Owner, class Pos>
static void emu_geo_stages(std::vector<Regs<Real, E>>& regs, std::vector<std::vector<cplx<Real>>>& bufs,
                           const std::vector<GeoSet<Real, L, E, Rad, SHIFT>>& geo, Owner owner, Pos pos) {
  if constexpr (I < Rad::count) {
    for (int s = 0; s < 2; ++s) {
      for (size_t tid = 0; tid < regs.size(); ++tid)
        geo_stage<Real, L, E, Rad, I, SHIFT, HALF && I == 0, PAD>(regs[tid].v[s], bufs[owner(tid)].data(), geo[tid],
                                                                  pos(tid));
      if constexpr (I < Rad::count - 1)
        for (size_t tid = 0; tid < regs.size(); ++tid)
          stage_gather<Real, L, E, PAD>(regs[tid].v[s], bufs[owner(tid)].data(), pos(tid));
    }
    emu_geo_stages<Real, L, E, Rad, I + 1, SHIFT, HALF, PAD>(regs, bufs, geo, owner, pos);
  }
}

template <typename Real, int L, int E, class Rad, int I, int Ns, int PAD, class Owner, class Pos>
static void emu_table_stages(std::vector<Regs<Real, E>>& regs, std::vector<std::vector<cplx<Real>>>& bufs,
                             const std::vector<cplx<Real>>& tw, Owner owner, Pos pos) {
  if constexpr (I < Rad::count) {
    constexpr int R = Rad::value[I];
    constexpr bool LAST = (I == Rad::count - 1);
    for (int s = 0; s < 2; ++s) {
      for (size_t tid = 0; tid < regs.size(); ++tid)
        stage_butterflies<Real, L, E, R, Ns, LAST, PAD>(regs[tid].v[s], bufs[owner(tid)].data(), tw.data(), pos(tid));
      if constexpr (!LAST) {
        for (size_t tid = 0; tid < regs.size(); ++tid)
          stage_gather<Real, L, E, PAD>(regs[tid].v[s], bufs[owner(tid)].data(), pos(tid));
      }
    }
    emu_table_stages<Real, L, E, Rad, I + 1, Ns * R, PAD>(regs, bufs, tw, owner, pos);
  }
}

template <typename Real, class PL, int DT>
static void prologue(cplx<Real> (&v)[2][PL::E1], const EvalDesc& ev, const SegDesc& sg, int n_det, int tile, int c,
                     int p) {
  if constexpr (DT > 0) {
    Pass1Data<Real, PL, DT> d;
    pass1_fetch<Real, PL, DT>(d, sg, tile, c, p);
    pass1_compute<Real, PL, DT>(v, d, pass1_point<Real, DT>(&ev));
  } else {
    pass1_prologue<Real, PL, 0>(v, ev, sg, n_det, tile, c, p);
  }
}

// The prologue of one thread for n_det detectors (as in the kernels, a
// compile-time count; `loop`: the run-time loop of the fused kernel).
template <typename Real, class PL>
static void any_prologue(cplx<Real> (&v)[2][PL::E1], const EvalDesc& ev, const SegDesc& sg, int n_det, bool loop,
                         int tile, int c, int p) {
  switch (loop ? 0 : n_det) {
#define FCAS_EMU_DT(DT) \
  case DT: return prologue<Real, PL, DT>(v, ev, sg, n_det, tile, c, p);
    FCAS_EMU_DT(0) FCAS_EMU_DT(1) FCAS_EMU_DT(2) FCAS_EMU_DT(3) FCAS_EMU_DT(4)
    FCAS_EMU_DT(5) FCAS_EMU_DT(6) FCAS_EMU_DT(7) FCAS_EMU_DT(8)
  }
}

template <typename Real, class PL>
static void run(const SegDesc& sg, const EvalDesc& ev, int n_det, std::vector<double>& series, double& bg,
                int& bj) {
  const int64_t N = PL::N;
  const int row_off = std::getenv("FCAS_EMU_ROW") ? std::atoi(std::getenv("FCAS_EMU_ROW")) : 0;
  std::vector<cplx<Real>> ws(2 * N);
  const int LP1 = lds_padded_len<kPad1>(PL::N1), LP2 = lds_padded_len<kPad2>(PL::N2);
  using Geo1 = GeoSet<Real, PL::N1, PL::E1, typename PL::Rad1, false>;
  using Geo2 = GeoSet<Real, PL::N2, PL::E2, typename PL::Rad2, !PL::THREE>;
  std::vector<Geo1> geo1(PL::T1);
  for (int tid = 0; tid < PL::T1; ++tid) geo1[tid].init(tid / PL::C);
  for (int tile = 0; tile < PL::TILES1; ++tile) {
    std::vector<Regs<Real, PL::E1>> regs(PL::T1), looped(PL::T1);
    std::vector<std::vector<cplx<Real>>> bufs(PL::C, std::vector<cplx<Real>>(LP1));
    for (int tid = 0; tid < PL::T1; ++tid) {
      any_prologue<Real, PL>(regs[tid].v, ev, sg, n_det, false, tile, tid % PL::C, tid / PL::C);
      any_prologue<Real, PL>(looped[tid].v, ev, sg, n_det, true, tile, tid % PL::C, tid / PL::C);
      for (int s = 0; s < 2; ++s)
        for (int q = 0; q < PL::E1 / 2; ++q)
          if (regs[tid].v[s][q].x != looped[tid].v[s][q].x || regs[tid].v[s][q].y != looped[tid].v[s][q].y) {
            std::fprintf(stderr, "the two prologues differ at tile %d thread %d\n", tile, tid);
            std::exit(8);
          }
    }
    emu_geo_stages<Real, PL::N1, PL::E1, typename PL::Rad1, 0, false, true, kPad1>(
        regs, bufs, geo1, [](size_t t) { return (int)(t % PL::C); }, [](size_t t) { return (int)(t / PL::C); });
    for (int tid = 0; tid < PL::T1; ++tid) pass1_store<Real, PL>(regs[tid].v, ws.data(), tile, tid % PL::C, tid / PL::C);
  }
  if constexpr (PL::THREE) {
    std::vector<cplx<Real>> twm(PL::NM);
    for (int m = 0; m < PL::NM; ++m) twm[m] = twiddle<Real>(m, PL::NM);
    const int LPM = lds_padded_len<kPadM>(PL::NM);
    for (int tile = 0; tile < PL::N1 * (PL::N2 / PL::CM); ++tile) {
      std::vector<Regs<Real, PL::EM>> regs(PL::TM);
      std::vector<std::vector<cplx<Real>>> bufs(PL::CM, std::vector<cplx<Real>>(LPM));
      for (int tid = 0; tid < PL::TM; ++tid) {
        passm_fetch<Real, PL>(regs[tid].v, ws.data(), tile, tid % PL::CM, tid / PL::CM);
        passm_twiddle_in<Real, PL>(regs[tid].v, tile, tid % PL::CM, tid / PL::CM);
      }
      emu_table_stages<Real, PL::NM, PL::EM, typename PL::RadM, 0, 1, kPadM>(
          regs, bufs, twm, [](size_t t) { return (int)(t % PL::CM); }, [](size_t t) { return (int)(t / PL::CM); });
      for (int tid = 0; tid < PL::TM; ++tid) {
        passm_twiddle_out<Real, PL>(regs[tid].v, tile, tid % PL::CM, tid / PL::CM);
        passm_store<Real, PL>(regs[tid].v, ws.data(), tile, tid % PL::CM, tid / PL::CM);
      }
    }
  }
  series.assign(N, -1.0);
  bg = -1;
  bj = 0x7fffffff;
  for (int tile = 0; tile < PL::TILES2; ++tile) {
    std::vector<Regs<Real, PL::E2>> regs(PL::T2);
    std::vector<std::vector<cplx<Real>>> bufs(PL::RW, std::vector<cplx<Real>>(LP2));
    std::vector<Geo2> geo2(PL::T2);
    for (int tid = 0; tid < PL::T2; ++tid) {
      const int r = tid / PL::P2, p = tid % PL::P2;
      pass2_fetch<Real, PL>(regs[tid].v, ws.data(), tile, r, p);
      if (PL::THREE) geo2[tid].init(p);
      else geo2[tid].init(p, (tile * PL::RW + r + row_off) % PL::N1, PL::N1);
    }
    emu_geo_stages<Real, PL::N2, PL::E2, typename PL::Rad2, 0, !PL::THREE, false, kPad2>(
        regs, bufs, geo2, [](size_t t) { return (int)(t / PL::P2); }, [](size_t t) { return (int)(t % PL::P2); });
    for (int tid = 0; tid < PL::T2; ++tid) {
      const int r = tid / PL::P2, p = tid % PL::P2;
      const int j0 = row_base<PL>(tile * PL::RW + r);
      for (int q = 0; q < PL::E2; ++q) {
        const int64_t j = j0 + (int64_t)PL::ROWS2 * (p + q * PL::P2);
        if (series.at(j) != -1.0) { std::fprintf(stderr, "sample %lld written twice\n", (long long)j); std::exit(4); }
        series.at(j) = (double)(norm2(regs[tid].v[0][q]) + norm2(regs[tid].v[1][q]));
      }
      Real gs[PL::E2], g;
      int j;
      for (int q = 0; q < PL::E2; ++q) gs[q] = norm2(regs[tid].v[0][q]) + norm2(regs[tid].v[1][q]);
      pass2_best_of<Real, PL>(gs, tile, r, p, g, j, 0, N);
      if (better((double)g, j, bg, bj)) { bg = (double)g; bj = j; }
    }
  }
  for (int64_t j = 0; j < N; ++j)
    if (series[j] < 0) { std::fprintf(stderr, "sample %lld never written\n", (long long)j); std::exit(5); }
}

template <typename Real>
static int main_t(int plan, int n_det, int k_lo, int k_hi, double df, double f_star, const std::string& in,
                  const std::string& out) {
  auto pos = read_all<double>(in + ".pos");
  auto ten = read_all<double>(in + ".ten");
  auto sig = read_all<double>(in + ".sigma");
  auto b = read_all<double>(in + ".b");
  auto th = read_all<double>(in + ".theta");
  auto y = read_all<cplx<Real>>(in + ".y");
  const int K = k_hi - k_lo + 1;
  if ((int)b.size() != K || (int)y.size() != K * n_det || (int)pos.size() != 3 * n_det) {
    std::fprintf(stderr, "input sizes do not match\n");
    return 6;
  }
  NetDesc net{};
  net.n_det = n_det;
  net.f_star = f_star;
  std::memcpy(net.pos, pos.data(), sizeof(double) * 3 * n_det);
  std::memcpy(net.ten, ten.data(), sizeof(double) * 9 * n_det);
  SegDesc sg{};
  sg.y = y.data();
  sg.b = b.data();
  sg.n = kPlans[plan].n;
  sg.k_lo = k_lo;
  sg.k_hi = k_hi;
  sg.plan = plan;
  sg.registered = 1;
  sg.dk1 = (int32_t)(kPlans[plan].n / kPlans[plan].e1);
  sg.df = df;
  for (int i = 0; i < n_det; ++i) sg.sigma[i] = sig[i];
  EvalDesc ev{};
  setup_one(net, sg, th.data(), ev);
  std::vector<double> series;
  double bg;
  int bj;
#define FCAS_EMU_CASE(id, ...)                                                                         \
  case id: {                                                                                           \
    using PL = std::conditional_t<std::is_same_v<Real, float>, PlanF##id, PlanD##id>;                  \
    run<Real, PL>(sg, ev, n_det, series, bg, bj);                                                      \
    break;                                                                                             \
  }
  switch (plan) {
    FCAS_PLAN_LIST(FCAS_EMU_CASE)
    default:
      return 7;
  }
  FILE* f = std::fopen(out.c_str(), "wb");
  std::fwrite(series.data(), sizeof(double), series.size(), f);
  const double tail[2] = {bg, (double)bj};
  std::fwrite(tail, sizeof(double), 2, f);
  std::fclose(f);
  return 0;
}

// Checks the fused-schedule sequence for cnt evaluations with lag L and S
// slots: every (kind, ep, tile) appears exactly once, a pass-2 tile comes after
// all pass-1 tiles of its evaluation, and a pass-1 tile comes after all pass-2
// tiles of the evaluation that used its slot before (ep - S).
static int check_schedule(int cnt, int L, int S, int T1, int T2) {
  const int total = cnt * (T1 + T2);
  std::vector<int> pos1((size_t)cnt * T1, -1), pos2((size_t)cnt * T2, -1);
  for (int i = 0; i < total; ++i) {
    int kind, ep, tile;
    fused_decode(i, cnt, L, T1, T2, kind, ep, tile);
    if (ep < 0 || ep >= cnt) return 10;
    if (kind == 1) {
      if (tile < 0 || tile >= T1 || pos1.at((size_t)ep * T1 + tile) != -1) return 11;
      pos1[(size_t)ep * T1 + tile] = i;
    } else if (kind == 2) {
      if (tile < 0 || tile >= T2 || pos2.at((size_t)ep * T2 + tile) != -1) return 12;
      pos2[(size_t)ep * T2 + tile] = i;
    } else {
      return 13;
    }
  }
  for (int ep = 0; ep < cnt; ++ep) {
    int last1 = -1, first1 = total, last2 = -1, first2 = total;
    for (int t = 0; t < T1; ++t) {
      last1 = std::max(last1, pos1[(size_t)ep * T1 + t]);
      first1 = std::min(first1, pos1[(size_t)ep * T1 + t]);
    }
    for (int t = 0; t < T2; ++t) first2 = std::min(first2, pos2[(size_t)ep * T2 + t]);
    if (last1 >= first2) return 14;   // pass 2 before its pass 1
    if (ep >= S) {
      for (int t = 0; t < T2; ++t) last2 = std::max(last2, pos2[(size_t)(ep - S) * T2 + t]);
      if (last2 >= first1) return 15;   // slot reused too early
    }
  }
  return 0;
}

int main(int argc, char** argv) {
  if (argc == 7 && std::string(argv[1]) == "schedule") {
    return check_schedule(std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]), std::atoi(argv[5]),
                          std::atoi(argv[6]));
  }
  if (argc != 10) {
    std::fprintf(stderr, "usage: %s prec plan n_det k_lo k_hi df f_star in_prefix out\n", argv[0]);
    return 1;
  }
  const int prec = std::atoi(argv[1]), plan = std::atoi(argv[2]), n_det = std::atoi(argv[3]);
  const int k_lo = std::atoi(argv[4]), k_hi = std::atoi(argv[5]);
  const double df = std::atof(argv[6]), f_star = std::atof(argv[7]);
  return prec ? main_t<double>(plan, n_det, k_lo, k_hi, df, f_star, argv[8], argv[9])
              : main_t<float>(plan, n_det, k_lo, k_hi, df, f_star, argv[8], argv[9]);
}
