// fitness_tiles.hpp -- the two passes of the coherent-fitness evaluation, per
// work item and per thread, written once for the gfx950 kernels and the CPU
// emulator used by the tests.
//
// For one parameter point the library forms, for every in-band bin k (Sec. II.D),
//   w^i_k = y^i_k exp(2 pi i [Phi_k + k dly_i])     (template phase and the
//            detector delay as an exact frequency-domain shift, eq.
//            data_template_innprod; y already carries 4 df f^-7/6 / (S sigma))
//   W_m(k) = sum_i Q_im w^i_k,  m = 0, 1
// where the columns of Q are an orthonormal basis of span(diag(sigma) U).  By
// linearity the inverse FFTs of W_0, W_1 give a_m(j) = sum_i Q_im z^i_j, and
//   Gamma^2_j = |a_0(j)|^2 + |a_1(j)|^2 = z_j^H Q Q^T z_j,
// the log-likelihood ratio maximised over the four amplitudes (Sec. II.C).
//
// The length-N inverse FFT is a four-step transform, N = N1 N2,
//   k = k1 N2 + k2,  j = j1 + N1 j2,
//   pass 1 (per column k2): B(j1, k2) = w_N^{k2 j1} sum_{k1} W(k1 N2 + k2) w_N1^{k1 j1}
//   pass 2 (per row j1):    a(j1 + N1 j2) = sum_{k2} B(j1, k2) w_N2^{k2 j2}
// with B stored row-major [series][j1][k2] in the workspace.  Lengths too long
// for two passes insert a middle pass (see Plan below).
#pragma once

#include <stdint.h>

#include "fft_core.hpp"

namespace fcas {

constexpr int kMaxDet = 8;

// Per registered segment (device resident).
struct SegDesc {
  const void* y;        // [K][n_det] complex (float2 or double2 by precision)
  const double* b;      // [K] (f_k / f*)^(-1/3)
  int64_t n;            // samples
  int32_t k_lo, k_hi;   // inclusive in-band bins
  int32_t plan;         // FFT plan index
  int32_t registered;   // 1 once fcas_set_segment has completed
  int32_t dk1;          // the plan's pass-1 register stride in bins (P1 W1)
  int32_t reserved;
  double df;            // 1 / T
  double sigma[kMaxDet];
  int64_t j_lo, j_hi;   // coalescence samples searched: j_lo <= j < j_hi
};

// Per parameter point, written by the set-up kernel.
struct EvalDesc {
  double coef[4];             // Phi_k = coef0 b^5 + coef1 b^3 + coef2 b^2 + coef3 b (cycles)
  double dly[kMaxDet];        // Delta^i * df: delay ramp in cycles per bin
  double q[kMaxDet][2];       // orthonormal basis of span(diag(sigma) U), FP64
  float qf[kMaxDet][2];       // same, rounded to float
  double v[kMaxDet][2];       // V = diag(sigma) U (kept for the gradient)
  double step1[kMaxDet][2];   // exp(2 pi i dk1 (dly_i - dly_0)): ramp of detector i relative to
                              // detector 0 across one pass-1 register stride
  float step1f[kMaxDet][2];   // same, rounded to float
  int32_t seg;
  int32_t status;             // 1 evaluate, 0 outside the rectangle, -2 bad segment
  int32_t plan;
  int32_t rank;               // rank of V (0, 1 or 2)
};

// Network, search rectangle and band reference frequency (device resident).
struct NetDesc {
  int32_t n_det;
  int32_t max_segments;
  double pos[kMaxDet][3];
  double ten[kMaxDet][3][3];
  double box_lo[4], box_hi[4];
  double f_star;
};

constexpr double kPi = 3.14159265358979323846;
constexpr double kC = 299792458.0;

// ---------------------------------------------------------------------------
// Set-up of one parameter point, FP64 (chirp times, delays, antenna patterns,
// orthonormal basis).  Sec. II.B (chirp times), Sec. II (eq. detresponse:
// delays, antenna pattern matrix), Sec. II.C (U = F(psi = 0)).
//
// Written once for two executions: `Dets` is either a loop over the
// detectors (setup_one, one thread per point) or a group of lanes with one
// detector each, whose sums over detectors are lane reductions (the kernel).
// A detector's values stay in registers (DetPoint) until the descriptor is
// written.
// ---------------------------------------------------------------------------
struct SkyFrame {
  double n[3], ex[3], ey[3];   // propagation direction and wave axes (-alpha_hat, delta_hat)
};

// 1 / cbrt(x) and 1 / sqrt(x).
FCAS_HD double inv_cbrt(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return rcbrt(x);
#else
  return 1.0 / std::cbrt(x);
#endif
}
FCAS_HD double inv_sqrt(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return rsqrt(x);
#else
  return 1.0 / std::sqrt(x);
#endif
}

// Phase coefficients (cycles) of a point.  With x = 5 tau15 / (32 pi tau0),
// v0 = x^(1/3) and eta = 1 / (8 fs tau15 v0^2),
//   tau1 = 5 / (192 pi fs eta v0^3) (743/336 + 11/4 eta)
//   tau2 = 5 / (128 pi fs eta v0) (3058673/1016064 + 5429/1008 eta + 617/144 eta^2),
// where 1 / (fs eta) = 8 tau15 v0^2: the two quotients that are left do not
// wait for each other.
FCAS_HD void setup_phase(double tau0, double tau15, double fs, double coef[4]) {
  const double x = 5.0 * tau15 / (32.0 * kPi * tau0);
  const double r = inv_cbrt(x), r2 = r * r, v0 = x * r2;
  const double eta = r2 * (1.0 / (8.0 * fs * tau15));
  const double tau1 = (40.0 / (192.0 * kPi)) * tau15 * r * (743.0 / 336.0 + 2.75 * eta);
  const double tau2 = (40.0 / (128.0 * kPi)) * tau15 * v0 *
                      (3058673.0 / 1016064.0 + eta * (5429.0 / 1008.0 + eta * (617.0 / 144.0)));
  coef[0] = fs * 0.6 * tau0;
  coef[1] = fs * tau1;
  coef[2] = -fs * 1.5 * tau15;
  coef[3] = fs * 3.0 * tau2;
}

// The sky frame from the sines and cosines of alpha and delta.
FCAS_HD void setup_sky(double sa, double ca, double sd, double cd, SkyFrame& fr) {
  fr.n[0] = cd * ca; fr.n[1] = cd * sa; fr.n[2] = sd;
  fr.ex[0] = sa; fr.ex[1] = -ca; fr.ex[2] = 0.0;
  fr.ey[0] = -sd * ca; fr.ey[1] = -sd * sa; fr.ey[2] = cd;
}

FCAS_HD void setup_point(const NetDesc& net, const double* th, double coef[4], SkyFrame& fr) {
  setup_phase(th[2], th[3], net.f_star, coef);
  double sa, ca, sd, cd;
  sincos(th[0], &sa, &ca);
  sincos(th[1], &sd, &cd);
  setup_sky(sa, ca, sd, cd, fr);
}

// Delay ramp of detector i in cycles per bin of width df (delay relative to
// the geocentre).
FCAS_HD double detector_delay(const NetDesc& net, double df, const SkyFrame& fr, int i) {
  const double* r = net.pos[i];
  return (fr.n[0] * r[0] + fr.n[1] * r[1] + fr.n[2] * r[2]) * (df * (-1.0 / kC));
}

// What the set-up computes of one detector.
struct DetPoint {
  double dly;        // delay ramp, cycles per bin
  double step[2];    // its pass-1 step relative to detector 0
  double v[2];       // row of V
  double q[2];       // row of Q
};

// Delay ramp and row of V of detector i, of a segment with bin width df and
// template norm sigma_i.
FCAS_HD void setup_detector(const NetDesc& net, double df, double sigma_i, const SkyFrame& fr, int i, DetPoint& d) {
  d.dly = detector_delay(net, df, fr, i);
  double up = 0.0, uc = 0.0;
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) {
      const double t = net.ten[i][a][b];
      up += t * (fr.ex[a] * fr.ex[b] - fr.ey[a] * fr.ey[b]);
      uc += t * (fr.ex[a] * fr.ey[b] + fr.ey[a] * fr.ex[b]);
    }
  d.v[0] = sigma_i * up;
  d.v[1] = sigma_i * uc;
}

// Its ramp across one pass-1 register stride of dk1 bins, relative to
// detector 0's delay ramp dly0.
FCAS_HD void setup_step(int dk1, double dly0, DetPoint& d) {
  const double ps = (double)dk1 * (d.dly - dly0);
  sincos_rev(ps - rint(ps), &d.step[1], &d.step[0]);
}

// Orthonormal basis Q of span(V): modified Gram-Schmidt, twice, larger
// column first; q[1] holds the residual of the second column until it is
// normalised.  Returns the rank (0, 1 or 2).
template <class Dets>
FCAS_HD int setup_basis(Dets& dets) {
  const double n0 = dets.sum([](const DetPoint& d) { return d.v[0] * d.v[0]; });
  const double n1 = dets.sum([](const DetPoint& d) { return d.v[1] * d.v[1]; });
  const double vf = n0 + n1;
  const bool second = n1 > n0;   // the larger column
  const double na = second ? n1 : n0;
  dets.each([](DetPoint& d) { d.q[0] = d.q[1] = 0.0; });
  int rank = 0;
  if (na > 0.0) {
    rank = 1;
    const double ia = inv_sqrt(na);
    dets.each([&](DetPoint& d) {
      d.q[0] = (second ? d.v[1] : d.v[0]) * ia;
      d.q[1] = second ? d.v[0] : d.v[1];
    });
    for (int pass = 0; pass < 2; ++pass) {
      const double dot = dets.sum([](const DetPoint& d) { return d.q[0] * d.q[1]; });
      dets.each([&](DetPoint& d) { d.q[1] -= dot * d.q[0]; });
    }
    const double nb = dets.sum([](const DetPoint& d) { return d.q[1] * d.q[1]; });
    const bool full = sqrt(nb) > 1e-10 * sqrt(vf);
    if (full) rank = 2;
    const double ib = full ? inv_sqrt(nb) : 0.0;
    dets.each([&](DetPoint& d) { d.q[1] *= ib; });
  }
  return rank;
}

// Detector i's entries of a point's descriptor.
FCAS_HD void store_detector(EvalDesc& ev, int i, const DetPoint& d) {
  ev.dly[i] = d.dly;
  for (int m = 0; m < 2; ++m) {
    ev.v[i][m] = d.v[m];
    ev.q[i][m] = d.q[m];
    ev.qf[i][m] = (float)d.q[m];
    ev.step1[i][m] = d.step[m];
    ev.step1f[i][m] = (float)d.step[m];
  }
}

// The detectors as a loop of one thread.
struct DetLoop {
  int n_det;
  DetPoint p[kMaxDet];
  template <class F> FCAS_HD double sum(F f) const {
    double acc = 0.0;
    for (int i = 0; i < n_det; ++i) acc += f(p[i]);
    return acc;
  }
  template <class F> FCAS_HD void each(F f) {
    for (int i = 0; i < n_det; ++i) f(p[i]);
  }
};

FCAS_HD void setup_one(const NetDesc& net, const SegDesc& sg, const double* th, EvalDesc& ev) {
  SkyFrame fr;
  setup_point(net, th, ev.coef, fr);
  DetLoop dets{};
  dets.n_det = net.n_det;
  for (int i = 0; i < net.n_det; ++i) {
    setup_detector(net, sg.df, sg.sigma[i], fr, i, dets.p[i]);
    setup_step(sg.dk1, dets.p[0].dly, dets.p[i]);
  }
  ev.rank = setup_basis(dets);
  for (int i = 0; i < net.n_det; ++i) store_detector(ev, i, dets.p[i]);
}

// Common phase of bin k in cycles, b = (f_k / f*)^(-1/3): FP64 throughout.
FCAS_HD double common_phase(const double* coef, double b) {
  const double b2 = b * b;
  return b * (coef[3] + b * (coef[2] + b * (coef[1] + coef[0] * b2)));
}

template <typename Real> struct Basis;
template <> struct Basis<float> {
  FCAS_HD static float get(const EvalDesc& e, int i, int m) { return e.qf[i][m]; }
};
template <> struct Basis<double> {
  FCAS_HD static double get(const EvalDesc& e, int i, int m) { return e.q[i][m]; }
};

template <typename Real> FCAS_HD cplx<Real> ramp_step(const EvalDesc& e, int i);
template <> FCAS_HD cplx<float> ramp_step<float>(const EvalDesc& e, int i) {
  return mk<float>(e.step1f[i][0], e.step1f[i][1]);
}
template <> FCAS_HD cplx<double> ramp_step<double>(const EvalDesc& e, int i) {
  return mk<double>(e.step1[i][0], e.step1[i][1]);
}

// ---------------------------------------------------------------------------
// One Stockham stage of the middle pass for one series of one transform (see
// fft_core.hpp), twiddles from a table.  Either leaves the outputs in registers (last stage) or scatters them to the
// transform's LDS buffer, to be gathered back in natural strided order.
// ---------------------------------------------------------------------------
template <typename Real, int L, int E, int R, int Ns, bool LAST, int PAD>
FCAS_HD void stage_butterflies(cplx<Real>* vs, cplx<Real>* buf, const cplx<Real>* tw, int t) {
  constexpr int P = L / E;
  constexpr int B = E / R;
  static_assert(E % R == 0, "radix must divide the elements per thread");
#pragma unroll
  for (int b = 0; b < B; ++b) {
    const int v = t + b * P;
    cplx<Real> x[R];
#pragma unroll
    for (int p = 0; p < R; ++p) x[p] = vs[b + p * B];
    if constexpr (Ns > 1) {
#pragma unroll
      for (int p = 1; p < R; ++p) x[p] = mul(x[p], tw[stockham_tw(v, Ns, R, p, L)]);
    }
    dft<R>(x);
    if constexpr (LAST) {
#pragma unroll
      for (int p = 0; p < R; ++p) vs[b + p * B] = x[p];
    } else {
#pragma unroll
      for (int p = 0; p < R; ++p) buf[lds_pad<PAD>(stockham_dst(v, Ns, R, p))] = x[p];
    }
  }
}

template <typename Real, int L, int E, int PAD>
FCAS_HD void stage_gather(cplx<Real>* vs, const cplx<Real>* buf, int t) {
  constexpr int P = L / E;
#pragma unroll
  for (int q = 0; q < E; ++q) vs[q] = buf[lds_pad<PAD>(t + q * P)];
}

// ---------------------------------------------------------------------------
// The stages of the two main passes.  A thread's twiddle factors depend on
// its place in the transform alone (pass 1), or on that and the row (pass 2),
// so they are formed once and kept in registers while the thread takes one
// point after the other (GeoSet).
//
// SHIFT transforms by x[k] exp(2 pi i k theta / L), theta = j1 / n1, first:
// the four-step twiddle w_N^{k2 j1} of pass 2.  It needs no products of its
// own: a stage of radix R after sub-length Ns then has the ratio
//   s = exp(2 pi i ((v mod Ns) + theta) / (Ns R)).
// ---------------------------------------------------------------------------
template <int L, int E, class Rad, bool SHIFT>
struct GeoShape {
  static constexpr int P = L / E;
  static constexpr int sub(int i) {   // product of the radices before stage i
    int n = 1;
    for (int k = 0; k < i; ++k) n *= Rad::value[k];
    return n;
  }
  // butterflies of stage i with factors of their own (they share them where
  // their places agree mod the sub-length)
  static constexpr int sets(int i) { return P % sub(i) == 0 ? 1 : E / Rad::value[i]; }
  static constexpr bool twiddled(int i) { return SHIFT || i > 0; }
  static constexpr int offset(int i) {
    int n = 0;
    for (int k = 0; k < i; ++k)
      if (twiddled(k)) n += sets(k) * geo_count(Rad::value[k]);
    return n;
  }
  static constexpr int count = offset(Rad::count) > 0 ? offset(Rad::count) : 1;
};

template <typename Real, int L, int E, class Rad, bool SHIFT>
struct GeoSet {
  using Shape = GeoShape<L, E, Rad, SHIFT>;
  cplx<Real> w[Shape::count];

  // factors of thread t (of P per transform); SHIFT: for theta = j1 / n1
  FCAS_HD void init(int t, int j1 = 0, int n1 = 1) { init_stage<0>(t, j1, n1); }

  template <int I>
  FCAS_HD void init_stage(int t, int j1, int n1) {
    if constexpr (I < Rad::count) {
      constexpr int R = Rad::value[I], Ns = Shape::sub(I);
      if constexpr (Shape::twiddled(I)) {
#pragma unroll
        for (int b = 0; b < Shape::sets(I); ++b) {
          const int v = (t + b * Shape::P) % Ns;
          if constexpr (SHIFT)
            geo_factors<R>(w + Shape::offset(I) + b * geo_count(R), v * n1 + j1, Ns * R * n1);
          else
            geo_factors<R>(w + Shape::offset(I) + b * geo_count(R), v, Ns * R);
        }
      }
      init_stage<I + 1>(t, j1, n1);
    }
  }
};

// Stage I for one series of one transform: inputs in registers; outputs left
// there (last stage) or scattered to the transform's LDS buffer.
template <typename Real, int L, int E, class Rad, int I, bool SHIFT, bool HALF, int PAD>
FCAS_HD void geo_stage(cplx<Real>* vs, cplx<Real>* buf, const GeoSet<Real, L, E, Rad, SHIFT>& g, int t) {
  using Shape = GeoShape<L, E, Rad, SHIFT>;
  constexpr int P = Shape::P, R = Rad::value[I], B = E / R, Ns = Shape::sub(I);
  constexpr bool LAST = (I == Rad::count - 1);
  static_assert(E % R == 0, "radix must divide the elements per thread");
  static_assert(!HALF || (I == 0 && B == 1 && !SHIFT), "half-zero inputs only in an untwiddled first stage");
#pragma unroll
  for (int b = 0; b < B; ++b) {
    const int v = t + b * P;
    cplx<Real> x[R];
#pragma unroll
    for (int p = 0; p < (HALF ? R / 2 : R); ++p) x[p] = vs[b + p * B];
    if constexpr (HALF)
      dft_half<R>(x);
    else if constexpr (Shape::twiddled(I))
      dft_geo<R>(x, g.w + Shape::offset(I) + (Shape::sets(I) == 1 ? 0 : b) * geo_count(R));
    else
      dft<R>(x);
    if constexpr (LAST) {
#pragma unroll
      for (int p = 0; p < R; ++p) vs[b + p * B] = x[p];
    } else {
#pragma unroll
      for (int p = 0; p < R; ++p) buf[lds_pad<PAD>(stockham_dst(v, Ns, R, p))] = x[p];
    }
  }
}

// Compile-time description of a plan.
// Two-pass plans (NM = 1): N = N1 * N2,
//   pass 1: C columns per work item, P1 = N1 / E1 threads per column
//   pass 2: RW rows per work item,   P2 = N2 / E2 threads per row
// Three-pass plans (NM > 1): N = N1 * NM * N2 with
//   k = k1 NM N2 + km N2 + k2,  j = j1 + N1 jm + N1 NM j2,
//   pass 1 (per column km N2 + k2 of its W1 = NM N2): the length-N1 transform over k1,
//           stored as B1[j1][km N2 + k2]
//   middle pass (per j1 and k2; CM adjacent k2 per work item, PM = NM / EM
//           threads per transform): times w_N^{j1 (km N2 + k2)}, the
//           length-NM transform over km, times w_{NM N2}^{jm k2}, stored in
//           place as B2[j1][jm N2 + k2]
//   pass 2 (per row j1 NM + jm, contiguous): the length-N2 transform over k2
//           and the maximum of |a_0|^2 + |a_1|^2 over its samples
// which is the four-step factorisation applied twice: both passes' row
// segments stay contiguous, so every store and load moves whole 64-byte or
// longer pieces even when N1 N2 exceeds what one work item can hold.
// LDS padding of the exchanges (see lds_pad): one spare element in 16 for all
// passes (on gfx950 pass 1 runs 1.7x slower unpadded, pass 2 ~8%).
constexpr int kPad1 = 4, kPad2 = 4, kPadM = 4;

template <int N1_, int E1_, class Rad1_, int C_, int N2_, int E2_, class Rad2_, int RW_, int NM_ = 1, int EM_ = 1,
          class RadM_ = Radices<1>, int CM_ = 1>
struct Plan {
  static constexpr int N1 = N1_, E1 = E1_, C = C_, N2 = N2_, E2 = E2_, RW = RW_;
  static constexpr int NM = NM_, EM = EM_, CM = CM_;
  using Rad1 = Rad1_;
  using Rad2 = Rad2_;
  using RadM = RadM_;
  static constexpr bool THREE = NM > 1;
  static constexpr int W1 = NM * N2;                        // columns of pass 1 (its output row length)
  static constexpr int ROWS2 = N1 * NM;                     // rows of pass 2
  static constexpr int64_t N = (int64_t)N1 * NM * N2;
  static constexpr int P1 = N1 / E1, P2 = N2 / E2, PM = NM / EM;
  static constexpr int T1 = C * P1, T2 = RW * P2, TM = CM * PM;   // threads per work item
  static constexpr int TILES1 = W1 / C, TILES2 = ROWS2 / RW;      // work items per evaluation
  static constexpr int TILESM = THREE ? N1 * (N2 / CM) : 0;
  static constexpr int DK1 = P1 * W1;                       // bin stride between a pass-1 thread's registers
  static constexpr int PARTS2 = TILES2;                     // pass-2 partials (one per work item)
  static_assert(Rad1::product() == N1, "pass-1 radices must multiply to N1");
  static_assert(Rad2::product() == N2, "pass-2 radices must multiply to N2");
  static_assert(RadM::product() == NM, "middle-pass radices must multiply to NM");
  static_assert(N1 % E1 == 0 && N2 % E2 == 0 && NM % EM == 0, "elements per thread must divide the length");
  static_assert(W1 % C == 0 && ROWS2 % RW == 0 && N2 % CM == 0, "tiles must divide the transform");
  static_assert(T2 % 64 == 0 && (64 % P2 == 0 || P2 % 64 == 0), "pass-2 rows and wavefronts must nest");
  // the middle pass works in place: at least one work-group barrier (between
  // two stages) separates an item's loads from its stores
  static_assert(!THREE || RadM::count >= 2, "the middle pass needs two or more stages");
  static_assert(N < ((int64_t)1 << 30), "sample and bin indices are 32-bit");
};

// First output sample of pass-2 row `row`; the row's samples follow at a
// stride of ROWS2.
template <class PL>
FCAS_HD int row_base(int row) {
  if constexpr (PL::THREE) {
    const int j1 = row / PL::NM;
    return j1 + PL::N1 * (row - j1 * PL::NM);
  } else {
    return row;
  }
}

// ---------------------------------------------------------------------------
// Pass 1, thread (c, p) of column tile `tile`: prologue into registers.
// Register q holds k1 = p + q P1, i.e. bin k = k1 W1 + k2.  Only positive
// frequencies are in band (k <= k_hi < N/2), so registers q >= E1/2
// (k1 >= N1/2) are always zero and are left unset: the first stage reads
// only the lower half.
//
// With the delay ramps r_i(k) = exp(2 pi i k dly_i) and the template phase
// Phi_k, W_m(k) = exp(2 pi i Phi_k) sum_i Q_im y^i_k r_i(k).  Detector 0's ramp
// is taken out of the sum into the common factor,
//   W_m(k) = e(k) [Q_0m y^0_k + sum_{i>0} Q_im y^i_k r'_i(k)],
//   e(k) = exp(2 pi i (Phi_k + k dly_0)),  r'_i(k) = exp(2 pi i k (dly_i - dly_0)),
// so detector 0 needs no ramp.  e is one sine/cosine per bin of an FP64 phase
// reduced mod 1; r'_i is exact (FP64-reduced) at the thread's first bin and
// advanced by the constant factor exp(2 pi i (P1 W1)(dly_i - dly_0)) of the
// point's descriptor from register to register.  Out-of-band registers read
// bin k_lo and are cleared once, so no lane branches.
// ---------------------------------------------------------------------------
// Segment data one pass-1 thread needs for a work item: y of its in-band
// registers and detectors, and the basis b of those bins (DT > 0 only).
template <typename Real, class PL, int DT>
struct Pass1Data {
  static constexpr int QH = PL::E1 / 2;
  cplx<Real> y[DT > 0 ? DT : 1][QH];
  double b[QH];
  int k0;
};

template <typename Real, class PL, int DT>
FCAS_HD void pass1_fetch(Pass1Data<Real, PL, DT>& d, const SegDesc& sg, int tile, int c, int p) {
  constexpr int QH = PL::E1 / 2;
  constexpr int DK = PL::DK1;
  static_assert(DT > 0, "prefetch needs a compile-time detector count");
  const int k2 = tile * PL::C + c;
  d.k0 = p * PL::W1 + k2;
  const FCAS_AS_GLOBAL cplx<Real>* y = global_view((const cplx<Real>*)sg.y);
  const FCAS_AS_GLOBAL double* bt = global_view(sg.b);
#pragma unroll
  for (int q = 0; q < QH; ++q) {
    const int k = d.k0 + q * DK;
    const bool in = (k >= sg.k_lo) && (k <= sg.k_hi);
    const int kk = in ? k - sg.k_lo : 0;
    d.b[q] = bt[kk];
#pragma unroll
    for (int i = 0; i < DT; ++i) {
      const cplx<Real> u = y[(int64_t)kk * DT + i];
      d.y[i][q] = in ? u : mk<Real>(0, 0);
    }
  }
}

// What the pass-1 arithmetic reads of a point's descriptor, in the working
// precision: phase coefficients, delay ramps, basis Q and ramp steps of the
// DT detectors.  `ev` points to an EvalDesc (through the constant address
// space in the kernels, so that these uniform values are scalar loads held in
// scalar registers).
template <typename Real, int DT>
struct Pass1Point {
  double coef[4];
  double dly[DT];
  Real q[DT][2];
  Real step[DT][2];
};

template <typename Real, int DT, class P>
FCAS_HD Pass1Point<Real, DT> pass1_point(P ev) {
  Pass1Point<Real, DT> r;
#pragma unroll
  for (int k = 0; k < 4; ++k) r.coef[k] = ev->coef[k];
#pragma unroll
  for (int i = 0; i < DT; ++i) {
    r.dly[i] = ev->dly[i];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      if constexpr (sizeof(Real) == 4) {
        r.q[i][m] = ev->qf[i][m];
        r.step[i][m] = ev->step1f[i][m];
      } else {
        r.q[i][m] = ev->q[i][m];
        r.step[i][m] = ev->step1[i][m];
      }
    }
  }
  return r;
}

// e(k) = exp(2 pi i (Phi_k + k dly_0)) for an in-band bin k with basis value
// b, 0 otherwise (Ev: a descriptor with the phase coefficients `coef` and the
// delay ramps `dly`).
template <typename Real, class Ev>
FCAS_HD cplx<Real> band_phase(const Ev& ev, double b, int k, bool in = true) {
  const double ph = common_phase(ev.coef, b) + (double)k * ev.dly[0];
  Real s, cc;
  sincos_rev((Real)(ph - rint(ph)), &s, &cc);
  return in ? mk<Real>(cc, s) : mk<Real>(0, 0);
}

// Ramp r'_i of detector i > 0 at the thread's first bin k0 (FP64 reduction).
template <typename Real, class Ev>
FCAS_HD cplx<Real> first_ramp(const Ev& ev, int i, int k0) {
  const double ph0 = (double)k0 * (ev.dly[i] - ev.dly[0]);
  Real s, cc;
  sincos_rev((Real)(ph0 - rint(ph0)), &s, &cc);
  return mk<Real>(cc, s);
}

// The prologue arithmetic on prefetched data (same results as pass1_prologue).
template <typename Real, class PL, int DT>
FCAS_HD void pass1_compute(cplx<Real> (&v)[2][PL::E1], const Pass1Data<Real, PL, DT>& d,
                           const Pass1Point<Real, DT>& ev) {
  constexpr int QH = PL::E1 / 2;
  {
    const Real q0 = ev.q[0][0], q1 = ev.q[0][1];
#pragma unroll
    for (int q = 0; q < QH; ++q) {
      const cplx<Real> u = d.y[0][q];
      v[0][q] = mk<Real>(q0 * u.x, q0 * u.y);
      v[1][q] = mk<Real>(q1 * u.x, q1 * u.y);
    }
  }
#pragma unroll
  for (int i = 1; i < DT; ++i) {
    cplx<Real> ramp = first_ramp<Real>(ev, i, d.k0);
    const cplx<Real> step = mk<Real>(ev.step[i][0], ev.step[i][1]);
    const Real q0 = ev.q[i][0], q1 = ev.q[i][1];
#pragma unroll
    for (int q = 0; q < QH; ++q) {
      const cplx<Real> u = mul(d.y[i][q], ramp);
      v[0][q] = mk<Real>(v[0][q].x + q0 * u.x, v[0][q].y + q0 * u.y);
      v[1][q] = mk<Real>(v[1][q].x + q1 * u.x, v[1][q].y + q1 * u.y);
      if (q + 1 < QH) ramp = mul(ramp, step);
    }
  }
#pragma unroll
  for (int q = 0; q < QH; ++q) {
    const cplx<Real> e = band_phase<Real>(ev, d.b[q], d.k0 + q * PL::DK1);
    v[0][q] = mul(v[0][q], e);
    v[1][q] = mul(v[1][q], e);
  }
}

// DT > 0: the detector count is the compile-time constant DT (loops unrolled,
// every load of the thread issued up front); DT = 0: n_det at run time.
template <typename Real, class PL, int DT = 0>
FCAS_HD void pass1_prologue(cplx<Real> (&v)[2][PL::E1], const EvalDesc& ev, const SegDesc& sg, int n_det_rt,
                            int tile, int c, int p) {
  constexpr int QH = PL::E1 / 2;
  constexpr int DK = PL::DK1;
  const int n_det = DT > 0 ? DT : n_det_rt;
  const int k2 = tile * PL::C + c;
  const int k0 = p * PL::W1 + k2;
  const cplx<Real>* y = (const cplx<Real>*)sg.y;
  bool in[QH];
  int kk[QH];
#pragma unroll
  for (int q = 0; q < QH; ++q) {
    const int k = k0 + q * DK;
    in[q] = (k >= sg.k_lo) && (k <= sg.k_hi);
    kk[q] = in[q] ? k - sg.k_lo : 0;
  }
  {
    const Real q0 = Basis<Real>::get(ev, 0, 0), q1 = Basis<Real>::get(ev, 0, 1);
#pragma unroll
    for (int q = 0; q < QH; ++q) {
      const cplx<Real> u = y[(int64_t)kk[q] * n_det];
      v[0][q] = mk<Real>(q0 * u.x, q0 * u.y);
      v[1][q] = mk<Real>(q1 * u.x, q1 * u.y);
    }
  }
#pragma unroll
  for (int i = 1; i < (DT > 0 ? DT : kMaxDet); ++i) {
    if (DT == 0 && i >= n_det) break;
    cplx<Real> ramp = first_ramp<Real>(ev, i, k0);
    const cplx<Real> step = ramp_step<Real>(ev, i);
    const Real q0 = Basis<Real>::get(ev, i, 0), q1 = Basis<Real>::get(ev, i, 1);
#pragma unroll
    for (int q = 0; q < QH; ++q) {
      const cplx<Real> u = mul(y[(int64_t)kk[q] * n_det + i], ramp);
      v[0][q] = mk<Real>(v[0][q].x + q0 * u.x, v[0][q].y + q0 * u.y);
      v[1][q] = mk<Real>(v[1][q].x + q1 * u.x, v[1][q].y + q1 * u.y);
      if (q + 1 < QH) ramp = mul(ramp, step);
    }
  }
#pragma unroll
  for (int q = 0; q < QH; ++q) {
    const cplx<Real> e = band_phase<Real>(ev, sg.b[kk[q]], k0 + q * DK, in[q]);
    v[0][q] = mul(v[0][q], e);
    v[1][q] = mul(v[1][q], e);
  }
}

// Pass 1 epilogue: store B[m][j1][k2] (the four-step twiddle is applied when
// the next pass loads the rows).
template <typename Real, class PL, bool NT = false>
FCAS_HD void pass1_store_series(cplx<Real> (&v)[PL::E1], cplx<Real>* slot, int s, int tile, int c, int p) {
  static_assert(2 * (int64_t)PL::N * sizeof(cplx<Real>) < (int64_t(1) << 31), "byte offsets fit in 31 bits");
  const StreamOut<Real> out(slot, 2 * (int64_t)PL::N);
  const int o = p * PL::W1 + tile * PL::C + c;      // row j1 = p, column k2
#pragma unroll
  for (int q = 0; q < PL::E1; ++q) out.template store<NT>(o, s * (int)PL::N + q * PL::P1 * PL::W1, v[q]);   // row p + q P1
}
template <typename Real, class PL, bool NT = false>
FCAS_HD void pass1_store(cplx<Real> (&v)[2][PL::E1], cplx<Real>* slot, int tile, int c, int p) {
  pass1_store_series<Real, PL, NT>(v[0], slot, 0, tile, c, p);
  pass1_store_series<Real, PL, NT>(v[1], slot, 1, tile, c, p);
}

// ---------------------------------------------------------------------------
// Middle pass of a three-pass plan, thread (c, p) of tile `tile`: the tile is
// pass-1 row j1 = tile / (N2 / CM) and the CM adjacent columns k2 from
// (tile mod (N2 / CM)) CM; register q holds km = p + q PM on input and
// jm = p + q PM on output.
// ---------------------------------------------------------------------------
template <class PL>
FCAS_HD void passm_coords(int tile, int c, int& j1, int& k2) {
  constexpr int KT = PL::N2 / PL::CM;
  j1 = tile / KT;
  k2 = (tile - j1 * KT) * PL::CM + c;
}

// The middle-pass functions act on S series held in registers, series s0
// onwards (S = 2, s0 = 0: both).
template <typename Real, class PL, int S>
FCAS_HD void passm_fetch(cplx<Real> (&v)[S][PL::EM], const cplx<Real>* slot, int tile, int c, int p, int s0 = 0) {
  int j1, k2;
  passm_coords<PL>(tile, c, j1, k2);
  const cplx<Real>* at = slot + (int64_t)s0 * PL::N + (int64_t)j1 * PL::W1 + k2;
#pragma unroll
  for (int q = 0; q < PL::EM; ++q) {
    const int o = (p + q * PL::PM) * PL::N2;
#pragma unroll
    for (int s = 0; s < S; ++s) v[s][q] = stream_load(at + s * PL::N + o);
  }
}

// Multiplies register q of every series by t st^(q - EM/2): exact in the middle,
// advanced by a constant factor from register to register upwards and downwards
// from there.  (Half the steps of one run over all registers leave half its
// error, which dominated that of the long lengths.)
template <typename Real, int EM, int S>
FCAS_HD void passm_twiddle(cplx<Real> (&v)[S][EM], cplx<Real> t, cplx<Real> st) {
  constexpr int MID = EM / 2;
  const cplx<Real> back = mk<Real>(st.x, -st.y);
  cplx<Real> up = t, down = mul(t, back);
#pragma unroll
  for (int q = MID; q < EM; ++q) {
#pragma unroll
    for (int s = 0; s < S; ++s) v[s][q] = mul(v[s][q], up);
    if (q + 1 < EM) up = mul(up, st);
  }
#pragma unroll
  for (int q = MID - 1; q >= 0; --q) {
#pragma unroll
    for (int s = 0; s < S; ++s) v[s][q] = mul(v[s][q], down);
    if (q > 0) down = mul(down, back);
  }
}

// w_N^{j1 (km N2 + k2)} on input.
template <typename Real, class PL, int S>
FCAS_HD void passm_twiddle_in(cplx<Real> (&v)[S][PL::EM], int tile, int c, int p) {
  int j1, k2;
  passm_coords<PL>(tile, c, j1, k2);
  passm_twiddle<Real, PL::EM, S>(
      v, twiddle<Real>(j1 * ((p + PL::EM / 2 * PL::PM) * PL::N2 + k2), (int)PL::N),   // < N1 W1 = N
      twiddle<Real>(j1 * (PL::PM * PL::N2), (int)PL::N));
}

// w_{NM N2}^{jm k2} on output.
template <typename Real, class PL, int S>
FCAS_HD void passm_twiddle_out(cplx<Real> (&v)[S][PL::EM], int tile, int c, int p) {
  int j1, k2;
  passm_coords<PL>(tile, c, j1, k2);
  passm_twiddle<Real, PL::EM, S>(v, twiddle<Real>((p + PL::EM / 2 * PL::PM) * k2, PL::W1),   // < NM N2 = W1
                                 twiddle<Real>(PL::PM * k2, PL::W1));
}

// Store B2[m][j1][jm N2 + k2], over the elements the tile loaded.
template <typename Real, class PL, int S>
FCAS_HD void passm_store(cplx<Real> (&v)[S][PL::EM], cplx<Real>* slot, int tile, int c, int p, int s0 = 0) {
  int j1, k2;
  passm_coords<PL>(tile, c, j1, k2);
  cplx<Real>* at = slot + (int64_t)s0 * PL::N + (int64_t)j1 * PL::W1 + k2;
#pragma unroll
  for (int q = 0; q < PL::EM; ++q) {
    const int o = (p + q * PL::PM) * PL::N2;
#pragma unroll
    for (int s = 0; s < S; ++s) stream_store(at + s * PL::N + o, v[s][q]);
  }
}

// Pass 2 prologue: thread (r, p) of row tile `tile` reads row tile RW + r,
// register q holds k2 = p + q P2.  In a two-pass plan the row is j1, and the
// four-step twiddle w_N^{k2 j1} is the shift of the row's transform (GeoSet);
// in a three-pass plan the middle pass has applied it.
template <typename Real, class PL>
FCAS_HD void pass2_fetch(cplx<Real> (&v)[2][PL::E2], const cplx<Real>* slot, int tile, int r, int p) {
  const int j1 = tile * PL::RW + r;
  const int64_t row = (int64_t)j1 * PL::N2;
#pragma unroll
  for (int q = 0; q < PL::E2; ++q) {
    const int k2 = p + q * PL::P2;
    v[0][q] = stream_load(slot + row + k2);
    v[1][q] = stream_load(slot + PL::N + row + k2);
  }
}

// Pass 2 epilogue: Gamma^2_j = |a_0|^2 + |a_1|^2 (g) at j = row_base + ROWS2 (p + q P2),
// for j_lo <= j < j_hi; the thread's largest value and, among equal values,
// its smallest j (value -1 if none of its samples is in range).
template <typename Real, class PL>
FCAS_HD void pass2_best_of(const Real (&g)[PL::E2], int tile, int r, int p, Real& best, int& best_j, int64_t j_lo,
                           int64_t j_hi) {
  const int j0 = row_base<PL>(tile * PL::RW + r);
  const int lo = j_lo > 0 ? (int)j_lo : 0;
  const int hi = j_hi < PL::N ? (int)j_hi : (int)PL::N;
  best = (Real)-1;
  best_j = 0x7fffffff;
#pragma unroll
  for (int q = 0; q < PL::E2; ++q) {
    const int j = j0 + PL::ROWS2 * (p + q * PL::P2);
    if (g[q] > best && j >= lo && j < hi) {   // j grows with q: ties keep the smaller j
      best = g[q];
      best_j = j;
    }
  }
}

// Work item `item` of the fused schedule (cnt evaluations, lag L, T1 pass-1
// and T2 pass-2 tiles each): kind 1 / 2 = pass 1 / pass 2, list position ep,
// tile.  Sequence: [P1(0..L-1)] then rounds [P1(L + r) P2(r)] then [P2(cnt-L..cnt-1)].
FCAS_HD void fused_decode(int item, int cnt, int L, int T1, int T2, int& kind, int& ep, int& tile) {
  const int T = T1 + T2;
  if (item < L * T1) {
    kind = 1; ep = item / T1; tile = item - ep * T1;
    return;
  }
  const int j = item - L * T1, mid = (cnt - L) * T;
  if (j < mid) {
    const int r = j / T, w = j - r * T;
    if (w < T1) { kind = 1; ep = L + r; tile = w; }
    else { kind = 2; ep = r; tile = w - T1; }
  } else {
    const int k = j - mid;
    kind = 2; ep = (cnt - L) + k / T2; tile = k - (k / T2) * T2;
  }
}

// (g, j) ordering used by every reduction: larger g wins, then smaller j.
template <typename Real>
FCAS_HD bool better(Real g, int j, Real g_ref, int j_ref) {
  return g > g_ref || (g == g_ref && j < j_ref);
}

}  // namespace fcas
