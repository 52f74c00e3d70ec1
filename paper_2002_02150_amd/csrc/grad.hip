// grad.hip -- dGamma^2/dtheta at the maximising sample j* (held fixed).
//
// Gamma^2 = z^H P z with z^i = sum_k a^i_k,  a^i_k = y^i_k exp(2 pi i [Phi_k + k dly_i + k j*/N]),
// P the projector onto span(V), V = diag(sigma) U(alpha, delta).  For a
// parameter t:
//   d z^i   = 2 pi i [ sum_p (d coef_p / dt) sum_k a_k b_k^{e_p} + (d dly_i / dt) sum_k a_k k ]
//   d Gamma^2 = 2 Re[(P z)^H dz] + 2 Re[r^H dV w],   w = (V^T V)^-1 V^T z,  r = z - V w,
// the second term being z^H dP z for the derivative of an orthogonal projector.
#include "grad_kernels.hpp"

#include "setup_kernels.hpp"

namespace fcas {

// Sums NV doubles per lane over the 64 lanes of a wavefront: while the count
// is even, half of the values go to the other half of the lanes (NV/2
// exchanges instead of NV), the rest is a butterfly.  `base` receives the
// index of the lane's first total, the count of totals it holds is returned
// (v[0 .. count)); lanes whose low bits agree hold the same totals.
template <int NV, int OFF>
__device__ __forceinline__ int wave_totals(double* v, int lane, int& base) {
  if constexpr (OFF == 0) {
    return NV;
  } else if constexpr (NV % 2 == 0) {
    constexpr int H = NV / 2;
    const bool up = (lane & OFF) != 0;
#pragma unroll
    for (int m = 0; m < H; ++m) {
      const double send = up ? v[m] : v[H + m], keep = up ? v[H + m] : v[m];
      v[m] = keep + __shfl_xor(send, OFF, 64);
    }
    if (up) base += H;
    return wave_totals<H, OFF / 2>(v, lane, base);
  } else {
#pragma unroll
    for (int m = 0; m < NV; ++m) v[m] += __shfl_xor(v[m], OFF, 64);
    return wave_totals<NV, OFF / 2>(v, lane, base);
  }
}

// Blocks (point, group of DT detectors, part): each part sums a strided share
// of the in-band bins into six complex FP64 partial sums per detector; the
// chain kernel adds the parts in a fixed order (deterministic).
//
// Bound by vector instructions: 12 FP64 multiply-adds per bin and detector,
// plus the phase.  A thread takes every detector of its group at a bin, so
// that the template phase, the powers of b and the sample ramp k j*/N (cycles)
// are formed once per bin; the ramp's numerator k j* mod N advances by a
// constant from bin to bin (an add and a conditional subtract: exact for
// every N).  4096 points of 4 x 131072 samples: 2.96 ms with one detector per
// block, a 64-bit remainder and a division per bin and twelve tree sums;
// 1.35 ms so (0.7 of the vector instruction rate).
template <typename Real, int DT>
__global__ void __launch_bounds__(kAdjThreads) k_adjoint_sums(const SegDesc* __restrict__ segs,
                                                              const EvalDesc* __restrict__ evals,
                                                              const int32_t* __restrict__ argmax, int n_det,
                                                              int parts, double* __restrict__ sums) {
  constexpr int NV = DT * kAdjSums * 2, NW = kAdjThreads / 64;
  const int e = blockIdx.x, i0 = blockIdx.y * DT, part = blockIdx.z;
  const EvalDesc& ev = evals[e];
  const int tid = threadIdx.x;
  // sums[e][i][part][sum][re, im]
  double* out = sums + ((int64_t)e * n_det * parts + part) * kAdjSums * 2;
  const int nd = n_det - i0 < DT ? n_det - i0 : DT;   // detectors of this group (the last may hold fewer)
  if (ev.status != 1) {
    if (tid < nd * kAdjSums * 2) {
      const int d = tid / (kAdjSums * 2);
      out[(int64_t)(i0 + d) * parts * kAdjSums * 2 + tid - d * (kAdjSums * 2)] = 0.0;
    }
    return;
  }
  const SegDesc& sg = segs[ev.seg];
  const int64_t N = sg.n;
  const int64_t jstar = argmax[e];
  const cplx<Real>* y = (const cplx<Real>*)sg.y + i0;
  const double* bt = sg.b;
  const int k_lo = sg.k_lo, k_hi = sg.k_hi;
  double dly[DT];
  int at[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) {
    at[d] = d < nd ? d : 0;   // a missing detector repeats the first one's; its sums are not written
    dly[d] = ev.dly[i0 + at[d]];
  }
  const double coef[4] = {ev.coef[0], ev.coef[1], ev.coef[2], ev.coef[3]};
  const double inv_n = 1.0 / (double)N;
  const int stride = kAdjThreads * parts;
  int k = k_lo + part * kAdjThreads + tid;
  uint32_t m = (uint32_t)(((int64_t)k * jstar) % N);
  const uint32_t dm = (uint32_t)(((int64_t)stride * jstar) % N), nn = (uint32_t)N;
  double acc[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) acc[c] = 0.0;
  for (; k <= k_hi; k += stride) {
    const int kk = k - k_lo;
    const double b = bt[kk];
    cplx<Real> yv[DT];
#pragma unroll
    for (int d = 0; d < DT; ++d) yv[d] = y[(int64_t)kk * n_det + at[d]];
    const double phc = common_phase(coef, b);
    const double ramp = (double)m * inv_n;
    m += dm;
    m = m >= nn ? m - nn : m;
    const double b2 = b * b, b3 = b2 * b, b5 = b3 * b2;
    const double kd = (double)k;
#pragma unroll
    for (int d = 0; d < DT; ++d) {
      const double ph = kd * dly[d] + phc + ramp;
      const double r = ph - rint(ph);
      Real sn, cs;
      sincos_rev((Real)r, &sn, &cs);
      const cplx<Real> a = mul(yv[d], mk<Real>(cs, sn));
      const double ax = (double)a.x, ay = (double)a.y;
      double* s = acc + d * kAdjSums * 2;
      s[0] += ax;
      s[1] += ay;
      s[2] += b5 * ax;
      s[3] += b5 * ay;
      s[4] += b3 * ax;
      s[5] += b3 * ay;
      s[6] += b2 * ax;
      s[7] += b2 * ay;
      s[8] += b * ax;
      s[9] += b * ay;
      s[10] += kd * ax;
      s[11] += kd * ay;
    }
  }
  __shared__ double red[NW][NV];
  int base = 0;
  const int held = wave_totals<NV, 32>(acc, tid & 63, base);
  // lanes that hold the same totals write the same values
  for (int c = 0; c < held; ++c) red[tid >> 6][base + c] = acc[c];
  __syncthreads();
  if (tid < nd * kAdjSums * 2) {
    double t = red[0][tid];
#pragma unroll
    for (int w = 1; w < NW; ++w) t += red[w][tid];
    const int d = tid / (kAdjSums * 2);
    out[(int64_t)(i0 + d) * parts * kAdjSums * 2 + tid - d * (kAdjSums * 2)] = t;
  }
}

// d coef / d tau0, d coef / d tau1.5 for coef = f* (0.6 tau0, tau1, -1.5 tau1.5, 3 tau2).
__device__ void coef_derivatives(double tau0, double tau15, double fs, double dc[2][4]) {
  const double v0 = cbrt(5.0 * tau15 / (32.0 * kPi * tau0));
  const double eta = 1.0 / (8.0 * fs * tau15 * v0 * v0);
  // logarithmic derivatives of v0 and eta
  const double dlv[2] = {-1.0 / (3.0 * tau0), 1.0 / (3.0 * tau15)};
  const double dle[2] = {2.0 / (3.0 * tau0), -5.0 / (3.0 * tau15)};
  const double A1 = 5.0 / (192.0 * kPi * fs), A2 = 5.0 / (128.0 * kPi * fs);
  const double iv3 = 1.0 / (v0 * v0 * v0), iv = 1.0 / v0;
  const double B0 = 3058673.0 / 1016064.0, B1 = 5429.0 / 1008.0, B2 = 617.0 / 144.0;
  for (int q = 0; q < 2; ++q) {
    // tau1 = A1 [ (743/336) eta^-1 v0^-3 + (11/4) v0^-3 ]
    const double dtau1 = A1 * ((743.0 / 336.0) / eta * iv3 * (-dle[q] - 3.0 * dlv[q]) + 2.75 * iv3 * (-3.0 * dlv[q]));
    // tau2 = A2 [ B0 eta^-1 v0^-1 + B1 v0^-1 + B2 eta v0^-1 ]
    const double dtau2 = A2 * (B0 / eta * iv * (-dle[q] - dlv[q]) + B1 * iv * (-dlv[q]) + B2 * eta * iv * (dle[q] - dlv[q]));
    dc[q][0] = fs * (q == 0 ? 0.6 : 0.0);
    dc[q][1] = fs * dtau1;
    dc[q][2] = fs * (q == 1 ? -1.5 : 0.0);
    dc[q][3] = fs * 3.0 * dtau2;
  }
}

// One wavefront per point: its lanes add the parts of the six sums (fixed
// order, deterministic), then apply the chain rule in FP64, lane 8 q + i
// holding detector i for parameter q (alpha, delta, tau0, tau1.5); sums over
// detectors are butterflies inside a group of 8 lanes.  Bound by the latency
// of its dependent FP64 operations (8 points: 14 us when one thread did it).
// Returns component q in the lanes of group q (0 for a point not evaluated);
// S: LDS of kMaxDet kAdjSums 2 doubles.
__device__ __forceinline__ double chain_rule(const NetDesc& net, const SegDesc* __restrict__ segs,
                                             const EvalDesc* __restrict__ evals, const double* __restrict__ theta,
                                             const double* __restrict__ sums, int parts, int e, double* S) {
  const int lane = threadIdx.x;
  const EvalDesc& ev = evals[e];
  if (ev.status != 1) return 0.0;
  const int D = net.n_det;
  const int q = (lane >> 3) & 3, i = lane & 7;   // lanes 32..63 repeat lanes 0..31
  const bool on = i < D;
  // everything that does not depend on the sums is read first
  const SegDesc& sg = segs[ev.seg];
  const double df = sg.df, sigma = on ? sg.sigma[i] : 0.0;
  const double* th = theta + 4 * (int64_t)e;
  const double alpha = th[0], delta = th[1], tau0 = th[2], tau15 = th[3];
  const double q0 = on ? ev.q[i][0] : 0.0, q1 = on ? ev.q[i][1] : 0.0;
  const double v0 = on ? ev.v[i][0] : 0.0, v1 = on ? ev.v[i][1] : 0.0;
  const bool full = (ev.rank == 2);
  double pos[3] = {0.0, 0.0, 0.0}, ten[3][3] = {};
  if (on)
    for (int a = 0; a < 3; ++a) {
      pos[a] = net.pos[i][a];
      for (int b = 0; b < 3; ++b) ten[a][b] = net.ten[i][a][b];
    }
  for (int m = lane; m < D * kAdjSums * 2; m += 64) {
    const int d = m / (kAdjSums * 2), c = m - d * (kAdjSums * 2);
    const double* s = sums + ((int64_t)e * D + d) * parts * kAdjSums * 2 + c;
    double t = 0.0;
    // batches of eight loads in flight
    int part = 0;
    for (; part + 8 <= parts; part += 8) {
      double u[8];
#pragma unroll
      for (int w = 0; w < 8; ++w) u[w] = s[(part + w) * kAdjSums * 2];
      t += ((u[0] + u[1]) + (u[2] + u[3])) + ((u[4] + u[5]) + (u[6] + u[7]));
    }
    for (; part < parts; ++part) t += s[part * kAdjSums * 2];
    S[m] = t;
  }
  double sa, ca, sd, cd;
  sincos(alpha, &sa, &ca);
  sincos(delta, &sd, &cd);
  const double ex[3] = {sa, -ca, 0.0}, ey[3] = {-sd * ca, -sd * sa, cd};
  // derivatives of n, e_X = -alpha_hat, e_Y = delta_hat with respect to alpha (q = 0) or delta
  const bool qa = (q == 0);
  const double dn[3] = {qa ? -cd * sa : -sd * ca, qa ? cd * ca : -sd * sa, qa ? 0.0 : cd};
  const double dex[3] = {qa ? ca : 0.0, qa ? sa : 0.0, 0.0};
  const double dey[3] = {qa ? sd * sa : -cd * ca, qa ? -sd * ca : -cd * sa, qa ? 0.0 : -sd};
  const double ddl = -(dn[0] * pos[0] + dn[1] * pos[1] + dn[2] * pos[2]) / kC * df;
  double up = 0.0, uc = 0.0;
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) {
      const double d = ten[a][b];
      up += d * (dex[a] * ex[b] + ex[a] * dex[b] - dey[a] * ey[b] - ey[a] * dey[b]);
      uc += d * (dex[a] * ey[b] + ex[a] * dey[b] + dey[a] * ex[b] + ey[a] * dex[b]);
    }
  const double dV0 = sigma * up, dV1 = sigma * uc;
  double dc[2][4];
  coef_derivatives(tau0, tau15, net.f_star, dc);
  __syncthreads();   // S
  double Si[kAdjSums * 2];
  for (int c = 0; c < kAdjSums * 2; ++c) Si[c] = on ? S[i * kAdjSums * 2 + c] : 0.0;
  const double zr = Si[0], zi = Si[1];
  // P z = Q (Q^T z)
  const double c0r = sum8(q0 * zr), c0i = sum8(q0 * zi), c1r = sum8(q1 * zr), c1i = sum8(q1 * zi);
  const double pz_r = q0 * c0r + q1 * c1r, pz_i = q0 * c0i + q1 * c1i;
  // w = (V^T V)^-1 V^T z (rank two only), r = z - V w
  double wr0 = 0, wi0 = 0, wr1 = 0, wi1 = 0, rr = 0, ri = 0;
  if (full) {
    const double G00 = sum8(v0 * v0), G01 = sum8(v0 * v1), G11 = sum8(v1 * v1);
    const double br0 = sum8(v0 * zr), bi0 = sum8(v0 * zi), br1 = sum8(v1 * zr), bi1 = sum8(v1 * zi);
    const double det = G00 * G11 - G01 * G01;
    wr0 = (G11 * br0 - G01 * br1) / det; wi0 = (G11 * bi0 - G01 * bi1) / det;
    wr1 = (G00 * br1 - G01 * br0) / det; wi1 = (G00 * bi1 - G01 * bi0) / det;
    rr = zr - (v0 * wr0 + v1 * wr1);
    ri = zi - (v0 * wi0 + v1 * wi1);
  }
  // d z^i = 2 pi i * s, s = sum_p dcoef_p S_p + ddly S_k
  double sr = 0.0, si = 0.0;
  if (q >= 2) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const double d = q == 2 ? dc[0][p] : dc[1][p];
      sr += d * Si[(1 + p) * 2];
      si += d * Si[(1 + p) * 2 + 1];
    }
  } else {
    sr = ddl * Si[10];
    si = ddl * Si[11];
  }
  const double twopi = 2.0 * kPi;
  const double dzr = -twopi * si, dzi = twopi * sr;
  // 2 Re(conj(Pz_i) dz_i)
  double acc = 2.0 * (pz_r * dzr + pz_i * dzi);
  if (q < 2 && full) {
    // 2 Re(conj(r_i) (dV_i0 w_0 + dV_i1 w_1))
    const double tr = dV0 * wr0 + dV1 * wr1;
    const double ti = dV0 * wi0 + dV1 * wi1;
    acc += 2.0 * (rr * tr + ri * ti);
  }
  return sum8(acc);
}

__global__ void __launch_bounds__(64) k_chain(const NetDesc* __restrict__ netp, const SegDesc* __restrict__ segs,
                                              const EvalDesc* __restrict__ evals, const double* __restrict__ theta,
                                              const double* __restrict__ sums, int parts, int n,
                                              double* __restrict__ grad) {
  __shared__ double S[kMaxDet * kAdjSums * 2];
  const int e = blockIdx.x, lane = threadIdx.x;
  const double g = chain_rule(*netp, segs, evals, theta, sums, parts, e, S);
  if (lane < 32 && (lane & 7) == 0) grad[4 * (int64_t)e + (lane >> 3)] = g;
}


// One polish step around its fitness batch, two kernels of one wavefront per
// point (bound by latency: as five kernels a step of 8 points took 23 us more).
//
// Before it: the gradient by the chain rule, the trials
//   theta_t = theta + step_frac 2^-t w^2 g / |w g|, t = 0..T-1
// (w = widths of the search rectangle, same segment as the point) and their
// set-up, eight at a time.  `evals` holds the points' descriptors, apart from the
// trials' (`trial_evals`), which other work-groups write meanwhile.
__global__ void __launch_bounds__(64) k_polish_trials(const NetDesc* __restrict__ netp,
                                                      const SegDesc* __restrict__ segs,
                                                      const EvalDesc* __restrict__ evals,
                                                      const double* __restrict__ theta,
                                                      const int32_t* __restrict__ seg,
                                                      const double* __restrict__ sums, int parts, int trials,
                                                      double step_frac, double* __restrict__ cand,
                                                      EvalDesc* __restrict__ trial_evals, int32_t* __restrict__ lists,
                                                      int32_t* __restrict__ counts, int list_stride,
                                                      int32_t* __restrict__ err) {
  __shared__ double S[kMaxDet * kAdjSums * 2], th_s[8][4];
  const NetDesc& net = *netp;
  const int e = blockIdx.x, lane = threadIdx.x, k = lane >> 3, d = lane & 3;
  const SetupSeg q = setup_seg_load(net, segs, seg, e, true);
  const double gq = chain_rule(net, segs, evals, theta, sums, parts, e, S);
  double g[4], w[4], nrm = 0.0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    g[c] = __shfl(gq, 8 * c, 64);
    w[c] = net.box_hi[c] - net.box_lo[c];
    nrm += (w[c] * g[c]) * (w[c] * g[c]);
  }
  nrm = sqrt(nrm);
  const double gd = d == 0 ? g[0] : d == 1 ? g[1] : d == 2 ? g[2] : g[3];
  const double wd = d == 0 ? w[0] : d == 1 ? w[1] : d == 2 ? w[2] : w[3];
  const double td = theta[4 * (int64_t)e + d];
  for (int t0 = 0; t0 < trials; t0 += 8) {
    const int t = t0 + k;
    const double s = ldexp(step_frac, -t);
    const double x = td + (nrm > 0.0 ? s * wd * wd * gd / nrm : 0.0);
    const int64_t o = (int64_t)e * trials + t;
    if ((lane & 7) < 4) {
      th_s[k][d] = x;
      if (t < trials) cand[4 * o + d] = x;
    }
    __syncthreads();
    setup_group(net, q, th_s[k], (int)o, t < trials, trial_evals, lists, counts, list_stride, 1, err);
    __syncthreads();
  }
}

// After it: the trials' fitness from their pass-2 partials, each point moved to
// its best trial if that raises its fitness, and (more) the descriptors of the
// points for the next step; the work-list counts are cleared.
template <typename Real>
__global__ void __launch_bounds__(64) k_polish_select(const NetDesc* __restrict__ netp,
                                                      const SegDesc* __restrict__ segs, EvalDesc* __restrict__ evals,
                                                      double* __restrict__ theta, const int32_t* __restrict__ seg,
                                                      double* __restrict__ fitness, int32_t* __restrict__ argmax,
                                                      const double* __restrict__ cand,
                                                      const EvalDesc* __restrict__ trial_evals,
                                                      const Real* __restrict__ part_g,
                                                      const int32_t* __restrict__ part_j, int part_stride,
                                                      const int32_t* __restrict__ plan_parts2, int trials,
                                                      int32_t* __restrict__ counts,
                                                      unsigned long long* __restrict__ evaluated, int more,
                                                      int32_t* __restrict__ err) {
  __shared__ double f_s[kMaxTrials], th_s[4];
  __shared__ int32_t j_s[kMaxTrials];
  const NetDesc& net = *netp;
  const int e = blockIdx.x, lane = threadIdx.x, k = lane >> 3;
  const int64_t first = (int64_t)e * trials;
  const SetupSeg q = setup_seg_load(net, segs, seg, e, more && k == 0);
  if (e == 0 && lane < kNumPlans) {
    const int c = counts[lane];
    counts[lane] = 0;
    if (c) atomicAdd(evaluated, (unsigned long long)c);
  }
  for (int t0 = 0; t0 < trials; t0 += 8) {
    const int t = t0 + k;
    if (t < trials) {
      double f;
      int j;
      PointPartials<Real, 8> pp;
      pp.load(trial_evals[first + t], part_g, part_j, part_stride, (int)(first + t), lane & 7);
      pp.load_count(plan_parts2);
      finalize_value<Real, 8>(pp, part_g, part_j, part_stride, (int)(first + t), lane & 7, f, j);
      if ((lane & 7) == 0) {
        f_s[t] = f;
        j_s[t] = j;
      }
    }
  }
  __syncthreads();
  int best = -1;
  double fb = fitness[e];
  for (int t = 0; t < trials; ++t)
    if (f_s[t] > fb) {
      fb = f_s[t];
      best = t;
    }
  if (lane < 4) {
    const double x = best >= 0 ? cand[4 * (first + best) + lane] : theta[4 * (int64_t)e + lane];
    th_s[lane] = x;
    if (best >= 0) theta[4 * (int64_t)e + lane] = x;
  }
  if (best >= 0 && lane == 0) {
    fitness[e] = fb;
    argmax[e] = j_s[best];
  }
  if (!more) return;
  __syncthreads();
  setup_group(net, q, th_s, e, k == 0, evals, nullptr, nullptr, 0, 0, err);
}

// Detectors per adjoint block: every detector up to four (24 registers of
// sums each), networks of five to eight in two groups.
static int adj_group(int n_det) { return n_det <= 4 ? n_det : (n_det + 1) / 2; }
static int grad_parts(int n, int n_det, int64_t bins) { return adjoint_parts(n, n_det <= 4 ? 1 : 2, bins); }

hipError_t launch_polish_trials(const GradBuffers& g, const NetDesc* net, const SegDesc* segs, const EvalDesc* evals,
                                const double* theta, const int32_t* seg, int n, int n_det, int trials,
                                double step_frac, double* cand, EvalDesc* trial_evals, int32_t* lists,
                                int32_t* counts, int list_stride, int64_t bins, int32_t* err, hipStream_t s) {
  hipLaunchKernelGGL(k_polish_trials, dim3(n), dim3(64), 0, s, net, segs, evals, theta, seg, g.sums,
                     grad_parts(n, n_det, bins), trials, step_frac, cand, trial_evals, lists, counts, list_stride, err);
  return hipGetLastError();
}

hipError_t launch_polish_select(int precision, const NetDesc* net, const SegDesc* segs, EvalDesc* evals,
                                double* theta, const int32_t* seg, double* fitness, int32_t* argmax,
                                const double* cand, const EvalDesc* trial_evals, const void* part_g,
                                const int32_t* part_j, int part_stride, const int32_t* plan_parts2, int n, int trials,
                                int32_t* counts, unsigned long long* evaluated, int more, int32_t* err,
                                hipStream_t s) {
  if (precision == 0)
    hipLaunchKernelGGL(k_polish_select<float>, dim3(n), dim3(64), 0, s, net, segs, evals, theta, seg, fitness, argmax,
                       cand, trial_evals, (const float*)part_g, part_j, part_stride, plan_parts2, trials, counts,
                       evaluated, more, err);
  else
    hipLaunchKernelGGL(k_polish_select<double>, dim3(n), dim3(64), 0, s, net, segs, evals, theta, seg, fitness, argmax,
                       cand, trial_evals, (const double*)part_g, part_j, part_stride, plan_parts2, trials, counts,
                       evaluated, more, err);
  return hipGetLastError();
}

int alloc_grad_buffers(GradBuffers& g, int max_batch, int n_det) {
  g.max_batch = max_batch;
  g.n_det = n_det;
  // n * adjoint_parts(n, ...) <= n + 1024 for every n
  const size_t entries = ((size_t)max_batch + 1024) * n_det;
  const size_t bytes = entries * kAdjSums * 2 * sizeof(double);
  if (hipMalloc((void**)&g.sums, bytes) != hipSuccess) {
    g.sums = nullptr;
    return -5;
  }
  return 0;
}

void free_grad_buffers(GradBuffers& g) {
  if (g.sums) hipFree(g.sums);
  g.sums = nullptr;
}

hipError_t launch_adjoint(int precision, const GradBuffers& g, const SegDesc* segs, const EvalDesc* evals,
                          const int32_t* argmax, int n, int n_det, int64_t bins, hipStream_t s) {
  const int parts = grad_parts(n, n_det, bins);
  const int dt = adj_group(n_det);
  const dim3 grid(n, (n_det + dt - 1) / dt, parts), block(kAdjThreads);
#define FCAS_ADJOINT(DT)                                                                                    \
  case DT:                                                                                                  \
    if (precision == 0)                                                                                     \
      hipLaunchKernelGGL((k_adjoint_sums<float, DT>), grid, block, 0, s, segs, evals, argmax, n_det, parts, \
                         g.sums);                                                                           \
    else                                                                                                    \
      hipLaunchKernelGGL((k_adjoint_sums<double, DT>), grid, block, 0, s, segs, evals, argmax, n_det, parts, \
                         g.sums);                                                                           \
    break;
  switch (dt) {
    FCAS_ADJOINT(1)
    FCAS_ADJOINT(2)
    FCAS_ADJOINT(3)
    FCAS_ADJOINT(4)
    default:
      return hipErrorInvalidValue;
  }
#undef FCAS_ADJOINT
  return hipGetLastError();
}

hipError_t launch_gradient(int precision, const GradBuffers& g, const NetDesc* net, const SegDesc* segs,
                           const EvalDesc* evals, const double* theta, const int32_t* argmax, int n, int n_det,
                           double* grad, int64_t bins, hipStream_t s) {
  const hipError_t e = launch_adjoint(precision, g, segs, evals, argmax, n, n_det, bins, s);
  if (e != hipSuccess) return e;
  const int parts = grad_parts(n, n_det, bins);
  hipLaunchKernelGGL(k_chain, dim3(n), dim3(64), 0, s, net, segs, evals, theta, g.sums, parts, n, grad);
  return hipGetLastError();
}

}  // namespace fcas
