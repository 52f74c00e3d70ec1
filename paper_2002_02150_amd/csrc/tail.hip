// tail.hip -- the end of one PSO iteration in one launch: the fitness of the
// run's points from their pass-2 partials (finalize), the swarm update
// (Sec. III), and the set-up of the next points with their work-list entries.
// One work-group per run, 8 lanes per particle.  Each phase runs the same
// device code as the separate finalize, pso_step and set-up kernels, so an
// iteration ends with the same fitness, swarm and descriptors bit for bit.
#include <algorithm>

#include "launch.hpp"
#include "pso_kernels.hpp"
#include "setup_kernels.hpp"

namespace fcas {

// Bound by latency: about a thousand dependent instructions and four round
// trips to memory, on as many CUs as there are runs.  So lane d of a
// particle's group (d + 4 the same) takes coordinate d, whatever does not
// depend on the fitness is read and drawn before it, the run's best is found
// by a wavefront of its own, and the next position goes from lane to lane.
// One run of 40 particles, two detectors, FP64: 8.6 us with a thread per
// particle and its fitness through memory, 7.1 so (search runs, four detectors: 10.8, 9.0).
template <typename Real>
__global__ void __launch_bounds__(kTailMaxThreads) k_pso_tail(PsoDev p, TailArgs t) {
  constexpr int PM = kTailMaxParticles;
  constexpr int NW = (sizeof(NetDesc) + 7) / 8;
  static_assert(sizeof(NetDesc) % 8 == 0 && NW <= 2 * 64, "two words of the network per thread");
  __shared__ double s_pf[PM], s_px[4 * PM], s_net[NW];
  __shared__ int32_t s_pj[PM];
  const PsoShared sh{s_pf, s_px, s_pj};
  const int r = blockIdx.x, tid = threadIdx.x, P = p.n_particles;
  const int g = tid & 7, d = tid & 3;
  const bool on = (tid >> 3) < P;
  const int k = on ? tid >> 3 : 0;   // the particle of this thread's group; a group without one reads the first's
  const int64_t e = (int64_t)r * P + k;
  // first round trip
  double nw[2];
  for (int u = 0; u < 2; ++u) {
    const int at = tid + u * blockDim.x;
    nw[u] = ((const double*)t.net)[at < NW ? at : 0];
  }
  SetupSeg q{};
  q.s = t.seg_ids[e];
  const int iter = p.iteration[0];
  const double run_best = p.best_f[r];
  const double x = p.x[4 * e + d], v = p.v[4 * e + d];
  double pbx = p.pbest_x[4 * e + d], pb = p.pbest_f[e];
  int32_t pbj = p.pbest_j[e];
  PointPartials<Real, 8> pp;
  pp.load(t.evals[e], (const Real*)t.part_g, t.part_j, t.part_stride, (int)e, g);
  const bool counter = r == 0 && tid < kNumPlans;
  const int count = t.counts_cur[counter ? tid : 0];
  // second round trip: what those values lead to
  pp.load_count(t.plan_parts2);
  setup_seg_fields(q, t.net->max_segments, t.net->n_det, t.segs);
  // even lanes draw stream 2, odd lanes stream 3, and neighbours exchange
  uint32_t c[4];
  random4(p.seed, (uint32_t)(iter + 1), k, r, 2 + (g & 1), c);
  const uint32_t even = d & 2 ? c[2] : c[0], odd = d & 2 ? c[3] : c[1];
  const uint32_t own = d & 1 ? odd : even;
  const uint32_t other = __builtin_amdgcn_update_dpp(0, d & 1 ? even : odd, 0xb1, 0xf, 0xf, true);
  const double r1 = uniform(d & 1 ? other : own), r2 = uniform(d & 1 ? own : other);
  const double w = pso_inertia(p, iter);
  const double lo = d & 2 ? (d & 1 ? p.lo[3] : p.lo[2]) : (d & 1 ? p.lo[1] : p.lo[0]);
  const double span = d & 2 ? (d & 1 ? p.span[3] : p.span[2]) : (d & 1 ? p.span[1] : p.span[0]);
  for (int u = 0; u < 2; ++u)
    if (tid + u * blockDim.x < NW) s_net[tid + u * blockDim.x] = nw[u];
  double f;
  int j;
  finalize_value<Real, 8>(pp, (const Real*)t.part_g, t.part_j, t.part_stride, (int)e, g, f, j);
  // Every load has arrived before the first store leaves: loads and stores
  // complete in one order, and a value that may still be on its way when a
  // store follows it can only be awaited together with the store.
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
  const bool better = f > pb;
  pb = better ? f : pb;
  pbj = better ? j : pbj;
  pbx = better ? x : pbx;
  if (on && g < 4) {
    s_px[4 * k + d] = pbx;
    if (better) p.pbest_x[4 * e + d] = pbx;
    if (g == 0) {
      s_pf[k] = pb;
      s_pj[k] = pbj;
      if (better) {
        p.pbest_f[e] = pb;
        p.pbest_j[e] = pbj;
      }
      t.fitness[e] = f;
      t.argmax[e] = j;
    }
  }
  if (counter) {
    // running total of points evaluated in this iteration (one thread per
    // plan); its list counts are cleared for the iteration after next (the
    // appends below go to the other list set)
    t.counts_cur[tid] = 0;
    if (count) atomicAdd(t.evaluated, (unsigned long long)count);
  }
  __syncthreads();   // the run's personal bests and the network are in LDS
  double vn, xn;
  pso_move(p, w, r1, r2, x, v, pbx, s_px[4 * pso_local_best(s_pf, k, P) + d], vn, xn);
  const double td = pso_theta(lo, span, xn);
  if (on && g < 4) {
    p.v[4 * e + d] = vn;
    p.x[4 * e + d] = xn;
    t.theta[4 * e + d] = td;
  }
  if (t.setup) {
    // the four coordinates from the lanes of the quad
    const double th[4] = {dpp_double<0x00>(td), dpp_double<0x55>(td), dpp_double<0xaa>(td), dpp_double<0xff>(td)};
    setup_group(*(const NetDesc*)s_net, q, th, (int)e, on, t.evals, t.lists_next, t.counts_next, t.list_stride, 1,
                t.err);
  }
  // by the last wavefront, which usually has no particles
  const int lane = tid - ((int)blockDim.x - 64);
  if (lane >= 0) {
    if (lane == 0) pso_advance(p, iter);
    pso_run_best(p, sh, run_best, r, lane);
  }
}

hipError_t launch_pso_tail(int precision, const PsoDev& p, const TailArgs& t, hipStream_t s) {
  if (p.n_particles < 1 || p.n_particles > kTailMaxParticles) return hipErrorInvalidValue;
  // one wavefront more than the particles fill, where there is room for it
  const int threads = std::min((8 * p.n_particles / 64 + 1) * 64, kTailMaxThreads);
  static_assert(kNumPlans <= 64, "one thread per plan count");
  if (precision == 0)
    hipLaunchKernelGGL(k_pso_tail<float>, dim3(p.n_runs), dim3(threads), 0, s, p, t);
  else
    hipLaunchKernelGGL(k_pso_tail<double>, dim3(p.n_runs), dim3(threads), 0, s, p, t);
  return hipGetLastError();
}

}  // namespace fcas
