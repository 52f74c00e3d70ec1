// setup_kernels.hpp -- the per-point set-up on the device: eight lanes per
// point, the descriptor and the append to its plan's work list.  Used by the
// set-up kernel of every fitness call and by the kernel that ends a PSO
// iteration.
#pragma once

#include "eval_kernels.hpp"

namespace fcas {

// A double from the lane that a DPP control names.
template <int CTRL>
__device__ __forceinline__ double dpp_double(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Sum over an aligned group of 8 lanes, in every lane: pairs, quads (both quad
// permutations), then the two quads (each lane reads its mirror image in the
// group of 8).  The same additions as a butterfly of shuffles, without the
// LDS round trip of each.
__device__ __forceinline__ double sum8(double x) {
  x += dpp_double<0xb1>(x);    // quad_perm 1,0,3,2
  x += dpp_double<0x4e>(x);    // quad_perm 2,3,0,1
  x += dpp_double<0x141>(x);   // row_half_mirror
  return x;
}

// The detectors of one point as a group of 8 lanes, lane g holding detector g;
// sums over detectors are butterfly reductions inside the group of eight
// (every lane gets the same, order-independent total: IEEE addition commutes).
struct DetLanes {
  bool on;       // this lane holds a detector
  DetPoint p;
  template <class F> __device__ double sum(F f) const { return sum8(on ? f(p) : 0.0); }
  template <class F> __device__ void each(F f) { f(p); }
};
static_assert(kMaxDet == 8, "one lane per detector slot in a group of 8");

// What the set-up of one point reads of its segment: the segment id, whether
// it can be evaluated, and the segment's plan, bin width, pass-1 register
// stride and (lane g) detector g's template norm.
struct SetupSeg {
  int32_t s, ok, plan, dk1;
  double df, sigma_g;
};

// The fields of segment q.s.
__device__ __forceinline__ void setup_seg_fields(SetupSeg& q, int max_segments, int n_det,
                                                 const SegDesc* __restrict__ segs) {
  // the descriptor is read ahead of the check; a bad id reads segment 0's
  const bool in_table = q.s >= 0 && q.s < max_segments;
  const SegDesc& sg = segs[in_table ? q.s : 0];
  q.ok = in_table && sg.registered;
  q.plan = sg.plan;
  q.dk1 = sg.dk1;
  q.df = sg.df;
  const int g = threadIdx.x & 7;
  q.sigma_g = g < n_det ? sg.sigma[g] : 0.0;
}

__device__ __forceinline__ SetupSeg setup_seg_load(const NetDesc& net, const SegDesc* __restrict__ segs,
                                                   const int32_t* __restrict__ seg_ids, int e, bool valid) {
  SetupSeg q{};
  if (!valid) return q;
  q.s = seg_ids[e];
  setup_seg_fields(q, net.max_segments, net.n_det, segs);
  return q;
}

// Sine and cosine of x, reduced to half turns by the product with 1 / pi in two
// parts (no branch on the size of x: |x| < 2^52).
__device__ __forceinline__ void sincos_turns(double x, double* s, double* c) {
  const double i1 = 0x1.45f306dc9c883p-2, i2 = -0x1.6b01ec5417056p-56;   // 1 / pi
  const double t = x * i1, k = rint(t);
  const double e = __builtin_fma(x, i2, __builtin_fma(x, i1, -t));
  double sn, cs;
  sincospi((t - k) + e, &sn, &cs);
  const bool odd = k != 2.0 * rint(0.5 * k);
  *s = odd ? -sn : sn;
  *c = odd ? -cs : cs;
}

// Whether a point lies in the search rectangle (finite, bounds included).
__device__ __forceinline__ bool inside_box(const NetDesc& net, const double* th) {
  bool inside = true;
  for (int d = 0; d < 4; ++d) {
    const double t = th[d];
    inside = inside && isfinite(t) && t >= net.box_lo[d] && t <= net.box_hi[d];
  }
  return inside;
}

// The FP64 set-up of a point in the rectangle by a group of 8 lanes (lane g):
// phase coefficients and rank in every lane, detector g in dets.p.  Bound by
// the latency of about 400 dependent FP64 operations, so its chains are kept
// short: roots and their reciprocals in one (inv_cbrt, inv_sqrt), no quotient
// that waits for another, no branch on the size of an angle (3.1 -> 2.3 us of
// the kernel that ends a PSO iteration).
__device__ __forceinline__ int setup_math(const NetDesc& net, const SetupSeg& q, const double* th, int g,
                                          double coef[4], DetLanes& dets) {
  SkyFrame fr;
  setup_phase(th[2], th[3], net.f_star, coef);
  // one sine and cosine for both angles: odd lanes take delta's
  double s1, c1;
  sincos_turns(g & 1 ? th[1] : th[0], &s1, &c1);
  const double s2 = dpp_double<0xb1>(s1), c2 = dpp_double<0xb1>(c1);
  setup_sky(g & 1 ? s2 : s1, g & 1 ? c2 : c1, g & 1 ? s1 : s2, g & 1 ? c1 : c2, fr);
  dets.on = g < net.n_det;
  setup_detector(net, q.df, q.sigma_g, fr, dets.on ? g : 0, dets.p);
  // detector 0's delay ramp, from lane 0 of the group (by its quad, then the
  // other quad's mirror image)
  const double d0 = dpp_double<0x00>(dets.p.dly), d1 = dpp_double<0x141>(d0);
  setup_step(q.dk1, g < 4 ? d0 : d1, dets.p);
  return setup_basis(dets);
}

// Set-up of point e (valid) by the 8-lane group holding it, given its segment
// (setup_seg_load) and its parameters th[4]: status, the FP64 set-up with the
// per-detector work spread over the lanes, and (build_lists) the append to
// its plan's work list.  Every lane of the wavefront calls it, lanes without
// a point with valid = false: list entries of one wavefront that share a plan
// are appended with a single atomic.
__device__ __forceinline__ void setup_group(const NetDesc& net, const SetupSeg& q, const double* th, int e,
                                            bool valid, EvalDesc* __restrict__ evals, int32_t* __restrict__ lists,
                                            int32_t* __restrict__ counts, int list_stride, int build_lists,
                                            int32_t* __restrict__ err) {
  const int lane = threadIdx.x & 63, g = threadIdx.x & 7;
  int plan = -1;   // on lane 0 of a group: plan of a point to append to its list, else -1
  if (valid) {
    EvalDesc& ev = evals[e];
    if (!q.ok) {
      if (g == 0) {
        ev.seg = q.s;
        ev.status = -2;
        ev.plan = 0;
        atomicOr(err, 1);
      }
    } else {
      const bool inside = inside_box(net, th);
      if (inside) {
        double coef[4];
        DetLanes dets{};
        const int rank = setup_math(net, q, th, g, coef, dets);
        if (dets.on) store_detector(ev, g, dets.p);
        if (g == 0) {
          for (int k = 0; k < 4; ++k) ev.coef[k] = coef[k];
          ev.rank = rank;
          if (build_lists) plan = q.plan;
        }
      }
      if (g == 0) {
        ev.seg = q.s;
        ev.plan = q.plan;
        ev.status = inside ? 1 : 0;
      }
    }
  }
  unsigned long long todo = __ballot(plan >= 0);
  while (todo) {
    const int leader = __ffsll((long long)todo) - 1;
    const int lp = __shfl(plan, leader, 64);
    const unsigned long long same = __ballot(plan == lp);
    int base = 0;
    if (lane == leader) base = atomicAdd(counts + lp, __popcll(same));
    base = __shfl(base, leader, 64);
    if (plan == lp) lists[(int64_t)lp * list_stride + base + __popcll(same & ((1ull << lane) - 1))] = e;
    todo &= ~same;
  }
}

}  // namespace fcas
