// direct_kernels.hpp -- pass 1 of a small call with the points' set-up inside.
#pragma once

#include "setup_kernels.hpp"

namespace fcas {

// Every dword of a work-group-uniform value moved to scalar registers.
template <class T>
__device__ __forceinline__ T uniform_copy(const T& x) {
  static_assert(sizeof(T) % 4 == 0, "dwords");
  constexpr int W = sizeof(T) / 4;
  struct Words { int32_t w[W]; };
  Words u = __builtin_bit_cast(Words, x);
#pragma unroll
  for (int k = 0; k < W; ++k) u.w[k] = __builtin_amdgcn_readfirstlane(u.w[k]);
  return __builtin_bit_cast(T, u);
}

// Work-group b: tile b mod TILES1 of point b / TILES1.  Its first wavefront
// sets the point up (every work-group of the point does, in LDS; tile 0's also
// writes the descriptor) while the segment data are on their way, so a call
// that gives no work-group a second point needs no set-up kernel, no work list
// and no reads of a descriptor that another kernel wrote.  Bound by latency
// (the set-up's dependent operations, one round of the tile's transform): one
// point of 131072 samples, set-up kernel and pass 1 4.2 + 8.2 us, this one 9.2.
template <typename Real, class PL, int DT>
__global__ void __launch_bounds__(PL::T1) __attribute__((amdgpu_waves_per_eu(PassTune<Real, PL, DT>::waves1)))
k_pass1_direct(PassArgs a, DirectArgs d) {
  constexpr int LP = PassLds<Real, PL>::LP1;
  __shared__ cplx<Real> lds[PassLds<Real, PL>::X1];
  __shared__ Pass1Point<Real, DT> shared_point;
  const int tid = threadIdx.x;
  const int e = blockIdx.x / PL::TILES1, tile = blockIdx.x - e * PL::TILES1;
  const bool writer = tile == 0;
  EvalDesc& ev = d.evals[e];
  const NetDesc& net = *d.net;
  const int s = *const_view(d.seg_ids + e);
  // the descriptor is read ahead of the check; a bad id reads segment 0's
  const bool in_table = s >= 0 && s < const_view(d.net)->max_segments;
  const SegDesc sg = *const_view(a.segs + (in_table ? s : 0));
  if (!in_table || !sg.registered || sg.plan != d.plan) {
    if (writer && tid == 0) {
      ev.seg = s;
      ev.status = -2;
      ev.plan = 0;
      atomicOr(d.err, 1);
    }
    return;
  }
  const double* th = d.theta + 4 * (int64_t)e;
  if (!inside_box(net, th)) {
    if (writer && tid == 0) {
      ev.seg = s;
      ev.status = 0;
      ev.plan = sg.plan;
    }
    return;
  }
  const int c = tid % PL::C, p = tid / PL::C;
  Pass1Data<Real, PL, DT> data;
  pass1_fetch<Real, PL, DT>(data, sg, tile, c, p);
  if (tid < 64) {
    const int g = tid & 7;
    SetupSeg q{};
    q.dk1 = sg.dk1;
    q.df = sg.df;
    q.sigma_g = g < net.n_det ? a.segs[s].sigma[g] : 0.0;
    double coef[4];
    DetLanes dets{};
    const int rank = setup_math(net, q, th, g, coef, dets);
    if (tid < DT) {
      shared_point.dly[tid] = dets.p.dly;
      for (int m = 0; m < 2; ++m) {
        shared_point.q[tid][m] = (Real)dets.p.q[m];
        shared_point.step[tid][m] = (Real)dets.p.step[m];
      }
    }
    if (tid == 0)
      for (int k = 0; k < 4; ++k) shared_point.coef[k] = coef[k];
    if (writer) {
      if (tid < DT) store_detector(ev, tid, dets.p);
      if (tid == 0) {
        for (int k = 0; k < 4; ++k) ev.coef[k] = coef[k];
        ev.rank = rank;
        ev.seg = s;
        ev.status = 1;
        ev.plan = sg.plan;
        atomicAdd(d.evaluated, 1ull);
      }
    }
  }
  Pass1Geo<Real, PL> geo;
  geo.init(p);
  __syncthreads();
  cplx<Real> v[2][PL::E1];
  pass1_compute<Real, PL, DT>(v, data, uniform_copy(shared_point));
  cplx<Real>* buf0 = lds + c * LP;
  cplx<Real>* buf1 = PassTune<Real, PL>::joint1 ? lds + (PL::C + c) * LP : buf0;
  pass1_transform<Real, PL, false>(v, (cplx<Real>*)a.ws + (int64_t)e * 2 * PL::N, buf0, buf1, geo, tile, c, p);
}

}  // namespace fcas
