// eval_kernels.hpp -- gfx950 kernels of fitness_eval_batch (included by the
// per-precision translation units).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "fitness_tiles.hpp"
#include "plans.hpp"
#include "rules.hpp"

// Build-time overrides of the occupancy each pass kernel is compiled for
// (waves per SIMD; -1: the per-plan choice of PassTune below).
#ifndef FCAS_PASS1_WAVES
#define FCAS_PASS1_WAVES (-1)
#endif
#ifndef FCAS_PASS2_WAVES
#define FCAS_PASS2_WAVES (-1)
#endif

namespace fcas {

// Settings of the pass kernels of one plan.
//   joint: both series of a transform exchange through LDS in one step (two
//   buffers, half the synchronisations), else one after the other through one
//   buffer, the first stored before the second's stages begin, which takes
//   half the LDS and, in pass 1, leaves the second series in its half-full
//   input registers meanwhile.
//   waves: occupancy the kernel is compiled for (waves per SIMD).
// Float transforms of 8-element threads fit in 128 VGPRs: 4 waves; pass 1 of
// 12 or 16 elements with its data kept takes 190-210 (320 points of 196608 in
// 192-point columns: 199 us at 2 waves, 212 at 3 with spills).  Double: 3 waves
// for 8 elements, 2 for more (12 elements spill 97 VGPRs at 3: 40 points of
// 98304 95 us a call, 71 at 2).
//   keep: pass 1 holds a tile's segment data in registers from point to point
//   (where they leave room for the transform), else it reads them again.
template <typename Real, class PL, int DT = 1>
struct PassTune {
  static constexpr bool f32 = sizeof(Real) == 4;
  static constexpr bool joint1 = f32 && PL::E1 <= 12, joint2 = f32 && PL::E2 <= 12;
  static constexpr int data1 = (DT * 2 * (int)sizeof(Real) / 4 + 2) * (PL::E1 / 2);   // registers of the segment data
  static constexpr bool keep = data1 <= (f32 && PL::E1 > 8 ? 80 : 40);
  static constexpr int waves1 = FCAS_PASS1_WAVES >= 0 ? FCAS_PASS1_WAVES : !f32 ? (PL::E1 == 8 ? 3 : 2) : PL::E1 == 8 ? 4 : 2;
  static constexpr int waves2 = FCAS_PASS2_WAVES >= 0 ? FCAS_PASS2_WAVES : (f32 && PL::E2 == 8 ? 4 : 3);
};

struct PassArgs {
  const SegDesc* segs;
  const EvalDesc* evals;
  const int32_t* list;     // evaluation indices of this plan, in list order (null: a direct call, see DirectArgs)
  const int32_t* count;    // number of entries in `list`
  void* ws;                // workspace: cap slots of 2 N complex
  void* part_g;            // [max_batch][part_stride] partial maxima (Real)
  int32_t* part_j;         // [max_batch][part_stride] their samples
  int32_t part_stride;     // partials per evaluation slot (>= the plan's PARTS2)
  int32_t nt;              // pass-1 stores (StorePolicy)
  int32_t n_det;
  int32_t chunk_begin;     // first list position handled by this launch
  int32_t cap;             // workspace slots (positions per launch)
};

// What a direct call adds to pass 1 (k_pass1_direct): the points themselves.
// Such a call has one plan, one launch and no work lists; pass 2 takes point e
// at position e and passes over those not evaluated.
struct DirectArgs {
  const NetDesc* net;
  const double* theta;
  const int32_t* seg_ids;
  EvalDesc* evals;
  int32_t* err;
  unsigned long long* evaluated;
  int32_t plan;            // the launch's plan: a segment of another one is refused
};

// Number of list positions one launch handles: the chunk [chunk_begin,
// chunk_begin + cap) of the plan's list, cut to the count the set-up kernel
// wrote.
__device__ __forceinline__ int launch_span(const PassArgs& a) {
  if (!a.list) return a.cap;   // a direct call: every point, in order
  const int cnt = *a.count - a.chunk_begin;
  return cnt < 0 ? 0 : (cnt > a.cap ? a.cap : cnt);
}

// ---------------------------------------------------------------------------
// Pass 1: prologue (template phase, delays, projection) + length-N1 column
// FFTs + four-step twiddle, for C columns of one evaluation per work item.
// ---------------------------------------------------------------------------
// Orders the LDS writes of a stage before the reads of the next.  When every
// transform is held by threads of one wavefront (WAVE), the lanes of that wave
// are the only writers and readers of its buffer: waiting for the wave's own
// LDS operations and keeping the compiler from moving accesses across is
// enough.  Otherwise the whole work-group synchronises.
template <bool WAVE>
__device__ __forceinline__ void lds_exchange_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// All stages of the middle pass for the S series (1 or 2) of one transform held
// in registers, which take turns in the LDS buffer.
template <typename Real, int L, int E, class Rad, int I, int Ns, int PAD, int S>
__device__ __forceinline__ void run_stages(cplx<Real> (&v)[S][E], cplx<Real>* buf, const cplx<Real>* tw, int t) {
  if constexpr (I < Rad::count) {
    constexpr int R = Rad::value[I];
    constexpr bool LAST = (I == Rad::count - 1);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      stage_butterflies<Real, L, E, R, Ns, LAST, PAD>(v[s], buf, tw, t);
      if constexpr (!LAST) {
        __syncthreads();
        stage_gather<Real, L, E, PAD>(v[s], buf, t);
        __syncthreads();
      }
    }
    run_stages<Real, L, E, Rad, I + 1, Ns * R, PAD, S>(v, buf, tw, t);
  }
}

// The stages of passes 1 and 2, with their factors in registers: of one
// series, or of both exchanging together.
template <typename Real, int L, int E, class Rad, int I, bool SHIFT, bool HALF, bool WAVE, int PAD>
__device__ __forceinline__ void run_geo_series(cplx<Real> (&v)[E], cplx<Real>* buf,
                                               const GeoSet<Real, L, E, Rad, SHIFT>& g, int t) {
  if constexpr (I < Rad::count) {
    geo_stage<Real, L, E, Rad, I, SHIFT, HALF && I == 0, PAD>(v, buf, g, t);
    if constexpr (I < Rad::count - 1) {
      lds_exchange_sync<WAVE>();
      stage_gather<Real, L, E, PAD>(v, buf, t);
      lds_exchange_sync<WAVE>();
    }
    run_geo_series<Real, L, E, Rad, I + 1, SHIFT, HALF, WAVE, PAD>(v, buf, g, t);
  }
}

template <typename Real, int L, int E, class Rad, int I, bool SHIFT, bool HALF, bool WAVE, int PAD>
__device__ __forceinline__ void run_geo_joint(cplx<Real> (&v)[2][E], cplx<Real>* buf0, cplx<Real>* buf1,
                                              const GeoSet<Real, L, E, Rad, SHIFT>& g, int t) {
  if constexpr (I < Rad::count) {
    geo_stage<Real, L, E, Rad, I, SHIFT, HALF && I == 0, PAD>(v[0], buf0, g, t);
    geo_stage<Real, L, E, Rad, I, SHIFT, HALF && I == 0, PAD>(v[1], buf1, g, t);
    if constexpr (I < Rad::count - 1) {
      lds_exchange_sync<WAVE>();
      stage_gather<Real, L, E, PAD>(v[0], buf0, t);
      stage_gather<Real, L, E, PAD>(v[1], buf1, t);
      lds_exchange_sync<WAVE>();
    }
    run_geo_joint<Real, L, E, Rad, I + 1, SHIFT, HALF, WAVE, PAD>(v, buf0, buf1, g, t);
  }
}

// Pass 1 of one item from its prologue's values to the workspace slot `out`.
template <typename Real, class PL>
using Pass1Geo = GeoSet<Real, PL::N1, PL::E1, typename PL::Rad1, false>;
template <typename Real, class PL, bool NT>
__device__ __forceinline__ void pass1_transform(cplx<Real> (&v)[2][PL::E1], cplx<Real>* out, cplx<Real>* buf0,
                                                cplx<Real>* buf1, const Pass1Geo<Real, PL>& g, int tile, int c,
                                                int p) {
  using Rad = typename PL::Rad1;
  if constexpr (PassTune<Real, PL>::joint1) {
    run_geo_joint<Real, PL::N1, PL::E1, Rad, 0, false, true, false, kPad1>(v, buf0, buf1, g, p);
    pass1_store<Real, PL, NT>(v, out, tile, c, p);
  } else {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      run_geo_series<Real, PL::N1, PL::E1, Rad, 0, false, true, false, kPad1>(v[s], buf0, g, p);
      pass1_store_series<Real, PL, NT>(v[s], out, s, tile, c, p);
    }
  }
}

// Pass 2 of one item from its rows: Gamma^2 of the thread's samples.
template <class PL>
constexpr bool kRowInWave = (64 % PL::P2) == 0;
template <typename Real, class PL>
using Pass2Geo = GeoSet<Real, PL::N2, PL::E2, typename PL::Rad2, !PL::THREE>;
template <typename Real, class PL, bool WAVE>
__device__ __forceinline__ void pass2_transform(cplx<Real> (&v)[2][PL::E2], Real (&g)[PL::E2], cplx<Real>* buf0,
                                                cplx<Real>* buf1, const Pass2Geo<Real, PL>& geo, int p) {
  using Rad = typename PL::Rad2;
  if constexpr (PassTune<Real, PL>::joint2) {
    run_geo_joint<Real, PL::N2, PL::E2, Rad, 0, !PL::THREE, false, WAVE, kPad2>(v, buf0, buf1, geo, p);
#pragma unroll
    for (int q = 0; q < PL::E2; ++q) g[q] = norm2(v[0][q]) + norm2(v[1][q]);
  } else {
    run_geo_series<Real, PL::N2, PL::E2, Rad, 0, !PL::THREE, false, WAVE, kPad2>(v[0], buf0, geo, p);
#pragma unroll
    for (int q = 0; q < PL::E2; ++q) g[q] = norm2(v[0][q]);
    run_geo_series<Real, PL::N2, PL::E2, Rad, 0, !PL::THREE, false, WAVE, kPad2>(v[1], buf0, geo, p);
#pragma unroll
    for (int q = 0; q < PL::E2; ++q) g[q] = g[q] + norm2(v[1][q]);
  }
}

// Work of passes 1 and 2: work-group b of a grid of TILES * G takes one tile
// of every G-th point of the launch, so what belongs to the tile (its segment
// data, twiddle factors, addresses) stays in registers from point to point,
// while the work-groups of a group, which start together, are on the tiles of
// one point at a time: their stores and loads cover whole rows of the
// workspace between them (with the points of a tile in one work-group after
// the other instead, pass 1 of 131072 lost what the fewer instructions gave,
// and 262144, with 64-byte row pieces, 15%).
template <int TILES>
__device__ __forceinline__ void tile_of_block(int block, int nblocks, int& tile, int& first, int& step) {
  tile = block % TILES;
  first = block / TILES;
  step = nblocks / TILES;
}

// Point (evaluation index) at list position `pos` of the launch, and its
// segment's descriptor: uniform across the work-group, read as scalar loads.
__device__ __forceinline__ int list_entry(const PassArgs& a, int pos) {
  return a.list ? *const_view(a.list + pos) : pos;
}

__device__ __forceinline__ SegDesc segment_of(const PassArgs& a, int e) {
  const int seg = const_view(a.evals + e)->seg;
  return *const_view(a.segs + seg);
}

// LDS exchange buffers of the two passes: padded length of one transform and
// elements per work-group.
template <typename Real, class PL>
struct PassLds {
  static constexpr int LP1 = lds_padded_len<kPad1>(PL::N1), LP2 = lds_padded_len<kPad2>(PL::N2);
  static constexpr int X1 = (PassTune<Real, PL>::joint1 ? 2 : 1) * PL::C * LP1;
  static constexpr int X2 = (PassTune<Real, PL>::joint2 ? 2 : 1) * PL::RW * LP2;
};

// Whether a launch of `span` points stores non-temporally.  Points of one
// segment usually stand together, so its first and last point tell whether it
// holds several (either policy gives the same results).
__device__ __forceinline__ bool streams_rows(const PassArgs& a, int span) {
  if (a.nt != kStoreBySegments) return a.nt == kStoreStreamed;
  return const_view(a.evals + list_entry(a, a.chunk_begin))->seg !=
         const_view(a.evals + list_entry(a, a.chunk_begin + span - 1))->seg;
}

// Pass 1 on the share of work-group `block` of `nblocks`.  The segment data of
// the tile are read when the segment changes and stay in registers for the
// points that follow.
template <typename Real, class PL, int DT>
__device__ __forceinline__ void pass1_body(const PassArgs& a, cplx<Real>* lds, int block, int nblocks) {
  constexpr int LP = PassLds<Real, PL>::LP1;
  const int tid = threadIdx.x;
  const int span = launch_span(a);
  int tile, slot, step;
  tile_of_block<PL::TILES1>(block, nblocks, tile, slot, step);
  if (slot >= span) return;
  const int c = tid % PL::C, p = tid / PL::C;
  cplx<Real>* buf0 = lds + c * LP;
  cplx<Real>* buf1 = PassTune<Real, PL>::joint1 ? lds + (PL::C + c) * LP : buf0;
  int cur_seg = -1;
  Pass1Data<Real, PL, DT> d;
  Pass1Geo<Real, PL> g;
  g.init(p);
  const bool nt = streams_rows(a, span);
  for (; slot < span; slot += step) {
    const int e = list_entry(a, a.chunk_begin + slot);
    const int seg = const_view(a.evals + e)->seg;
    if (!PassTune<Real, PL, DT>::keep || seg != cur_seg) {
      const SegDesc sg = *const_view(a.segs + seg);
      pass1_fetch<Real, PL, DT>(d, sg, tile, c, p);
      cur_seg = seg;
    }
    cplx<Real> v[2][PL::E1];
    pass1_compute<Real, PL, DT>(v, d, pass1_point<Real, DT>(const_view(a.evals + e)));
    cplx<Real>* out = (cplx<Real>*)a.ws + (int64_t)slot * 2 * PL::N;
    if (nt)
      pass1_transform<Real, PL, true>(v, out, buf0, buf1, g, tile, c, p);
    else
      pass1_transform<Real, PL, false>(v, out, buf0, buf1, g, tile, c, p);
  }
}

template <typename Real, int L, int T>
__device__ __forceinline__ void init_twiddles(cplx<Real>* tw) {
  for (int m = threadIdx.x; m < L; m += T) tw[m] = twiddle<Real>(m, L);
  __syncthreads();
}

template <typename Real, class PL, int DT>
__global__ void __launch_bounds__(PL::T1)
    __attribute__((amdgpu_waves_per_eu(PassTune<Real, PL, DT>::waves1))) k_pass1(PassArgs a) {
  __shared__ cplx<Real> lds[PassLds<Real, PL>::X1];
  pass1_body<Real, PL, DT>(a, lds, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------
// Middle pass of the three-pass plans: length-NM transforms over the pass-1
// output, in place (see Plan).  Each work item takes CM adjacent columns of
// one pass-1 row, so every load and store instruction moves CM * 8 bytes of
// contiguous row per transform element (128 bytes at CM = 16).
// ---------------------------------------------------------------------------
// Series per work item and software prefetch of the middle pass.  Measured on
// the hour-long plans: the series taking turns in LDS (half the LDS) runs 1.75x
// faster than both at once; a second register set for prefetching then gains
// nothing, and neither does one series per work item (117 instead of 240 VGPRs,
// twice the waves per SIMD, 4% slower): the pass moves its 32 N bytes per point
// at the rate of a device copy.
constexpr int kPassmSeries = 2;         // series per work item (1: each series its own item)
constexpr bool kPassmPrefetch = false;

// Work item -> (list position in the launch, first series, tile); the items
// of one point run series by series, tiles in order.
template <class PL>
__device__ __forceinline__ void passm_decode(int item, int& slot, int& s0, int& tile) {
  constexpr int PER_SERIES = PL::TILESM, PER_SLOT = (2 / kPassmSeries) * PL::TILESM;
  slot = item / PER_SLOT;
  const int r = item - slot * PER_SLOT;
  const int g = r / PER_SERIES;
  s0 = g * kPassmSeries;
  tile = r - g * PER_SERIES;
}

template <typename Real, class PL>
__device__ __forceinline__ void passm_fetch_item(cplx<Real> (&v)[kPassmSeries][PL::EM], const PassArgs& a,
                                                 int item, int c, int p) {
  int slot, s0, tile;
  passm_decode<PL>(item, slot, s0, tile);
  passm_fetch<Real, PL>(v, (const cplx<Real>*)a.ws + (int64_t)slot * 2 * PL::N, tile, c, p, s0);
}

template <typename Real, class PL>
__device__ __forceinline__ void passm_item(cplx<Real> (&v)[kPassmSeries][PL::EM], const PassArgs& a, int item,
                                           cplx<Real>* buf, const cplx<Real>* tw, int c, int p) {
  int slot, s0, tile;
  passm_decode<PL>(item, slot, s0, tile);
  passm_twiddle_in<Real, PL>(v, tile, c, p);
  run_stages<Real, PL::NM, PL::EM, typename PL::RadM, 0, 1, kPadM>(v, buf, tw, p);
  passm_twiddle_out<Real, PL>(v, tile, c, p);
  passm_store<Real, PL>(v, (cplx<Real>*)a.ws + (int64_t)slot * 2 * PL::N, tile, c, p, s0);
}

// Middle pass on the items of `a` taken by work-group `block` of `nblocks`;
// with kPassmPrefetch the next item's loads are in flight while one is
// transformed (two register sets).  Items cover disjoint workspace elements,
// so a prefetch never reads what another item stores.
template <typename Real, class PL>
__device__ __forceinline__ void passm_body(const PassArgs& a, cplx<Real>* lds, const cplx<Real>* tw, int block,
                                           int nblocks) {
  constexpr int LP = lds_padded_len<kPadM>(PL::NM);
  const int tid = threadIdx.x;
  const int items = launch_span(a) * (2 / kPassmSeries) * PL::TILESM;
  const int c = tid % PL::CM, p = tid / PL::CM;
  cplx<Real>* buf = lds + c * LP;
  if constexpr (kPassmPrefetch) {
    cplx<Real> va[kPassmSeries][PL::EM], vb[kPassmSeries][PL::EM];
    int item = block;
    if (item < items) passm_fetch_item<Real, PL>(va, a, item, c, p);
    while (item < items) {
      const int next = item + nblocks;
      if (next < items) passm_fetch_item<Real, PL>(vb, a, next, c, p);
      passm_item<Real, PL>(va, a, item, buf, tw, c, p);
      if (next >= items) break;
      item = next + nblocks;
      if (item < items) passm_fetch_item<Real, PL>(va, a, item, c, p);
      passm_item<Real, PL>(vb, a, next, buf, tw, c, p);
    }
  } else {
    for (int item = block; item < items; item += nblocks) {
      cplx<Real> v[kPassmSeries][PL::EM];
      passm_fetch_item<Real, PL>(v, a, item, c, p);
      passm_item<Real, PL>(v, a, item, buf, tw, c, p);
    }
  }
}

template <typename Real, class PL>
__global__ void __launch_bounds__(PL::TM) k_passm(PassArgs a) {
  static_assert(PL::THREE, "two-pass plans have no middle pass");
  __shared__ cplx<Real> lds[PL::CM * lds_padded_len<kPadM>(PL::NM)];
  __shared__ cplx<Real> tw[PL::NM];
  init_twiddles<Real, PL::NM, PL::TM>(tw);
  passm_body<Real, PL>(a, lds, tw, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------
// Pass 2: length-N2 row FFTs, |a_0|^2 + |a_1|^2 and its maximum over the rows
// of one work item -> one partial (value, sample) per work item.  When every
// row transform lies inside one wavefront the items need no work-group
// barrier; rows longer than a wavefront's share synchronise the work-group.
// ---------------------------------------------------------------------------
// The largest value over the 64 lanes of a wavefront (no lane holds a NaN).
__device__ __forceinline__ float wave_max(float x) {
  auto step = [](float v, auto ctrl) {
    const int b = __builtin_bit_cast(int, v);
    return __builtin_fmaxf(
        v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(b, b, decltype(ctrl)::value, 0xf, 0xf, false)));
  };
  x = step(x, std::integral_constant<int, 0x111>{});   // row_shr 1, 2, 4, 8
  x = step(x, std::integral_constant<int, 0x112>{});
  x = step(x, std::integral_constant<int, 0x114>{});
  x = step(x, std::integral_constant<int, 0x118>{});
  x = step(x, std::integral_constant<int, 0x142>{});   // row_bcast 15, 31: lane 63 holds the maximum
  x = step(x, std::integral_constant<int, 0x143>{});
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}
__device__ __forceinline__ double wave_max(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double o = __shfl_xor(x, off, 64);
    x = o > x ? o : x;
  }
  return x;
}

// The largest Gamma^2 in range of one wavefront's rows and its smallest
// sample, written to *out_g / *out_j by one lane.  Over the whole series it
// takes the maximum of the values alone first; the lane that holds it then
// looks for its sample.  A restricted range, several lanes with the same value
// or none with any take the general reduction of (value, sample) pairs.  (That
// reduction for every row cost 82 instructions of pass 2's 642; this one 37.)
template <typename Real, class PL>
__device__ __forceinline__ void pass2_rows_best(const Real (&gs)[PL::E2], int tile, int64_t j_lo, int64_t j_hi,
                                                int r, int p, int lane, Real* out_g, int* out_j) {
  if (j_lo <= 0 && j_hi >= PL::N) {
    Real m = (Real)-1;   // a NaN is never the larger of two
#pragma unroll
    for (int q = 0; q < PL::E2; ++q)
      m = sizeof(Real) == 4 ? (Real)__builtin_fmaxf((float)m, (float)gs[q]) : gs[q] > m ? gs[q] : m;
    const Real top = wave_max(m);
    const unsigned long long tie = __ballot(m == top);
    if (top >= (Real)0 && (tie & (tie - 1)) == 0) {
      if (m == top) {
        int q = PL::E2 - 1;
#pragma unroll
        for (int k = PL::E2 - 2; k >= 0; --k) q = gs[k] == m ? k : q;
        *out_g = m;
        *out_j = row_base<PL>(tile * PL::RW + r) + PL::ROWS2 * (p + q * PL::P2);
      }
      return;
    }
  }
  Real g;
  int j;
  pass2_best_of<Real, PL>(gs, tile, r, p, g, j, j_lo, j_hi);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const Real go = __shfl_xor(g, off, 64);
    const int jo = __shfl_xor(j, off, 64);
    if (better(go, jo, g, j)) {
      g = go;
      j = jo;
    }
  }
  if (lane == 0) {
    *out_g = g;
    *out_j = j;
  }
}

// One wavefront's best rows, exchanged within the work-group (two sets, used
// in turn: a set is rewritten only after the next item's barrier).
template <typename Real, class PL>
struct RowsBest {
  Real g[2][PL::T2 / 64];
  int j[2][PL::T2 / 64];
};

// The partial of a work item: the best of its wavefronts.
template <typename Real, class PL>
__device__ __forceinline__ void pass2_join(const Real (&gs)[PL::E2], const PassArgs& a, int e, int tile,
                                           int64_t j_lo, int64_t j_hi, int r, int p, RowsBest<Real, PL>& red, int turn) {
  constexpr int NW = PL::T2 / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  pass2_rows_best<Real, PL>(gs, tile, j_lo, j_hi, r, p, lane, &red.g[turn][wave], &red.j[turn][wave]);
  __syncthreads();
  if (threadIdx.x == 0) {
    Real g = red.g[turn][0];
    int j = red.j[turn][0];
#pragma unroll
    for (int w = 1; w < NW; ++w)
      if (better(red.g[turn][w], red.j[turn][w], g, j)) {
        g = red.g[turn][w];
        j = red.j[turn][w];
      }
    const int64_t o = (int64_t)e * a.part_stride + tile;
    ((Real*)a.part_g)[o] = g;
    a.part_j[o] = j;
  }
}

// Pass 2 on the share of work-group `block` of `nblocks`.
template <typename Real, class PL>
__device__ __forceinline__ void pass2_body(const PassArgs& a, cplx<Real>* lds, RowsBest<Real, PL>& red, int block,
                                           int nblocks) {
  constexpr int LP = PassLds<Real, PL>::LP2;
  const int tid = threadIdx.x;
  const int span = launch_span(a);
  int tile, slot, step;
  tile_of_block<PL::TILES2>(block, nblocks, tile, slot, step);
  if (slot >= span) return;
  const int p = tid % PL::P2, r = tid / PL::P2;
  cplx<Real>* buf0 = lds + r * LP;
  cplx<Real>* buf1 = PassTune<Real, PL>::joint2 ? lds + (PL::RW + r) * LP : buf0;
  int turn = 0;
  Pass2Geo<Real, PL> geo;
  geo.init(p, tile * PL::RW + r, PL::THREE ? 1 : PL::N1);
  for (; slot < span; slot += step) {
    const int e = list_entry(a, a.chunk_begin + slot);
    if (!a.list && const_view(a.evals + e)->status != 1) continue;
    cplx<Real> v[2][PL::E2];
    pass2_fetch<Real, PL>(v, (const cplx<Real>*)a.ws + (int64_t)slot * 2 * PL::N, tile, r, p);
    const SegDesc sg = segment_of(a, e);
    const int64_t j_lo = sg.j_lo, j_hi = sg.j_hi;
    // row transforms held by one wavefront exchange through LDS without a
    // work-group barrier
    Real g[PL::E2];
    pass2_transform<Real, PL, kRowInWave<PL>>(v, g, buf0, buf1, geo, p);
    pass2_join<Real, PL>(g, a, e, tile, j_lo, j_hi, r, p, red, turn);
    turn ^= 1;
  }
}

template <typename Real, class PL>
__global__ void __launch_bounds__(PL::T2)
    __attribute__((amdgpu_waves_per_eu(PassTune<Real, PL>::waves2))) k_pass2(PassArgs a) {
  __shared__ cplx<Real> lds[PassLds<Real, PL>::X2];
  __shared__ RowsBest<Real, PL> red;
  pass2_body<Real, PL>(a, lds, red, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------
// Finalize: Gamma^2 and j* of a point from its pass-2 partials; -inf / -1
// outside the rectangle, NaN / -2 for a bad segment.  By a group of G lanes
// (aligned, every lane of the group calling it): the largest value, then
// smallest sample, is unique, so any grouping of the reduction gives the same
// result.
// ---------------------------------------------------------------------------
// What is read of a point before its number of partials is known: its status
// and plan, and the first batch of partials, whether or not it has left that
// many.
template <typename Real, int G>
struct PointPartials {
  static constexpr int B = G >= 64 ? 2 : 8;   // loads per lane in flight before any is compared
  Real gv[B];
  int jv[B];
  int status, plan, count;   // count: partials of a point of that plan

  __device__ __forceinline__ void load(const EvalDesc& ev, const Real* __restrict__ part_g,
                                       const int32_t* __restrict__ part_j, int part_stride, int e, int g) {
    const Real* pg = part_g + (int64_t)e * part_stride;
    const int32_t* pj = part_j + (int64_t)e * part_stride;
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int t = g + G * u < part_stride ? g + G * u : 0;
      gv[u] = pg[t];
      jv[u] = pj[t];
    }
    status = ev.status;
    plan = ev.plan;
  }
  __device__ __forceinline__ void load_count(const int32_t* __restrict__ plan_parts2) { count = plan_parts2[plan]; }
};

template <typename Real, int G>
__device__ __forceinline__ void finalize_value(PointPartials<Real, G>& pp, const Real* __restrict__ part_g,
                                               const int32_t* __restrict__ part_j, int part_stride, int e, int g,
                                               double& fitness, int& argmax) {
  constexpr int B = PointPartials<Real, G>::B;
  const Real* pg = part_g + (int64_t)e * part_stride;
  const int32_t* pj = part_j + (int64_t)e * part_stride;
  Real(&gv)[B] = pp.gv;
  int(&jv)[B] = pp.jv;
  const int status = pp.status;
  Real bg = (Real)-1;
  int bj = 0x7fffffff;
  if (status == 1) {
    const int nt = pp.count;
    for (int t0 = g;;) {
#pragma unroll
      for (int u = 0; u < B; ++u)
        if (t0 + G * u < nt && better(gv[u], jv[u], bg, bj)) {
          bg = gv[u];
          bj = jv[u];
        }
      t0 += G * B;
      if (t0 - g >= nt) break;
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int t = t0 + G * u < nt ? t0 + G * u : 0;
        gv[u] = pg[t];
        jv[u] = pj[t];
      }
    }
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) {
      const Real go = __shfl_xor(bg, off, G);
      const int jo = __shfl_xor(bj, off, G);
      if (better(go, jo, bg, bj)) {
        bg = go;
        bj = jo;
      }
    }
  }
  fitness = status == 1 ? (double)bg : status == 0 ? -INFINITY : NAN;
  argmax = status == 1 ? bj : status == 0 ? -1 : -2;
}

// The same, written to the call's outputs.
template <typename Real, int G>
__device__ __forceinline__ void finalize_group(const EvalDesc& ev, const Real* __restrict__ part_g,
                                               const int32_t* __restrict__ part_j, int part_stride,
                                               const int32_t* __restrict__ plan_parts2, int e, int g,
                                               double* __restrict__ fitness, int32_t* __restrict__ argmax) {
  double f;
  int j;
  PointPartials<Real, G> pp;
  pp.load(ev, part_g, part_j, part_stride, e, g);
  pp.load_count(plan_parts2);
  finalize_value<Real, G>(pp, part_g, part_j, part_stride, e, g, f, j);
  if (g == 0) {
    fitness[e] = f;
    argmax[e] = j;
  }
}

template <typename Real>
__global__ void __launch_bounds__(256) k_finalize(const EvalDesc* __restrict__ evals, const Real* __restrict__ part_g,
                                                  const int32_t* __restrict__ part_j, int n, int part_stride,
                                                  const int32_t* __restrict__ plan_parts2,
                                                  int32_t* __restrict__ counts,
                                                  unsigned long long* __restrict__ evaluated,
                                                  double* __restrict__ fitness, int32_t* __restrict__ argmax) {
  const int e = blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
  if (blockIdx.x == 0 && threadIdx.x < kNumPlans) {
    // running total of points evaluated (inside the rectangle); the passes of
    // this call are done with the list counts, which start the next call at 0
    const int c = counts[threadIdx.x];
    counts[threadIdx.x] = 0;
    if (c) atomicAdd(evaluated, (unsigned long long)c);
  }
  if (e >= n) return;
  finalize_group<Real, 64>(evals[e], part_g, part_j, part_stride, plan_parts2, e, threadIdx.x & 63, fitness, argmax);
}

}  // namespace fcas

namespace fcas {

// ---------------------------------------------------------------------------
// Fused persistent schedule: both passes of every evaluation of one plan in
// a single launch.  Work items (TILES1 pass-1 tiles and TILES2 pass-2 tiles per
// evaluation) form a software pipeline in which pass-1 tiles of evaluation
// e + L interleave with pass-2 tiles of evaluation e:
//   [P1(0) .. P1(L-1)] [P1(L) P2(0)] [P1(L+1) P2(1)] ... [P2(cnt-L) .. P2(cnt-1)]
// Work-group w takes items w, w + G, w + 2G, ... (G <= resident work-groups),
// so ALU-bound pass-1 tiles and bandwidth-bound pass-2 tiles run side by side
// and only S = `slots` evaluations occupy the workspace (S > L), small enough
// to stay in the memory-side cache.  A pass-2 tile waits for its evaluation's
// pass-1 tiles; a pass-1 tile waits for the pass-2 tiles of the evaluation that
// last used its slot.  Both are earlier in the sequence, so the wait always
// ends; each wait is also bounded (on overflow an error flag is set and the
// item proceeds).
// ---------------------------------------------------------------------------
struct FusedArgs {
  PassArgs p;
  int32_t* done1;    // [max_batch] pass-1 tiles finished, per list position
  int32_t* done2;    // [max_batch] pass-2 tiles finished, per list position
  int32_t* err;      // error flags (bit 1: a wait exceeded its bound)
  int32_t lag;       // L
  int32_t slots;     // S
  int32_t max_spin;  // polls before a wait gives up
};

__device__ __forceinline__ void wait_count(const int32_t* ctr, int target, int max_spin, int32_t* err) {
  if (threadIdx.x == 0) {
    int spins = 0;
    while (__hip_atomic_load(ctr, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (++spins > max_spin) {
        __hip_atomic_fetch_or(err, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      __builtin_amdgcn_s_sleep(4);
    }
  }
  __syncthreads();
}

__device__ __forceinline__ void signal_count(int32_t* ctr) {
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename Real, class PL>
__global__ void __launch_bounds__(PL::T1) k_fused(FusedArgs f) {
  static_assert(PL::T1 == PL::T2, "the fused schedule needs equal work-item sizes");
  static_assert(!PL::THREE, "the fused schedule covers two-pass plans");
  constexpr int LP1 = lds_padded_len<kPad1>(PL::N1), LP2 = lds_padded_len<kPad2>(PL::N2);
  constexpr int LDSN = 2 * ((PL::C * LP1 > PL::RW * LP2) ? PL::C * LP1 : PL::RW * LP2);
  constexpr int T1 = PL::TILES1, T2 = PL::TILES2, T = T1 + T2;
  __shared__ cplx<Real> lds[LDSN];
  __shared__ RowsBest<Real, PL> red;
  const PassArgs& a = f.p;
  const int tid = threadIdx.x;
  const int cnt = *a.count;
  const int L = f.lag < cnt ? f.lag : cnt;
  const int total = cnt * T;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    int kind, ep, tile;
    fused_decode(item, cnt, L, T1, T2, kind, ep, tile);
    const int slot = ep % f.slots;
    cplx<Real>* ws = (cplx<Real>*)a.ws + (int64_t)slot * 2 * PL::N;
    const int e = a.list[ep];
    if (kind == 1) {
      if (ep >= f.slots) wait_count(f.done2 + (ep - f.slots), T2, f.max_spin, f.err);
      const EvalDesc& ev = a.evals[e];
      const SegDesc& sg = a.segs[ev.seg];
      const int c = tid % PL::C, p = tid / PL::C;
      cplx<Real> v[2][PL::E1];
      Pass1Geo<Real, PL> geo;
      geo.init(p);
      pass1_prologue<Real, PL>(v, ev, sg, a.n_det, tile, c, p);
      pass1_transform<Real, PL, false>(v, ws, lds + c * LP1, lds + (PL::C + c) * LP1, geo, tile, c, p);
      signal_count(f.done1 + ep);
    } else {
      wait_count(f.done1 + ep, T1, f.max_spin, f.err);
      const int p = tid % PL::P2, r = tid / PL::P2;
      cplx<Real> v[2][PL::E2];
      pass2_fetch<Real, PL>(v, ws, tile, r, p);
      Pass2Geo<Real, PL> geo;
      geo.init(p, tile * PL::RW + r, PL::N1);
      Real g[PL::E2];
      pass2_transform<Real, PL, false>(v, g, lds + r * LP2, lds + (PL::RW + r) * LP2, geo, p);
      const SegDesc sg = segment_of(a, e);
      pass2_join<Real, PL>(g, a, e, tile, sg.j_lo, sg.j_hi, r, p, red, 0);
      signal_count(f.done2 + ep);
    }
  }
}

}  // namespace fcas
