// pso_kernels.hpp -- lbest particle swarm (Sec. III) on the device.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fcas {

struct PsoDev {
  int32_t n_runs, n_particles, n_iter;
  double w0, w1, c1, c2, vmax;
  uint64_t seed;
  double lo[4], span[4];     // theta = lo + x * span
  double* x;
  double* v;
  double* pbest_x;
  double* pbest_f;
  int32_t* pbest_j;
  double* best_x;
  double* best_f;
  int32_t* best_j;
  int32_t* iteration;
};

__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += W0;
      k1 += W1;
    }
    const uint32_t lo0 = M0 * c[0], hi0 = __umulhi(M0, c[0]);
    const uint32_t lo1 = M1 * c[2], hi1 = __umulhi(M1, c[2]);
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
  }
}

// A random word as a number in (0, 1): (c + 1/2) 2^-32.
__device__ __forceinline__ double uniform(uint32_t c) { return ((double)c + 0.5) * 2.3283064365386962890625e-10; }

__device__ __forceinline__ void random4(uint64_t seed, uint32_t it, uint32_t particle, uint32_t run, uint32_t stream,
                                        uint32_t c[4]) {
  c[0] = it;
  c[1] = particle;
  c[2] = run;
  c[3] = stream;
  philox4x32_10(c, (uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32));
}
__device__ __forceinline__ void uniforms4(uint64_t seed, uint32_t it, uint32_t particle, uint32_t run,
                                          uint32_t stream, double u[4]) {
  uint32_t c[4];
  random4(seed, it, particle, run, stream, c);
#pragma unroll
  for (int d = 0; d < 4; ++d) u[d] = uniform(c[d]);
}

__device__ __forceinline__ double clampv(double v, double vmax) {
  v = v < -vmax ? -vmax : v;
  return v > vmax ? vmax : v;
}

// The pieces of an iteration (Sec. III).  Streams 2 and 3 of the generator are
// the random numbers of the cognitive and the social term.
__device__ __forceinline__ double pso_inertia(const PsoDev& p, int iter) {
#pragma clang fp contract(off)
  return p.n_iter <= 1 ? p.w0 : p.w0 - (p.w0 - p.w1) * ((double)iter / (double)(p.n_iter - 1));
}

// One coordinate's move: velocity vn and position xn from the random numbers
// r1 and r2, the personal best pbx and the local best lbx.
__device__ __forceinline__ void pso_move(const PsoDev& p, double w, double r1, double r2, double x, double v,
                                         double pbx, double lbx, double& vn, double& xn) {
#pragma clang fp contract(off)
  const double t0 = w * v;
  const double t1 = (p.c1 * r1) * (pbx - x);
  const double t2 = (p.c2 * r2) * (lbx - x);
  vn = clampv((t0 + t1) + t2, p.vmax);
  xn = x + vn;
}
__device__ __forceinline__ double pso_theta(double lo, double span, double xn) {
#pragma clang fp contract(off)
  return lo + xn * span;
}

// Particle i's local best among itself and its two neighbours on the ring,
// pf: the personal bests of the run's P particles.
__device__ __forceinline__ int pso_local_best(const double* pf, int i, int P) {
  const int prev = i == 0 ? P - 1 : i - 1, next = i == P - 1 ? 0 : i + 1;
  int lb = prev;
  if (pf[i] > pf[lb]) lb = i;
  if (pf[next] > pf[lb]) lb = next;
  return lb;
}

// LDS of one run's update: personal-best fitness pf[P], positions px[P][4]
// and samples pj[P] after this iteration's personal-best update.
struct PsoShared {
  double* pf;
  double* px;
  int32_t* pj;
};

// The run's best so far, by one wavefront: the first particle with the largest
// personal best (lane l scans particles l, l + 64, ...; then a butterfly keeps
// the larger value, the smaller index among equal ones).
__device__ __forceinline__ void pso_run_best(const PsoDev& p, const PsoShared& sh, double run_best, int r, int lane) {
  double bv = -INFINITY;
  int b = 0x7fffffff;
  for (int k = lane; k < p.n_particles; k += 64)
    if (b == 0x7fffffff || sh.pf[k] > bv) {
      bv = sh.pf[k];
      b = k;
    }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double ov = __shfl_xor(bv, off, 64);
    const int ob = __shfl_xor(b, off, 64);
    if (ob != 0x7fffffff && (b == 0x7fffffff || ov > bv || (ov == bv && ob < b))) {
      bv = ov;
      b = ob;
    }
  }
  if (lane == 0 && sh.pf[b] > run_best) {
    p.best_f[r] = sh.pf[b];
    p.best_j[r] = sh.pj[b];
    for (int d = 0; d < 4; ++d) p.best_x[4 * r + d] = sh.px[4 * b + d];
  }
}

// The iteration count advances once every run has read it: each run's
// work-group counts itself in iteration[1] after that (a device-scope atomic,
// by one thread), and the last one stores count + 1 and clears the tally.
__device__ __forceinline__ void pso_advance(const PsoDev& p, int iter) {
  const int done = __hip_atomic_fetch_add(p.iteration + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (done != p.n_runs - 1) return;
  __hip_atomic_store(p.iteration + 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(p.iteration, iter + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS bytes of one run's update (PsoShared) for P particles.
constexpr size_t pso_shared_bytes(int P) { return (size_t)P * (sizeof(double) * 5 + sizeof(int32_t)); }

hipError_t launch_pso_init(const PsoDev& p, double* theta_out, hipStream_t s);
hipError_t launch_pso_step(const PsoDev& p, const double* fitness, const int32_t* argmax, double* theta_next,
                           hipStream_t s);
hipError_t launch_pso_best(const PsoDev& p, int runs_per_group, int runs_used, double* out_f, double* out_theta,
                           int32_t* out_j, int32_t* out_run, hipStream_t s);

}  // namespace fcas
