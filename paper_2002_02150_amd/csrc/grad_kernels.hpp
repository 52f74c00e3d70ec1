// grad_kernels.hpp -- fixed-sample adjoint of the coherent fitness.
#pragma once

#include <hip/hip_runtime.h>

#include "eval_kernels.hpp"

namespace fcas {

// Per point and detector, six complex sums over the in-band bins at j*:
// [0] z^i, [1..4] sum a_k b_k^{5,3,2,1}, [5] sum a_k k.
constexpr int kAdjSums = 6;
constexpr int kAdjThreads = 256;      // threads of an adjoint block

constexpr int kMaxTrials = 32;        // trials of a polish step

struct GradBuffers {
  double* sums = nullptr;   // [n][n_det][parts][kAdjSums][2]
  int max_batch = 0;
  int n_det = 0;
};

// `bins` below: in-band bins of the longest segment in use (adjoint_parts).
int alloc_grad_buffers(GradBuffers& g, int max_batch, int n_det);
void free_grad_buffers(GradBuffers& g);
hipError_t launch_gradient(int precision, const GradBuffers& g, const NetDesc* net, const SegDesc* segs,
                           const EvalDesc* evals, const double* theta, const int32_t* argmax, int n, int n_det,
                           double* grad, int64_t bins, hipStream_t s);

// The adjoint sums alone, and the two kernels of a polish step (grad.hip).
hipError_t launch_adjoint(int precision, const GradBuffers& g, const SegDesc* segs, const EvalDesc* evals,
                          const int32_t* argmax, int n, int n_det, int64_t bins, hipStream_t s);
hipError_t launch_polish_trials(const GradBuffers& g, const NetDesc* net, const SegDesc* segs, const EvalDesc* evals,
                                const double* theta, const int32_t* seg, int n, int n_det, int trials,
                                double step_frac, double* cand, EvalDesc* trial_evals, int32_t* lists,
                                int32_t* counts, int list_stride, int64_t bins, int32_t* err, hipStream_t s);
hipError_t launch_polish_select(int precision, const NetDesc* net, const SegDesc* segs, EvalDesc* evals,
                                double* theta, const int32_t* seg, double* fitness, int32_t* argmax,
                                const double* cand, const EvalDesc* trial_evals, const void* part_g,
                                const int32_t* part_j, int part_stride, const int32_t* plan_parts2, int n, int trials,
                                int32_t* counts, unsigned long long* evaluated, int more, int32_t* err,
                                hipStream_t s);

}  // namespace fcas
