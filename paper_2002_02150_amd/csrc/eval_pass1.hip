// eval_pass1.hip -- pass 1 of every plan for one precision and detector count
// (compiled once per pair: FCAS_REAL = float or double, FCAS_DT = 1..8).
#include "direct_kernels.hpp"
#include "launch.hpp"

namespace fcas {

template <typename Real>
struct PlansOf;
#define FCAS_PLAN_F(id, ...) using P##id = PlanF##id;
#define FCAS_PLAN_D(id, ...) using P##id = PlanD##id;
template <>
struct PlansOf<float> {
  FCAS_PLAN_LIST(FCAS_PLAN_F)
};
template <>
struct PlansOf<double> {
  FCAS_PLAN_LIST(FCAS_PLAN_D)
};

#define FCAS_CASE_P1(id, ...)                                                                        \
  case id: {                                                                                         \
    using PL = PlansOf<FCAS_REAL>::P##id;                                                            \
    launch_k(k_pass1<FCAS_REAL, PL, FCAS_DT>, dim3(grid), dim3(PL::T1), s, e0, e1, a);               \
    break;                                                                                           \
  }

template <>
hipError_t launch_pass1_dt<FCAS_REAL, FCAS_DT>(int plan, const PassArgs& a, int grid, hipStream_t s, hipEvent_t e0,
                                               hipEvent_t e1) {
  switch (plan) {
    FCAS_PLAN_LIST(FCAS_CASE_P1)
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

#define FCAS_CASE_DIRECT(id, ...)                                                                              \
  case id: {                                                                                                   \
    using PL = PlansOf<FCAS_REAL>::P##id;                                                                      \
    launch_k(k_pass1_direct<FCAS_REAL, PL, FCAS_DT>, dim3(n * PL::TILES1), dim3(PL::T1), s, e0, e1, a, d);     \
    break;                                                                                                     \
  }

template <>
hipError_t launch_direct_dt<FCAS_REAL, FCAS_DT>(int plan, const PassArgs& a, const DirectArgs& d, int n, hipStream_t s,
                                                hipEvent_t e0, hipEvent_t e1) {
  switch (plan) {
    FCAS_PLAN_LIST(FCAS_CASE_DIRECT)
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace fcas
