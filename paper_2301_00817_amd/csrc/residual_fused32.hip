// The RK stage kernel in the FP32-storage form (FP32 stage states, metrics
// and fluxes; FP64 Q^(0) and stage accumulation).  The kernel template is in
// fused_stage.hpp; this translation unit keeps the default instruction
// scheduling, under which the FP32 kernel fits four waves per SIMD without
// spilling.
#include "fused_stage.hpp"

namespace lesjet {

template <>
FusedPlan fused_plan<float>(const Grid& g, int num_cu) {
  double cost;
  return tile_plan<float, false>(g, num_cu, &cost);
}

template <>
hipError_t launch_fused<float>(const float* Q, const float* M, const Grid& g, const Phys<float>& ph,
                        FusedPlan plan, int epi, float* out, const double* Q0, double* Q64, double alpha, const double* dt,
                        const Phys<double>& ph64, unsigned long long* maxbits, int lag, float* visc,
                        const double* dyn, const ProdTab& pt, hipStream_t s) {
  return launch_fused_tile<float, false>(
      Q, M, g, ph, plan.kc, epi, out, Q0, Q64, alpha, dt, ph64, maxbits, lag, visc, dyn, pt, s);
}

}  // namespace lesjet
