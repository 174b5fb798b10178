// The RK stage kernel in FP64 (plain form), narrow tile, and the choice of the
// tile.  The kernel template is in fused_stage.hpp; each precision and tile is
// its own translation unit, the FP64 ones scheduled for instruction-level
// parallelism by the build, the FP32 one with the default scheduling (each
// measured faster for its kernel).
#include "fused_stage.hpp"

namespace lesjet {

extern template hipError_t launch_fused_tile<double, true>(
    const double*, const double*, const Grid&, const Phys<double>&, int, int, double*, const double*, double*, double,
    const double*, const Phys<double>&, unsigned long long*, int, double*, const double*, const ProdTab&,
    hipStream_t);

// The tile that takes fewer (rounds) x (planes per block); the wide one on a
// tie, as it computes fewer halo columns.  Narrow against wide, a residual:
// 16^3 13.8 / 15.0 us, 61 x 43 x 50 24.5 / 25.9 us (narrow chosen); 32^3
// curvilinear 17.8 / 17.6 us, 64^3 curvilinear 31.9 / 31.4 us, 173 x 67 x 90 60.7 /
// 56.8 us, 29 x 200 x 200 89 / 69 us, 128^3 curvilinear 141 / 133 us, 320 x 200 x
// 160 459 / 416 us, 200^3 curvilinear 495 / 440 us (wide chosen).
template <>
FusedPlan fused_plan<double>(const Grid& g, int num_cu) {
  double cn, cw;
  const FusedPlan n = tile_plan<double, false>(g, num_cu, &cn);
  const FusedPlan w = tile_plan<double, true>(g, num_cu, &cw);
  return cw <= cn ? w : n;
}

template <>
hipError_t launch_fused<double>(const double* Q, const double* M, const Grid& g,
                                const Phys<double>& ph, FusedPlan plan, int epi, double* out, const double* Q0,
                                double* Q64, double alpha, const double* dt,
                                const Phys<double>& ph64, unsigned long long* maxbits, int lag,
                                double* visc, const double* dyn, const ProdTab& pt, hipStream_t s) {
  return plan.wide
             ? launch_fused_tile<double, true>(
                   Q, M, g, ph, plan.kc, epi, out, Q0, Q64, alpha, dt, ph64, maxbits, lag, visc, dyn, pt, s)
             : launch_fused_tile<double, false>(
                   Q, M, g, ph, plan.kc, epi, out, Q0, Q64, alpha, dt, ph64, maxbits, lag, visc, dyn, pt, s);
}

}  // namespace lesjet
