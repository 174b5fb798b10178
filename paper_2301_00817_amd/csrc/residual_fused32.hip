// The RK stage kernel in the FP32-storage form (FP32 stage states, metrics
// and fluxes; FP64 Q^(0) and stage accumulation), narrow tile, and the choice of
// the tile.  The kernel template is in fused_stage.hpp; the FP32 translation
// units keep the default instruction scheduling, under which residuals and stages
// 1-4 fit four waves per SIMD without spilling.
#include "fused_stage.hpp"

namespace lesjet {

extern template hipError_t launch_fused_tile<float, true>(
    const float*, const float*, const Grid&, const Phys<float>&, int, int, float*, const double*, double*, double,
    const double*, const Phys<double>&, unsigned long long*, int, float*, const double*, const ProdTab&,
    hipStream_t);

// The chunk length is the narrow tile's (states depend on it by their rounding,
// not on the tile: the two give the same bits); the wide tile, which computes 14 %
// fewer columns but keeps eight waves in step, where it saves a round of
// blocks.  Narrow against wide, a step: 222^3 curvilinear 2.51 / 2.42 ms (5 / 4
// rounds), 300 x 210 x 200 2.08 / 2.01 (7 / 6), 256 x 256 x 360 4.01 / 4.01 (10 /
// 9), 320^3 curvilinear 6.93 / 6.82 (12 / 10), 512 x 256 x 360 7.57 / 7.46 (20 /
// 18), 800 x 400 x 320 15.75 / 15.10 (36 / 31) (wide chosen); 61 x 43 x 50 0.184 /
// 0.188, 95^3 curvilinear 0.308 / 0.317 (1 / 1), 288 x 160 x 128 1.06 / 1.09 (3 /
// 3), 256^3 curvilinear 3.90 / 3.89 (7 / 7) (narrow chosen).
template <>
FusedPlan fused_plan<float>(const Grid& g, int num_cu) {
  double cost;
  FusedPlan p = tile_plan<float, false>(g, num_cu, &cost);
  const long long chunks = (g.nth + p.kc - 1) / p.kc;
  const auto rounds = [&](int x, int y, int per_cu) {
    const long long blocks = (long long)((g.nx + x - 3) / (x - 2)) * ((g.nr + y - 3) / (y - 2)) * chunks;
    return (blocks + (long long)num_cu * per_cu - 1) / ((long long)num_cu * per_cu);
  };
  using N = Tile<float, false>;
  using W = Tile<float, true>;
  p.wide = rounds(W::X, W::Y, W::PER_CU) < rounds(N::X, N::Y, N::PER_CU);
  return p;
}

template <>
hipError_t launch_fused<float>(const float* Q, const float* M, const Grid& g, const Phys<float>& ph,
                        FusedPlan plan, int epi, float* out, const double* Q0, double* Q64, double alpha, const double* dt,
                        const Phys<double>& ph64, unsigned long long* maxbits, int lag, float* visc,
                        const double* dyn, const ProdTab& pt, hipStream_t s) {
  return plan.wide
             ? launch_fused_tile<float, true>(
                   Q, M, g, ph, plan.kc, epi, out, Q0, Q64, alpha, dt, ph64, maxbits, lag, visc, dyn, pt, s)
             : launch_fused_tile<float, false>(
                   Q, M, g, ph, plan.kc, epi, out, Q0, Q64, alpha, dt, ph64, maxbits, lag, visc, dyn, pt, s);
}

}  // namespace lesjet
