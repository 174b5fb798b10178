// The RK stage kernel in FP64 (plain form), wide tile.
#include "fused_stage.hpp"

namespace lesjet {

template hipError_t launch_fused_tile<double, true>(
    const double*, const double*, const Grid&, const Phys<double>&, int, int, double*, const double*, double*, double,
    const double*, const Phys<double>&, unsigned long long*, int, double*, const double*, const ProdTab&,
    hipStream_t);

}  // namespace lesjet
