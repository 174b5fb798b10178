// The RK stage kernel in the FP32-storage form, wide tile.
#include "fused_stage.hpp"

namespace lesjet {

template hipError_t launch_fused_tile<float, true>(
    const float*, const float*, const Grid&, const Phys<float>&, int, int, float*, const double*, double*, double,
    const double*, const Phys<double>&, unsigned long long*, int, float*, const double*, const ProdTab&,
    hipStream_t);

}  // namespace lesjet
