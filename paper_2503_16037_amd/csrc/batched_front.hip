// The sweeps of many wavelengths that mark or visit the front (see batched_sweep.hpp).
#include "batched_sweep.hpp"

namespace sg {

void launch_spmm_front(Scene &s, hipStream_t st, int grid, const float *rhs, const float *x, float *y, int monitor,
                       int front) {
    if (front > kFrontFirst) launch_wide<float, float, float, false, kFrontOn>(s, st, grid, rhs, x, y, monitor, front);
    else launch_wide<float, float, float, false, kFrontFirst>(s, st, grid, rhs, x, y, monitor, front);
}

}  // namespace sg
