// The FP64 residual of all wavelengths: the sweep kernels in residual mode (batched_sweep.hpp).
#include "batched_sweep.hpp"

namespace sg {

void launch_bresidual64(Scene &s, hipStream_t st, int grid, const double *x64, float *r32) {
    launch_wide<double, float, double, true, 0>(s, st, grid, nullptr, x64, r32, 1, 0);
}

void launch_bresidual32(Scene &s, hipStream_t st, int grid, const float *x, float *r32) {
    launch_wide<float, float, double, true, 0>(s, st, grid, nullptr, x, r32, 1, 0);
}

}  // namespace sg
