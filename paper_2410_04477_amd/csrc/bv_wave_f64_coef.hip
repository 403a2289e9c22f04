// One-wave matrix-core kernels, FP64 instantiations: conditional-mean weights and
// variances of single points, for the simulator (the kernel is in wave_kernel.hpp).
#include "wave_kernel.hpp"

namespace bv {

hipError_t launch_wave_f64_coef(int g, const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  return launch_wave_t<double, 7>(g, a, thp, grid, s);
}

}  // namespace bv
