// One-wave matrix-core kernels, FP64 instantiations: prediction
// (the kernel is in wave_kernel.hpp).
#include "wave_kernel.hpp"

namespace bv {

hipError_t launch_wave_f64_pred(int g, const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  return launch_wave_t<double, 4>(g, a, thp, grid, s);
}

}  // namespace bv
