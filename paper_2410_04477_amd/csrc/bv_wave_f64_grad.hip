// One-wave matrix-core kernels, FP64 instantiations: gradient in one launch, factor in the registers
// (the kernel is in wave_kernel.hpp).
#include "wave_kernel.hpp"

namespace bv {

hipError_t launch_wave_f64_grad(int g, const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  return launch_wave_t<double, 5>(g, a, thp, grid, s);
}

}  // namespace bv
