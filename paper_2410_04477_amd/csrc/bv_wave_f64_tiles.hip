// One-wave matrix-core kernels, FP64 instantiations: gradient in one launch through the tile buffer
// (the kernel is in wave_kernel.hpp).
#include "wave_kernel.hpp"

namespace bv {

hipError_t launch_wave_f64_tiles(int g, const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  return launch_wave_t<double, 1>(g, a, thp, grid, s);
}

}  // namespace bv
