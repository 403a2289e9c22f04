// One-wave matrix-core kernels, FP64 instantiations: conditional-mean weights and
// variances of single points, for the simulator (the kernel is in wave_rows.hpp).
#include "wave_rows.hpp"

namespace bv {

hipError_t launch_wave_f64_coef(int g, const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  switch (g) {
    case 1: return launch_rows_g<1, true>(a, thp, grid, s);
    case 2: return launch_rows_g<2, true>(a, thp, grid, s);
    case 3: return launch_rows_g<3, true>(a, thp, grid, s);
    case 4: return launch_rows_g<4, true>(a, thp, grid, s);
    case 5: return launch_rows_g<5, true>(a, thp, grid, s);
    case 6: return launch_rows_g<6, true>(a, thp, grid, s);
    case 7: return launch_rows_g<7, true>(a, thp, grid, s);
    case 8: return launch_rows_g<8, true>(a, thp, grid, s);
    case 9: return launch_rows_g<9, true>(a, thp, grid, s);
    case 10: return launch_rows_g<10, true>(a, thp, grid, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bv
