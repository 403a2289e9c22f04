// One-wave matrix-core kernels, FP64 value of G = 7 to 10 (the kernel is in
// wave_rows.hpp).
#include "wave_rows.hpp"

namespace bv {

hipError_t launch_rows_value(int g, const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  switch (g) {
    case 7: return launch_rows_g<7, false>(a, thp, grid, s);
    case 8: return launch_rows_g<8, false>(a, thp, grid, s);
    case 9: return launch_rows_g<9, false>(a, thp, grid, s);
    case 10: return launch_rows_g<10, false>(a, thp, grid, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bv
