// One-wave matrix-core kernels, FP64 instantiations of the value and of the
// two-launch gradient (the kernel is in wave_kernel.hpp; the one-launch gradient
// and the prediction are in sources of their own, so that they compile side by side).
#include "wave_kernel.hpp"

namespace bv {

hipError_t launch_wave_f64(int g, int mode, const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  // Value: from G = 7 on a wave has its SIMD to itself and the kernel that keeps the
  // row solves off the LDS is the faster one (n = 1e6, m = 120, G = 9: 3.74 ms with the
  // general kernel, 3.43 with it); G = 11 exceeds the registers of both and stays.
  if (mode == 0)
    return g >= 7 && g <= 10 ? launch_rows_value(g, a, thp, grid, s) : launch_wave_t<double, 0>(g, a, thp, grid, s);
  if (mode == 1) return launch_wave_f64_tiles(g, a, thp, grid, s);
  if (mode == 5) return launch_wave_f64_grad(g, a, thp, grid, s);
  if (mode == 4) return launch_wave_f64_pred(g, a, thp, grid, s);
  if (mode == 6) return launch_wave_t<double, 6>(g, a, thp, grid, s);
  if (mode == 3) return launch_wave_t<double, 3>(g, a, thp, grid, s);
  return hipErrorInvalidValue;
}

bool wave_fits(int g, bool fp32) { return g >= 1 && g <= (fp32 ? kWaveMaxG32 : kWaveMaxG64); }

hipError_t launch_wave(int g, bool fp32, int mode, const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  if (!wave_fits(g, fp32)) return hipErrorInvalidValue;
  if (a.gen) return fp32 ? launch_wave_gen_f32(g, mode, a, thp, grid, s) : launch_wave_gen_f64(g, mode, a, thp, grid, s);
  return fp32 ? launch_wave_f32(g, mode, a, thp, grid, s) : launch_wave_f64(g, mode, a, thp, grid, s);
}

}  // namespace bv
