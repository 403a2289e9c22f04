// Sequential Vecchia simulator (data generator for the synthetic workloads):
// points in a given (random) order, point i drawn from N(c_i^T y_N(i), s_i)
// given its nearest earlier points N(i).  The weights c_i and variances s_i
// come from the coefficient mode of the one-wave kernels (one wave per point,
// FP64; the four-wave kernels above 10 tile rows).  The recursion runs as a data
// flow: waves take the points in order and wait for the values of a point's
// neighbours, which points taken earlier produce, so some wave can always go on.
// Each value is a fixed function of the inputs (bit-for-bit reproducible).
// Lists with a neighbour that is not earlier in the order run in passes instead: a
// point is drawn in the first pass in which all of its neighbours were drawn in
// earlier passes.
#include <string.h>

#include <algorithm>
#include <vector>

#include "internal.hpp"

namespace bv {

__global__ void unit_blocks_kernel(int* __restrict__ bp, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i <= n) bp[i] = i;
}

// Whether every neighbour comes earlier in the order (late is set where one does not).
__global__ void sim_check_kernel(const int* __restrict__ nbr_ptr, const int* __restrict__ nbr_idx, int n,
                                 int* __restrict__ late) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), ln = threadIdx.x & 63;
  if (i >= n) return;
  const int o1 = nbr_ptr[i + 1];
  bool bad = false;
  for (int q = nbr_ptr[i] + ln; q < o1; q += 64) bad |= nbr_idx[q] < 0 || nbr_idx[q] >= i;
  if (bad) *late = 1;
}

// A value that is not drawn yet: a NaN that no arithmetic produces (results are
// written with NaNs made canonical).
constexpr unsigned long long kNotDrawn = 0x7ff8c0de51a1d00dull;

__global__ void sim_clear_kernel(unsigned long long* __restrict__ y, int64_t total, int* __restrict__ ticket, int nt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < total) y[i] = kNotDrawn;
  if (i < nt) ticket[i] = 0;
}

// One wave per point at a time, blockIdx.y the data set.  The point's weights and
// neighbour indices are read while the wave waits; the neighbours' values are
// polled where they are (value and readiness in one word, device-scope accesses,
// as the producer may run on another XCD).  Every neighbour index is below the
// point's, and points are taken in order, so the earliest unfinished point never
// waits; the poll count is bounded all the same, and a wave that reaches the bound
// says so and gives up.  20,000 points, 150 neighbours, 24 sets: the chain of
// dependent points is about 1,200 long (94 ms as 1,216 passes over all points).
constexpr int kSimPolls = 1 << 20;
constexpr int kSimRegs = 4;   // neighbours per lane in registers (up to 256; more are read again)
__global__ void __launch_bounds__(256)
sim_flow_kernel(const int* __restrict__ nbr_ptr, const int* __restrict__ nbr_idx, const double* __restrict__ coef,
                int64_t coef_stride, const double* __restrict__ cvar, const double* __restrict__ z,
                unsigned long long* __restrict__ y, int n, int* __restrict__ ticket, int* __restrict__ stuck) {
  const int ln = threadIdx.x & 63, t = blockIdx.y;
  const double* cf = coef + (size_t)t * coef_stride;
  unsigned long long* yt = y + (size_t)t * n;
  // All lanes store the result.  With `if (lane == 0)` around the store as well as
  // the ticket the compiler joined the end of one turn to the start of the next for
  // the other lanes, which then took ticket 0 again and again and never left.
  for (;;) {
    int i = 0;
    if (ln == 0) i = atomicAdd(&ticket[t], 1);
    __builtin_amdgcn_wave_barrier();
    i = __builtin_amdgcn_readfirstlane(i);
    if (i >= n) return;
    const int o0 = nbr_ptr[i], cnt = nbr_ptr[i + 1] - o0;
    const double noise = sqrt(cvar[(size_t)t * n + i]) * z[(size_t)t * n + i];
    double acc = 0.0;
    bool ok = true;
    for (int base = 0; base < cnt; base += 64 * kSimRegs) {
      int idx[kSimRegs];
      double w[kSimRegs];
      unsigned long long v[kSimRegs];
#pragma unroll
      for (int k = 0; k < kSimRegs; ++k) {
        const int q = base + 64 * k + ln;
        idx[k] = q < cnt ? nbr_idx[o0 + q] : -1;
        w[k] = q < cnt ? cf[o0 + q] : 0.0;
        v[k] = q < cnt ? kNotDrawn : 0ull;
      }
      int polls = 0;
      for (;;) {
        bool wait = false;
#pragma unroll
        for (int k = 0; k < kSimRegs; ++k)
          if (v[k] == kNotDrawn) {
            v[k] = __hip_atomic_load(&yt[idx[k]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wait |= v[k] == kNotDrawn;
          }
        if (!__any(wait)) break;
        __builtin_amdgcn_s_sleep(1);
        ++polls;
        if (polls >= kSimPolls ||
            (polls % 1024 == 0 && __hip_atomic_load(stuck, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
          ok = false;
          break;
        }
      }
#pragma unroll
      for (int k = 0; k < kSimRegs; ++k)
        if (idx[k] >= 0) acc += w[k] * __longlong_as_double((long long)v[k]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (!ok) {   // gives up, and with it every wave that waits
      __hip_atomic_store(stuck, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    const double r = acc + noise;   // the same in every lane
    const unsigned long long bits = r == r ? (unsigned long long)__double_as_longlong(r) : 0x7ff8000000000000ull;
    __hip_atomic_store(&yt[i], bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// grid.y runs over the data sets that share the design (same neighbour lists)
__global__ void sim_pass_kernel(const int* __restrict__ nbr_ptr, const int* __restrict__ nbr_idx,
                                const double* __restrict__ coef, int64_t coef_stride, const double* __restrict__ cvar,
                                const double* __restrict__ z, double* __restrict__ y, int* __restrict__ done, int n,
                                int pass, int* __restrict__ ndone) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int t = blockIdx.y;
  if (i >= n) return;
  int* dn = done + (size_t)t * (n + 8);
  if (dn[i] != 0) return;
  const int o0 = nbr_ptr[i], o1 = nbr_ptr[i + 1];
  const double* cf = coef + (size_t)t * coef_stride;
  const double* yy = y + (size_t)t * n;
  double acc = 0.0;
  for (int q = o0; q < o1; ++q) {
    const int j = nbr_idx[q];
    const int dj = dn[j];
    if (dj == 0 || dj >= pass) return;  // a neighbour is not drawn yet
    acc += cf[q] * yy[j];
  }
  y[(size_t)t * n + i] = acc + sqrt(cvar[(size_t)t * n + i]) * z[(size_t)t * n + i];
  dn[i] = pass;
  atomicAdd(ndone, 1);
}

}  // namespace bv

using namespace bv;

namespace {
constexpr int kCoefMaxG = 10;   // tile rows of the one-wave coefficient kernels
inline size_t al256s(size_t x) { return (x + 255) & ~(size_t)255; }
struct SimLayout {
  size_t bp, cfg, sched, counts, stats, coef, cvar, flag, done, total;
};
SimLayout sim_layout(int64_t n, int64_t nnz, int64_t nt) {
  SimLayout L;
  size_t o = 0;
  L.bp = o;     o = al256s(o + sizeof(int) * (n + 1));
  L.cfg = o;    o = al256s(o + sizeof(int) * n);
  L.sched = o;  o = al256s(o + sizeof(int) * n);
  L.counts = o; o = al256s(o + sizeof(int) * 64);
  L.stats = o;  o = al256s(o + sizeof(unsigned long long) * 8 + sizeof(int) * (16 + 32));
  L.coef = o;   o = al256s(o + sizeof(double) * (nnz > 0 ? nnz : 1) * nt);
  L.cvar = o;   o = al256s(o + sizeof(double) * n * nt);
  L.flag = o;   o = al256s(o + sizeof(int) * n * nt);
  L.done = o;   o = al256s(o + sizeof(int) * (n + 8) * nt + 64);
  L.total = o;
  return L;
}
template <typename P> P* at(void* base, size_t off) { return reinterpret_cast<P*>(static_cast<char*>(base) + off); }
}  // namespace

#define SCHECK(x)                              \
  do {                                         \
    hipError_t e_ = (x);                       \
    if (e_ != hipSuccess) return VECCHIA_EHIP; \
  } while (0)

extern "C" size_t vecchia_simulate_workspace_size(int64_t n, int64_t nnz, int32_t ntheta) {
  if (n <= 0 || nnz < 0 || ntheta <= 0) return 0;
  return sim_layout(n, nnz, ntheta).total;
}

extern "C" int vecchia_simulate(const double* locs_ord, int64_t n, int32_t d, const int32_t* nbr_ptr,
                                const int32_t* nbr_idx, const vecchia_theta* theta, int32_t ntheta, const double* z,
                                double* y, void* workspace, size_t ws_bytes, void* stream) {
  if (!locs_ord || !nbr_ptr || !nbr_idx || !theta || !z || !y || !workspace) return VECCHIA_EINVAL;
  if (n <= 0 || d < 1 || d > 3 || n >= ((int64_t)1 << 31)) return VECCHIA_EINVAL;
  if (ntheta < 1 || ntheta > kMaxThetaPerLaunch || (int64_t)ntheta * (n + 8) >= ((int64_t)1 << 31))
    return VECCHIA_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  int hnnz = 0;
  SCHECK(hipMemcpyAsync(&hnnz, nbr_ptr + n, sizeof(int), hipMemcpyDeviceToHost, s));
  SCHECK(hipStreamSynchronize(s));
  const SimLayout L = sim_layout(n, hnnz, ntheta);
  if (ws_bytes < L.total) return VECCHIA_ENOMEM;
  ThetaPack thp;
  memset(&thp, 0, sizeof(thp));
  for (int q = 0; q < ntheta; ++q) {
    const vecchia_theta& t = theta[q];
    if (!(t.sigma2 > 0) || !(t.range > 0) || !(t.nugget >= 0)) return VECCHIA_EINVAL;
    ThetaDev& o = thp.t[q];
    if (t.nu == 0.5) o.nu_code = 0;
    else if (t.nu == 1.5) o.nu_code = 1;
    else if (t.nu == 2.5) o.nu_code = 2;
    else return VECCHIA_EUNSUPPORTED;
    o.sigma2 = t.sigma2;
    o.nugget = t.nugget;
    o.inv_range = 1.0 / t.range;
    for (int k = 0; k < 3; ++k) o.inv_scale[k] = k < d ? 1.0 / (t.range * t.aniso[k]) : 0.0;
  }
  int* bp = at<int>(workspace, L.bp);
  int* cfg = at<int>(workspace, L.cfg);
  int* sched = at<int>(workspace, L.sched);
  int* counts = at<int>(workspace, L.counts);
  unsigned long long* stats = at<unsigned long long>(workspace, L.stats);
  int* maxes = reinterpret_cast<int*>(stats + 8);
  const int ni = (int)n;
  hipLaunchKernelGGL(unit_blocks_kernel, dim3((ni + 256) / 256), dim3(256), 0, s, bp, ni);
  SCHECK(launch_fill_int(counts, 64, 0, s));
  int* lmax_cfg = maxes + 16;
  SCHECK(launch_fill_int(reinterpret_cast<int*>(stats), 16 + 16 + 32, 0, s));
  SCHECK(launch_classify(bp, nbr_ptr, ni, cfg, counts, stats, maxes, lmax_cfg, kEngineMfmaWg, 1, s));
  int hc[32], hmax[4];
  SCHECK(hipMemcpyAsync(hc, counts, sizeof(hc), hipMemcpyDeviceToHost, s));
  SCHECK(hipMemcpyAsync(hmax, maxes, sizeof(hmax), hipMemcpyDeviceToHost, s));
  SCHECK(hipStreamSynchronize(s));
  if (hmax[3] > 0) return hmax[0] > VECCHIA_MAX_JOINT ? VECCHIA_EUNSUPPORTED : VECCHIA_EINVAL;
  int hoff[32], acc = 0;
  for (int c = 0; c < kMfmaMaxG; ++c) {
    hoff[c] = acc;
    acc += hc[c];
  }
  SCHECK(hipMemcpyAsync(counts + 32, hoff, sizeof(int) * kMfmaMaxG, hipMemcpyHostToDevice, s));
  SCHECK(launch_fill_int(counts, 32, 0, s));
  SCHECK(launch_scatter(cfg, ni, counts + 32, counts, sched, s));
  AdjArgs a;
  memset(&a, 0, sizeof(a));
  a.locs = locs_ord;
  a.y = nullptr;
  a.block_ptr = bp;
  a.nbr_ptr = nbr_ptr;
  a.nbr_idx = nbr_idx;
  a.ntheta = ntheta;
  a.bc = ni;
  a.coef_stride = hnnz;
  a.d = d;
  a.ldx = mfma_ldx(1);
  a.flag = at<int>(workspace, L.flag);
  a.coef = at<double>(workspace, L.coef);
  a.cvar = at<double>(workspace, L.cvar);
  for (int c = 0; c < kMfmaMaxG; ++c) {
    if (hc[c] == 0) continue;
    a.sched = sched + hoff[c];
    a.nsched = hc[c];
    if (c + 1 <= kCoefMaxG) SCHECK(launch_wave_f64_coef(c + 1, a, thp, hc[c] * ntheta, s));
    else SCHECK(launch_mfma(c + 1, false, 2, a, thp, hc[c] * ntheta, s));
  }
  int* done = at<int>(workspace, L.done);
  // recursion: counts[0] a neighbour that is not earlier, [1] a wave that gave up,
  // done[0 ..] the tickets of the sets
  SCHECK(launch_fill_int(counts, 2, 0, s));
  hipLaunchKernelGGL(sim_check_kernel, dim3((ni + 3) / 4), dim3(256), 0, s, nbr_ptr, nbr_idx, ni, counts);
  SCHECK(hipGetLastError());
  int flags[2];
  SCHECK(hipMemcpyAsync(flags, counts, sizeof(flags), hipMemcpyDeviceToHost, s));
  SCHECK(hipStreamSynchronize(s));
  const int64_t ny = n * ntheta;   // (y over z: the passes read z[i] before they write y[i])
  if (flags[0] == 0 && (y + ny <= z || z + ny <= y)) {
    unsigned long long* yw = reinterpret_cast<unsigned long long*>(y);
    hipLaunchKernelGGL(sim_clear_kernel, dim3((unsigned)((ny + 255) / 256)), dim3(256), 0, s, yw, ny, done, ntheta);
    // about 2,048 waves in all, no more than a sixteenth of the points of a set
    const int per = std::max(1, std::min(512 / ntheta, (ni + 63) / 64));
    hipLaunchKernelGGL(sim_flow_kernel, dim3(per, ntheta), dim3(256), 0, s, nbr_ptr, nbr_idx, a.coef, (int64_t)hnnz,
                       a.cvar, z, yw, ni, done, counts + 1);
    SCHECK(hipGetLastError());
    SCHECK(hipMemcpyAsync(flags, counts, sizeof(flags), hipMemcpyDeviceToHost, s));
    SCHECK(hipStreamSynchronize(s));
    return flags[1] ? VECCHIA_EHIP : VECCHIA_OK;
  }
  // recursion in passes
  int* ndone = done + (size_t)(n + 8) * ntheta;
  SCHECK(launch_fill_int(done, (ni + 8) * ntheta + 8, 0, s));
  const int target = ni * ntheta;
  int total = 0;
  for (int pass = 1; total < target; pass += 16) {
    for (int q = 0; q < 16; ++q)
      hipLaunchKernelGGL(sim_pass_kernel, dim3((ni + 255) / 256, ntheta), dim3(256), 0, s, nbr_ptr, nbr_idx, a.coef,
                         (int64_t)hnnz, a.cvar, z, y, done, ni, pass + q, ndone);
    SCHECK(hipGetLastError());
    int prev = total;
    SCHECK(hipMemcpyAsync(&total, ndone, sizeof(int), hipMemcpyDeviceToHost, s));
    SCHECK(hipStreamSynchronize(s));
    if (total == prev) return VECCHIA_EINVAL;  // no progress: a neighbour index is not earlier
  }
  return VECCHIA_OK;
}
