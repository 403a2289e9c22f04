// Learned warm start for the block Vecchia MLE: binned empirical
// semivariogram features and the kernels that train / run a small MLP
// (96 -> 256 -> 256 -> 3, ReLU) on the GPU.
//
// Variogram: for each data set, all pairs of a subset of k points; pair (i, j),
// i < j, with 0 < h <= h_max falls in bin floor(h / h_max * nbins) (clamped to
// nbins - 1), decided in FP64.  Bin sums of (y_i - y_j)^2 and counts accumulate
// per workgroup in LDS (FP64 sums), workgroup partials are reduced in a fixed
// order, and the features are gamma_k / s2 (gamma_k = sum / (2 N_k), s2 = subset variance)
// placed in the data set's smoothness slot (one-hot over nu in {1/2, 3/2, 5/2}).
//
// GEMM: C = op(A) op(B) with BF16 operands on the matrix cores
// (v_mfma_f32_16x16x16_bf16, FP32 accumulation); the epilogue adds a bias,
// applies ReLU, or multiplies by the ReLU mask of a pre-activation (backward).
// Operands are FP32 in memory (master copies) and rounded to BF16 (round to
// nearest even) as they are loaded; mode FP32 uses plain FP32 FMAs instead.
#include <math.h>
#include <string.h>

#include "internal.hpp"

namespace bv {

// ------------------------------------------------------------- variogram --

constexpr int VG_T = 256;
constexpr int VG_MAXBINS = 64;
constexpr int VG_STAGE = 2048;  // partials staged in LDS at once
static_assert(VG_MAXBINS <= VG_T && VG_MAXBINS <= VG_STAGE, "one thread per bin");
constexpr int VG_COPIES = 16;   // copies of each bin's sum in LDS, by lane

// Bin of a pair at squared distance d2, or -1: the integer that the definition
// decides in FP64 without fused multiply-add, h = sqrt(d2), 0 < h <= hmax,
// floor(h / hmax * nbins).  An estimate good to 1e-14 decides it unless it falls
// within 1e-9 of an integer; only those pairs evaluate the definition itself (and all
// pairs where hmax is so small that the 1e-300 below shows: scale is a NaN then).
__device__ __forceinline__ int vg_bin(double d2, double hmax, double scale, int nbins) {
  const double x = d2 + 1e-300;
  const double y = __builtin_amdgcn_rsq(x);
  const double g = x * y;
  const double e = __builtin_fma(-g, y, 1.0);
  const double t = __builtin_fma(g * e, __builtin_fma(e, 0.375, 0.5), g) * scale;
  const double fl = floor(t), fr = t - fl;
  if (fr > 1e-9 && fr < 1.0 - 1e-9) return fl < (double)nbins ? (int)fl : -1;
  {
#pragma clang fp contract(off)
    const double h = sqrt(d2);
    const int bin = (h > 0.0 && h <= hmax) ? (int)(h / hmax * (double)nbins) : -1;
    return bin < nbins ? bin : nbins - 1;
  }
}

// grid: (row chunks, groups of S data sets).  Workgroup g of a group handles rows
// i = g, g + gridDim.x, ... against all j > i, once for the S sets that share a
// design (S = 1 where each has its own).  What bounds it: one LDS addition per
// pair and set; a bin's sum is kept VG_COPIES times, by lane, so that the
// lanes of a wave meet on few addresses, and the distances are formed once for
// S sets.  64 sets of 4,096 points: 923 us with one copy and one set at a time,
// 296 so (no change with 32 copies); two sets 220 and 152 us, although six of the
// eight sums go unused.
template <int S, int T>
__global__ void __launch_bounds__(T)
variogram_pairs_kernel(const double* __restrict__ locs, int64_t locs_stride, const double* __restrict__ y,
                       int64_t y_stride, int k, int nsets, int nbins, double hmax, double* __restrict__ part_sum,
                       unsigned* __restrict__ part_cnt) {
  extern __shared__ __align__(16) unsigned char vg_smem[];
  double* ssum = reinterpret_cast<double*>(vg_smem);                                   // [S][nbins][VG_COPIES]
  unsigned* scnt = reinterpret_cast<unsigned*>(ssum + (size_t)S * nbins * VG_COPIES);   // [nbins][VG_COPIES]
  const int b0 = blockIdx.y * S;
  const double* L = locs + (size_t)b0 * locs_stride;
  const int per = nbins * VG_COPIES;
  for (int q = threadIdx.x; q < S * per; q += T) ssum[q] = 0.0;
  for (int q = threadIdx.x; q < per; q += T) scnt[q] = 0u;
  __syncthreads();
  const int copy = threadIdx.x & (VG_COPIES - 1);
  const double scale = hmax > 1e-130 ? (double)nbins / hmax : (double)NAN;
  const double* Y[S];
#pragma unroll
  for (int u = 0; u < S; ++u) Y[u] = y + (size_t)(b0 + u < nsets ? b0 + u : nsets - 1) * y_stride;
  for (int i = blockIdx.x; i < k - 1; i += gridDim.x) {
    const double xi = L[2 * i], yi = L[2 * i + 1];
    double vi[S];
#pragma unroll
    for (int u = 0; u < S; ++u) vi[u] = Y[u][i];
    for (int j = i + 1 + threadIdx.x; j < k; j += T) {
      double d2, vj[S];
#pragma unroll
      for (int u = 0; u < S; ++u) vj[u] = Y[u][j];
      {
#pragma clang fp contract(off)
        const double dx = L[2 * j] - xi, dy = L[2 * j + 1] - yi;
        d2 = dx * dx + dy * dy;
      }
      const int bin = vg_bin(d2, hmax, scale, nbins);
      if (bin >= 0) {
        const int o = bin * VG_COPIES + copy;
#pragma unroll
        for (int u = 0; u < S; ++u) {
          const double dv = vj[u] - vi[u];
          atomicAdd(&ssum[u * per + o], dv * dv);
        }
        atomicAdd(&scnt[o], 1u);
      }
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < S * nbins; q += T) {
    const int u = q / nbins, bin = q - u * nbins;
    if (b0 + u >= nsets) continue;
    double sum = 0.0;
    unsigned cnt = 0u;
    for (int c = 0; c < VG_COPIES; ++c) {
      sum += ssum[u * per + bin * VG_COPIES + c];
      cnt += scnt[bin * VG_COPIES + c];
    }
    const size_t o = ((size_t)(b0 + u) * gridDim.x + blockIdx.x) * nbins + bin;
    part_sum[o] = sum;
    part_cnt[o] = cnt;
  }
}

template <int S, int T>
hipError_t launch_pairs(const double* locs, int64_t locs_stride, const double* y, int64_t y_stride, int k, int nsets,
                        int nbins, double hmax, int nchunks, double* ps, unsigned* pc, hipStream_t s) {
  const size_t lds = (size_t)nbins * VG_COPIES * (S * sizeof(double) + sizeof(unsigned));
  hipLaunchKernelGGL((variogram_pairs_kernel<S, T>), dim3(nchunks, (nsets + S - 1) / S), dim3(T), lds, s, locs,
                     locs_stride, y, y_stride, k, nsets, nbins, hmax, ps, pc);
  return hipGetLastError();
}

// one workgroup per data set: fixed-order reduction of the partials, subset
// variance, normalised features in the nu slot
__global__ void __launch_bounds__(VG_T)
variogram_features_kernel(const double* __restrict__ y, int64_t y_stride, int k, int nbins, int nchunks,
                          const double* __restrict__ part_sum, const unsigned* __restrict__ part_cnt,
                          const int* __restrict__ nu_slot, int nslots, float* __restrict__ feat,
                          double* __restrict__ gamma_out) {
  __shared__ double s1[VG_T], s2[VG_T], ps[VG_STAGE];
  __shared__ unsigned pc[VG_STAGE];
  const int b = blockIdx.x;
  const double* Y = y + (size_t)b * y_stride;
  double a1 = 0.0, a2 = 0.0;
#pragma unroll 16
  for (int i = threadIdx.x; i < k; i += VG_T) {
    const double v = Y[i];
    a1 += v;
    a2 += v * v;
  }
  s1[threadIdx.x] = a1;
  s2[threadIdx.x] = a2;
  __syncthreads();
  for (int s = VG_T / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      s1[threadIdx.x] += s1[threadIdx.x + s];
      s2[threadIdx.x] += s2[threadIdx.x + s];
    }
    __syncthreads();
  }
  const double mean = s1[0] / k;
  const double var = s2[0] / k - mean * mean;
  const int slot = nu_slot[b];
  for (int q = threadIdx.x; q < nbins * nslots; q += VG_T) feat[(size_t)b * nbins * nslots + q] = 0.f;
  __syncthreads();
  // the partials through LDS, VG_STAGE at a time, then one thread per bin in chunk order
  double sum = 0.0;
  unsigned long long cnt = 0;
  const int q = threadIdx.x, step = VG_STAGE / nbins;
  for (int c0 = 0; c0 < nchunks; c0 += step) {
    const int nc = nchunks - c0 < step ? nchunks - c0 : step;
    const size_t o = ((size_t)b * nchunks + c0) * nbins;
    __syncthreads();
#pragma unroll 8
    for (int e = threadIdx.x; e < nc * nbins; e += VG_T) {
      ps[e] = part_sum[o + e];
      pc[e] = part_cnt[o + e];
    }
    __syncthreads();
    if (q < nbins) {
#pragma unroll 8
      for (int c = 0; c < nc; ++c) {
        sum += ps[c * nbins + q];
        cnt += pc[c * nbins + q];
      }
    }
  }
  if (q < nbins) {
    const double g = cnt ? sum / (2.0 * (double)cnt) : 0.0;
    if (gamma_out) gamma_out[(size_t)b * nbins + q] = g;
    feat[(size_t)b * nbins * nslots + (size_t)slot * nbins + q] = (float)(g / var);
  }
}

// ------------------------------------------------------------------- GEMM --

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ short f32_to_bf16_rne(float f) {
  unsigned u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (short)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));  // inf / nan
  u += 0x7fffu + ((u >> 16) & 1u);
  return (short)(u >> 16);
}

struct GemmArgs {
  const float* A;
  const float* B;
  float* C;
  const float* bias;   // length N or NULL
  const float* mask;   // pre-activation of the same shape as C (ReLU backward) or NULL
  float* Z;            // if non-NULL, pre-activation output (before ReLU)
  int M, N, K;
  int lda, ldb, ldc;
  int ta, tb;          // op(A) = A^T if ta (A stored K x M), op(B) = B^T if tb (B stored N x K)
  int act;             // 0 none, 1 ReLU
  int beta_accum;      // 1: C += result
};

__device__ __forceinline__ float ldA(const GemmArgs& g, int m, int k) {
  if (m >= g.M || k >= g.K) return 0.f;
  return g.ta ? g.A[(size_t)k * g.lda + m] : g.A[(size_t)m * g.lda + k];
}
__device__ __forceinline__ float ldB(const GemmArgs& g, int k, int n) {
  if (n >= g.N || k >= g.K) return 0.f;
  return g.tb ? g.B[(size_t)n * g.ldb + k] : g.B[(size_t)k * g.ldb + n];
}

__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, int m, int n, float v) {
  if (m >= g.M || n >= g.N) return;
  const size_t o = (size_t)m * g.ldc + n;
  if (g.bias) v += g.bias[n];
  if (g.Z) g.Z[o] = v;
  if (g.act == 1) v = v > 0.f ? v : 0.f;
  if (g.mask) v = g.mask[o] > 0.f ? v : 0.f;
  if (g.beta_accum) v += g.C[o];
  g.C[o] = v;
}

// One workgroup of four waves per 16 x 16 output tile, BF16 MFMA over K in steps of
// 16.  The layers are small (256 x 256 x 256 is 256 tiles), so a launch lasts as
// long as its loads: the waves read the operands of 16 steps together, round them
// and lay them out in LDS as the matrix instruction takes them, and the first wave
// multiplies, step by step in the order of K.  256^3: 23 us with one wave and
// one step at a time, 11 us with one wave and eight steps in flight, 7-8 us so.
constexpr int GEMM_T = 256, GEMM_STEPS = 16;
struct GemmLds {
  bf16x4 a[GEMM_STEPS][64], b[GEMM_STEPS][64];
};
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, int m0, int n0, GemmLds& lds) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int row = l & 15, kq = (l >> 4) * 4;
  constexpr int PER = GEMM_STEPS / 4;   // steps of one wave
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  // whole tiles along M and N read without bounds checks (K is checked per group)
  const bool inside = m0 + 16 <= g.M && n0 + 16 <= g.N;
  const float* pa = g.A + (g.ta ? (size_t)kq * g.lda + m0 + row : (size_t)(m0 + row) * g.lda + kq);
  const float* pb = g.B + (g.tb ? (size_t)(n0 + row) * g.ldb + kq : (size_t)kq * g.ldb + n0 + row);
  const int sa = g.ta ? g.lda : 1, sb = g.tb ? 1 : g.ldb;
  for (int k0 = 0; k0 < g.K; k0 += 16 * GEMM_STEPS) {
    const int left = (g.K - k0 + 15) / 16, steps = left < GEMM_STEPS ? left : GEMM_STEPS;
    float a[PER][4], b[PER][4];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int kk = k0 + 16 * (w * PER + q);
      if (inside && kk + 16 <= g.K) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          a[q][j] = pa[(size_t)(kk + j) * sa];
          b[q][j] = pb[(size_t)(kk + j) * sb];
        }
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          a[q][j] = ldA(g, m0 + row, kk + kq + j);
          b[q][j] = ldB(g, kk + kq + j, n0 + row);
        }
      }
    }
    __syncthreads();   // the first wave is done with the previous group
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      bf16x4 av, bv;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        av[j] = f32_to_bf16_rne(a[q][j]);
        bv[j] = f32_to_bf16_rne(b[q][j]);
      }
      lds.a[w * PER + q][l] = av;
      lds.b[w * PER + q][l] = bv;
    }
    __syncthreads();
    if (w == 0)
      for (int q = 0; q < steps; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(lds.a[q][l], lds.b[q][l], acc, 0, 0, 0);
  }
  // accumulator: lane l holds rows 4*(l/16) + r of column l % 16
  if (w == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) gemm_epilogue(g, m0 + kq + r, n0 + row, acc[r]);
  }
}

__global__ void __launch_bounds__(GEMM_T) gemm_bf16_kernel(GemmArgs g) {
  __shared__ GemmLds lds;
  gemm_tile(g, blockIdx.y * 16, blockIdx.x * 16, lds);
}

// One wave per tile and one step at a time: the same products in the same order.
__global__ void __launch_bounds__(64) gemm_bf16_wave_kernel(GemmArgs g) {
  const int l = threadIdx.x, row = l & 15, kq = (l >> 4) * 4;
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < g.K; k0 += 16) {
    bf16x4 a, b;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[j] = f32_to_bf16_rne(ldA(g, m0 + row, k0 + kq + j));
      b[j] = f32_to_bf16_rne(ldB(g, k0 + kq + j, n0 + row));
    }
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) gemm_epilogue(g, m0 + kq + r, n0 + row, acc[r]);
}
// With fewer than eight steps two or three of a workgroup's four waves have nothing to
// load; once the tiles fill the chip several times over, one wave per tile is the faster
// kernel: M x 256 x K, four waves / one wave, 20,000 x 32 50 / 25 us, x 64 55 / 44,
// x 96 66 / 64, x 128 79 / 83; 4,096 x 32 13.5 / 8.4, x 96 18.8 / 16.6, and 2,000 x 96
// (2,000 tiles) 11.1 / 10.8 and with A transposed 8.7 / 11.0.
constexpr int GEMM_WAVE_K = 128, GEMM_WAVE_TILES = 4096;

// FP32 reference mode: 16 x 16 tile per 256 threads, plain FMAs
__global__ void __launch_bounds__(256) gemm_f32_kernel(GemmArgs g) {
  const int n = blockIdx.x * 16 + (threadIdx.x & 15);
  const int m = blockIdx.y * 16 + (threadIdx.x >> 4);
  float acc = 0.f;
  for (int k = 0; k < g.K; ++k) acc += ldA(g, m, k) * ldB(g, k, n);
  gemm_epilogue(g, m, n, acc);
}

// --------------------------------------------------------- loss / adam ---

// MSE over all B x D entries: dOut = 2 (out - T) / (B D); loss partials per workgroup
__global__ void __launch_bounds__(256)
mse_kernel(const float* __restrict__ out, const float* __restrict__ tgt, int total, float* __restrict__ dout,
           double* __restrict__ loss_part) {
  __shared__ double s[256];
  double acc = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const float d = out[i] - tgt[i];
    dout[i] = 2.f * d / (float)total;
    acc += (double)d * (double)d;
  }
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int q = 128; q > 0; q >>= 1) {
    if (threadIdx.x < q) s[threadIdx.x] += s[threadIdx.x + q];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss_part[blockIdx.x] = s[0] / (double)total;
}

// column sums of an M x N matrix (bias gradients): a workgroup of 256 threads takes
// 16 columns, reads 256 rows of them together into LDS, and one thread per column
// adds them in row order (one load at a time took 23 us for 256 rows)
constexpr int CS_COLS = 16, CS_ROWS = 256;
struct ColsumLds {
  float x[CS_ROWS][CS_COLS + 1];
};
__device__ __forceinline__ void colsum_columns(const float* __restrict__ X, int M, int N, int ld, int n0,
                                               float* __restrict__ out, ColsumLds& lds) {
  const int c = threadIdx.x & (CS_COLS - 1), r0 = threadIdx.x / CS_COLS, n = n0 + c;
  float acc = 0.f;
  for (int m0 = 0; m0 < M; m0 += CS_ROWS) {
    const int rows = M - m0 < CS_ROWS ? M - m0 : CS_ROWS;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < CS_ROWS / 16; ++q) {
      const int r = r0 + 16 * q;
      if (r < rows && n < N) lds.x[r][c] = X[(size_t)(m0 + r) * ld + n];
    }
    __syncthreads();
    if (r0 == 0 && n < N) {
#pragma unroll 16
      for (int r = 0; r < rows; ++r) acc += lds.x[r][c];
    }
  }
  if (r0 == 0 && n < N) out[n] = acc;
}

__global__ void __launch_bounds__(256) colsum_kernel(const float* __restrict__ X, int M, int N, int ld,
                                                     float* __restrict__ out) {
  __shared__ ColsumLds lds;
  colsum_columns(X, M, N, ld, blockIdx.x * CS_COLS, out, lds);
}

// Up to two products and a column sum that need nothing of each other in one
// launch: workgroup w belongs to the first product whose tiles end above it, the
// workgroups after all tiles sum columns.
constexpr int GROUP_MAX = 2;
struct GroupArgs {
  GemmArgs g[GROUP_MAX];
  int tiles[GROUP_MAX];   // running count of 16 x 16 tiles
  int ng;
  const float* cs_x;      // column sums: M x N, to cs_out (null: none)
  float* cs_out;
  int cs_m, cs_n, cs_ld;
};
__global__ void __launch_bounds__(GEMM_T) gemm_group_kernel(GroupArgs a) {
  __shared__ union {
    GemmLds g;
    ColsumLds c;
  } lds;
  const int w = blockIdx.x;
#pragma unroll
  for (int q = 0; q < GROUP_MAX; ++q) {
    if (q < a.ng && w < a.tiles[q]) {
      const int t = w - (q ? a.tiles[q ? q - 1 : 0] : 0);
      const int nt = (a.g[q].N + 15) / 16;
      gemm_tile(a.g[q], t / nt * 16, t % nt * 16, lds.g);
      return;
    }
  }
  colsum_columns(a.cs_x, a.cs_m, a.cs_n, a.cs_ld, (w - a.tiles[a.ng - 1]) * CS_COLS, a.cs_out, lds.c);
}

// Adam (Kingma & Ba) with bias correction; t is the 1-based step
__device__ __forceinline__ void adam_one(float* __restrict__ p, const float* __restrict__ gr, float* __restrict__ m,
                                         float* __restrict__ v, int i, float lr, float b1, float b2, float eps,
                                         float c1, float c2) {
  const float g = gr[i];
  const float mi = b1 * m[i] + (1.f - b1) * g;
  const float vi = b2 * v[i] + (1.f - b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ gr, float* __restrict__ m,
                            float* __restrict__ v, int n, float lr, float b1, float b2, float eps, float c1,
                            float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) adam_one(p, gr, m, v, i, lr, b1, b2, eps, c1, c2);
}

// the six parameter arrays of the network in one launch, their elements one after
// the other
struct AdamGroup {
  float* p[6];
  const float* g[6];
  float* m[6];
  float* v[6];
  int end[6];   // running count of elements
};
__global__ void adam_group_kernel(AdamGroup a, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
#pragma unroll
  for (int q = 0; q < 6; ++q)
    if (i < a.end[q]) {
      adam_one(a.p[q], a.g[q], a.m[q], a.v[q], i - (q ? a.end[q - 1] : 0), lr, b1, b2, eps, c1, c2);
      return;
    }
}

}  // namespace bv

using namespace bv;

#define LCHECK(x)                              \
  do {                                         \
    hipError_t e_ = (x);                       \
    if (e_ != hipSuccess) return VECCHIA_EHIP; \
  } while (0)

extern "C" size_t vecchia_variogram_workspace_size(int32_t nsets, int32_t nbins, int32_t nchunks) {
  if (nsets <= 0 || nbins <= 0 || nchunks <= 0) return 0;
  return (size_t)nsets * nchunks * nbins * (sizeof(double) + sizeof(unsigned)) + 256;
}

extern "C" int vecchia_variogram(const double* locs, int64_t locs_stride, const double* y, int64_t y_stride,
                                 int32_t nsets, int32_t k, int32_t nbins, double hmax, const int32_t* nu_slot,
                                 int32_t nslots, float* features, double* gamma, int32_t nchunks, void* workspace,
                                 size_t ws_bytes, void* stream) {
  if (!locs || !y || !nu_slot || !features || !workspace) return VECCHIA_EINVAL;
  if (nsets <= 0 || k < 2 || nbins <= 0 || nbins > VG_MAXBINS || !(hmax > 0) || nslots <= 0 || nchunks <= 0)
    return VECCHIA_EINVAL;
  if (ws_bytes < vecchia_variogram_workspace_size(nsets, nbins, nchunks)) return VECCHIA_ENOMEM;
  hipStream_t s = (hipStream_t)stream;
  double* ps = static_cast<double*>(workspace);
  unsigned* pc = reinterpret_cast<unsigned*>(ps + (size_t)nsets * nchunks * nbins);
  // eight sets at a time on a shared design (four above 32 bins): at most 36 kB of
  // LDS, four workgroups of eight waves per compute unit.  2 to 16 sets of 4,096
  // points take 152 us at 32 bins and 109 us at 64, one set 153 us; with one set at a
  // time 220 to 318 us.
  if (locs_stride == 0 && nsets > 1 && nbins <= 32)
    LCHECK((launch_pairs<8, 512>(locs, 0, y, y_stride, k, nsets, nbins, hmax, nchunks, ps, pc, s)));
  else if (locs_stride == 0 && nsets > 1)
    LCHECK((launch_pairs<4, 512>(locs, 0, y, y_stride, k, nsets, nbins, hmax, nchunks, ps, pc, s)));
  else
    LCHECK((launch_pairs<1, VG_T>(locs, locs_stride, y, y_stride, k, nsets, nbins, hmax, nchunks, ps, pc, s)));
  hipLaunchKernelGGL(variogram_features_kernel, dim3(nsets), dim3(VG_T), 0, s, y, y_stride, k, nbins, nchunks, ps,
                     pc, nu_slot, nslots, features, gamma);
  LCHECK(hipGetLastError());
  return VECCHIA_OK;
}

extern "C" int vecchia_gemm(const float* A, const float* B, float* C, const float* bias, const float* mask, float* Z,
                            int32_t M, int32_t N, int32_t K, int32_t lda, int32_t ldb, int32_t ldc, int32_t ta,
                            int32_t tb, int32_t act, int32_t accumulate, int32_t use_bf16, void* stream) {
  if (!A || !B || !C || M <= 0 || N <= 0 || K <= 0) return VECCHIA_EINVAL;
  GemmArgs g;
  memset(&g, 0, sizeof(g));
  g.A = A;
  g.B = B;
  g.C = C;
  g.bias = bias;
  g.mask = mask;
  g.Z = Z;
  g.M = M;
  g.N = N;
  g.K = K;
  g.lda = lda;
  g.ldb = ldb;
  g.ldc = ldc;
  g.ta = ta;
  g.tb = tb;
  g.act = act;
  g.beta_accum = accumulate;
  const dim3 grid((N + 15) / 16, (M + 15) / 16);
  if (use_bf16 && K < GEMM_WAVE_K && (int64_t)grid.x * grid.y >= GEMM_WAVE_TILES)
    hipLaunchKernelGGL(gemm_bf16_wave_kernel, grid, dim3(64), 0, (hipStream_t)stream, g);
  else if (use_bf16)
    hipLaunchKernelGGL(gemm_bf16_kernel, grid, dim3(GEMM_T), 0, (hipStream_t)stream, g);
  else
    hipLaunchKernelGGL(gemm_f32_kernel, grid, dim3(256), 0, (hipStream_t)stream, g);
  LCHECK(hipGetLastError());
  return VECCHIA_OK;
}

extern "C" int vecchia_mse(const float* out, const float* target, int32_t total, float* dout, double* loss_part,
                           int32_t nparts, void* stream) {
  if (!out || !target || !dout || !loss_part || total <= 0 || nparts <= 0) return VECCHIA_EINVAL;
  hipLaunchKernelGGL(mse_kernel, dim3(nparts), dim3(256), 0, (hipStream_t)stream, out, target, total, dout, loss_part);
  LCHECK(hipGetLastError());
  return VECCHIA_OK;
}

extern "C" int vecchia_colsum(const float* X, int32_t M, int32_t N, int32_t ld, float* out, void* stream) {
  if (!X || !out || M <= 0 || N <= 0) return VECCHIA_EINVAL;
  hipLaunchKernelGGL(colsum_kernel, dim3((N + CS_COLS - 1) / CS_COLS), dim3(256), 0, (hipStream_t)stream, X, M, N, ld, out);
  LCHECK(hipGetLastError());
  return VECCHIA_OK;
}

extern "C" int vecchia_adam(float* param, const float* grad, float* m, float* v, int64_t n, double lr, double beta1,
                            double beta2, double eps, int64_t step, void* stream) {
  if (!param || !grad || !m || !v || n <= 0 || step < 1) return VECCHIA_EINVAL;
  const float c1 = (float)(1.0 - pow(beta1, (double)step));
  const float c2 = (float)(1.0 - pow(beta2, (double)step));
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, param, grad,
                     m, v, (int)n, (float)lr, (float)beta1, (float)beta2, (float)eps, c1, c2);
  LCHECK(hipGetLastError());
  return VECCHIA_OK;
}

// One training step of the three-layer network (see vecchia.h): eight launches
// where the separate entry points take eighteen, with the same operations in the
// same order for every value.  The workspace holds the activations, then the
// gradients.
namespace {
struct MlpLayout {
  size_t z1, a1, z2, a2, out, dout, dz2, dz1, grad[6], total;   // in floats
};
MlpLayout mlp_layout(int64_t b, const int32_t* n) {
  MlpLayout L;
  size_t o = 0;
  auto take = [&](int64_t k) {
    const size_t at = o;
    o += ((size_t)k + 63) & ~(size_t)63;
    return at;
  };
  L.z1 = take(b * n[1]);
  L.a1 = take(b * n[1]);
  L.z2 = take(b * n[2]);
  L.a2 = take(b * n[2]);
  L.out = take(b * n[3]);
  L.dout = take(b * n[3]);
  L.dz2 = take(b * n[2]);
  L.dz1 = take(b * n[1]);
  for (int q = 0; q < 3; ++q) {
    L.grad[2 * q] = take((int64_t)n[q] * n[q + 1]);
    L.grad[2 * q + 1] = take(n[q + 1]);
  }
  L.total = o;
  return L;
}
bool mlp_sizes_ok(int64_t b, const int32_t* n) {
  if (!n || b <= 0 || b > (1 << 20)) return false;
  for (int q = 0; q < 4; ++q)
    if (n[q] <= 0 || n[q] > 16384) return false;
  return b * n[3] < ((int64_t)1 << 31) - (1 << 24);   // the loss kernel counts the outputs in 32 bits
}
// C (M x N) = op(A) op(B), all row-major without gaps
GemmArgs mlp_gemm(const float* A, const float* B, float* C, int M, int N, int K, int ta, int tb) {
  GemmArgs g;
  memset(&g, 0, sizeof(g));
  g.A = A;
  g.B = B;
  g.C = C;
  g.M = M;
  g.N = N;
  g.K = K;
  g.lda = ta ? M : K;
  g.ldb = tb ? K : N;
  g.ldc = N;
  g.ta = ta;
  g.tb = tb;
  return g;
}
hipError_t launch_group(GroupArgs& a, hipStream_t s) {
  int w = 0;
  for (int q = 0; q < a.ng; ++q) {
    w += ((a.g[q].M + 15) / 16) * ((a.g[q].N + 15) / 16);
    a.tiles[q] = w;
  }
  if (a.cs_x) w += (a.cs_n + CS_COLS - 1) / CS_COLS;
  hipLaunchKernelGGL(gemm_group_kernel, dim3(w), dim3(GEMM_T), 0, s, a);
  return hipGetLastError();
}
}  // namespace

extern "C" size_t vecchia_mlp_step_workspace_size(int32_t batch, const int32_t* sizes) {
  return mlp_sizes_ok(batch, sizes) ? sizeof(float) * mlp_layout(batch, sizes).total : 0;
}

extern "C" int vecchia_mlp_step(const float* X, const float* target, int32_t batch, const int32_t* sizes,
                                float* const* params, float* const* m, float* const* v, double* loss_part,
                                int32_t nparts, double lr, double beta1, double beta2, double eps, int64_t step,
                                void* workspace, size_t ws_bytes, void* stream) {
  if (!X || !target || !params || !m || !v || !loss_part || !workspace || nparts <= 0 || step < 1) return VECCHIA_EINVAL;
  if (!mlp_sizes_ok(batch, sizes)) return VECCHIA_EINVAL;
  if ((int64_t)batch * sizes[3] + 256 * (int64_t)nparts > INT32_MAX) return VECCHIA_EINVAL;   // and in strides of its grid
  for (int q = 0; q < 6; ++q)
    if (!params[q] || !m[q] || !v[q]) return VECCHIA_EINVAL;
  const MlpLayout L = mlp_layout(batch, sizes);
  if (ws_bytes < sizeof(float) * L.total) return VECCHIA_ENOMEM;
  hipStream_t s = (hipStream_t)stream;
  float* w = static_cast<float*>(workspace);
  const int B = batch, n0 = sizes[0], n1 = sizes[1], n2 = sizes[2], n3 = sizes[3];
  float* z[2] = {w + L.z1, w + L.z2};
  float* act[2] = {w + L.a1, w + L.a2};
  float* grad[6];
  for (int q = 0; q < 6; ++q) grad[q] = w + L.grad[q];
  // forward: act = relu(Z = in W^T + b), out without the ReLU
  const float* in = X;
  for (int q = 0; q < 3; ++q) {
    GroupArgs a;
    memset(&a, 0, sizeof(a));
    a.ng = 1;
    a.g[0] = mlp_gemm(in, params[2 * q], q < 2 ? act[q] : w + L.out, B, sizes[q + 1], sizes[q], 0, 1);
    a.g[0].bias = params[2 * q + 1];
    if (q < 2) {
      a.g[0].Z = z[q];
      a.g[0].act = 1;
    }
    LCHECK(launch_group(a, s));
    in = act[q < 2 ? q : 1];
  }
  hipLaunchKernelGGL(mse_kernel, dim3(nparts), dim3(256), 0, s, w + L.out, target, B * n3, w + L.dout, loss_part);
  LCHECK(hipGetLastError());
  // backward: per layer the weight gradient d^T in, the bias gradient and the
  // gradient of the layer below, (d W) where Z > 0
  const float* d = w + L.dout;
  float* below[3] = {nullptr, w + L.dz1, w + L.dz2};
  const int width[4] = {n0, n1, n2, n3};
  for (int q = 2; q >= 0; --q) {
    GroupArgs a;
    memset(&a, 0, sizeof(a));
    a.ng = q > 0 ? 2 : 1;
    a.g[0] = mlp_gemm(d, q > 0 ? act[q - 1] : X, grad[2 * q], width[q + 1], width[q], B, 1, 0);
    if (q > 0) {
      a.g[1] = mlp_gemm(d, params[2 * q], below[q], B, width[q], width[q + 1], 0, 0);
      a.g[1].mask = z[q - 1];
    }
    a.cs_x = d;
    a.cs_out = grad[2 * q + 1];
    a.cs_m = B;
    a.cs_n = width[q + 1];
    a.cs_ld = width[q + 1];
    LCHECK(launch_group(a, s));
    d = below[q];
  }
  AdamGroup ag;
  int end = 0;
  for (int q = 0; q < 6; ++q) {
    ag.p[q] = params[q];
    ag.g[q] = grad[q];
    ag.m[q] = m[q];
    ag.v[q] = v[q];
    end += (q & 1) ? width[q / 2 + 1] : width[q / 2] * width[q / 2 + 1];
    ag.end[q] = end;
  }
  const float c1 = (float)(1.0 - pow(beta1, (double)step));
  const float c2 = (float)(1.0 - pow(beta2, (double)step));
  hipLaunchKernelGGL(adam_group_kernel, dim3((unsigned)((end + 255) / 256)), dim3(256), 0, s, ag, (float)lr,
                     (float)beta1, (float)beta2, (float)eps, c1, c2);
  LCHECK(hipGetLastError());
  return VECCHIA_OK;
}
