// FP64 value of the blocks above the register capacity (m_i + l_i > 175): one
// workgroup of four waves per block, left-looking by panels of four tile columns.
//
// What bounds it.  P^3 / 3 products per block on the matrix cores (64 cycles per
// 16 x 16 x 4 instruction) and the panel updates' re-reading of the factor,
// which for the blocks in flight exceeds every cache.  So the output of a panel is
// kept in accumulators, two row tiles by four tile columns per wave: an element of
// the factor is read P / 64 times instead of P / 16, one tile load feeds two to
// four products, the matrix itself is generated in the accumulators and never
// stored, and only the factor is written.  Tiles are stored as the operands
// of 16 x 16 x 4 products in lane order, 2 KB whole instead of columns of 128 B.
//
// The accumulators hold the transposed negated tile, -C_IJ^T: register q of lane
// (lr, lg) is row lr, column 4 q + lg, which is also the layout of an operand of
// four columns.  The row solves L_IJ = C_IJ L_JJ^-T therefore need no data
// movement: four columns are one product with the inverse of the 4 x 4 diagonal
// block, its result is the operand of the updates of the columns to the right.
// Only 4 x 4 inverses are used (inverses of whole tiles would lose accuracy
// with the condition of 16 columns).
//
// n = 20,000 in 1,500 blocks, m = 450 (p about 463, nu = 3/2): 5.41 ms with one
// tile column per panel and divisions in the row solves, 1.88 ms now.  Of the time the
// matrix cores work 42 % and the vector units 20 % (they share their
// cycles); the rest is waiting, mostly at the barriers around the diagonal
// blocks.  5.0 GB are read and 1.2 GB written past the L2, 3.3 TB/s where a copy
// reaches 4.9.  Measured and
// not better: three waves per SIMD (2.44 ms, scratch), the panel operands
// prefetched as the row operands are (2.16), neither prefetched (2.07).
#include "internal.hpp"

#include <type_traits>

namespace bv {

namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef double d2_t __attribute__((ext_vector_type(2), aligned(8)));

constexpr int W = 4;   // tile columns of a panel
constexpr int R = 2;   // row tiles of a wave in the row stage

__device__ __forceinline__ d4_t mma(double a, double b, d4_t c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// one wave's LDS accesses in program order across its lanes
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// operand s = 0..3 of a stored tile (columns 4 s .. 4 s + 3), the lane's element
struct Operand {
  d2_t v[2];
  __device__ __forceinline__ double operator[](int s) const { return v[s >> 1][s & 1]; }
};
__device__ __forceinline__ Operand load_tile(const double* tile, int ln) {
  Operand o;
  o.v[0] = *reinterpret_cast<const d2_t*>(tile + 2 * ln);
  o.v[1] = *reinterpret_cast<const d2_t*>(tile + 128 + 2 * ln);
  return o;
}

}  // namespace

// Two workgroups' waves per SIMD (256 registers): 64 accumulator registers, 48 of
// operands and the row operands of the next K step.
__global__ void __launch_bounds__(256, 2) bv_large_f64_kernel(LargeArgs a, ThetaPack thp) {
  __shared__ double sop[W * (W + 1) / 2][4][64];   // factor tiles of the panel's diagonal block, as operands
  __shared__ double sinv[W][4][16];                // negated inverses of its 4 x 4 diagonal blocks
  __shared__ double spub[4][16];                   // four columns of the diagonal tile being factored
  __shared__ double scol[4][16 * W];               // coordinates and y of the panel's columns
  __shared__ double spiv[16 * W], sw[16 * W];      // their pivots and border entries
  const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), ln = tid & 63, lr = ln & 15, lg = ln >> 4;
  const int total = a.list ? *a.list_count : a.nsched * a.ntheta;
  double* M = reinterpret_cast<double*>(a.ws) + (size_t)blockIdx.x * a.slot_elems;
  const d4_t zero = {0.0, 0.0, 0.0, 0.0};
  for (int wi = blockIdx.x; wi < total; wi += gridDim.x) {
    int b, tt;
    if (a.list) {
      const int e = a.list[wi];
      tt = e / a.bc;
      b = e - tt * a.bc;
    } else {
      tt = wi / a.nsched;
      b = a.sched[wi - tt * a.nsched];
    }
    const ThetaDev& th = thp.t[tt];
    const int b0 = a.block_ptr[b], b1 = a.block_ptr[b + 1];
    const int n0 = a.nbr_ptr[b], n1 = a.nbr_ptr[b + 1];
    const int l = b1 - b0, m = n1 - n0, p = m + l;
    const int G = (p + 1 + 15) >> 4, P = 16 * G;
    const size_t ld = (size_t)P;
    double* cs = M + ld * ld;   // cs[k * P + i]: coordinates in units of range / log2(e), so e^-x is the exp2 of a distance
    const int d = a.d;
    const double nug = th.nugget;
    const MaternCoef<double> mc(th.nu_code);
    const double ns0 = -th.sigma2, ns1 = ns0 * mc.c1 * kLn2, ns2 = ns0 * mc.c2 * (kLn2 * kLn2);
    // tile (I, K) of the factor, K < I: operands of four columns, [pair of operands][lane][operand]
    auto tile = [&](int I, int K) { return M + ((size_t)K * G + I) * 256; };
    __syncthreads();
    for (int i = tid; i < P; i += 256) {
      const int gi = i < m ? a.nbr_idx[n0 + i] : (b0 + i - m);
      for (int k = 0; k < 3; ++k) {
        double v = 0.0;
        if (i < p && k < d) v = (a.locs[(size_t)gi * d + k] - a.locs[(size_t)b0 * d + k]) * (th.inv_scale[k] * kLog2E);
        cs[k * ld + i] = v;
      }
    }
    // rows of tile I as the accumulators hold them
    double ci[3];
    auto row_coords = [&](int I) {
#pragma unroll
      for (int k = 0; k < 3; ++k) ci[k] = cs[k * ld + I * 16 + lr];
    };
    // -C_IJ^T before the updates; column tile c of the panel
    auto generate = [&](int I, int J, int c) __attribute__((always_inline)) {
      double dx[4], dy[4], dz[4], u[4];
      Exp2Parts e[4];
      d4_t v;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = c * 16 + 4 * r + lg;
        dx[r] = ci[0] - scol[0][j];
        dy[r] = ci[1] - scol[1][j];
        dz[r] = ci[2] - scol[2][j];
      }
      distance_exp2neg4<false>(dx, dy, dz, u, e);
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = MaternCoef<double>::neg_cov_log2(u[r], e[r], ns0, ns1, ns2);
      const int i = I * 16 + lr;
      if (I == J) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] -= 4 * r + lg == lr ? nug : 0.0;
      }
      if (I == G - 1) {   // the only row tile with rows from p on: row p holds y, later ones the identity
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = J * 16 + 4 * r + lg;
          const double yb = -scol[3][c * 16 + 4 * r + lg], id = i == j ? -1.0 : 0.0;
          const double rest = ((i == p) & (j < p)) ? yb : id;
          v[r] = ((i < p) & (j < p)) ? v[r] : rest;
        }
      }
      __builtin_amdgcn_sched_barrier(0);   // one tile at a time: their temporaries together would spill
      return v;
    };
    const double guard = a.fp32_guard == 2 ? INFINITY
        : a.fp32_guard ? fmax(0.5 * th.nugget, (double)p * 1.1920928955078125e-07 * (th.sigma2 + th.nugget))
        : 0.0;
    double acc_ll = 0.0;
    int flag = 0;
    for (int J0 = 0; J0 < G; J0 += W) {
      __threadfence_block();
      __syncthreads();   // the rows of the last panel (and the coordinates) are stored, its LDS is read
      if (tid < 16 * W) {
        const int j = J0 * 16 + tid;
        const bool in = j < P;
#pragma unroll
        for (int k = 0; k < 3; ++k) scol[k][tid] = in ? cs[k * ld + j] : 0.0;
        scol[3][tid] = j < p ? a.y[j < m ? a.nbr_idx[n0 + j] : (b0 + j - m)] : 0.0;
      }
      __syncthreads();
      // ---- diagonal block: wave w holds row tile J0 + w, its columns 0 .. w
      const int I = J0 + wv;
      const bool mine = I < G;
      d4_t acc[W];
      if (mine) {
        row_coords(I);
#pragma unroll
        for (int c = 0; c < W; ++c)
          if (c <= wv) acc[c] = generate(I, J0 + c, c);
#pragma nounroll
        for (int K = 0; K < J0; ++K) {
          const Operand own = load_tile(tile(I, K), ln);
          Operand o[W];
#pragma unroll
          for (int c = 0; c < W; ++c) o[c] = load_tile(tile(J0 + c <= I ? J0 + c : I, K), ln);
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < W; ++c)
              if (c <= wv) acc[c] = mma(o[c][s], own[s], acc[c]);
        }
      }
#pragma unroll
      for (int c = 0; c < W; ++c) {
        if (J0 + c >= G) break;
        if (wv == c) {
          // tile (c, c), four columns at a time: every lane factors the 4 x 4 block and solves its row
          const int q0 = (J0 + c) * 16;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            wave_order();
            spub[lg][lr] = -acc[c][q];
            wave_order();
            double D[4][4], x[4], rinv[4], piv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              x[i] = spub[i][lr];
#pragma unroll
              for (int j = 0; j <= i; ++j) D[i][j] = spub[j][4 * q + i];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const bool real = q0 + 4 * q + k < p;   // columns from p on: no factor
#pragma unroll
              for (int j = 0; j < k; ++j) {
                D[k][k] -= D[k][j] * D[k][j];
                x[k] -= x[j] * D[k][j];
              }
              piv[k] = real ? D[k][k] : 1.0;
              rinv[k] = real ? rsqrt_fast(piv[k]) : 0.0;
#pragma unroll
              for (int i = k + 1; i < 4; ++i) {
#pragma unroll
                for (int j = 0; j < k; ++j) D[i][k] -= D[i][j] * D[k][j];
                D[i][k] *= rinv[k];
              }
              x[k] *= rinv[k];
            }
            // the lane's element of the four columns, and row lg of the negated inverse
            double v = lg == 0 ? x[0] : lg == 1 ? x[1] : lg == 2 ? x[2] : x[3];
            v = lr >= 4 * q + lg ? v : 0.0;
            sop[c * (c + 1) / 2 + c][q][ln] = v;
            double z[4];   // column lr & 3 of the inverse
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              z[i] = (lr & 3) == i ? 1.0 : 0.0;
#pragma unroll
              for (int j = 0; j < i; ++j) z[i] -= D[i][j] * z[j];
              z[i] *= rinv[i];
            }
            if (ln < 4) {
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                sinv[c][q][4 * i + ln] = -z[i];
                spiv[c * 16 + 4 * q + i] = piv[i];
              }
            }
            if (I == G - 1 && lr == (p & 15)) sw[c * 16 + 4 * q + lg] = v;
            if (q < 3) acc[c] = mma(v, v, acc[c]);
          }
        }
        __syncthreads();
        if (c + 1 < W) {
          double x[4];
          if (mine && wv > c) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const double ai = lr < 4 ? sinv[c][q][4 * (lr & 3) + lg] : 0.0;
              x[q] = mma(ai, acc[c][q], zero)[0];
              if (q < 3) acc[c] = mma(sop[c * (c + 1) / 2 + c][q][ln], x[q], acc[c]);
              sop[wv * (wv + 1) / 2 + c][q][ln] = x[q];
              if (I == G - 1 && lr == (p & 15)) sw[c * 16 + 4 * q + lg] = x[q];
            }
          }
          __syncthreads();
          if (mine && wv > c) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int e = c + 1; e < W; ++e)
                if (e <= wv) acc[e] = mma(sop[e * (e + 1) / 2 + c][q][ln], x[q], acc[e]);
          }
        }
      }
      // ---- rows below: the row tiles are split evenly over the waves (the larger
      // shares go round from panel to panel), each takes R at a time and then
      // single ones
      {
        const int rows = G - J0 - W, share = rows > 0 ? rows >> 2 : 0, more = rows > 0 ? rows & 3 : 0;
        const int turn = (wv + (J0 >> 2) + wi) & 3;
        int I0 = J0 + W + turn * share + (turn < more ? turn : more);
        const int Ie = I0 + share + (turn < more ? 1 : 0);
        auto row_tiles = [&](auto N_c) __attribute__((always_inline)) {
          constexpr int N = decltype(N_c)::value;
          d4_t t[N][W];
          int It[N];
#pragma unroll
          for (int i = 0; i < N; ++i) {
            It[i] = I0 + i;
            row_coords(It[i]);
#pragma unroll
            for (int c = 0; c < W; ++c) t[i][c] = generate(It[i], J0 + c, c);
          }
          if (J0 > 0) {
            Operand x[N];
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = load_tile(tile(It[i], 0), ln);
#pragma nounroll
            for (int K = 0; K < J0; ++K) {
              const int Kn = K + 1 < J0 ? K + 1 : K;
              Operand xn[N], o[W];
#pragma unroll
              for (int c = 0; c < W; ++c) o[c] = load_tile(tile(J0 + c, K), ln);
#pragma unroll
              for (int i = 0; i < N; ++i) xn[i] = load_tile(tile(It[i], Kn), ln);
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int c = 0; c < W; ++c)
#pragma unroll
                  for (int i = 0; i < N; ++i) t[i][c] = mma(o[c][s], x[i][s], t[i][c]);
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int i = 0; i < N; ++i) x[i] = xn[i];
            }
          }
#pragma unroll
          for (int c = 0; c < W; ++c) {
            Operand x[N];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const double ai = lr < 4 ? sinv[c][q][4 * (lr & 3) + lg] : 0.0;
#pragma unroll
              for (int i = 0; i < N; ++i) x[i].v[q >> 1][q & 1] = mma(ai, t[i][c][q], zero)[0];
#pragma unroll
              for (int e = c; e < W; ++e) {
                if (e == c && q == 3) continue;
                const double le = sop[e * (e + 1) / 2 + c][q][ln];
#pragma unroll
                for (int i = 0; i < N; ++i) t[i][e] = mma(le, x[i][q], t[i][e]);
              }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
              double* out = tile(It[i], J0 + c);
              *reinterpret_cast<d2_t*>(out + 2 * ln) = x[i].v[0];
              *reinterpret_cast<d2_t*>(out + 128 + 2 * ln) = x[i].v[1];
              if (It[i] == G - 1 && lr == (p & 15)) {
#pragma unroll
                for (int q = 0; q < 4; ++q) sw[c * 16 + 4 * q + lg] = x[i][q];
              }
            }
          }
        };
        for (; I0 + R <= Ie; I0 += R) row_tiles(std::integral_constant<int, R>());
        for (; I0 < Ie; ++I0) row_tiles(std::integral_constant<int, 1>());
      }
      __syncthreads();
      // pivots and border entries of the panel: the first wave keeps running sums
      if (tid < 16 * W) {
        const int k = J0 * 16 + tid;
        if (k < p) {
          const double dd = spiv[tid];
          if (!(dd > guard)) flag |= a.fp32_guard ? 1 : 2;
          if (!(dd > 0.0)) flag |= 2;
          if (k >= m) acc_ll += log(dd) + sw[tid] * sw[tid];
        }
      }
    }
    if (wv == 0) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        acc_ll += __shfl_xor(acc_ll, off);
        flag |= __shfl_xor(flag, off);
      }
    }
    if (tid == 0) {
      const size_t o = (size_t)tt * a.bc + b;
      a.partial[o] = (flag & 2) && !a.fp32_guard ? __builtin_nan("") : -0.5 * (acc_ll + (double)l * kLog2Pi);
      a.flag[o] = flag | a.flag_or;
    }
  }
}

hipError_t launch_large_f64(const LargeArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  hipLaunchKernelGGL(bv_large_f64_kernel, dim3(grid), dim3(256), 0, s, a, thp);
  return hipGetLastError();
}

}  // namespace bv
