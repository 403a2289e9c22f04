// One-wave FP64 kernels on transposed tiles: the value of a block, and the
// conditional-mean weights and variance of single points for the simulator.
//
// The accumulators hold the transposed negated tile, -C_IJ^T: register q of lane
// (lr, lg) is row lr, column 4 q + lg of the tile, which is also the layout of
// an operand of four columns.  Of each panel of four columns only the diagonal tile's
// part passes through LDS (one element per lane); the other row tiles are solved by one
// product with the negated inverse of the 4 x 4 block, whose result is the
// operand of the updates.  The general kernel (wave_kernel.hpp) keeps its tiles
// untransposed, as its contraction of the gradient wants them, and writes and reads
// the whole panel through LDS.
//
// What bounds it: one wave per SIMD from G = 6 or 7 on, so every wait shows.  G = 9: a
// wave lives 154,000 cycles, of which 795 matrix products take 51,000, other vector
// instructions 56,000, and waits (LDS, the gathers, results of the products and of
// the pivots' chains) the rest.
// n = 1e6, m = 120 (G = 9), value: 3.74 ms with the general kernel, 3.43 now.
// Simulator, 24 sets of n = 20,000, m = 150 (G = 10): 80.4 ms with the general
// kernel, 58.8 now (both with part of the tiles in scratch).
#pragma once
#include "wave_kernel.hpp"

namespace bv {

// Tile columns eliminated before the others are generated: 55 tiles (G = 10) exceed
// the register file, 45 do not, so the first column is factored alone and
// waits in LDS, and its updates are applied to every other tile as that is generated.
template <int G> constexpr int rows_deferred() { return G >= 10 ? 1 : 0; }
template <int G, bool COEF> constexpr int rows_min_waves() {
  // the most at which the weights keep nearly all tiles in registers (bytes of scratch per
  // lane: 100 at G = 5, 20, 412, 924 and 956 at G = 7 to 10, where one wave has all
  // registers already); the value has G >= 7 only (none, 12 at G = 10)
  return G <= 2 ? 4 : G <= 3 ? 3 : G <= 5 ? 2 : 1;
}
// LDS elements: coordinates, y, pivots, border row, the published columns, the first
// tile column, and for the weights the 4 x 4 inverses and one tile
template <int G, bool COEF> constexpr int rows_lds_elems() {
  return 6 * 16 * G + 64 + rows_deferred<G>() * G * 256 + (COEF ? 64 * G + 16 * 17 : 0);
}

template <int CTRL> __device__ __forceinline__ double dpp_row(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
// sum over the 16 lanes of equal lg, in every one of them
__device__ __forceinline__ double row_sum(double v) {
  v += dpp_row<0x128>(v);
  v += dpp_row<0x124>(v);
  v += dpp_row<0x122>(v);
  v += dpp_row<0x121>(v);
  return v;
}

template <int G, bool COEF>
__global__ void __launch_bounds__(64, (rows_min_waves<G, COEF>())) bv_rows_kernel(AdjArgs a, ThetaPack thp) {
  constexpr int P = 16 * G, DEF = rows_deferred<G>(), H = G - DEF;
  constexpr bool STAGED = rows_min_waves<G, COEF>() == 1;
  typedef WMma<double> M;
  typedef M::acc acc_t;
  extern __shared__ __align__(16) double rsm[];
  double* su = rsm;             // coordinates in units of range / log2(e) relative to the block's first point
  double* sy = su + 3 * P;      // y (weights: the solution)
  double* spiv = sy + P;        // pivots
  double* sw = spiv + P;        // border row of the factor
  double* spub = sw + P;        // four columns of a diagonal tile, [column][row]
  double* scol0 = spub + 64;    // factor tiles of column 0 as operands (deferred)
  double* sinv = scol0 + DEF * G * 256;   // weights: negated 4 x 4 inverses, by rows
  double* stile = sinv + 64 * G;          // weights: a diagonal tile, [row * 17 + column]
  const int ln = threadIdx.x, lr = ln & 15, lg = ln >> 4;
  const int total = a.list ? *a.list_count : a.nsched * a.ntheta;
  const int wi = blockIdx.x;
  if (wi >= total) return;
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
  const int brow = COEF ? m : p;   // the row whose factor entries are kept: y_J, or the point's own
  const double* org = a.locs + (size_t)b0 * a.d;
  {
    // all rows' indices before their points, all points before the first store (as
    // in the general kernel; rows past p read the block's first point)
    constexpr int NR = (P + 63) / 64;
    int gi[NR];
    double yv[NR], x[NR][3], og[3];
#pragma unroll
    for (int q = 0; q < NR; ++q) gi[q] = 0;
    if (m > 0) {
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const int i = ln + 64 * q;
        gi[q] = a.nbr_idx[n0 + (i < m ? i : m - 1)];
      }
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int i = ln + 64 * q;
      if (i >= m) gi[q] = i < p ? b0 + i - m : b0;
      yv[q] = COEF ? 0.0 : a.y[gi[q]];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      og[k] = k < a.d ? org[k] : 0.0;
#pragma unroll
      for (int q = 0; q < NR; ++q) x[q][k] = k < a.d ? a.locs[(size_t)gi[q] * a.d + k] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int i = ln + 64 * q;
      if (i < P) {
        sy[i] = i < p ? yv[q] : 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k)
          su[k * P + i] = i < p && k < a.d ? (x[q][k] - og[k]) * (th.inv_scale[k] * kLog2E) : 0.0;
      }
    }
  }
  wave_lds_sync();
  const MaternCoef<double> mc(th.nu_code);
  const double nug = th.nugget, ns0 = -th.sigma2, ns1 = ns0 * mc.c1 * kLn2, ns2 = ns0 * mc.c2 * kLn2 * kLn2;

  // ---- one tile of the bordered matrix; cj: its columns' coordinates ---------
  auto col_coords = [&](int J, double (&cj)[4][3]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int k = 0; k < 3; ++k) cj[r][k] = su[k * P + J * 16 + 4 * r + lg];
  };
  auto generate = [&](int I, int J, const double (&cj)[4][3]) __attribute__((always_inline)) {
    const int i = I * 16 + lr;
    const double si0 = su[i], si1 = su[P + i], si2 = su[2 * P + i];
    double dx[4], dy[4], dz[4], u[4];
    Exp2Parts e[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      dx[r] = si0 - cj[r][0];
      dy[r] = si1 - cj[r][1];
      dz[r] = si2 - cj[r][2];
    }
    distance_exp2neg4<STAGED>(dx, dy, dz, u, e);
    acc_t v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = MaternCoef<double>::neg_cov_log2(u[r], e[r], ns0, ns1, ns2);
    if (I == J) {
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] -= 4 * r + lg == lr ? nug : 0.0;
    }
    if (I >= (p >> 4)) {   // rows that hold no point: the border row p, identity after it
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = J * 16 + 4 * r + lg;
        const double id = i == j ? -1.0 : 0.0;
        const double rest = !COEF && ((i == p) & (j < p)) ? -sy[j] : id;
        v[r] = ((i < p) & (j < p)) ? v[r] : rest;
      }
    }
    return v;
  };

  // ---- four columns: Cholesky of the 4 x 4 block D (the same in every lane); the
  // operand that solves the rows: element (lr, lg) of its negated inverse, lr < 4 -----
  auto read_block = [&](int q, double (&D)[4][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j) D[i][j] = spub[j * 16 + 4 * q + i];
  };
  const int kreal = COEF ? m : p;   // columns with a factor (the point's own column only has a pivot)
  auto factor_block = [&](int k0, double (&D)[4][4]) __attribute__((always_inline)) {
    double rinv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int j = 0; j < k; ++j) D[k][k] = __builtin_fma(-D[k][j], D[k][j], D[k][k]);
      rinv[k] = k0 + k < kreal ? rsqrt_fast(D[k][k]) : 0.0;
#pragma unroll
      for (int i = k + 1; i < 4; ++i) {
#pragma unroll
        for (int j = 0; j < k; ++j) D[i][k] = __builtin_fma(-D[i][j], D[k][j], D[i][k]);
        D[i][k] *= rinv[k];
      }
    }
    double z[4];   // row lr & 3 of the negated inverse
#pragma unroll
    for (int c = 3; c >= 0; --c) {
      z[c] = (lr & 3) == c ? -1.0 : 0.0;
#pragma unroll
      for (int j = c + 1; j < 4; ++j) z[c] = __builtin_fma(-z[j], D[j][c], z[c]);
      z[c] *= rinv[c];
    }
    if (ln == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) spiv[k0 + k] = D[k][k];
    }
    const double lo = lg & 1 ? z[1] : z[0], hi = lg & 1 ? z[3] : z[2];
    const double op = lr < 4 ? (lg & 2 ? hi : lo) : 0.0;
    if (COEF && lr < 4) sinv[4 * k0 + 4 * lr + lg] = op;
    return op;
  };
  // tile column K: c(I) its tiles, update(v, q) the tiles right of it
  const acc_t zero = {0.0, 0.0, 0.0, 0.0};
  auto eliminate = [&](auto K_c, auto&& c, auto&& update) __attribute__((always_inline)) {
    BV_CV(K);
    double D[4][4];
    wave_lds_sync();
    spub[ln] = -c(K_c)[0];
    wave_lds_sync();
    read_block(0, D);
    static_for<0, 4>(BV_CI(q) {
      BV_CV(q);
      const double op = factor_block(K * 16 + 4 * q, D);
      double v[G];
      static_for<K, G>(BV_CI(I) {
        BV_CV(I);
        v[I] = M::op(op, c(I_c)[q], zero)[0];
      });
      v[K] = lr >= 4 * q + lg ? v[K] : 0.0;
      if constexpr (q < 3) {
        // the diagonal tile first: its next four columns go to LDS and come back
        // while the other tiles are updated
        c(K_c) = M::op(v[K], v[K], c(K_c));
        wave_lds_sync();
        spub[ln] = -c(K_c)[q + 1];
        wave_lds_sync();
        read_block(q + 1, D);
        static_for<K + 1, G>(BV_CI(I) {
          BV_CV(I);
          c(I_c) = M::op(v[K], v[I], c(I_c));
        });
      }
      static_for<K, G>(BV_CI(I) {   // the border row's entries
        BV_CV(I);
        if (I == (brow >> 4) && lr == (brow & 15)) sw[K * 16 + 4 * q + lg] = v[I];
      });
      update(v, q_c);
    });
  };

  acc_t acc[H * (H + 1) / 2];
  // weights: the finished columns, as operands (values of their own: as elements of
  // the tiles they kept all eight registers of each tile together and spilled)
  double fin[COEF ? H * (H + 1) / 2 : 1][4];
  auto tx = [](int I, int J) constexpr { return (I - DEF) * (I - DEF + 1) / 2 + J - DEF; };
  if constexpr (DEF == 1) {
    acc_t c0[G];
    double cj[4][3];
    col_coords(0, cj);
    static_for<0, G>(BV_CI(I) {
      BV_CV(I);
      c0[I] = generate(I, 0, cj);
      __builtin_amdgcn_sched_barrier(0);
    });
    eliminate(std::integral_constant<int, 0>{},
              [&](auto I_c) __attribute__((always_inline)) -> acc_t& { return c0[decltype(I_c)::value]; },
              [&](const double (&v)[G], auto q_c) __attribute__((always_inline)) {
                static_for<0, G>(BV_CI(I) {
                  BV_CV(I);
                  scol0[I * 256 + decltype(q_c)::value * 64 + ln] = v[I];
                });
              });
    wave_lds_sync();
  }
  static_for<DEF, G>(BV_CI(J) {
    BV_CV(J);
    double cj[4][3];
    col_coords(J, cj);
    static_for<J, G>(BV_CI(I) {
      BV_CV(I);
      constexpr int t = tx(I, J);
      acc[t] = generate(I, J, cj);
      if constexpr (DEF == 1) {
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[t] = M::op(scol0[J * 256 + q * 64 + ln], scol0[I * 256 + q * 64 + ln], acc[t]);
      }
      // where the tiles outgrow the VGPRs the finished tile leaves them now
      if constexpr (STAGED && t < 32) asm volatile("" : "+a"(acc[t]));
      __builtin_amdgcn_sched_barrier(0);
    });
  });
  static_for<DEF, G>(BV_CI(K) {
    BV_CV(K);
    if (K * 16 >= p) return;
    eliminate(K_c,
              [&](auto I_c) __attribute__((always_inline)) -> acc_t& { return acc[tx(decltype(I_c)::value, K)]; },
              [&](const double (&v)[G], auto q_c) __attribute__((always_inline)) {
                static_for<K + 1, G>(BV_CI(I) {
                  BV_CV(I);
                  static_for<K + 1, I + 1>(BV_CI(J) {
                    BV_CV(J);
                    acc[tx(I, J)] = M::op(v[J], v[I], acc[tx(I, J)]);
                  });
                });
                if constexpr (COEF) {
                  static_for<K, G>(BV_CI(I) {
                    BV_CV(I);
                    double& f = fin[tx(I, K)][decltype(q_c)::value];
                    f = v[I];
                    if constexpr (STAGED) asm volatile("" : "+a"(f));
                  });
                }
              });
  });
  wave_lds_sync();

  const size_t o = (size_t)tt * a.bc + b;
  if constexpr (!COEF) {
    // ---- log-determinant, quadratic form and pivot guard ----------------------
    const double guard = a.fp32_guard == 2 ? INFINITY
        : a.fp32_guard ? fmax(0.5 * th.nugget, (double)p * 1.1920928955078125e-07 * (th.sigma2 + th.nugget))
        : 0.0;
    double acc_ll = 0.0;
    int flag = 0;
    for (int k = ln; k < p; k += 64) {
      const double dd = spiv[k];
      if (!(dd > guard)) flag |= a.fp32_guard ? 1 : 2;
      if (!(dd > 0.0)) flag |= 2;
      if (k >= m) acc_ll += log(dd) + sw[k] * sw[k];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      acc_ll += __shfl_down(acc_ll, off, 64);
      flag |= __shfl_down(flag, off, 64);
    }
    if (ln == 0) {
      a.partial[o] = (flag & 2) && !a.fp32_guard ? __builtin_nan("") : -0.5 * (acc_ll + (double)l * kLog2Pi);
      a.flag[o] = flag | a.flag_or;
    }
  } else {
    // ---- weights L_N^-T w, tile column by tile column from the last.  The rows
    // below contribute per lane (row lr, its four columns) and are summed over the
    // 16 lanes; inside the tile the contraction over rows is a product with the
    // transposed tile (through LDS), four rows at a time, after the 4 x 4 solve.
    // Rows from m on hold zeros.
    double* sx = sy;
    static_for_down<0, G>(BV_CI(K) {
      BV_CV(K);
      if (K * 16 >= m) {
        if (lg == 0) sx[K * 16 + lr] = 0.0;
        return;
      }
      auto tile = [&](auto I_c, int q) __attribute__((always_inline)) -> double {
        constexpr int I = decltype(I_c)::value;
        if constexpr (K < DEF) return scol0[I * 256 + q * 64 + ln];
        else return fin[tx(I, K < DEF ? DEF : K)][q];
      };
      wave_lds_sync();
#pragma unroll
      for (int q = 0; q < 4; ++q) stile[lr * 17 + 4 * q + lg] = tile(K_c, q);
      acc_t s;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        double v = 0.0;
        static_for<K + 1, G>(BV_CI(I) {
          BV_CV(I);
          v = __builtin_fma(tile(I_c, q), sx[I * 16 + lr], v);
          __builtin_amdgcn_sched_barrier(0);
        });
        const int c = K * 16 + 4 * q + lg;
        s[q] = c < m ? row_sum(v) - sw[c] : 0.0;
      }
      wave_lds_sync();
      double x[4];
      static_for_down<0, 4>(BV_CI(q) {
        BV_CV(q);
        const double it = lr < 4 ? sinv[64 * K + 16 * q + 4 * lg + (lr & 3)] : 0.0;
        x[q] = M::op(it, s[q], zero)[0];
        if (lr == 0) sx[K * 16 + 4 * q + lg] = x[q];
        if constexpr (q > 0) s = M::op(stile[(4 * q + lg) * 17 + lr], x[q], s);
        __builtin_amdgcn_sched_barrier(0);
      });
      wave_lds_sync();
    });
    wave_lds_sync();
    for (int j = ln; j < m; j += 64) a.coef[(size_t)tt * a.coef_stride + n0 + j] = sx[j];
    if (ln == 0) a.cvar[o] = spiv[m];
  }
}

template <int G, bool COEF>
static hipError_t launch_rows_g(const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  constexpr size_t lds = sizeof(double) * rows_lds_elems<G, COEF>();
  hipLaunchKernelGGL((bv_rows_kernel<G, COEF>), dim3(grid), dim3(64), lds, s, a, thp);
  return hipGetLastError();
}

}  // namespace bv
