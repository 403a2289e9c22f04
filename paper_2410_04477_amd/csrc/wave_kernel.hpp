// One-wave matrix-core kernels for the per-block chain of Alg. 1.
//
// A single wave (64 lanes, the whole workgroup) evaluates one block for one
// theta.  The bordered joint matrix [[K_J, .], [y_J^T, .]] (p + 1 rows, padded
// to P = 16 G with identity) lives in the wave's accumulator registers as the
// G (G + 1) / 2 lower-triangular 16 x 16 tiles of the v_mfma_*_16x16x4
// instructions; every lane generates its own Matern entries.  With the tile
// loops unrolled (G is a template parameter) every tile index is static, so
// the matrix never leaves the register file.
//
// Factorisation: right-looking Cholesky in panels of four columns.  Per panel,
// the lanes holding its columns write them to LDS; every lane factors the
// 4 x 4 diagonal block (all lanes compute the same values in lockstep, so the
// redundancy costs nothing); each lane solves up to ceil((P - 16 K) / 64)
// panel rows, or in FP64 forms the entries that its matrix-core operands need
// (the TRSM / TRSV of Alg. 1; the border row becomes
// w = L^-1 y_J); the trailing tiles take one rank-4 MFMA each (the Schur
// update).  What bounds it: matrix-core and vector operations of FP32 and FP64
// share the same units on gfx950 (a wave that alternates them takes the sum of
// their times), so a block costs its MFMA time plus its vector instructions,
// and at one wave per SIMD every wait as well.  FP64, n = 1e6, m = 120: value
// 4.68 -> 3.73 ms (3.43 with the kernel of wave_rows.hpp), prediction of 1e5 points
// 1.12 -> 0.76 ms; n = 1e5, m = 60: value and gradient 757 -> 490 us (square root,
// exponential and 1 / sqrt from the hardware estimates, masks only in the edge
// tiles, row panels, two waves per SIMD up to G = 5 or 6).  Lanes exchange panel data
// through LDS with wavefront-scope fences, so a panel costs no cross-wave synchronisation.  Pivots d_k and
// border entries w_k (k >= m) give log det and the quadratic form, summed in
// FP64.
//
// Adjoint: X = L^-T [ w | [z; 0] | [0; I_l] ] is pure MFMA work tile row by
// tile row, X_K <- inv(L_KK)^T X_K, then X_J -= L_KJ^T X_K for the rows above;
// W = alpha alpha^T - b b^T - X_R X_R^T is formed tile by tile with MFMA and
// contracted against dK regenerated entry by entry (FP64 across tiles):
// d l_i = 1/2 <W, dK>.  MODE 5 keeps the factor in the registers (the
// diagonal inverses formed during the factorisation from 16 rows appended to
// each panel) and takes its A operands from the accumulator registers;
// MODE 1 stores the factor tiles to the item's slot of a global tile buffer,
// inverts the diagonal blocks there (16 lanes per block, all blocks in one
// pass) and reads its A operands from the buffer; MODES 2 + 3 split the two
// halves over two launches, and MODES 6 + 3 likewise with a left-looking
// factorisation (FP64 above G = 9).
#pragma once

#include <utility>

#include "internal.hpp"

namespace bv {

// Compile-time loops: the body receives std::integral_constant<int, i>, so
// accumulator tile indices are constants whatever the unroller decides.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}
template <int B, int E, typename F>  // E - 1 down to B
__device__ __forceinline__ void static_for_down(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, E - 1>{});
    static_for_down<B, E - 1>(f);
  }
}
#define BV_CI(name) [&](auto name##_c) __attribute__((always_inline))
#define BV_CV(name) constexpr int name = decltype(name##_c)::value

typedef float w32x4_t __attribute__((ext_vector_type(4)));
typedef double w64x4_t __attribute__((ext_vector_type(4)));

template <typename T> struct WMma;
template <> struct WMma<float> {
  typedef w32x4_t acc;
  static __device__ __forceinline__ acc op(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // tile row held by accumulator register r of lane group g
  static __device__ __forceinline__ constexpr int row(int g, int r) { return 4 * g + r; }
  static __device__ __forceinline__ float rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
  // position, inside a tile stored in accumulator order (lane * 4 + register),
  // of element (4 s + l / 16, l % 16): the A operand of lane l for k-step s
  // when the stored tile is used transposed
  static __device__ __forceinline__ constexpr int aop(int l, int s) { return ((l & 15) + 16 * s) * 4 + (l >> 4); }
  // position of element (i, j) of a tile stored in accumulator order
  static __device__ __forceinline__ constexpr int at(int i, int j) { return (j + 16 * (i >> 2)) * 4 + (i & 3); }
};
template <> struct WMma<double> {
  typedef w64x4_t acc;
  static __device__ __forceinline__ acc op(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ constexpr int row(int g, int r) { return g + 4 * r; }
  static __device__ __forceinline__ double rsqrt(double x) { return rsqrt_fast(x); }
  static __device__ __forceinline__ constexpr int aop(int l, int s) { return l * 4 + s; }
  static __device__ __forceinline__ constexpr int at(int i, int j) { return (j + 16 * (i & 3)) * 4 + (i >> 2); }
};

// lower-triangular tile (I, J), J <= I, in row-major packed order
__host__ __device__ constexpr int tix(int I, int J) { return I * (I + 1) / 2 + J; }

constexpr int kStageStride = 260;   // staged 16 x 16 tiles, padded so tiles four apart fall in different banks

__host__ __device__ constexpr int wave_max(int x, int y) { return x > y ? x : y; }

// The kernels below run one wave per workgroup, and a wave's LDS operations
// are performed in issue order, so lanes exchange data through LDS with a
// wavefront-scope fence (it keeps the compiler from moving LDS accesses across
// it) and no wait for the LDS traffic.  Exchanges through global memory (the
// tile buffer of mode 1, the stored tile columns of mode 6) keep the workgroup
// barrier.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// elements of the panel: four columns of P rows; in the modes that form the diagonal
// inverses during the factorisation also 16 appended rows, and the panel is the
// scratch of a 16 x 16 transposition too (which exceeds four columns up to G = 2)
__host__ __device__ constexpr int wave_panel(int G, bool einv) {
  return einv ? wave_max(4 * (16 * G + 16), 256) : 4 * 16 * G;
}
__host__ __device__ constexpr int wave_lds_elems(int G, int mode) {
  // su (3 P) for the whole kernel, then a work region: the panel and sy, sdk, swk
  // (P each) during the factorisation; for the adjoint, one chunk of right-hand sides
  // (P x (wave_chunk(G) + 1), plus 32 elements that reads of the last row's
  // unused columns may touch), which also holds the G staged diagonal tiles
  // before the first chunk
  // (mode 5 keeps the border row w of the factor after that, 16 G elements)
  return 3 * 16 * G + wave_max(wave_panel(G, mode == 2 || mode == 5 || mode == 6) + 3 * 16 * G,
                               mode == 0 || mode == 2 || mode == 4 || mode == 6 ? 0
                               : (16 * (wave_chunk(G) + 1) > kStageStride
                                      ? 16 * G * (wave_chunk(G) + 1) + 32
                                      : G * kStageStride)) +
         (mode == 5 ? 16 * G : 0);
}

// bytes before the Bessel form's table in the LDS
__host__ __device__ constexpr int wave_table_offset(int elem, int G, int mode) {
  return (elem * wave_lds_elems(G, mode) + 15) / 16 * 16;
}

// Waves per SIMD that a kernel's registers have to allow (512 per lane and SIMD).
// A wave's matrix-core and vector instructions share the FP32 / FP64 units (one
// wave that mixes them takes the sum of their times), so more waves only hide
// latency; two already do, and the first bound below that keeps every tile in
// registers is taken.  FP64 (8 registers a tile and lane): value and prediction
// kernels 4, 3 and 2 waves up to G = 2, 4, 6; the one-launch gradient, whose
// contraction holds more beside the tiles, 2 up to G = 5 (n = 1e5, m = 60 value and
// gradient: 631 us with one wave per SIMD).  FP32: 5 up to G = 5 (96 registers).
template <typename T, int G, int MODE, bool GEN>
constexpr int wave_min_waves() {
  if (MODE == 6) return 2;
  if (sizeof(T) == 8) {
    if (MODE == 1 || MODE == 3) return 1;
    // Bessel form: the call's own registers, so two waves where the tiles leave room without scratch
    if (GEN) return G <= 3 || (G == 4 && MODE != 5) ? 2 : 1;
    if (MODE == 5) return G <= 5 ? 2 : 1;
    return G <= 2 ? 4 : G <= 4 ? 3 : G <= 6 ? 2 : 1;
  }
  if (MODE == 0 && G <= 5) return 5;
  return G <= 9 || MODE == 3 ? 2 : 1;
}

// Modes: 0 value; 1 value and gradient in one launch; 2 value and the factor
// tiles to the tile buffer; 3 gradient from those tiles (a second launch that
// holds no tiles in registers, so it runs more waves per SIMD than mode 1);
// 4 prediction (Alg. 2): the block rows are new locations, the border row
// carries y_N and zeros, and only the neighbour columns are eliminated, which
// leaves the Schur complement -- the conditional covariance of the block and,
// in the border row, minus its conditional mean -- in the trailing tiles.
// 5 value and gradient in one launch with the factor kept in the registers
// through the back-substitution (no tile buffer; right-hand sides in passes
// of wave_chunk(G), at G = 9 one pass only: l + 2 <= wave_chunk(G)).
// 6 value and the factor tiles to the tile buffer, as mode 2, but left-looking
// by tile columns: a tile column is generated when its turn comes, updated
// with the stored columns to its left (MFMA, operands read back from the
// buffer), factored in its four panels and stored, so that only one tile
// column is in the registers at a time (FP64 classes above G = 9, whose tiles
// exceed the register file); mode 3 takes the adjoint from its tiles.
// (The FP64 value above G = 6 and the simulator's weights have a kernel of their
// own, wave_rows.hpp.)
// GEN: covariances by the Bessel form for any nu instead of the closed forms.
template <typename T, int G, int MODE, bool GEN>
__global__ void __launch_bounds__(64, (wave_min_waves<T, G, MODE, GEN>())) bv_wave_kernel(AdjArgs a, ThetaPack thp) {
  constexpr int P = 16 * G;
  constexpr int NT = G * (G + 1) / 2;
  typedef WMma<T> M;
  typedef typename M::acc acc_t;
  extern __shared__ __align__(16) unsigned char smem[];
  T* su = reinterpret_cast<T*>(smem);  // scaled coordinates relative to the block's first point, su[k * P + i]
  // closed forms: the coordinates carry a factor log2(e), so e^-x is the exp2 of
  // the distance (one instruction in FP32, no argument reduction by ln 2 in FP64)
  // and the polynomial coefficients carry powers of ln 2
  constexpr double UNIT = GEN ? 1.0 : kLog2E;
  // The FP64 gradient at G = 9 (45 tiles, 360 registers, with the right-hand sides'
  // working set) fits the registers without scratch only with masks instead of
  // branches in the generation, the panel kept by columns and one nest of updates.
  // The value at G = 11 and the prediction from G = 10 on (Bessel form: 11) exceed them
  // either way, and spill less so: 3,000 blocks, value at G = 11 610 us by rows
  // (with 752 bytes of scratch), 464 so (612; 521 before the row panels); prediction at
  // G = 11 766 and 563 us (1,220 and 868), at G = 10 387 and 325 us (612 and 356), but
  // at G = 9 224 and 256 us.
  constexpr bool TIGHT = sizeof(T) == 8 && ((MODE == 5 && G == 9) || ((MODE == 0 || MODE == 4) && G >= (GEN ? 11 : 10)));
  constexpr bool STAGED = wave_min_waves<T, G, MODE, GEN>() == 1;
  T* work = su + 3 * P;
  // MODE 5 appends 16 rows to the panel (the identity rows whose elimination
  // gives the inverse of each diagonal tile of the factor)
  constexpr bool LEFT = MODE == 6;                // left-looking by tile columns
  constexpr bool INREG = MODE == 5;                // factor kept in the registers
  constexpr bool EINV = INREG || MODE == 2 || LEFT;   // diagonal inverses formed during the factorisation
  constexpr int PS = EINV ? P + 16 : P;            // panel column stride
  constexpr int PANEL = wave_panel(G, EINV);
  static_assert(3 * P + PANEL + 3 * P <= wave_lds_elems(G, MODE), "factorisation LDS");
  T* sy = work + PANEL;                // border row y_J
  T* sdk = sy + P;                     // pivots d_k
  T* swk = sdk + P;                    // border entries w_k

  const int ln = threadIdx.x, lr = ln & 15, lg = ln >> 4;
  const int total = a.list ? *a.list_count : a.nsched * a.ntheta;
  const int wi = blockIdx.x + a.item_base;
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
  const int l = b1 - b0, m = n1 - n0;
  // prediction pads the neighbour rows with identity up to a panel boundary
  const int mq = MODE == 4 ? pred_rows(m) : m;
  const int p = mq + l;
  // rows that hold a point (the rest of the P rows are identity padding)
  // (no short circuits: as branches they made the compiler drop a mask of gen_tile)
  auto real_row = [&](int i) __attribute__((always_inline)) {
    return (int)(i < p) & ((int)(MODE != 4) | (int)(i < m) | (int)(i >= mq));
  };
  if (MODE == 4 && l == 0) return;
  const double* org = (MODE == 4 ? a.locs2 : a.locs) + (size_t)b0 * a.d;   // coordinate origin: the block's first point

  // All rows' indices are read before any of their points, and all points before
  // any is stored (rows that hold none read the block's first point or the last
  // neighbour): the wave waits for two loads in turn whatever its rows, not two
  // per 64 rows (FP32 value and gradient at n = 1e6 3.10 -> 3.02 ms, prediction at
  // n = 1e5 770 -> 751 us).  With three and more waves per SIMD the others cover
  // it, and 64 rows at a time need fewer registers; mode 6 has none to spare either
  // (left to itself the loop costs it scratch at G = 10, rolled at G = 11).
  constexpr int NR = wave_min_waves<T, G, MODE, GEN>() <= 2 && MODE != 6 ? (P + 63) / 64 : 1;
  constexpr int ROLL = MODE == 6 && G == 10 ? 1 : (P + 63) / 64;
#pragma unroll ROLL
  for (int row0 = 0; row0 < P; row0 += 64 * NR) {
    int gi[NR];
    T yv[NR];
    double x[NR][3];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      gi[q] = 0;
      yv[q] = T(0);
    }
    if (m > 0) {
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const int i = row0 + ln + 64 * q;
        gi[q] = a.nbr_idx[n0 + (i < m ? i : m - 1)];
      }
    }
    if (MODE == 4 && m > 0) {   // the border row is [y_N, 0]
#pragma unroll
      for (int q = 0; q < NR; ++q) yv[q] = T(a.y[gi[q]]);
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int i = row0 + ln + 64 * q;
      if (i >= m) gi[q] = i >= mq && i < p ? b0 + i - mq : b0;
    }
    if (MODE != 3 && MODE != 4) {
#pragma unroll
      for (int q = 0; q < NR; ++q) yv[q] = T(a.y[gi[q]]);
    }
    double og[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      og[k] = 0.0;
      if (k < a.d) {
        og[k] = org[k];
#pragma unroll
        for (int q = 0; q < NR; ++q)
          x[q][k] = (MODE == 4 && row0 + ln + 64 * q >= m ? a.locs2 : a.locs)[(size_t)gi[q] * a.d + k];
      } else {
#pragma unroll
        for (int q = 0; q < NR; ++q) x[q][k] = 0.0;
      }
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int i = row0 + ln + 64 * q;
      if (i < P) {
        const bool real = real_row(i);
        if (MODE != 3) sy[i] = real && (MODE != 4 || i < m) ? yv[q] : T(0);
#pragma unroll
        for (int k = 0; k < 3; ++k)
          su[k * P + i] = real && k < a.d ? T((x[q][k] - og[k]) * (th.inv_scale[k] * UNIT)) : T(0);
      }
    }
  }
  wave_lds_sync();
  const size_t o = (size_t)tt * a.bc + b;
  // tile slot (MODE 1-3, 6): the NT factor tiles (MODES 2, 6: the diagonal
  // ones replaced by their inverses), then the border row w (16 G elements)
  constexpr int SLOT = NT * 256 + 16 * G;
  T* Lg = reinterpret_cast<T*>(a.tiles) + (size_t)(wi - a.item_base) * SLOT;
  double acc_ll = 0.0;
  int flag = 0;
  const MaternCoef<T> mc(th.nu_code);   // closed forms
  // Bessel form, FP64: the table of this order, after the rest of the LDS.  (FP32
  // rounds the FP64 function; it keeps the function by single distances, whose last
  // bits differ, as a changed rounding of one covariance moves the FP32 results.)
  constexpr bool BES4 = GEN && sizeof(T) == 8;
  double* const table = reinterpret_cast<double*>(smem + wave_table_offset(sizeof(T), G, MODE));
  LdsDouble* const btab = (LdsDouble*)table;
  if constexpr (BES4) {
    bessel_table(table, th.bes, ln);
    wave_lds_sync();
  }
  acc_t acc[NT];   // the bordered matrix, then its factor (unused by MODE 3)
  if constexpr (MODE != 3) {   // MODE 3 starts from the factor tiles of a MODE 2 or 6 launch

  // ---- generate the bordered joint matrix in the accumulator tiles ----------
  const T sig2 = T(th.sigma2), nug = T(th.nugget);
  // closed forms: -sigma2 (1 + c1 x + c2 x^2) e^-x with the scale and sign in
  // the coefficients
  T ns0 = T(0), ns1 = T(0), ns2 = T(0);
  if constexpr (!GEN) {
    ns0 = -sig2;
    ns1 = T(-th.sigma2 * (double)mc.c1 * kLn2);
    ns2 = T(-th.sigma2 * (double)mc.c2 * kLn2 * kLn2);
  }
  // tile row I's coordinates (row M::row(lg, r) of the tile in ri[r]) and the
  // generation of one tile
  auto row_coords = [&](int I, T (&ri)[4][3]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = I * 16 + M::row(lg, r);
      ri[r][0] = su[i];
      ri[r][1] = su[P + i];
      ri[r][2] = su[2 * P + i];
    }
  };
  auto gen_tile = [&](auto I_c, auto J_c, const T (&ri)[4][3]) __attribute__((always_inline)) {
    constexpr int I = decltype(I_c)::value, J = decltype(J_c)::value;
    const int j = J * 16 + lr;
    const T sj0 = su[j], sj1 = su[P + j], sj2 = su[2 * P + j];
    T dx[4], dy[4], dz[4], u[4];
    typename ExpOf<T>::type e[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      dx[r] = ri[r][0] - sj0;
      dy[r] = ri[r][1] - sj1;
      dz[r] = ri[r][2] - sj2;
    }
    BesselOut bes;
    if constexpr (!GEN) {
      distance_exp2neg4<STAGED>(dx, dy, dz, u, e);
    } else if constexpr (!BES4) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double rho, g;
        matern_general((double)distance<T>(dx[r], dy[r], dz[r]), th.bes, &rho, &g);
        bes[r] = rho;
      }
    } else {
      Bessel4 x;
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = (double)distance<T>(dx[r], dy[r], dz[r]);
      bes = bessel4<0>(x, btab);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // the tiles hold the negated matrix (updates add L L^T)
      T v;
      if constexpr (GEN) v = -(sig2 * T(bes[r]));
      else v = mc.neg_cov_log2(u[r], e[r], ns0, ns1, ns2);
      if constexpr (I == J) v -= (M::row(lg, r) == lr) ? nug : T(0);   // the nugget: same-index pairs only
      acc[tix(I, J)][r] = v;
    }
    // Rows and columns that hold no point: only the tile rows from p on (and,
    // for prediction, the tiles of the padding between neighbours and block)
    // have any, so the others skip the masks (a wave-uniform branch).
    if (TIGHT || I >= (p >> 4) || (MODE == 4 && (I == (m >> 4) || J == (m >> 4)))) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = I * 16 + M::row(lg, r);
        const T v = acc[tix(I, J)][r];
        acc[tix(I, J)][r] = real_row(i) & real_row(j) ? v : (i == j) ? T(-1) : T(0);
      }
      if (I == (p >> 4)) {  // border row p: y_J
        const T yb = sy[j];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const T v = acc[tix(I, J)][r];
          acc[tix(I, J)][r] = (int)(I * 16 + M::row(lg, r) == p) & (int)(j < p) ? -yb : v;
        }
      }
    }
    // Where the tiles outgrow the VGPRs the finished tile goes to the accumulator
    // registers now, so that the generated values do not pile up until the first
    // update: by D = 0 * 0 + C.  (Asking for the move itself is cheaper, but where other
    // tiles are in scratch the compiler lost tiles asked for like this: with the
    // calls of the Bessel form, and at G = 11.)
    constexpr bool ONE = sizeof(T) == 8 && wave_min_waves<T, G, MODE, GEN>() == 1;
    if constexpr (sizeof(T) == 8 ? ONE || (LEFT && G == 10) : !(G <= 9 && (MODE == 5 || MODE == 2))) {
      acc[tix(I, J)] = M::op(T(0), T(0), acc[tix(I, J)]);
    }
  };
  if constexpr (!LEFT) {   // the whole matrix now (mode 6: a tile column at a time)
    static_for<0, G>(BV_CI(I) {
      T ri[4][3];
      row_coords(decltype(I_c)::value, ri);
      static_for<0, decltype(I_c)::value + 1>(BV_CI(J) { gen_tile(I_c, J_c, ri); });
    });
  }

  // ---- factorisation, four columns per step -----------------------------------
  T* pan = work;  // pan[c * PS + row], c < 4
  // MODES 5, 2 and 6: the 16 rows appended below the matrix while tile column K is
  // eliminated, R = e_j^T at column 16 K + j (zero left of the tile column,
  // so earlier columns leave them untouched).  After the tile column they hold
  // R L_KK^-T = L_KK^-T, and the transpose of that, inv(L_KK), replaces L_KK
  // in the tiles (nothing in the factorisation reads L_KK afterwards).  Held
  // negated like the matrix tiles.
  acc_t einv;
  // columns c0 .. c0 + 3 of tile column Kc to the panel
  auto publish = [&](auto Kc_c, int c0) __attribute__((always_inline)) {
    constexpr int Kc = decltype(Kc_c)::value;
    if (lr >= c0 && lr < c0 + 4) {
      static_for<Kc, G>(BV_CI(I) {
        BV_CV(I);
#pragma unroll
        for (int r = 0; r < 4; ++r) pan[(lr - c0) * PS + I * 16 + M::row(lg, r)] = acc[tix(I, Kc)][r];
      });
      if (EINV) {
#pragma unroll
        for (int r = 0; r < 4; ++r) pan[(lr - c0) * PS + P + M::row(lg, r)] = einv[r];
      }
    }
  };
  // the panel at column k0: 4 x 4 diagonal block (same values in every lane),
  // then its rows from the diagonal tile down (zero above the block, L_dd in
  // it, TRSM below); pivots and border entries to LDS
  auto factor_panel = [&](auto Kf_c, int k0) __attribute__((always_inline)) {
    constexpr int i0 = 16 * decltype(Kf_c)::value;
    T Ld[4][4], rinv[4], piv[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) Ld[r][c] = r >= c ? -pan[c * PS + k0 + r] : T(0);   // panel holds -A
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      // (columns at and beyond p come out as whatever the border row makes of
      // them; the pass below sets them to identity)
      T dsum = Ld[c][c];
#pragma unroll
      for (int j = 0; j < c; ++j) dsum -= Ld[c][j] * Ld[c][j];
      piv[c] = dsum;
      const T ri = M::rsqrt(dsum);
      rinv[c] = ri;
      Ld[c][c] = dsum * ri;
#pragma unroll
      for (int r = c + 1; r < 4; ++r) {
        T v = Ld[r][c];
#pragma unroll
        for (int j = 0; j < c; ++j) v -= Ld[r][j] * Ld[c][j];
        Ld[r][c] = v * ri;
      }
    }
    constexpr int NCH = (PS - i0 + 63) / 64;   // 64-row chunks of the panel
    // every chunk's entries are read before any is used (the row index is
    // clamped into the panel; the clamped lanes store nothing)
    T pv[NCH][4];
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      const int i = i0 + ln + 64 * q;
      const int ic = i < PS ? i : PS - 1;
#pragma unroll
      for (int c = 0; c < 4; ++c) pv[q][c] = pan[c * PS + ic];
    }
    // every lane runs the substitution, which also yields the rows of the
    // diagonal block up to their diagonal (the operations that formed Ld); right
    // of the diagonal there, and above the block, is zero.  Only the first chunk
    // holds such rows (i0 + 64 > k0 + 3).  An appended row j stands for column
    // i0 + j.  FP64 takes all chunks in step (independent chains: a dependent
    // operation waits as long as two issue), FP32 one after the other (fewer
    // registers; its dependent operations do not wait).
    constexpr int QB = sizeof(T) == 8 && !TIGHT ? NCH : 1;
#pragma unroll
    for (int q0 = 0; q0 < NCH; q0 += QB) {
      T x[QB][4];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int q = 0; q < QB; ++q) {
          const int i = i0 + ln + 64 * (q0 + q);
          T v = -pv[q0 + q][c];
#pragma unroll
          for (int j = 0; j < c; ++j) v -= x[q][j] * Ld[c][j];
          x[q][c] = v * rinv[c];
          if (q0 + q == 0) x[q][c] = (i < P ? i : i0 + (i - P)) - k0 < c && i < P ? T(0) : x[q][c];
        }
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const int i = i0 + ln + 64 * (q0 + q);
        if (i < PS) {
#pragma unroll
          for (int c = 0; c < 4; ++c) pan[c * PS + i] = x[q][c];
          if (i == p) {
#pragma unroll
            for (int c = 0; c < 4; ++c) swk[k0 + c] = x[q][c];
          }
        }
      }
    }
    if (k0 + 4 > p) {
      // the panel holds padding columns (at and beyond p, the last ones): they
      // become identity columns.  What the substitution wrote there fed only
      // later columns of the panel, which are padding too.
#pragma unroll
      for (int q = 0; q < NCH; ++q) {
        const int i = i0 + ln + 64 * q;
        if (i < PS) {
          const int di = (i < P ? i : i0 + (i - P)) - k0;
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (k0 + c >= p) pan[c * PS + i] = di == c ? T(1) : T(0);
        }
      }
    }
    if (ln == 0) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        sdk[k0 + c] = piv[c];
      }
    }
  };

  const int kend = MODE == 4 ? mq : p;   // columns to eliminate
  auto init_einv = [&](auto K_c) __attribute__((always_inline)) {
    BV_CV(K);
    // -e_j for the columns the loop below eliminates; columns it skips (at
    // and beyond kend: the border column and the padding) keep +e_j, the
    // identity of the inverse there
#pragma unroll
    for (int r = 0; r < 4; ++r)
      einv[r] = M::row(lg, r) == lr ? (K * 16 + lr < kend ? T(-1) : T(1)) : T(0);
  };
  // inv(L_KK) = (L_KK^-T)^T into the diagonal tile, transposed through LDS
  auto finish_einv = [&](auto K_c) __attribute__((always_inline)) {
    BV_CV(K);
#pragma unroll
    for (int r = 0; r < 4; ++r) pan[lr * 16 + M::row(lg, r)] = einv[r];
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[tix(K, K)][r] = pan[M::row(lg, r) * 16 + lr];
    wave_lds_sync();
  };
  // FP64 (ROWPAN): the panel is kept by rows, pan[row * 4 + c], and its rows are
  // solved where the matrix instructions want them.  Lane (lr, lg) needs column lg
  // of L for row lr of each row tile: it forms row lg of the inverse of the 4 x 4
  // block, z, once per panel (10 operations) and v[I] = sum_c A[row][c] z[c], 4
  // products per row tile.  The substitution by rows costs fewer operations but
  // needs its results written to LDS and read back in this layout, one more
  // exchange in each panel's chain of dependent steps.  Products with the inverse add
  // about 10 % to the rounding error of a block; up to G = 3, where that is the largest
  // part of it and a panel has one or two row tiles, each lane substitutes along its row
  // instead and keeps one of the four results (SUBST).  Per-block error against 80 bits,
  // products / substitution: joint sizes to 33 3.8e-14 / 3.35e-14, to 48 4.6e-14 / 4.1e-14
  // (nu = 1/2, noise gradient: 3.1e-14 / 2.3e-14).  It costs 1 to 8 %: 12,000 blocks of 8
  // points and 26 neighbours, value 70.6 / 74.3 us, with the gradient 173 / 178,
  // prediction 59 / 63; at 2,000 points 17.8 us either way.
  constexpr bool ROWPAN = sizeof(T) == 8 && !LEFT && !TIGHT;
  constexpr bool SUBST = G <= 3;
  auto publish_rows = [&](auto Kc_c, int c0) __attribute__((always_inline)) {
    constexpr int Kc = decltype(Kc_c)::value;
    if (lr >= c0 && lr < c0 + 4) {
      static_for<Kc, G>(BV_CI(I) {
        BV_CV(I);
#pragma unroll
        for (int r = 0; r < 4; ++r) pan[(I * 16 + M::row(lg, r)) * 4 + lr - c0] = acc[tix(I, Kc)][r];
        __builtin_amdgcn_sched_barrier(0);   // one tile's copies at a time in the VGPRs
      });
      if (EINV) {
#pragma unroll
        for (int r = 0; r < 4; ++r) pan[(P + M::row(lg, r)) * 4 + lr - c0] = einv[r];
      }
    }
  };
  // lower part of the 4 x 4 block at column k0 of the published panel (-A)
  auto read_block = [&](int k0, T (&D)[4][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c <= r; ++c) D[r][c] = pan[(k0 + r) * 4 + c];
  };
  // Cholesky of the block (same values in every lane), pivots to LDS; z = -(row
  // lg of the inverse), the sign for the panel's -A; SUBST: z = 1 / (the factor's diagonal)
  auto factor_block = [&](int k0, T (&D)[4][4], T (&z)[4]) __attribute__((always_inline)) {
    if (k0 + 4 > p) {   // columns at and beyond p: identity
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c <= r; ++c)
          if (k0 + r >= p) D[r][c] = r == c ? T(-1) : T(0);
    }
    T piv[4], rinv[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int j = 0; j < c; ++j) D[c][c] += D[c][j] * D[c][j];
      piv[c] = -D[c][c];
      rinv[c] = M::rsqrt(piv[c]);
#pragma unroll
      for (int r = c + 1; r < 4; ++r) {
#pragma unroll
        for (int j = 0; j < c; ++j) D[r][c] += D[r][j] * D[c][j];
        D[r][c] = -D[r][c] * rinv[c];
      }
    }
    if constexpr (SUBST) {
#pragma unroll
      for (int c = 0; c < 4; ++c) z[c] = rinv[c];
    } else {
#pragma unroll
      for (int c = 3; c >= 0; --c) {
        T v = lg == c ? T(-1) : T(0);
#pragma unroll
        for (int j = c + 1; j < 4; ++j) v -= z[j] * D[j][c];
        z[c] = v * rinv[c];
      }
    }
    if (ln == 0) {
#pragma unroll
      for (int c = 0; c < 4; ++c) sdk[k0 + c] = piv[c];
    }
  };
  // v[I] (and ve, the appended rows) of the published panel; border entries to LDS
  auto solve_rows = [&](auto K_c, int k0, const T (&D)[4][4], const T (&z)[4], T (&v)[G], T& ve) __attribute__((always_inline)) {
    BV_CV(K);
    // the next row tile's entries are read before the current one's products
    // (no more: the scheduler would read all of them first and spill)
    T cur[4], nxt[4];
    auto fetch = [&](int row, T (&d)[4]) __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < 4; ++c) d[c] = pan[row * 4 + c];
    };
    auto solved = [&]() __attribute__((always_inline)) {   // entry lg of the solved row, from its published entries cur
      if constexpr (SUBST) {
        T x[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          x[c] = -cur[c];
#pragma unroll
          for (int j = 0; j < c; ++j) x[c] -= x[j] * D[c][j];
          x[c] *= z[c];
        }
        const T lo = lg & 1 ? x[1] : x[0], hi = lg & 1 ? x[3] : x[2];
        return lg & 2 ? hi : lo;
      } else {
        return cur[0] * z[0] + cur[1] * z[1] + (cur[2] * z[2] + cur[3] * z[3]);
      }
    };
    fetch(16 * K + lr, cur);
    static_for<K, G + (EINV ? 1 : 0)>(BV_CI(I) {
      BV_CV(I);
      if constexpr (I + 1 < G + (EINV ? 1 : 0)) fetch((I + 1) * 16 + lr, nxt);
      if constexpr (I < G) v[I] = solved();
      else ve = solved();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < 4; ++c) cur[c] = nxt[c];
    });
    // above the block, and right of the diagonal in it, L is zero (columns at and
    // beyond p have entries in rows from p on only, which nothing reads)
    if (lr < k0 - 16 * K + lg) v[K] = T(0);
    // the border row's entries of the four columns
    fetch(p, cur);
    const T w = solved();
    if (lr == 0) swk[k0 + lg] = w;
  };

  static_for<0, G>(BV_CI(K) {
    BV_CV(K);
    if (K * 16 >= kend) return;
    if constexpr (LEFT) {
      // tile column K: generated now, then updated with the stored columns to
      // its left, C_IK += L_IJ L_KJ^T (J < K, 16-wide contractions as four
      // k-steps; both operands take element (lane % 16, 4 s + lane / 16) of
      // their stored tile)
      static_for<K, G>(BV_CI(I) {
        BV_CV(I);
        T ri[4][3];
        row_coords(I, ri);
        gen_tile(std::integral_constant<int, I>{}, std::integral_constant<int, K>{}, ri);
      });
      for (int Jp = 0; Jp < K; ++Jp) {
        const T* LK = Lg + (size_t)(K * (K + 1) / 2 + Jp) * 256;
        T bq[4];
#pragma unroll
        for (int sq = 0; sq < 4; ++sq) bq[sq] = LK[M::at(lr, 4 * sq + lg)];
        static_for<K, G>(BV_CI(I) {
          BV_CV(I);
          const T* LI = Lg + (size_t)(I * (I + 1) / 2 + Jp) * 256;
          T aq[4];
#pragma unroll
          for (int sq = 0; sq < 4; ++sq) aq[sq] = LI[M::at(lr, 4 * sq + lg)];
#pragma unroll
          for (int sq = 0; sq < 4; ++sq) acc[tix(I, K)] = M::op(aq[sq], bq[sq], acc[tix(I, K)]);
        });
      }
    }
    if constexpr (EINV && !ROWPAN) init_einv(K_c);
    if constexpr (ROWPAN) {
      // One step per panel: its rows are solved, then tile column K (which holds the
      // next panel) takes the rank-4 update and the next panel is published and its
      // block read before the update of the other tiles is issued, which covers
      // the LDS exchange.
      constexpr bool KEEP = MODE != 0 && MODE != 4;   // the finished columns stay in the tiles
      T D[4][4];
      if constexpr (EINV) init_einv(K_c);
      publish_rows(K_c, 0);
      wave_lds_sync();
      read_block(K * 16, D);
#pragma nounroll
      for (int c0 = 0;; c0 += 4) {
        const int k0 = K * 16 + c0;
        T z[4], v[G], ve = T(0);
        factor_block(k0, D, z);
        solve_rows(K_c, k0, D, z, v, ve);
        const bool next = c0 + 4 < 16 && k0 + 4 < kend;
        if (MODE == 4 ? c0 + 4 < 16 : next) {   // (prediction: the block's columns may start in this tile)
          static_for<K, G>(BV_CI(I) {
            BV_CV(I);
            acc[tix(I, K)] = M::op(v[I], v[K], acc[tix(I, K)]);
          });
          if (EINV) einv = M::op(ve, v[K], einv);
        }
        if constexpr (KEEP) {
          wave_lds_sync();
          static_for<K, G>(BV_CI(I) {
            BV_CV(I);
            pan[(I * 16 + lr) * 4 + lg] = v[I];
          });
          if (EINV) pan[(P + lr) * 4 + lg] = ve;
          wave_lds_sync();
          if (lr >= c0 && lr < c0 + 4) {
            static_for<K, G>(BV_CI(I) {
              BV_CV(I);
#pragma unroll
              for (int r = 0; r < 4; ++r) acc[tix(I, K)][r] = pan[(I * 16 + M::row(lg, r)) * 4 + lr - c0];
            });
            if (EINV) {
#pragma unroll
              for (int r = 0; r < 4; ++r) einv[r] = pan[(P + M::row(lg, r)) * 4 + lr - c0];
            }
          }
        }
        wave_lds_sync();
        static_for<K + 1, G>(BV_CI(I) {
          BV_CV(I);
          static_for<K + 1, I + 1>(BV_CI(J) {
            BV_CV(J);
            acc[tix(I, J)] = M::op(v[I], v[J], acc[tix(I, J)]);
          });
        });
        if (next) publish_rows(K_c, c0 + 4);
        wave_lds_sync();
        if (next) read_block(k0 + 4, D);
        if (!next) break;
      }
      if constexpr (EINV) finish_einv(K_c);
    } else
    if constexpr (sizeof(T) == 4 && (MODE == 5 || MODE == 2)) {
      // FP32 gradient, one step per panel of four columns: the rank-4 update of tile
      // column K first (the next panel's columns are in it) and the finished
      // columns kept, then the next panel is published before the update of
      // the tiles right of column K is issued, and its factorisation follows
      // while the matrix core still works on that update.  (FP64 keeps the
      // plain order: its tiles leave no registers for the longer-lived panel;
      // the value and prediction kernels measured faster in it as well.)
      publish(std::integral_constant<int, K>{}, 0);
      wave_lds_sync();
      factor_panel(K_c, K * 16);
      wave_lds_sync();
#pragma nounroll
      for (int c0 = 0;; c0 += 4) {
        T v[G];
        static_for<K, G>(BV_CI(I) {
          BV_CV(I);
          v[I] = pan[lg * PS + I * 16 + lr];
        });
        // the tile column's last panel leaves no column of it to update
        const bool next = c0 + 4 < 16 && K * 16 + c0 + 4 < kend;
        if (next) {
          static_for<K, G>(BV_CI(I) {
            BV_CV(I);
            acc[tix(I, K)] = M::op(v[I], v[K], acc[tix(I, K)]);
          });
          if (EINV) einv = M::op(pan[lg * PS + P + lr], v[K], einv);
        }
        if (MODE != 0 && MODE != 4 && lr >= c0 && lr < c0 + 4) {
          // keep the finished factor columns in the tiles
          static_for<K, G>(BV_CI(I) {
            BV_CV(I);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[tix(I, K)][r] = pan[(lr - c0) * PS + I * 16 + M::row(lg, r)];
          });
          if (EINV) {
#pragma unroll
            for (int r = 0; r < 4; ++r) einv[r] = pan[(lr - c0) * PS + P + M::row(lg, r)];
          }
        }
        // the rank-4 update of the tiles right of tile column K
        auto trailing = [&]() __attribute__((always_inline)) {
          static_for<K + 1, G>(BV_CI(I) {
            BV_CV(I);
            static_for<K + 1, I + 1>(BV_CI(J) {
              BV_CV(J);
              acc[tix(I, J)] = M::op(v[I], v[J], acc[tix(I, J)]);
            });
          });
        };
        wave_lds_sync();
        if (next) publish(std::integral_constant<int, K>{}, c0 + 4);
        wave_lds_sync();
        trailing();
        if (!next) break;
        factor_panel(K_c, K * 16 + c0 + 4);
        wave_lds_sync();
      }
    } else {
#pragma nounroll
      for (int c0 = 0; c0 < 16; c0 += 4) {
        const int k0 = K * 16 + c0;
        if (k0 >= kend) break;
        publish(std::integral_constant<int, K>{}, c0);
        wave_lds_sync();
        factor_panel(K_c, k0);
        wave_lds_sync();
        T v[G];
        static_for<K, G>(BV_CI(I) {
          BV_CV(I);
          v[I] = pan[lg * PS + I * 16 + lr];
        });
        if constexpr (TIGHT) {
          static_for<K, G>(BV_CI(I) {
            BV_CV(I);
            static_for<K, I + 1>(BV_CI(J) {
              BV_CV(J);
              acc[tix(I, J)] = M::op(v[I], v[J], acc[tix(I, J)]);
            });
          });
          if (EINV) einv = M::op(pan[lg * PS + P + lr], v[K], einv);
        } else {
          // the tile column itself, unless this was its last panel
          if (c0 + 4 < 16) {
            static_for<K, G>(BV_CI(I) {
              BV_CV(I);
              acc[tix(I, K)] = M::op(v[I], v[K], acc[tix(I, K)]);
            });
            if (EINV) einv = M::op(pan[lg * PS + P + lr], v[K], einv);
          }
          if constexpr (!LEFT) {   // the tiles right of it (mode 6 updates those when their turn comes)
            static_for<K + 1, G>(BV_CI(I) {
              BV_CV(I);
              static_for<K + 1, I + 1>(BV_CI(J) {
                BV_CV(J);
                acc[tix(I, J)] = M::op(v[I], v[J], acc[tix(I, J)]);
              });
            });
          }
        }
        if (MODE != 0 && MODE != 4 && lr >= c0 && lr < c0 + 4) {
          // keep the finished factor columns in the tiles
          static_for<K, G>(BV_CI(I) {
            BV_CV(I);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[tix(I, K)][r] = pan[(lr - c0) * PS + I * 16 + M::row(lg, r)];
          });
          if (EINV) {
#pragma unroll
            for (int r = 0; r < 4; ++r) einv[r] = pan[(lr - c0) * PS + P + M::row(lg, r)];
          }
        }
        wave_lds_sync();
      }
    }
    if constexpr (EINV && !ROWPAN) finish_einv(K_c);
    if constexpr (LEFT) {
      // the finished tile column to the item's slot; the later columns read it
      // back through global memory (hence the workgroup barrier)
      static_for<K, G>(BV_CI(I) {
        BV_CV(I);
#pragma unroll
        for (int r = 0; r < 4; ++r) Lg[(I * (I + 1) / 2 + K) * 256 + ln * 4 + r] = acc[tix(I, K)][r];
      });
      __syncthreads();
    }
  });

  if constexpr (MODE == 4) {
    // ---- prediction outputs from the trailing tiles (they hold -A) ------------
    int bad = 0;
    for (int k = ln; k < m; k += 64) bad |= !((double)sdk[k] > 0.0);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) bad |= __shfl_xor(bad, off, 64);
    const double nanv = __builtin_nan("");
    double* pm = a.out_mean + b0;
    double* pv = a.out_var + b0;
    double* pc = a.out_cov ? a.out_cov + (size_t)b * a.ldc * a.ldc : nullptr;
    static_for<0, G>(BV_CI(I) {
      BV_CV(I);
      if (I * 16 > p) return;
      static_for<0, I + 1>(BV_CI(J) {
        BV_CV(J);
        if (J * 16 + 15 < mq) return;
        const int j = J * 16 + lr;
        if (j < mq || j >= p) return;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = I * 16 + M::row(lg, r);
          const double v = (double)acc[tix(I, J)][r];
          if (i == p) {
            pm[j - mq] = bad ? nanv : v;            // border row: -(-mu)
          } else if (i >= j && i < p) {
            const double c = bad ? nanv : -v;       // Schur complement: Sigma_B
            if (i == j) pv[j - mq] = c;
            if (pc) {
              pc[(size_t)(i - mq) * a.ldc + (j - mq)] = c;
              pc[(size_t)(j - mq) * a.ldc + (i - mq)] = c;
            }
          }
        }
      });
    });
    return;
  }

  // ---- log-determinant, quadratic form and pivot guard (FP64) -----------------
  const double guard = a.fp32_guard == 2 ? INFINITY
      : a.fp32_guard ? fmax(0.5 * th.nugget, (double)p * 1.1920928955078125e-07 * (th.sigma2 + th.nugget))
      : 0.0;
  for (int k = ln; k < p; k += 64) {
    const double dd = (double)sdk[k];
    if (!(dd > guard)) flag |= a.fp32_guard ? 1 : 2;
    if (!(dd > 0.0)) flag |= 2;
    if (k >= m) {
      const double wk = (double)swk[k];
      // FP32 pivots: log2 by the hardware (about 1 ulp of the FP32 value)
      const double lgd = sizeof(T) == 4 ? (double)__builtin_amdgcn_logf((float)sdk[k]) * kLn2 : log(dd);
      acc_ll += lgd + wk * wk;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    acc_ll += __shfl_down(acc_ll, off, 64);
    flag |= __shfl_down(flag, off, 64);
  }
  if (MODE == 0 || MODE == 2 || MODE == 6) {
    if (ln == 0) {
      a.partial[o] = (flag & 2) && !a.fp32_guard ? __builtin_nan("") : -0.5 * (acc_ll + (double)l * kLog2Pi);
      a.flag[o] = flag | a.flag_or;
    }
  }
  if (MODE == 0) return;
  if constexpr (!INREG) {
    // the factor leaves the registers for this item's slot of the tile buffer
    // (accumulator order, 256 elements per tile), so the adjoint's phases do not
    // hold the tiles in registers
    if constexpr (!LEFT) {   // (mode 6 stored its tiles column by column)
      static_for<0, NT>(BV_CI(t) {
        BV_CV(t);
#pragma unroll
        for (int r = 0; r < 4; ++r) Lg[t * 256 + ln * 4 + r] = acc[t][r];
      });
    }
    // the border row w = L^-1 y_J (the diagonal tiles no longer hold it in MODES 2, 6)
    for (int j = ln; j < P; j += 64) Lg[NT * 256 + j] = j < p ? swk[j] : T(0);
    __syncthreads();
  }
  if (MODE == 2 || MODE == 6) return;
  } else {
    flag = a.flag[o];   // written by the factorisation launch
  }

  constexpr int CH = wave_chunk(G);   // right-hand sides per pass
  constexpr int NQ = (CH + 15) / 16;             // 16-column tiles of one pass
  constexpr int LDX = CH + 1;
  // with CH < 32 the second 16-column tile is partly outside a row: its reads
  // there are harmless (other columns of the MFMA results), its writes masked
  auto colok = [&](int q) __attribute__((always_inline)) { return (q + 1) * 16 <= CH || q * 16 + lr < CH; };
  constexpr int GM = G > 1 ? G - 1 : 1;   // tile rows above a diagonal step, at most
  const int nr = l + 2;
  const int Gp = (p + 15) >> 4;
  T* X = work;   // X[row * LDX + col], one chunk of right-hand sides
  // clears X (and the 32 elements after it) with 16-byte stores
  auto zero_x = [&]() __attribute__((always_inline)) {
    constexpr int V = 16 / (int)sizeof(T);
    static_assert((P * LDX + 32) % V == 0 && (3 * P * sizeof(T)) % 16 == 0, "16-byte stores into X");
    typedef T vec_t __attribute__((ext_vector_type(V)));
    vec_t* xv = reinterpret_cast<vec_t*>(X);
    for (int e = ln; e < (P * LDX + 32) / V; e += 64) xv[e] = vec_t(0);
  };

  const T irange = T(th.inv_range);
  T dh0 = T(0), dh1 = T(0), dh2 = T(0);   // closed forms: d rho / d range coefficients over the range
  if constexpr (!GEN) {
    dh0 = T((double)mc.g0 * th.inv_range * kLn2);
    dh1 = T((double)mc.g1 * th.inv_range * kLn2 * kLn2);
    dh2 = T((double)mc.g2 * th.inv_range * kLn2 * kLn2 * kLn2);
  }
  // d/d sigma2 needs no entry of dK: with d K_J / d sigma2 = (K_J - nugget I) / sigma2,
  // <W, K_J> = ||w||^2 - ||w_N||^2 - l (the quadratic forms of y_J and y_N, and
  // tr(X_R^T K_J X_R) = l) and tr W = 2 d l / d nugget, so that
  // d l / d sigma2 = (sum_{k >= m} w_k^2 - l - nugget tr W) / (2 sigma2)
  double g1 = 0.0, g2 = 0.0, qb = 0.0, g3 = 0.0;   // g3: <W, d rho / d nu> (Bessel form, on request)
  const bool want_nu = GEN && a.gnu != nullptr;
  // FP32 Bessel form: one distance at a time
  auto drange = [&](T x) __attribute__((always_inline)) {
    double rho, g;
    matern_general((double)x, th.bes, &rho, &g);
    return T(g) * irange;
  };
  auto drange_dnu = [&](T x, T& dr, T& dn) __attribute__((always_inline)) {
    double rho, g, v;
    matern_general_dnu((double)x, th.bes, &rho, &g, &v);
    dr = T(g) * irange;
    dn = T(v);
  };
  // W = alpha alpha^T - b b^T - X_R X_R^T over the right-hand sides [cb, cb + nc)
  // held in X, contracted with dK regenerated entry by entry
  auto contract = [&](int cb, int nc) __attribute__((always_inline)) {
    // the next tile's MFMA chain is issued before this tile's contraction
    const int nk = (nc + 3) >> 2;
    for (int I = 0; I < Gp; ++I) {
      T av[CH / 4];
#pragma unroll
      for (int kq = 0; kq < CH / 4; ++kq) {
        const int q = 4 * kq + lg;
        av[kq] = (cb + q == 0 ? T(1) : T(-1)) * X[(I * 16 + lr) * LDX + q];
      }
      T ri[4][3];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = I * 16 + M::row(lg, r);
        ri[r][0] = su[i];
        ri[r][1] = su[P + i];
        ri[r][2] = su[2 * P + i];
      }
      auto wtile = [&](int J) __attribute__((always_inline)) {
        // all B operands are read before the first product (the reads stay in
        // the row: 4 kq + lg < CH), so the chain waits for LDS once
        T xb[CH / 4];
#pragma unroll
        for (int kq = 0; kq < CH / 4; ++kq) xb[kq] = X[(J * 16 + lr) * LDX + 4 * kq + lg];
        acc_t c;
#pragma unroll
        for (int r = 0; r < 4; ++r) c[r] = T(0);
#pragma unroll
        for (int kq = 0; kq < CH / 4; ++kq)
          if (kq < nk) c = M::op(av[kq], xb[kq], c);
        return c;
      };
      // (with two FP64 waves per SIMD the other wave covers it, and there are no
      // registers for a second tile)
      constexpr bool AHEAD = !(sizeof(T) == 8 && wave_min_waves<T, G, MODE, GEN>() >= 2);
      acc_t cn;
      if constexpr (AHEAD) cn = wtile(0);
      for (int J = 0; J <= I; ++J) {
        acc_t c;
        if constexpr (AHEAD) {
          c = cn;
          if (J < I) cn = wtile(J + 1);
        } else {
          c = wtile(J);
        }
        const int j = J * 16 + lr;
        const T sj0 = su[j], sj1 = su[P + j], sj2 = su[2 * P + j];
        T s1 = T(0), s2 = T(0), s3 = T(0);
        T dx[4], dy[4], dz[4], u[4];
        typename ExpOf<T>::type e[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          dx[r] = ri[r][0] - sj0;
          dy[r] = ri[r][1] - sj1;
          dz[r] = ri[r][2] - sj2;
        }
        BesselOut bes;   // g of the four, then their d rho / d nu
        if constexpr (!GEN) {
          distance_exp2neg4<STAGED>(dx, dy, dz, u, e);
        } else if constexpr (BES4) {
          Bessel4 x;
#pragma unroll
          for (int r = 0; r < 4; ++r) x[r] = (double)distance<T>(dx[r], dy[r], dz[r]);
          bes = want_nu ? bessel4<2>(x, btab) : bessel4<1>(x, btab);
        }
        auto entry = [&](int r) __attribute__((always_inline)) {
          if constexpr (BES4) {
            s1 += c[r] * (T(bes[r]) * irange);
            if (want_nu) s3 += c[r] * T(bes[r + 4]);
          } else if constexpr (GEN) {
            const T x = distance<T>(dx[r], dy[r], dz[r]);
            if (want_nu) {
              T dr, dn;
              drange_dnu(x, dr, dn);
              s1 += c[r] * dr;
              s3 += c[r] * dn;
            } else {
              s1 += c[r] * drange(x);
            }
          } else {
            s1 += c[r] * mc.drange_log2(u[r], e[r], dh0, dh1, dh2);
          }
        };
        if ((I + 1) * 16 <= p) {   // a tile inside the point rows (wave-uniform)
#pragma unroll
          for (int r = 0; r < 4; ++r) entry(r);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (I * 16 + M::row(lg, r) < p && j < p) entry(r);
        }
        if (I == J) {   // d K / d nugget is the identity
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (M::row(lg, r) == lr && j < p) s2 += c[r];
        }
        const double wgt = I == J ? 1.0 : 2.0;
        g1 += wgt * (double)s1;
        g2 += (double)s2;
        if (GEN) g3 += wgt * (double)s3;
      }
    }
  };

  if constexpr (INREG) {
    // ---- factor kept in the registers (its diagonal tiles already replaced by
    // their inverses), CH right-hand sides per pass ---------------------------
    // border row of the bordered factor, w = L^-1 y_J, from the factorisation's
    // LDS record to LDS past the right-hand sides (which overwrite the record)
    T* sw = work + wave_max(PANEL + 3 * P, P * LDX + 32);
    static_assert(3 * P + wave_max(PANEL + 3 * P, P * LDX + 32) + P <= wave_lds_elems(G, MODE), "LDS of w");
    for (int j = ln; j < P; j += 64) {
      const T w = j < p ? swk[j] : T(0);
      sw[j] = w;
      if (j >= m && j < p) qb += (double)w * (double)w;
    }
    for (int cb = 0; cb < nr; cb += CH) {
    const int nc = nr - cb < CH ? nr - cb : CH;
    wave_lds_sync();
    // columns cb .. cb + nc - 1 of the right-hand sides [ w | [z; 0] | [0; I_l] ]
    zero_x();
    wave_lds_sync();
    for (int c = ln; c < nc; c += 64)
      if (cb + c >= 2) X[(m + cb + c - 2) * LDX + c] = T(1);
    if (cb == 0) {
      for (int j = ln; j < p; j += 64) {
        X[j * LDX] = sw[j];
        if (j < m) X[j * LDX + 1] = sw[j];
      }
    }
    wave_lds_sync();
    // X <- L^-T X, tile row by tile row from the bottom.  Every product
    // contracts over the rows of a factor tile, so the accumulator registers
    // serve as the A operand as they are: k-step s of lane (i, k) takes
    // register s, i.e. row M::row(k, s) of the tile, and the B operand takes
    // the same row of X.  The diagonal step's result, in accumulator layout,
    // is then directly the B operand of the updates of the rows above.
    // (all NQ column tiles every step: the columns at and beyond nc are zero
    // and stay zero, so no step branches on the chunk width)
    static_for_down<0, G>(BV_CI(K) {
      BV_CV(K);
      if (K >= Gp) return;
      acc_t dq[NQ];
      T xb[NQ][4];
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int sb = 0; sb < 4; ++sb) xb[q][sb] = X[(K * 16 + M::row(lg, sb)) * LDX + q * 16 + lr];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
#pragma unroll
        for (int r = 0; r < 4; ++r) dq[q][r] = T(0);
#pragma unroll
        for (int sb = 0; sb < 4; ++sb) dq[q] = M::op(acc[tix(K, K)][sb], xb[q][sb], dq[q]);
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (colok(q)) {
#pragma unroll
          for (int r = 0; r < 4; ++r) X[(K * 16 + M::row(lg, r)) * LDX + q * 16 + lr] = dq[q][r];
        }
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) dq[q][r] = -dq[q][r];
      // rows above: X_J -= L_KJ^T X_K
      static_for<0, K>(BV_CI(J) {
        BV_CV(J);
        acc_t cj[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int r = 0; r < 4; ++r) cj[q][r] = X[(J * 16 + M::row(lg, r)) * LDX + q * 16 + lr];
#pragma unroll
        for (int sb = 0; sb < 4; ++sb)
#pragma unroll
          for (int q = 0; q < NQ; ++q) cj[q] = M::op(acc[tix(K, J)][sb], dq[q][sb], cj[q]);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          if (colok(q)) {
#pragma unroll
            for (int r = 0; r < 4; ++r) X[(J * 16 + M::row(lg, r)) * LDX + q * 16 + lr] = cj[q][r];
          }
      });
      wave_lds_sync();
    });
    contract(cb, nc);
    if constexpr (!wave_regadj_passes(G, sizeof(T) == 4)) break;   // one pass: nr <= CH
    }
  } else {
  // border row p of the bordered factor: w = L^-1 y_J, stored after the tiles
  constexpr int NW = (P + 63) / 64;
  T wreg[NW];
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    const int j = ln + 64 * k;
    wreg[k] = j < p ? Lg[NT * 256 + j] : T(0);
    if (j >= m && j < p) qb += (double)wreg[k] * (double)wreg[k];
  }

  // ---- inverses of the diagonal 16 x 16 blocks of L (MODE 1; MODE 3 reads the
  // ones its factorisation launch formed) ---------------------------------------
  if constexpr (MODE == 1) {
  // all Gp blocks staged at once (the border row and the padding become
  // identity rows); lane (c = l % 16, g = l / 16) forms column c of inv(L_KK)
  // for K = g, g + 4, g + 8 by forward substitution, three independent chains
  {
    constexpr int NB = (G + 3) / 4;   // blocks per lane group
    for (int K = 0; K < Gp; ++K) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rw = M::row(lg, r);
        const int i = K * 16 + rw, j = K * 16 + lr;
        T v = Lg[(K * (K + 1) / 2 + K) * 256 + ln * 4 + r];
        if (i >= p || j >= p) v = (i == j) ? T(1) : T(0);
        X[K * kStageStride + rw * 16 + lr] = v;
      }
    }
    wave_lds_sync();
    const int c = lr;
    T x[NB][16];
    const T* Lk[NB];
#pragma unroll
    for (int jb = 0; jb < NB; ++jb) {
      const int K = lg + 4 * jb;
      Lk[jb] = X + (K < Gp ? K : 0) * kStageStride;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
#pragma unroll
      for (int jb = 0; jb < NB; ++jb) {
        T sum = T(0);
#pragma unroll
        for (int k = 0; k < i; ++k) sum += Lk[jb][i * 16 + k] * x[jb][k];
        const T rd = T(1) / Lk[jb][i * 16 + i];
        x[jb][i] = i < c ? T(0) : (i == c ? rd : -sum * rd);
      }
    }
#pragma unroll
    for (int jb = 0; jb < NB; ++jb) {
      const int K = lg + 4 * jb;
      if (K < Gp) {
        T* dst = Lg + (K * (K + 1) / 2 + K) * 256;
#pragma unroll
        for (int i = 0; i < 16; ++i) dst[M::at(i, c)] = x[jb][i];
      }
    }
  }
  }   // MODE 1
  __syncthreads();

  // ---- X <- L^-T X and the contraction, CH right-hand sides per pass ---------
  for (int cb = 0; cb < nr; cb += CH) {
    const int nc = nr - cb < CH ? nr - cb : CH;
    const int nq = (nc + 15) >> 4;
    wave_lds_sync();
    zero_x();
    wave_lds_sync();
    // column cb + c of [ w | [z; 0] | [0; I_l] ]
    for (int c = ln; c < nc; c += 64)
      if (cb + c >= 2) X[(m + cb + c - 2) * LDX + c] = T(1);
    if (cb == 0) {
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const int j = ln + 64 * k;
        if (j < p) {
          X[j * LDX] = wreg[k];
          if (j < m) X[j * LDX + 1] = wreg[k];
        }
      }
    }
    wave_lds_sync();
    for (int K = Gp - 1; K >= 0; --K) {
      const T* Lrow = Lg + (K * (K + 1) / 2) * 256;   // tile row K: tiles (K, 0..K)
      // A operands from the tile buffer: inv(L_KK)^T and -L_KJ^T, J < K
      T ad[4];
#pragma unroll
      for (int sb = 0; sb < 4; ++sb) ad[sb] = Lrow[K * 256 + M::aop(ln, sb)];
      T aj[GM][4];
#pragma unroll
      for (int J = 0; J < GM; ++J)
        if (J < K) {
#pragma unroll
          for (int sb = 0; sb < 4; ++sb) aj[J][sb] = -Lrow[J * 256 + M::aop(ln, sb)];
        }
      // diagonal step: X_K <- inv(L_KK)^T X_K
      acc_t dq[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int r = 0; r < 4; ++r) dq[q][r] = T(0);
        if (q < nq) {
#pragma unroll
          for (int sb = 0; sb < 4; ++sb) dq[q] = M::op(ad[sb], X[(K * 16 + 4 * sb + lg) * LDX + q * 16 + lr], dq[q]);
        }
      }
      wave_lds_sync();
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (q < nq && colok(q)) {
#pragma unroll
          for (int r = 0; r < 4; ++r) X[(K * 16 + M::row(lg, r)) * LDX + q * 16 + lr] = dq[q][r];
        }
      wave_lds_sync();
      // rows above: X_J -= L_KJ^T X_K (all tiles loaded first, then the MFMA chains)
      if (K > 0) {
        T bq[2][4];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int sb = 0; sb < 4; ++sb) bq[q][sb] = X[(K * 16 + 4 * sb + lg) * LDX + q * 16 + lr];
        acc_t cj[GM][2];
#pragma unroll
        for (int J = 0; J < GM; ++J)
          if (J < K) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
              if (q < nq) {
#pragma unroll
                for (int r = 0; r < 4; ++r) cj[J][q][r] = X[(J * 16 + M::row(lg, r)) * LDX + q * 16 + lr];
              }
          }
#pragma unroll
        for (int sb = 0; sb < 4; ++sb)
#pragma unroll
          for (int J = 0; J < GM; ++J)
#pragma unroll
            for (int q = 0; q < 2; ++q)
              if (J < K && q < nq) cj[J][q] = M::op(aj[J][sb], bq[q][sb], cj[J][q]);
#pragma unroll
        for (int J = 0; J < GM; ++J)
          if (J < K) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
              if (q < nq && colok(q)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) X[(J * 16 + M::row(lg, r)) * LDX + q * 16 + lr] = cj[J][q][r];
              }
          }
        wave_lds_sync();
      }
    }

    contract(cb, nc);
  }
  }   // MODE != 5
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    qb += __shfl_down(qb, off, 64);
    if (GEN) g3 += __shfl_down(g3, off, 64);
    g1 += __shfl_down(g1, off, 64);
    g2 += __shfl_down(g2, off, 64);
  }
  if (ln == 0) {
    const bool bad = (flag & 2) && !a.fp32_guard;
    if (MODE == 1 || MODE == 5) {
      a.partial[o] = bad ? __builtin_nan("") : -0.5 * (acc_ll + (double)l * kLog2Pi);
      a.flag[o] = flag | a.flag_or;
    }
    a.gpart[3 * o + 0] = bad ? __builtin_nan("") : 0.5 * (qb - (double)l - th.nugget * g2) / th.sigma2;
    a.gpart[3 * o + 1] = bad ? __builtin_nan("") : 0.5 * th.sigma2 * g1;
    a.gpart[3 * o + 2] = bad ? __builtin_nan("") : 0.5 * g2;
    if (want_nu) a.gnu[o] = bad ? __builtin_nan("") : 0.5 * th.sigma2 * g3;
  }
}

template <typename T, int G, int MODE, bool GEN>
static hipError_t launch_wave_g(const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  const size_t lds = GEN && sizeof(T) == 8 ? (size_t)wave_table_offset(sizeof(T), G, MODE) + kBesselBytes
                                           : sizeof(T) * (size_t)wave_lds_elems(G, MODE);
  hipLaunchKernelGGL((bv_wave_kernel<T, G, MODE, GEN>), dim3(grid), dim3(64), lds, s, a, thp);
  return hipGetLastError();
}

template <typename T, int MODE, bool GEN = false>
static hipError_t launch_wave_t(int g, const AdjArgs& a, const ThetaPack& thp, int grid, hipStream_t s) {
  if constexpr (MODE == 5) {   // factor kept in the registers: up to G = 9 (FP32: 10)
    switch (g) {
      case 1: return launch_wave_g<T, 1, MODE, GEN>(a, thp, grid, s);
      case 2: return launch_wave_g<T, 2, MODE, GEN>(a, thp, grid, s);
      case 3: return launch_wave_g<T, 3, MODE, GEN>(a, thp, grid, s);
      case 4: return launch_wave_g<T, 4, MODE, GEN>(a, thp, grid, s);
      case 5: return launch_wave_g<T, 5, MODE, GEN>(a, thp, grid, s);
      case 6: return launch_wave_g<T, 6, MODE, GEN>(a, thp, grid, s);
      case 7: return launch_wave_g<T, 7, MODE, GEN>(a, thp, grid, s);
      case 8: return launch_wave_g<T, 8, MODE, GEN>(a, thp, grid, s);
      case 9: return launch_wave_g<T, 9, MODE, GEN>(a, thp, grid, s);
#if BV_REGADJ_MAX_G32 >= 10
      case 10:   // FP32 only (one wave per SIMD)
        if constexpr (sizeof(T) == 4) return launch_wave_g<T, 10, MODE, GEN>(a, thp, grid, s);
        return hipErrorInvalidValue;
#endif
      default: return hipErrorInvalidValue;
    }
  } else if constexpr (MODE == 6) {   // left-looking factorisation: FP64 above G = 9
    if constexpr (sizeof(T) == 8) {
      if (g == 10) return launch_wave_g<T, 10, MODE, GEN>(a, thp, grid, s);
      if (g == 11) return launch_wave_g<T, 11, MODE, GEN>(a, thp, grid, s);
    }
    return hipErrorInvalidValue;
  } else if constexpr (MODE == 2 || MODE == 3) {   // split gradient: only the classes that use it
    // (FP32: factorisation by mode 2; FP64: by mode 6, adjoint by mode 3 in both)
    if constexpr (sizeof(T) == 4 || MODE == 3) {
      if constexpr (sizeof(T) == 8 || BV_REGADJ_MAX_G32 < 10) {
        if (g == 10) return launch_wave_g<T, 10, MODE, GEN>(a, thp, grid, s);
      }
      if (g == 11) return launch_wave_g<T, 11, MODE, GEN>(a, thp, grid, s);
    }
    return hipErrorInvalidValue;
  } else if constexpr (MODE == 1 && sizeof(T) == 8) {
    // the classes that neither keep the factor in registers nor split: G = 9 with
    // several passes of right-hand sides, and the Bessel form above it
    if (g == 9) return launch_wave_g<T, 9, MODE, GEN>(a, thp, grid, s);
    if constexpr (GEN) {
      if (g == 10) return launch_wave_g<T, 10, MODE, GEN>(a, thp, grid, s);
      if (g == 11) return launch_wave_g<T, 11, MODE, GEN>(a, thp, grid, s);
    }
    return hipErrorInvalidValue;
  } else if constexpr (MODE == 1) {   // FP32 G >= 10 use the split gradient
    switch (g) {
      case 1: return launch_wave_g<T, 1, MODE, GEN>(a, thp, grid, s);
      case 2: return launch_wave_g<T, 2, MODE, GEN>(a, thp, grid, s);
      case 3: return launch_wave_g<T, 3, MODE, GEN>(a, thp, grid, s);
      case 4: return launch_wave_g<T, 4, MODE, GEN>(a, thp, grid, s);
      case 5: return launch_wave_g<T, 5, MODE, GEN>(a, thp, grid, s);
      case 6: return launch_wave_g<T, 6, MODE, GEN>(a, thp, grid, s);
      case 7: return launch_wave_g<T, 7, MODE, GEN>(a, thp, grid, s);
      case 8: return launch_wave_g<T, 8, MODE, GEN>(a, thp, grid, s);
      case 9: return launch_wave_g<T, 9, MODE, GEN>(a, thp, grid, s);
      default: return hipErrorInvalidValue;
    }
  } else if constexpr (MODE == 0 && sizeof(T) == 8 && !GEN) {   // (G = 7 .. 10: wave_rows.hpp)
    switch (g) {
      case 1: return launch_wave_g<T, 1, MODE, GEN>(a, thp, grid, s);
      case 2: return launch_wave_g<T, 2, MODE, GEN>(a, thp, grid, s);
      case 3: return launch_wave_g<T, 3, MODE, GEN>(a, thp, grid, s);
      case 4: return launch_wave_g<T, 4, MODE, GEN>(a, thp, grid, s);
      case 5: return launch_wave_g<T, 5, MODE, GEN>(a, thp, grid, s);
      case 6: return launch_wave_g<T, 6, MODE, GEN>(a, thp, grid, s);
      case 11: return launch_wave_g<T, 11, MODE, GEN>(a, thp, grid, s);
      default: return hipErrorInvalidValue;
    }
  } else {
  switch (g) {
    case 1: return launch_wave_g<T, 1, MODE, GEN>(a, thp, grid, s);
    case 2: return launch_wave_g<T, 2, MODE, GEN>(a, thp, grid, s);
    case 3: return launch_wave_g<T, 3, MODE, GEN>(a, thp, grid, s);
    case 4: return launch_wave_g<T, 4, MODE, GEN>(a, thp, grid, s);
    case 5: return launch_wave_g<T, 5, MODE, GEN>(a, thp, grid, s);
    case 6: return launch_wave_g<T, 6, MODE, GEN>(a, thp, grid, s);
    case 7: return launch_wave_g<T, 7, MODE, GEN>(a, thp, grid, s);
    case 8: return launch_wave_g<T, 8, MODE, GEN>(a, thp, grid, s);
    case 9: return launch_wave_g<T, 9, MODE, GEN>(a, thp, grid, s);
    case 10: return launch_wave_g<T, 10, MODE, GEN>(a, thp, grid, s);
    case 11: return launch_wave_g<T, 11, MODE, GEN>(a, thp, grid, s);
    default: return hipErrorInvalidValue;
  }
  }
}

}  // namespace bv
