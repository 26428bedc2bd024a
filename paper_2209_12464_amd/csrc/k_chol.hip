// Cholesky factor of the float64 Gram matrix, G = R^T R (R upper): the
// middle step of each CholeskyQR pass (orth() and qr() of the paper,
// computed as an unpivoted QR with a positive diagonal in R).
//
// For d <= 256, one workgroup of 16 waves, right-looking over 16-row blocks k of the
// upper triangle.  The 16 x 16 tiles of G on and above the diagonal are held in
// registers (MFMA 16x16x4 accumulator layout: lane l holds rows l/16 + 4 s, column
// l % 16) by 12 waves, dealt to them row by row.  The other 4 waves, one a SIMD,
// eliminate a block row: a lane has one column of it and all 16 rows, and each row
// of 16 lanes a copy of the diagonal tile, so that a pivot's multipliers come from
// the neighbour lanes and diagonal tile, panel and L_kk^-1 (the columns of the
// identity) take their steps together, without MFMA or LDS in between.  Per k:
//   A. the 4 waves eliminate block row k (in LDS) and put it back, while the 12
//      do the rest of step k - 1, G_ij -= R_ti^T R_tj for t = k - 1 and i > k (MFMA),
//      and store block row k - 1 of R;
//   B. the 12 bring row k + 1 up to date with row k and put it in LDS.
// (With 16 tile columns 36 of the 12 slots' registers a lane are spilled.)
// What bounds it is the chain of A and B: about 3500 + 1500 cycles a step at 2.1
// GHz, of which the 16 pivots' row operations are 1000 (240 FMAs of 4 cycles), and
// with many tiles the float64 MFMAs of A (64 cycles each, 4 a tile, in the same
// pipes as the elimination).  Before, the wave that owned the diagonal tile took it
// in blocks of 4 pivots on wave-uniform scalars and MFMAs (5400 cycles), and panel
// and update followed.  This kernel before and after (traced): d = 64
// 15.6 -> 12.0 us, 110 30.5 -> 23.6, 176 51 -> 35, 192 59 -> 41, 210 75 -> 55.
// Columns whose pivot is <= tol * (their original squared norm) are marked
// dependent: their L column is zero, their R diagonal is 1 (so R stays
// invertible for the solve) and the caller replaces the matching columns of
// Q with random directions.
//
// Fast path for the second CholeskyQR pass: G = I + E with E small.  The
// upper-triangular F with F + F^T = E (F = triu(E, 1) + diag(E) / 2) gives
// R = I + F with R^T R = G + F^T F, so Q = Q1 R^-1 is orthonormal up to
// ~||F||_2^2 <= ||E||_F^2 / 4.  The host passes the largest ||E||_F that keeps
// this below the output precision; then R = I + F, R^-1 = I - F (to the same
// order) is written explicitly and the solve becomes a plain product.
#include "common.h"
#include "grouped.h"
#include "kernels.h"

#include <algorithm>
#include <utility>

namespace rqlp {

constexpr int kChE = 4;                    // waves that eliminate (one per SIMD)
constexpr int kChU = 12;                   // waves that hold the tiles
constexpr int kChWaves = kChE + kChU;
constexpr int kChThreads = kChWaves * kWave;

__device__ inline void tile_of(int t, int T, int& i, int& j) {
  // upper triangle of T x T tiles, row by row: t = i T - i (i - 1) / 2 + j - i
  i = 0;
  while (t >= T - i) t -= T - i++;
  j = i + t;
}

// 1/x and 1/sqrt(x) to float64 accuracy: the hardware estimate (relative error
// about 2^-24) and one third-order correction, y (1 + e + e^2) with e = 1 - x y
// and y (1 + e/2 + 3 e^2/8) with e = 1 - x y^2, as accurate as two Newton steps
// (about an ulp) with fewer dependent operations on the pivot chain.
__device__ __forceinline__ double rcp_f64(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, y, 1.0);
  return fma(y, fma(e, e, e), y);
}
__device__ __forceinline__ double rsqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// The value of lane C of each row of 16 lanes, in all of the row's lanes.
template <int C>
__device__ __forceinline__ double row_bcast(double v) {
  const long long b = __double_as_longlong(v);
  return __longlong_as_double(__builtin_amdgcn_update_dpp((long long)0, b, 0x150 + C, 0xf, 0xf, true));  // row_newbcast
}

// W_i += sp[i] tw and S_i += sp[i] ts, sp[i] taken from lane i of each row of 16
// lanes by the FMA itself (a move of its own for each sp[i] makes a chain of two
// instructions, twice the time: one wave a SIMD has nothing to hide it with).  A
// value written by a vector instruction can be read across lanes two instructions
// later: FIRST, at a pivot's first rows, waits for what came before, and for what
// the compiler does with these rows next.
#define RQLP_ROW_FMA(d, t, i) \
  "v_fmac_f64_dpp %[" d "], %[sp], %[" t "] row_newbcast:%[" i "] row_mask:0xf bank_mask:0xf\n\t"
#define RQLP_ROW_FMA2                                       \
  RQLP_ROW_FMA("w0", "tw", "i") RQLP_ROW_FMA("w1", "tw", "j") \
  RQLP_ROW_FMA("s0", "ts", "i") RQLP_ROW_FMA("s1", "ts", "j")
template <int I, bool FIRST>
__device__ __forceinline__ void row_fma2(double sp, double& s0, double& w0, double& s1, double& w1, double ts,
                                         double tw) {
  if constexpr (FIRST)
    asm volatile("s_nop 1\n\t" RQLP_ROW_FMA2 "s_nop 1"
                 : [s0] "+&v"(s0), [w0] "+&v"(w0), [s1] "+&v"(s1), [w1] "+&v"(w1)
                 : [sp] "v"(sp), [ts] "v"(ts), [tw] "v"(tw), [i] "i"(I), [j] "i"(I + 1));
  else
    asm volatile(RQLP_ROW_FMA2
                 : [s0] "+&v"(s0), [w0] "+&v"(w0), [s1] "+&v"(s1), [w1] "+&v"(w1)
                 : [sp] "v"(sp), [ts] "v"(ts), [tw] "v"(tw), [i] "i"(I), [j] "i"(I + 1));
}
template <int I>
__device__ __forceinline__ void row_fma1(double sp, double& s0, double& w0, double ts, double tw) {
  asm volatile("s_nop 1\n\t" RQLP_ROW_FMA("w0", "tw", "i") RQLP_ROW_FMA("s0", "ts", "i") "s_nop 1"
               : [s0] "+&v"(s0), [w0] "+&v"(w0)
               : [sp] "v"(sp), [ts] "v"(ts), [tw] "v"(tw), [i] "i"(I));
}
#undef RQLP_ROW_FMA2
#undef RQLP_ROW_FMA

// Pivot P of the elimination of a 16-row slab: S[i] holds row i of the diagonal
// tile (lane c of each row of 16 lanes: column c), W[i] row i of this lane's own
// column.  Rows below lose S[P][i] / d times row P, and row P goes to LDS as it is
// (its factor 1 / sqrt(d) is left to those who read it).  S[P][i] and not S[i][P],
// which rounds differently: the identity's columns have to see the very entries that
// become R, or X R - I is a thousand times as large (1.5e-11 for 1.2e-14 at d = 110),
// and R of the two passes with it less accurate (at condition 4e5 1.8e-15 for 7e-16,
// at 3e7 1.9e-13 for 1.1e-15).  What lies below the diagonal is not used.  d, the pivot, and r = 1 / d are in every lane and become the
// next ones, taken on a chain of their own (a reciprocal, a product and one FMA from
// pivot to pivot) whose operations stand between the rows' and hide behind them.  dv
// and rv collect d and -r, lane c those of column c.  CHECK: a pivot at or below thr is a dependent column, it
// eliminates nothing, and its row is zero outside the diagonal tile (`panel`
// lanes); a branch at every pivot costs half as much again as the elimination, so
// it is first done without.
template <bool CHECK, int P, int LD>
__device__ __forceinline__ void pivot_step(double (&S)[kTile], double (&W)[kTile], double& d, double& r, double& dv,
                                           double& rv, double thr, int lc, bool panel, double* put, double* put_s) {
  dv = lc == P ? d : dv;
  if (CHECK && __any(!(d > row_bcast<P>(thr)))) {  // (the same in every lane)
    put[P * LD] = panel ? 0.0 : W[P];
    put_s[P * LD] = 0.0;
    rv = lc == P ? 0.0 : rv;
    if constexpr (P + 1 < kTile) {
      d = row_bcast<P + 1>(S[P + 1]);
      r = rcp_f64(d);
    }
    return;
  }
  put[P * LD] = W[P];
  put_s[P * LD] = S[P];  // (the same from every wave and row of 16 lanes)
  rv = lc == P ? -r : rv;
  if constexpr (P + 1 < kTile) {
    const double next = row_bcast<P + 1>(S[P + 1]), b = row_bcast<P + 1>(S[P]);
    const double ts = -r * S[P], tw = -r * W[P];
    d = fma(-(b * r), b, next);  // (b b leaves the range at columns of norm 1e77 and 1e-81)
    double y = 0.0, e = 0.0;
    auto rows = [&]<int I>(std::integral_constant<int, I>) {  // rows P + 1 + 2 I, P + 2 + 2 I
      constexpr int i = P + 1 + 2 * I;
      if constexpr (i + 1 < kTile) row_fma2<i, I == 0>(S[P], S[i], W[i], S[i + 1], W[i + 1], ts, tw);
      else if constexpr (i < kTile) row_fma1<i>(S[P], S[i], W[i], ts, tw);
    };
    // 1 / d as rcp_f64 takes it, an operation after each pair of rows
    y = __builtin_amdgcn_rcp(d);
    __builtin_amdgcn_sched_barrier(0);
    rows(std::integral_constant<int, 0>{});
    rows(std::integral_constant<int, 1>{});
    e = fma(-d, y, 1.0);
    __builtin_amdgcn_sched_barrier(0);
    rows(std::integral_constant<int, 2>{});
    e = fma(e, e, e);
    __builtin_amdgcn_sched_barrier(0);
    rows(std::integral_constant<int, 3>{});
    r = fma(y, e, y);
    __builtin_amdgcn_sched_barrier(0);
    rows(std::integral_constant<int, 4>{});
    rows(std::integral_constant<int, 5>{});
    rows(std::integral_constant<int, 6>{});
    rows(std::integral_constant<int, 7>{});
  }
}

template <bool CHECK, int LD>
__device__ __forceinline__ void eliminate(double (&S)[kTile], double (&W)[kTile], double& dv, double& rv, double thr,
                                          int lc, bool panel, double* put, double* put_s) {
  double d = row_bcast<0>(S[0]), r = rcp_f64(d);
  [&]<int... P>(std::integer_sequence<int, P...>) {
    (pivot_step<CHECK, P, LD>(S, W, d, r, dv, rv, thr, lc, panel, put, put_s), ...);
  }(std::make_integer_sequence<int, kTile>{});
}

// Workgroup barrier for data passed in LDS: stores to memory in flight are not
// waited for.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Fast path of the second CholeskyQR pass: when ||G - I||_F < fast_tol
// (from the nesq partial sums the Gram reduction wrote; every workgroup adds
// them in the same fixed order), all workgroups write their share of
// R = I + F and R^-1 = I - F, and the call returns true.
__device__ inline bool chol_fast_path(const double* __restrict__ G, int d, int dp, double* __restrict__ R,
                                      double* __restrict__ Rinv16, int32_t* __restrict__ flags, double fast_tol,
                                      const double* __restrict__ esq, int nesq, int32_t* __restrict__ mode,
                                      double* __restrict__ Xfull, double* red, int nw, int bid, int nblk) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double ss = 0.0;
  for (int e = tid; e < nesq; e += blockDim.x) ss += esq[e];
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  if (lane == 0) red[wave] = ss;
  __syncthreads();
  double tot = 0.0;
  for (int w = 0; w < nw; ++w) tot += red[w];
  if (tot < fast_tol * fast_tol) {  // false for NaN
    for (int e = bid * blockDim.x + tid; e < dp * dp; e += nblk * blockDim.x) {
      const int i = e / dp, j = e - (e / dp) * dp;
      double f = 0.0;  // F[i][j]
      if (i < d && j < d && i <= j) {
        const double g = G[(int64_t)i * dp + j];
        f = (i < j) ? g : 0.5 * (g - 1.0);
      }
      const double id = (i == j) ? 1.0 : 0.0;
      R[(int64_t)i * dp + j] = id + f;
      Xfull[(int64_t)i * dp + j] = id - f;
      if ((i >> 4) == (j >> 4))
        Rinv16[(int64_t)(i >> 4) * kTile * kTile + (i & 15) * kTile + (j & 15)] = id - f;
    }
    for (int i = bid * blockDim.x + tid; i < dp; i += nblk * blockDim.x) flags[i] = 0;
    if (bid == 0 && tid == 0) *mode = 2;  // explicit inverse already written
    return true;
  }
  __syncthreads();
  return false;
}

// G (dp x dp block, row stride ld; R the same) is factored in registers.
// Standalone (block = 0): the whole matrix, with the fast path, and *mode
// set to 1 or 0.  As a diagonal block of a larger factorization (block =
// 1): nothing is done when *mode == 2, the dependence test takes the
// original diagonal from gdiag0, and *mode is only lowered to 0.
// The body is shared by the one-matrix kernel and the grouped kernel that
// factors many matrices in one launch (bid, nblk: this workgroup's index
// and the workgroup count of its matrix).
template <int TMAX>
__device__ __attribute__((always_inline)) inline void chol_body(const double* __restrict__ G, int ld, int d, int dp,
                                                    double* __restrict__ R,
                                                    double* __restrict__ Rinv16,
                                                    int32_t* __restrict__ flags, DevInfo* info,
                                                    int pass_id, double tol, double fast_tol,
                                                    const double* __restrict__ esq, int nesq,
                                                    int32_t* __restrict__ mode,
                                                    double* __restrict__ Xfull,
                                                    const double* __restrict__ gdiag0, int block, int bid, int nblk) {
  constexpr int SLOTS = (TMAX * (TMAX + 1) / 2 + kChU - 1) / kChU;
  // slab[k & 1]: block row k of D^1/2 R, D the pivots, and behind it D^1/2 R_kk (upper
  // part), D^1/2 L_kk^-1 and columns of scratch; beside it -1/D, D^-1/2 and R_kk's
  // diagonal; grow: the block row of G that is eliminated next.
  // Its row stride is 16 mod 32 values, so that the four rows an MFMA operand
  // takes spread over the banks.
  constexpr int RD = TMAX * kTile, XD = RD + kTile, LD = XD + 2 * kTile;
  constexpr int ZD = XD + kTile;
  static_assert(TMAX % 2 == 0 && TMAX <= 4 * kChE && TMAX <= 2 * kChU, "slab stride and width");
  __shared__ double slab[2][kTile][LD], grow[kTile][LD];
  __shared__ double nrd[2][kTile], rsd[2][kTile], diag[2][kTile];
  __shared__ double Gdiag[TMAX * kTile];
  __shared__ double red[kChWaves];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = dp / kTile;
  const int lr = lane >> 4, lc = lane & 15;  // MFMA accumulator layout: row lr + 4 r, col lc

  if (block) {
    if (*mode == 2) return;
  } else if (fast_tol > 0.0 && chol_fast_path(G, d, dp, R, Rinv16, flags, fast_tol, esq, nesq, mode, Xfull, red,
                                              kChWaves, bid, nblk)) {
    return;
  }
  if (bid != 0) return;  // the factorization runs in one workgroup

  // ---------------- full factorization ----------------
  for (int i = tid; i < dp; i += kChThreads)
    Gdiag[i] = (i < d) ? (gdiag0 ? gdiag0[i] : G[(int64_t)i * ld + i]) : 1.0;

  if (wave >= kChE) {
    // ---- tiles: slot sl of this wave holds tile (i, j), j >= i, packed as i + 256 j ----
    const int ntiles = T * (T + 1) / 2;
    doublex4 tile[SLOTS];
    int tij[SLOTS];
#pragma unroll
    for (int sl = 0; sl < SLOTS; ++sl) {
      const int t = wave - kChE + kChU * sl;
      int i0 = 0, j0 = 0;
      if (t < ntiles) tile_of(t, T, i0, j0);
      tij[sl] = __builtin_amdgcn_readfirstlane(t < ntiles ? i0 + 256 * j0 : -1);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double v = 0.0;
        if (t < ntiles) {
          const int row = i0 * kTile + lr + 4 * r, col = j0 * kTile + lc;
          v = (row < d && col < d) ? G[(int64_t)row * ld + col] : (row == col ? 1.0 : 0.0);
        }
        tile[sl][r] = v;
      }
    }
    auto publish = [&](const doublex4& t, int j) {
#pragma unroll
      for (int r = 0; r < 4; ++r) grow[lr + 4 * r][j * kTile + lc] = t[r];
    };
    // G_ij -= R_ki^T R_kj
    auto update = [&](const double (*from)[LD], const double (&f)[4], doublex4& t, int i, int j) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        t = Mfma<double>::mma(from[ks * 4 + lr][i * kTile + lc] * f[ks], from[ks * 4 + lr][j * kTile + lc], t);
    };
    // the first slot of this wave whose tile is in row i or below
    auto first = [&](int i) {
      const int t = i < T ? i * T - i * (i - 1) / 2 : ntiles;
      return (t - (wave - kChE) + kChU - 1) / kChU;  // (t >= 0; a negative numerator gives 0)
    };
    // block row k of R, L_kk^-T's block to memory
    auto store = [&](int k) {
      const double (*from)[LD] = slab[k & 1];
      const double* scale = rsd[k & 1];
      const int u = wave - kChE;
      double* Rk = R + (int64_t)k * kTile * ld;
      for (int c = (u >> 2) * kWave + lane; c < dp; c += (kChU / 4) * kWave) {
        const bool in_diag = (c >> 4) == k;
        const int from_c = in_diag ? RD + lc : c;
        double v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = 4 * (u & 3) + q;
          v[q] = from[row][from_c] * scale[row];
          v[q] = in_diag && lc == row ? diag[k & 1][row] : v[q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = 4 * (u & 3) + q;
          Rk[(int64_t)row * ld + c] = c < k * kTile + (in_diag ? row : 0) ? 0.0 : v[q];
        }
      }
      if (u >= kChU - 4) {
        const int e = (u - (kChU - 4)) * kWave + lane;
        Rinv16[(int64_t)k * kTile * kTile + e] = from[e & 15][XD + (e >> 4)] * scale[e & 15];
      }
    };
#pragma unroll
    for (int sl = 0; sl < SLOTS; ++sl)
      if (tij[sl] >= 0 && (tij[sl] & 255) == 0) publish(tile[sl], tij[sl] >> 8);
    double f[4] = {0.0, 0.0, 0.0, 0.0};  // -1/D of the step, for this lane's rows
    lds_barrier();
    for (int k = 0; k < T; ++k) {
      // opaque to the optimizer: otherwise the LDS addresses of every slot are
      // hoisted out of this loop and held in vector registers the tiles need
#pragma unroll
      for (int sl = 0; sl < SLOTS; ++sl) asm volatile("" : "+s"(tij[sl]));
      // rows are in order, so the tiles of rows > k are the slots from first(k + 1)
      // on, those of row k + 1 (at most two) the ones before first(k + 2)
      const int s1 = first(k + 1), s2 = first(k + 2);
      if (k > 0) {  // the rest of step k - 1, while row k is eliminated
        // (half of the waves store first, so that the matrix cores stay busy)
        if (wave & 1) store(k - 1);
#pragma unroll
        for (int g = 0; g < SLOTS; g += 3)
          if (g + 3 > s1) {
#pragma unroll
            for (int sl = g; sl < min(g + 3, SLOTS); ++sl)
              if (sl >= s1 && tij[sl] >= 0) update(slab[(k - 1) & 1], f, tile[sl], tij[sl] & 255, tij[sl] >> 8);
          }
        if (!(wave & 1)) store(k - 1);
      }
      lds_barrier();  // R's block row k is in slab[k & 1]
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) f[ks] = nrd[k & 1][ks * 4 + lr];
#pragma unroll
      for (int g = 0; g < SLOTS; g += 3)  // (by threes: a skipped branch is a tenth of a tile's update)
        if (g + 3 > s1 && g < s2) {
#pragma unroll
          for (int sl = g; sl < min(g + 3, SLOTS); ++sl)
            if (sl >= s1 && sl < s2) {
              update(slab[k & 1], f, tile[sl], k + 1, tij[sl] >> 8);
              publish(tile[sl], tij[sl] >> 8);
            }
        }
      lds_barrier();  // G's block row k + 1 is in grow
    }
    store(T - 1);
    return;
  }

  // ---- block rows: lane group g of wave w takes the columns of tile k + 4 w + g,
  // the first of all those of the identity (for R_kk^-T) ----
  const int idx = 4 * wave + lr;
  int ndep = 0;
  lds_barrier();
  for (int k = 0; k < T; ++k) {
    double (*sk)[LD] = slab[k & 1];
    double dv = 0.0;
    const double thr = tol * Gdiag[k * kTile + lc];
    if (4 * wave < T - k) {
      __builtin_amdgcn_s_setprio(3);  // the elimination is the chain of the whole factorization
      const bool mine = idx < T - k;
      int c = lc;  // (opaque: what is computed from it is not kept in registers from step to step)
      asm volatile("" : "+v"(c));
      const double* dcol = &grow[0][k * kTile + c];
      const double* wcol = &grow[0][(k + (mine ? idx : 0)) * kTile + c];
      double* put = &sk[0][idx == 0 ? XD + c : (mine ? (k + idx) * kTile + c : ZD + c)];
      double S[kTile], W[kTile], rv = 0.0;
      auto fetch = [&] {
#pragma unroll
        for (int p = 0; p < kTile; ++p) {
          S[p] = dcol[p * LD];
          W[p] = wcol[p * LD];
        }
#pragma unroll
        for (int p = 0; p < kTile; ++p) W[p] = idx == 0 ? (p == c ? 1.0 : 0.0) : W[p];
      };
      fetch();
      eliminate<false, LD>(S, W, dv, rv, thr, c, idx > 0, put, &sk[0][RD + c]);
      if (__builtin_expect(__any(!(dv > thr)), 0)) {  // a dependent column
        fetch();
        eliminate<true, LD>(S, W, dv, rv, thr, c, idx > 0, put, &sk[0][RD + c]);
      }
      if (wave == 0 && lr == 0) nrd[k & 1][lc] = rv;
      __builtin_amdgcn_s_setprio(0);
    }
    lds_barrier();  // R's block row k is in slab[k & 1]
    if (wave == 0) {  // (read after the next barrier)
      const bool dep = !(dv > thr);
      const double rs = dep ? 1.0 : rsqrt_f64(dv);
      if (lr == 0) {
        rsd[k & 1][lc] = rs;
        diag[k & 1][lc] = dep ? 1.0 : dv * rs;
        flags[k * kTile + lc] = dep;
      }
      ndep += __popcll(__ballot(dep) & 0xffff);
    }
    lds_barrier();  // G's block row k + 1 is in grow
  }
  // the explicit R^-1 (formed next by the inverse kernel) serves the solve
  // unless a column was dependent
  if (tid == 0) {
    if (!block) *mode = ndep ? 0 : 1;
    else if (ndep) *mode = 0;
    if (ndep) {
      atomicAdd(&info->completed_cols, ndep);
      atomicCAS(&info->breakdown_pass, 0, pass_id);
    }
  }
}

template <int TMAX>
__global__ __launch_bounds__(kChThreads) void chol_kernel(const double* __restrict__ G, int ld, int d, int dp,
                                                    double* __restrict__ R, double* __restrict__ Rinv16,
                                                    int32_t* __restrict__ flags, DevInfo* info, int pass_id,
                                                    double tol, double fast_tol, const double* __restrict__ esq,
                                                    int nesq, int32_t* __restrict__ mode,
                                                    double* __restrict__ Xfull, const double* __restrict__ gdiag0,
                                                    int block) {
  chol_body<TMAX>(G, ld, d, dp, R, Rinv16, flags, info, pass_id, tol, fast_tol, esq, nesq, mode, Xfull, gdiag0,
                       block, blockIdx.x, gridDim.x);
}

// Many independent matrices in one launch (argument table in device
// memory): workgroups start[p] .. start[p + 1] - 1 belong to matrix p.
struct CholRecArgs {
  const double* G;
  double* R;
  double* Rinv16;
  int32_t* flags;
  DevInfo* info;
  const double* esq;
  int32_t* mode;
  double* Xfull;
  const double* gdiag0;
  double tol, fast_tol;
  int ld, d, dp, pass_id, nesq, block;
};

template <int TMAX>
__global__ __launch_bounds__(kChThreads) void chol_grouped(const CholRecArgs* __restrict__ a,
                                                        const int* __restrict__ start, int count) {
  const int p = group_find(start, count, blockIdx.x);
  const CholRecArgs g = a[p];
  chol_body<TMAX>(device_ptr(g.G), g.ld, g.d, g.dp, device_ptr(g.R), device_ptr(g.Rinv16), device_ptr(g.flags),
                  device_ptr(g.info), g.pass_id, g.tol, g.fast_tol, device_ptr(g.esq), g.nesq, device_ptr(g.mode),
                  device_ptr(g.Xfull), device_ptr(g.gdiag0), g.block, (int)blockIdx.x - start[p],
                  start[p + 1] - start[p]);
}

template <int TMAX>
void chol_grouped_launch(const void* args, const int* start, int count, unsigned blocks, hipStream_t s) {
  hipLaunchKernelGGL((chol_grouped<TMAX>), dim3(blocks), dim3(kChThreads), 0, s, (const CholRecArgs*)args,
                     start, count);
}

// ---------------- d > 256: blocked over register-sized diagonal blocks ----------------
// The matrix is cut into nb diagonal blocks of at most 256 columns.  For
// each block b in turn: R_bb = chol(G_bb) (chol_kernel in block mode), then,
// unless b is the last block, X_bb = R_bb^-1 (inverse kernel),
// R_b,r = X_bb^T G_b,r for the columns r after the block (rows of dependent
// columns zero), and the trailing update G_r,r -= R_b,r^T R_b,r (both
// triangles, in place).  The panel and update spread over many workgroups;
// only the diagonal blocks run in one.

// Fast path of the second pass (all workgroups), else the original diagonal
// into gd0 (for the dependence test of later blocks) and *mode = 1.
__device__ __attribute__((always_inline)) inline void chol_prep_body(const double* __restrict__ G, int d, int dp,
                                                                     double* __restrict__ R,
                                                                     double* __restrict__ Rinv16,
                                                                     int32_t* __restrict__ flags, double fast_tol,
                                                                     const double* __restrict__ esq, int nesq,
                                                                     int32_t* __restrict__ mode,
                                                                     double* __restrict__ Xfull,
                                                                     double* __restrict__ gd0, int bid, int nblk) {
  __shared__ double red[16];
  if (fast_tol > 0.0 && chol_fast_path(G, d, dp, R, Rinv16, flags, fast_tol, esq, nesq, mode, Xfull, red, 16, bid, nblk))
    return;
  if (bid != 0) return;
  for (int i = threadIdx.x; i < dp; i += blockDim.x) gd0[i] = (i < d) ? G[(int64_t)i * dp + i] : 1.0;
  if (threadIdx.x == 0) *mode = 1;
}

__global__ __launch_bounds__(1024) void chol_prep_kernel(const double* __restrict__ G, int d, int dp,
                                                      double* __restrict__ R, double* __restrict__ Rinv16,
                                                      int32_t* __restrict__ flags, double fast_tol,
                                                      const double* __restrict__ esq, int nesq,
                                                      int32_t* __restrict__ mode, double* __restrict__ Xfull,
                                                      double* __restrict__ gd0) {
  chol_prep_body(G, d, dp, R, Rinv16, flags, fast_tol, esq, nesq, mode, Xfull, gd0, blockIdx.x, gridDim.x);
}

struct CholPrepArgs {
  const double* G;
  double* R;
  double* Rinv16;
  int32_t* flags;
  const double* esq;
  int32_t* mode;
  double* Xfull;
  double* gd0;
  double fast_tol;
  int d, dp, nesq;
};

__global__ __launch_bounds__(1024) void chol_prep_grouped(const CholPrepArgs* __restrict__ a,
                                                       const int* __restrict__ start, int count) {
  const int p = group_find(start, count, blockIdx.x);
  const CholPrepArgs g = a[p];
  chol_prep_body(device_ptr(g.G), g.d, g.dp, device_ptr(g.R), device_ptr(g.Rinv16), device_ptr(g.flags), g.fast_tol,
                 device_ptr(g.esq), g.nesq, device_ptr(g.mode), device_ptr(g.Xfull), device_ptr(g.gd0),
                 (int)blockIdx.x - start[p], start[p + 1] - start[p]);
}

void chol_prep_grouped_launch(const void* args, const int* start, int count, unsigned blocks, hipStream_t s) {
  hipLaunchKernelGGL(chol_prep_grouped, dim3(blocks), dim3(1024), 0, s, (const CholPrepArgs*)args, start, count);
}

// R[b, r] = X_bb^T G[b, r] (one wave per 16 x 16 output tile, float64 MFMA)
// and R[r, b] = 0; X_bb is upper triangular, so tile row I needs only the
// first 16 (I + 1) rows of X_bb and G.
__device__ __attribute__((always_inline)) inline void chol_panel_body(const double* __restrict__ G, int ld, int off,
                                                                      int db, int rest, const double* __restrict__ X,
                                                                      double* __restrict__ R,
                                                                      const int32_t* __restrict__ flags,
                                                                      const int32_t* __restrict__ mode, int bid) {
  if (*mode == 2) return;
  const int nI = db / kTile;
  const int I = bid % nI, J = bid / nI;
  const int lane = threadIdx.x, lr = lane >> 4, lc = lane & 15;
  const double* Xb = X + (int64_t)off * ld + off;
  const double* Gb = G + (int64_t)off * ld + off + db;
  doublex4 acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u] = Mfma<double>::zero();
  const int kend = (I + 1) * kTile;
  for (int t0 = 0; t0 < kend; t0 += kTile) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {  // A[m][kk] = X_bb[t][I*16+m], B[kk][n] = G_b,r[t][J*16+n]
      const int t = t0 + 4 * u + lr;
      acc[u] = Mfma<double>::mma(Xb[(int64_t)t * ld + I * kTile + lc], Gb[(int64_t)t * ld + J * kTile + lc],
                                 acc[u]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = I * kTile + lr + 4 * r, col = J * kTile + lc;
    const double v = ((acc[0][r] + acc[1][r]) + acc[2][r]) + acc[3][r];
    R[(int64_t)(off + row) * ld + off + db + col] = flags[off + row] ? 0.0 : v;
    R[(int64_t)(off + db + col) * ld + off + row] = 0.0;
  }
}

__global__ __launch_bounds__(64) void chol_panel_kernel(const double* __restrict__ G, int ld, int off, int db,
                                                     int rest, const double* __restrict__ X,
                                                     double* __restrict__ R, const int32_t* __restrict__ flags,
                                                     const int32_t* __restrict__ mode) {
  chol_panel_body(G, ld, off, db, rest, X, R, flags, mode, blockIdx.x);
}

struct CholPanelArgs {
  const double* G;
  const double* X;
  double* R;
  const int32_t* flags;
  const int32_t* mode;
  int ld, off, db, rest;
};

__global__ __launch_bounds__(64) void chol_panel_grouped(const CholPanelArgs* __restrict__ a,
                                                      const int* __restrict__ start, int count) {
  const int p = group_find(start, count, blockIdx.x);
  const CholPanelArgs g = a[p];
  chol_panel_body(device_ptr(g.G), g.ld, g.off, g.db, g.rest, device_ptr(g.X), device_ptr(g.R), device_ptr(g.flags),
                  device_ptr(g.mode), (int)blockIdx.x - start[p]);
}

void chol_panel_grouped_launch(const void* args, const int* start, int count, unsigned blocks, hipStream_t s) {
  hipLaunchKernelGGL(chol_panel_grouped, dim3(blocks), dim3(64), 0, s, (const CholPanelArgs*)args, start, count);
}

// G[r, r] -= R[b, r]^T R[b, r] (one wave per 16 x 16 tile of the square
// trailing block, K = db)
__device__ __attribute__((always_inline)) inline void chol_syrk_body(double* __restrict__ G, int ld, int off, int db,
                                                                     int rest, const double* __restrict__ R,
                                                                     const int32_t* __restrict__ mode, int bid) {
  if (*mode == 2) return;
  const int nI = rest / kTile;
  const int I = bid % nI, J = bid / nI;
  const int lane = threadIdx.x, lr = lane >> 4, lc = lane & 15;
  const double* Rb = R + (int64_t)off * ld + off + db;
  doublex4 acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u] = Mfma<double>::zero();
  for (int t0 = 0; t0 < db; t0 += kTile) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + 4 * u + lr;
      acc[u] = Mfma<double>::mma(Rb[(int64_t)t * ld + I * kTile + lc], Rb[(int64_t)t * ld + J * kTile + lc],
                                 acc[u]);
    }
  }
  double* Gt = G + (int64_t)(off + db + I * kTile) * ld + off + db + J * kTile;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    Gt[(int64_t)(lr + 4 * r) * ld + lc] -= ((acc[0][r] + acc[1][r]) + acc[2][r]) + acc[3][r];
}

__global__ __launch_bounds__(64) void chol_syrk_kernel(double* __restrict__ G, int ld, int off, int db, int rest,
                                                    const double* __restrict__ R, const int32_t* __restrict__ mode) {
  chol_syrk_body(G, ld, off, db, rest, R, mode, blockIdx.x);
}

struct CholSyrkArgs {
  double* G;
  const double* R;
  const int32_t* mode;
  int ld, off, db, rest;
};

__global__ __launch_bounds__(64) void chol_syrk_grouped(const CholSyrkArgs* __restrict__ a,
                                                     const int* __restrict__ start, int count) {
  const int p = group_find(start, count, blockIdx.x);
  const CholSyrkArgs g = a[p];
  chol_syrk_body(device_ptr(g.G), g.ld, g.off, g.db, g.rest, device_ptr(g.R), device_ptr(g.mode),
                 (int)blockIdx.x - start[p]);
}

void chol_syrk_grouped_launch(const void* args, const int* start, int count, unsigned blocks, hipStream_t s) {
  hipLaunchKernelGGL(chol_syrk_grouped, dim3(blocks), dim3(64), 0, s, (const CholSyrkArgs*)args, start, count);
}

// One diagonal block (or the whole matrix) of T = db / 16 tile columns, by the
// smallest of three variants that holds it: their T (T + 1) / 2 upper tiles take 5,
// 9 or 12 register slots of each of the 12 waves, and their slabs 75, 105 or 120 KB
// of LDS.
static hipError_t launch_chol_reg(const double* G, int ld, int d, int db, double* R, double* Rinv16,
                                  int32_t* flags, void* info, int pass_id, double tol, double fast_tol,
                                  const double* esq, int nesq, int32_t* mode, double* Xfull, const double* gdiag0,
                                  int block, hipStream_t s) {
  const int T = db / kTile;
  const unsigned grid = (!block && fast_tol > 0.0) ? 16 : 1;  // extra workgroups only help the fast path
  const CholRecArgs a{G, R, Rinv16, flags, (DevInfo*)info, esq, mode, Xfull, gdiag0, tol, fast_tol, ld, d, db, pass_id,
                      nesq, block};
#define RQLP_CHOL_LAUNCH(S)                                                                                        \
  do {                                                                                                             \
    if (!record_launch(&chol_grouped_launch<S>, a, grid))                                                       \
      hipLaunchKernelGGL((chol_kernel<S>), dim3(grid), dim3(kChThreads), 0, s, G, ld, d, db, R, Rinv16, flags,       \
                         (DevInfo*)info, pass_id, tol, fast_tol, esq, nesq, mode, Xfull, gdiag0, block);             \
  } while (0)
  if (T <= 10) RQLP_CHOL_LAUNCH(10);
  else if (T <= 14) RQLP_CHOL_LAUNCH(14);
  else RQLP_CHOL_LAUNCH(16);
#undef RQLP_CHOL_LAUNCH
  return hipGetLastError();
}

hipError_t launch_chol(double* G, int d, int dp, double* R, double* Rinv16, int32_t* flags,
                       void* info, int pass_id, double fast_tol, const double* esq, int nesq,
                       int32_t* mode, double* Xfull, double* gd0, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const double tol = 64.0 * (double)d * 2.220446049250313e-16;
  if (ev0) (void)hipEventRecord(ev0, s);
  hipError_t e = hipSuccess;
  if (dp <= kCholRegMax) {
    e = launch_chol_reg(G, dp, d, dp, R, Rinv16, flags, info, pass_id, tol, fast_tol, esq, nesq, mode, Xfull,
                        nullptr, 0, s);
  } else {
    const unsigned pg = fast_tol > 0.0 ? 16 : 1;
    if (!record_launch(&chol_prep_grouped_launch,
                       CholPrepArgs{G, R, Rinv16, flags, esq, mode, Xfull, gd0, fast_tol, d, dp, nesq}, pg))
      hipLaunchKernelGGL(chol_prep_kernel, dim3(pg), dim3(1024), 0, s, G, d, dp, R, Rinv16, flags, fast_tol, esq, nesq,
                         mode, Xfull, gd0);
    const int T = dp / kTile;
    const int nb = (int)ceil_div(T, kCholRegMax / kTile);
    int t0 = 0;
    for (int b = 0; b < nb && e == hipSuccess; ++b) {
      const int tb = (T - t0) / (nb - b);  // equal shares, the larger ones first
      const int tbs = tb + ((T - t0) % (nb - b) ? 1 : 0);
      const int off = t0 * kTile, db = tbs * kTile, rest = dp - off - db;
      const int dl = std::max(0, std::min(d - off, db));
      e = launch_chol_reg(G + (int64_t)off * dp + off, dp, dl, db, R + (int64_t)off * dp + off,
                          Rinv16 + (int64_t)t0 * kTile * kTile, flags + off, info, pass_id, tol, 0.0, esq, nesq,
                          mode, Xfull, gd0 + off, 1, s);
      if (e == hipSuccess && rest > 0) {
        e = launch_trinv_block(R + (int64_t)off * dp + off, Rinv16 + (int64_t)t0 * kTile * kTile, dp, tbs, mode,
                               Xfull + (int64_t)off * dp + off, s);
        if (e != hipSuccess) break;
        const unsigned npb = (unsigned)(tbs * (rest / kTile)), nsb = (unsigned)((rest / kTile) * (rest / kTile));
        if (!record_launch(&chol_panel_grouped_launch, CholPanelArgs{G, Xfull, R, flags, mode, dp, off, db, rest}, npb))
          hipLaunchKernelGGL(chol_panel_kernel, dim3(npb), dim3(kWave), 0, s, G, dp, off, db, rest, Xfull, R, flags,
                             mode);
        if (!record_launch(&chol_syrk_grouped_launch, CholSyrkArgs{G, R, mode, dp, off, db, rest}, nsb))
          hipLaunchKernelGGL(chol_syrk_kernel, dim3(nsb), dim3(kWave), 0, s, G, dp, off, db, rest, R, mode);
        e = hipGetLastError();
      }
      t0 += tbs;
    }
  }
  if (ev1) (void)hipEventRecord(ev1, s);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace rqlp
