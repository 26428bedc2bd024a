// SVD of the small d x d factor (Remark 1 of Section III-B: an SVD of the
// middle factor turns RU-QLP into an SVD-like decomposition), float64,
// d <= 544, by one-sided (Hestenes) Jacobi with column blocks.
//
// The columns of X = M are rotated in pairs until they are mutually
// orthogonal: X V-bar = U-bar Sigma, with V-bar the product of the
// rotations.  A rotation of columns p, q zeroes their inner product:
//     zeta = (||x_q||^2 - ||x_p||^2) / (2 x_p.x_q),
//     t = sign(zeta) / (|zeta| + sqrt(1 + zeta^2)),  c = 1 / sqrt(1 + t^2),  s = c t,
//     x_p <- c x_p - s x_q,   x_q <- s x_p + c x_q.
// Each column carries its column of V-bar below it (length 2 dp: x_j, then
// v_j, starting from e_j).  The padded columns (dp a multiple of 16) are split
// into nb blocks of 16.  One step pairs every block with another (a round-robin
// tournament over the blocks, so a sweep of nb - 1 steps meets every pair of
// blocks; with nb odd one block meets none).
//
// A step on the 32 columns of a block pair is a contraction, a small
// eigenproblem and a contraction: the Gram matrix G = X^T X on the matrix cores,
// the rotations on G alone (J^T G J, 16 disjoint pairs a round, all 32 x 32
// values in one pass), their product J kept beside it, and X <- X J, V <- V J
// on the matrix cores.  At a sweep's first step every pair of the 32 columns is
// met (15 rounds within the blocks, 16 across), at later steps the 256 pairs
// across.  G is computed afresh from X at every step, so that its rounding
// errors reach no further than one step's choice of angles, and any angle is an
// exact rotation.  A pair counts as orthogonal when
// |x_p.x_q| <= dp eps ||x_p|| ||x_q||; a sweep whose fresh G's show no other
// ends the iteration.
//
// What bounds it is latency: at most 17 pairs of blocks at once (of 256 CUs), a
// chain of rounds in each and a grid barrier after each step.  Hence 16 columns
// to a block (half the steps of 8, at the same number of rounds), rounds that
// touch 32 x 32 values in LDS instead of 2 dp x 32 (about 860 cycles each, with
// one barrier, against a reduction over a column and its update), the angles
// from the hardware's estimates and one Newton step, J's accumulation one round
// behind on waves of its own, and V's product one step behind on workgroups of its
// own.  At d = 210 (10 sweeps of 13 steps) a step takes 35 thousand cycles: load 4,
// G 6, rounds 14, X J 5, barrier 5.  All sweeps run in one cooperative launch.
// Measured against blocks of 8 columns rotated in place (the whole call, L
// factors): d = 100 1204 -> 981 us, 210 3270 -> 2141, 320 6381 -> 3842, 400 9108 ->
// 5683; singular values nearer to 64-bit references, vectors as near.
//
// Finally sigma_j = ||x_j||, the columns are sorted by descending sigma
// (stable), u_j = x_j / sigma_j (zero when sigma_j = 0), and each pair of vectors
// is signed so that the entry of largest magnitude of v_j is positive (the first
// such entry on ties).
#include "common.h"
#include "kernels.h"

namespace rqlp {

constexpr int kSvW = 16;              // columns per block
constexpr int kSvCols = 2 * kSvW;     // columns of a block pair
constexpr int kSvThreads = 512;

inline size_t svd_align(size_t b) { return (b + 255) & ~(size_t)255; }

// 1/sqrt(x) for finite positive x: the hardware estimate (relative error about
// 2^-24) with one third-order correction, y (1 + e/2 + 3 e^2/8) with e = 1 - x
// y^2, within an ulp or two like two Newton steps but with a shorter dependent
// chain on the critical path of every rotation.
__device__ __forceinline__ double rsqrt_nr(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// XV: dp columns of length 2 dp, column j = (M[:, j] zero-padded, e_j).
template <typename T>
__global__ __launch_bounds__(256) void svd_init_kernel(const T* __restrict__ M, int64_t ldm, int d, int dp,
                                                       double* __restrict__ XV, int32_t* __restrict__ flags,
                                                       int nflags, unsigned* __restrict__ counter) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < (int64_t)dp * 2 * dp) {
    const int j = (int)(e / (2 * dp)), r = (int)(e % (2 * dp));
    XV[e] = r < dp ? ((j < d && r < d) ? (double)M[(int64_t)r * ldm + j] : 0.0) : (r - dp == j ? 1.0 : 0.0);
  }
  if (e < nflags) flags[e] = 0;
  if (e == 0) *counter = 0;
}

// ---------------------------------------------------------------------------
// The sweeps.
constexpr int kGS = kSvCols + 1;  // LDS row stride of G and J (doubles)
constexpr int kXPad = 2;          // LDS column stride of X: dp + kXPad (16-byte aligned columns)

// Pair i (0 .. 15) of round r: columns u < v of the block pair's 32.  Rounds
// 0 .. 15 pair every column of the first block with every one of the second;
// rounds 16 .. 30 (a sweep's first step) play a round-robin within each block.
__device__ inline void svd_pair(int r, int i, int& u, int& v) {
  if (r < kSvW) {
    u = i;
    v = kSvW + ((i + r) & (kSvW - 1));
  } else {
    constexpr int n = kSvW - 1;
    const int k = r - kSvW, h = i >> 3, j = i & 7;  // block h, pair j of 8
    int x = j == 0 ? 0 : 1 + (j - 1 + k) % n, y = 1 + (n - 1 - j + k) % n;
    if (x > y) {
      const int t = x;
      x = y;
      y = t;
    }
    u = kSvW * h + x;
    v = kSvW * h + y;
  }
}

// A value from the next lane of each row of 16 (cyclic).
__device__ __forceinline__ double row_next(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x12F, 0xf, 0xf, false);  // row_ror:15
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x12F, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Whether columns with squared norms a, d and inner product b are still to be
// made orthogonal: |b| sqrt(a d)^-1 above working accuracy 1 / itol.  (b, not a d,
// takes the factor: a square of a negligible b leaves the range first.)  Never for
// b = 0, also where the rounding of earlier rotations left a or d negative.
__device__ __forceinline__ bool svd_needs(double a, double b, double d, double itol) {
  const double w = b * itol;
  return b != 0.0 && w * w > a * d;
}

// The rotation x_u <- c x_u - s x_v, x_v <- s x_u + c x_v that does it: with h =
// d - a and r = sqrt(h^2 + 4 b^2), t = 2 sign(h) b / (|h| + r) (the t above),
// c = 1 / sqrt(1 + t^2), s = c t; c = 1, s = 0 where none is needed.  t is taken
// from the hardware estimates (relative error about 2^-23) with one Newton step on
// b t^2 + h t - b = 0, whose derivative at the root is +-r: three FMAs, an error of
// 2^-44.  (Without it the last rotations leave 2^-22 of b, up to the bound of
// svd_needs, and nearby singular vectors are that much less accurate.)  c takes one
// Newton step more than its estimate's correction: what c and s are off by is a
// factor of the columns' norms, and a column takes some ten rotations with every
// other (singular values at d = 320: relative error 4.2e-14, 6.7e-14 without, for
// 1.5 % of the time; scaling c and s to c^2 + s^2 = 1 gives 1.6e-15 for 6 %).
// Values whose squares leave the range are scaled first (a whole wave at once;
// rare).
__device__ __forceinline__ void svd_rotation(double a, double b, double d, double itol, double& c, double& s) {
  double h = d - a, b2 = b + b;
  double x = fma(b2, b2, h * h);
  const bool rot = svd_needs(a, b, d, itol);
  if (__builtin_expect(__any(rot && !(x > 1e-290 && x < 1e290)), 0)) {
    const int e = -__builtin_amdgcn_frexp_exp(fabs(h) + fabs(b2));
    h = __builtin_amdgcn_ldexp(h, e);
    b2 = __builtin_amdgcn_ldexp(b2, e);
    x = fma(b2, b2, h * h);
  }
  const double y = __builtin_amdgcn_rsq(x), hb = 0.5 * b2;
  const double t0 = (h < 0.0 ? -b2 : b2) * __builtin_amdgcn_rcp(fma(x, y, fabs(h)));
  const double f = fma(fma(hb, t0, h), t0, -hb);
  const double t = fma(h < 0.0 ? f : -f, y, t0);
  const double q = fma(t, t, 1.0), z0 = rsqrt_nr(q);
  const double z = fma(0.5 * z0, fma(-q * z0, z0, 1.0), z0);
  c = rot ? z : 1.0;
  s = rot ? z * t : 0.0;
}

// Grid-wide barrier of the resident workgroups (a cooperative launch); `phase`
// counts this workgroup's barriers.  Every wave's stores are out before the
// workgroup arrives; one thread writes them back beyond this chiplet's L2 and
// afterwards discards what its caches hold of the others'.
__device__ inline void svd_grid_barrier(unsigned* counter, unsigned nwg, unsigned phase) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned target = nwg * phase;
    while (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
}

// Blocks of pair `pr` at `step` of the tournament over nbe (even) positions;
// a block index of nb or more is the bye of an odd nb.
__device__ inline void svd_blocks(int pr, int step, int nbe, int& ba, int& bb) {
  const int pb = nbe - 1 - pr;
  ba = pr == 0 ? 0 : 1 + (pr - 1 + step) % (nbe - 1);
  bb = 1 + (pb - 1 + step) % (nbe - 1);
}

// One step for block pair `pr`: its 32 x-columns, their Gram matrix, the
// rotations on the Gram matrix (accumulated in J), X <- X J, and J for the
// workgroup that applies it to V.  PING: two copies of G in LDS, one barrier
// per round; else one copy and two barriers (the widest matrices).
template <bool PING>
__device__ __attribute__((always_inline)) inline void svd_step(double* __restrict__ XV, int dp, int nb, int nbe, int pr,
                                                              int step, int sweep, int32_t* __restrict__ flags,
                                                              double itol, double* smem, double2* cs,
                                                              double* __restrict__ Jout, int32_t* __restrict__ jflag) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane >> 4, lc = lane & 15;
  const int xs = dp + kXPad;
  double* Xs = smem;                       // [32][xs]
  double* G = smem + kSvCols * xs;         // [PING ? 2 : 1][32][kGS]
  double* J = G + (PING ? 2 : 1) * kSvCols * kGS;  // [32][kGS]
  int ba, bb;
  svd_blocks(pr, step, nbe, ba, bb);
  // the bye's block has no columns: nothing across, pairs within at step 0
  const bool bye = ba >= nb || bb >= nb;
  if (bye && step > 0) {
    if (tid == 0) *jflag = 0;
    return;
  }
  const int len = 2 * dp;
  auto column = [&](int c) { return c < kSvW ? ba * kSvW + c : bb * kSvW + c - kSvW; };

  // ---- the x-columns into LDS (16 bytes per load, batches in flight) ----
  {
    const int hv = dp / 2, total = kSvCols * hv;  // double2 values
    constexpr int kLd = 8;
    for (int e0 = tid; e0 < total; e0 += kLd * kSvThreads) {
      double2 v[kLd];
#pragma unroll
      for (int j = 0; j < kLd; ++j) {
        const int e = e0 + j * kSvThreads;
        v[j] = double2{0.0, 0.0};
        if (e < total) {
          const int c = e / hv, o = e - c * hv, col = column(c);
          if (col < nb * kSvW) v[j] = *reinterpret_cast<const double2*>(XV + (int64_t)col * len + 2 * o);
        }
      }
#pragma unroll
      for (int j = 0; j < kLd; ++j) {
        const int e = e0 + j * kSvThreads;
        if (e < total) {
          const int c = e / hv, o = e - c * hv;
          *reinterpret_cast<double2*>(Xs + c * xs + 2 * o) = v[j];
        }
      }
    }
  }
  __syncthreads();

  // ---- G = X^T X: waves 0 .. 3 (one per SIMD, which the float64 MFMAs fill)
  // take every fourth group of 4 rows, then their sums are added in a tree ----
  {
    doublex4 g[3];  // blocks (0,0), (0,1), (1,1)
#pragma unroll
    for (int t = 0; t < 3; ++t) g[t] = Mfma<double>::zero();
    double* part = G;  // [2 or 3][3][256], before G holds anything
    if (wave < 4) {  // (the next group's values are read before this one's products)
      const double* x0 = Xs + lc * xs + lr;
      const double* x1 = Xs + (lc + kSvW) * xs + lr;
      double a0 = x0[4 * wave], a1 = x1[4 * wave];
      for (int k = 4 * wave; k < dp; k += 16) {
        const int kn = k + 16 < dp ? k + 16 : k;
        const double n0 = x0[kn], n1 = x1[kn];
        g[0] = Mfma<double>::mma(a0, a0, g[0]);
        g[1] = Mfma<double>::mma(a0, a1, g[1]);
        g[2] = Mfma<double>::mma(a1, a1, g[2]);
        a0 = n0;
        a1 = n1;
      }
    }
    auto put = [&](int slot) {
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[(slot * 3 + t) * 256 + r * 64 + lane] = g[t][r];
    };
    auto take = [&](int slot) {
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) g[t][r] += part[(slot * 3 + t) * 256 + r * 64 + lane];
    };
    if (wave == 2 || wave == 3) put(wave - 2);
    if (PING && wave == 1) put(2);  // (three slots fit beside two copies of G)
    __syncthreads();
    if (PING) {
      if (wave == 0) {
        take(2);
        take(0);
        take(1);
      }
    } else {
      if (wave < 2) take(wave);
      __syncthreads();
      if (wave == 1) put(0);
      __syncthreads();
      if (wave == 0) take(0);
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = lr + 4 * r;
        G[m * kGS + lc] = g[0][r];
        G[m * kGS + kSvW + lc] = g[1][r];
        G[(kSvW + lc) * kGS + m] = g[1][r];
        G[(kSvW + m) * kGS + kSvW + lc] = g[2][r];
      }
    }
    for (int e = tid; e < kSvCols * kSvCols; e += kSvThreads) J[(e >> 5) * kGS + (e & 31)] = (e >> 5) == (e & 31);
  }
  __syncthreads();

  // ---- does any pair of this step need a rotation? ----
  {
    bool need = false;
    for (int e = tid; e < kSvCols * kSvCols; e += kSvThreads) {
      const int u = e >> 5, v = e & 31;
      if (u < v && (step == 0 || (u < kSvW && v >= kSvW)))
        need |= svd_needs(G[u * kGS + u], G[u * kGS + v], G[v * kGS + v], itol);
    }
    if (__syncthreads_or(need) == 0) {
      if (tid == 0) *jflag = 0;
      return;
    }
  }
  // columns that are not finite (or whose norms aren't) are left out: the same
  // bits in every wave
  const double gd = G[(lane & 31) * kGS + (lane & 31)];
  const unsigned skip = (unsigned)__ballot(!(gd < __builtin_inf()));
  if (__builtin_expect(skip != 0, 0)) {
    __syncthreads();  // (every wave has read the diagonal)
    for (int e = tid; e < kSvCols * kSvCols; e += kSvThreads)
      if (((skip >> (e >> 5)) | (skip >> (e & 31))) & 1) G[(e >> 5) * kGS + (e & 31)] = 0.0;
    for (int e = tid; e < kSvCols * dp; e += kSvThreads)
      if ((skip >> (e / dp)) & 1) Xs[(e / dp) * xs + e % dp] = 0.0;
    __syncthreads();
  }

  // ---- rounds: threads 0 .. 255 own the 2 x 2 blocks (pair i, pair j) of G;
  // threads 256 .. 511 rows 2 i, 2 i + 1 of J, one round behind, with the
  // rotations the first write ----
  int cur = 0;
  auto g_round = [&](int r, int par) {
    const double* Gr = G + cur * kSvCols * kGS;
    double* Gw = PING ? G + (cur ^ 1) * kSvCols * kGS : G;
    const int i = tid >> 4, j = tid & 15;
    int ui, vi, uj, vj;
    svd_pair(r, i, ui, vi);
    svd_pair(r, j, uj, vj);
    const double ai = Gr[ui * kGS + ui], bi = Gr[ui * kGS + vi], di = Gr[vi * kGS + vi];
    const double aj = Gr[uj * kGS + uj], bj = Gr[uj * kGS + vj], dj = Gr[vj * kGS + vj];
    const double a = Gr[ui * kGS + uj], b = Gr[ui * kGS + vj], c = Gr[vi * kGS + uj], d = Gr[vi * kGS + vj];
    double ci, si, cj, sj;
    svd_rotation(ai, bi, di, itol, ci, si);
    svd_rotation(aj, bj, dj, itol, cj, sj);
    if (i == j) cs[par * kSvW + i] = double2{ci, si};
    const double t1 = ci * a - si * c, t2 = ci * b - si * d, t3 = si * a + ci * c, t4 = si * b + ci * d;
    if (!PING) __syncthreads();
    Gw[ui * kGS + uj] = cj * t1 - sj * t2;
    Gw[ui * kGS + vj] = sj * t1 + cj * t2;
    Gw[vi * kGS + uj] = cj * t3 - sj * t4;
    Gw[vi * kGS + vj] = sj * t3 + cj * t4;
  };
  const int jrow = 2 * ((tid >> 4) & 15), jp = tid & 15;
  double* J0 = J + jrow * kGS;
  double* J1 = J0 + kGS;
  const bool forg = tid < 256;
  if (step == 0) {  // within the blocks (J through LDS)
    auto j_round = [&](int r, int par) {
      int u, v;
      svd_pair(r, jp, u, v);
      const double2 w = cs[par * kSvW + jp];
      const double p0 = J0[u], q0 = J0[v], p1 = J1[u], q1 = J1[v];
      J0[u] = w.x * p0 - w.y * q0;
      J0[v] = w.y * p0 + w.x * q0;
      J1[u] = w.x * p1 - w.y * q1;
      J1[v] = w.y * p1 + w.x * q1;
    };
    for (int k = 0; k < kSvW - 1; ++k) {
      if (forg) {
        g_round(kSvW + k, k & 1);
      } else {
        if (k > 0) j_round(kSvW + k - 1, (k - 1) & 1);
        if (!PING) __syncthreads();
      }
      __syncthreads();
      if (PING) cur ^= 1;
    }
    if (!forg) j_round(2 * kSvW - 2, (kSvW - 2) & 1);
    __syncthreads();
  }
  // across the blocks: pair j's second column moves one on from round to
  // round, so J's values stay in registers and pass from lane to lane
  double p0 = J0[jp], q0 = J0[kSvW + jp], p1 = J1[jp], q1 = J1[kSvW + jp];
  auto j_cross = [&](int par) {
    const double2 w = cs[par * kSvW + jp];
    const double n0 = w.x * p0 - w.y * q0, m0 = w.y * p0 + w.x * q0;
    const double n1 = w.x * p1 - w.y * q1, m1 = w.y * p1 + w.x * q1;
    p0 = n0;
    p1 = n1;
    q0 = row_next(m0);
    q1 = row_next(m1);
  };
  const int cross = bye ? 0 : kSvW;
  for (int k = 0; k < cross; ++k) {
    if (forg) {
      g_round(k, k & 1);
    } else {
      if (k > 0) j_cross((k - 1) & 1);
      if (!PING) __syncthreads();
    }
    __syncthreads();
    if (PING) cur ^= 1;
  }
  if (!forg && !bye) {
    j_cross((kSvW - 1) & 1);
    J0[jp] = p0;
    J0[kSvW + jp] = q0;
    J1[jp] = p1;
    J1[kSvW + jp] = q1;
  }
  __syncthreads();

  // ---- J to memory, X <- X J as J^T X (rows of X along the lanes, so that the
  // stores are runs of 16 values of a column) ----
  for (int e = tid; e < kSvCols * kSvCols; e += kSvThreads) Jout[e] = J[(e >> 5) * kGS + (e & 31)];
  if (tid == 0) {
    *jflag = 1;
    flags[sweep] = 1;
  }
  double ja[2][8];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) ja[m][ks] = J[(4 * ks + lr) * kGS + kSvW * m + lc];
  for (int row0 = 16 * wave; row0 < dp; row0 += 16 * (kSvThreads / 64)) {
    doublex4 acc[2];
    acc[0] = acc[1] = Mfma<double>::zero();
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const double x = Xs[(4 * ks + lr) * xs + row0 + lc];
      acc[0] = Mfma<double>::mma(ja[0][ks], x, acc[0]);
      acc[1] = Mfma<double>::mma(ja[1][ks], x, acc[1]);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int col = column(kSvW * m + lr + 4 * r);
        if (col < nb * kSvW && !((skip >> (kSvW * m + lr + 4 * r)) & 1)) XV[(int64_t)col * len + row0 + lc] = acc[m][r];
      }
  }
}

// V <- V J for the pair and step whose J is given (the same blocks).
__device__ __attribute__((always_inline)) inline void svd_apply_v(double* __restrict__ XV, int dp, int nb, int nbe,
                                                                  int pr, int step, const double* __restrict__ Jin) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane >> 4, lc = lane & 15;
  int ba, bb;
  svd_blocks(pr, step, nbe, ba, bb);
  const int len = 2 * dp;
  auto column = [&](int c) { return c < kSvW ? ba * kSvW + c : bb * kSvW + c - kSvW; };
  double ja[2][8];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) ja[m][ks] = Jin[(4 * ks + lr) * kSvCols + kSvW * m + lc];
  for (int row0 = 16 * wave; row0 < dp; row0 += 16 * (kSvThreads / 64)) {
    double x[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const int col = column(4 * ks + lr);
      x[ks] = col < nb * kSvW ? XV[(int64_t)col * len + dp + row0 + lc] : 0.0;
    }
    doublex4 acc[2];
    acc[0] = acc[1] = Mfma<double>::zero();
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      acc[0] = Mfma<double>::mma(ja[0][ks], x[ks], acc[0]);
      acc[1] = Mfma<double>::mma(ja[1][ks], x[ks], acc[1]);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int col = column(kSvW * m + lr + 4 * r);
        if (col < nb * kSvW) XV[(int64_t)col * len + dp + row0 + lc] = acc[m][r];
      }
  }
}

// Every sweep, in one cooperative launch of 2 np workgroups (np = ceil(nb / 2)
// block pairs): the first np rotate X, the others apply each step's J to V one
// step later.  Jbuf: [2][np][32 x 32], jflags: [2][np], by the step's parity.
template <bool PING>
__global__ __launch_bounds__(kSvThreads) void svd_sweeps_kernel(double* __restrict__ XV, int dp, int nb,
                                                                int32_t* __restrict__ flags, int max_sweeps,
                                                                double itol, double* __restrict__ Jbuf,
                                                                int32_t* __restrict__ jflags,
                                                                unsigned* __restrict__ counter) {
  extern __shared__ __attribute__((aligned(16))) double svd_smem[];
  __shared__ double2 cs[2 * kSvW];  // rotations of two rounds
  const int nbe = (nb + 1) & ~1, np = nbe / 2;
  const bool forx = (int)blockIdx.x < np;
  const int pr = forx ? blockIdx.x : blockIdx.x - np;
  unsigned phase = 0;
  int prev = -1, par = 0;  // the step before (V's), parity of this one
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    for (int step = 0; step < nbe - 1; ++step) {
      if (forx)
        svd_step<PING>(XV, dp, nb, nbe, pr, step, sweep, flags, itol, svd_smem, cs,
                       Jbuf + (int64_t)(par * np + pr) * kSvCols * kSvCols, jflags + par * np + pr);
      else if (prev >= 0 && jflags[(par ^ 1) * np + pr])
        svd_apply_v(XV, dp, nb, nbe, pr, prev, Jbuf + (int64_t)((par ^ 1) * np + pr) * kSvCols * kSvCols);
      svd_grid_barrier(counter, 2 * np, ++phase);  // the next step reads columns other workgroups wrote
      prev = step;
      par ^= 1;
    }
    if (flags[sweep] == 0) break;  // the same value for every workgroup after the barrier
  }
  if (!forx && jflags[(par ^ 1) * np + pr])
    svd_apply_v(XV, dp, nb, nbe, pr, prev, Jbuf + (int64_t)((par ^ 1) * np + pr) * kSvCols * kSvCols);
}

// sigma_j, the sign of each pair and the descending order (one workgroup):
// sig[o], src[o] (the column that goes to place o) and sgn[o].  Columns that are
// not a number come last, so that src is a permutation whatever the input holds.
__global__ __launch_bounds__(1024) void svd_order_kernel(const double* __restrict__ XV, int d, int dp, const int32_t* __restrict__ flags,
                                                         int nflags, double* __restrict__ sig_out,
                                                         int32_t* __restrict__ src, double* __restrict__ sgn_out,
                                                         DevInfo* __restrict__ info) {
  __shared__ double sig[kDMax];
  __shared__ double sgn[kDMax];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int j = wave; j < d; j += 16) {
    const double* X = XV + (int64_t)j * 2 * dp;  // x_j, then v_j
    double ss = 0.0, best = -1.0;
    int bi = 0;
    for (int r = lane; r < d; r += 64) {
      const double x = X[r];
      ss = fma(x, x, ss);
      const double v = fabs(X[dp + r]);
      if (v > best) { best = v; bi = r; }  // first index of the lane's largest
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      ss += __shfl_xor(ss, off);
      const double ob = __shfl_xor(best, off);
      const int oi = __shfl_xor(bi, off);
      if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
    }
    ss = __shfl(ss, 0);
    bi = __shfl(bi, 0);
    if (lane == 0) {
      sig[j] = ss == ss ? sqrt(ss) : -1.0;  // (-1: not a number)
      sgn[j] = X[dp + bi] < 0.0 ? -1.0 : 1.0;
    }
  }
  __syncthreads();
  for (int j = tid; j < d; j += blockDim.x) {
    const double sj = sig[j];
    int rank = 0;
    for (int i = 0; i < d; ++i) rank += (sig[i] > sj) || (sig[i] == sj && i < j);
    sig_out[rank] = sj < 0.0 ? __builtin_nan("") : sj;
    src[rank] = j;
    sgn_out[rank] = sgn[j];
  }
  if (tid == 0 && flags[nflags - 1] != 0) info->status = 5;  // no convergence in nflags sweeps
}

// U[r][o] = sgn x_j[r] / sigma_j (0 if sigma_j = 0), V[r][o] = sgn v_j[r],
// S[o] = sigma_j with j = src[o]; row-major outputs.
template <typename T>
__global__ __launch_bounds__(256) void svd_out_kernel(const double* __restrict__ XV, int d, int dp, const double* __restrict__ sig,
                                                      const int32_t* __restrict__ src,
                                                      const double* __restrict__ sgn, T* __restrict__ U,
                                                      int64_t ldu, T* __restrict__ S, T* __restrict__ V,
                                                      int64_t ldv) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)d * d) return;
  const int o = (int)(e / d), r = (int)(e % d);  // consecutive threads: consecutive rows of one column
  const double* X = XV + (int64_t)src[o] * 2 * dp;  // x_j, then v_j
  const double s = sig[o], g = sgn[o];
  U[(int64_t)r * ldu + o] = (T)(s > 0.0 ? g * X[r] / s : 0.0);
  V[(int64_t)r * ldv + o] = (T)(g * X[dp + r]);
  if (r == 0) S[o] = (T)s;
}

// Workspace: XV, sweep flags, sigma, signs, source columns, the rotations of
// two steps and their flags, the barrier's counter.
struct SvdWs { size_t flags, sig, sgn, src, jbuf, jflags, counter, total; };
static SvdWs svd_ws(int d) {
  const int dp = svd_padded(d), np = (dp / kSvW + 1) / 2;
  SvdWs w;
  size_t o = svd_align((size_t)dp * 2 * dp * sizeof(double));
  auto put = [&](size_t bytes) { const size_t at = o; o += svd_align(bytes); return at; };
  w.flags = put(kSvSweeps * sizeof(int32_t));
  w.sig = put((size_t)d * sizeof(double));
  w.sgn = put((size_t)d * sizeof(double));
  w.src = put((size_t)d * sizeof(int32_t));
  w.jbuf = put((size_t)2 * np * kSvCols * kSvCols * sizeof(double));
  w.jflags = put((size_t)2 * np * sizeof(int32_t));
  w.counter = put(sizeof(unsigned));
  w.total = o;
  return w;
}
size_t svd_ws_bytes(int d) { return svd_ws(d).total; }

template <typename T>
hipError_t launch_svd_small(const T* M, int64_t ldm, int d, T* U, int64_t ldu, T* S, T* V, int64_t ldv, void* ws,
                            void* info, hipStream_t s) {
  if (d < 1 || d > kDMax) return hipErrorInvalidValue;
  const int dp = svd_padded(d), nb = dp / kSvW, np = (nb + 1) / 2;
  const SvdWs w = svd_ws(d);
  char* p = (char*)ws;
  double* XV = (double*)p;
  int32_t* flags = (int32_t*)(p + w.flags);
  double* sig = (double*)(p + w.sig);
  double* sgn = (double*)(p + w.sgn);
  int32_t* src = (int32_t*)(p + w.src);
  double* jbuf = (double*)(p + w.jbuf);
  int32_t* jflags = (int32_t*)(p + w.jflags);
  unsigned* counter = (unsigned*)(p + w.counter);
  const int64_t tot = (int64_t)dp * 2 * dp;
  hipLaunchKernelGGL((svd_init_kernel<T>), dim3((unsigned)ceil_div(tot, 256)), dim3(256), 0, s, M, ldm, d, dp, XV,
                     flags, kSvSweeps, counter);
  // two copies of G while they fit beside X in 160 KB (dp <= 528)
  auto lds = [&](int copies) {
    return ((size_t)kSvCols * (dp + kXPad) + (size_t)(copies + 1) * kSvCols * kGS) * sizeof(double);
  };
  const bool ping = lds(2) + 1024 <= 160 * 1024;
  const size_t shmem = lds(ping ? 2 : 1);
  const void* fn = ping ? reinterpret_cast<const void*>(svd_sweeps_kernel<true>)
                        : reinterpret_cast<const void*>(svd_sweeps_kernel<false>);
  if (shmem > 65536) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (e != hipSuccess) return e;
  }
  double itol = 1.0 / ((double)dp * 1.1102230246251565e-16);
  int max_sweeps = kSvSweeps;
  void* args[] = {&XV, (void*)&dp, (void*)&nb, &flags, &max_sweeps, &itol, &jbuf, &jflags, &counter};
  // at most 34 workgroups of one CU each: the whole grid is resident at once
  const hipError_t e = hipLaunchCooperativeKernel(fn, dim3((unsigned)(2 * np)), dim3(kSvThreads), args,
                                                  (unsigned)shmem, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(svd_order_kernel, dim3(1), dim3(1024), 0, s, XV, d, dp, flags, kSvSweeps, sig, src, sgn,
                     (DevInfo*)info);
  hipLaunchKernelGGL((svd_out_kernel<T>), dim3((unsigned)ceil_div((int64_t)d * d, 256)), dim3(256), 0, s, XV, d, dp,
                     sig, src, sgn, U, ldu, S, V, ldv);
  return hipGetLastError();
}

template hipError_t launch_svd_small<float>(const float*, int64_t, int, float*, int64_t, float*, float*, int64_t,
                                            void*, void*, hipStream_t);
template hipError_t launch_svd_small<double>(const double*, int64_t, int, double*, int64_t, double*, double*,
                                             int64_t, void*, void*, hipStream_t);

}  // namespace rqlp
