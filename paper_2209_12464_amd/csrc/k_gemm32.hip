// Dense float32 products with A, Y = A X (NN) and Y = A^T X (TN), on the bfloat16
// matrix cores: the sketch, power-step and projection products of Algorithms 1 and
// 2 and rqlp_gemm.
//
// Each float is split exactly into three bfloat16 parts, x = h + m + l (8 + 8
// + 8 significand bits, each part the rounding of what the parts before it
// leave), and a product a x is taken as the six partial products
//     a_l x_h + a_h x_l + a_m x_m + a_m x_h + a_h x_m + a_h x_h,
// each exact in float32, accumulated in float32.  The three products left out
// (m l, l m, l l) are below 2^-24 of a x together, float32's own rounding of it,
// and a 32x32x16 MFMA adds 16 products into its accumulator at a time, so that a
// dot product sees fewer roundings than with the float32 MFMA.
// bfloat16 has float32's range, so one constant factor serves; six bfloat16
// MFMAs have 16/6 = 2.7 times the rate of the float32 MFMA.  Measured, one product
// with its split-K reduction: 6000 x 3000 x 110: 41 us (float32 MFMA 92), 8000
// x 8000 x 210: 163 us (320), where it is the chip's power that binds (the
// clock falls to 2.0 GHz, 1.8 at 20000 x 15000; 1.05-1.17 PFLOP/s of bfloat16,
// what the vendor's large matrix products reach here); relative error against
// float64 at 6000 x 3000 x 110 3.9e-7 (float32 MFMA 4.1e-7).
//
// Range: the parts are multiples of 2^-133, bfloat16's smallest denormal, and
// float32's values of 2^-149.  Both operands are therefore multiplied by 2^16, so
// that every value is the sum of its parts, and the sums by 2^-32.  What leaves the
// range on the way (values from 2^112, sums from 2^96) or is not finite shows as an
// output that is not finite, and sends its wave's 32 rows through the float32 MFMA
// again, straight from the inputs.  (Without the factors small values lose parts,
// and a guard on the size of the outputs either misses them, where the other
// operand is large, or redoes the far parts of a split reduction over a matrix that
// decays: a 4000 x 3000 Gaussian kernel times 110 columns took 200 us, now 35 us.)
//
// Tiles: a workgroup owns 32 WAVES rows (256 or 128) and up to 288 columns of Y;
// wave w the rows 32 w .. and every column, as NB blocks of 32 x 32.  So each value
// of A is loaded, split and used by one wave only, and goes from memory straight to
// the registers of its MFMA operands, split while the other half step's MFMAs run.
// X is split by the workgroup on its way to LDS (once per reduction step, stored as
// whole operand fragments, double buffered) and read back without bank conflicts.
// The reduction is split over workgroups (split-K) and the partial slabs are summed
// in a fixed order; an output's summation order depends on the split only, not on
// the row tile.
//
// BLOCKED (decompositions): the six partial products of 16 reduction indices are
// summed by themselves and the sum is added to the accumulator, one rounding of it
// in the place of six: relative error against float64 2.5e-7 instead of 5.1e-7 at
// 8000 x 8000 x 210, 2.1e-7 instead of 3.9e-7 at 6000 x 3000 x 110, for 5 to 10 %
// more time (168 -> 180 us, 41 -> 46 us; 2700 x 2700 x 270 46 -> 51).  What several
// products, and the orthonormalizations between them, make of their rounding errors
// adds up; a product by itself (rqlp_gemm) is as accurate as on the float32 MFMA
// without.  The additions stand between the MFMAs of the next block (after them:
// another 5 %) and take a second block's worth of registers, so that with eight
// waves 224 columns are the most (8000 x 8000 x 256: 225 us in two passes, 270 in
// one that spills).
//
// Two float16 parts of each operand and three products, with a scale for each row of
// A, took 112 us at 8000 x 8000 x 210, but held 22 to 23 bits of a value (fewer of
// one far below its row's largest) where float32 has 24, and L's errors grew by it.
#include "common.h"
#include "grouped.h"
#include "kernels.h"

#include <type_traits>

namespace rqlp {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// four floats at any float's alignment (the target takes unaligned vector loads)
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kBK = 32;
constexpr float kLift = 0x1p16f;

// two floats to packed bfloat16, round to nearest even
__device__ inline uint32_t pk_bf16(float a, float b) {
  const floatx2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// The three parts of a pair of values times kLift, packed.
__device__ inline void split3(float x0, float x1, uint32_t* part) {
  const uint32_t h = pk_bf16(x0 * kLift, x1 * kLift);
  const float r0 = fmaf(x0, kLift, -__uint_as_float(h << 16)), r1 = fmaf(x1, kLift, -__uint_as_float(h & 0xffff0000u));
  const uint32_t m = pk_bf16(r0, r1);
  part[0] = h;
  part[1] = m;
  part[2] = pk_bf16(r0 - __uint_as_float(m << 16), r1 - __uint_as_float(m & 0xffff0000u));
}

__device__ inline floatx16 mma(u32x4 a, u32x4 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

}  // namespace

// One workgroup's share: tile `logical` = split * mtiles + slab.
// Lane l of a wave holds operand row (A) or column (X) l % 32; its reduction
// indices of half step h (16 of a step's 32) are 16 h + 8 (j / 4) + 4 (l / 32)
// + j % 4, j = 0..7: any assignment serves as long as both operands share it,
// and this one lets a lane load A in runs of four.
template <int NB, bool TRANS, int WAVES, bool BLOCKED>
__device__ __attribute__((always_inline)) inline void gemm32_body(
    const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb, float* __restrict__ C,
    int64_t ldc, int64_t cslice, int M, int N, int K, int kchunk, int mtiles, int nst, int logical) {
  constexpr int BM = 32 * WAVES, BN = 32 * NB, THREADS = 64 * WAVES;
  constexpr int UNITS = 4 * BN;                           // (column, half step, lane half): 8 values of X each
  constexpr int UPT = (UNITS + THREADS - 1) / THREADS;
  __shared__ u32x4 Bs[2][NB * 2 * 3 * 64];                // [block][half step][part][lane]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lc = lane & 31, g = lane >> 5;
  const int split = logical / mtiles;
  const int mt = logical - split * mtiles;
  const int m0 = mt * BM + wave * 32;
  const int kbeg = split * kchunk;
  const int kend = min(K, kbeg + kchunk);

  // rows past M are read from row M - 1 and not stored
  const int arow = min(m0 + lc, M - 1);
  const float* pa = TRANS ? A + (int64_t)(kbeg + 4 * g) * lda + arow : A + (int64_t)arow * lda + kbeg + 4 * g;

  // this thread's units: LDS slot and first reduction index; a unit past the
  // last one or a column past N reads a valid place, and its values go nowhere
  // (columns past N are stored as zero)
  int ul[UPT], uk[UPT];
  const float* pb[UPT];
#pragma unroll
  for (int u = 0; u < UPT; ++u) {
    const int e = tid + THREADS * u;
    const int n = e % BN, hg = (e / BN) & 3, h = hg >> 1, gg = hg & 1;
    uk[u] = 16 * h + 4 * gg;
    ul[u] = ((n >> 5) * 2 + h) * 3 * 64 + gg * 32 + (n & 31);
    pb[u] = B + (int64_t)(kbeg + uk[u]) * ldb + min(n, N - 1);
  }

  float araw[2][8], braw[UPT][8];
  u32x4 ap[2][3];   // this wave's A operands: parts of the two half steps
  u32x4 bp[UPT][3];  // parts of the units on their way to LDS
  auto load_a = [&](auto Hc, const float* p) {  // half step H of the step at p
    constexpr int H = decltype(Hc)::value;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (TRANS) {
#pragma unroll
        for (int e = 0; e < 4; ++e) araw[H][4 * i + e] = p[(int64_t)(16 * H + 8 * i + e) * lda];
      } else {
        const floatx4u v = *reinterpret_cast<const floatx4u*>(p + 16 * H + 8 * i);
#pragma unroll
        for (int e = 0; e < 4; ++e) araw[H][4 * i + e] = v[e];
      }
    }
  };
  auto load_b = [&](int u) {
#pragma unroll
    for (int j = 0; j < 8; ++j) braw[u][j] = pb[u][(int64_t)(8 * (j >> 2) + (j & 3)) * ldb];
    pb[u] += (int64_t)kBK * ldb;
  };
  // the first step: n <= kBK values, zeros after them (read from the n-th)
  auto load_first = [&](int n) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int kk = 8 * (i >> 2) + (i & 3), ko = min(kk, n - 1 - 4 * g);
      const float v = pa[TRANS ? (int64_t)ko * lda : (int64_t)ko];
      araw[i >> 3][i & 7] = 4 * g + kk < n ? v : 0.f;
    }
    pa += TRANS ? (int64_t)n * lda : (int64_t)n;
#pragma unroll
    for (int u = 0; u < UPT; ++u) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int kk = 8 * (j >> 2) + (j & 3);
        const float v = pb[u][(int64_t)min(kk, n - 1 - uk[u]) * ldb];
        braw[u][j] = uk[u] + kk < n ? v : 0.f;
      }
      pb[u] += (int64_t)n * ldb;
    }
  };
  auto split_a = [&](int h, int p) {  // pair p of half step h
    uint32_t x[3];
    split3(araw[h][2 * p], araw[h][2 * p + 1], x);
#pragma unroll
    for (int q = 0; q < 3; ++q) ap[h][q][p] = x[q];
  };
  auto split_b = [&](int u, int p, int buf) {  // pair p of unit u, stored with its last pair
    uint32_t x[3];
    split3(braw[u][2 * p], braw[u][2 * p + 1], x);
#pragma unroll
    for (int q = 0; q < 3; ++q) bp[u][q][p] = x[q];
    if (p == 3 && ((u + 1) * THREADS <= UNITS || tid + THREADS * u < UNITS)) {
#pragma unroll
      for (int q = 0; q < 3; ++q) Bs[buf][ul[u] + 64 * q] = bp[u][q];
    }
  };
  // every LDS access of the step done; the loads in flight stay so
  auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  floatx16 acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = (floatx16)0.0f;

  // One half step: the partial products of each column block, the parts of
  // the next block read from LDS meanwhile; after each block's MFMAs a share
  // of the splits that the coming half steps need (the other half's A values
  // and, for the units of this parity, X values for the other LDS buffer), so
  // that the vector work runs under the matrix work of the same wave.
  u32x4 b[2][3];
  auto fetch = [&](int buf, int t) {
    const u32x4* bs = Bs[buf] + lane;
    const int h = t / NB, nb = t % NB;
#pragma unroll
    for (int q = 0; q < 3; ++q) b[t & 1][q] = bs[((nb * 2 + h) * 3 + q) * 64];
  };
  // partial product x of half step H, smallest first
  auto product = [&](auto Hc, int x, int cur, floatx16 c) {
    const int pA = x == 0 ? 2 : (x == 2 || x == 3) ? 1 : 0;
    const int pB = x == 1 ? 2 : (x == 2 || x == 4) ? 1 : 0;
    return mma(ap[decltype(Hc)::value][pA], b[cur][pB], c);
  };
  auto splits = [&](auto Hc, int buf, int w0, int w1) {  // pairs w0 .. w1 - 1 of half step H's
    constexpr int H = decltype(Hc)::value;
    constexpr int NU = (UPT + 1 - H) / 2;  // units H, H + 2, ...
#pragma unroll
    for (int w = w0; w < w1; ++w) {
      if (w < 4 * NU) {
        split_b(H + 2 * (w / 4), w % 4, buf ^ 1);
      } else {
        split_a(H ^ 1, w - 4 * NU);
      }
    }
  };
  floatx16 sums[2];  // BLOCKED: this block's and the last one's sums over a half step
  auto half_step = [&](auto Hc, int buf) {
    constexpr int H = decltype(Hc)::value;
    constexpr int PAIRS = 4 + 4 * ((UPT + 1 - H) / 2);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int t = H * NB + nb, cur = t & 1;
      if (t + 1 < 2 * NB) fetch(buf, t + 1);
      __builtin_amdgcn_sched_barrier(0);
      const int w0 = nb * PAIRS / NB, w1 = (nb + 1) * PAIRS / NB;
      if constexpr (BLOCKED) {
        floatx16& sum = sums[cur];
        sum = (floatx16)0.0f;
#pragma unroll
        for (int x = 0; x < 6; ++x) {
          sum = product(Hc, x, cur, sum);
          if (t > 0) {
#pragma unroll
            for (int r = x * 16 / 6; r < (x + 1) * 16 / 6; ++r) acc[(t + NB - 1) % NB][r] += sums[cur ^ 1][r];
          }
          splits(Hc, buf, w0 + x * (w1 - w0) / 6, w0 + (x + 1) * (w1 - w0) / 6);
          __builtin_amdgcn_sched_barrier(0);
        }
        // (opaque: the additions stay here, or every sum of the step is kept)
        if (t > 0) asm volatile("" : "+v"(acc[(t + NB - 1) % NB]));
      } else {
#pragma unroll
        for (int x = 0; x < 6; ++x) acc[nb] = product(Hc, x, cur, acc[nb]);
        splits(Hc, buf, w0, w1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (BLOCKED && H == 1) {
      acc[NB - 1] += sums[1];
      asm volatile("" : "+v"(acc[NB - 1]));
    }
  };
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;

  // a split that is no whole number of steps takes the short one first
  const int nsteps = kbeg < kend ? (kend - kbeg + kBK - 1) / kBK : 0;
  const int64_t astep = TRANS ? (int64_t)kBK * lda : (int64_t)kBK;
  if (nsteps > 0) {
    load_first(kend - kbeg - (nsteps - 1) * kBK);
#pragma unroll
    for (int u = 0; u < UPT; ++u)
#pragma unroll
      for (int p = 0; p < 4; ++p) split_b(u, p, 0);
#pragma unroll
    for (int p = 0; p < 4; ++p) split_a(0, p);
    if (nsteps > 1) {
#pragma unroll
      for (int u = 0; u < UPT; ++u) load_b(u);
      load_a(H0{}, pa);
    }
    barrier();
    int buf = 0;
    for (int s = 0; s < nsteps; ++s) {
      // here: Bs[buf] and ap[0] hold step s, araw[1] its other half; braw and
      // araw[0] hold (or await) step s + 1, where pa points (in the last step
      // they are left-overs, split into places that are not read again)
      fetch(buf, 0);
      half_step(H0{}, buf);
      if (s + 2 < nsteps) {
#pragma unroll
        for (int u = 0; u < UPT; u += 2) load_b(u);
      }
      if (s + 1 < nsteps) load_a(H1{}, pa);
      half_step(H1{}, buf);
      if (s + 2 < nsteps) {
#pragma unroll
        for (int u = 1; u < UPT; u += 2) load_b(u);
        pa += astep;
        load_a(H0{}, pa);
      }
      barrier();
      buf ^= 1;
    }
  }

  // outputs the split cannot vouch for: this wave's rows again in float32
  bool bad = false;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      bad |= !(fabsf(acc[nb][r]) < __builtin_inff());
      acc[nb][r] *= 1.f / (kLift * kLift);
    }
  if (__any(bad)) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = (floatx16)0.0f;
    constexpr int kRun = 4;  // pairs of reduction indices loaded together
    for (int k0 = kbeg; k0 < kend; k0 += 2 * kRun) {
      float a[kRun], x[kRun][NB];
#pragma unroll
      for (int i = 0; i < kRun; ++i) {
        const int k = k0 + 2 * i + g;
        const bool kin = k < kend;
        a[i] = kin ? A[TRANS ? (int64_t)k * lda + arow : (int64_t)arow * lda + k] : 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const int n = nb * 32 + lc;
          x[i][nb] = (kin && n < N) ? B[(int64_t)k * ldb + n] : 0.f;
        }
      }
#pragma unroll
      for (int i = 0; i < kRun; ++i)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], x[i][nb], acc[nb], 0, 0, 0);
    }
  }

  float* Cs = C + (int64_t)split * cslice;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int col = nb * 32 + lc;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = m0 + 8 * (r >> 2) + 4 * g + (r & 3);
      if (row < M && col < nst) Cs[(int64_t)row * ldc + col] = col < N ? acc[nb][r] : 0.f;
    }
  }
}

template <int NB, bool TRANS, int WAVES, bool BLOCKED>
__global__ __launch_bounds__(64 * WAVES, 2) void gemm32_kernel(const float* __restrict__ A, int64_t lda,
                                                               const float* __restrict__ B, int64_t ldb,
                                                               float* __restrict__ C, int64_t ldc, int64_t cslice,
                                                               int M, int N, int K, int kchunk, int mtiles, int nst) {
  gemm32_body<NB, TRANS, WAVES, BLOCKED>(A, lda, B, ldb, C, ldc, cslice, M, N, K, kchunk, mtiles, nst,
                                xcd_remap(blockIdx.x, gridDim.x));
}

struct Gemm32Args {
  const float* A;
  const float* B;
  float* C;
  int64_t lda, ldb, ldc, cslice;
  int M, N, K, kchunk, mtiles, nst;
};

template <int NB, bool TRANS, int WAVES, bool BLOCKED>
__global__ __launch_bounds__(64 * WAVES, 2) void gemm32_grouped(const Gemm32Args* __restrict__ a,
                                                                const int* __restrict__ start, int count) {
  const int p = group_find(start, count, blockIdx.x);
  const Gemm32Args x = a[p];
  gemm32_body<NB, TRANS, WAVES, BLOCKED>(device_ptr(x.A), x.lda, device_ptr(x.B), x.ldb, device_ptr(x.C), x.ldc, x.cslice, x.M,
                                x.N, x.K, x.kchunk, x.mtiles, x.nst, (int)blockIdx.x - start[p]);
}

template <int NB, bool TRANS, int WAVES, bool BLOCKED>
void gemm32_grouped_launch(const void* args, const int* start, int count, unsigned blocks, hipStream_t s) {
  hipLaunchKernelGGL((gemm32_grouped<NB, TRANS, WAVES, BLOCKED>), dim3(blocks), dim3(64 * WAVES), 0, s, (const Gemm32Args*)args,
                     start, count);
}

template <int NB, bool TRANS, int WAVES, bool BLOCKED>
static void launch_nb32(const Gemm32Args& x, int grid, hipStream_t s) {
  if (!record_launch(&gemm32_grouped_launch<NB, TRANS, WAVES, BLOCKED>, x, (unsigned)grid))
    hipLaunchKernelGGL((gemm32_kernel<NB, TRANS, WAVES, BLOCKED>), dim3((unsigned)grid), dim3(64 * WAVES), 0, s, x.A,
                       x.lda, x.B, x.ldb, x.C, x.ldc, x.cslice, x.M, x.N, x.K, x.kchunk, x.mtiles, x.nst);
}

template <bool TRANS, int WAVES, bool BLOCKED>
static void dispatch_nb32(const Gemm32Args& x, int grid, hipStream_t s) {
  switch ((int)ceil_div(x.N, 32)) {
    case 1: launch_nb32<1, TRANS, WAVES, BLOCKED>(x, grid, s); break;
    case 2: launch_nb32<2, TRANS, WAVES, BLOCKED>(x, grid, s); break;
    case 3: launch_nb32<3, TRANS, WAVES, BLOCKED>(x, grid, s); break;
    case 4: launch_nb32<4, TRANS, WAVES, BLOCKED>(x, grid, s); break;
    case 5: launch_nb32<5, TRANS, WAVES, BLOCKED>(x, grid, s); break;
    case 6: launch_nb32<6, TRANS, WAVES, BLOCKED>(x, grid, s); break;
    case 7: launch_nb32<7, TRANS, WAVES, BLOCKED>(x, grid, s); break;
    case 8:
      if constexpr (!(BLOCKED && WAVES == 8)) launch_nb32<8, TRANS, WAVES, BLOCKED>(x, grid, s);
      break;
    default:  // (at most gemm32_max_cols)
      if constexpr (!(BLOCKED && WAVES == 8)) launch_nb32<9, TRANS, WAVES, BLOCKED>(x, grid, s);
  }
}

template <bool BLOCKED>
static void dispatch_tile32(const Gemm32Args& x, int mb, int trans, int grid, hipStream_t s) {
  if (mb == 4) {
    if (trans) dispatch_nb32<true, 8, BLOCKED>(x, grid, s);
    else dispatch_nb32<false, 8, BLOCKED>(x, grid, s);
  } else {
    if (trans) dispatch_nb32<true, 4, BLOCKED>(x, grid, s);
    else dispatch_nb32<false, 4, BLOCKED>(x, grid, s);
  }
}

int gemm32_max_cols(const GemmArgs<float>& g) { return g.blocked && g.mb == 4 ? 224 : 288; }

// One column pass (g.B and g.N are the pass's own).
void launch_gemm32_tiles(const GemmArgs<float>& g, int grid, float* C, int64_t ldc, int64_t cslice, int nst,
                         hipStream_t s) {
  const Gemm32Args x{g.A, g.B, C, g.lda, g.ldb, ldc, cslice, g.M, g.N, g.K, g.kchunk, g.mtiles, nst};
  if (g.blocked) dispatch_tile32<true>(x, g.mb, g.trans, grid, s);
  else dispatch_tile32<false>(x, g.mb, g.trans, grid, s);
}

}  // namespace rqlp
