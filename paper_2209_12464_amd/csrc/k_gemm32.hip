// Dense float32 products with A, Y = A X (NN) and Y = A^T X (TN), on the
// float16 matrix cores: the sketch, power-step and projection products of
// Algorithms 1 and 2, whose X is a Gaussian test matrix or a basis.
//
// Every value is scaled by a power of two and split into two float16 parts,
// x s = h + l (11 + 11 significand bits and the sign of l: within half an ulp
// of float32, rms 2^-24.6 of x), and a product is taken as the three partial
// products a_l x_h + a_h x_l + a_h x_h, each exact in float32, accumulated in
// float32; the fourth, a_l x_l, is 2^-24.8 of a x (rms).  A 32x32x16 MFMA adds
// 16 products into its accumulator at a time, so a dot product sees fewer
// roundings than with the float32 MFMA, which dominate both: the relative
// error against float64 at 8000 x 8000 x 210 is 3.7e-7, with the float32
// MFMA 5.7e-7.  Three float16 MFMAs have 16/3 = 5.3 times the rate of the
// float32 MFMA.
//
// Range: X is scaled by the caller's power of two (g.xscale), A by one of its
// own per row of op(A), taken from the first reduction step and lowered when
// a later value asks for it (what was accumulated follows), so that the
// largest value of a row so far lies in [2^7, 2^15) and float16's smallest
// step is at most 2^-31 of it.  What is left to float32: an output that is
// not finite (a part of an infinity, or of an X value past the range) or is
// nonzero below 2^-96 (inputs whose parts no scale of float32's range can
// hold) sends its wave's 32 rows through the float32 MFMA again, straight from
// the inputs.
//
// Tiles: a workgroup owns 32 WAVES rows (256 or 128) and up to 288 columns of
// Y; wave w the rows 32 w .. and every column, as NB blocks of 32 x 32.  So
// each value of A is loaded, split and used by one wave only: A goes from
// memory straight to the registers of its MFMA operands (two reduction steps
// of 32 ahead), split while the other half step's MFMAs run, and only X passes
// through LDS.  X is split once per product by a kernel of its own, into whole
// operand fragments in the order the product reads them, so that a step's
// tile is one contiguous run copied straight to LDS (a ring of three stages,
// two steps ahead, one barrier per step) and read back without bank
// conflicts.  The reduction is split over workgroups (split-K) and the partial
// slabs are summed in a fixed order; an output's summation order depends on
// the split only, not on the row tile.
//
// Measured, one product with X's split (4-5 us) and the split-K reduction
// (10 us at 8000 x 224): 8000 x 8000 x 210 112 us (float32 MFMA 268 / 288),
// 20000 x 15000 x 224 424 us, 6000 x 3000 x 110 36 us (65), 2700 x 2700 x 288
// 40 us (90).  At 8000 x 8000 the main kernel takes 98 us; the MFMAs alone are
// 40, A's 256 MB at the card's copy rate 50; what is left is the latency
// between a step's parts (without any global load it still takes 82 us: LDS
// reads, conversions and one barrier per step) and the partial slabs' 57 MB.
// Tried on the way: X split by each workgroup on its way to LDS, no separate
// kernel (125-141 us); X tiles and A one step ahead (122); X's fragments read
// one block ahead of their products (122).
#include "common.h"
#include "grouped.h"
#include "kernels.h"

#include <type_traits>

namespace rqlp {

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// four floats at any float's alignment (the target takes unaligned vector loads)
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int kBK = 32;      // reduction step

// A pair of values times s as two packed float16 parts.
__device__ inline void split2(float x0, float x1, float s, uint32_t& hi, uint32_t& lo) {
  const f16x2 h = {(_Float16)(x0 * s), (_Float16)(x1 * s)};
  const f16x2 l = {(_Float16)fmaf(x0, s, -(float)h.x), (_Float16)fmaf(x1, s, -(float)h.y)};
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, l);
}

__device__ inline floatx16 mma(u32x4 a, u32x4 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// 2^e for -126 <= e <= 127
__device__ inline float pow2(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }

// s_waitcnt immediate: at most n vector memory operations outstanding
constexpr int vm_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

}  // namespace

// ---------------------------------------------------------------------------
// X (K x N floats, ldb) into operand fragments: block (step s, column block
// b) holds, for each half step h and part p, 64 lanes of 16 bytes, lane l the
// values of column 32 b + l % 32 at reduction indices 32 s + 16 h + 8 (l / 32)
// .. + 7; zero past K and N.  Column blocks of one pass (cwb blocks, the last
// pass what remains) lie together: pass, step, block.  Memory-bound (4 bytes
// in, 4 out per value); one wave per (block, half step).
__device__ __attribute__((always_inline)) inline void xsplit_body(const float* __restrict__ B, int64_t ldb, int K, int N,
                                                                  float xs, int steps, int nblk, int cwb,
                                                                  u32x4* __restrict__ out, int bid) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t t = (int64_t)bid * 4 + wave;  // (step, block, half step), half step fastest
  const int h = (int)(t & 1);
  const int64_t sb = t >> 1;
  const int s = (int)(sb / nblk), b = (int)(sb % nblk);
  if (s >= steps) return;
  const int n = 32 * b + (lane & 31), k0 = kBK * s + 16 * h + 8 * (lane >> 5);
  float x[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) x[j] = (n < N && k0 + j < K) ? B[(int64_t)(k0 + j) * ldb + n] : 0.f;
  u32x4 hi, lo;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    uint32_t a, c;
    split2(x[2 * p], x[2 * p + 1], xs, a, c);
    hi[p] = a;
    lo[p] = c;
  }
  const int pass = b / cwb, first = pass * cwb;
  const int width = nblk - first < cwb ? nblk - first : cwb;
  u32x4* o = out + ((int64_t)steps * first + (int64_t)s * width + (b - first)) * 256 + h * 128 + lane;
  o[0] = hi;
  o[64] = lo;
}

__global__ __launch_bounds__(256) void xsplit_kernel(const float* __restrict__ B, int64_t ldb, int K, int N, float xs,
                                                     int steps, int nblk, int cwb, u32x4* __restrict__ out) {
  xsplit_body(B, ldb, K, N, xs, steps, nblk, cwb, out, blockIdx.x);
}

struct XsplitArgs {
  const float* B;
  u32x4* out;
  int64_t ldb;
  int K, N, steps, nblk, cwb;
  float xs;
};

__global__ __launch_bounds__(256) void xsplit_grouped(const XsplitArgs* __restrict__ a, const int* __restrict__ start,
                                                      int count) {
  const int p = group_find(start, count, blockIdx.x);
  const XsplitArgs x = a[p];
  xsplit_body(device_ptr(x.B), x.ldb, x.K, x.N, x.xs, x.steps, x.nblk, x.cwb, device_ptr(x.out),
              (int)blockIdx.x - start[p]);
}

void xsplit_grouped_launch(const void* args, const int* start, int count, unsigned blocks, hipStream_t s) {
  hipLaunchKernelGGL(xsplit_grouped, dim3(blocks), dim3(256), 0, s, (const XsplitArgs*)args, start, count);
}

size_t gemm32_split_bytes(int64_t K, int N) { return (size_t)round_up(K, kBK) * round_up(N, 32) * 4; }

void launch_xsplit(const GemmArgs<float>& g, int cw, hipStream_t s) {
  const int steps = (int)ceil_div(g.K, kBK), nblk = (int)ceil_div(g.N, 32), cwb = cw / 32;
  const unsigned blocks = (unsigned)ceil_div((int64_t)steps * nblk * 2, 4);
  const XsplitArgs x{g.B, (u32x4*)g.xsplit, g.ldb, g.K, g.N, steps, nblk, cwb, g.xscale};
  if (!record_launch(&xsplit_grouped_launch, x, blocks))
    hipLaunchKernelGGL(xsplit_kernel, dim3(blocks), dim3(256), 0, s, x.B, x.ldb, x.K, x.N, x.xs, steps, nblk, cwb, x.out);
}

// ---------------------------------------------------------------------------
// One workgroup's share: tile `logical` = split * mtiles + slab.  Xf: the
// fragments of this column pass; B, ldb: its values, for the float32 path.
template <int NB, bool TRANS, int WAVES>
__device__ __attribute__((always_inline)) inline void gemm32_body(
    const float* __restrict__ A, int64_t lda, const u32x4* __restrict__ Xf, const float* __restrict__ B, int64_t ldb,
    float* __restrict__ C, int64_t ldc, int64_t cslice, int M, int N, int K, int kchunk, int mtiles, int nst, float xs,
    int logical) {
  constexpr int BM = 32 * WAVES;
  constexpr int NLOADS = 4 * NB;              // 1 KB wave loads per X tile
  constexpr int LB = (NLOADS + WAVES - 1) / WAVES;  // per wave (the last ones of a wave may repeat a load)
  constexpr int AH = TRANS ? 8 : 2;           // loads per half step of A
  // LDS ring of X tiles; with 8 waves (one workgroup per CU) a tile is
  // requested two steps before its use, with 4 (two workgroups) one
  constexpr int kStages = WAVES == 8 ? 4 : 3;
  __shared__ __attribute__((aligned(1024))) u32x4 Bs[kStages][NB * 256];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lc = lane & 31, g = lane >> 5;
  const int split = logical / mtiles;
  const int mt = logical - split * mtiles;
  const int m0 = mt * BM + wave * 32;
  const int kbeg = split * kchunk;
  const int kend = min(K, kbeg + kchunk);
  // a split that is no whole number of steps takes its short step first
  const int nsteps = kbeg < kend ? (kend - kbeg + kBK - 1) / kBK : 0;
  const int nshort = nsteps > 0 ? kend - kbeg - (nsteps - 1) * kBK : 0;  // 1 .. 32
  const bool ragged = nshort != kBK;
  // the i-th step taken (past the end, the last: such loads are not used)
  auto step_id = [&](int i) {
    i = min(i, nsteps - 1);
    return ragged ? (i == 0 ? nsteps - 1 : i - 1) : i;
  };

  // Operand row of lane l: l % 32; its reduction indices in half step h:
  // 16 h + 8 (l / 32) .. + 7.  NN loads rows l % 16 and 16 + l % 16, four
  // values at 4 (l / 16) each (64 consecutive bytes of a row per load), and a
  // half-row swap between the two puts every value in its place.  Rows past M
  // are read from row M - 1 and not stored.
  const int arow = min(m0 + lc, M - 1);
  const float* p0;
  const float* p1;
  if constexpr (TRANS) {
    p0 = A + (int64_t)(kbeg + 8 * g) * lda + arow;
    p1 = p0;
  } else {
    p0 = A + (int64_t)min(m0 + (lane & 15), M - 1) * lda + kbeg + 4 * (lane >> 4);
    p1 = A + (int64_t)min(m0 + 16 + (lane & 15), M - 1) * lda + kbeg + 4 * (lane >> 4);
  }
  // A split that is one short step has no whole step to load ahead (loads are
  // issued all the same): they go to the first bytes of X's fragments instead.
  const float *q0 = p0, *q1 = p1;
  int64_t ldq = lda;
  if (ragged && nsteps == 1) {
    q0 = q1 = (const float*)Xf;
    ldq = 0;
  }
  float raw[2][2][8];  // loaded values: [parity of the step][half step]
  auto load_a = [&](auto Pc, auto Hc, int i) {
    constexpr int P = decltype(Pc)::value, H = decltype(Hc)::value;
    const int64_t ko = (int64_t)step_id(i) * kBK + 16 * H;
    if constexpr (TRANS) {
      const float* p = q0 + ko * ldq;
#pragma unroll
      for (int j = 0; j < 8; ++j) raw[P][H][j] = p[(int64_t)j * ldq];
    } else {
      const floatx4u u = *reinterpret_cast<const floatx4u*>(q0 + ko);
      const floatx4u v = *reinterpret_cast<const floatx4u*>(q1 + ko);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        raw[P][H][e] = u[e];
        raw[P][H][4 + e] = v[e];
      }
    }
  };
  // the short first step: zeros from its nshort-th value on (read from the
  // last one)
  auto load_short = [&] {
    const int64_t ko = (int64_t)(nsteps - 1) * kBK;
    const int c = TRANS ? 8 * g : 4 * (lane >> 4);  // in p0 and p1 already
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int kk = 16 * h + (TRANS ? j : j & 3);
        const int64_t k = ko + min(kk, nshort - 1 - c);
        const float v = TRANS || j < 4 ? p0[TRANS ? k * lda : k] : p1[k];
        raw[0][h][j] = c + kk < nshort ? v : 0.f;
      }
  };
  auto issue_x = [&](int i) {  // X tile of step i into its ring stage
    const u32x4* src = Xf + ((int64_t)(kbeg / kBK + step_id(i)) * NB) * 256;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)src, 0, NB * 4096, 0x00027000);
    u32x4* dst = Bs[i % kStages];
#pragma unroll
    for (int u = 0; u < LB; ++u) {
      const int j = min(wave + WAVES * u, NLOADS - 1);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(dst + 64 * j), 16, lane * 16, j * 1024, 0, 0);
    }
  };

  floatx16 acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = (floatx16)0.0f;

  // The scale of operand row arow: 2^-ea, as the factor `as`; values from
  // athr on need another.  A row whose largest value so far is m takes the
  // scale that puts m into [2^7, 2^8).
  int ea = 0;
  float as = 1.f, athr = 0.f;
  u32x4 ap[2][2];  // this wave's A operands: [half step][part]
  auto set_scale = [&](float m) {
    ea = max((int)(__float_as_uint(m) >> 23) - 127 - 7, -120);
    as = pow2(-ea);
    athr = ea + 15 < 128 ? pow2(ea + 15) : __builtin_inff();
  };
  auto place = [&](auto Pc, auto Hc) {  // every value to its lane (see above)
    constexpr int P = decltype(Pc)::value, H = decltype(Hc)::value;
    if constexpr (!TRANS) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const u32x2 r = __builtin_bit_cast(
            u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(raw[P][H][e]), __float_as_uint(raw[P][H][4 + e]),
                                                    false, false));
        raw[P][H][e] = __uint_as_float(r[0]);
        raw[P][H][4 + e] = __uint_as_float(r[1]);
      }
    }
  };
  auto absmax = [&](auto Pc, auto Hc) {
    constexpr int P = decltype(Pc)::value, H = decltype(Hc)::value;
    float m = fabsf(raw[P][H][0]);
#pragma unroll
    for (int j = 1; j < 8; ++j) m = fmaxf(m, fabsf(raw[P][H][j]));
    return m;
  };
  // Rows with a value too large for their scale take another, and what they
  // have accumulated and the other half's parts, still to be multiplied,
  // follow.
  // (Not for what was loaded past the last step.)
  auto check_scale = [&](auto Pc, auto Hc, bool used) {
    constexpr int H = decltype(Hc)::value;
    float m = absmax(Pc, Hc);
    if (__builtin_expect(!__any(used && m >= athr), 1)) return;
    m = fmaxf(m, __shfl_xor(m, 32));
    const int eo = ea;
    if (m >= athr) set_scale(m);
    const int de = max(eo - ea, -250);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int dr = __shfl(de, 8 * (r >> 2) + 4 * g + (r & 3));
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[nb][r] = ldexpf(acc[nb][r], dr);
      __builtin_amdgcn_sched_barrier(0);
    }
    const _Float16 f = (_Float16)ldexpf(1.f, de);
    const f16x8 fv = {f, f, f, f, f, f, f, f};
#pragma unroll
    for (int q = 0; q < 2; ++q)
      ap[H ^ 1][q] = __builtin_bit_cast(u32x4, __builtin_bit_cast(f16x8, ap[H ^ 1][q]) * fv);
  };
  auto split_a = [&](auto Pc, auto Hc, int p) {  // pair p
    constexpr int P = decltype(Pc)::value, H = decltype(Hc)::value;
    uint32_t x, y;
    split2(raw[P][H][2 * p], raw[P][H][2 * p + 1], as, x, y);
    ap[H][0][p] = x;
    ap[H][1][p] = y;
  };

  // One half step: the partial products of each column block.  A block's
  // fragments are read from LDS two blocks ahead, each part into the registers
  // its last product has just freed (across steps, too: `nx` is the next tile
  // in the second half step), and the A values (SP, SH) that the next half
  // step needs are split along the way, so that the vector work runs under the
  // matrix work.
  u32x4 b[2][2];
  auto fetch = [&](const u32x4* bs, int t, int q) { b[t & 1][q] = bs[(t % NB * 4 + t / NB * 2 + q) * 64]; };
  auto half_step = [&](auto Hc, auto SPc, const u32x4* bs, const u32x4* nx, bool used) {
    constexpr int H = decltype(Hc)::value;
    using SHc = std::integral_constant<int, H ^ 1>;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int t = H * NB + nb, cur = t & 1;
      // one column block: two blocks ahead would be the next tile already in
      // the first half step, when it need not be there yet
      constexpr bool AHEAD = NB > 1 || H == 1;
      const u32x4* fs = t + 2 < 2 * NB ? bs : nx;
      const int ft = t + 2 < 2 * NB ? t + 2 : t + 2 - 2 * NB;
      if constexpr (NB == 1 && H == 1) {
        fetch(nx, 0, 0);
        fetch(nx, 0, 1);
      }
      acc[nb] = mma(ap[H][1], b[cur][0], acc[nb]);
      acc[nb] = mma(ap[H][0], b[cur][0], acc[nb]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (AHEAD) fetch(fs, ft, 0);
      __builtin_amdgcn_sched_barrier(0);
      acc[nb] = mma(ap[H][0], b[cur][1], acc[nb]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (AHEAD) fetch(fs, ft, 1);
      if (nb == 0) {
        place(SPc, SHc{});
        check_scale(SPc, SHc{}, used);
      }
#pragma unroll
      for (int w = nb * 4 / NB; w < (nb + 1) * 4 / NB; ++w) split_a(SPc, SHc{}, w);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;

  // Step i of parity P.  At its start raw holds (or awaits) half step 1 of
  // step i, step i + 1 and half step 0 of step i + 2, and the ring tile i and
  // (awaited) the kStages - 2 after it.
  auto step = [&](auto Pc, int i) {
    constexpr int P = decltype(Pc)::value;
    using Qc = std::integral_constant<int, P ^ 1>;
    const u32x4* bs = Bs[i % kStages] + lane;
    const u32x4* nx = Bs[(i + 1) % kStages] + lane;
    half_step(I0{}, Pc, bs, nx, true);
    load_a(Pc, I1{}, i + 2);
    // This wave's loads of tile i + 1 are done once at most the loads issued
    // after it are pending: at least 3 half steps of A and, if there is one,
    // tile i + 2 (8 waves), or 2 half steps of A.  (A's loads are issued in
    // every step, so that they can be counted.)
    if (WAVES == 8 && i + 2 < nsteps) __builtin_amdgcn_s_waitcnt(vm_imm(3 * AH + LB));
    else __builtin_amdgcn_s_waitcnt(vm_imm(WAVES == 8 ? 3 * AH : 2 * AH));
    // Every wave's part of tile i + 1 is in, and every wave has consumed tile
    // i - 1, whose stage is filled again (a plain barrier: the loads in flight
    // stay so).
    asm volatile("s_barrier" ::: "memory");
    if (i + kStages - 1 < nsteps) issue_x(i + kStages - 1);
    half_step(I1{}, Qc{}, bs, nx, i + 1 < nsteps);
    load_a(Qc{}, I0{}, i + 3);
  };

  if (nsteps > 0) {
    if (ragged) {
      load_short();
    } else {
      load_a(I0{}, I0{}, 0);
      load_a(I0{}, I1{}, 0);
    }
    issue_x(0);
    load_a(I1{}, I0{}, 1);
    load_a(I1{}, I1{}, 1);
    if (nsteps > 1) issue_x(1);
    if (kStages > 3 && nsteps > 2) issue_x(2);
    {  // the first scales, from the whole first step
      place(I0{}, I0{});
      place(I0{}, I1{});
      const float m = fmaxf(absmax(I0{}, I0{}), absmax(I0{}, I1{}));
      place(I0{}, I1{});  // (its own inverse: step 0 places half step 1 again)
      set_scale(fmaxf(m, __shfl_xor(m, 32)));
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) split_a(I0{}, I0{}, p);
    // tile 0 (and whatever else has been requested so far)
    __builtin_amdgcn_s_waitcnt(vm_imm(0));
    asm volatile("s_barrier" ::: "memory");
    load_a(I0{}, I0{}, 2);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int q = 0; q < 2; ++q) fetch(Bs[0] + lane, t, q);
    int i = 0;
    for (; i + 1 < nsteps; i += 2) {
      step(I0{}, i);
      step(I1{}, i + 1);
    }
    if (i < nsteps) step(I0{}, i);
  }

  {  // undo the scales
    const int ex = 127 - (int)(__float_as_uint(xs) >> 23);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int er = __shfl(ea, 8 * (r >> 2) + 4 * g + (r & 3)) + ex;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[nb][r] = ldexpf(acc[nb][r], er);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // outputs the split cannot vouch for: this wave's rows again in float32
  bool bad = false;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float v = fabsf(acc[nb][r]);
      bad |= !(v < __builtin_inff()) || (v < 0x1p-96f && v != 0.f);
    }
  if (__any(bad)) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = (floatx16)0.0f;
    for (int k0 = kbeg; k0 < kend; k0 += 2) {
      const int k = k0 + g;
      const bool kin = k < kend;
      const float a = kin ? A[TRANS ? (int64_t)k * lda + arow : (int64_t)arow * lda + k] : 0.f;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int n = nb * 32 + lc;
        const float x = (kin && n < N) ? B[(int64_t)k * ldb + n] : 0.f;
        acc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, x, acc[nb], 0, 0, 0);
      }
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

template <int NB, bool TRANS, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 2) void gemm32_kernel(const float* __restrict__ A, int64_t lda,
                                                               const u32x4* __restrict__ Xf,
                                                               const float* __restrict__ B, int64_t ldb,
                                                               float* __restrict__ C, int64_t ldc, int64_t cslice,
                                                               int M, int N, int K, int kchunk, int mtiles, int nst,
                                                               float xs) {
  gemm32_body<NB, TRANS, WAVES>(A, lda, Xf, B, ldb, C, ldc, cslice, M, N, K, kchunk, mtiles, nst, xs,
                                xcd_remap(blockIdx.x, gridDim.x));
}

struct Gemm32Args {
  const float* A;
  const u32x4* Xf;
  const float* B;
  float* C;
  int64_t lda, ldb, ldc, cslice;
  int M, N, K, kchunk, mtiles, nst;
  float xs;
};

template <int NB, bool TRANS, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 2) void gemm32_grouped(const Gemm32Args* __restrict__ a,
                                                                const int* __restrict__ start, int count) {
  const int p = group_find(start, count, blockIdx.x);
  const Gemm32Args x = a[p];
  gemm32_body<NB, TRANS, WAVES>(device_ptr(x.A), x.lda, device_ptr(x.Xf), device_ptr(x.B), x.ldb, device_ptr(x.C),
                                x.ldc, x.cslice, x.M, x.N, x.K, x.kchunk, x.mtiles, x.nst, x.xs,
                                (int)blockIdx.x - start[p]);
}

template <int NB, bool TRANS, int WAVES>
void gemm32_grouped_launch(const void* args, const int* start, int count, unsigned blocks, hipStream_t s) {
  hipLaunchKernelGGL((gemm32_grouped<NB, TRANS, WAVES>), dim3(blocks), dim3(64 * WAVES), 0, s, (const Gemm32Args*)args,
                     start, count);
}

template <int NB, bool TRANS, int WAVES>
static void launch_nb32(const Gemm32Args& x, int grid, hipStream_t s) {
  if (!record_launch(&gemm32_grouped_launch<NB, TRANS, WAVES>, x, (unsigned)grid))
    hipLaunchKernelGGL((gemm32_kernel<NB, TRANS, WAVES>), dim3((unsigned)grid), dim3(64 * WAVES), 0, s, x.A, x.lda,
                       x.Xf, x.B, x.ldb, x.C, x.ldc, x.cslice, x.M, x.N, x.K, x.kchunk, x.mtiles, x.nst, x.xs);
}

template <bool TRANS, int WAVES>
static void dispatch_nb32(const Gemm32Args& x, int grid, hipStream_t s) {
  switch ((int)ceil_div(x.N, 32)) {
    case 1: launch_nb32<1, TRANS, WAVES>(x, grid, s); break;
    case 2: launch_nb32<2, TRANS, WAVES>(x, grid, s); break;
    case 3: launch_nb32<3, TRANS, WAVES>(x, grid, s); break;
    case 4: launch_nb32<4, TRANS, WAVES>(x, grid, s); break;
    case 5: launch_nb32<5, TRANS, WAVES>(x, grid, s); break;
    case 6: launch_nb32<6, TRANS, WAVES>(x, grid, s); break;
    case 7: launch_nb32<7, TRANS, WAVES>(x, grid, s); break;
    case 8: launch_nb32<8, TRANS, WAVES>(x, grid, s); break;
    default: launch_nb32<9, TRANS, WAVES>(x, grid, s); break;
  }
}

// One column pass from column c0 (g.B and g.N are the pass's own).
void launch_gemm32_tiles(const GemmArgs<float>& g, int c0, int grid, float* C, int64_t ldc, int64_t cslice, int nst,
                         hipStream_t s) {
  if (!g.xsplit) {
    launch_gemm32_any(g, grid, C, ldc, cslice, nst, s);
    return;
  }
  const u32x4* Xf = (const u32x4*)g.xsplit + ceil_div(g.K, kBK) * (c0 / 32) * 256;
  const Gemm32Args x{g.A, Xf, g.B, C, g.lda, g.ldb, ldc, cslice, g.M, g.N, g.K, g.kchunk, g.mtiles, nst, g.xscale};
  if (g.mb == 4) {
    if (g.trans) dispatch_nb32<true, 8>(x, grid, s);
    else dispatch_nb32<false, 8>(x, grid, s);
  } else {
    if (g.trans) dispatch_nb32<true, 4>(x, grid, s);
    else dispatch_nb32<false, 4>(x, grid, s);
  }
}

}  // namespace rqlp
