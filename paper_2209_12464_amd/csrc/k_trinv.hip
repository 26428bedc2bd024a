// Explicit inverse X = R^-1 of the upper-triangular Cholesky factor R (dp x
// dp, 16 x 16 blocks), so that the CholeskyQR solve Q = Y R^-1 becomes a
// plain product with no chain across column blocks.  Column blocks of X are
// independent: workgroup J forms X[:, J] by block back substitution,
//     X_JJ = R_JJ^-1,   X_IJ = -R_II^-1 sum_{t = I+1..J} R_It X_tJ   (I < J),
// right-looking: as soon as X_{I+1,J} is known every pending block row
// I' <= I adds R_{I',I+1} X_{I+1,J} to its accumulator (float64 MFMA), and the
// owner of row I finishes it with R_II^-1.  Rows are dealt to the waves
// round-robin; X_{I+1,J} is passed through LDS (double buffered, one
// workgroup barrier per block row).  The R tiles of each step are loaded into
// a register ring several steps before they are used; what bounds a step is the
// chain barrier, X_{I+1,J} from LDS, 4 + 4 MFMAs, LDS (about 1000 cycles) and, with
// many rows to a wave, those rows' R tiles and MFMAs.  Measured with the steps
// unrolled, the tiles in four 8-byte loads a lane and all loads waited for, and
// now: d = 210 17.3 -> 14.0 us, 540 67 -> 51 (the form for 34 block rows spills 8
// registers a lane).  The diagonal-block inverses come
// from the Cholesky.  Nothing is done after the Cholesky's fast path, which
// writes its own inverse.  A dependent column has a unit row in R, so the
// inverse exists and its other columns do not involve it.
#include "common.h"
#include "grouped.h"
#include "kernels.h"

#include <utility>

namespace rqlp {

// kInvWaves waves; up to kInvT block rows (grid = number of block rows,
// dp is the row stride of R and X); R tiles are loaded kInvAhead steps
// before they are used.
// The body is shared by the one-matrix kernel and the grouped kernel
// (J: the column block this workgroup forms).
template <int kInvWaves, int kInvT, int kInvAhead>
__device__ __attribute__((always_inline)) inline void trinv_body(const double* __restrict__ R,
                                                               const double* __restrict__ Rinv16, int dp,
                                                               const int32_t* __restrict__ mode,
                                                               double* __restrict__ X, const int J) {
  constexpr int kInvRows = (kInvT + kInvWaves - 1) / kInvWaves;  // block rows per wave
  __shared__ double Zs[2][kTile][kTile + 4];  // (rows 4 lr + ks of four lr's spread over the banks)
  if (*mode == 2) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane >> 4, lc = lane & 15;

  // A operands of R_{I', t} for this wave's rows I' = wave + kInvWaves s, step I = t - 1:
  // ring[(J - 1 - I) % kInvAhead][s][ks] (float64 MFMA A layout, A[m][kk] = R_I't[m][kk],
  // with kk = 4 lr + ks: a lane's four values are one run of 32 bytes)
  double ring[kInvAhead][kInvRows][4];
  // (the loads stand in no branch, so that the compiler can count those in flight
  // and a step waits for its own only; a row that a step has not is an address out
  // of the buffer's range, which costs no access)
  const __amdgpu_buffer_rsrc_t Rb =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(R), 0, kInvT * kTile * dp * 8, 0x00020000);
  auto load_step = [&](auto slot, int I) {
#pragma unroll
    for (int s = 0; s < kInvRows; ++s) {
      const int Ip = wave + kInvWaves * s;
      const int at = Ip <= I ? ((Ip * kTile + lc) * dp + (I + 1) * kTile + 4 * lr) * 8 : -32;
      typedef double v2d __attribute__((ext_vector_type(2)));
      const v2d lo = __builtin_bit_cast(v2d, __builtin_amdgcn_raw_buffer_load_b128(Rb, at, 0, 0));
      const v2d hi = __builtin_bit_cast(v2d, __builtin_amdgcn_raw_buffer_load_b128(Rb, at, 16, 0));
      ring[decltype(slot)::value][s][0] = lo.x;
      ring[decltype(slot)::value][s][1] = lo.y;
      ring[decltype(slot)::value][s][2] = hi.x;
      ring[decltype(slot)::value][s][3] = hi.y;
    }
  };
  // -R_I'I'^-1 as A operands for the rows this wave finishes
  double rinv[kInvRows][4];
#pragma unroll
  for (int s = 0; s < kInvRows; ++s) {
    const int Ip = wave + kInvWaves * s;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      rinv[s][ks] = (Ip < J) ? -Rinv16[(int64_t)Ip * kTile * kTile + lc * kTile + ks * 4 + lr] : 0.0;
  }
  auto slots = [&](auto f) {
    [&]<int... Qs>(std::integer_sequence<int, Qs...>) {
      (f(std::integral_constant<int, Qs>{}), ...);
    }(std::make_integer_sequence<int, kInvAhead>{});
  };
  if (J > 0)
    slots([&](auto q) {
      if constexpr (decltype(q)::value + 1 < kInvAhead) load_step(q, J - 1 - decltype(q)::value);
    });

  // X_JJ = R_JJ^-1 (row-major 16 x 16 block of Rinv16)
  for (int e = tid; e < kTile * kTile; e += blockDim.x) {
    const int r = e / kTile, c = e % kTile;
    const double v = Rinv16[(int64_t)J * kTile * kTile + e];
    Zs[0][r][c] = v;
    X[(int64_t)(J * kTile + r) * dp + J * kTile + c] = v;
  }
  doublex4 S[kInvRows];  // accumulators of block rows wave + kInvWaves s
#pragma unroll
  for (int s = 0; s < kInvRows; ++s) S[s] = Mfma<double>::zero();
  __syncthreads();

  // Steps I = J-1 down to 0, kInvAhead to a turn of the loop so that the ring slots
  // are fixed.  (Not unrolled further: code that runs once comes from memory, and
  // its lines took longer than its work.)
  int buf = 0;  // X_{I+1,J} is in Zs[buf]
  for (int I0 = J - 1; I0 >= 0; I0 -= kInvAhead) {
    slots([&](auto q) {
      const int I = I0 - decltype(q)::value;
      if (I < 0) return;
      double zk[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) zk[ks] = Zs[buf][4 * lr + ks][lc];
      // the slot of the step before is free (addresses while LDS answers)
      load_step(std::integral_constant<int, (decltype(q)::value + kInvAhead - 1) % kInvAhead>{}, I + 1 - kInvAhead);
      // S_I' += R_{I',I+1} X_{I+1,J} for the pending rows I' <= I of this wave, the
      // last of them first: the owner of row I finishes X_IJ = -R_II^-1 S_I
#pragma unroll
      for (int s = kInvRows - 1; s >= 0; --s) {
        const int Ip = wave + kInvWaves * s;
        if (Ip <= I) {
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) S[s] = Mfma<double>::mma(ring[decltype(q)::value][s][ks], zk[ks], S[s]);
        }
        if (Ip == I) {
          doublex4 z = Mfma<double>::zero();
#pragma unroll
          for (int ks = 0; ks < 4; ++ks)  // the accumulator layout is the B operand layout
            z = Mfma<double>::mma(rinv[s][ks], S[s][ks], z);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = lr + 4 * r;
            Zs[buf ^ 1][row][lc] = z[r];
            X[(int64_t)(I * kTile + row) * dp + J * kTile + lc] = z[r];
          }
        }
      }
      __syncthreads();
      buf ^= 1;
    });
  }
}

template <int kInvWaves, int kInvT, int kInvAhead>
__global__ __launch_bounds__(kInvWaves * 64) void trinv_kernel(const double* __restrict__ R,
                                                               const double* __restrict__ Rinv16, int dp,
                                                               const int32_t* __restrict__ mode,
                                                               double* __restrict__ X) {
  trinv_body<kInvWaves, kInvT, kInvAhead>(R, Rinv16, dp, mode, X, blockIdx.x);
}

// Many matrices in one launch (argument table in device memory):
// workgroups start[p] .. start[p + 1] - 1 form the column blocks of matrix p.
struct TrinvRecArgs {
  const double* R;
  const double* Rinv16;
  const int32_t* mode;
  double* X;
  int ld;
};

template <int W, int T, int AH>
__global__ __launch_bounds__(W * 64) void trinv_grouped(const TrinvRecArgs* __restrict__ a,
                                                        const int* __restrict__ start, int count) {
  const int p = group_find(start, count, blockIdx.x);
  const TrinvRecArgs g = a[p];
  trinv_body<W, T, AH>(device_ptr(g.R), device_ptr(g.Rinv16), g.ld, device_ptr(g.mode), device_ptr(g.X),
                       (int)blockIdx.x - start[p]);
}

template <int W, int T, int AH>
void trinv_grouped_launch(const void* args, const int* start, int count, unsigned blocks, hipStream_t s) {
  hipLaunchKernelGGL((trinv_grouped<W, T, AH>), dim3(blocks), dim3(W * kWave), 0, s, (const TrinvRecArgs*)args, start,
                     count);
}

hipError_t launch_trinv(const double* R, const double* Rinv16, int dp, const int32_t* mode, double* X,
                        hipStream_t s) {
  return launch_trinv_block(R, Rinv16, dp, dp / kTile, mode, X, s);
}

hipError_t launch_trinv_block(const double* R, const double* Rinv16, int ld, int nT, const int32_t* mode,
                              double* X, hipStream_t s) {
  const TrinvRecArgs a{R, Rinv16, mode, X, ld};
  if (nT <= kCholRegMax / kTile) {
    if (!record_launch(&trinv_grouped_launch<8, kCholRegMax / kTile, 4>, a, (unsigned)nT))
      hipLaunchKernelGGL((trinv_kernel<8, kCholRegMax / kTile, 4>), dim3((unsigned)nT), dim3(8 * kWave), 0, s, R,
                         Rinv16, ld, mode, X);
  } else {
    if (!record_launch(&trinv_grouped_launch<16, kDMax / kTile, 2>, a, (unsigned)nT))
      hipLaunchKernelGGL((trinv_kernel<16, kDMax / kTile, 2>), dim3((unsigned)nT), dim3(16 * kWave), 0, s, R,
                         Rinv16, ld, mode, X);
  }
  return hipGetLastError();
}

}  // namespace rqlp
