// Back-transformation of eigenvectors by the stored Householder reflectors of a
// tridiagonal or Hessenberg reduction (device part of the small eigensolvers).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ka {

// x + its 16-lane rotations by 8, 4, 2, 1: the sum over a row of 16 lanes, the same in each
template <int ROR>
__device__ __forceinline__ double row_rotate(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x120 + ROR, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x120 + ROR, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

__device__ __forceinline__ double row_sum16(double x) {
  x += row_rotate<8>(x);
  x += row_rotate<4>(x);
  x += row_rotate<2>(x);
  x += row_rotate<1>(x);
  return x;
}

// the sum over a wave, the same in each lane
__device__ __forceinline__ double wave_sum(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, row_sum16(x));
  auto row = [&](int l) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, l), hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
  };
  return (row(0) + row(16)) + (row(32) + row(48));
}

// One wave per 4 vectors, 16 lanes per vector.  Lane r of a vector holds its
// elements r, r + 16, ... (NS of them, n <= 16 NS) in registers; for each
// reflector the 16 lanes form the dot product, then update their own elements.
// No barriers: every wave walks the reflectors on its own, requesting them kD
// ahead.  Reflector j: rows j + 1 .. n - 1 of column j of A (n x n), times beta[j].
// Element i of vector `col` at V[i ld + col].
//
// The time is the chain over the reflectors, about 0.5 us each: 59 us for a
// Rayleigh-Ritz step of the solve for 50 Galerkin pairs with blocks of 16.  (303 us with one thread per
// vector and a reflector at a time through LDS; 150 us like this without
// leaving out the elements a reflector does not reach.)
template <int NS>
__device__ __forceinline__ void back_wave(const double* __restrict__ A, const double* __restrict__ beta, int n,
                                          double* __restrict__ V, int64_t ld, int col, bool act) {
  constexpr int kD = NS <= 16 ? 4 : (NS <= 32 ? 2 : 1);
  const int r = threadIdx.x & 15;
  double x[NS], v[kD][NS], b[kD];
  int zero = 0;
  asm("" : "+v"(zero));   // beta through vector loads too: scalar loads return in any order, and each wait takes all
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = r + 16 * s;
    x[s] = (act && i < n) ? V[(int64_t)i * ld + col] : 0.0;
  }
  uint32_t at[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) at[s] = r + 16 * s < n ? r + 16 * s : n - 1;
  // (16 elements that a reflector does not reach are neither read nor changed)
  auto load = [&](int d, int j) {
    if (j < 0) return;
    const double* a = A + (int64_t)j * n;
    b[d] = beta[j + zero];
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (16 * s + 15 > j) v[d][s] = a[at[s]];
  };
#pragma unroll
  for (int d = 0; d < kD; ++d) load(d, n - 3 - d);
  for (int j0 = n - 3; j0 >= 0; j0 -= kD) {
#pragma unroll
    for (int d = 0; d < kD; ++d) {
      const int j = j0 - d;
      if (j < 0) break;
      double dot = 0.0;
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (16 * s + 15 > j) {
          const int i = r + 16 * s;
          v[d][s] = (i > j && i < n) ? v[d][s] : 0.0;
          dot += v[d][s] * x[s];
        }
      const double sc = b[d] == 0.0 ? 0.0 : b[d] * row_sum16(dot);
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (16 * s + 15 > j) x[s] -= sc * v[d][s];
      load(d, j - kD);
    }
  }
  if (act)
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int i = r + 16 * s;
      if (i < n) V[(int64_t)i * ld + col] = x[s];
    }
}

}  // namespace ka
