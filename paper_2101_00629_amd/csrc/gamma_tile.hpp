// Pieces shared by the kernel-product tiles of gamma.hip (FP32 and split BF16)
// and gamma_f16x3.hip (split FP16): work-item mapping, kernel exponent, row
// boxes and the centred Gram form.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ka_internal.hpp"

namespace ka {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef double d4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr int kXcds = 8;        // MI355X: workgroups are dealt to the 8 XCDs round-robin by id
constexpr int kCT = 64;         // columns per LDS tile
// MFMA accumulators are flushed into running totals every 2 tiles (128
// columns, 32 chained MFMAs per FP32 accumulator): FP64 totals in the FP32
// path, FP32 totals in the BF16x3 path.  The FP32 chain length is
// what sets the arithmetic noise of the product: measured on the 287,496-point
// Gaussian operator, 8-tile chains gave 1.8e-6 relative error on the smallest
// of 200 eigenvalues (1.4% of the largest), 2-tile chains 3.8e-7, at the same
// speed within 1%.
constexpr int kFlushTiles = 2;
constexpr double kL2FitBytes = 3.0 * (1 << 20);   // column data per split that an XCD's L2 keeps


// (row block, split) of this workgroup.  Grouped grid (xcd_splits > 0): a 1-D
// grid of row_blocks * xcd_splits workgroups; workgroup id L runs on XCD
// L % 8, and the XCD's own sequence L / 8 walks split by split (all row
// blocks of a split back to back), splits x, x + 8, ... on XCD x.  Returns
// false for padding workgroups (split beyond the real split count).
__device__ __forceinline__ bool gamma_item(const GammaLaunch& a, int64_t& rblk, int& split) {
  if (a.xcd_splits == 0) {
    rblk = blockIdx.x;
    split = blockIdx.y;
    return true;
  }
  const int64_t L = blockIdx.x;
  const int x = (int)(L % kXcds);
  const int64_t j = L / kXcds;
  rblk = j % a.row_blocks;
  split = x + kXcds * (int)(j / a.row_blocks);
  return split < a.nsplit;
}

template <int KERNEL>
__device__ __forceinline__ float pair_exponent(float dx, float dy, float dz) {
  if constexpr (KERNEL == KA_GAUSSIAN) {
    float s = dx * dx;
    s = __builtin_fmaf(dy, dy, s);
    return __builtin_fmaf(dz, dz, s);
  } else {
    return (__builtin_fabsf(dx) + __builtin_fabsf(dy)) + __builtin_fabsf(dz);
  }
}

__device__ __forceinline__ float load_coord(const float* p, int64_t i, int stride, int k, float scale) {
  return p[i * stride + k] * scale;
}

// Centred Gram form of the Gaussian exponent (shown for the FP32 path).  With c the centre
// of the bounding box of a workgroup's rows, xt = x - c and yt = y - c (scaled
// coordinates),
//     2^-|x - y|^2 = 2^-|xt|^2 * 2^((2 yt) . xt - |yt|^2),
// so the exponents of 16 x 16 pairs, less the row term, are one
// v_mfma_f32_16x16x4_f32: A holds (2 yt, -|yt|^2) of 16 columns and B holds
// (xt, 1) of 16 rows; the row factor 2^-|xt|^2 multiplies the finished row of
// the product.  Lane l of the result holds row l % 16 against four columns,
// which is where the kernel product's A operand expects Gamma when column
// 4 * (m % 4) + m / 4 of the group is put in A row m: result entry r of lane l
// is then column 4 r + l / 16, the column of k-slot l / 16 in product step
// 4 r.  This replaces three differences and three multiply-adds per pair by
// 1/64 of an MFMA.  Rounding: the terms are of size R^2 (R the half-diagonal
// of the rows' box) where the difference form's are of size |x - y|^2, so the
// form is taken only for boxes with R^2 <= kGramR2 in scaled units (the
// exponent is then off by a few units of 2^-24 R^2 at most, Gamma by ln 2
// times that relative, and the factored terms stay below 2^(R^2)); wider row
// blocks keep the difference form.  Row blocks of tensor-grid points in their
// natural order qualify at the workload sizes: R^2 = 9.0 on the 66^3 cube at
// ell = 0.2 (18.0 for the blocks that straddle two z-layers), at most 11.5 on
// the quarter annulus r in [1, 2] at ell = 0.5.  The cut takes in the
// straddling blocks on purpose: workgroups of one launch that run the two
// forms at different speeds drift apart in their column streams and stop
// sharing the XCD's L2 (measured on the 66^3 launch with a cut of 16: 5x the
// HBM fetch, 29.7 GB against 5.9 GB per launch).
constexpr float kGramR2 = 20.f;

// Bounding box of a wave's rows (lanes l and l + 16 hold the same rows) into
// the wave's entry of s_box: lo in [0..2], hi in [4..6].
template <int RB>
__device__ __forceinline__ void gram_box_put(const float* rx, const float* ry, const float* rz, int lane, int wave,
                                             float (*s_box)[8]) {
  float lo[3] = {rx[0], ry[0], rz[0]}, hi[3] = {rx[0], ry[0], rz[0]};
#pragma unroll
  for (int rb = 1; rb < RB; ++rb) {
    lo[0] = fminf(lo[0], rx[rb]); hi[0] = fmaxf(hi[0], rx[rb]);
    lo[1] = fminf(lo[1], ry[rb]); hi[1] = fmaxf(hi[1], ry[rb]);
    lo[2] = fminf(lo[2], rz[rb]); hi[2] = fmaxf(hi[2], rz[rb]);
  }
#pragma unroll
  for (int o = 1; o < 16; o <<= 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lo[k] = fminf(lo[k], __shfl_xor(lo[k], o));
      hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], o));
    }
  if (lane < 3) {
    s_box[wave][lane] = lane == 0 ? lo[0] : (lane == 1 ? lo[1] : lo[2]);
    s_box[wave][4 + lane] = lane == 0 ? hi[0] : (lane == 1 ? hi[1] : hi[2]);
  }
}

// After gram_box_put on every wave: a barrier, then the centre of the
// workgroup's box and whether the Gram form applies (uniform over the
// workgroup).  The barrier also orders this read before any later rewrite of
// s_box: every wave passes at least one more barrier before its next item.
__device__ __forceinline__ bool gram_box_take(float (*s_box)[8], float& cx, float& cy, float& cz) {
  __syncthreads();
  float lo[3], hi[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    lo[k] = fminf(fminf(s_box[0][k], s_box[1][k]), fminf(s_box[2][k], s_box[3][k]));
    hi[k] = fmaxf(fmaxf(s_box[0][4 + k], s_box[1][4 + k]), fmaxf(s_box[2][4 + k], s_box[3][4 + k]));
  }
  cx = 0.5f * (lo[0] + hi[0]);
  cy = 0.5f * (lo[1] + hi[1]);
  cz = 0.5f * (lo[2] + hi[2]);
  const float ex = 0.5f * (hi[0] - lo[0]), ey = 0.5f * (hi[1] - lo[1]), ez = 0.5f * (hi[2] - lo[2]);
  return __builtin_amdgcn_readfirstlane((int)(ex * ex + ey * ey + ez * ez <= kGramR2)) != 0;
}

// A-operand data of one column in the Gram form: (2 yt, -|yt|^2) from the raw
// coordinates.
__device__ __forceinline__ float4 gram_column(float4 raw, float scale, float cx, float cy, float cz) {
  const float tx = raw.x * scale - cx, ty = raw.y * scale - cy, tz = raw.z * scale - cz;
  return make_float4(2.f * tx, 2.f * ty, 2.f * tz, -__builtin_fmaf(tz, tz, __builtin_fmaf(ty, ty, tx * tx)));
}

// The row factor 2^-|xt|^2 of the Gram form.
__device__ __forceinline__ double gram_row_factor(const GammaLaunch& a, int64_t row, float cx, float cy, float cz) {
  const float tx = load_coord(a.xr, row, a.xr_stride, 0, a.coord_scale) - cx;
  const float ty = load_coord(a.xr, row, a.xr_stride, 1, a.coord_scale) - cy;
  const float tz = load_coord(a.xr, row, a.xr_stride, 2, a.coord_scale) - cz;
  return exp2(-(double)__builtin_fmaf(tz, tz, __builtin_fmaf(ty, ty, tx * tx)));
}

// Row box of a work item and whether the centred Gram form applies to it
// (Gaussian kernel only); contains a workgroup barrier.
template <int RB>
__device__ __forceinline__ bool gram_rows(const GammaLaunch& a, int64_t rblk, float (*s_box)[8], float& cx,
                                          float& cy, float& cz) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t row0 = rblk * (4 * 16 * RB) + wave * 16 * RB;
  float rx[RB], ry[RB], rz[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    int64_t r = row0 + 16 * rb + (lane & 15);
    if (r >= a.nr) r = a.nr - 1;
    rx[rb] = load_coord(a.xr, r, a.xr_stride, 0, a.coord_scale);
    ry[rb] = load_coord(a.xr, r, a.xr_stride, 1, a.coord_scale);
    rz[rb] = load_coord(a.xr, r, a.xr_stride, 2, a.coord_scale);
  }
  gram_box_put<RB>(rx, ry, rz, lane, wave, s_box);
  return gram_box_take(s_box, cx, cy, cz);
}

}  // namespace ka
