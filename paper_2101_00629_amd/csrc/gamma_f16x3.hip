// Split-FP16 kernel product: the FP32 product of gamma.hip with its
// contraction on the FP16 matrix cores.
//
// Contraction.  A value x of FP32 is kept as the sum of two FP16 parts, hi =
// fp16(x) and lo = fp16(x - hi): 11 + 11 significant bits and lo's sign, so
// three quarters of all values are exact and the others 2^-23 |x| off.  Then
// Gamma Y = hi hi + hi lo + lo hi, three v_mfma_f32_16x16x32_f16 that
// accumulate in FP32; the dropped lo lo is below 2^-22 of the product and of
// either sign.  (The scheme of Markidis et al. 2018 and Ootomo & Yokota 2022
// for FP32 products on FP16 matrix units.)  The cross terms have accumulators
// of their own: they are 2^11 smaller, so only the hi hi chain (16 MFMAs per
// 512 columns) rounds at the size of the sum, and the result is closer to FP64
// than that of FP32 MFMAs (relative 2-norm error, N(0, 1) blocks: 1.8e-7
// against 3.9e-7 at 287,496^2, b = 64, Gaussian; 1.5-1.9e-7 against 2.0-2.5e-7
// at 12,167^2, b = 16).
//
// Range.  FP16 has 5 exponent bits where FP32 has 8.  Every vector of Y has a
// scale per group of 512 columns that takes its largest entry there just below
// 2^15, and every row a scale per group that takes Gamma at the row's distance
// from the group's bounding box just below 2^15 (both powers of two; the FP64
// totals undo them).  What is lost is relative accuracy below 2^-16 of the
// largest Gamma or Y of a group, an absolute 2^-40 of that.  Groups with
// values that are not finite are added pair by pair (no scale would hold).
//
// Exponents (Gaussian).  16 x 16 exponents -|x - y|^2 come from one
// v_mfma_f32_16x16x32_f16.  Coordinates (scaled, relative to the launch's
// centre, its middle row, FP64) are split as h + l with h on a lattice of 1/64:
//   -(x - y)^2 = -(hx - hy)^2 + 2 hx ly + 2 hy lx + 2 lx ly
//                - (2 hy + ly) ly - (2 hx + lx) lx.
// The unit sums eight products at a time, in the order of the k index, into
// the FP32 accumulator (measured: products aligned to the block's largest with
// two more bits than FP32, then rounded to nearest).  The first block holds
// the lattice part, whose terms and sum are multiples of 2^-12 below 2^12 and
// so exact; the other three hold the small terms, one coordinate each, every
// factor in as many FP16 parts as it has bits.  Nothing cancels, so the
// exponent is rounded at its own size (FP32 in the centred Gram form of
// gamma.hip: at the size of the row block), and the operands do not depend on
// the workgroup: the pre-pass forms them once.  The last term, the row's own,
// is a factor of the row.  The form is exact within |coordinate| < 31 and
// |point|^2 < 2000 (scaled units: 26 correlation lengths each way); workgroups
// that meet a point outside it take differences on the VALU, as the
// exponential kernel does.
//
// What bounds it (287,496^2, b = 64, Gaussian, 32.5 ms = 2.54e12 pairs/s against
// 91 ms on the FP32 matrix cores): matrix cores 54% and VALU 65% of the cycles,
// 23% of them together, so that either is busy 97% of the time, at 2.0 GHz (the
// power limit; 2.4 GHz nominal).  The same instructions without any memory
// access, on random operands, run at 3.1e12 (b = 64), 4.4e12 (b = 32; the
// kernel 3.9e12) and 5.5e12 (b = 16; 5.0e12) pairs/s.  v_mfma_f32_32x32x16_f16
// was no faster there (2.9-3.1e12 at b = 64).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "gamma_tile.hpp"
#include "ka_internal.hpp"

namespace ka {

typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef float f2v __attribute__((ext_vector_type(2)));

// Columns that share one scale per vector of Y; their sums go to the FP64
// totals together.
constexpr int kGroup = 512;
constexpr int kGroupTiles = kGroup / kCT;
constexpr int kPreThreads = 1024;           // of the pre-pass, one workgroup per group
constexpr int kXEntries = 256;              // uint4 of column operands per tile
constexpr float kLat = 64.f;                // 1 / spacing of the coordinate lattice

enum { kBadValue = 1, kOffLattice = 2 };   // flags of a column group

template <int B>
constexpr int h16_entries() { return (kCT / 32) * (B / 16) * 64; }   // uint4 per 64-column tile and part

__device__ __forceinline__ bool finite_bits(float x) {
  return (__builtin_bit_cast(uint32_t, x) & 0x7f800000u) != 0x7f800000u;
}

__device__ __forceinline__ uint32_t pack_h2(float a, float b) {
  const f2v v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, h2v));
}

__device__ __forceinline__ float half_of(float x) { return (float)(_Float16)x; }

// a value that is the same in every lane, in a scalar register
__device__ __forceinline__ float uniform(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}

// Scaled FP64 coordinate relative to the launch's centre
__device__ __forceinline__ double lattice_coord(const GammaLaunch& a, float x, double c) {
  return (double)x * ((double)a.coord_scale + (double)a.coord_scale_lo) - c;
}

// The launch's centre: its middle row, on the lattice.
__device__ __forceinline__ void launch_centre(const GammaLaunch& a, double (&c)[3]) {
  const float* x = a.xr + (a.nr / 2) * a.xr_stride;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double v = rint(lattice_coord(a, x[k], 0.0) * kLat) / kLat;
    c[k] = v - v == 0.0 ? v : 0.0;
  }
}

struct LatticePoint {
  float h[3], l[3];   // coordinate = h + l, h on the lattice
  bool ok;            // in the range where the Gram form is exact
};

__device__ __forceinline__ LatticePoint lattice_point(const GammaLaunch& a, const float* x, const double (&c)[3]) {
  LatticePoint p;
  float n = 0.f;
  p.ok = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double t = lattice_coord(a, x[k], c[k]);
    const bool in = fabs(t) < 31.0;
    p.ok = p.ok && in;
    const double h = in ? rint(t * kLat) / kLat : 0.0;
    p.h[k] = (float)h;
    p.l[k] = in ? (float)(t - h) : 0.f;
    n += p.h[k] * p.h[k];
  }
  p.ok = p.ok && n < 2000.f;
  return p;
}

// ---------------------------------------------------------------------------
// pre-pass: Y and the column points into FP16 operands
//
// One workgroup of 1024 threads per group of 512 columns: a thread holds 8, 16
// or 32 values of one vector of Y, all loaded before use, so a launch of a few
// groups is one memory latency long (256 threads that read the group twice took
// 80 us for 3,375 columns at b = 64, where the product itself takes 25).
// Y's fragments lie as the product's LDS tiles hold them: entry (ks NT + t) 64
// + lane of a 64-column tile is the MFMA B operand of vectors 16 t .. + 15 and
// columns 32 ks .. + 31 (lane 16 g + n: vector n, columns 8 g .. + 7), hi parts
// first.  Vectors that do not count (a block application of fewer than b leaves
// there what an earlier one wrote) are taken as zero: the groups' flags are
// common to all vectors.  Gram operands: fragment (ks, w), lane 16 q + m is block q of column
// 32 ks + 8 (m / 4) + 4 w + m % 4, the column whose exponent the product wants
// in result m % 4 of lane group m / 4.
// ---------------------------------------------------------------------------
template <int B>
__device__ __forceinline__ void split16_group(const GammaLaunch& a, int kernel, int64_t g, float (*s_m)[B], float* s_up,
                                              int* s_flag, float (*s_b)[8]) {
  constexpr int NT = B / 16;
  constexpr int G = kGroup, GT = kGroupTiles;
  constexpr int PARTS = kPreThreads / B;
  constexpr int CPT = G / PARTS;        // columns per thread: 8, 16 or 32
  constexpr int E = h16_entries<B>();
  const int j = threadIdx.x % B, part = threadIdx.x / B;
  const int64_t c0 = g * G + part * CPT;
  float y[CPT];
#pragma unroll
  for (int u = 0; u < CPT; ++u) y[u] = c0 + u < a.nc && j < a.nv ? a.Y[(c0 + u) * B + j] : 0.f;
  float m = 0.f;
  int flag = 0;
#pragma unroll
  for (int u = 0; u < CPT; ++u) {
    if (!finite_bits(y[u])) flag |= kBadValue;
    m = fmaxf(m, __builtin_fabsf(y[u]));
  }
  if (threadIdx.x == 0) *s_flag = 0;
  s_m[part][j] = m;
  // the column points: their places on the lattice, and the group's box
  double c[3];
  launch_centre(a, c);
  LatticePoint p;
  const int64_t col = g * G + threadIdx.x;
  const bool in = threadIdx.x < G && col < a.nc;
  float x[3] = {0.f, 0.f, 0.f}, lo[3], hi[3];
  if (in)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      x[k] = a.xc[col * a.xc_stride + k];
      if (!finite_bits(x[k])) flag |= kBadValue;
    }
  p = lattice_point(a, x, c);
  if (in && !p.ok) flag |= kOffLattice;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float t = (float)lattice_coord(a, x[k], c[k]);
    lo[k] = in ? t : INFINITY;
    hi[k] = in ? t : -INFINITY;
    if (!in || !p.ok) p.h[k] = p.l[k] = 0.f;
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lo[k] = fminf(lo[k], __shfl_xor(lo[k], o));
      hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], o));
    }
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      s_b[threadIdx.x >> 6][k] = lo[k];
      s_b[threadIdx.x >> 6][4 + k] = hi[k];
    }
  __syncthreads();
  if (flag) atomicOr(s_flag, flag);
#pragma unroll
  for (int q = 0; q < PARTS; ++q) m = fmaxf(m, s_m[q][j]);
  int ex = 0;
  if (m > 0.f && finite_bits(m)) (void)__builtin_frexpf(m, &ex);   // m in [2^(ex-1), 2^ex)
  const int up = 15 - ex;                                             // |y| 2^up < 2^15
  if (part == 0) {
    s_up[j] = (float)up;
    a.yup[g * B + j] = (float)up;
  }
  __syncthreads();
  const bool bad = (*s_flag & kBadValue) != 0;   // its columns are added by the product's slow loop instead
  if (threadIdx.x == 0) {
    float* b = a.gbox + 8 * g;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      float l = s_b[0][k], h = s_b[0][4 + k];
#pragma unroll
      for (int w = 1; w < G / 64; ++w) {
        l = fminf(l, s_b[w][k]);
        h = fmaxf(h, s_b[w][4 + k]);
      }
      b[k] = bad ? -1e30f : l;
      b[4 + k] = bad ? 1e30f : h;
    }
    b[3] = (float)*s_flag;
    b[7] = 0.f;
  }
  if (kernel == KA_GAUSSIAN && threadIdx.x < G) {
    // fragment (ks, half), lane 16 q + m of the column's tile
    const int cg = threadIdx.x, ct = cg & 31, vec = cg & 63;
    uint4* dst = a.xs + (g * GT + cg / kCT) * kXEntries + (((cg & 63) >> 5) * 2 + ((ct >> 2) & 1)) * 64 +
                 4 * (ct >> 3) + (ct & 3);
    // (a column that is none, or of a group that is not finite, is put so far
    // off that Gamma is zero whatever the row's scale)
    const float n = bad || !in ? -30000.f : -(p.h[0] * p.h[0] + p.h[1] * p.h[1] + p.h[2] * p.h[2]);
    // the last slot meets a zero of the rows' operand: it carries the scale of vector `vec`
    dst[0] = make_uint4(pack_h2(p.h[0], p.h[1]), pack_h2(p.h[2], n), pack_h2(n - half_of(n), 1.f),
                        pack_h2(1.f, vec < B ? s_up[vec] : 0.f));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float l = p.l[k] * kLat, b = -l * (2.f * p.h[k] + p.l[k]);
      const float b1 = b - half_of(b);
      dst[16 * (k + 1)] = make_uint4(pack_h2(l, l - half_of(l)), pack_h2(p.h[k] / kLat, p.h[k] / kLat), pack_h2(l, b),
                                     pack_h2(b1, b1 - half_of(b1)));
    }
  }
#pragma unroll
  for (int v = 0; v < CPT / 8; ++v) {
    const int cg = part * CPT + 8 * v;        // in the group
    uint32_t h[4], l[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float y0 = bad ? 0.f : __builtin_ldexpf(y[8 * v + 2 * u], up);
      const float y1 = bad ? 0.f : __builtin_ldexpf(y[8 * v + 2 * u + 1], up);
      h[u] = pack_h2(y0, y1);
      l[u] = pack_h2(y0 - half_of(y0), y1 - half_of(y1));
    }
    const int64_t T = g * GT + cg / kCT;
    const int r = ((cg % kCT) / 32 * NT + j / 16) * 64 + 16 * ((cg % 32) / 8) + (j & 15);
    a.ys[2 * E * T + r] = make_uint4(h[0], h[1], h[2], h[3]);
    a.ys[2 * E * T + E + r] = make_uint4(l[0], l[1], l[2], l[3]);
  }
}

template <int B>
__global__ __launch_bounds__(kPreThreads) void gamma_split16_kernel(GammaLaunch a, int kernel) {
  __shared__ float s_m[kPreThreads / B][B];
  __shared__ float s_up[B];
  __shared__ float s_b[kPreThreads / 64][8];
  __shared__ int s_flag;
  split16_group<B>(a, kernel, blockIdx.x, s_m, s_up, &s_flag, s_b);
}

// ---------------------------------------------------------------------------
// product
//
// A workgroup of 4 waves owns 64 RB rows; columns stream through LDS in tiles
// of 64.  A step is 16 rows x 32 columns, 8 pairs per lane: while its MFMAs
// run, the wave forms the kernel values of the next step (exponents ready) and
// starts the exponents of the one after.  The vector work is cut into 12 pieces
// set between the MFMAs; a scheduling barrier after each keeps them there.
// (Splitting a value costs a multiply, one half of a packed conversion, a
// v_fma_mix_f32 and another half: 8 cycles of vector issue a pair.  Two
// v_fma_mix{lo,hi}_f16 would do it in two instructions, but these issue at half
// rate: 16 cycles.)
//
// Tiles go from memory straight to LDS, Y three tiles ahead and the column
// operands four, with one barrier per tile.  It stands before the last step:
// by then every LDS read of the tile has been issued and waited for, the loads
// it waits for were issued two barriers before, and the next tile's operands
// arrive while the last step's MFMAs run.  yl is read again for the next 32
// columns as soon as its last MFMA is issued, yh after the step, so one set of
// registers is enough; that is what the second accumulator costs at b = 64.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef __attribute__((address_space(4))) float uniform_float;   // read through the scalar cache

// 16 bytes per lane from base + voff to LDS at `lds` (uniform) + 16 lane.  In
// assembly because the compiler, which cannot tell the slots of a ring apart,
// waits for every load to LDS before each later read of it; the kernel waits
// by count at its barriers instead.  It has no register result.
__device__ __forceinline__ void load_to_lds(const void* base, uint32_t voff, void* lds) {
  const uint32_t l = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr)lds);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(l), "v"(voff), "s"(base)
               : "memory", "m0");
}

constexpr int kYRing = 3;     // tiles of Y in LDS
constexpr int kVm0 = (7 << 4) | (15 << 8);   // s_waitcnt: vmcnt(0) alone
constexpr int kXRing = 4;     // tiles of column operands in LDS

// Scaled FP32 coordinate relative to a workgroup's centre (difference form; row_centre)
__device__ __forceinline__ float centred(const GammaLaunch& a, float x, float c) {
  return __builtin_fmaf(x, a.coord_scale_lo, __builtin_fmaf(x, a.coord_scale, -c));
}

// Centre of a workgroup's rows along direction k for the difference form: the
// middle of their box, or zero where that would cost a row accuracy.  A
// coordinate is rounded at its distance from the centre, half the box's extent
// at most.  That is taken if no row lies nearer to zero than that, or if it is
// below 16 (Gaussian) or 32 scaled units: two coordinates 2^-21 (2^-20) off
// change an exponent d^2 with d <= 2 by 4e-6 at most (a distance by 2e-6).  One
// row far from the others of its block must not round theirs away.
template <int KERNEL>
__device__ __forceinline__ float row_centre(const float (*s_box)[8], int k, float mid) {
  const float lo = fminf(fminf(s_box[0][k], s_box[1][k]), fminf(s_box[2][k], s_box[3][k]));
  const float hi = fmaxf(fmaxf(s_box[0][4 + k], s_box[1][4 + k]), fmaxf(s_box[2][4 + k], s_box[3][4 + k]));
  const float half = 0.5f * (hi - lo), nearest = fmaxf(lo, -hi);
  // (rows at infinity: zero)
  return finite_bits(mid) && half <= fmaxf(nearest, KERNEL == KA_GAUSSIAN ? 16.f : 32.f) ? mid : 0.f;
}

template <int KERNEL, int B, int RB, bool GRAM>
__device__ __forceinline__ void gamma_h16_tile(const GammaLaunch& a, int64_t rblk, int split,
                                               uint4 (*s_x)[kXEntries], uint4 (*s_y)[2 * h16_entries<B>()],
                                               float c0, float c1, float c2, const double (&cl)[3], int flags,
                                               const float (*s_row)[64 * RB], float (*s_inv)[64 * RB]) {
  constexpr int NT = B / 16;
  constexpr int KS = kCT / 32;
  constexpr int S = KS * RB;                 // steps per tile: 16 rows x 32 columns each
  constexpr int E = h16_entries<B>();
  constexpr int G = kGroup, GT = kGroupTiles;
  constexpr int ROWS = 4 * 16 * RB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = lane >> 4;
  const int64_t row0 = rblk * ROWS + wave * 16 * RB;
  const int64_t c_begin = (int64_t)split * a.cols_per_split;
  const int64_t c_end = (c_begin + a.cols_per_split < a.nc) ? c_begin + a.cols_per_split : a.nc;

  // rows: Gram operand and factor, or centred coordinates
  h8v bx[RB];
  float Sr[RB], rx[RB], ry[RB], rz[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    int64_t r = row0 + 16 * rb + (lane & 15);
    if (r >= a.nr) r = a.nr - 1;
    const float* xr = a.xr + r * a.xr_stride;
    if constexpr (GRAM) {
      const LatticePoint p = lattice_point(a, xr, cl);
      const float m = -(p.h[0] * p.h[0] + p.h[1] * p.h[1] + p.h[2] * p.h[2]);
      const float h = q == 1 ? p.h[0] : (q == 2 ? p.h[1] : p.h[2]);
      const float l = (q == 1 ? p.l[0] : (q == 2 ? p.l[1] : p.l[2])) * kLat;
      const uint4 w0 = make_uint4(pack_h2(2.f * p.h[0], 2.f * p.h[1]), pack_h2(2.f * p.h[2], 1.f), pack_h2(1.f, m),
                                  pack_h2(m - half_of(m), 0.f));
      const uint4 w1 = make_uint4(pack_h2(2.f * h / kLat, 2.f * h / kLat), pack_h2(2.f * l, 2.f * (l - half_of(l))),
                                  pack_h2(2.f * l / (kLat * kLat), 1.f / kLat), pack_h2(1.f / kLat, 1.f / kLat));
      bx[rb] = __builtin_bit_cast(h8v, q == 0 ? w0 : w1);
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < 3; ++k) t -= (2.0 * p.h[k] + p.l[k]) * (double)p.l[k];
      Sr[rb] = (float)exp2(t);
    } else {
      // (a row at infinity stays there: Gamma = 0)
      auto row = [&](float x, float c) {
        const float t = centred(a, x, c);
        return finite_bits(t) ? t : x * a.coord_scale;
      };
      rx[rb] = row(xr[0], c0);
      ry[rb] = row(xr[1], c1);
      rz[rb] = row(xr[2], c2);
      Sr[rb] = 1.f;
    }
  }

  // Scale of a row's kernel values for the columns of group g, a power of two
  // just short of taking Gamma at the distance of the row from the group's box
  // to 2^15; the inverse goes to s_inv for the sums of the group (`par` its
  // parity).  Row points are read from LDS: this runs once per group.
  // The distance must not come out larger than the kernel's exponents have it,
  // or Gamma passes 2^16.  Box and row are rounded to FP32 relative to the
  // launch's centre, the exponents' coordinates relative to the workgroup's.  On
  // the lattice (below 31 units) that is nothing next to the factor of two in
  // hand; differences may be of any size, and there each gap is shortened by the
  // roundings it can hold: one of row and box, two each of the coordinates in a
  // difference, 6 of 2^-24, taken as 8.
  float Sg[RB];
  float gb[6];   // box of the next group
  const float off[3] = {uniform(__builtin_fabsf((float)cl[0]) + __builtin_fabsf(c0)),
                        uniform(__builtin_fabsf((float)cl[1]) + __builtin_fabsf(c1)),
                        uniform(__builtin_fabsf((float)cl[2]) + __builtin_fabsf(c2))};
  auto load_box = [&](int64_t g) {
    const uniform_float* b = (const uniform_float*)(uintptr_t)(a.gbox + 8 * (g < a.ngroups ? g : 0));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      gb[k] = b[k];
      gb[3 + k] = b[4 + k];
    }
  };
  auto row_scales = [&](int par) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int r = wave * 16 * RB + 16 * rb + (lane & 15);
      float d = 0.f;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float x = s_row[k][r];
        float gap = fmaxf(gb[k] - x, x - gb[3 + k]);
        if constexpr (!GRAM) {
          const float far = fmaxf(__builtin_fabsf(x), fmaxf(__builtin_fabsf(gb[k]), __builtin_fabsf(gb[3 + k])));
          gap -= 0x1p-21f * (far + off[k]);
        }
        gap = fmaxf(gap, 0.f);
        d += KERNEL == KA_GAUSSIAN ? gap * gap : gap;
      }
      const int up = 15 + (int)fminf(0.999f * d, 110.f);
      Sg[rb] = __builtin_ldexpf(Sr[rb], up);
      if (lane < 16) s_inv[par][r] = __builtin_ldexpf(1.f, -up);
    }
  };
  load_box(c_begin / G);
  row_scales(0);

  const f4v zero4 = {0.f, 0.f, 0.f, 0.f};
  f4v acc[RB][NT], accx[RB][NT];
  d4v tot[RB][NT];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      acc[rb][t] = zero4;
      accx[rb][t] = zero4;
      tot[rb][t] = (d4v){0.0, 0.0, 0.0, 0.0};
    }

  const int64_t ntile = (c_end - c_begin + kCT - 1) / kCT;
  const int64_t T0 = c_begin / kCT;
  // Y of tile ty and the column operands of tile tx on their way to LDS; past
  // the end the last tile again, so that every call counts the same loads.
  // Difference form: wave w < 3 takes coordinate w of the tile's columns, wave
  // 3 the scales.
  float raw = 0.f;
  auto fetch = [&](int64_t ty, int64_t tx, int yslot, int xslot) {
    ty = T0 + (ty < ntile ? ty : ntile - 1);
    tx = T0 + (tx < ntile ? tx : ntile - 1);
    if constexpr (!GRAM) {
      int64_t c = tx * kCT + lane;
      if (c >= a.nc) c = a.nc - 1;             // meets Y = 0
      raw = wave < 3 ? a.xc[c * a.xc_stride + wave] : a.yup[tx / GT * B + (lane & (B - 1))];
    }
    const uint4* src = a.ys + ty * (2 * E);
#pragma unroll
    for (int v = 0; v < 2 * E / kThreads; ++v) {
      const int e = v * kThreads + wave * 64;
      load_to_lds(src + e, 16u * lane, &s_y[yslot][e]);
    }
    if constexpr (GRAM) {
      const uint4* sx = a.xs + tx * kXEntries;
      load_to_lds(sx + wave * 64, 16u * lane, &s_x[xslot][wave * 64]);
    }
  };
  constexpr int kLoads = NT + (GRAM ? 1 : 0);   // loads to LDS per call and wave
  const float cw = wave == 0 ? c0 : (wave == 1 ? c1 : c2);
  auto stash = [&](int slot) {
    if constexpr (!GRAM) {
      float t = raw;
      if (wave < 3) {
        t = centred(a, raw, cw);
        if (!finite_bits(t)) t = 1e18f;        // Gamma = 0 here; its group is added by the slow loop
      }
      reinterpret_cast<float*>(&s_x[slot][0])[wave * kCT + lane] = t;
    }
  };
  uint4 ax[2];
  float4 px[2], py[2], pz[2];
  auto load_x = [&](int slot, int ks) {
    if constexpr (GRAM) {
      ax[0] = s_x[slot][(2 * ks) * 64 + lane];
      ax[1] = s_x[slot][(2 * ks + 1) * 64 + lane];
    } else {
      const float4* s = reinterpret_cast<const float4*>(&s_x[slot][0]) + (32 * ks + 8 * q) / 4;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        px[h] = s[h];
        py[h] = s[kCT / 4 + h];
        pz[h] = s[2 * kCT / 4 + h];
      }
    }
  };
  f4v d[2];
  auto gram = [&](int rb) {
    d[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8v, ax[0]), bx[rb], zero4, 0, 0, 0);
    d[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8v, ax[1]), bx[rb], zero4, 0, 0, 0);
  };
  auto comp = [](const float4 (&v)[2], int u) {
    const float4 w = v[u >> 2];
    return (u & 3) == 0 ? w.x : ((u & 3) == 1 ? w.y : ((u & 3) == 2 ? w.z : w.w));
  };
  float e[8];
  uint32_t nh[4], nl[4];
  auto kernel_values = [&](int u, int rb, const f4v (&dd)[2]) {
#pragma unroll
    for (int v = 2 * u; v < 2 * u + 2; ++v) {
      if constexpr (GRAM) e[v] = __builtin_amdgcn_exp2f(dd[v >> 2][v & 3]);
      else
        e[v] = __builtin_amdgcn_exp2f(-pair_exponent<KERNEL>(rx[rb] - comp(px, v), ry[rb] - comp(py, v), rz[rb] - comp(pz, v)));
    }
  };
  auto hi_part = [&](int u, int rb) {
    uint32_t w = pack_h2(e[2 * u] * Sg[rb], e[2 * u + 1] * Sg[rb]);
    asm("" : "+v"(w));
    nh[u] = w;
  };
  auto lo_part = [&](int u, int rb) {
    const h2v p = __builtin_bit_cast(h2v, nh[u]);
    float l0 = __builtin_fmaf(e[2 * u], Sg[rb], -(float)p[0]), l1 = __builtin_fmaf(e[2 * u + 1], Sg[rb], -(float)p[1]);
    asm("" : "+v"(l0), "+v"(l1));   // (v_fma_mix_f32 and one packed conversion: 6 cycles less than two v_fma_mix{lo,hi}_f16)
    nl[u] = pack_h2(l0, l1);
  };
  // the vector work of a step in 12 pieces, in an order that leaves each exp time to finish
  auto atom = [&](int i, int rb, const f4v (&dd)[2]) {
    constexpr int kind[12] = {0, 0, 1, 0, 2, 1, 0, 2, 1, 2, 1, 2};
    constexpr int idx[12] = {0, 1, 0, 2, 0, 1, 3, 1, 2, 2, 3, 3};
    if (kind[i] == 0) kernel_values(idx[i], rb, dd);
    else if (kind[i] == 1) hi_part(idx[i], rb);
    else lo_part(idx[i], rb);
  };
  h8v yh[NT], yl[NT];
  auto load_yh = [&](int slot, int ks) {
#pragma unroll
    for (int t = 0; t < NT; ++t) yh[t] = __builtin_bit_cast(h8v, s_y[slot][(ks * NT + t) * 64 + lane]);
  };
  auto load_yl = [&](int slot, int ks) {
#pragma unroll
    for (int t = 0; t < NT; ++t) yl[t] = __builtin_bit_cast(h8v, s_y[slot][E + (ks * NT + t) * 64 + lane]);
  };
  h8v gh, gl;
  auto take = [&]() {
    gh = __builtin_bit_cast(h8v, make_uint4(nh[0], nh[1], nh[2], nh[3]));
    gl = __builtin_bit_cast(h8v, make_uint4(nl[0], nl[1], nl[2], nl[3]));
  };

#pragma unroll
  for (int v = 0; v < kXRing; ++v) {
    fetch(v < kYRing ? v : kYRing - 1, v, v < kYRing ? v : kYRing - 1, v);
    stash(v);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  load_x(0, 0);
  load_yl(0, 0);
  load_yh(0, 0);
  if constexpr (GRAM) gram(0);
  {
    const f4v dd[2] = {d[0], d[1]};
#pragma unroll
    for (int i = 0; i < 12; ++i) atom(i, 0, dd);
  }
  take();
  if constexpr (GRAM) {
    gram(1);
    if (RB == 2) load_x(0, 1);
  }
  // scale of vector 16 t + lane % 16 of the group whose last tile is in `slot`
  auto scale_up = [&](int slot, int t) {
    const int vec = 16 * t + (lane & 15), ct = vec & 31;
    if constexpr (GRAM) {
      const uint4* x = &s_x[slot][((vec >> 5) * 2 + ((ct >> 2) & 1)) * 64 + 4 * (ct >> 3) + (ct & 3)];
      return (int)(float)reinterpret_cast<const _Float16*>(x)[7];
    } else {
      return (int)reinterpret_cast<const float*>(&s_x[slot][0])[3 * kCT + vec];
    }
  };

  int yc = 0, xc = 0;   // LDS slots of the tile in work
  int par = 0;          // parity of its group
  for (int64_t ti = 0; ti < ntile; ++ti) {
    int up[NT];
    const bool last = ((T0 + ti + 1) & (GT - 1)) == 0 || ti + 1 == ntile;   // of its group
    const int yn = yc + 1 < kYRing ? yc + 1 : 0, xn = (xc + 1) & (kXRing - 1);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int ks = s / RB, rb = s % RB;
      if (s == S - 1) {
#pragma unroll
        for (int t = 0; t < NT; ++t) up[t] = scale_up(xc, t);
        // All reads of this tile from LDS are done.  Wait for the next tile's
        // Y and the next but one's operands (their loads were issued two
        // barriers ago), then refill this tile's place.
        stash((xc + 3) & (kXRing - 1));
        if (last) {   // from here on the vector work is the next group's
          row_scales(par ^ 1);
        }
        __builtin_amdgcn_s_waitcnt(kLoads | (7 << 4));   // vmcnt(kLoads), lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (ti + 1 < ntile) fetch(ti + 3, ti + 4, yc, xc);
      }
      if (s == 0 && last) load_box((T0 + ti + 1) / GT);
      // step s: its MFMAs, the vector work of step s + 1 (exponents in d) and the exponents of step s + 2
      const f4v dd[2] = {d[0], d[1]};
      if constexpr (GRAM) {
        gram((s + 2) % RB);
        if ((s + 3) % RB == 0) load_x(s + 3 >= S ? xn : xc, ((s + 3) % S) / RB);
      } else {
        if ((s + 1) % RB == 0) load_x(s + 1 >= S ? xn : xc, ((s + 1) % S) / RB);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 3 * NT; ++i) {
        const int t = i % NT, part = i / NT;
        // hi lo and lo hi in sums of their own: 2^11 smaller, their roundings do not count
        f4v& dst = part == 1 ? acc[rb][t] : accx[rb][t];
        dst = __builtin_amdgcn_mfma_f32_16x16x32_f16(part == 2 ? gl : gh, part == 0 ? yl[t] : yh[t], dst, 0, 0, 0);
        constexpr int per = 12 / (3 * NT);
#pragma unroll
        for (int v = 0; v < per; ++v) atom(i * per + v, (s + 1) % RB, dd);
        if (rb == RB - 1 && i == NT - 1) load_yl(ks + 1 < KS ? yc : yn, (ks + 1) % KS);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (rb == RB - 1) load_yh(ks + 1 < KS ? yc : yn, (ks + 1) % KS);
      take();
    }
    if (last) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const float4 inv4 = *reinterpret_cast<const float4*>(&s_inv[par][wave * 16 * RB + 16 * rb + 4 * q]);
        const float inv[4] = {inv4.x, inv4.y, inv4.z, inv4.w};
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const double f = __builtin_ldexp(1.0, -up[t]);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            tot[rb][t][r] = __builtin_fma((double)((acc[rb][t][r] + accx[rb][t][r]) * inv[r]), f, tot[rb][t][r]);
          acc[rb][t] = zero4;
          accx[rb][t] = zero4;
        }
      }
      par ^= 1;
    }
    yc = yn;
    xc = xn;
  }
  __builtin_amdgcn_s_waitcnt(kVm0);   // no load to LDS outlives the tile loop

  // Groups with a value that is not finite in Y or in the points: their
  // operands are zero above, and they are added here as they stand, one pair
  // at a time, so that infinities and NaN come out as from FP32 products.
  if (flags & kBadValue) {
    for (int64_t g = c_begin / G; g * G < c_end; ++g) {
      if (((int)a.gbox[8 * g + 3] & kBadValue) == 0) continue;
      for (int64_t c = g * G > c_begin ? g * G : c_begin; c < (g + 1) * G && c < c_end; ++c) {
        const float* y = a.xc + c * a.xc_stride;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int64_t row = row0 + 16 * rb + 4 * q + r;
            const float* x = a.xr + (row < a.nr ? row : a.nr - 1) * a.xr_stride;
            const float k = __builtin_amdgcn_exp2f(-pair_exponent<KERNEL>(
                x[0] * a.coord_scale - y[0] * a.coord_scale, x[1] * a.coord_scale - y[1] * a.coord_scale,
                x[2] * a.coord_scale - y[2] * a.coord_scale));
#pragma unroll
            for (int t = 0; t < NT; ++t) tot[rb][t][r] += (double)(k * a.Y[c * B + 16 * t + (lane & 15)]);
          }
      }
    }
  }

  float* out = a.nsplit > 1 ? a.partial + (size_t)split * a.nr * B : a.Z;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = row0 + 16 * rb + 4 * q + r;
      if (row < a.nr) {
        const double f = (double)(a.out_scale * (a.rs ? a.rs[row] : 1.0f));
#pragma unroll
        for (int t = 0; t < NT; ++t) out[row * B + 16 * t + (lane & 15)] = (float)(f * tot[rb][t][r]);
      }
    }
  }
}

// Waves per SIMD: as many as the registers allow (b = 16: 165; b = 32 and 64:
// up to 250, most of them sums).
template <int B>
constexpr int h16_waves() { return B == 16 ? 3 : 2; }

template <int KERNEL, int B, int RB>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(h16_waves<B>(), h16_waves<B>())))
void gamma_f16x3_kernel(GammaLaunch a) {
  __shared__ uint4 s_x[kXRing][kXEntries];
  __shared__ uint4 s_y[kYRing][2 * h16_entries<B>()];
  constexpr int ROWS = 64 * RB;
  __shared__ float s_box[4][8];
  __shared__ float s_row[3][ROWS];
  __shared__ float s_inv[2][ROWS];
  __shared__ int s_flags;
  int64_t rblk;
  int split;
  if (!gamma_item(a, rblk, split)) return;
  double cl[3];
  launch_centre(a, cl);
  float c0, c1, c2;
  (void)gram_rows<RB>(a, rblk, s_box, c0, c1, c2);
  c0 = uniform(row_centre<KERNEL>(s_box, 0, c0));
  c1 = uniform(row_centre<KERNEL>(s_box, 1, c1));
  c2 = uniform(row_centre<KERNEL>(s_box, 2, c2));
  // the rows' points relative to the launch's centre, whether they are on the
  // lattice, and the flags of the columns' groups
  int flags = 0;
  for (int r = threadIdx.x; r < ROWS; r += kThreads) {
    const int64_t row = rblk * ROWS + r;
    const float* x = a.xr + (row < a.nr ? row : a.nr - 1) * a.xr_stride;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float t = (float)lattice_coord(a, x[k], cl[k]);
      s_row[k][r] = t;
    }
    if (KERNEL == KA_GAUSSIAN && !lattice_point(a, x, cl).ok) flags |= kOffLattice;
  }
  const int64_t c0s = (int64_t)split * a.cols_per_split;
  const int64_t g0 = c0s / kGroup, g1 = (c0s + a.cols_per_split + kGroup - 1) / kGroup;
  for (int64_t g = g0 + threadIdx.x; g < g1 && g < a.ngroups; g += kThreads) flags |= (int)a.gbox[8 * g + 3];
  if (threadIdx.x == 0) s_flags = 0;
  __syncthreads();
  if (flags) atomicOr(&s_flags, flags);
  __syncthreads();
  flags = __builtin_amdgcn_readfirstlane(s_flags);
  if constexpr (KERNEL == KA_GAUSSIAN) {
    if (!(flags & kOffLattice)) {
      gamma_h16_tile<KERNEL, B, RB, true>(a, rblk, split, s_x, s_y, c0, c1, c2, cl, flags, s_row, s_inv);
      return;
    }
  }
  gamma_h16_tile<KERNEL, B, RB, false>(a, rblk, split, s_x, s_y, c0, c1, c2, cl, flags, s_row, s_inv);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <int B, int RB>
static hipError_t launch_b(const GammaLaunch& a, int kernel, dim3 grid, hipStream_t s) {
  hipLaunchKernelGGL(gamma_split16_kernel<B>, dim3((unsigned)a.ngroups), dim3(kPreThreads), 0, s, a, kernel);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (kernel == KA_GAUSSIAN)
    hipLaunchKernelGGL((gamma_f16x3_kernel<KA_GAUSSIAN, B, RB>), grid, dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((gamma_f16x3_kernel<KA_EXP_L1, B, RB>), grid, dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_gamma_f16x3(const GammaLaunch& a, int kernel, int b, dim3 grid, hipStream_t s) {
  switch (b) {
    case 16: return launch_b<16, 4>(a, kernel, grid, s);
    case 32: return launch_b<32, 4>(a, kernel, grid, s);
    case 64: return launch_b<64, 2>(a, kernel, grid, s);
    default: return hipErrorInvalidValue;
  }
}

// scratch: Y's fragments, the points' operands, the scales, the boxes
size_t gamma_f16x3_bytes(int64_t nc, int b) {
  const size_t ng = ((size_t)nc + kGroup - 1) / kGroup;
  return ng * (kGroup * (b * 4 + 64) + b * sizeof(float) + 8 * sizeof(float));
}

void gamma_f16x3_place(GammaLaunch& a, int b, void* work) {
  const size_t ng = ((size_t)a.nc + kGroup - 1) / kGroup;
  char* p = (char*)work;
  a.ys = (uint4*)p;
  p += ng * kGroup * b * 4;
  a.xs = (uint4*)p;
  p += ng * kGroup * 64;
  a.yup = (float*)p;
  p += ng * b * sizeof(float);
  a.gbox = (float*)p;
  a.ngroups = (int64_t)ng;
}

}  // namespace ka
