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
// totals undo them).  Below 2^-16 of its largest a value loses bits, below 2^-40
// all of them.  What would show that in a result is formed in FP32:
// - columns with an entry that is not finite or below 2^-22 of its vector's
//   largest in the group (2^-18 off in FP16 parts), and all columns of a group
//   with no more than 64 that are not zero, are marked by the pre-pass, left out
//   of the FP16 operands and added as they stand; where half of an item's
//   columns are marked, all of it is formed so;
// - rows (in vectors with zeros or very small entries, single entries) whose
//   results are below 2^-19 of what the groups' boxes promise, which may be what
//   was lost (lossy_results), are done again; where that is a quarter of an item's
//   rows, all of it.
// So what is lost is below 2^-19 of a result, or below 2^-126 |Y| (groups at
// exponents past 86, where the loss is below FP32's least value).  Not seen: a low
// result in a vector without very small entries, in a row whose other results are
// not low (a row without near columns, and at the nearest of them a small entry).
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
// What bounds it (287,496^2, b = 64, Gaussian, 32.2 to 33.4 ms on several cards =
// 2.5e12 pairs/s, against 91 ms on the FP32 matrix cores): matrix cores 53% and
// VALU 61% of the cycles, 22% of them together, so that either is busy 91% of the
// time, at 2.0 GHz (the power limit; 2.4 GHz nominal).  The same instructions without any memory
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

constexpr int kFewColumns = 64;             // a group with no more columns that are not zero (half of it at most) has them added in FP32
constexpr int kNoScale = 200;               // "scale" of a vector that is zero in a group

enum { kOffLattice = 1, kGaps = 2, kMarks = 4 };   // flags of a column group, and kMarks times its columns in FP32

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
struct SplitShared {
  float b[kPreThreads / 64][8];           // boxes of the waves' columns
  uint32_t bad[kGroup / 32], nz[kGroup / 32], point[kGroup / 32];   // a bit per column
  uint32_t gap[2];                        // a bit per vector
  int flag;
};

template <int B>
__device__ __forceinline__ void split16_group(const GammaLaunch& a, int kernel, int64_t g, float (*s_m)[B], float* s_up,
                                              SplitShared& sh) {
  constexpr int NT = B / 16;
  constexpr int G = kGroup, GT = kGroupTiles;
  constexpr int PARTS = kPreThreads / B;
  constexpr int CPT = G / PARTS;        // columns per thread: 8, 16 or 32; a wave has 32
  constexpr int E = h16_entries<B>();
  const int j = threadIdx.x % B, part = threadIdx.x / B;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int bit0 = part * CPT % 32;     // this thread's first column in its wave's word
  const int64_t c0 = g * G + part * CPT;
  float y[CPT];
#pragma unroll
  for (int u = 0; u < CPT; ++u) y[u] = c0 + u < a.nc && j < a.nv ? a.Y[(c0 + u) * B + j] : 0.f;
  uint32_t most = 0, least = ~0u;   // of the entries' magnitudes, as bits
#pragma unroll
  for (int u = 0; u < CPT; ++u) {
    const uint32_t v = __builtin_bit_cast(uint32_t, y[u]) & 0x7fffffffu;
    most = most > v ? most : v;
    least = least < v ? least : v;
  }
  float m = __builtin_bit_cast(float, most);   // largest finite entry
  if (!finite_bits(m)) {
    m = 0.f;
#pragma unroll
    for (int u = 0; u < CPT; ++u) m = fmaxf(m, finite_bits(y[u]) ? __builtin_fabsf(y[u]) : 0.f);
  }
  if (threadIdx.x == 0) sh.flag = 0;
  if (threadIdx.x < 2) sh.gap[threadIdx.x] = 0;
  s_m[part][j] = m;
  // the column points: their places on the lattice, and the group's box
  double c[3];
  launch_centre(a, c);
  LatticePoint p;
  const int64_t col = g * G + threadIdx.x;
  bool in = threadIdx.x < G && col < a.nc;
  float x[3] = {0.f, 0.f, 0.f}, lo[3], hi[3];
  bool far = false;   // at infinity, or there once scaled
  if (in)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      x[k] = a.xc[col * a.xc_stride + k];
      far = far || !finite_bits(x[k] * a.coord_scale);
    }
  const uint64_t far_cols = __ballot(far);
  if (lane < 2 && threadIdx.x < G) sh.point[2 * wave + lane] = (uint32_t)(far_cols >> (32 * lane));
  in = in && !far;
  p = lattice_point(a, x, c);
  const bool off = in && !p.ok;
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
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      sh.b[wave][k] = lo[k];
      sh.b[wave][4 + k] = hi[k];
    }
  __syncthreads();
  if (off) atomicOr(&sh.flag, (int)kOffLattice);
#pragma unroll
  for (int q = 0; q < PARTS; ++q) m = fmaxf(m, s_m[q][j]);
  int ex = 0;
  if (m > 0.f) (void)__builtin_frexpf(m, &ex);   // m in [2^(ex-1), 2^ex)
  const int up = m > 0.f ? 15 - ex : kNoScale;                        // |y| 2^up < 2^15
  if (part == 0) {
    s_up[j] = (float)up;
    a.yup[g * B + j] = (float)up;
  }
  // columns with a value that the parts do not hold: not finite, or below 2^-22
  // of the largest (2^-7 where FP16's last place is 2^-24: 2^-18 off); vectors
  // with such values, or zeros; columns that are not zero.  Most waves have none
  // of the odd ones.
  const float low = m > 0.f ? __builtin_ldexpf(1.f, ex - 22) : 0.f;
  uint32_t bad = 0, nz = ~0u;
  if (__any(j < a.nv && (least < __builtin_bit_cast(uint32_t, low) || least == 0 || most >= 0x7f800000u))) {
    nz = 0;
    bool gap = m == 0.f;
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const bool some = y[u] != 0.f, small = __builtin_fabsf(y[u]) < low;
      if (some) nz |= 1u << u;
      if (some && (small || !finite_bits(y[u]))) bad |= 1u << u;
      gap = gap || (small && c0 + u < a.nc);
    }
    if (gap && j < a.nv) atomicOr(&sh.gap[j / 32], 1u << (j % 32));
    bad <<= bit0;
    nz <<= bit0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      bad |= __shfl_xor(bad, o);
      nz |= __shfl_xor(nz, o);
    }
  }
  if (lane == 0) {
    sh.bad[wave] = bad;
    sh.nz[wave] = nz;
  }
  __syncthreads();
  int count = 0;
#pragma unroll
  for (int w = 0; w < G / 32; ++w) count += __builtin_popcount(sh.nz[w]);
  // (not a short last group: its box is that of its few columns.  b = 64, 100,000 x
  // 568 takes 58 us so, and 89 with the last 56 columns in FP32)
  const int cols = (int)(a.nc - g * G < G ? a.nc - g * G : G);
  const bool few = count <= kFewColumns && 2 * count <= cols;
  auto exact_word = [&](int w) { return sh.bad[w] | sh.point[w] | (few ? sh.nz[w] : 0u); };
  if (threadIdx.x < G / 32) a.gmask[g * (G / 32) + threadIdx.x] = exact_word(threadIdx.x);
  if (threadIdx.x < 2) a.ggap[2 * g + threadIdx.x] = sh.gap[threadIdx.x];
  if (wave == kPreThreads / 64 - 1) {   // box, flags and largest entry (rounded down to a power of two); a wave without points
    int marks = lane < G / 32 ? __builtin_popcount(exact_word(lane & (G / 32 - 1))) : 0;
#pragma unroll
    for (int o = 1; o < G / 32; o <<= 1) marks += __shfl_xor(marks, o);   // (lane 3 has them)
    float size = few || up == kNoScale ? 0.f : __builtin_ldexpf(1.f, 14 - up);   // (lane: vector lane % B)
#pragma unroll
    for (int o = 1; o < B; o <<= 1) size = fmaxf(size, __shfl_xor(size, o));
    const int flags = sh.flag | ((sh.gap[0] | sh.gap[1]) != 0 ? (int)kGaps : 0) | marks * kMarks;
    float* b = a.gbox + 8 * g;
    if (lane < 3) {
      float l = sh.b[0][lane], h = sh.b[0][4 + lane];
#pragma unroll
      for (int w = 1; w < G / 64; ++w) {
        l = fminf(l, sh.b[w][lane]);
        h = fmaxf(h, sh.b[w][4 + lane]);
      }
      // A row's distance from the box has to be a lower bound of its distances
      // from the columns as the product forms them.  Box and row are rounded at
      // their size relative to the launch's centre (once each), the two
      // coordinates of a difference relative to the row block's (twice each),
      // which is no further from a row than zero or 32 units (row_centre).  With
      // a row as far off as the box that is 6 of 2^-24, taken as 8; what a row
      // further off adds is 2^-21 of the distance, inside the product's 0.999.
      const float ck = (float)(lane == 0 ? c[0] : (lane == 1 ? c[1] : c[2]));
      const float wide = 0x1p-21f * (fmaxf(__builtin_fabsf(l), __builtin_fabsf(h)) + __builtin_fabsf(ck) + 32.f);
      b[lane] = l <= h ? l - wide : l;
      b[4 + lane] = l <= h ? h + wide : h;
    } else if (lane == 3) {
      b[3] = (float)flags;
      b[7] = size;
    }
  }
  if (kernel == KA_GAUSSIAN && threadIdx.x < G) {
    // fragment (ks, half), lane 16 q + m of the column's tile
    const int cg = threadIdx.x, ct = cg & 31, vec = cg & 63;
    uint4* dst = a.xs + (g * GT + cg / kCT) * kXEntries + (((cg & 63) >> 5) * 2 + ((ct >> 2) & 1)) * 64 +
                 4 * (ct >> 3) + (ct & 3);
    // (a column that is none, or is at infinity, is put so far off that Gamma is
    // zero whatever the row's scale)
    const float n = !in ? -30000.f : -(p.h[0] * p.h[0] + p.h[1] * p.h[1] + p.h[2] * p.h[2]);
    // the last slot meets a zero of the rows' operand: it carries the scale of vector `vec`
    dst[0] = make_uint4(pack_h2(p.h[0], p.h[1]), pack_h2(p.h[2], n), pack_h2(n - half_of(n), 1.f),
                        pack_h2(1.f, vec < B ? s_up[vec] : 0.f));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float l = p.l[k] * kLat;
      float b = -l * (2.f * p.h[k] + p.l[k]);
      // (one value for its part and for what that leaves: a product rounded straight
      // to FP16 in the one and by way of FP32 in the other is a last place off, 2^-13
      // in the exponent, for one column in some thousands)
      asm("" : "+v"(b));
      const float b1 = b - half_of(b);
      dst[16 * (k + 1)] = make_uint4(pack_h2(l, l - half_of(l)), pack_h2(p.h[k] / kLat, p.h[k] / kLat), pack_h2(l, b),
                                     pack_h2(b1, b1 - half_of(b1)));
    }
  }
  if (const uint32_t exact = exact_word(wave) >> bit0)
#pragma unroll
    for (int u = 0; u < CPT; ++u) y[u] = exact >> u & 1 ? 0.f : y[u];
#pragma unroll
  for (int v = 0; v < CPT / 8; ++v) {
    const int cg = part * CPT + 8 * v;        // in the group
    uint32_t h[4], l[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = 8 * v + 2 * u;
      const float y0 = __builtin_ldexpf(y[e], up), y1 = __builtin_ldexpf(y[e + 1], up);
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
  __shared__ SplitShared sh;
  split16_group<B>(a, kernel, blockIdx.x, s_m, s_up, sh);
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

// ---------------------------------------------------------------------------
// columns and rows in FP32
//
// What FP16 parts do not hold is formed as FP32 values, contracted by FP32 MFMAs
// and added to FP64 totals every 128 columns.  Exponents come from differences
// of FP64 coordinates, rounded once: no centre has to be chosen, and a pair costs
// six FP64 operations and a conversion where FP32 with as much accuracy would
// take twice as many.  All of 85,184^2 at b = 64 takes 11.7 ms so (11.4
// exponential), 8.0 in the FP32 tiles of gamma.hip with their rounding of
// coordinates, and 2.8 in FP16 parts; b = 16 5.2, 2.9 and 1.5 ms.  Blocks without
// such values pay for the look-out: 12,167^2 at b = 16 62.8 -> 66.2 us, 6,500^2 at
// b = 64 53.5 -> 57.9, 70,000^2 at b = 32 exponential 1.77 -> 1.80 ms, 287,496^2 at
// b = 64 32.0 -> 32.1 ms.
// ---------------------------------------------------------------------------
template <int KERNEL>
__device__ __forceinline__ float exact_value(const double (&x)[3], const double (&y)[3]) {
  const double dx = x[0] - y[0], dy = x[1] - y[1], dz = x[2] - y[2];
  const double e = KERNEL == KA_GAUSSIAN ? __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx)) : (fabs(dx) + fabs(dy)) + fabs(dz);
  return __builtin_amdgcn_exp2f((float)-e);
}

__device__ __forceinline__ void exact_point(const GammaLaunch& a, const float* p, double (&x)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) x[k] = lattice_coord(a, p[k], 0.0);
}

// The n columns column(0), column(1), ... against RB groups of 16 rows, added to
// `tot`; sixteen at a time, the operands of the next sixteen or 32 on their way.
template <int KERNEL, int B, int RB, class Column>
__device__ __forceinline__ void exact_columns(const GammaLaunch& a, const double (&x)[RB][3], int columns,
                                              Column column, d4v (&tot)[RB][B / 16]) {
  constexpr int NT = B / 16;
  const int n = __builtin_amdgcn_readfirstlane(columns);
  const int q = (threadIdx.x & 63) >> 4, l16 = threadIdx.x & 15;
  float p[2][4][3], y[2][4][NT];
  auto load = [&](int i0, float (&lp)[4][3], float (&ly)[4][NT]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int i = i0 + 4 * s + q;
      const int64_t c = column(i < n ? i : n - 1);
#pragma unroll
      for (int k = 0; k < 3; ++k) lp[s][k] = a.xc[c * a.xc_stride + k];
#pragma unroll
      for (int t = 0; t < NT; ++t) ly[s][t] = a.Y[c * B + 16 * t + l16];
    }
  };
  f4v acc[RB][NT];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[rb][t] = (f4v){0.f, 0.f, 0.f, 0.f};
  auto work = [&](int i0, const float (&wp)[4][3], const float (&wy)[4][NT]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (i0 + 4 * s >= n) break;   // (a mark or two as a rule)
      const bool on = i0 + 4 * s + q < n;
      double z[3];
      exact_point(a, wp[s], z);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        float e = exact_value<KERNEL>(x[rb], z);
        asm("" : "+v"(e));   // (or each value gets a branch of its own)
        e = on ? e : 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[rb][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(e, on ? wy[s][t] : 0.f, acc[rb][t], 0, 0, 0);
      }
    }
  };
  if (n <= 0) return;
  load(0, p[0], y[0]);
  if (n > 16) load(16, p[1], y[1]);
  for (int i0 = 0; i0 < n; i0 += 32) {
    work(i0, p[0], y[0]);
    if (i0 + 32 < n) load(i0 + 32, p[0], y[0]);
    __builtin_amdgcn_sched_barrier(0);
    work(i0 + 16, p[1], y[1]);
    if (i0 + 48 < n) load(i0 + 48, p[1], y[1]);
    __builtin_amdgcn_sched_barrier(0);
    if ((i0 & 127) == 96 || i0 + 32 >= n)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          tot[rb][t] += __builtin_convertvector(acc[rb][t], d4v);
          acc[rb][t] = (f4v){0.f, 0.f, 0.f, 0.f};
        }
  }
}

__device__ __forceinline__ double row_factor(const GammaLaunch& a, int64_t row) {
  return (double)(a.out_scale * (a.rs ? a.rs[row] : 1.0f));
}

// Adds the columns of [c_begin, c_end) that are marked in a.gmask to `tot`: as a
// rule a few (of N(0, 1) blocks one in 80,000 at b = 16), listed in s_few in any
// order; else they are gathered in their order from up to 8192 columns at a time.
constexpr int kFewMarks = 64;
constexpr int kListColumns = 32 * kThreads;
static_assert(sizeof(uint16_t) * kListColumns <= sizeof(uint4) * kXRing * kXEntries, "the list takes the operands' place in LDS");

template <int KERNEL, int B, int RB>
__device__ __forceinline__ void add_marked_columns(const GammaLaunch& a, int64_t row0, int64_t c_begin, int64_t c_end,
                                                   const int* s_few, int n_few, void* s_list, int* s_cnt,
                                                   d4v (&tot)[RB][B / 16]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double x[RB][3];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int64_t r = row0 + 16 * rb + (lane & 15);
    exact_point(a, a.xr + (r < a.nr ? r : a.nr - 1) * a.xr_stride, x[rb]);
  }
  if (n_few <= kFewMarks) {
    int* list = reinterpret_cast<int*>(s_list);
    if ((int)threadIdx.x < n_few) {   // sorted, so that sums don't depend on the order of arrival
      const int v = s_few[threadIdx.x];
      int at = 0;
      for (int k = 0; k < n_few; ++k) at += s_few[k] < v;
      list[at] = v;
    }
    __syncthreads();
    exact_columns<KERNEL, B, RB>(a, x, n_few, [&](int i) { return c_begin + list[i]; }, tot);
    return;
  }
  uint16_t* list = reinterpret_cast<uint16_t*>(s_list);
  for (int64_t cb = c_begin; cb < c_end; cb += kListColumns) {
    // a word of 32 columns per thread (splits start at whole words, and no
    // column past the last is marked)
    uint32_t w = cb + 32 * (int)threadIdx.x < c_end ? a.gmask[cb / 32 + threadIdx.x] : 0u;
    const int own = __builtin_popcount(w);
    int k = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(k, o);
      if (lane >= o) k += v;
    }
    __syncthreads();   // the list and counts of the columns before have been read
    if (lane == 63) s_cnt[wave] = k;
    __syncthreads();
    int at = k - own, n = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (v < wave) at += s_cnt[v];
      n += s_cnt[v];
    }
    for (; w; w &= w - 1) list[at++] = (uint16_t)(32 * threadIdx.x + __builtin_ctz(w));
    __syncthreads();
    exact_columns<KERNEL, B, RB>(a, x, n, [&](int i) { return cb + list[i]; }, tot);
  }
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
                                               float c0, float c1, float c2, const double (&cl)[3],
                                               const float (*s_row)[64 * RB], float (*s_inv)[64 * RB],
                                               const int* s_few, int marks, int* s_cnt, d4v (&tot)[RB][B / 16]) {
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

#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int t = 0; t < NT; ++t) tot[rb][t] = (d4v){0.0, 0.0, 0.0, 0.0};
  if (marks > 0) {
    add_marked_columns<KERNEL, B, RB>(a, row0, c_begin, c_end, s_few, marks, &s_x[0][0], s_cnt, tot);
    __syncthreads();   // the list has been read
  }

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
  // or Gamma passes 2^16: the pre-pass widens the boxes by what roundings can do.
  float Sg[RB];
  float gb[6];   // box of the next group
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
        const float x = s_row[k][r], gap = fmaxf(fmaxf(gb[k] - x, x - gb[3 + k]), 0.f);
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
  f4v acc[RB][NT], accx[RB][NT];   // (tot comes with the columns that are added in FP32)
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      acc[rb][t] = zero4;
      accx[rb][t] = zero4;
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
        if (!finite_bits(t)) t = 1e18f;        // Gamma = 0 here: the column is added in FP32
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
}

// the sum of s over the workgroup, in every thread
__device__ __forceinline__ double block_sum(double s, double* s_sum) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  __syncthreads();   // the sums before have been read
  if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = s;
  __syncthreads();
  return (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
}

// Which stored results may have lost what matters: entries (i B + vector, i the
// row's place) into s_entry, whole rows into s_list.  A low result is not
// cancellation if no vector of the row comes out larger for its size (a hole
// between scattered columns; results that are not finite don't count): the row.  In a vector with zeros or very small
// entries the near columns may be among these: the entry, unless the group that
// could give most holds enough of |Gamma| |Y|; the rows, if the entries are many.
// (N(0, 1) blocks of 287,496 x 64: a dozen entries in 50 row blocks get as far
// as the check of the group, none further.)
//
// Where the columns are split, those of this item may all be far from a row and
// their sum low for the boxes, but nothing beside that of another split.  So a
// single column anywhere whose part of |Gamma| |Y| outweighs what this item and as
// many others could lose is enough to leave a result as it is (`weighs`): the
// column in the row's place (the row itself where rows and columns are the same
// points), then the nearest of 16 in the group whose box is nearest.  Without this,
// rows are done again in the items next to their own when correlation lengths are
// short (us, without / with): b = 16, 5,280 points of a half cylinder, ell a 15th of
// its height, 57 / 36; b = 32, 4,312 points of a quarter annulus, ell = 0.12, 96 /
// 43; 11,968 points of it 111 / 95; b = 64, 85,184 points of the cube, ell = 0.1,
// sines over the cube 12.4 / 3.1 ms.
constexpr float kLostCut = 0x1p-19f;
constexpr float kFarExponent = 86.f;   // from here on 2^-40 of a kernel value is below FP32's least, 2^-126
constexpr int kEntries = 64;
constexpr uint16_t kNoEntry = 0xffff;   // (an entry is below 256 rows times 64 vectors)

struct Lossy {
  int rows, entries;
};

template <int B>
struct LossyShared {
  float size[kThreads];       // largest entry of vector t % B, over part of the groups, then [0 .. B) over all
  uint32_t gap[kThreads];     // whether it has zeros or very small entries
  uint32_t rows[8], some[8];  // a bit per row; of rows with entries
  double sum[4];
  int n;
};

template <int KERNEL, int B, int RB>
__device__ __forceinline__ Lossy lossy_results(const GammaLaunch& a, int64_t row0, int64_t c_begin, int64_t c_end,
                                               int64_t g0, int64_t g1, const float* out,
                                               const float (*s_row)[64 * RB], float* s_lost, const int* s_best,
                                               LossyShared<B>& sh, uint16_t* s_list, uint16_t* s_entry, bool rows) {
  constexpr int NT = B / 16, ROWS = 64 * RB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = lane >> 4, l16 = lane & 15;
  float v_size = 0.f;
  uint32_t v_gap = 0;
  for (int64_t g = g0 + threadIdx.x / B; g < g1 && g < a.ngroups; g += kThreads / B) {
    const int vec = threadIdx.x % B, up = (int)a.yup[g * B + vec];
    if (up != kNoScale) v_size = fmaxf(v_size, __builtin_ldexpf(1.f, 14 - up));
    v_gap |= a.ggap[2 * g + vec / 32] >> (vec % 32) & 1;
  }
  sh.size[threadIdx.x] = v_size;
  sh.gap[threadIdx.x] = v_gap;
  if (threadIdx.x < 8) sh.rows[threadIdx.x] = sh.some[threadIdx.x] = 0;
  if (threadIdx.x == 0) sh.n = 0;
  __syncthreads();
  if (threadIdx.x < B)
    for (int v = threadIdx.x + B; v < kThreads; v += B) {
      v_size = fmaxf(v_size, sh.size[v]);
      v_gap |= sh.gap[v];
    }
  __syncthreads();
  if (threadIdx.x < B) {
    sh.size[threadIdx.x] = v_size;
    sh.gap[threadIdx.x] = v_gap;
  }
  __syncthreads();
  float largest = 0.f;
  for (int v = 0; v < B; ++v) largest = fmaxf(largest, sh.size[v]);
  auto value = [&](const float* x, int64_t c) {
    float d = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float t = __builtin_fabsf(x[k] - a.xc[c * a.xc_stride + k]) * a.coord_scale;
      d += KERNEL == KA_GAUSSIAN ? t * t : t;
    }
    return __builtin_amdgcn_exp2f(-d);
  };
  // the column in a row's place, and the least that a column has to add to a row's
  // |Gamma| |Y| in a vector of size 1
  auto in_place = [&](int i) { return (int64_t)((double)(row0 + i) * (double)a.nc / (double)a.nr); };
  auto cut = [&](int i) { return (float)a.nsplit * kLostCut * s_lost[i] / largest; };
  // leaves rows as they are that a column outweighs (s_lost 0); true if others are left
  auto leave_rows = [&](bool left) {
    const float* xr = a.xr + (left ? row0 + threadIdx.x : row0) * a.xr_stride;
    const float x[3] = {xr[0], xr[1], xr[2]};
    auto weighs = [&](int64_t c) {
      const float e = value(x, c), least = cut(threadIdx.x);
      int all = 1;
      for (int v = 0; v < B; v += 16) {
        float4 y[4];   // (all at once: one by one they are four waits)
#pragma unroll
        for (int u = 0; u < 4; ++u) y[u] = reinterpret_cast<const float4*>(a.Y + c * B + v)[u];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float* size = &sh.size[v + 4 * u];   // (zero for vectors that do not count)
          all &= (int)(e * __builtin_fabsf(y[u].x) >= least * size[0]) | (int)(size[0] == 0.f);
          all &= (int)(e * __builtin_fabsf(y[u].y) >= least * size[1]) | (int)(size[1] == 0.f);
          all &= (int)(e * __builtin_fabsf(y[u].z) >= least * size[2]) | (int)(size[2] == 0.f);
          all &= (int)(e * __builtin_fabsf(y[u].w) >= least * size[3]) | (int)(size[3] == 0.f);
        }
      }
      return all != 0;
    };
    const bool had = left;
    if (left) left = !weighs(in_place(threadIdx.x));
    if (a.nsplit > 1 && __syncthreads_or(left)) {
      if (left) {
        int64_t near = 0, at = 0;
        float most = -1.f;
        const int64_t step = (a.ngroups + 127) / 128;
        for (int64_t g = 0; g < a.ngroups; g += step) {
          const uniform_float* b = (const uniform_float*)(uintptr_t)(a.gbox + 8 * g);
          float d = 0.f;
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const float t = s_row[k][threadIdx.x], gap = fmaxf(fmaxf(b[k] - t, t - b[4 + k]), 0.f);
            d += KERNEL == KA_GAUSSIAN ? gap * gap : gap;
          }
          const float v = __builtin_amdgcn_exp2f(-d) * b[7];
          if (v > most) {
            most = v;
            near = g;
          }
        }
        most = -1.f;
#pragma unroll 4
        for (int k = 0; k < 16; ++k) {
          const int64_t c = near * kGroup + (k * (k + 1) / 2 * 29 & (kGroup - 1));
          const float v = c < a.nc ? value(x, c) : -1.f;
          if (v > most) {
            most = v;
            at = c;
          }
        }
        left = !weighs(at);
      }
    }
    if (had && !left) s_lost[threadIdx.x] = 0.f;
    return __syncthreads_or(left) != 0;
  };
  const uint32_t word = threadIdx.x / 32, bit = threadIdx.x % 32;
  if (rows && !leave_rows(threadIdx.x < ROWS && row0 + threadIdx.x < a.nr && s_lost[threadIdx.x % ROWS] > 0.f)) return {0, 0};
  float size[NT];   // of vectors 16 t + l16, the largest 1
  bool gap[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    size[t] = largest > 0.f ? sh.size[16 * t + l16] / largest : 0.f;
    gap[t] = sh.gap[16 * t + l16] != 0;
  }
  for (int rb = 0; rb < RB; ++rb) {
    float z[4][NT];   // (all at once: row by row they are four waits)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = row0 + wave * 16 * RB + 16 * rb + 4 * q + r;
#pragma unroll
      for (int t = 0; t < NT; ++t) z[r][t] = out[(row < a.nr ? row : a.nr - 1) * B + 16 * t + l16];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = wave * 16 * RB + 16 * rb + 4 * q + r;
      const bool in = row0 + i < a.nr;
      const double lost = in ? fabs(row_factor(a, in ? row0 + i : a.nr - 1)) * (double)(kLostCut * s_lost[i]) : 0.0;
      bool low[NT], all = lost > 0.0, any = false;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        low[t] = fabs((double)z[r][t]) < lost * (double)size[t];
        any = any || low[t];
        all = all && (low[t] || size[t] == 0.f || !finite_bits(z[r][t]));
      }
      const bool whole = (__ballot(all) >> (16 * q) & 0xffff) == 0xffff && (__ballot(any) >> (16 * q) & 0xffff) != 0;
      if (whole && l16 == 0) atomicOr(&sh.rows[i / 32], 1u << (i % 32));
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (low[t] && gap[t] && !whole) {
          const int at = atomicAdd(&sh.n, 1);
          if (at < kEntries) s_entry[at] = (uint16_t)(i * B + 16 * t + l16);
          atomicOr(&sh.some[i / 32], 1u << (i % 32));
        }
    }
  }
  __syncthreads();
  const int found = sh.n;
  const bool many = found > kEntries;
  // (many entries: the rows that have them)
  if (many && !rows) (void)leave_rows(threadIdx.x < ROWS && (sh.some[threadIdx.x % ROWS / 32] >> bit & 1) != 0);
  if (!many && (int)threadIdx.x < found) {
    const int e = s_entry[threadIdx.x], i = e / B, vec = e % B;
    const int64_t c = in_place(i);
    const float* xr = a.xr + (row0 + i) * a.xr_stride;
    const float x[3] = {xr[0], xr[1], xr[2]};
    if (value(x, c) * __builtin_fabsf(a.Y[c * B + vec]) >= cut(i) * sh.size[vec]) s_entry[threadIdx.x] = kNoEntry;
  }
  __syncthreads();
  Lossy n = {0, 0};
  for (int k = 0; k < (many ? 0 : found); ++k) {
    if (s_entry[k] == kNoEntry) continue;
    const int e = s_entry[k], i = e / B, vec = e % B;
    const int64_t c = (g0 + s_best[i]) * kGroup + threadIdx.x;
    double s = 0.0, x[3], z[3];
    exact_point(a, a.xr + (row0 + i) * a.xr_stride, x);
#pragma unroll
    for (int u = 0; u < kGroup / kThreads; ++u) {
      const int64_t cu = c + u * kThreads;
      if (cu < c_begin || cu >= c_end) continue;
      exact_point(a, a.xc + cu * a.xc_stride, z);
      s += (double)(exact_value<KERNEL>(x, z) * __builtin_fabsf(a.Y[cu * B + vec]));
    }
    s = block_sum(s, sh.sum);
    if (!(s >= (double)(kLostCut * s_lost[i]) * (double)(sh.size[vec] / largest))) {
      if (threadIdx.x == 0) s_entry[n.entries] = (uint16_t)e;   // (n.entries <= k, and all have read entry k)
      ++n.entries;
    }
  }
  if (many) {
    if (threadIdx.x < ROWS && s_lost[threadIdx.x] == 0.f) atomicAnd(&sh.some[word], ~(1u << bit));
    __syncthreads();
  }
  int at = 0;
  uint32_t own = 0;
  for (int w = 0; w < ROWS / 32; ++w) {
    const uint32_t bits = sh.rows[w] | (many ? sh.some[w] : 0u);
    if (w < (int)word) at += __builtin_popcount(bits);
    if (w == (int)word) own = bits;
    n.rows += __builtin_popcount(bits);
  }
  if (own >> bit & 1) s_list[at + __builtin_popcount(own & ((1u << bit) - 1))] = (uint16_t)threadIdx.x;
  __syncthreads();   // (also: what is done again has been written)
  return n;
}

// Rows row0 + s_list[0 .. n) again, all columns of [c_begin, c_end) in FP32:
// 16 rows at a time, a quarter of the columns per wave.
template <int KERNEL, int B>
__device__ __forceinline__ void redo_rows(const GammaLaunch& a, int64_t row0, const uint16_t* s_list, int n,
                                          int64_t c_begin, int64_t c_end, double (*s_sum)[16 * B], float* out) {
  constexpr int NT = B / 16;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i0 = 0; i0 < n; i0 += 16) {
    const int i = i0 + (lane & 15);
    double x[1][3];
    exact_point(a, a.xr + (row0 + s_list[i < n ? i : n - 1]) * a.xr_stride, x[0]);
    d4v tot[1][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) tot[0][t] = (d4v){0.0, 0.0, 0.0, 0.0};
    const int64_t part = (c_end - c_begin + 3) / 4, c0 = c_begin + wave * part;
    exact_columns<KERNEL, B, 1>(a, x, (int)(c_end - c0 < part ? c_end - c0 : part), [&](int k) { return c0 + k; }, tot);
    __syncthreads();   // the sums of the rows before have been read
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) s_sum[wave][(4 * (lane >> 4) + r) * B + 16 * t + (lane & 15)] = tot[0][t][r];
    __syncthreads();
    for (int e = threadIdx.x; e < 16 * B; e += kThreads)
      if (i0 + e / B < n) {
        const int64_t row = row0 + s_list[i0 + e / B];
        out[row * B + e % B] = (float)(row_factor(a, row) * ((s_sum[0][e] + s_sum[1][e]) + (s_sum[2][e] + s_sum[3][e])));
      }
  }
}

// One entry again: a column per thread at a time, eight on their way.
template <int KERNEL, int B>
__device__ __forceinline__ void redo_entry(const GammaLaunch& a, int64_t row, int vec, int64_t c_begin, int64_t c_end,
                                           double* s_sum, float* out) {
  double x[3], s = 0.0;
  exact_point(a, a.xr + row * a.xr_stride, x);
  for (int64_t cb = c_begin; cb < c_end; cb += 8 * kThreads) {
    float p[8][3], y[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t c = cb + u * kThreads + threadIdx.x, cc = c < c_end ? c : c_end - 1;
#pragma unroll
      for (int k = 0; k < 3; ++k) p[u][k] = a.xc[cc * a.xc_stride + k];
      y[u] = a.Y[cc * B + vec];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      double z[3];
      exact_point(a, p[u], z);
      const float e = exact_value<KERNEL>(x, z);
      if (cb + u * kThreads + threadIdx.x < c_end) s += (double)e * (double)y[u];
    }
  }
  s = block_sum(s, s_sum);
  if (threadIdx.x == 0) out[row * B + vec] = (float)(row_factor(a, row) * s);
}

// One work item.  False where it has to be formed in FP32 as a whole: half of its
// columns or more are marked (not begun), or a quarter of its rows to be done
// again.
template <int KERNEL, int B, int RB>
__device__ __forceinline__ bool gamma_h16_item(const GammaLaunch& a, int64_t rblk, int split, uint4 (*s_x)[kXEntries],
                                               uint4 (*s_y)[2 * h16_entries<B>()], float (*s_box)[8]) {
  constexpr int ROWS = 64 * RB;
  __shared__ float s_row[3][ROWS];
  __shared__ float s_inv[2][ROWS];
  __shared__ float s_lost[ROWS];
  __shared__ int s_best[ROWS];
  __shared__ int s_flags, s_marks, s_size, s_look, s_cnt[4], s_few[kFewMarks];
  __shared__ uint32_t s_gap[2];
  const int64_t row0 = rblk * ROWS;
  const int64_t c0s = (int64_t)split * a.cols_per_split;
  const int64_t c1s = c0s + a.cols_per_split < a.nc ? c0s + a.cols_per_split : a.nc;
  const int64_t g0 = c0s / kGroup, g1 = (c1s + kGroup - 1) / kGroup;
  // (the first loads of what follows the rows' box)
  const int64_t own = row0 + threadIdx.x % ROWS;
  const float* xr = a.xr + (own < a.nr ? own : a.nr - 1) * a.xr_stride;
  const float x[3] = {xr[0], xr[1], xr[2]};
  const int64_t g_own = g0 + threadIdx.x < g1 ? g0 + threadIdx.x : g0;
  float flag_own = a.gbox[8 * g_own + 3], size_own = a.gbox[8 * g_own + 7];
  if (threadIdx.x == 0) s_flags = s_marks = s_size = s_look = 0;   // (gram_rows has a barrier)
  if (threadIdx.x < 2) s_gap[threadIdx.x] = 0;
  double cl[3];
  launch_centre(a, cl);
  float c0, c1, c2;
  (void)gram_rows<RB>(a, rblk, s_box, c0, c1, c2);
  c0 = uniform(row_centre<KERNEL>(s_box, 0, c0));
  c1 = uniform(row_centre<KERNEL>(s_box, 1, c1));
  c2 = uniform(row_centre<KERNEL>(s_box, 2, c2));
  // the flags of the columns' groups, their marked columns and the largest size of Y
  int flags = 0, size = 0;
  for (int64_t g = g0 + threadIdx.x; g < g1; g += kThreads) {
    if (g > g_own) {
      flag_own = a.gbox[8 * g + 3];
      size_own = a.gbox[8 * g + 7];
    }
    const int f = (int)flag_own;
    flags |= f & (kMarks - 1);
    size = max(size, __builtin_bit_cast(int, size_own));   // (not negative: in order as integers too)
    if (const int n = f / kMarks; n > kFewMarks) {   // (without the flags: what is counted as few is listed)
      atomicAdd(&s_marks, n);
    } else if (n > 0) {
      uint4 m[kGroup / 128];   // (all at once: word by word they are 16 waits)
#pragma unroll
      for (int k = 0; k < kGroup / 128; ++k) m[k] = reinterpret_cast<const uint4*>(a.gmask + g * (kGroup / 32))[k];
#pragma unroll
      for (int k = 0; k < kGroup / 32; ++k)
        for (uint32_t w = k % 4 == 0 ? m[k / 4].x : (k % 4 == 1 ? m[k / 4].y : (k % 4 == 2 ? m[k / 4].z : m[k / 4].w)); w; w &= w - 1) {
          const int64_t c = g * kGroup + 32 * k + __builtin_ctz(w);
          if (c < c0s || c >= c1s) continue;
          const int at = atomicAdd(&s_marks, 1);
          if (at < kFewMarks) s_few[at] = (int)(c - c0s);
        }
    }
  }
  // the rows' points relative to the launch's centre, and whether they are on the
  // lattice
  if (threadIdx.x < ROWS) {
#pragma unroll
    for (int k = 0; k < 3; ++k) s_row[k][threadIdx.x] = (float)lattice_coord(a, x[k], cl[k]);
    if (KERNEL == KA_GAUSSIAN && !lattice_point(a, x, cl).ok) flags |= kOffLattice;
  }
  if (size) atomicMax(&s_size, size);
  if (flags) atomicOr(&s_flags, flags);
  __syncthreads();
  flags = __builtin_amdgcn_readfirstlane(s_flags);
  const int marks = __builtin_amdgcn_readfirstlane(s_marks);
  if (2 * (int64_t)marks >= c1s - c0s) return false;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = lane >> 4;
  d4v tot[RB][B / 16];
  if (KERNEL == KA_GAUSSIAN && !(flags & kOffLattice))
    gamma_h16_tile<KERNEL, B, RB, true>(a, rblk, split, s_x, s_y, c0, c1, c2, cl, s_row, s_inv, s_few, marks, s_cnt, tot);
  else
    gamma_h16_tile<KERNEL, B, RB, false>(a, rblk, split, s_x, s_y, c0, c1, c2, cl, s_row, s_inv, s_few, marks, s_cnt, tot);

  // A kernel value is good to 2^-40 of what it could be at the row's distance
  // from the box of its group.  s_lost has the sum over the groups of what they
  // could give; each pair's loss is 2^-40 of that, all of a row's, with random
  // roundings, 2^-38, and a result below 2^-19 of it may owe that to columns that
  // are all much further off than the boxes.  It takes a load or more per group,
  // so first: is a result low if all groups were at the row?
  const double largest = (double)(kLostCut * (float)(g1 - g0)) * (double)__builtin_bit_cast(float, s_size);
  bool low = false;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      bool all = true, any = false;   // (a result that is not finite says nothing of the others)
#pragma unroll
      for (int t = 0; t < B / 16; ++t) {
        const double z = fabs(tot[rb][t][r]);
        any = any || z < largest;
        all = all && (z < largest || !(z < INFINITY));
      }
      low = low || (all && any);
    }
  if (__any(low && (lane & 15) < a.nv) && lane == 0) s_look = 1;
  __syncthreads();
  const bool look = s_look || (flags & kGaps);
  if (look) {
    if (flags & kGaps)
      for (int64_t g = 2 * g0 + threadIdx.x; g < 2 * g1; g += kThreads)
        if (const uint32_t gaps = a.ggap[g]) atomicOr(&s_gap[g & 1], gaps);
    if (threadIdx.x < ROWS) {
      float x[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) x[k] = s_row[k][threadIdx.x];
      float lost = 0.f, most = 0.f;
      int best = 0;
#pragma unroll 4
      for (int64_t g = g0; g < g1; ++g) {
        const uniform_float* b = (const uniform_float*)(uintptr_t)(a.gbox + 8 * g);
        float d = 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const float gap = fmaxf(fmaxf(b[k] - x[k], x[k] - b[4 + k]), 0.f);
          d += KERNEL == KA_GAUSSIAN ? gap * gap : gap;
        }
        const float v = d < kFarExponent ? __builtin_amdgcn_exp2f(-d) * b[7] : 0.f;
        lost += v;
        if (v > most) {
          most = v;
          best = (int)(g - g0);
        }
      }
      s_lost[threadIdx.x] = lost;
      s_best[threadIdx.x] = best;
    }
    __syncthreads();
  }
  float* out = a.nsplit > 1 ? a.partial + (size_t)split * a.nr * B : a.Z;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = row0 + wave * 16 * RB + 16 * rb + 4 * q + r;
      if (row < a.nr) {
        const double f = row_factor(a, row);
#pragma unroll
        for (int t = 0; t < B / 16; ++t) out[row * B + 16 * t + (lane & 15)] = (float)(f * tot[rb][t][r]);
      }
    }
  if (!look) return true;
  bool some = false, whole = false;   // (a low entry is of interest in a vector with gaps only)
  const uint32_t gaps = s_gap[0], gaps_hi = B == 64 ? s_gap[1] : 0u;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int r0 = wave * 16 * RB + 16 * rb + 4 * q;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double lost = row0 + r0 + r < a.nr ? (double)(kLostCut * s_lost[r0 + r]) : 0.0;
      bool all = true, any = false;
#pragma unroll
      for (int t = 0; t < B / 16; ++t) {
        const double z = fabs(tot[rb][t][r]);
        const bool low = z < lost;
        some = some || (low && ((t < 2 ? gaps : gaps_hi) >> (16 * (t & 1) + (lane & 15)) & 1) != 0);
        any = any || low;
        all = all && (low || !(z < INFINITY));
      }
      whole = whole || ((__ballot(all) >> (16 * q) & 0xffff) == 0xffff && (__ballot(any) >> (16 * q) & 0xffff) != 0);
    }
  }
  const bool rows = __syncthreads_or(whole) != 0;
  if (!rows && !((flags & kGaps) && __syncthreads_or(some))) return true;
  uint16_t* s_list = reinterpret_cast<uint16_t*>(&s_x[0][0]);
  constexpr size_t kPlace = sizeof(uint4) * kYRing * 2 * h16_entries<B>();
  static_assert(sizeof(LossyShared<B>) <= kPlace && sizeof(double) * 64 * B <= kPlace, "both take the place of Y's tiles");
  const Lossy n = lossy_results<KERNEL, B, RB>(a, row0, c0s, c1s, g0, g1, out, s_row, s_lost, s_best,
                                               *reinterpret_cast<LossyShared<B>*>(&s_y[0][0]), s_list, s_list + ROWS, rows);
  if (4 * n.rows >= ROWS) return false;
  if (n.rows > 0)
    redo_rows<KERNEL, B>(a, row0, s_list, n.rows, c0s, c1s, reinterpret_cast<double(*)[16 * B]>(&s_y[0][0]), out);
  for (int i = 0; i < n.entries; ++i)
    redo_entry<KERNEL, B>(a, row0 + s_list[ROWS + i] / B, s_list[ROWS + i] % B, c0s, c1s,
                          reinterpret_cast<double*>(&s_y[0][0]), out);
  return true;
}

// One work item, all of it in FP32.
template <int KERNEL, int B, int RB>
__device__ __forceinline__ void exact_item(const GammaLaunch& a, int64_t rblk, int split) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row0 = (rblk * 4 + wave) * (16 * RB);
  const int64_t c_begin = (int64_t)split * a.cols_per_split;
  const int64_t c_end = c_begin + a.cols_per_split < a.nc ? c_begin + a.cols_per_split : a.nc;
  double x[RB][3];
  d4v tot[RB][B / 16];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int64_t r = row0 + 16 * rb + (lane & 15);
    exact_point(a, a.xr + (r < a.nr ? r : a.nr - 1) * a.xr_stride, x[rb]);
#pragma unroll
    for (int t = 0; t < B / 16; ++t) tot[rb][t] = (d4v){0.0, 0.0, 0.0, 0.0};
  }
  exact_columns<KERNEL, B, RB>(a, x, (int)(c_end - c_begin), [&](int i) { return c_begin + i; }, tot);
  float* out = a.nsplit > 1 ? a.partial + (size_t)split * a.nr * B : a.Z;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = row0 + 16 * rb + 4 * (lane >> 4) + r;
      if (row < a.nr)
#pragma unroll
        for (int t = 0; t < B / 16; ++t) out[row * B + 16 * t + (lane & 15)] = (float)(row_factor(a, row) * tot[rb][t][r]);
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
  __shared__ float s_box[4][8];
  int64_t rblk;
  int split;
  if (!gamma_item(a, rblk, split)) return;
  if (!gamma_h16_item<KERNEL, B, RB>(a, rblk, split, s_x, s_y, s_box)) exact_item<KERNEL, B, RB>(a, rblk, split);
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

// scratch: Y's fragments, the points' operands, the scales, the boxes, the marks
size_t gamma_f16x3_bytes(int64_t nc, int b) {
  const size_t ng = ((size_t)nc + kGroup - 1) / kGroup;
  return ng * (kGroup * (b * 4 + 64) + b * sizeof(float) + 8 * sizeof(float) + kGroup / 8 + 8);
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
  p += ng * 8 * sizeof(float);
  a.gmask = (uint32_t*)p;
  p += ng * (kGroup / 8);
  a.ggap = (uint32_t*)p;
  a.ngroups = (int64_t)ng;
}

}  // namespace ka
