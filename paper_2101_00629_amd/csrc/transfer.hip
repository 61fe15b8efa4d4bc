// Kronecker mode products: the "linear or nearly linear" steps of both
// matrix-free operators (paper Sec. 3.1: L^-T, M, B~^-T, J and their
// transposes; Sec. 3.2 / Algorithm 1: R at the quadrature points, J W
// scaling, the LU backsolve of Z).  A Kronecker matrix A3 (x) A2 (x) A1 acts
// on a block as three mode products, each contracting one tensor index with
// a small dense univariate matrix.
//
// One kernel serves all of them.  A product is a small matrix times a long
// one whose columns ("fibers") are the other tensor indices and the vectors;
// a block's layout (column-major at the API, point-major around the kernel
// product) is only the strides of those three indices, so the products at the
// two ends of a block application change the layout as they go.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ka_internal.hpp"

namespace ka {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ inline d4 mfma_k4(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ inline f4 mfma_k4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

struct ModeLaunch {
  const void* in;
  void* out;
  const void* matT;       // nk x m
  const float* scale;     // optional, at sc0 x + sc1 y + sc2 z + scm r
  int nk, m;              // contracted length, output rows
  int d0, d1;             // fiber q = x + d0 (y + d1 z)
  int64_t nfib;
  int64_t in0, in1, in2, ink;      // strides of x, y, z and of the contracted index
  int64_t out0, out1, out2, outm;
  int64_t sc0, sc1, sc2, scm;
  int kg;                 // groups of 16 contracted indices per matrix chunk in LDS
};

// out(r, q) = sum_c mat[r, c] in(c, q) on the matrix cores (f64 or f32
// 16 x 16 x 4): A = mat (rows r), B = in (columns q).  Lane l holds A (row
// l % 16, k = l / 16), B (k = l / 16, column l % 16) and of the accumulator
// column l % 16, rows l / 16 + 4 i (f64) or 4 (l / 16) + i (f32), i < 4.
// Which contracted index is "k" and which output row is "row" are free as long
// as both operands agree: lane group l / 16 takes the contracted indices
// 4 (l / 16) .. + 3 of each group of 16 and (f64, by permuting the rows of A)
// holds the output rows 4 (l / 16) .. + 3, so a fiber that is contiguous
// (INU) or an output that is (OUTU) moves in 128-byte pieces, and fibers that
// lie side by side do so across the lanes.  A wave takes 16 fibers, a
// workgroup of eight waves 128 in turn; the matrix is in LDS in operand order,
// in chunks of kg groups (reloaded only where it does not fit at once).
// Inputs are requested a group ahead, across the ends of a workgroup's tiles.
// Past the end of a fiber both operands are zero; fibers past the last repeat
// it and are not stored.
//
// Bound by memory where blocks are large, by latency where they are small.  A
// 66^3 block of 64 FP64 vectors is 147 MB in and 147 MB out, 74 us for a
// device copy, and its products take 44 us of the f64 matrix cores: 95 us on
// average over the three directions, column-major at both ends (before, one
// thread per fiber and 33 rows: 138 us, and 150 us for two transposes).  A 23^3
// block of 16 vectors: 5.7 us (before, 13 us).  Eight waves of one fiber tile
// per matrix ran the two in 361 and 138 us (three, and twelve products and the
// kernel product of a block application), four waves of two tiles in 371 and
// 156 us; two waves in 361 and 155 us, the small one waiting for the matrix.
constexpr int kThreads = 512;
constexpr int kFibers = kThreads / 4;   // per workgroup: 16 per wave

template <typename TIn, typename TAcc, typename TOut, int MT, bool INU, bool OUTU>
__global__ __launch_bounds__(kThreads, 6) void mode_kernel(ModeLaunch p) {
  using V4 = typename std::conditional<std::is_same<TAcc, double>::value, d4, f4>::type;
  constexpr bool F64 = std::is_same<TAcc, double>::value;
  extern __shared__ double lds_raw[];
  TAcc* As = reinterpret_cast<TAcc*>(lds_raw);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int m0 = blockIdx.y * (16 * MT);
  const int ng = (p.nk + 15) / 16;
  const int tail = p.nk - 16 * (ng - 1);      // 1 .. 16 in the last group
  const int tsteps = tail == 16 ? 4 : (tail + 3) / 4;
  const int64_t ntile = (p.nfib + kFibers - 1) / kFibers;

  // matrix chunk from group g0: slot ((g - g0) 4 + s) MT + t of 64 lanes
  auto fill = [&](int g0) {
    const int n = (ng - g0 < p.kg ? ng - g0 : p.kg) * 4 * MT * 64;
    const TAcc* matT = (const TAcc*)p.matT;
    for (int i = threadIdx.x; i < n; i += kThreads) {
      const int l = i & 63, slot = i >> 6;
      const int t = slot % MT, gs = slot / MT;
      const int g = g0 + (gs >> 2), s = gs & 3;
      const int ll = l & 15, kk = l >> 4;
      const int r = m0 + 16 * t + (F64 ? 4 * (ll & 3) + (ll >> 2) : ll);
      const int c = 16 * g + (g == ng - 1 && tail != 16 ? 4 * s + kk : 4 * kk + s);
      As[i] = r < p.m && c < p.nk ? matT[(int64_t)c * p.m + r] : (TAcc)0;
    }
  };
  auto split = [&](int64_t q, int64_t& x, int64_t& y, int64_t& z) {
    if (p.nfib <= 0x7fffffff) {
      const unsigned u = (unsigned)q, v = u / (unsigned)p.d0, w = v / (unsigned)p.d1;
      x = u - v * (unsigned)p.d0;
      y = v - w * (unsigned)p.d1;
      z = w;
    } else {
      const int64_t v = q / p.d0;
      x = q - v * p.d0;
      z = v / p.d1;
      y = v - z * p.d1;
    }
  };
  // the loader: runs one group ahead of the products
  int64_t ltile = blockIdx.x;
  int lg = 0;
  const TIn* src;
  auto locate = [&]() {
    int64_t q = ltile * kFibers + 16 * wave + li, x, y, z;
    q = q < p.nfib ? q : p.nfib - 1;
    split(q, x, y, z);
    src = (const TIn*)p.in + (x * p.in0 + y * p.in1 + z * p.in2);
  };
  auto load = [&](TIn (&v)[4]) {
    if (ltile >= ntile) return;
    if (lg + 1 < ng || tail == 16) {
      const int64_t o = 16 * lg + 4 * lk;
#pragma unroll
      for (int s = 0; s < 4; ++s) v[s] = INU ? src[o + s] : src[(o + s) * p.ink];
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int c = 16 * lg + 4 * s + lk;
        const TIn w = src[(int64_t)(c < p.nk ? c : p.nk - 1) * (INU ? 1 : p.ink)];
        v[s] = c < p.nk ? w : (TIn)0;
      }
    }
    if (++lg == ng) {
      lg = 0;
      ltile += gridDim.x;
      if (ltile < ntile) locate();
    }
  };

  V4 acc[MT];
  int64_t tile = blockIdx.x;
  auto clear = [&]() {
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = (V4){0, 0, 0, 0};
  };
  auto store = [&]() {
    const int64_t q = tile * kFibers + 16 * wave + li;
    if (q >= p.nfib) return;
    int64_t x, y, z;
    split(q, x, y, z);
    int r = m0 + 4 * lk;
    const int64_t om = OUTU ? 1 : p.outm;
    TOut* o = (TOut*)p.out + (x * p.out0 + y * p.out1 + z * p.out2 + r * om);
    const float* sc = p.scale ? p.scale + (x * p.sc0 + y * p.sc1 + z * p.sc2 + r * p.scm) : nullptr;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (r + i < p.m) {
          TAcc v = acc[t][i];
          if (sc) v *= (TAcc)sc[i * p.scm];
          o[i * om] = (TOut)v;
        }
      }
      r += 16;
      o += 16 * om;
      if (sc) sc += 16 * p.scm;
    }
  };

  TIn v[4], w[4];
  locate();
  load(v);
  if (p.kg >= ng) {
    fill(0);
    __syncthreads();
  }
  for (; tile < ntile; tile += gridDim.x) {
    clear();
    int gl = 0;   // group within the matrix chunk in LDS
#pragma unroll 1
    for (int g = 0; g < ng; ++g) {
      if (p.kg < ng && (gl == p.kg || g == 0)) {
        __syncthreads();
        fill(g);
        __syncthreads();
        gl = 0;
      }
      load(w);
      __builtin_amdgcn_sched_barrier(0);
      const TAcc* A = As + gl++ * (4 * MT * 64) + lane;
      const int steps = g + 1 < ng ? 4 : tsteps;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (s < steps) {
#pragma unroll
          for (int t = 0; t < MT; ++t) acc[t] = mfma_k4(A[(s * MT + t) * 64], (TAcc)v[s], acc[t]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 4; ++s) v[s] = w[s];
    }
    store();
  }
}

template <typename TIn, typename TAcc, typename TOut, int MT, bool INU, bool OUTU>
static hipError_t launch_mode_mt(ModeLaunch& p, hipStream_t s) {
  const int ng = (p.nk + 15) / 16;
  const int group = 4 * MT * 64 * (int)sizeof(TAcc);   // bytes of a group's matrix operands
  p.kg = std::min(ng, 65536 / group);
  const int64_t ntile = (p.nfib + kFibers - 1) / kFibers;
  // workgroups that are resident at once, each with as many tiles as any other
  const int64_t res = 256 * std::max(1, std::min(3, 163840 / (p.kg * group)));
  const int64_t rounds = (ntile + res - 1) / res;
  const dim3 grid((unsigned)((ntile + rounds - 1) / rounds), (unsigned)((p.m + 16 * MT - 1) / (16 * MT)));
  hipLaunchKernelGGL((mode_kernel<TIn, TAcc, TOut, MT, INU, OUTU>), grid, dim3(kThreads), (size_t)p.kg * group, s, p);
  return hipGetLastError();
}

template <typename TIn, typename TAcc, typename TOut, bool INU, bool OUTU>
static hipError_t launch_mode_io(ModeLaunch& p, hipStream_t s) {
  // 16 MT rows per pass over the input: up to 80 in one, longer modes in equal passes
  const int mt = (p.m + 15) / 16, passes = (mt + 4) / 5;
  switch ((mt + passes - 1) / passes) {
    case 1: return launch_mode_mt<TIn, TAcc, TOut, 1, INU, OUTU>(p, s);
    case 2: return launch_mode_mt<TIn, TAcc, TOut, 2, INU, OUTU>(p, s);
    case 3: return launch_mode_mt<TIn, TAcc, TOut, 3, INU, OUTU>(p, s);
    case 4: return launch_mode_mt<TIn, TAcc, TOut, 4, INU, OUTU>(p, s);
    default: return launch_mode_mt<TIn, TAcc, TOut, 5, INU, OUTU>(p, s);
  }
}

// The fiber indices x, y, z: with a point-major block at either end the
// vectors come first, else the directions in memory order.
template <typename TIn, typename TAcc, typename TOut>
static hipError_t launch_mode(const ModeArgs& a, hipStream_t s) {
  const int nk = a.n_in[a.mode];
  const int64_t nfib = (int64_t)a.n_in[0] * a.n_in[1] * a.n_in[2] / std::max(nk, 1) * a.nv;
  if (nfib == 0 || a.m == 0 || nk == 0) return hipSuccess;
  ModeLaunch p;
  p.in = a.in;
  p.out = a.out;
  p.matT = a.matT;
  p.scale = a.out_scale;
  p.nk = nk;
  p.m = a.m;
  p.nfib = nfib;
  p.kg = 0;
  // strides of the two other directions and of the contracted one, in points
  const int da = a.mode == 0 ? 1 : 0, db = a.mode == 2 ? 1 : 2;
  int no[3] = {a.n_in[0], a.n_in[1], a.n_in[2]};
  no[a.mode] = a.m;
  const int64_t si[3] = {1, a.n_in[0], (int64_t)a.n_in[0] * a.n_in[1]};
  const int64_t so[3] = {1, no[0], (int64_t)no[0] * no[1]};
  const bool ipt = a.in_layout == LAYOUT_PT, opt = a.out_layout == LAYOUT_PT;
  const int64_t ip = ipt ? a.in_ld : 1, iv = ipt ? 1 : a.in_ld;     // strides of a point and of a vector
  const int64_t op = opt ? a.out_ld : 1, ov = opt ? 1 : a.out_ld;
  p.ink = si[a.mode] * ip;
  p.outm = so[a.mode] * op;
  p.scm = so[a.mode];
  if (ipt || opt) {          // x: vectors, y and z: directions
    p.d0 = a.nv;
    p.d1 = a.n_in[da];
    p.in0 = iv, p.in1 = si[da] * ip, p.in2 = si[db] * ip;
    p.out0 = ov, p.out1 = so[da] * op, p.out2 = so[db] * op;
    p.sc0 = 0, p.sc1 = so[da], p.sc2 = so[db];
  } else {                   // x and y: directions, z: vectors
    p.d0 = a.n_in[da];
    p.d1 = a.n_in[db];
    p.in0 = si[da], p.in1 = si[db], p.in2 = iv;
    p.out0 = so[da], p.out1 = so[db], p.out2 = ov;
    p.sc0 = so[da], p.sc1 = so[db], p.sc2 = 0;
  }
  // (INU and OUTU are instantiated where the operators need them; the others
  // are right for any stride)
  constexpr bool kInCol = std::is_same<TIn, double>::value, kOutCol = std::is_same<TOut, double>::value;
  const bool inu = kInCol && p.ink == 1, outu = kOutCol && p.outm == 1;
  if (inu && outu) return launch_mode_io<TIn, TAcc, TOut, kInCol, kOutCol>(p, s);
  if (inu) return launch_mode_io<TIn, TAcc, TOut, kInCol, false>(p, s);
  if (outu) return launch_mode_io<TIn, TAcc, TOut, false, kOutCol>(p, s);
  return launch_mode_io<TIn, TAcc, TOut, false, false>(p, s);
}

hipError_t launch_mode_f64(const ModeArgs& a, hipStream_t s) { return launch_mode<double, double, double>(a, s); }
hipError_t launch_mode_f64_to_f32(const ModeArgs& a, hipStream_t s) { return launch_mode<double, float, float>(a, s); }
hipError_t launch_mode_f32(const ModeArgs& a, hipStream_t s) { return launch_mode<float, float, float>(a, s); }
hipError_t launch_mode_f32_to_f64(const ModeArgs& a, hipStream_t s) { return launch_mode<float, float, double>(a, s); }
hipError_t launch_mode_f32in_f64(const ModeArgs& a, hipStream_t s) { return launch_mode<float, double, double>(a, s); }

// Layout changes between the column-major API blocks (element (i, j) at
// i + j ld) and the point-major operator blocks (at i ld + j), through LDS
// tiles of 64 points x 64 vectors so that both sides are read and written in
// memory order.  kPad keeps the transposed LDS reads free of bank conflicts.
constexpr int kTP = 64;
constexpr int kPad = 1;

// point-major TIn (ld_in) -> column-major TOut (ld_out), divided by div[i] if given
template <typename TIn, typename TOut>
__global__ __launch_bounds__(256) void pt_to_col_kernel(const TIn* __restrict__ in, int64_t ld_in,
                                                        TOut* __restrict__ out, int64_t ld_out, int64_t npts, int nv,
                                                        const double* __restrict__ div) {
  __shared__ double t[kTP][kTP + kPad];
  const int64_t p0 = (int64_t)blockIdx.x * kTP;
  const int j0 = blockIdx.y * kTP;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int pp = ty; pp < kTP; pp += 4) {          // read point rows: lanes over vectors
    const int64_t p = p0 + pp;
    const int j = j0 + tx;
    if (p < npts && j < nv) t[pp][tx] = (double)in[p * ld_in + j];
  }
  __syncthreads();
  for (int jj = ty; jj < kTP; jj += 4) {          // write columns: lanes over points
    const int64_t p = p0 + tx;
    const int j = j0 + jj;
    if (p < npts && j < nv) {
      const double v = t[tx][jj];
      out[p + (int64_t)j * ld_out] = (TOut)(div ? v / div[p] : v);
    }
  }
}

static dim3 tile_grid(int64_t npts, int nv) {
  return dim3((unsigned)((npts + kTP - 1) / kTP), (unsigned)((nv + kTP - 1) / kTP));
}

hipError_t cast_pt32_to_col64(const float* in, int64_t ld_in, double* out, int64_t ld_out, int64_t npts, int nv,
                              const double* div, hipStream_t s) {
  if (npts * nv == 0) return hipSuccess;
  hipLaunchKernelGGL((pt_to_col_kernel<float, double>), tile_grid(npts, nv), dim3(256), 0, s, in, ld_in, out, ld_out,
                     npts, nv, div);
  return hipGetLastError();
}

}  // namespace ka
