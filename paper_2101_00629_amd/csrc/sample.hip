// Sampling of the truncated Karhunen-Loeve expansion (paper Sec. 2, eq. kle):
//   alpha_M(x, s) = mu + sum_{i < M} sqrt(lambda_i) phi_i(x) xi_i(s)
// on a tensor grid of parametric points, for draws xi passed in.
//
// phi_i is the eigenfunction with coefficient column i of V in the problem's
// trial space (Galerkin: B-splines over sqrt|det DF|; collocation: the NURBS
// functions, or B_j / W on a general NURBS volume), scaled to unit L^2(D)
// norm (the expansion assumes orthonormal eigenfunctions).  Galerkin:
// int_D phi^2 = v^T Z v exactly, with Z = Z_3 x Z_2 x Z_1 the mass matrix.
// Collocation: int_D phi^2 by the collocation rule's Gauss points.
//
// Device work: Kronecker mode products in FP64 (Z v, or the eigenfunction
// values at the Gauss points; the values at the grid for Phi), fixed-order
// column reductions, and the field product F = mu + Phi diag(sqrt(lambda) /
// ||phi||) Xi on the FP64 matrix cores.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "ka_internal.hpp"

#define HIP_TRY(expr)                                                                    \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess) return ka::fail(KA_ERR_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

namespace ka {

typedef double d4v __attribute__((ext_vector_type(4)));

// Column dot products out[i] = sum_q w[q] A[q + i lda] B[q + i ldb] (w optional),
// in two fixed-order passes: workgroup (c, i) sums chunk c of column i, then
// one thread per column adds the chunk sums in order.
__global__ __launch_bounds__(256) void wdot_partial_kernel(const double* __restrict__ A, int64_t lda,
                                                           const double* __restrict__ B, int64_t ldb,
                                                           const double* __restrict__ w, int64_t Q, int64_t clen,
                                                           double* __restrict__ part) {
  __shared__ double red[256];
  const int i = blockIdx.y;
  const int64_t q0 = (int64_t)blockIdx.x * clen;
  const int64_t q1 = (q0 + clen < Q) ? q0 + clen : Q;
  const double* a = A + (int64_t)i * lda;
  const double* b = B + (int64_t)i * ldb;
  double s = 0.0;
  for (int64_t q = q0 + threadIdx.x; q < q1; q += 256) s += (w ? w[q] : 1.0) * a[q] * b[q];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[(int64_t)i * gridDim.x + blockIdx.x] = red[0];
}

__global__ void wdot_final_kernel(const double* __restrict__ part, int nchunk, int n, double* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
  for (int c = 0; c < nchunk; ++c) s += part[(int64_t)i * nchunk + c];
  out[i] = s;
}

// XiT[s + k Sp] = sqrt(lambda[k] / norm2[k]) Xi[k + s ldxi] for k < Kp, s < Sp,
// zero past K and S: the draws scaled, laid out sample-fastest and padded to
// whole MFMA tiles.  A norm that is not positive and finite sets *bad.
__global__ void xi_scale_kernel(const double* __restrict__ Xi, int64_t ldxi, int K, int S, int Kp, int64_t Sp,
                                const double* __restrict__ lambda, const double* __restrict__ norm2,
                                double* __restrict__ XiT, double* __restrict__ bad) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)Kp * Sp) return;
  const int s = (int)(id % Sp), k = (int)(id / Sp);
  double v = 0.0;
  if (k < K) {
    const double n = norm2[k];
    if (!(n > 0.0) || !(n - n == 0.0)) *bad = 1.0;
    if (s < S) v = sqrt(lambda[k] / n) * Xi[k + (int64_t)s * ldxi];
  }
  XiT[id] = v;
}

// F[p + s ldf] = mu + sum_k Phi[p + k ldp] XiT[s + k Sp].
//
// v_mfma_f64_16x16x4f64 with A = XiT^T (rows: samples) and B = Phi^T
// (columns: points), so a lane's 16 consecutive points land in consecutive
// addresses.  Operand layout (gfx950): A lane l holds (row l % 16, k = l / 16),
// B lane l holds (k = l / 16, column l % 16), accumulator register r of lane l
// holds (row l / 16 + 4 r, column l % 16).  A workgroup of 2 x 2 waves covers
// kFS samples x kFP points (each wave kU x kT MFMA tiles).  Workgroups
// are dealt to the 8 XCDs round-robin by id; the id mapping gives each XCD
// whole point-tiles (all their sample tiles back to back), so a tile of Phi
// is fetched from HBM into one L2 once.
//
// Bound by its stores and the FP64 matrix cores alike: a 64^3 grid, 1000
// samples and M = 50 write 2.1 GB (0.37 ms at the 5.7 TB/s of a plain fill) and
// take 2.7e10 flops (0.35 ms at 78 TFLOP/s).  A workgroup therefore walks
// `tiles` sample tiles of its points in one pipeline of k-steps: operands are
// requested two steps ahead across the tile ends, and a tile's stores go out
// while the next one's MFMAs run.  Operands past the edges are read at the edge
// and meet zeros of XiT, so no load is conditional.  The fields are not read
// again here: their stores are non-temporal.  At that size, with the products
// around it: 2846 us with conditional loads in each step and one tile per
// workgroup, 1095 us with unconditional ones ahead, 1024 us with the
// non-temporal stores, 982 / 959 / 950 / 926 us walking 1 / 2 / 4 / 8 tiles.
constexpr int kU = 2, kT = 4;                       // 16 x 16 MFMA tiles per wave: samples x points
constexpr int kFS = 2 * 16 * kU, kFP = 2 * 16 * kT;  // workgroup tile (2 x 2 waves)
constexpr int kMaxTiles = 8;                         // sample tiles per workgroup

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
void kl_field_kernel(const double* __restrict__ Phi, int64_t ldp, int64_t P, const double* __restrict__ XiT, int S,
                     int64_t Sp, int K, double mu, const double* __restrict__ bad, double* __restrict__ F, int64_t ldf,
                     int64_t n_pt, int n_sg, int tiles) {
  const int64_t L = blockIdx.x;
  const int64_t j = L / 8;
  const int64_t pt = (L % 8) + 8 * (j / n_sg);
  const int sg = (int)(j % n_sg);
  if (pt >= n_pt || *bad != 0.0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int64_t p0 = pt * kFP + (wave & 1) * (16 * kT);
  const int s_first = sg * tiles * kFS + (wave >> 1) * (16 * kU);
  const int left = (int)(Sp / kFS) - sg * tiles;
  const int ntile = left < tiles ? left : tiles;
  int64_t po[kT];
#pragma unroll
  for (int t = 0; t < kT; ++t) {
    const int64_t p = p0 + 16 * t + li;
    po[t] = p < P ? p : P - 1;
  }
  const int nk = (K + 3) / 4;
  // operands of the next k-step in turn (rows 4 c + lk of XiT^T and Phi^T),
  // past the last tile's end those of its first steps again
  int lc = 0, lt = 0;
  auto load = [&](double (&a)[kU], double (&b)[kT]) {
    const int k = 4 * lc + lk;
    const double* x = XiT + k * Sp + (s_first + lt * kFS + li);
#pragma unroll
    for (int u = 0; u < kU; ++u) a[u] = x[16 * u];
    const double* f = Phi + (int64_t)(k < K ? k : K - 1) * ldp;
#pragma unroll
    for (int t = 0; t < kT; ++t) b[t] = f[po[t]];
    if (++lc == nk) {
      lc = 0;
      if (lt + 1 < ntile) ++lt;
    }
  };
  d4v acc[kU][kT];
  auto step = [&](const double (&a)[kU], const double (&b)[kT]) {
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int t = 0; t < kT; ++t) acc[u][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[t], acc[u][t], 0, 0, 0);
  };
  double a0[kU], b0[kT], a1[kU], b1[kT];
  load(a0, b0);
  load(a1, b1);
  for (int tile = 0; tile < ntile; ++tile) {
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int t = 0; t < kT; ++t) acc[u][t] = (d4v){0.0, 0.0, 0.0, 0.0};
    // each step's operands are replaced as soon as its MFMAs are issued; the
    // scheduling barriers keep the compiler from sinking the loads
    int c = 0;
    for (; c + 2 <= nk; c += 2) {
      step(a0, b0);
      load(a0, b0);
      __builtin_amdgcn_sched_barrier(0);
      step(a1, b1);
      load(a1, b1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (c < nk) {
      step(a0, b0);
#pragma unroll
      for (int u = 0; u < kU; ++u) a0[u] = a1[u];
#pragma unroll
      for (int t = 0; t < kT; ++t) b0[t] = b1[t];
      load(a1, b1);
    }
    const int s0 = s_first + tile * kFS + lk;
    double* row = F + (int64_t)s0 * ldf + p0 + li;
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int t = 0; t < kT; ++t)
          if (s0 + 16 * u + 4 * r < S && p0 + 16 * t + li < P)
            __builtin_nontemporal_store(mu + acc[u][t][r], row + 16 * t);   // (one rounding at mu's size, not one per step)
        row += 4 * ldf;
      }
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
namespace {

// Workspace of one call, carved from the problem's kept buffer: sizes are
// collected first (256-byte aligned), then the buffer grows if needed.
struct KlArena {
  std::vector<size_t> off;
  size_t total = 0;
  size_t add(size_t doubles) {
    off.push_back(total);
    total += (std::max<size_t>(doubles, 1) * sizeof(double) + 255) / 256 * 256;
    return off.size() - 1;
  }
};

ModeArgs col_mode(const double* in, int64_t in_ld, double* out, int64_t out_ld, const int dims[3], int mode, int m,
                  const double* matT, int nv) {
  ModeArgs a;
  a.in = in;
  a.in_layout = LAYOUT_COL;
  a.in_ld = in_ld;
  a.out = out;
  a.out_layout = LAYOUT_COL;
  a.out_ld = out_ld;
  for (int k = 0; k < 3; ++k) a.n_in[k] = dims[k];
  a.mode = mode;
  a.m = m;
  a.matT = matT;
  a.nv = nv;
  a.out_scale = nullptr;
  return a;
}

// (E_3 x E_2 x E_1) V[:, 0 : nv] -> out (column-major, ld = m0 m1 m2), from the transposes of E_k
hipError_t kron_eval(const int n[3], const int m[3], double* const ET[3], const double* V, int64_t ldv,
                     int nv, double* t1, double* t2, double* out, int64_t ld_out, hipStream_t s) {
  const int d0[3] = {n[0], n[1], n[2]};
  const int d1[3] = {m[0], n[1], n[2]};
  const int d2[3] = {m[0], m[1], n[2]};
  const int64_t l1 = (int64_t)m[0] * n[1] * n[2], l2 = (int64_t)m[0] * m[1] * n[2];
  hipError_t e = launch_mode_f64(col_mode(V, ldv, t1, l1, d0, 0, m[0], ET[0], nv), s);
  if (e == hipSuccess) e = launch_mode_f64(col_mode(t1, l1, t2, l2, d1, 1, m[1], ET[1], nv), s);
  if (e == hipSuccess) e = launch_mode_f64(col_mode(t2, l2, out, ld_out, d2, 2, m[2], ET[2], nv), s);
  return e;
}

}  // namespace

}  // namespace ka

using namespace ka;

extern "C" int ka_kl_sample(ka_problem* p, int M, const double* lambda_host, const double* V_dev, int64_t ldv,
                            const int npts[3], const double* grid_host, int nsamples, const double* xi_dev,
                            int64_t ldxi, double mu, double* field_dev, int64_t ldf, void* stream) {
  Problem* P = reinterpret_cast<Problem*>(p);
  if (!P) return fail(KA_ERR_ARG, "problem is NULL");
  if (!lambda_host || !V_dev || !npts || !grid_host || !xi_dev || !field_dev) return fail(KA_ERR_ARG, "NULL argument");
  if (M < 1 || M > P->N) return fail(KA_ERR_ARG, "M must be in 1..N");
  if (nsamples < 1) return fail(KA_ERR_ARG, "nsamples must be >= 1");
  if (ldv < P->N || ldxi < M) return fail(KA_ERR_ARG, "leading dimension too small");
  if (!std::isfinite(mu)) return fail(KA_ERR_ARG, "mu must be finite");
  for (int i = 0; i < M; ++i)
    if (!(lambda_host[i] >= 0) || !std::isfinite(lambda_host[i])) return fail(KA_ERR_ARG, "eigenvalues must be finite and >= 0");
  int64_t Pts = 1;
  size_t off = 0;
  std::vector<Vec> grid(3);
  for (int k = 0; k < 3; ++k) {
    if (npts[k] < 1 || npts[k] > (1 << 20)) return fail(KA_ERR_ARG, "npts must be in 1..2^20");
    grid[k].assign(grid_host + off, grid_host + off + npts[k]);
    off += npts[k];
    for (double x : grid[k])
      if (!(x >= 0.0 && x <= 1.0)) return fail(KA_ERR_ARG, "grid coordinates must lie in [0, 1]");
    Pts *= npts[k];
  }
  if (Pts > ((int64_t)1 << 34)) return fail(KA_ERR_ARG, "grid too large");
  if (ldf < Pts) return fail(KA_ERR_ARG, "ldf must be >= the number of grid points");
  hipStream_t s = stream ? (hipStream_t)stream : P->stream;
  const ka_desc& d = P->d;
  const bool coll = d.method == KA_COLLOCATION;
  const bool nurbs = d.domain == KA_NURBS;
  const bool dir_weights = coll && !nurbs;   // collocation NURBS factors per direction (closed-form domains)
  const Geometry& geo = P->geo;

  // univariate trial matrices at the grid (and, for collocation, at the Gauss points of the norms)
  std::vector<Mat> Eq(3), Eg(3);
  std::vector<Vec> xq(3), wq(3);
  int n[3], mq[3], mg[3];
  for (int k = 0; k < 3; ++k) {
    const int pk = d.degree[k];
    const Vec& t = P->tsol[k];
    n[k] = P->n[k];
    mg[k] = npts[k];
    mq[k] = n[k];
    if (!trial_matrix_1d(geo, dir_weights, t, pk, k, grid[k], Eg[k]))
      return fail(KA_ERR_SINGULAR, "weight interpolation matrix is singular");
    if (coll && !P->kl_omega) {
      element_gauss(t, d.nq > 0 ? d.nq : pk + 1, xq[k], wq[k]);
      if (!trial_matrix_1d(geo, dir_weights, t, pk, k, xq[k], Eq[k]))
        return fail(KA_ERR_SINGULAR, "weight interpolation matrix is singular");
      mq[k] = (int)xq[k].size();
    } else if (coll) {
      mq[k] = P->kl_mq[k];
    }
  }
  // collocation: weights of int_D phi^2 at the Gauss points, |det DF| (times 1 / W^2 on a NURBS volume)
  const int64_t Q = (int64_t)mq[0] * mq[1] * mq[2];
  std::vector<double> omega;
  if (coll && !P->kl_omega) {
    omega.resize(Q);
    for (int64_t i = 0; i < Q; ++i) {
      const int64_t a1 = i % mq[0], a2 = (i / mq[0]) % mq[1], a3 = i / ((int64_t)mq[0] * mq[1]);
      const double xh[3] = {xq[0][a1], xq[1][a2], xq[2][a3]};
      double x[3], J, W;
      geo.eval(xh, x, &J, &W);
      omega[i] = wq[0][a1] * wq[1][a2] * wq[2][a3] * J / (W * W);
    }
  }
  // per-point scale of phi on the grid: Galerkin 1/sqrt|det DF|, NURBS
  // collocation 1/W.  On the closed-form domains |det DF| is a product of
  // functions of one coordinate each (the box: a constant; the quarter annulus:
  // r(eta) |C x C'|(xi)), taken into the rows of the univariate matrices.
  if (!coll && !nurbs) {
    auto det = [&](int k, double x) {
      double xh[3] = {0.5, 0.5, 0.5}, y[3], J;
      if (k >= 0) xh[k] = x;
      geo.eval(xh, y, &J, nullptr);
      return J;
    };
    const double J0 = det(-1, 0.0);
    for (int k = 0; k < 3; ++k)
      for (int a = 0; a < Eg[k].rows; ++a) {
        const double f = 1.0 / std::sqrt(k == 0 ? det(k, grid[k][a]) : det(k, grid[k][a]) / J0);
        for (int j = 0; j < Eg[k].cols; ++j) Eg[k](a, j) *= f;
      }
  }
  std::vector<double> gscale;
  if (nurbs) {
    gscale.resize(Pts);
    for (int64_t i = 0; i < Pts; ++i) {
      const int64_t a1 = i % mg[0], a2 = (i / mg[0]) % mg[1], a3 = i / ((int64_t)mg[0] * mg[1]);
      const double xh[3] = {grid[0][a1], grid[1][a2], grid[2][a3]};
      double x[3], J, W;
      geo.eval(xh, x, &J, &W);
      gscale[i] = coll ? 1.0 / W : 1.0 / std::sqrt(J);
    }
  }

  // collocation norm data: computed on the first call, kept by the problem
  auto keep = [&](const std::vector<double>& v) -> double* {
    void* p = nullptr;
    const size_t bytes = std::max<size_t>(v.size(), 1) * sizeof(double);
    if (hipMalloc(&p, bytes) != hipSuccess) return nullptr;
    P->allocs.push_back({p, bytes});
    P->device_bytes += bytes;
    if (hipMemcpy(p, v.data(), v.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) return nullptr;
    return (double*)p;
  };
  if (coll && !P->kl_omega) {
    for (int k = 0; k < 3; ++k) {
      P->kl_EqT[k] = keep(transpose(Eq[k]).a);
      if (!P->kl_EqT[k]) return fail(KA_ERR_OOM, "device allocation failed in ka_kl_sample");
      P->kl_mq[k] = mq[k];
    }
    P->kl_omega = keep(omega);
    if (!P->kl_omega) return fail(KA_ERR_OOM, "device allocation failed in ka_kl_sample");
  }
  // this call's workspace; the host's data (transposed grid matrices,
  // eigenvalues, the cleared flag) go up in one copy
  const int64_t tq = std::max((int64_t)mq[0] * n[1] * n[2], (int64_t)mq[0] * mq[1] * n[2]);
  const int64_t tg = std::max((int64_t)mg[0] * n[1] * n[2], (int64_t)mg[0] * mg[1] * n[2]);
  const int64_t clen = std::max<int64_t>(8192, (Q + 255) / 256);
  const int nchunk = (int)((Q + clen - 1) / clen);
  const int Kp = (M + 3) / 4 * 4;
  const int64_t Sp = ((int64_t)nsamples + kFS - 1) / kFS * kFS;
  std::vector<double> up;
  size_t oET[3];
  for (int k = 0; k < 3; ++k) {
    const Mat ET = transpose(Eg[k]);
    oET[k] = up.size();
    up.insert(up.end(), ET.a.begin(), ET.a.end());
  }
  const size_t olam = up.size();
  up.insert(up.end(), lambda_host, lambda_host + M);
  const size_t obad = up.size();
  up.push_back(0.0);
  // Vectors that go through the mode products together: up to 128 (a block of 16
  // to 64 leaves small grids latency-bound), but no more than 1 GiB of
  // intermediate blocks takes, or 32: on a grid that is fine in two directions
  // only these are larger than everything else.
  const double per_vector = (2.0 * (double)std::max(tq, tg) + (double)Q) * sizeof(double);
  int chunk = std::min(M, (int)std::max(32.0, std::min(128.0, (double)(1 << 30) / per_vector)));
  KlArena ar;
  size_t iup, it1, it2, iUq, ipart, inorm, iPhi, igs, iXi;
  for (;;) {
    ar = KlArena();
    iup = ar.add(up.size());
    it1 = ar.add((size_t)std::max(tq, tg) * chunk);
    it2 = ar.add((size_t)std::max(tq, tg) * chunk);
    iUq = ar.add((size_t)Q * chunk);
    ipart = ar.add((size_t)nchunk * chunk);
    inorm = ar.add(M);
    iPhi = ar.add((size_t)Pts * M);
    igs = ar.add(gscale.size());
    iXi = ar.add((size_t)Kp * Sp);
    if (P->kl_bytes >= ar.total) break;
    if (P->kl_buf) {
      (void)hipStreamSynchronize(s);
      (void)hipFree(P->kl_buf);
      P->kl_buf = nullptr;
      P->kl_bytes = 0;
    }
    if (hipMalloc(&P->kl_buf, ar.total) == hipSuccess) {
      P->kl_bytes = ar.total;
      break;
    }
    (void)hipGetLastError();
    P->kl_buf = nullptr;
    if (chunk <= 32) return fail(KA_ERR_OOM, "device allocation failed in ka_kl_sample");
    chunk = 32;
  }
  auto at = [&](size_t i) { return (double*)((char*)P->kl_buf + ar.off[i]); };
  double* up_d = at(iup);
  HIP_TRY(hipMemcpyAsync(up_d, up.data(), up.size() * sizeof(double), hipMemcpyHostToDevice, s));
  double *EqTd[3], *EgTd[3];
  for (int k = 0; k < 3; ++k) {
    EqTd[k] = coll ? P->kl_EqT[k] : P->Zk[k];    // Galerkin: Z v with the mass matrices (symmetric)
    EgTd[k] = up_d + oET[k];
  }
  double* t1 = at(it1);
  double* t2 = at(it2);
  double* Uq = at(iUq);
  const double* omega_d = coll ? P->kl_omega : nullptr;
  double* part = at(ipart);
  double* norms2 = at(inorm);
  double* Phi = at(iPhi);
  double* gscale_d = gscale.empty() ? nullptr : at(igs);
  if (gscale_d) HIP_TRY(hipMemcpyAsync(gscale_d, gscale.data(), gscale.size() * sizeof(double), hipMemcpyHostToDevice, s));
  double* XiT = at(iXi);

  for (int c0 = 0; c0 < M; c0 += chunk) {
    const int nv = std::min(chunk, M - c0);
    const double* Vc = V_dev + (int64_t)c0 * ldv;
    // collocation: phi at the Gauss points, norms^2 = sum omega phi^2; Galerkin: Z v, norms^2 = v^T Z v
    HIP_TRY(kron_eval(n, mq, EqTd, Vc, ldv, nv, t1, t2, Uq, Q, s));
    hipLaunchKernelGGL(wdot_partial_kernel, dim3(nchunk, nv), dim3(256), 0, s, Uq, Q, coll ? (const double*)Uq : Vc,
                       coll ? Q : ldv, omega_d, Q, clen, part);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(wdot_final_kernel, dim3((nv + 63) / 64), dim3(64), 0, s, part, nchunk, nv, norms2 + c0);
    HIP_TRY(hipGetLastError());
    HIP_TRY(kron_eval(n, mg, EgTd, Vc, ldv, nv, t1, t2, Phi + (int64_t)c0 * Pts, Pts, s));
  }
  if (gscale_d) HIP_TRY(scale_rows(Phi, Pts, M, Pts, gscale_d, s));
  double* bad_d = up_d + obad;
  const int64_t tot = Kp * Sp;
  hipLaunchKernelGGL(xi_scale_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, xi_dev, ldxi, M, nsamples,
                     Kp, Sp, up_d + olam, norms2, XiT, bad_d);
  HIP_TRY(hipGetLastError());
  const int64_t n_pt = (Pts + kFP - 1) / kFP;
  // as many sample tiles per workgroup as leave 2048 workgroups (8 on each CU,
  // twice what is resident)
  const int n_tiles = (int)(Sp / kFS);
  const int tiles = (int)std::max<int64_t>(1, std::min<int64_t>(kMaxTiles, n_pt * n_tiles / 2048));
  const int n_st = (n_tiles + tiles - 1) / tiles;
  const int64_t grid_wg = 8 * ((n_pt + 7) / 8) * (int64_t)n_st;
  if (grid_wg > ((int64_t)1 << 31) - 1) return fail(KA_ERR_ARG, "field too large for one launch");
  hipLaunchKernelGGL(kl_field_kernel, dim3((unsigned)grid_wg), dim3(256), 0, s, Phi, Pts, Pts, XiT, nsamples, Sp, M,
                     mu, bad_d, field_dev, ldf, n_pt, n_st, tiles);
  HIP_TRY(hipGetLastError());
  double bad = 0.0;
  HIP_TRY(hipMemcpyAsync(&bad, bad_d, sizeof(double), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));   // the host vectors copied above live until here
  if (bad != 0.0) return fail(KA_ERR_SINGULAR, "an eigenfunction has zero L2 norm");   // (no field was written)
  return KA_OK;
}
