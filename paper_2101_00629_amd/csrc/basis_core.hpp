// Orthonormal basis of the span of a set of vectors, from their Gram matrix,
// for the thick restart of the non-symmetric (collocation) eigensolver: the
// kept Ritz vectors S (columns of the projected space) are in general not
// orthogonal, and the restarted Krylov basis is X S W with W such that S W
// has orthonormal columns.
//
// Diagonal-pivoted Cholesky of the positive semi-definite G = S^T S: at step
// j the largest remaining diagonal entry is moved to position j (rows and
// columns swapped), R(j, j) is its square root, row j of R is the rest of
// row j divided by it, and the trailing block loses the outer product of that
// row.  The remaining diagonal entries are the squared distances of the
// remaining vectors from the span of the chosen ones, so the factorisation
// stops at the first pivot at or below cut * max_i G(i, i): the vectors from
// there on are dependent on the chosen ones to that accuracy.  With the r
// chosen pivots P^T G P = R^T R (leading r x r), and W = P[:, :r] R^-1.
// (Textbook pivoted Cholesky, e.g. Golub and Van Loan Sec. 4.2.8; the rank cut
// replaces the eigenvalue cut of a Gram eigendecomposition.)
//
// Written once over a team of threads (tid(), size(), sync(), and
// argmax(v, i): the index i of the largest v over the threads that look for one
// together, the smallest index among equals, -1 when no thread has one (i < 0),
// returned to every thread), so the same source runs as one
// workgroup on the device and as one thread in the host unit tests.
#pragma once
#include <math.h>
#include <stddef.h>

#ifndef KA_HD
#ifdef __HIPCC__
#define KA_HD __host__ __device__
#else
#define KA_HD
#endif
#endif
#ifndef KA_FORCEINLINE
#define KA_FORCEINLINE __attribute__((always_inline)) inline
#endif

namespace ka {

// 1 / sqrt(x) of a finite x > 0, to an ulp or two (the device's own square root
// and division are chains several times as long)
KA_HD inline double rsqrt_pos(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  double y = __builtin_amdgcn_rsq(x);
  for (int i = 0; i < 2; ++i) {
    const double e = __builtin_fma(-x * y, y, 1.0);
    y = __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
  }
  return y;
#else
  return 1.0 / sqrt(x);
#endif
}

// the threads that look for a maximum together: the whole team, unless it says otherwise
template <class Team>
KA_HD int argmax_lane(const Team& tm) { return tm.tid(); }
template <class Team>
KA_HD int argmax_lanes(const Team& tm) { return tm.size(); }

KA_HD inline size_t pchol_basis_work(int n) { return (size_t)n * n + 2 * (size_t)n; }   // doubles

// G: n x n (column-major, leading dimension ldg), symmetric positive
// semi-definite.  work: team-shared, pchol_basis_work(n) doubles (fast memory
// where it fits): the working copy, whose upper triangle becomes R and whose
// strictly lower triangle then holds R^-1 transposed, the diagonal of R^-1,
// and the pivot order.  W: n x n (leading dimension ldw): columns 0 .. r-1
// receive the basis coefficients, the others are left untouched.  Returns r
// (0 when G is zero).  Inlined, so that each caller accesses its work array
// with the instructions of that array's address space.
template <class Team>
KA_HD KA_FORCEINLINE int pchol_basis(Team& tm, const double* G, int ldg, int n, double cut, double* work, double* W, int ldw) {
  const int t = tm.tid(), NT = tm.size();
  if (n <= 0) return 0;
  // two-index loops: NI threads down a column, NG columns at once
  const int NI = NT < 32 ? NT : 32, NG = NT / NI, ti = t % NI, tg = t / NI;
  double* A = work;                         // working copy; R in its upper triangle
  double* xd = A + (size_t)n * n;           // diagonal of R^-1
  int* piv = reinterpret_cast<int*>(xd + n);
#define AA(i, j) A[(size_t)(j) * n + (i)]
#define XX(i, j) ((i) == (j) ? xd[i] : A[(size_t)(i) * n + (j)])   // R^-1 (i <= j), stored transposed below
  for (int l = tg; l < n; l += NG)
    for (int i = ti; i < n; i += NI) AA(i, l) = G[(size_t)l * ldg + i];
  for (int i = t; i < n; i += NT) piv[i] = i;
  tm.sync();
  const int al = argmax_lane(tm), an = argmax_lanes(tm);
  auto largest = [&](int lo) {                          // place of the largest diagonal entry from lo on
    int best = -1;
    double bv = -1.0;
    for (int i = lo + al; i < n; i += an)
      if (AA(i, i) > bv) {
        bv = AA(i, i);
        best = i;
      }
    return tm.argmax(bv, best);
  };
  const int i0 = largest(0);
  const double dmax = i0 >= 0 ? AA(i0, i0) : 0.0;
  int r = n;
  for (int j = 0; j < n; ++j) {
    const int p = largest(j);
    const double d = p >= 0 ? AA(p, p) : 0.0;
    if (!(d > cut * dmax) || !(d > 0.0)) {
      r = j;
      break;
    }
    const double inv = rsqrt_pos(d);
    tm.sync();
    if (p != j) {                                       // symmetric swap of rows and columns j and p
      for (int i = t; i < n; i += NT) {
        if (i == p) continue;
        double x;
        if (i != j) {
          x = AA(j, i);
          AA(j, i) = AA(p, i);
          AA(p, i) = x;
          x = AA(i, j);
          AA(i, j) = AA(i, p);
          AA(i, p) = x;
        } else {
          x = AA(j, j);
          AA(j, j) = AA(p, p);
          AA(p, p) = x;
          x = AA(j, p);
          AA(j, p) = AA(p, j);
          AA(p, j) = x;
          const int q = piv[j];
          piv[j] = piv[p];
          piv[p] = q;
        }
      }
      tm.sync();
    }
    if (t == 0) xd[j] = inv;
    // trailing block: A(i, l) -= R(j, i) R(j, l); row j itself is divided by its pivot at the end
    for (int l = j + 1 + tg; l < n; l += NG) {
      const double x = AA(j, l) * inv;
      for (int i = j + 1 + ti; i < n; i += NI) AA(i, l) -= (AA(j, i) * inv) * x;
    }
    tm.sync();
  }
  tm.sync();
  for (int l = 1 + tg; l < r; l += NG)
    for (int j = ti; j < l; j += NI) AA(j, l) *= xd[j];
  tm.sync();
  // X = R^-1 row by row from the bottom: X(i, i) = 1 / R(i, i) and
  // X(i, c) = -X(i, i) * sum_{k = i+1 .. c} R(i, k) X(k, c).  The sums of the
  // rows above are kept where X goes (the strictly lower triangle of the
  // working copy is free once R is done), and each finished row is added to all
  // of them at once: a step is one product per entry, not a sum of r of them.
  for (int c = tg; c < r; c += NG)
    for (int k = ti; k < c; k += NI) A[(size_t)k * n + c] = 0.0;
  tm.sync();
  for (int i = r - 1; i >= 0; --i) {
    const double d = xd[i];
    for (int k = tg; k < i; k += NG) {
      const double x = AA(k, i);
      for (int c = i + ti; c < r; c += NI) A[(size_t)k * n + c] += x * (c == i ? d : -d * A[(size_t)i * n + c]);
    }
    tm.sync();
  }
  for (int c = tg; c < r; c += NG)
    for (int k = ti; k < c; k += NI) A[(size_t)k * n + c] *= -xd[k];
  tm.sync();
  // W = P[:, :r] R^-1: row i of R^-1 lands in row piv[i] of W
  for (int c = tg; c < r; c += NG)
    for (int i = ti; i < n; i += NI) W[(size_t)c * ldw + piv[i]] = (i <= c) ? XX(i, c) : 0.0;
  tm.sync();
#undef AA
#undef XX
  return r;
}

}  // namespace ka
