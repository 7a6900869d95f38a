// Compile-time constants of the reference element shared by the step and
// adjoint kernels (gfx950): the time basis and the reconstruction's basis of
// shifted monomials, with the quadrature of monomial means on a triangle.
#pragma once

#include <hip/hip_runtime.h>

#include "common.h"

namespace aw {
// internal linkage: each kernel file folds these constants into its own code
namespace {

// Monomial coefficients of the Lagrange polynomials l_q on the time nodes
// q/M (q = 0..M) and of their integrals from 0, evaluated at compile time so
// that they enter the kernels as constants (the same polynomials as the host
// tables, built as products of the linear factors (tau - j/M) / ((q - j)/M)).
template <int M>
struct TimePoly {
  static constexpr int T = M + 1;
  struct Coef {
    double lag[T][T];
    double lint[T][T + 1];
  };
  static constexpr Coef make() {
    Coef c{};
    for (int q = 0; q < T; ++q) {
      double p[T] = {};
      p[0] = 1.0;
      int deg = 0;
      for (int j = 0; j < T; ++j) {
        if (j == q) continue;
        const double tj = double(j) / M, den = double(q - j) / M;
        double np[T] = {};
        for (int k = 0; k <= deg; ++k) {
          np[k + 1] += p[k] / den;
          np[k] -= p[k] * tj / den;
        }
        ++deg;
        for (int k = 0; k < T; ++k) p[k] = np[k];
      }
      c.lint[q][0] = 0.0;
      for (int k = 0; k < T; ++k) {
        c.lag[q][k] = p[k];
        c.lint[q][k + 1] = p[k] / (k + 1);
      }
    }
    return c;
  }
  static constexpr Coef c = make();
};

template <int M>
__device__ inline void time_basis(double tau, double l[M + 1]) {
  constexpr auto& C = TimePoly<M>::c;
#pragma unroll
  for (int q = 0; q <= M; ++q) {
    double s = C.lag[q][M];
#pragma unroll
    for (int k = M - 1; k >= 0; --k) s = s * tau + C.lag[q][k];
    l[q] = s;
  }
}

template <int M>
__device__ inline void time_antideriv(double tau, double L[M + 1]) {
  constexpr auto& C = TimePoly<M>::c;
#pragma unroll
  for (int q = 0; q <= M; ++q) {
    double s = C.lint[q][M + 1];
#pragma unroll
    for (int k = M; k >= 0; --k) s = s * tau + C.lint[q][k];
    L[q] = s;
  }
}

// Means of the monomials x^a y^b over the reference triangle (0,0), (1,0),
// (0,1): 2 a! b! / (a + b + 2)!, in the order of increasing degree, then b.
template <int M>
struct RefMeans {
  static constexpr double fact(int n) { return n <= 1 ? 1.0 : n * fact(n - 1); }
  struct Arr {
    double v[(M + 1) * (M + 2) / 2];
    constexpr double operator[](int k) const { return v[k]; }
  };
  static constexpr Arr make() {
    Arr r{};
    int k = 0;
    for (int d = 0; d <= M; ++d)
      for (int b = 0; b <= d; ++b) r.v[k++] = 2.0 * fact(d - b) * fact(b) / fact(d + 2);
    return r;
  }
  static constexpr Arr m = make();
};

// The reconstruction's basis: the monomials x^a y^b (1 <= a + b <= M, by
// degree, then b) minus their means on the reference triangle. For it, at
// compile time: the oscillation-indicator matrix (sum over all derivatives of
// orders 1..M of the integral of their products over the reference triangle,
// eq. eqn.sigma) and the values at the nodal lattice (i/M, j/M), i + j <= M,
// ordered by j then i. Integrals of x^p y^q over the triangle: p! q! / (p+q+2)!.
template <int M>
struct MonoBasis {
  static constexpr int nb = (M + 1) * (M + 2) / 2, nu = nb - 1;
  struct Coef {
    double sig[nu][nu];
    double node[nb][nu];
  };
  static constexpr double fact(int n) { return n <= 1 ? 1.0 : n * fact(n - 1); }
  static constexpr double falling(int n, int k) { return k == 0 ? 1.0 : n * falling(n - 1, k - 1); }
  static constexpr double ipow(double x, int n) { return n == 0 ? 1.0 : x * ipow(x, n - 1); }
  static constexpr Coef make() {
    Coef c{};
    int ea[nb] = {}, eb[nb] = {};
    int k = 0;
    for (int d = 0; d <= M; ++d)
      for (int b = 0; b <= d; ++b) {
        ea[k] = d - b;
        eb[k] = b;
        ++k;
      }
    for (int l = 1; l < nb; ++l)
      for (int m = 1; m < nb; ++m) {
        double s = 0.0;
        for (int ord = 1; ord <= M; ++ord)
          for (int be = 0; be <= ord; ++be) {
            const int al = ord - be;
            if (ea[l] < al || eb[l] < be || ea[m] < al || eb[m] < be) continue;
            const int p = ea[l] + ea[m] - 2 * al, q = eb[l] + eb[m] - 2 * be;
            s += falling(ea[l], al) * falling(eb[l], be) * falling(ea[m], al) * falling(eb[m], be) *
                 fact(p) * fact(q) / fact(p + q + 2);
          }
        c.sig[l - 1][m - 1] = s;
      }
    int n = 0;
    for (int j = 0; j <= M; ++j)
      for (int i = 0; i + j <= M; ++i) {
        const double x = double(i) / M, y = double(j) / M;
        for (int l = 1; l < nb; ++l)
          c.node[n][l - 1] = ipow(x, ea[l]) * ipow(y, eb[l]) -
                             2.0 * fact(ea[l]) * fact(eb[l]) / fact(ea[l] + eb[l] + 2);
        ++n;
      }
    return c;
  }
  static constexpr Coef c = make();
};

// Means of the monomials x^a y^b (a + b <= M) over a triangle with vertices
// (x[k], y[k]), in closed form: with the vertex sums S_x = sum x_k, S_y and the
// power sums P_pq = sum x_k^p y_k^q,
//   mean(x) = S_x / 3, mean(xy) = (S_x S_y + P_11) / 12,
//   mean(x^3) = (S_x^3 + 3 S_x P_20 + 2 P_30) / 60 and its polarised forms.
// About half the operations of a quadrature over the edge midpoints (M=2: 21
// instead of 40), no cancellation beyond that of the rule's own sums.
template <int M>
__device__ inline void monomial_means(const double x[3], const double y[3], double mm[]) {
  constexpr double third = 1.0 / 3.0;
  mm[0] = 1.0;
  const double sx = x[0] + x[1] + x[2], sy = y[0] + y[1] + y[2];
  mm[1] = sx * third;
  mm[2] = sy * third;
  if constexpr (M >= 2) {
    const double p20 = x[0] * x[0] + x[1] * x[1] + x[2] * x[2];
    const double p11 = x[0] * y[0] + x[1] * y[1] + x[2] * y[2];
    const double p02 = y[0] * y[0] + y[1] * y[1] + y[2] * y[2];
    constexpr double twelfth = 1.0 / 12.0;
    mm[3] = (sx * sx + p20) * twelfth;
    mm[4] = (sx * sy + p11) * twelfth;
    mm[5] = (sy * sy + p02) * twelfth;
    if constexpr (M >= 3) {
      double p30 = 0.0, p21 = 0.0, p12 = 0.0, p03 = 0.0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double xx = x[k] * x[k], yy = y[k] * y[k];
        p30 += xx * x[k];
        p21 += xx * y[k];
        p12 += x[k] * yy;
        p03 += yy * y[k];
      }
      constexpr double sixtieth = 1.0 / 60.0;
      const double sxx = sx * sx, syy = sy * sy;
      mm[6] = (sx * (sxx + 3.0 * p20) + 2.0 * p30) * sixtieth;
      mm[7] = (sy * (sxx + p20) + 2.0 * (sx * p11 + p21)) * sixtieth;
      mm[8] = (sx * (syy + p02) + 2.0 * (sy * p11 + p12)) * sixtieth;
      mm[9] = (sy * (syy + 3.0 * p02) + 2.0 * p03) * sixtieth;
    }
  }
}

// Least squares of a stencil by Householder reflections over blocks of rows
// held in registers. Row c is (a[c], b[c]): NU unknowns, four right-hand sides.
// A reflection clears a whole column of a block with one inverse square root
// and one reciprocal; Givens rotations, row by row, need one inverse square
// root per entry (55 at M=2 instead of 10) and twice the multiply-adds.
//
// block_qr: triangular factor of the first P >= NU rows, left in a[0..NU) (upper
// triangle) and b[0..NU).
template <int NU, int P>
__device__ inline void block_qr(double (&a)[P][NU], double (&b)[P][4]) {
#pragma unroll
  for (int k = 0; k < NU; ++k) {
    double s2 = 0.0;
#pragma unroll
    for (int p = k + 1; p < P; ++p) s2 += a[p][k] * a[p][k];
    const double al = a[k][k];
    const double mu2 = al * al + s2;
    if (mu2 == 0.0) continue;
    const double rmu = rsqrt(mu2);
    const double mu = mu2 * rmu;
    // reflection vector (v0, a[k+1..P)), v0 = al + sign(al) mu; 2 / v.v = rmu / (mu + |al|)
    const double v0 = al + copysign(mu, al);
    const double g = rmu * rcp_newton(mu + fabs(al)), gv = g * v0;
    auto reflect = [&](auto&& top, auto&& col) {
      double w = v0 * top();
#pragma unroll
      for (int p = k + 1; p < P; ++p) w += a[p][k] * col(p);
      const double gw = g * w;
      top() -= gv * w;
#pragma unroll
      for (int p = k + 1; p < P; ++p) col(p) -= gw * a[p][k];
    };
#pragma unroll
    for (int c = k + 1; c < NU; ++c)
      reflect([&]() -> double& { return a[k][c]; }, [&](int p) -> double& { return a[p][c]; });
#pragma unroll
    for (int v = 0; v < 4; ++v)
      reflect([&]() -> double& { return b[k][v]; }, [&](int p) -> double& { return b[p][v]; });
    a[k][k] = -copysign(mu, al);
  }
}

// block_fold: folds P further rows into the triangle (R, z).
template <int NU, int P>
__device__ inline void block_fold(double (&R)[NU][NU], double (&z)[NU][4], double (&a)[P][NU],
                                  double (&b)[P][4]) {
#pragma unroll
  for (int k = 0; k < NU; ++k) {
    double s2 = 0.0;
#pragma unroll
    for (int p = 0; p < P; ++p) s2 += a[p][k] * a[p][k];
    const double al = R[k][k];
    const double mu2 = al * al + s2;
    if (mu2 == 0.0) continue;
    const double rmu = rsqrt(mu2);
    const double mu = mu2 * rmu;
    const double v0 = al + copysign(mu, al);
    const double g = rmu * rcp_newton(mu + fabs(al)), gv = g * v0;
#pragma unroll
    for (int c = k + 1; c < NU; ++c) {
      double w = v0 * R[k][c];
#pragma unroll
      for (int p = 0; p < P; ++p) w += a[p][k] * a[p][c];
      const double gw = g * w;
      R[k][c] -= gv * w;
#pragma unroll
      for (int p = 0; p < P; ++p) a[p][c] -= gw * a[p][k];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double w = v0 * z[k][v];
#pragma unroll
      for (int p = 0; p < P; ++p) w += a[p][k] * b[p][v];
      const double gw = g * w;
      z[k][v] -= gv * w;
#pragma unroll
      for (int p = 0; p < P; ++p) b[p][v] -= gw * a[p][k];
    }
    R[k][k] = -copysign(mu, al);
  }
}

// Rows per block: the first block by block_qr, the others by block_fold.
template <int M>
struct LsBlocks {
  static constexpr int rows = (M + 1) * (M + 2) - 1;
  static constexpr int first = M == 1 ? 5 : M == 2 ? 6 : 10;
  static constexpr int next = M == 1 ? 0 : M == 2 ? 3 : 5;
};

// The triangle (R, z) of all rows; row(c, a, b) delivers rows c = 1, 2, ... in order.
template <int M, class Row>
__device__ inline void ls_triangle(double (&R)[MonoBasis<M>::nu][MonoBasis<M>::nu],
                                   double (&z)[MonoBasis<M>::nu][4], Row&& row) {
  constexpr int nu = MonoBasis<M>::nu;
  using B = LsBlocks<M>;
  {
    double a[B::first][nu], b[B::first][4];
#pragma unroll
    for (int p = 0; p < B::first; ++p) row(1 + p, a[p], b[p]);
    block_qr<nu, B::first>(a, b);
#pragma unroll
    for (int k = 0; k < nu; ++k) {
#pragma unroll
      for (int c = k; c < nu; ++c) R[k][c] = a[k][c];
#pragma unroll
      for (int v = 0; v < 4; ++v) z[k][v] = b[k][v];
    }
  }
  if constexpr (B::next > 0) {
    constexpr int full = (B::rows - B::first) / B::next, rest = (B::rows - B::first) % B::next;
#pragma unroll
    for (int f = 0; f < full; ++f) {
      double a[B::next][nu], b[B::next][4];
#pragma unroll
      for (int p = 0; p < B::next; ++p) row(1 + B::first + f * B::next + p, a[p], b[p]);
      block_fold<nu, B::next>(R, z, a, b);
    }
    if constexpr (rest > 0) {
      double a[rest][nu], b[rest][4];
#pragma unroll
      for (int p = 0; p < rest; ++p) row(1 + B::first + full * B::next + p, a[p], b[p]);
      block_fold<nu, rest>(R, z, a, b);
    }
  }
}

}  // namespace
}  // namespace aw
