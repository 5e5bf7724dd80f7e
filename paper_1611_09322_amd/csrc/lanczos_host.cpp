// Host FP64 tridiagonal square root for the full-mobility Krylov sample
// (Sec. II B.1 applies the same Lanczos process to M_r; Sec. III compares
// with it on the whole mobility, where the basis grows past what one
// wavefront's registers hold).
#include <cmath>
#include <vector>

#include "pse_internal.hpp"

namespace pse {

// s = T^{1/2} e_1 for the m x m symmetric tridiagonal T with diagonal d and
// off-diagonal e (e[i] couples i and i + 1), through its eigendecomposition
// T = Q diag(lambda) Q^T by implicit QL with shifts (Q accumulated; negative
// eigenvalues from rounding are taken as 0).  false if an eigenvalue does
// not converge in 60 sweeps.
bool tridiag_sqrt_e1_host(int m, const double *dd, const double *ee, double *s) {
  std::vector<double> d(dd, dd + m), e(m, 0.0), Q((size_t)m * m, 0.0);
  for (int i = 0; i + 1 < m; ++i) e[i] = ee[i];
  for (int i = 0; i < m; ++i) Q[(size_t)i * m + i] = 1.0;  // Q[row k][col j] at k m + j
  const double eps = 2.2e-16;
  for (int l = 0; l < m; ++l) {
    int iter = 0;
    while (true) {
      int mm = l;
      for (; mm < m - 1; ++mm) {
        const double sc = std::fabs(d[mm]) + std::fabs(d[mm + 1]);
        if (std::fabs(e[mm]) <= eps * sc) break;
      }
      if (mm == l) break;
      if (++iter > 60) return false;
      double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
      double r = std::hypot(g, 1.0);
      g = d[mm] - d[l] + e[l] / (g + std::copysign(r, g));
      double sn = 1.0, cs = 1.0, p = 0.0;
      bool deflated = false;
      for (int i = mm - 1; i >= l; --i) {
        const double f = sn * e[i], b = cs * e[i];
        r = std::hypot(f, g);
        e[i + 1] = r;
        if (r == 0.0) {
          d[i + 1] -= p;
          e[mm] = 0.0;
          deflated = true;
          break;
        }
        sn = f / r;
        cs = g / r;
        g = d[i + 1] - p;
        r = (d[i] - g) * sn + 2.0 * cs * b;
        p = sn * r;
        d[i + 1] = g + p;
        g = cs * r - b;
        for (int k = 0; k < m; ++k) {
          double *row = &Q[(size_t)k * m];
          const double q1 = row[i + 1], q0 = row[i];
          row[i + 1] = sn * q0 + cs * q1;
          row[i] = cs * q0 - sn * q1;
        }
      }
      if (deflated) continue;
      d[l] -= p;
      e[l] = g;
      e[mm] = 0.0;
    }
  }
  for (int k = 0; k < m; ++k) {
    double acc = 0.0;
    for (int j = 0; j < m; ++j) acc += Q[(size_t)k * m + j] * std::sqrt(d[j] > 0.0 ? d[j] : 0.0) * Q[j];
    s[k] = acc;
  }
  return true;
}

// Quadrature of the square root (Hale, Higham and Trefethen, "Computing A^alpha,
// log(A), and related matrix functions by contour integrals", SIAM J. Numer.
// Anal. 46, 2008, method 3): lambda^{1/2} = (2 / pi) int_0^inf lambda / (lambda + s^2) ds
// with s = k sc(u | 1 - k^2), u in (0, K'), by the midpoint rule in u, whose
// error decays as exp(-2 pi^2 N / (log(1 / k^2) + 3)): at N = 64 nodes and
// k^2 = 1e-13 it is below 2e-15 for every lambda in [k^2, 1].  sc is evaluated
// from sinh by descending Landen steps on the small modulus k (imaginary
// argument), which loses no digits near u = K'.
void lz_quadrature(double2 *tw) {
  const double k2 = kRootLow, k = std::sqrt(k2), pi = 3.14159265358979323846;
  double a = 1.0, b = k;
  for (int i = 0; i < 12; ++i) {  // arithmetic-geometric mean of 1 and k
    const double t = 0.5 * (a + b);
    b = std::sqrt(a * b);
    a = t;
  }
  const double Kp = pi / (2.0 * a);
  double ks[3], q = k2;
  for (double &x : ks) {
    const double kp = std::sqrt(1.0 - q);
    x = q / ((1.0 + kp) * (1.0 + kp));
    q = x * x;
  }
  for (int j = 0; j < kRootNodes; ++j) {
    double v = (j + 0.5) * Kp / kRootNodes;
    for (double x : ks) v /= 1.0 + x;
    double s = std::sinh(v);
    for (int i = 2; i >= 0; --i) s = (1.0 + ks[i]) * s / (1.0 - ks[i] * s * s);
    tw[j].x = k2 * s * s;
    tw[j].y = 2.0 * Kp * k / (pi * kRootNodes) * std::sqrt((1.0 + k2 * s * s) * (1.0 + s * s));
  }
}

}  // namespace pse
