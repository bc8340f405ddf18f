// Host FP64 dense linear algebra (no HIP dependency).
#pragma once
#include <cmath>
#include <cstdint>

namespace thc {
int host_cholesky(int64_t n, double* A);                     // lower factor in place; 0 on success
void host_tri_inverse_lower(int64_t n, const double* L, double* Linv);
int host_syev(int64_t n, double* A, double* w);              // eigenvectors in the columns of A

// sqrt(f^2 + g^2) without overflow or harmful underflow
inline double ql_norm(double f, double g) {
  const double t = f * f + g * g;
  return t > 1e-280 && t < 1e280 ? std::sqrt(t) : std::hypot(f, g);
}

// Implicit QL iteration with Wilkinson-type shifts on the symmetric tridiagonal (d, e), e[i] coupling i
// and i + 1 (Golub & Van Loan, Matrix Computations, Sec. 8.3): d becomes the eigenvalues, unsorted.
// The step sequence (shift from the leading 2 x 2 block, rotations chased up the tridiagonal) is the
// published tql2 procedure of Bowdler, Martin, Reinsch & Wilkinson (Numer. Math. 11, 293-306, 1968).
// Its plane rotations combine columns i, i + 1 of the eigenvector matrix (z_i <- c z_i - s z_i+1,
// z_i+1 <- s z_i + c z_i+1) and go to the sink in order: sink.sweep(l, m) before a sweep over
// i = m - 1 .. l, then sink.rotate(i, c, s).  Returns 0, 2 without convergence, or the sink's code.
template <class Sink>
int ql_iterate(int64_t n, double* d, double* e, Sink& sink) {
  for (int64_t l = 0; l < n; ++l) {
    int iter = 0;
    for (;;) {
      int64_t m = l;
      for (; m + 1 < n; ++m) {
        const double dd = std::fabs(d[m]) + std::fabs(d[m + 1]);
        if (std::fabs(e[m]) <= 1e-16 * dd) break;
      }
      if (m == l) break;
      if (++iter > 80) return 2;
      const int rc = sink.sweep(l, m);
      if (rc != 0) return rc;
      double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
      double r = ql_norm(g, 1.0);
      g = d[m] - d[l] + e[l] / (g + (g >= 0 ? r : -r));
      double s = 1.0, c = 1.0, pp = 0.0;
      bool underflow = false;
      for (int64_t i = m - 1; i >= l; --i) {
        const double f = s * e[i];
        const double b = c * e[i];
        r = ql_norm(f, g);
        e[i + 1] = r;
        if (r == 0.0) {
          d[i + 1] -= pp;
          e[m] = 0.0;
          underflow = true;
          break;
        }
        s = f / r;
        c = g / r;
        g = d[i + 1] - pp;
        r = (d[i] - g) * s + 2.0 * c * b;
        pp = s * r;
        d[i + 1] = g + pp;
        g = c * r - b;
        sink.rotate(i, c, s);
      }
      if (underflow) continue;
      d[l] -= pp;
      e[l] = g;
      e[m] = 0.0;
    }
  }
  return 0;
}
}  // namespace thc
