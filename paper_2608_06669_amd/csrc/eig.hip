// Explicitly shifted QR iteration in complex arithmetic (Golub & Van Loan,
// Matrix Computations, the shifted QR algorithm on Hessenberg matrices):
// on the active unreduced block, A - mu I = QR by Givens rotations and
// A <- RQ + mu I, with the Wilkinson shift (the eigenvalue of the trailing
// 2 x 2 block nearer its last diagonal entry) and an occasional ad hoc
// shift against cycling; a subdiagonal entry below eps times its diagonal
// neighbours is set to zero and the block splits. Complex arithmetic lets
// the conjugate pairs of a real matrix come out one at a time.
#include "eig.hpp"

#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdint>
#include <limits>
#include <vector>

namespace pnk {

bool hessenberg_eigenvalues(const double* H, int m, double* re, double* im) {
  using C = std::complex<double>;
  if (m <= 0) return true;
  std::vector<C> a((size_t)m * m);
  double anorm = 0.0;
  for (int i = 0; i < m; ++i)
    for (int j = 0; j < m; ++j) {
      const double x = j >= i - 1 ? H[(size_t)i * m + j] : 0.0;
      a[(size_t)i * m + j] = x;
      anorm += std::fabs(x);
    }
  auto A = [&](int i, int j) -> C& { return a[(size_t)i * m + j]; };
  std::vector<C> eig(m), cs(m), sn(m);
  const double eps = std::numeric_limits<double>::epsilon();
  int hi = m - 1, iter = 0;
  while (hi >= 0) {
    // the unreduced block [lo, hi]
    int lo = hi;
    while (lo > 0) {
      double s = std::abs(A(lo, lo)) + std::abs(A(lo - 1, lo - 1));
      if (s == 0.0) s = anorm;
      if (std::abs(A(lo, lo - 1)) <= eps * s) {
        A(lo, lo - 1) = 0.0;
        break;
      }
      --lo;
    }
    if (lo == hi) {
      eig[hi] = A(hi, hi);
      --hi;
      iter = 0;
      continue;
    }
    if (++iter > 60 * m + 100) return false;
    const C p = A(hi - 1, hi - 1), q = A(hi - 1, hi), r = A(hi, hi - 1), d = A(hi, hi);
    const C half = 0.5 * (p + d);
    const C disc = std::sqrt(half * half - (p * d - q * r));
    const C l1 = half + disc, l2 = half - disc;
    C mu = std::abs(l1 - d) < std::abs(l2 - d) ? l1 : l2;
    if (iter % 11 == 10) mu = d + 0.75 * std::abs(r);  // ad hoc shift
    for (int k = lo; k <= hi; ++k) A(k, k) -= mu;
    // A - mu I = Q R: G_k = [conj(c) conj(s); -s c] zeroes the subdiagonal
    for (int k = lo; k < hi; ++k) {
      const C x = A(k, k), y = A(k + 1, k);
      const double rr = std::hypot(std::abs(x), std::abs(y));
      const C c = rr == 0.0 ? C(1.0) : x / rr, s = rr == 0.0 ? C(0.0) : y / rr;
      for (int j = k; j <= hi; ++j) {
        const C u = A(k, j), v = A(k + 1, j);
        A(k, j) = std::conj(c) * u + std::conj(s) * v;
        A(k + 1, j) = -s * u + c * v;
      }
      cs[k] = c;
      sn[k] = s;
    }
    // R Q: the adjoints from the right, in order
    for (int k = lo; k < hi; ++k) {
      const C c = cs[k], s = sn[k];
      for (int i = lo; i <= std::min(k + 1, hi); ++i) {
        const C u = A(i, k), v = A(i, k + 1);
        A(i, k) = u * c + v * s;
        A(i, k + 1) = -u * std::conj(s) + v * std::conj(c);
      }
    }
    for (int k = lo; k <= hi; ++k) A(k, k) += mu;
  }
  for (int i = 0; i < m; ++i) {
    re[i] = eig[i].real();
    im[i] = eig[i].imag();
  }
  return true;
}

// Householder tridiagonalisation and the implicit QR step with Wilkinson
// shift (Golub & Van Loan, Matrix Computations, the symmetric QR algorithm).
// The transformations are applied to rows, so the inner loops are
// contiguous: about 3 n^3 flops for the reduction with its vectors and 5 n^3
// for the QR steps (0.8 ms of one core beside the card at n = 90, 5 ms at 180).
bool symmetric_eigen(const double* F, int n, double* eps, double* ut, bool* diagonal) {
  std::vector<double> a((size_t)n * n), vs((size_t)n * n, 0.0), beta(n, 0.0), e(n, 0.0), w(n);
  bool diag = true;
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) {
      const double x = 0.5 * (F[(size_t)i * n + j] + F[(size_t)j * n + i]);
      if (!std::isfinite(x)) return false;
      if (i != j && x != 0.0) diag = false;
      a[(size_t)i * n + j] = x;
    }
  *diagonal = diag;
  std::fill(ut, ut + (size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i) ut[(size_t)i * n + i] = 1.0;
  if (diag) {
    for (int i = 0; i < n; ++i) eps[i] = a[(size_t)i * n + i];
    return true;
  }
  // step k reflects rows and columns k + 1 .. n - 1 so that column k keeps one
  // entry below the diagonal: H = I - beta v v^T, v in row k of vs
  for (int k = 0; k + 2 < n; ++k) {
    double* v = &vs[(size_t)k * n];
    double tail = 0.0;
    for (int i = k + 2; i < n; ++i) tail = std::max(tail, std::fabs(a[(size_t)k * n + i]));
    e[k] = a[(size_t)k * n + k + 1];
    if (tail == 0.0) continue;
    const double scale = std::max(tail, std::fabs(e[k]));
    double nrm = 0.0;
    for (int i = k + 1; i < n; ++i) {
      v[i] = a[(size_t)k * n + i] / scale;
      nrm += v[i] * v[i];
    }
    nrm = std::sqrt(nrm);
    const double alpha = v[k + 1] > 0.0 ? -nrm : nrm;  // the entry that is kept
    v[k + 1] -= alpha;
    beta[k] = 1.0 / (nrm * (nrm + std::fabs(v[k + 1] + alpha)));
    e[k] = alpha * scale;
    // p = beta A v, w = p - (beta v.p / 2) v, A -= v w^T + w v^T
    double vp = 0.0;
    for (int i = k + 1; i < n; ++i) {
      const double* row = &a[(size_t)i * n];
      double t = 0.0;
      for (int j = k + 1; j < n; ++j) t += row[j] * v[j];
      w[i] = beta[k] * t;
      vp += v[i] * w[i];
    }
    const double h = 0.5 * beta[k] * vp;
    for (int i = k + 1; i < n; ++i) w[i] -= h * v[i];
    for (int i = k + 1; i < n; ++i) {
      double* row = &a[(size_t)i * n];
      const double vi = v[i], wi = w[i];
      for (int j = k + 1; j < n; ++j) row[j] -= vi * w[j] + wi * v[j];
    }
  }
  if (n >= 2) e[n - 2] = a[(size_t)(n - 2) * n + n - 1];
  for (int i = 0; i < n; ++i) eps[i] = a[(size_t)i * n + i];
  // F = Q T Q^T, Q = H_0 H_1 ..., accumulated from the last reflection (on
  // the rows of Q), then stored as its transpose
  {
    std::vector<double> q((size_t)n * n, 0.0);
    for (int i = 0; i < n; ++i) q[(size_t)i * n + i] = 1.0;
    for (int k = n - 3; k >= 0; --k) {
      if (beta[k] == 0.0) continue;
      const double* v = &vs[(size_t)k * n];
      std::fill(w.begin(), w.end(), 0.0);
      for (int i = k + 1; i < n; ++i) {
        const double* row = &q[(size_t)i * n];
        const double t = beta[k] * v[i];
        for (int j = k + 1; j < n; ++j) w[j] += t * row[j];
      }
      for (int i = k + 1; i < n; ++i) {
        double* row = &q[(size_t)i * n];
        const double t = v[i];
        for (int j = k + 1; j < n; ++j) row[j] -= t * w[j];
      }
    }
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) ut[(size_t)j * n + i] = q[(size_t)i * n + j];
  }
  const double tiny = std::numeric_limits<double>::epsilon();
  int hi = n - 1;
  for (int64_t sweeps = 0; hi > 0;) {
    if (std::fabs(e[hi - 1]) <= tiny * (std::fabs(eps[hi - 1]) + std::fabs(eps[hi]))) {
      e[hi - 1] = 0.0;
      --hi;
      continue;
    }
    if (++sweeps > 60 * (int64_t)n) return false;
    int lo = hi - 1;
    while (lo > 0 && std::fabs(e[lo - 1]) > tiny * (std::fabs(eps[lo - 1]) + std::fabs(eps[lo]))) --lo;
    // the eigenvalue of the trailing 2 x 2 block nearer its last entry
    const double dd = 0.5 * (eps[hi - 1] - eps[hi]), eb = e[hi - 1];
    const double root = std::hypot(dd, eb);
    const double mu = eps[hi] - eb * (eb / (dd + (dd >= 0.0 ? root : -root)));
    double x = eps[lo] - mu, z = e[lo];
    for (int k = lo; k < hi; ++k) {
      const double r = std::hypot(x, z);
      const double c = r != 0.0 ? x / r : 1.0, s = r != 0.0 ? z / r : 0.0;
      if (k > lo) e[k - 1] = r;
      const double d1 = eps[k], d2 = eps[k + 1], ek = e[k];
      const double cc = c * c, ss = s * s, cs = c * s;
      eps[k] = cc * d1 + 2.0 * cs * ek + ss * d2;
      eps[k + 1] = ss * d1 - 2.0 * cs * ek + cc * d2;
      e[k] = cs * (d2 - d1) + (cc - ss) * ek;
      if (k + 1 < hi) {
        x = e[k];
        z = s * e[k + 1];
        e[k + 1] *= c;
      }
      double* __restrict__ q0 = ut + (size_t)k * n;
      double* __restrict__ q1 = ut + (size_t)(k + 1) * n;
      for (int j = 0; j < n; ++j) {
        const double y0 = q0[j], y1 = q1[j];
        q0[j] = c * y0 + s * y1;
        q1[j] = c * y1 - s * y0;
      }
    }
  }
  return true;
}

}  // namespace pnk
