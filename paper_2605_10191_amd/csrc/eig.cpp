// Host eigensolvers for the Lanczos matrix and the Rayleigh-Ritz
// projection.  Symmetric tridiagonal: the implicit QL algorithm with
// Wilkinson-type shifts (Dubrulle, Martin and Wilkinson, Numer. Math. 12,
// 1968, the procedure known as imtql2).  Dense symmetric: Householder
// reduction to tridiagonal form (Golub and Van Loan, Sec. 8.3) followed by
// the tridiagonal solver.  Both run in O(n^3).
//
// The rows of the eigenvector matrix are independent of each other, but the
// work on one row is a chain (every rotation and every sum needs the one
// before), which a core runs at the latency of its additions.  They are
// therefore kept in panels of 16 rows, the 16 values of a column side by
// side, and go through the same operations in the same order together: the
// same bits, at n = 120 in 2.9 ms instead of 9.3 and at n = 240 in 15 instead
// of 69, of which the rotations' own scalar chain is 0.9 and 3.  Panels are
// shared among the host's threads with OpenMP once n reaches the thousands
// that thousands of wanted pairs bring (about 3,000 Lanczos vectors for 1,500
// pairs).
#include <algorithm>
#include <cmath>
#include <numeric>
#include <stdexcept>

#include "eig.hpp"

namespace polfed {

namespace {

// Rows updated per thread below which a loop stays serial.
constexpr long kParWork = 1L << 16;

// nz x n values in panels of kP rows: row k, column i at
// panel(k / kP)[i * kP + k % kP]; rows past nz are zero.
constexpr int kP = 16;
struct Panels {
  int n = 0, nz = 0, np = 0;
  std::vector<double> x;
  void init(int n_, int nz_) {
    n = n_;
    nz = nz_;
    np = (nz + kP - 1) / kP;
    x.assign((size_t)np * n * kP, 0.0);
  }
  double* panel(int p) { return x.data() + (size_t)p * n * kP; }
  double& at(int k, int i) { return x[((size_t)(k / kP) * n + i) * kP + k % kP]; }
};

// The kernels on panels, for the vector units of the machine it runs on (AVX2
// without FMA: the operations, and so the bits, are those of the base set).
#define POLFED_SIMD __attribute__((target_clones("avx2", "default")))

POLFED_SIMD void sweep_panel(double* __restrict__ z, int i_hi, int i_lo,
                             const double* __restrict__ cs, const double* __restrict__ sn) {
  double f[kP];  // z_{i+1} on its way down
  for (int k = 0; k < kP; ++k) f[k] = z[(size_t)(i_hi + 1) * kP + k];
  for (int i = i_hi; i >= i_lo; --i) {
    const double c = cs[i], s = sn[i];
    double* zi = z + (size_t)i * kP;
#pragma omp simd
    for (int k = 0; k < kP; ++k) {
      const double x = zi[k], y = f[k];
      zi[kP + k] = s * x + c * y;
      f[k] = c * x - s * y;
    }
  }
  for (int k = 0; k < kP; ++k) z[(size_t)i_lo * kP + k] = f[k];
}

// qr (m columns of a panel) <- qr (I - beta v v^T)
POLFED_SIMD void reflect_panel(double* __restrict__ qr, int m, const double* __restrict__ v,
                               double beta) {
  double t[kP] = {0};
  for (int j = 0; j < m; ++j) {
    const double vj = v[j];
#pragma omp simd
    for (int r = 0; r < kP; ++r) t[r] += qr[(size_t)j * kP + r] * vj;
  }
  for (int r = 0; r < kP; ++r) t[r] *= beta;
  for (int j = 0; j < m; ++j) {
    const double vj = v[j];
#pragma omp simd
    for (int r = 0; r < kP; ++r) qr[(size_t)j * kP + r] -= t[r] * vj;
  }
}

// p[0..len) = beta sum_j v_j a_j[0..len), len <= kChunk, rows of stride n
constexpr int kChunk = 32;
POLFED_SIMD void product_chunk(const double* __restrict__ a, int n, int m, int len,
                               const double* __restrict__ v, double beta,
                               double* __restrict__ p) {
  double t[kChunk] = {0};
  if (len == kChunk) {
    for (int j = 0; j < m; ++j) {
      const double vj = v[j];
      const double* row = a + (size_t)j * n;
#pragma omp simd
      for (int i = 0; i < kChunk; ++i) t[i] += row[i] * vj;
    }
  } else {
    for (int j = 0; j < m; ++j) {
      const double vj = v[j];
      const double* row = a + (size_t)j * n;
      for (int i = 0; i < len; ++i) t[i] += row[i] * vj;
    }
  }
  for (int i = 0; i < len; ++i) p[i] = beta * t[i];
}

// row -= vi q + qi v
POLFED_SIMD void update_row(double* __restrict__ row, int m, double vi,
                            const double* __restrict__ q, double qi,
                            const double* __restrict__ v) {
#pragma omp simd
  for (int j = 0; j < m; ++j) row[j] -= vi * q[j] + qi * v[j];
}

// Applies the rotations of one QL sweep, recorded for i = i_hi down to
// i_lo, to every row of Z: (z_i, z_{i+1}) <- (c z_i - s z_{i+1}, s z_i + c z_{i+1}).
void apply_sweep(Panels& Z, int i_hi, int i_lo, const std::vector<double>& cs,
                 const std::vector<double>& sn) {
  if (i_hi < i_lo) return;
  if (Z.nz == 1) {  // last components only: one chain
    double* z = Z.x.data();
    for (int i = i_hi; i >= i_lo; --i) {
      const double c = cs[i], s = sn[i], zf = z[(i + 1) * kP], zi = z[i * kP];
      z[(i + 1) * kP] = s * zi + c * zf;
      z[i * kP] = c * zi - s * zf;
    }
    return;
  }
  const long work = (long)Z.nz * (i_hi - i_lo + 1);
#pragma omp parallel for schedule(static) if (work > kParWork)
  for (int p = 0; p < Z.np; ++p) sweep_panel(Z.panel(p), i_hi, i_lo, cs.data(), sn.data());
}

// Implicit QL on d, e (see tridiag_eig); returns the ascending order.
std::vector<int> implicit_ql(int n, std::vector<double>& d, std::vector<double>& e, Panels& Z) {
  e.resize(n, 0.0);
  e[n - 1] = 0.0;
  const double eps = 2.220446049250313e-16;
  std::vector<double> cs(n), sn(n);
  for (int l = 0; l < n; ++l) {
    int iter = 0;
    for (;;) {
      int m = l;
      for (; m < n - 1; ++m) {
        const double dd = std::fabs(d[m]) + std::fabs(d[m + 1]);
        if (std::fabs(e[m]) <= eps * dd) break;
      }
      if (m == l) break;
      if (++iter > 200) throw std::runtime_error("tridiagonal QL did not converge");
      // shift from the leading 2x2 block
      double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
      double r = std::hypot(g, 1.0);
      g = d[m] - d[l] + e[l] / (g + (g >= 0 ? r : -r));
      double s = 1.0, c = 1.0, p = 0.0;
      int i = m - 1;
      bool deflated = false;
      for (; i >= l; --i) {
        const double f = s * e[i], b = c * e[i];
        r = std::hypot(f, g);
        e[i + 1] = r;
        if (r == 0.0) {  // underflow: split and restart
          d[i + 1] -= p;
          e[m] = 0.0;
          deflated = true;
          break;
        }
        s = f / r;
        c = g / r;
        g = d[i + 1] - p;
        r = (d[i] - g) * s + 2.0 * c * b;
        p = s * r;
        d[i + 1] = g + p;
        g = c * r - b;
        cs[i] = c;
        sn[i] = s;
      }
      // the rotations of this sweep: i = m - 1 down to the last one done
      apply_sweep(Z, m - 1, deflated ? i + 1 : l, cs, sn);
      if (deflated) continue;
      d[l] -= p;
      e[l] = g;
      e[m] = 0.0;
    }
  }
  std::vector<int> idx(n);
  std::iota(idx.begin(), idx.end(), 0);
  std::stable_sort(idx.begin(), idx.end(), [&](int a, int b) { return d[a] < d[b]; });
  std::vector<double> d2(n);
  for (int j = 0; j < n; ++j) d2[j] = d[idx[j]];
  d.swap(d2);
  return idx;
}

// Householder reduction of the symmetric row-major a to tridiagonal form,
// a = Q T Q^T; Q keeps only its rows q0..n-1 ((n - q0) x n), which start as
// the matching rows of the identity.
void tridiagonalize(int n, std::vector<double>& a, Panels& Q, int q0, std::vector<double>& d,
                    std::vector<double>& e) {
  const int nq = n - q0;
  Q.init(n, nq);
  for (int i = 0; i < nq; ++i) Q.at(i, q0 + i) = 1.0;
  std::vector<double> v(n), p(n), q(n);
  for (int k = 0; k + 2 < n; ++k) {
    const int m = n - k - 1;  // length of the column below the diagonal
    double xn = 0;
    for (int i = 0; i < m; ++i) xn += a[(size_t)(k + 1 + i) * n + k] * a[(size_t)(k + 1 + i) * n + k];
    xn = std::sqrt(xn);
    if (xn == 0.0) continue;
    const double x0 = a[(size_t)(k + 1) * n + k];
    const double alpha = x0 >= 0 ? -xn : xn;
    for (int i = 0; i < m; ++i) v[i] = a[(size_t)(k + 1 + i) * n + k];
    v[0] -= alpha;
    double vv = 0;
    for (int i = 0; i < m; ++i) vv += v[i] * v[i];
    if (vv == 0.0) continue;
    const double beta = 2.0 / vv;
    // p = beta * A_sub v, by rows of the symmetric A_sub: p += v_j A_j, so
    // that the sums of a chunk of p run side by side
    const bool par = (long)m * m > kParWork;
#pragma omp parallel for schedule(static) if (par)
    for (int i0 = 0; i0 < m; i0 += kChunk)
      product_chunk(&a[(size_t)(k + 1) * n + (k + 1) + i0], n, m, std::min(kChunk, m - i0),
                    v.data(), beta, &p[i0]);
    double vp = 0;
    for (int i = 0; i < m; ++i) vp += v[i] * p[i];
    const double Kc = 0.5 * beta * vp;
    for (int i = 0; i < m; ++i) q[i] = p[i] - Kc * v[i];
#pragma omp parallel for schedule(static) if (par)
    for (int i = 0; i < m; ++i)
      update_row(&a[(size_t)(k + 1 + i) * n + (k + 1)], m, v[i], q.data(), q[i], v.data());
    a[(size_t)(k + 1) * n + k] = alpha;
    a[(size_t)k * n + (k + 1)] = alpha;
    for (int i = 1; i < m; ++i) {
      a[(size_t)(k + 1 + i) * n + k] = 0.0;
      a[(size_t)k * n + (k + 1 + i)] = 0.0;
    }
    // Q <- Q H on columns k+1..n-1
#pragma omp parallel for schedule(static) if ((long)nq * m > kParWork)
    for (int g = 0; g < Q.np; ++g)
      reflect_panel(Q.panel(g) + (size_t)(k + 1) * kP, m, v.data(), beta);
  }
  d.assign(n, 0.0);
  e.assign(n > 1 ? n - 1 : 0, 0.0);
  for (int i = 0; i < n; ++i) d[i] = a[(size_t)i * n + i];
  for (int i = 0; i + 1 < n; ++i) e[i] = a[(size_t)(i + 1) * n + i];
}

std::vector<double> symmetric_copy(int n, const std::vector<double>& A) {
  std::vector<double> a((size_t)n * n);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j)
      a[(size_t)i * n + j] = 0.5 * (A[(size_t)i * n + j] + A[(size_t)j * n + i]);
  return a;
}

}  // namespace

void tridiag_eig(int n, std::vector<double>& d, std::vector<double> e, std::vector<double>& Z,
                 int nz) {
  if (n <= 0) return;
  Panels P;
  P.init(n, nz);
  for (int k = 0; k < nz; ++k)
    for (int i = 0; i < n; ++i) P.at(k, i) = Z[(size_t)k * n + i];
  const std::vector<int> idx = implicit_ql(n, d, e, P);
  for (int k = 0; k < nz; ++k)
    for (int j = 0; j < n; ++j) Z[(size_t)k * n + j] = P.at(k, idx[j]);
}

void sym_eig(int n, std::vector<double>& A, std::vector<double>& w,
             std::vector<double>& Zout) {
  // Work row-major on a symmetric copy (A is col-major; symmetric anyway).
  std::vector<double> a = symmetric_copy(n, A), d, e;
  Panels Q;  // rows: components, columns: eigenvectors
  tridiagonalize(n, a, Q, 0, d, e);
  const std::vector<int> idx = implicit_ql(n, d, e, Q);
  w = d;
  Zout.assign((size_t)n * n, 0.0);
  for (int j = 0; j < n; ++j)
    for (int i = 0; i < n; ++i) Zout[(size_t)j * n + i] = Q.at(i, idx[j]);
}

void sym_eig_tail(int n, const std::vector<double>& A, int r, std::vector<double>& w,
                  std::vector<double>& Ztail) {
  std::vector<double> a = symmetric_copy(n, A), d, e;
  r = std::min(std::max(r, 1), n);
  Panels Q;
  tridiagonalize(n, a, Q, n - r, d, e);
  const std::vector<int> idx = implicit_ql(n, d, e, Q);
  w = d;
  Ztail.assign((size_t)r * n, 0.0);
  for (int i = 0; i < r; ++i)
    for (int j = 0; j < n; ++j) Ztail[(size_t)i * n + j] = Q.at(i, idx[j]);
}

}  // namespace polfed
