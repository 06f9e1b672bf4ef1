// Kernel polynomial method for the density of states (Sec. 4.1 eq. dos_kpm
// and App. B): stochastic Chebyshev moments mu_n = Tr T_n(H~), estimated as
// the mean over R random vectors r of <r|T_n(H~)|r>, and the Jackson-damped
// density rho_KPM(x) = [mu_0 g_0 + 2 sum_{n>=1} mu_n g_n T_n(x)] /
// (pi sqrt(1 - x^2)).
//
// With t_n = T_n(H~) r, moment n of a vector is <r|t_n>.  (Two moments a step
// from <t_n|t_n> and <t_{n+1}|t_n>, by the product rules of the Chebyshev
// polynomials, take half the steps, 0.75 ms instead of 0.96 below, but 2
// <t_n|t_n> - <r|r> doubles the rounding: relative error of t-V chains against
// 80-bit arithmetic 2.2e-16 at L = 12 and 2.8e-16 at L = 16, from <r|t_n>
// 1.1e-16 at both.)  On short chains all vectors go through the resident
// recurrence at once, with the products formed in it: 200 moments of 32 vectors
// at L = 17 take 0.96 ms, with a step and two product launches per moment and
// vector 71.  Elsewhere the recurrence is the fused step kernel (a = 0, written
// over t_{n-1}) followed by a product.
#include <algorithm>
#include <cmath>

#include "internal.hpp"

namespace polfed {

namespace {

constexpr int kKpmCols = 64;       // vectors of one resident launch
constexpr int kDotBlocks = 1024;   // partial sums of a product
constexpr int kDotPartials = 8192; // and of all that wait to be added up

// vector c: uniform on [-sqrt 3, sqrt 3) (zero mean, unit variance), drawn as
// dev_random does from seed + c
__global__ void k_kpm_vectors(int64_t D, int nb, uint64_t seed, double* y) {
  const double w = sqrt(3.0);
  const int64_t n = D * nb;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = e / D, i = e - c * D;
    uint64_t z = seed + (uint64_t)c + 0x9E3779B97F4A7C15ull * (uint64_t)(i + 1);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    y[e] = w * ((double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0);
  }
}

// Sum over a workgroup of 256, valid in thread 0.
__device__ __forceinline__ double sum_256(double a) {
  __shared__ double red[4];
  for (int off = 32; off > 0; off >>= 1) a += __shfl_down(a, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0)
    for (int i = 0; i < 4; ++i) t += red[i];
  return t;
}

// part[block] = sums of x y.
__global__ __launch_bounds__(256) void k_dot_part(int64_t n, const double* __restrict__ x,
                                                  const double* __restrict__ y, double* part) {
  double a = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    a += x[i] * y[i];
  a = sum_256(a);
  if (threadIdx.x == 0) part[blockIdx.x] = a;
}

// out[block] = sum of part[block n .. block n + n)
__global__ __launch_bounds__(256) void k_sum_rows(const double* part, int n, double* out) {
  double a = 0;
  for (int i = threadIdx.x; i < n; i += 256) a += part[(int64_t)blockIdx.x * n + i];
  a = sum_256(a);
  if (threadIdx.x == 0) out[blockIdx.x] = a;
}

void sum_rows(hipStream_t s, const double* part, int n, int count, double* out) {
  hipLaunchKernelGGL(k_sum_rows, dim3((unsigned)count), dim3(256), 0, s, part, n, out);
  HIPC(hipGetLastError());
}

void draw_vectors(hipStream_t s, int64_t D, int nb, uint64_t seed, double* y) {
  const int64_t n = D * nb;
  if (!n) return;
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(8192, (n + 255) / 256));
  hipLaunchKernelGGL(k_kpm_vectors, dim3(g), dim3(256), 0, s, D, nb, seed, y);
  HIPC(hipGetLastError());
}

int dot_blocks(int64_t D) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(kDotBlocks, (D + 1023) / 1024));
}

void dot_part(hipStream_t s, int64_t D, const double* x, const double* y, double* part) {
  hipLaunchKernelGGL(k_dot_part, dim3((unsigned)dot_blocks(D)), dim3(256), 0, s, D, x, y, part);
  HIPC(hipGetLastError());
}

}  // namespace

size_t kpm_workspace(const polfed_op* op, int N, int R) {
  const size_t nd = (size_t)std::max<int64_t>(op->D, 1);
  return (3 * nd + kDotPartials + (size_t)N * R) * sizeof(double);
}

// The buffers of the resident recurrence of cols vectors at a time.
struct ResidentVectors {
  DevBuf v, X, Y, ws, part, d0;
  static size_t bytes(const polfed_op* op, int M, int cols) {
    return ((size_t)3 * op->D * cols + (size_t)cols * (dot_blocks(op->D) + 1)) * sizeof(double) +
           chain_res_moments_bytes(op, M, cols);
  }
  void alloc(const polfed_op* op, int M, int cols, bool draw) {
    const size_t n = (size_t)op->D * cols * sizeof(double);
    X.alloc(n);
    Y.alloc(n);
    ws.alloc(chain_res_moments_bytes(op, M, cols));
    part.alloc((size_t)cols * dot_blocks(op->D) * sizeof(double));
    d0.alloc((size_t)cols * sizeof(double));
    if (draw) v.alloc(n);
  }
};

// How many vectors go through the resident recurrence at a time: all, up to
// 64, or as many as there is room and memory for; 0: none (or not faster).
static int resident_width(hipStream_t s, const polfed_op* op, int M, int R, bool draw, size_t room,
                          ResidentVectors& r) {
  if (M < 4 || op->D < 1) return 0;
  op_tune(s, op, false);  // as the steps of the other way do
  for (int cols = std::min(R, kKpmCols); cols >= 1; cols /= 2) {
    if (ResidentVectors::bytes(op, M, cols) > room) continue;
    if (!chain_res_moments_fit(s, op, cols)) return 0;
    try {
      r.alloc(op, M, cols, draw);
      return cols;
    } catch (const Error& e) {
      if (e.code != POLFED_ERR_OOM) throw;
      r = ResidentVectors{};
    }
  }
  return 0;
}

void kpm_moments(polfed_ctx* ctx, const polfed_op* op, double E_c, double dE, int N, int R,
                 const double* rvecs, uint64_t seed, double* mu, size_t room) {
  REQUIRE(N >= 1 && R >= 1, "kpm: need N >= 1 moments and R >= 1 vectors");
  REQUIRE(dE > 0 && std::isfinite(dE) && std::isfinite(E_c), "kpm: need finite E_c, dE > 0");
  hipStream_t s = ctx->stream;
  const int64_t D = op->D;
  const int M = N - 1;  // steps
  const size_t nd = (size_t)std::max<int64_t>(D, 1);
  const int g = dot_blocks(D);
  // the vectors' moments add up in 80 bits (relative error over eight draws of
  // 32 vectors at L = 17 1.7e-16, in 64 bits 2.0e-16)
  std::vector<long double> acc(N, 0.0L);
  ResidentVectors res;
  const int cols = resident_width(s, op, M, R, !rvecs, room, res);
  if (cols > 0) {
    std::vector<double> dots((size_t)M * cols + 1), h0((size_t)cols);
    for (int c0 = 0; c0 < R; c0 += cols) {
      const int nb = std::min(cols, R - c0);
      const double* vc = rvecs ? rvecs + (size_t)c0 * D : res.v.as<double>();
      if (!rvecs) draw_vectors(s, D, nb, seed + (uint64_t)c0, res.v.as<double>());
      for (int c = 0; c < nb; ++c)
        dot_part(s, D, vc + (size_t)c * D, vc + (size_t)c * D,
                 res.part.as<double>() + (size_t)c * g);
      sum_rows(s, res.part.as<double>(), g, nb, res.d0.as<double>());
      HIPC(hipMemcpyAsync(h0.data(), res.d0.get(), (size_t)nb * sizeof(double), hipMemcpyDeviceToHost,
                          s));
      chain_res_moments(s, op, E_c, dE, M, cols, nb, vc, res.X.as<double>(), res.Y.as<double>(),
                        res.ws, dots.data());
      for (int c = 0; c < nb; ++c) {
        acc[0] += h0[c];
        for (int n = 1; n < N; ++n) acc[n] += dots[(size_t)(n - 1) * nb + c];
      }
    }
  } else {
    DevBuf r, ta(nd * sizeof(double)), tb(nd * sizeof(double)),
        part(kDotPartials * sizeof(double)), sums((size_t)N * R * sizeof(double));
    if (!rvecs) r.alloc(nd * sizeof(double));
    for (int c = 0; c < R; ++c) {
      const double* rv = rvecs ? rvecs + (size_t)c * D : r.as<double>();
      if (!rvecs) draw_vectors(s, D, 1, seed + (uint64_t)c, r.as<double>());
      // the products of as many moments as there is room for partial sums
      double* out = sums.as<double>() + (size_t)c * N;
      int have = 0;
      auto product = [&](const double* t) {
        dot_part(s, D, rv, t, part.as<double>() + (size_t)have * g);
        if (++have < kDotPartials / g) return;
        sum_rows(s, part.as<double>(), g, have, out);
        out += have;
        have = 0;
      };
      product(rv);
      // cur = t_n, prev = t_{n-1} (overwritten; t_0 is r itself, so the first
      // update writes to tb)
      const double* cur = rv;
      const double* prev = nullptr;
      for (int n = 1; n <= M; ++n) {
        const double f = n == 1 ? 1.0 : 2.0;
        double* nxt = n == 1 ? ta.as<double>()
                             : (prev == rv ? tb.as<double>() : const_cast<double*>(prev));
        op_step<double>(s, op, f / dE, -f * E_c / dE, 0.0, nullptr, cur, prev, nxt);
        product(nxt);
        prev = cur;
        cur = nxt;
      }
      if (have) sum_rows(s, part.as<double>(), g, have, out);
    }
    std::vector<double> h((size_t)N * R);
    HIPC(hipMemcpyAsync(h.data(), sums.get(), h.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    HIPC(hipStreamSynchronize(s));
    for (int c = 0; c < R; ++c)
      for (int n = 0; n < N; ++n) acc[n] += h[(size_t)c * N + n];
  }
  for (int n = 0; n < N; ++n) mu[n] = (double)(acc[n] / R);
}

// Jackson factors g_n for N moments (App. B eq. kernels_jackson_and_lorenz).
static double jackson(int n, int N) {
  const double a = M_PI / (N + 1);
  return ((N - n + 1) * std::cos(a * n) + std::sin(a * n) / std::tan(a)) / (N + 1);
}

void kpm_density(const double* mu, int N, const double* x, int nx, double* rho) {
  REQUIRE(N >= 1, "kpm: need N >= 1 moments");
  std::vector<double> c(N);
  for (int n = 0; n < N; ++n) c[n] = (n == 0 ? 1.0 : 2.0) * mu[n] * jackson(n, N);
  for (int j = 0; j < nx; ++j) {
    const double t = x[j];
    REQUIRE(t > -1.0 && t < 1.0, "kpm: evaluation points must lie in (-1, 1)");
    // sum_n c_n T_n(t) by Clenshaw's recurrence
    double b1 = 0, b2 = 0;
    for (int n = N - 1; n >= 1; --n) {
      const double b = c[n] + 2.0 * t * b1 - b2;
      b2 = b1;
      b1 = b;
    }
    const double sum = c[0] + t * b1 - b2;
    rho[j] = sum / (M_PI * std::sqrt(1.0 - t * t));
  }
}

double kpm_maxdos(const double* mu, int N, double lo, double hi) {
  constexpr int kGrid = 4096;
  std::vector<double> x;
  for (int j = 0; j < kGrid; ++j) {
    const double t = std::cos(M_PI * (j + 0.5) / kGrid);
    if (t >= lo && t <= hi) x.push_back(t);
  }
  REQUIRE(!x.empty(), "kpm: empty search interval");
  std::vector<double> rho(x.size());
  kpm_density(mu, N, x.data(), (int)x.size(), rho.data());
  return x[std::max_element(rho.begin(), rho.end()) - rho.begin()];
}

}  // namespace polfed
