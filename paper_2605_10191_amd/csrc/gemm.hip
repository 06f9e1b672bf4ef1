// FP64 products of tall matrices on the matrix cores (v_mfma_f64_16x16x4f64).
//
// The extraction of Sec. 4.3 forms u_i = V t_i for the selected Ritz vectors
// (a D x m basis times an m x n coefficient block), the projection of H on
// their span (an n x n product with inner dimension D) and the rotations of
// the Rayleigh-Ritz step; a block Gram-Schmidt pass of Sec. 2.2 forms
// C = V^T W and W -= V C.  All are dense FP64 contractions with one very
// long dimension D, so they run as output tiles of 64 x 64 (128 x 128 where the
// output is wide enough, see there) on the MFMA units:
//   - nn:  C (D x n) = A (D x m) B (m x n), or C -= A B; one workgroup per
//          64 x 64 tile of C, the inner dimension m in chunks of 32 staged
//          in LDS;
//   - tn:  G (n1 x n2) = A^T B with A (D x n1), B (D x n2); the long inner
//          dimension D is split over workgroups (at least 256 rows each),
//          whose partial tiles are summed in a fixed order by a second
//          kernel, so the result does not depend on timing.
// Each of the four waves of a workgroup computes a 32 x 32 quarter of the
// tile as 2 x 2 MFMA blocks of 16 x 16.  The MFMA's M index runs over the
// output columns and its N index over the output rows, so that the 16 lanes
// of a group hold consecutive rows of one column and every store of a wave
// writes 128-byte runs of four columns.
//
// Lane layout of v_mfma_f64_16x16x4f64 (wave64, checked on the device):
// lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] of the 16 x 4 and
// 4 x 16 operands and receives C[l / 16 + 4 r][l % 16], r = 0..3, of the
// 16 x 16 result.
#include <algorithm>

#include "internal.hpp"

namespace polfed {

namespace {

using d4 = __attribute__((ext_vector_type(4))) double;
constexpr int kT = 64;       // output tile edge
constexpr int kKC = 32;      // inner chunk staged per iteration
constexpr int kPad = 2;      // LDS row padding (doubles)
constexpr int kTnMinRows = 256;

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// The 2 x 2 blocks of a wave: MFMA A operand from sM ([k][M index]), B
// operand from sN ([k][N index]), over one staged chunk of kKC.
__device__ __forceinline__ void mfma_chunk(const double (*sM)[kT + kPad],
                                           const double (*sN)[kT + kPad], int wm, int wn,
                                           int lane, d4 (&acc)[2][2]) {
  const int li = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int ks = 0; ks < kKC; ks += 4) {
    double a[2], b[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      a[q] = sM[ks + lk][wm * 32 + q * 16 + li];
      b[q] = sN[ks + lk][wn * 32 + q * 16 + li];
    }
#pragma unroll
    for (int qm = 0; qm < 2; ++qm)
#pragma unroll
      for (int qn = 0; qn < 2; ++qn) acc[qm][qn] = mfma(a[qm], b[qn], acc[qm][qn]);
  }
}

// C = A B (SUB: C -= A B).  Tile (blockIdx.x: 64 rows of D, blockIdx.y: 64
// columns of n); MFMA M = columns of C, N = rows of C, K = m.
template <bool SUB>
__global__ __launch_bounds__(256) void k_gemm_nn(int64_t D, int m, int n, const double* A,
                                                 int64_t lda, const double* B, int64_t ldb,
                                                 double* C, int64_t ldc) {
  __shared__ double sA[kKC][kT + kPad];  // [k][row]
  __shared__ double sB[kKC][kT + kPad];  // [k][col]
  const int64_t I0 = (int64_t)blockIdx.x * kT;
  const int J0 = blockIdx.y * kT;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wn = w & 1, wm = w >> 1;  // wave's row half (N) and column half (M)
  d4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = d4{0, 0, 0, 0};
  for (int k0 = 0; k0 < m; k0 += kKC) {
    // A chunk: 64 rows x 32 k, coalesced along the rows of each column
#pragma unroll
    for (int q = 0; q < kT * kKC / 256; ++q) {
      const int idx = t + 256 * q, kk = idx / kT, ii = idx % kT;
      const int64_t r = I0 + ii;
      const int k = k0 + kk;
      sA[kk][ii] = (r < D && k < m) ? A[r + (int64_t)k * lda] : 0.0;
    }
    // B chunk: 32 k x 64 columns, coalesced along k within a column
#pragma unroll
    for (int q = 0; q < kT * kKC / 256; ++q) {
      const int idx = t + 256 * q, kk = idx % kKC, jj = idx / kKC;
      const int j = J0 + jj, k = k0 + kk;
      sB[kk][jj] = (j < n && k < m) ? B[k + (int64_t)j * ldb] : 0.0;
    }
    __syncthreads();
    mfma_chunk(sB, sA, wm, wn, lane, acc);
    __syncthreads();
  }
  const int li = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int qm = 0; qm < 2; ++qm)
#pragma unroll
    for (int qn = 0; qn < 2; ++qn) {
      const int64_t r = I0 + wn * 32 + qn * 16 + li;
      if (r >= D) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = J0 + wm * 32 + qm * 16 + lk + 4 * e;
        if (j < n) {
          double* p = C + r + (int64_t)j * ldc;
          if (SUB)
            *p -= acc[qm][qn][e];
          else
            *p = acc[qm][qn][e];
        }
      }
    }
}

// Partial G tiles: part[z] (n1 x n2, col-major) = A^T B over the rows of
// split z.  MFMA M = columns of A (rows of G), N = columns of B, K = rows.
__global__ __launch_bounds__(256) void k_gemm_tn(int64_t D, int n1, int n2, const double* A,
                                                 int64_t lda, const double* B, int64_t ldb,
                                                 int64_t rows_per, double* part) {
  __shared__ double sA[kKC][kT + kPad];  // [row][col of A]
  __shared__ double sB[kKC][kT + kPad];  // [row][col of B]
  const int J1 = blockIdx.x * kT, J2 = blockIdx.y * kT;
  const int64_t r0 = (int64_t)blockIdx.z * rows_per;
  const int64_t r1 = std::min<int64_t>(D, r0 + rows_per);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wn = w & 1, wm = w >> 1;
  d4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = d4{0, 0, 0, 0};
  for (int64_t k0 = r0; k0 < r1; k0 += kKC) {
#pragma unroll
    for (int q = 0; q < kT * kKC / 256; ++q) {
      const int idx = t + 256 * q, kk = idx % kKC, jj = idx / kKC;
      const int64_t r = k0 + kk;
      const int j1 = J1 + jj, j2 = J2 + jj;
      sA[kk][jj] = (r < r1 && j1 < n1) ? A[r + (int64_t)j1 * lda] : 0.0;
      sB[kk][jj] = (r < r1 && j2 < n2) ? B[r + (int64_t)j2 * ldb] : 0.0;
    }
    __syncthreads();
    mfma_chunk(sA, sB, wm, wn, lane, acc);
    __syncthreads();
  }
  const int li = lane & 15, lk = lane >> 4;
  double* P = part + (int64_t)blockIdx.z * n1 * n2;
#pragma unroll
  for (int qm = 0; qm < 2; ++qm)
#pragma unroll
    for (int qn = 0; qn < 2; ++qn) {
      const int j2 = J2 + wn * 32 + qn * 16 + li;
      if (j2 >= n2) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j1 = J1 + wm * 32 + qm * 16 + lk + 4 * e;
        if (j1 < n1) P[j1 + (int64_t)j2 * n1] = acc[qm][qn][e];
      }
    }
}

// ---- 128 x 128 tiles, for outputs wider than 64 columns ----
//
// Each wave computes a 64 x 64 quarter as 4 x 4 MFMA blocks, so an operand
// read from LDS serves four of them, and a column of A is read once for 128
// columns of C instead of for 64.  Chunks of 16 along the inner dimension are
// double buffered: the next one is on its way into registers while the matrix
// cores work, and one barrier a chunk suffices.  In LDS the operand that is
// read along the inner dimension lies with that dimension inside ([column]
// [k], rows of 17) and the other one outside ([k][row], rows of 144): both the
// stores and the MFMA's reads (16 consecutive rows or columns, two k at a
// time) then touch every bank once.
//
// FP64 TF on one MI355X (72.6 for a library product of 8192 square matrices),
// 64 x 64 tiles / these: nn 184,756 x 231 x 120 18.3 / 38, 705,432 x 800 x 400
// 20 / 46; tn 184,756 x 120 x 120 12 / 37, 705,432 x 400 x 400 15 / 35.  What
// is left is the chunk's barrier with two workgroups a CU (the accumulators
// and the chunk in flight take 240 registers) and, for 130 columns, padding.
constexpr int kW = 128;            // tile edge
constexpr int kKW = 16;            // inner chunk
constexpr int kLdK = kKW + 1;      // row of [column][k]
constexpr int kLdR = kW + 16;      // row of [k][row]
constexpr size_t kNnShm = 2 * (kKW * kLdR + kW * kLdK) * sizeof(double);
constexpr size_t kTnShm = 2 * (2 * kW * kLdK) * sizeof(double);

using Acc = d4[4][4];

__device__ __forceinline__ void clear(Acc& acc) {
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = d4{0, 0, 0, 0};
}

// C = A B (SUB: C -= A B).  MFMA M = columns of C, N = rows of C, K = m.  The
// column tiles of a row tile run one after another on one XCD.
template <bool SUB>
__global__ __launch_bounds__(256, 2) void k_gemm_nn_wide(int64_t D, int m, int n, int ny,
                                                         const double* A, int64_t lda,
                                                         const double* B, int64_t ldb, double* C,
                                                         int64_t ldc) {
  extern __shared__ __attribute__((aligned(16))) double shm[];
  double* const sA = shm;                    // [2][kKW][kLdR]
  double* const sB = shm + 2 * kKW * kLdR;   // [2][kW][kLdK]
  const int64_t local = blockIdx.x / 8;
  const int64_t I0 = ((local / ny) * 8 + blockIdx.x % 8) * kW;
  const int J0 = (int)(local % ny) * kW;
  if (I0 >= D) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wn = w & 1, wm = w >> 1;  // wave's row half (N) and column half (M)
  const int li = lane & 15, lk = lane >> 4;
  Acc acc;
  clear(acc);
  // this thread's part of a chunk: row t % 128, every second k; k t % 16,
  // every 16th column
  const int ar = t & (kW - 1), ak = t >> 7, bk = t & (kKW - 1), bj = t >> 4;
  const bool a_in = I0 + ar < D;
  const double* pa = A + (a_in ? I0 + ar : 0);
  double ra[8], rb[8];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int k = k0 + ak + 2 * q;
      ra[q] = a_in && k < m ? pa[(int64_t)k * lda] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int k = k0 + bk, j = J0 + bj + 16 * q;
      rb[q] = j < n && k < m ? B[k + (int64_t)j * ldb] : 0.0;
    }
  };
  auto store = [&](int b) {
#pragma unroll
    for (int q = 0; q < 8; ++q) sA[(b * kKW + ak + 2 * q) * kLdR + ar] = ra[q];
#pragma unroll
    for (int q = 0; q < 8; ++q) sB[(b * kW + bj + 16 * q) * kLdK + bk] = rb[q];
  };
  load(0);
  store(0);
  __syncthreads();
  for (int k0 = 0, b = 0; k0 < m; k0 += kKW, b ^= 1) {
    const bool more = k0 + kKW < m;
    if (more) load(k0 + kKW);
#pragma unroll
    for (int ks = 0; ks < kKW; ks += 4) {
      double x[4], y[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        x[q] = sB[(b * kW + wm * 64 + q * 16 + li) * kLdK + ks + lk];
        y[q] = sA[(b * kKW + ks + lk) * kLdR + wn * 64 + q * 16 + li];
      }
#pragma unroll
      for (int qm = 0; qm < 4; ++qm)
#pragma unroll
        for (int qn = 0; qn < 4; ++qn) acc[qm][qn] = mfma(x[qm], y[qn], acc[qm][qn]);
    }
    if (more) store(b ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int qn = 0; qn < 4; ++qn) {
    const int64_t r = I0 + wn * 64 + qn * 16 + li;
    if (r >= D) continue;
#pragma unroll
    for (int qm = 0; qm < 4; ++qm)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = J0 + wm * 64 + qm * 16 + lk + 4 * e;
        if (j < n) {
          double* p = C + r + (int64_t)j * ldc;
          if (SUB)
            *p -= acc[qm][qn][e];
          else
            *p = acc[qm][qn][e];
        }
      }
  }
}

// Partial G tiles as in k_gemm_tn.
__global__ __launch_bounds__(256, 2) void k_gemm_tn_wide(int64_t D, int n1, int n2,
                                                         const double* A, int64_t lda,
                                                         const double* B, int64_t ldb,
                                                         int64_t rows_per, double* part) {
  extern __shared__ __attribute__((aligned(16))) double shm[];
  double* const sA = shm;                   // [2][kW][kLdK]
  double* const sB = shm + 2 * kW * kLdK;
  const int J1 = blockIdx.x * kW, J2 = blockIdx.y * kW;
  const int64_t r0 = (int64_t)blockIdx.z * rows_per;
  const int64_t r1 = std::min<int64_t>(D, r0 + rows_per);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wn = w & 1, wm = w >> 1;
  const int li = lane & 15, lk = lane >> 4;
  Acc acc;
  clear(acc);
  const int kk = t & (kKW - 1), jj = t >> 4;
  double ra[8], rb[8];
  auto load = [&](int64_t k0) {
    const int64_t r = k0 + kk;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j1 = J1 + jj + 16 * q;
      ra[q] = r < r1 && j1 < n1 ? A[r + (int64_t)j1 * lda] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j2 = J2 + jj + 16 * q;
      rb[q] = r < r1 && j2 < n2 ? B[r + (int64_t)j2 * ldb] : 0.0;
    }
  };
  auto store = [&](int b) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      sA[(b * kW + jj + 16 * q) * kLdK + kk] = ra[q];
      sB[(b * kW + jj + 16 * q) * kLdK + kk] = rb[q];
    }
  };
  load(r0);
  store(0);
  __syncthreads();
  int b = 0;
  for (int64_t k0 = r0; k0 < r1; k0 += kKW, b ^= 1) {
    const bool more = k0 + kKW < r1;
    if (more) load(k0 + kKW);
#pragma unroll
    for (int ks = 0; ks < kKW; ks += 4) {
      double x[4], y[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        x[q] = sA[(b * kW + wm * 64 + q * 16 + li) * kLdK + ks + lk];
        y[q] = sB[(b * kW + wn * 64 + q * 16 + li) * kLdK + ks + lk];
      }
#pragma unroll
      for (int qm = 0; qm < 4; ++qm)
#pragma unroll
        for (int qn = 0; qn < 4; ++qn) acc[qm][qn] = mfma(x[qm], y[qn], acc[qm][qn]);
    }
    if (more) store(b ^ 1);
    __syncthreads();
  }
  double* P = part + (int64_t)blockIdx.z * n1 * n2;
#pragma unroll
  for (int qn = 0; qn < 4; ++qn) {
    const int j2 = J2 + wn * 64 + qn * 16 + li;
    if (j2 >= n2) continue;
#pragma unroll
    for (int qm = 0; qm < 4; ++qm)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j1 = J1 + wm * 64 + qm * 16 + lk + 4 * e;
        if (j1 < n1) P[j1 + (int64_t)j2 * n1] = acc[qm][qn][e];
      }
  }
}

// G (ldg) = sum over the splits of part: a workgroup takes 32 entries, its
// eight groups of 32 threads an eighth of the splits each, in split order, and
// the eight sums are added in that order (512 splits of 120 x 120: one thread
// an entry 129 us, this 10).
__global__ __launch_bounds__(256) void k_sum_splits(int n1, int n2, int nsplit, const double* part,
                                                    double* G, int64_t ldg) {
  __shared__ double red[8][32];
  const int x = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int64_t ne = (int64_t)n1 * n2, e = (int64_t)blockIdx.x * 32 + x;
  const int z0 = nsplit * g / 8, z1 = nsplit * (g + 1) / 8;
  double s = 0;
  if (e < ne) {
#pragma unroll 8
    for (int z = z0; z < z1; ++z) s += part[(int64_t)z * ne + e];
  }
  red[g][x] = s;
  __syncthreads();
  if (g != 0 || e >= ne) return;
  for (int q = 1; q < 8; ++q) s += red[q][x];
  G[(e % n1) + (e / n1) * ldg] = s;
}

}  // namespace

// Wide tiles where they are not mostly padding (the 64 x 64 ones also where
// one side fits them).
static bool tn_wide(int n1, int n2) { return n1 > kT && n2 > kT; }

// Two workgroups of wide tiles a CU, four of the others.
int gemm_tn_splits(int64_t D, int n1, int n2) {
  const int e = tn_wide(n1, n2) ? kW : kT, most = tn_wide(n1, n2) ? 512 : 1024;
  const int64_t tiles = (int64_t)((n1 + e - 1) / e) * ((n2 + e - 1) / e);
  int64_t z = (most + tiles - 1) / std::max<int64_t>(tiles, 1);
  z = std::min<int64_t>(z, std::max<int64_t>(1, D / kTnMinRows));
  return (int)std::max<int64_t>(1, std::min<int64_t>(z, 512));
}

size_t gemm_tn_workspace(int64_t D, int n1, int n2) {
  return (size_t)gemm_tn_splits(D, n1, n2) * (size_t)n1 * (size_t)n2 * sizeof(double);
}

void dev_gemm_nn(hipStream_t s, int64_t D, int m, int n, const double* A, int64_t lda,
                 const double* B, int64_t ldb, double* C, int64_t ldc, bool sub) {
  if (D <= 0 || n <= 0) return;
  if (m <= 0) {
    REQUIRE(sub, "gemm: empty inner dimension");
    return;  // C -= 0
  }
  REQUIRE((D + kT - 1) / kT < (int64_t(1) << 31), "gemm: too many rows");
  const int ny = (n + kW - 1) / kW;
  const int64_t rows = ((D + kW - 1) / kW + 7) / 8 * 8;
  // wide tiles while they fill the chip (D = 3,432, 158 x 70: 54 tiles of 64 x
  // 64 take 31 us, 27 wide ones 43; D = 48,620, 160 x 66: 84 and 68)
  if (n > kT && rows * ny >= 200) {
    REQUIRE(rows * ny < (int64_t(1) << 31), "gemm: too many tiles");
    const dim3 g((unsigned)(rows * ny));
    if (sub)
      hipLaunchKernelGGL(k_gemm_nn_wide<true>, g, dim3(256), kNnShm, s, D, m, n, ny, A, lda, B,
                         ldb, C, ldc);
    else
      hipLaunchKernelGGL(k_gemm_nn_wide<false>, g, dim3(256), kNnShm, s, D, m, n, ny, A, lda, B,
                         ldb, C, ldc);
    HIPC(hipGetLastError());
    return;
  }
  const dim3 grid((unsigned)((D + kT - 1) / kT), (unsigned)((n + kT - 1) / kT));
  if (sub)
    hipLaunchKernelGGL(k_gemm_nn<true>, grid, dim3(256), 0, s, D, m, n, A, lda, B, ldb, C, ldc);
  else
    hipLaunchKernelGGL(k_gemm_nn<false>, grid, dim3(256), 0, s, D, m, n, A, lda, B, ldb, C, ldc);
  HIPC(hipGetLastError());
}

void dev_gemm_tn(hipStream_t s, int64_t D, int n1, int n2, const double* A, int64_t lda,
                 const double* B, int64_t ldb, double* G, int64_t ldg) {
  if (n1 <= 0 || n2 <= 0) return;
  const int z = gemm_tn_splits(D, n1, n2);
  const int64_t rows_per = std::max<int64_t>(1, (D + z - 1) / z);
  DevBuf part(gemm_tn_workspace(D, n1, n2));
  const int e = tn_wide(n1, n2) ? kW : kT;
  const dim3 grid((unsigned)((n1 + e - 1) / e), (unsigned)((n2 + e - 1) / e), (unsigned)z);
  if (tn_wide(n1, n2))
    hipLaunchKernelGGL(k_gemm_tn_wide, grid, dim3(256), kTnShm, s, D, n1, n2, A, lda, B, ldb,
                       rows_per, part.as<double>());
  else
    hipLaunchKernelGGL(k_gemm_tn, grid, dim3(256), 0, s, D, n1, n2, A, lda, B, ldb, rows_per,
                       part.as<double>());
  const int64_t ne = (int64_t)n1 * n2;
  hipLaunchKernelGGL(k_sum_splits, dim3((unsigned)((ne + 31) / 32)), dim3(256), 0, s, n1, n2,
                     z, part.as<double>(), G, ldg);
  HIPC(hipGetLastError());
}

}  // namespace polfed
