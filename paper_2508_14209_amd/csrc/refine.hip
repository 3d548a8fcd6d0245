// refine.hip -- FP64 residual of the mixed-precision least-squares path.
//
// r = B - A X in FP64: A (d x n, FP32 or FP64, column-major) is promoted
// exactly, X (n x nrhs) is FP64, B has A's type, every product and sum is
// FP64.  Each thread takes V groups of four consecutive rows with 16-byte
// loads of every column of A and keeps the 4 V x nrhs sums in registers; X is
// staged in LDS.
//
// Bound by HBM: A is read once.  What decides the rate is how much of one
// column a workgroup reads before it goes on to the next, which is on another
// page: a sum over 8,388,608 x 256 FP32 read at 5.6 TB/s with 4 KB of a column
// at a time and at 6.8 TB/s with 64 KB and nontemporal loads.
#include <algorithm>

#include "ms_internal.h"

namespace ms {

// Four consecutive rows of a column, NT: by a nontemporal load.  The loads are
// aligned to the element only (a dword-aligned multi-dword global load is legal on
// CDNA), so a column may start at any element.
template <bool NT, typename TA>
__device__ __forceinline__ auto rows4(const TA *p) {
  typedef TA V __attribute__((ext_vector_type(4)));
  typedef TA Vu __attribute__((ext_vector_type(4), aligned(sizeof(TA))));
  const auto *g = (const __attribute__((address_space(1))) Vu *)p;
  return NT ? (V)__builtin_nontemporal_load(g) : (V)*g;
}

constexpr int kResXlds = 8192;  // most doubles of X staged in LDS (64 KB)

// FP32 data of more than the last-level cache's 256 MB is read by nontemporal loads,
// all else by ordinary ones: a solve reads A and B for the sketch and for each step,
// and what is cached stays so.  Eight steps, FP32: 600,000 x 128 (302 MB), 4 right-hand sides
// 1.46 ms cached, 1.41 nontemporal; 2,000,000 x 16 (153 MB) 0.70 and 0.77.  FP64:
// cached is as fast or faster at every size measured (3 to 8450 MB), 2,000,000 x 8,
// 1 right-hand side 0.51 and 0.58 ms, 4,194,304 x 256, 2 right-hand sides 14.2 and 14.4.
constexpr int64_t kResCached = (int64_t)256 << 20;

// The residuals of V groups of four rows, i0 + v * vstep each.  Unless LAST every
// row is inside the matrix; LAST (V = 1, d >= 4): the group that would end past row d
// starts at d - 4 instead and stores the rows that are its own.  x(j, c): X[j, c].
// U columns' loads are issued before their products.
template <typename TA, int RH, int V, int U, bool NT, bool LAST, typename XF>
__device__ __forceinline__ void residual_groups(int64_t i0, int64_t vstep, int64_t d, int n,
                                                int nrhs, const TA *__restrict__ A, int64_t lda,
                                                const TA *__restrict__ B, int64_t ldb, const XF &x,
                                                double *__restrict__ r, int64_t ldr) {
  static_assert(!LAST || V == 1, "one group");
  const int64_t g0 = LAST ? min(i0, d - 4) : i0;
  typedef TA V4 __attribute__((ext_vector_type(4)));
  double acc[V][4][RH];
#pragma unroll
  for (int v = 0; v < V; ++v)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < RH; ++c) acc[v][q][c] = 0.0;
  auto column = [&](int j, const V4 (&a)[V]) {
#pragma unroll
    for (int c = 0; c < RH; ++c) {
      const double xc = x(j, c);
#pragma unroll
      for (int v = 0; v < V; ++v)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[v][q][c] += (double)a[v][q] * xc;
    }
  };
  int j = 0;
  for (; j + U <= n; j += U) {
    V4 a[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v) a[u][v] = rows4<NT>(A + g0 + v * vstep + (int64_t)(j + u) * lda);
    __builtin_amdgcn_sched_barrier(0);   // all of them, or the compiler may put some off
#pragma unroll
    for (int u = 0; u < U; ++u) column(j + u, a[u]);
  }
  for (; j < n; ++j) {
    V4 a[V];
#pragma unroll
    for (int v = 0; v < V; ++v) a[v] = rows4<NT>(A + g0 + v * vstep + (int64_t)j * lda);
    column(j, a);
  }
#pragma unroll
  for (int c = 0; c < RH; ++c)
    if (c < nrhs) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const V4 b = rows4<NT>(B + g0 + v * vstep + (int64_t)c * ldb);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (!LAST || g0 + q >= i0)
            r[g0 + v * vstep + q + (int64_t)c * ldr] = (double)b[q] - acc[v][q][c];
      }
    }
}

// The residuals of a matrix of fewer than four rows, a row per thread.
template <typename TA, int RH, typename XF>
__device__ __forceinline__ void residual_rows(int64_t d, int n, int nrhs, const TA *__restrict__ A,
                                              int64_t lda, const TA *__restrict__ B, int64_t ldb,
                                              const XF &x, double *__restrict__ r, int64_t ldr) {
  const int64_t i = threadIdx.x;
  if (i >= d) return;
  double acc[RH];
#pragma unroll
  for (int c = 0; c < RH; ++c) acc[c] = 0.0;
#pragma unroll 4
  for (int j = 0; j < n; ++j) {
    const double a = (double)gload(A + i + (int64_t)j * lda);
#pragma unroll
    for (int c = 0; c < RH; ++c) acc[c] += a * x(j, c);
  }
#pragma unroll
  for (int c = 0; c < RH; ++c)
    if (c < nrhs) r[i + (int64_t)c * ldr] = (double)gload(B + i + (int64_t)c * ldb) - acc[c];
}

// RH: right-hand sides held (nrhs <= RH; the X of the missing ones is zero).
template <typename TA, bool XLDS, int RH, int T, int V, bool NT>
__global__ __launch_bounds__(T) void k_residual(int64_t d, int n, int nrhs,
                                                const TA *__restrict__ A, int64_t lda,
                                                const TA *__restrict__ B, int64_t ldb,
                                                const double *__restrict__ X, int64_t ldx,
                                                double *__restrict__ r, int64_t ldr) {
  extern __shared__ __align__(16) double xs[];  // xs[j * RH + c] = X[j, c]
  if (XLDS) {
    for (int t = threadIdx.x; t < n * RH; t += T) {
      const int c = t % RH, j = t / RH;
      xs[t] = c < nrhs ? X[j + (int64_t)c * ldx] : 0.0;
    }
    __syncthreads();
  }
  auto xv = [&](int j, int c) {
    return XLDS ? xs[j * RH + c] : c < nrhs ? X[j + (int64_t)c * ldx] : 0.0;
  };
  constexpr int64_t blk = (int64_t)4 * T * V;
  constexpr int U = V > 1 || (RH == 8 && sizeof(TA) == 8) ? 2 : 4;   // in flight, as the registers allow
  int64_t r0 = (int64_t)blockIdx.x * blk;
  for (; r0 + blk <= d; r0 += gridDim.x * blk)
    residual_groups<TA, RH, V, U, NT, false>(r0 + 4 * (int64_t)threadIdx.x, 4 * T, d, n, nrhs, A,
                                             lda, B, ldb, xv, r, ldr);
  // the last rows a group at a time (the matrix's last one to three row by row in one
  // lane, each element read for every right-hand side, were a chain of up to 3 n nrhs
  // loads: eight steps of 100,003 x 256 FP32, 8 right-hand sides, with the solve 6.7 ms,
  // now 2.6)
  if (r0 < d && d < 4) return residual_rows<TA, RH>(d, n, nrhs, A, lda, B, ldb, xv, r, ldr);
  for (int64_t i = r0 + 4 * (int64_t)threadIdx.x; i < d; i += 4 * T)
    residual_groups<TA, RH, 1, 4, false, true>(i, 0, d, n, nrhs, A, lda, B, ldb, xv, r, ldr);
}

template <typename TA, bool XLDS, int RH, int T, int V>
static void launch_residual_k(unsigned grid, int64_t d, int64_t n, int64_t nrhs, const TA *A,
                              int64_t lda, const TA *B, int64_t ldb, const double *X, int64_t ldx,
                              double *r, int64_t ldr, hipStream_t st) {
  const size_t lds = XLDS ? (size_t)n * RH * sizeof(double) : 0;
  if (sizeof(TA) == 4 && d * (n + nrhs) * 4 > kResCached)
    hipLaunchKernelGGL((k_residual<TA, XLDS, RH, T, V, sizeof(TA) == 4>), dim3(grid), dim3(T), lds,
                       st, d, (int)n, (int)nrhs, A, lda, B, ldb, X, ldx, r, ldr);
  else
    hipLaunchKernelGGL((k_residual<TA, XLDS, RH, T, V, false>), dim3(grid), dim3(T), lds, st, d,
                       (int)n, (int)nrhs, A, lda, B, ldb, X, ldx, r, ldr);
}

// T, V: the wide workgroup of this many right-hand sides, one to a compute unit (32 V T
// bytes of FP64, 16 V T of FP32 of a column at a time, as many as the registers of
// the sums allow), where its rounds are at least five sixths full; else 1024 rows at a
// time.  Eight steps, 1 right-hand side: 7,000,000 x 64 (0.83 full) FP64 6.23 ms wide, 6.43
// narrow, 9,000,000 (0.72) 8.6 and 8.1, 4,300,000 (0.51) 5.1 and 4.1 (FP32 3.48 and 3.52,
// 4.65 and 4.46, 2.75 and 2.35).
template <typename TA, int RH, int T, int V>
static hipError_t launch_residual_rh(int64_t d, int64_t n, int64_t nrhs, const TA *A, int64_t lda,
                                     const TA *B, int64_t ldb, const double *X, int64_t ldx,
                                     double *r, int64_t ldr, hipStream_t st) {
  const int64_t cus = dev_info().cus, round = cus * 4 * T * V;
  const bool wide = 6 * d >= 5 * round * ((d + round - 1) / round), xl = n * RH <= kResXlds;
  const unsigned gw = (unsigned)std::min<int64_t>((d + 4 * T * V - 1) / (4 * T * V), cus * (1024 / T));
  const unsigned gn = (unsigned)std::min<int64_t>((d + 1023) / 1024, cus * 8);
  if (wide && xl)
    launch_residual_k<TA, true, RH, T, V>(gw, d, n, nrhs, A, lda, B, ldb, X, ldx, r, ldr, st);
  else if (xl)
    launch_residual_k<TA, true, RH, 256, 1>(gn, d, n, nrhs, A, lda, B, ldb, X, ldx, r, ldr, st);
  else
    launch_residual_k<TA, false, RH, 256, 1>(gn, d, n, nrhs, A, lda, B, ldb, X, ldx, r, ldr, st);
  return hipGetLastError();
}

template <typename TA>
static hipError_t launch_residual_t(int64_t d, int64_t n, int64_t nrhs, const TA *A, int64_t lda,
                                    const TA *B, int64_t ldb, const double *X, int64_t ldx,
                                    double *r, int64_t ldr, hipStream_t st) {
  if (nrhs > 8 || nrhs < 1) return hipErrorInvalidValue;
  if (d <= 0) return hipSuccess;
  if (nrhs == 1) return launch_residual_rh<TA, 1, 1024, 4>(d, n, nrhs, A, lda, B, ldb, X, ldx, r, ldr, st);
  if (nrhs == 2) return launch_residual_rh<TA, 2, 1024, 2>(d, n, nrhs, A, lda, B, ldb, X, ldx, r, ldr, st);
  if (nrhs <= 4) return launch_residual_rh<TA, 4, 512, 4>(d, n, nrhs, A, lda, B, ldb, X, ldx, r, ldr, st);
  return launch_residual_rh<TA, 8, 512, 2>(d, n, nrhs, A, lda, B, ldb, X, ldx, r, ldr, st);
}

hipError_t launch_residual_f32(int64_t d, int64_t n, int64_t nrhs, const float *A, int64_t lda,
                               const float *B, int64_t ldb, const double *X, int64_t ldx,
                               double *r, int64_t ldr, hipStream_t st) {
  return launch_residual_t<float>(d, n, nrhs, A, lda, B, ldb, X, ldx, r, ldr, st);
}

hipError_t launch_residual_f64(int64_t d, int64_t n, int64_t nrhs, const double *A, int64_t lda,
                               const double *B, int64_t ldb, const double *X, int64_t ldx,
                               double *r, int64_t ldr, hipStream_t st) {
  return launch_residual_t<double>(d, n, nrhs, A, lda, B, ldb, X, ldx, r, ldr, st);
}

// Residuals of a batch: item = (problem, kBatchResRows rows), X staged in LDS
// once per item; B has A's type.  r_p is d x nrhs, column-major, ld d.  Two
// groups of four rows per thread at once (8 KB of an FP32 column), one where
// the sums of more than four right-hand sides take the registers.
template <typename TA>
__global__ __launch_bounds__(256) void k_batch_residual(
    int count, const ms_problem *__restrict__ P, const BatchEntry *__restrict__ E,
    const BatchTotals *__restrict__ tot, unsigned char *__restrict__ rarea) {
  constexpr int RH = kBatchMaxRefineRhs;
  constexpr bool NT = sizeof(TA) == 4;   // (a batch is mostly more than the cache holds)
  static_assert(kBatchResRows == 2048, "256 threads, two groups of four rows each");
  __shared__ __align__(16) double xs[kBatchMaxCols * RH];  // xs[j * rh + c] = X[j, c]
  const int64_t total = tot->res_items;
  for (int64_t it = blockIdx.x; it < total; it += gridDim.x) {
    const int p = batch_find_m<&BatchEntry::res_start>(E, count, it);
    const ms_problem &Q = P[p];
    const BatchEntry &e = E[p];
    if (!e.refine) continue;   // converged in an earlier step
    const int n = (int)Q.n, nrhs = (int)Q.nrhs;
    const int rh = nrhs <= 2 ? nrhs : nrhs <= 4 ? 4 : 8;
    const TA *A = static_cast<const TA *>(Q.A);
    const TA *B = static_cast<const TA *>(Q.B);
    const int64_t lda = Q.lda, ldb = Q.ldb, d = Q.d;
    double *r = reinterpret_cast<double *>(rarea + e.r_off);
    __syncthreads();  // the previous item's reads of xs are done
    for (int t = threadIdx.x; t < n * rh; t += 256) {
      const int j = t / rh, c = t - j * rh;
      xs[t] = c < nrhs ? gload(Q.X + j + (int64_t)c * Q.ldx) : 0.0;
    }
    __syncthreads();
    const int64_t r0 = (it - e.res_start) * kBatchResRows, i0 = r0 + 4 * (int64_t)threadIdx.x;
    const bool whole = r0 + kBatchResRows <= d;   // uniform
#define MS_BRES(RH_, V_)                                                                        \
  {                                                                                             \
    auto xv = [&](int j, int c) { return xs[j * RH_ + c]; };                                    \
    if (whole) {                                                                                \
      for (int v = 0; v < 2; v += V_)                                                           \
        residual_groups<TA, RH_, V_, 2, NT, false>(i0 + 1024 * v, 1024, d, n, nrhs, A, lda, B,  \
                                                   ldb, xv, r, d);                              \
    } else if (d >= 4) {                                                                        \
      for (int64_t i = i0; i < d; i += 1024)                                                    \
        residual_groups<TA, RH_, 1, 4, false, true>(i, 0, d, n, nrhs, A, lda, B, ldb, xv, r,    \
                                                    d);                                         \
    } else {                                                                                    \
      residual_rows<TA, RH_>(d, n, nrhs, A, lda, B, ldb, xv, r, d);                             \
    }                                                                                           \
  }
    if (rh == 1)
      MS_BRES(1, 2)
    else if (rh == 2)
      MS_BRES(2, 2)
    else if (rh == 4)
      MS_BRES(4, 2)
    else
      MS_BRES(8, 1)
#undef MS_BRES
  }
}

template <typename TA>
hipError_t launch_batch_residual(int count, const ms_problem *P, const BatchEntry *E,
                                 const BatchTotals *tot, unsigned char *rarea, int grid,
                                 hipStream_t st) {
  hipLaunchKernelGGL(k_batch_residual<TA>, dim3(grid), dim3(256), 0, st, count, P, E, tot,
                     rarea);
  return hipGetLastError();
}
template hipError_t launch_batch_residual<float>(int, const ms_problem *, const BatchEntry *,
                                                 const BatchTotals *, unsigned char *, int,
                                                 hipStream_t);
template hipError_t launch_batch_residual<double>(int, const ms_problem *, const BatchEntry *,
                                                  const BatchTotals *, unsigned char *, int,
                                                  hipStream_t);

// X += dX (n x nrhs).
__global__ void k_axpy_update(int n, int nrhs, const double *__restrict__ dX, double *X,
                              int64_t ldx) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)n * nrhs) return;
  const int c = (int)(t / n), i = (int)(t - (int64_t)c * n);
  X[i + (int64_t)c * ldx] += dX[t];
}

hipError_t launch_axpy_update(int64_t n, int64_t nrhs, const double *dX, double *X, int64_t ldx,
                              hipStream_t st) {
  const int64_t t = n * nrhs;
  hipLaunchKernelGGL(k_axpy_update, dim3((unsigned)((t + 255) / 256)), dim3(256), 0, st, (int)n,
                     (int)nrhs, dX, X, ldx);
  return hipGetLastError();
}

}  // namespace ms
