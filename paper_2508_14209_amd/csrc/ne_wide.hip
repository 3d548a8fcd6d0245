// ne_wide.hip -- the normal equations (Sec. 6.3's comparator) and the
// Cholesky stage of rand_cholQR (Alg. 5) for wide problems: n up to 256
// columns with up to 16 right-hand sides (n + nrhs <= 272).
//
//   W = V^T V with V = [X | B] (d x nc), X = A (normal equations) or
//   X = Q0 = A R0^{-1} (rand_cholQR), FP64; R1 = chol(W_XX); y = R1^{-T} W_XB;
//   x = R1^{-1} y.
//
// The Gram pass is a tall product, bound by the FP64 matrix cores
// (n (n + 1) + 2 n nrhs flops per row against 8 (n + nrhs) bytes).  One
// workgroup of eight waves per compute unit takes a contiguous share of the
// rows and forms the whole upper triangle of 16 x 16 tiles for it, so V is
// read from memory once: slabs of 16 rows of every column are staged in LDS
// (two buffers, one barrier per slab, the next slab's loads in flight while
// the current one is multiplied), laid out so that staging writes and fragment
// reads are both contiguous 16-byte accesses.  The tiles are dealt out to the
// waves in row-major runs of equal length (at most 20 accumulator tiles, 160
// of a lane's 256 registers).  With the fragments, the staged slab and its pointers
// that is more than there are for 8, 12 and 17 tile columns in FP64 (13, 22 and 12
// registers spilled, reloaded once a slab) and 12 and 17 in FP32 (8 and 1).  FP64 Q0
// beside FP32 B (rand_cholQR of FP32 data; 22 to 43 spilled at 8, 11, 12 and 17)
// loads and converts B's few columns one element at a time, so that each slab
// waits for them; it is not slower for it than the pass before was.  Where
// fewer than eight waves hold all the tiles (n + nrhs <= 192), two or four groups
// of waves each take their own 16 rows of a taller slab.  Every group writes its sums as packed tiles; an
// ordered pass adds them (the same bits on every run).
// 4,194,304 x 256 FP64, one right-hand side: 20.9 -> 6.2 ms (the upper triangle's
// 153 tiles: 53 TFLOP/s of the instruction's 77); 2 x 4-tile tasks per wave, which re-read
// V from L2 and waited for each slab's loads, were what it took before.
//
// The factorisation works on 64 x 64 blocks of the Gram matrix in place: the
// diagonal block by one wave, its block row by one workgroup per 64 columns
// (the right-hand sides are columns of the matrix, so this is the forward
// substitution too), the trailing blocks by one workgroup each on the matrix
// cores; one workgroup then solves backwards.  n = 256: 0.31 ms against 2.0 ms for
// one workgroup doing the block rows, the trailing blocks and the solves from
// memory.
#include <algorithm>
#include <type_traits>

#include "ms_internal.h"

namespace ms {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kGwT = 512;        // threads of a Gram workgroup (8 waves)
constexpr int kSolveN = 256;     // order of the largest factorisation

__device__ __forceinline__ v4d mma64w(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Shape of the Gram pass for NT tile columns: the upper triangle's tiles, the
// waves that hold them all (nw, at most 20 tiles each), the tiles per wave,
// and the wave groups of a workgroup, each with its own 16 rows of a slab.
struct GramShape {
  int ntiles, nw, tpw, groups;
};
constexpr GramShape gram_shape(int NT) {
  GramShape g{};
  g.ntiles = NT * (NT + 1) / 2;
  g.nw = 2;
  while (g.nw < 8 && (g.ntiles + g.nw - 1) / g.nw > 20) g.nw *= 2;
  g.tpw = (g.ntiles + g.nw - 1) / g.nw;
  g.groups = 8 / g.nw;
  return g;
}

// Tile t (row-major) of the upper triangle of an NT x NT tile grid.
struct GramTile {
  int it, jt;
};
__host__ __device__ constexpr GramTile gram_tile(int NT, int t) {
  int i = 0;
  while (t >= NT - i) {
    t -= NT - i;
    ++i;
  }
  return GramTile{i, i + t};
}

typedef double dvec2e __attribute__((ext_vector_type(2), aligned(8)));
typedef float fvec2e __attribute__((ext_vector_type(2), aligned(4)));
typedef double v2d __attribute__((ext_vector_type(2)));
// Two consecutive rows of a column as stored, and promoted to FP64.
template <typename T>
struct Pair;
template <>
struct Pair<double> {
  typedef dvec2e type;
};
template <>
struct Pair<float> {
  typedef fvec2e type;
};
template <typename T>
__device__ __forceinline__ typename Pair<T>::type rows2(const T *p) {
  return *(const __attribute__((address_space(1))) typename Pair<T>::type *)p;
}
template <typename P>
__device__ __forceinline__ v2d promote2(const P &x) {
  return v2d{(double)x[0], (double)x[1]};
}

// The products of a wave's tiles t0 .. t0 + tpw - 1 (the first one first) for
// one 16-row slab (slab: this lane's slot of tile column 0, first half).  Per
// half slab the tiles go two at a time, their products alternating (a product
// depends on the one before it on the same tile), the next two tiles'
// fragments read meanwhile and no further ones: they would not fit next to
// the accumulators.  Slots past the last tile repeat it and are not stored.
template <int NT>
__device__ __forceinline__ void gram_products(const unsigned char *slab, int t0, GramTile first,
                                              v4d (&acc)[gram_shape(NT).tpw]) {
  constexpr int TPW = gram_shape(NT).tpw, LAST = gram_shape(NT).ntiles - 1;
  {
    GramTile g = first;
    auto frag = [&](int t) { return *reinterpret_cast<const v2d *>(slab + t * 2048); };
    // fragments of the next tile in the list (g: the tile after it)
    int t = t0;
    auto next = [&](v2d &fi, v2d &fj) {
      fi = frag(g.it);
      fj = frag(g.jt);
      const bool row = g.jt == NT - 1, last = t >= LAST;
      g.it += row && !last;
      g.jt = last ? g.jt : row ? g.it : g.jt + 1;
      ++t;
    };
    v2d fi0, fj0, fi1, fj1;
    next(fi0, fj0);
    next(fi1, fj1);
#pragma unroll
    for (int s = 0; s < TPW; s += 2) {
      v2d ni0 = fi0, nj0 = fj0, ni1 = fi1, nj1 = fj1;
      if (s + 2 < TPW) next(ni0, nj0);
      if (s + 3 < TPW) next(ni1, nj1);
      __builtin_amdgcn_sched_barrier(0);   // the reads first: they are used a pair later
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        acc[s] = mma64w(fi0[r], fj0[r], acc[s]);
        if (s + 1 < TPW) acc[s + 1] = mma64w(fi1[r], fj1[r], acc[s + 1]);
      }
      fi0 = ni0;
      fi1 = ni1;
      fj0 = nj0;
      fj1 = nj1;
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Slab s: rows [s * 16 * groups, ...); its LDS image is, for each group and
// tile column, two 1 KB halves of 64 slots of 16 bytes: slot l of half hh
// holds rows 8 hh + 2 (l / 16) and the next one of column l % 16.  Lane l of a
// fragment read takes slot l of a half; the two rows it gets are the same for
// both operands of a product, whose k order is free.
// Bound by the matrix cores: tpw 16 x 16 x 4 products per wave for every four
// rows, at two waves a SIMD; NT is a template argument so that the tile lists
// and the staged slots per thread have static counts.
template <typename TX, typename TB, int NT>
__global__ __launch_bounds__(kGwT, 2) void k_gram_wide(int64_t d, const TX *__restrict__ X,
                                                       int64_t ldx, const TB *__restrict__ B,
                                                       int64_t ldb, int nx, int nc, int nchunks,
                                                       double *__restrict__ part) {
  extern __shared__ __align__(16) unsigned char gsm[];
  constexpr GramShape gs = gram_shape(NT);
  constexpr int TPW = gs.tpw;
  constexpr int kSlots = gs.groups * NT * 128;          // 16-byte slots of a slab
  constexpr int kQ = (kSlots + kGwT - 1) / kGwT;        // slots a thread stages
  constexpr int kRows = 16 * gs.groups;                 // rows of a slab
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave / gs.nw, wv = wave - grp * gs.nw;
  const int64_t nslab = (d + kRows - 1) / kRows;
  const int64_t s0 = nslab * blockIdx.x / nchunks, s1 = nslab * (blockIdx.x + 1) / nchunks;

  const GramTile tile0 = gram_tile(NT, min(wv * TPW, gs.ntiles - 1));
  // staging: thread tid owns slots tid + 512 q; its row within the group's 16
  // and its column within the tile are the same for every q.  Columns past nc
  // read the last column and are zeroed.  The values are held as stored until
  // the write to LDS (promoted at once when X and B differ in type).
  const int myrow = 8 * ((tid >> 6) & 1) + 2 * ((tid >> 4) & 3);
  const int mycol = tid & 15;
  constexpr bool kSame = std::is_same<TX, TB>::value;
  using P2 = typename Pair<typename std::conditional<kSame, TX, double>::type>::type;
  P2 stg[kQ];
  const TX *px[kQ];   // row 0 of the slot's rows in slab 0 (X, or B of the same type)
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const int ft = min((tid >> 7) + 4 * q, gs.groups * NT - 1);   // group * NT + tile column
    const int c = min(16 * (ft - ft / NT * NT) + mycol, nc - 1);
    const int64_t off = c < nx ? (int64_t)c * ldx : (int64_t)(c - nx) * ldb;
    const TX *base = X;
    if constexpr (kSame) base = c < nx ? X : B;
    px[q] = base + off + 16 * (ft / NT) + myrow;
  }
  // rows r, r + 1 (zero past d) of slot q of slab s
  auto two = [&](const auto *p, int64_t r) {
    double x0 = 0.0, x1 = 0.0;
    if (r < d) x0 = (double)gload(p);
    if (r + 1 < d) x1 = (double)gload(p + 1);
    return P2{(decltype(P2{}[0]))x0, (decltype(P2{}[0]))x1};
  };
  auto fetch = [&](int64_t s, bool full) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const TX *p = px[q] + s * kRows;
      if constexpr (kSame) {
        if (full) {
          stg[q] = rows2(p);
          continue;
        }
      }
      const int ft = min((tid >> 7) + 4 * q, gs.groups * NT - 1);
      const int64_t r = s * kRows + 16 * (ft / NT) + myrow;
      if constexpr (kSame) {
        stg[q] = two(p, r);
      } else {
        const bool isb = min(16 * (ft - ft / NT * NT) + mycol, nc - 1) >= nx;
        if (full && !isb) {
          stg[q] = rows2(p);
        } else if (isb) {
          const int c = min(16 * (ft - ft / NT * NT) + mycol, nc - 1);
          stg[q] = two(B + (int64_t)(c - nx) * ldb + r, r);
        } else {
          stg[q] = two(p, r);
        }
      }
    }
  };
  auto put = [&](unsigned char *buf) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int ft = (tid >> 7) + 4 * q;
      const int f = ft - ft / NT * NT;
      const v2d x = 16 * f + mycol < nc ? promote2(stg[q]) : v2d{0.0, 0.0};
      if (ft < gs.groups * NT) *reinterpret_cast<v2d *>(buf + (tid + kGwT * q) * 16) = x;
    }
  };

  v4d acc[TPW];
#pragma unroll
  for (int s = 0; s < TPW; ++s) acc[s] = v4d{0.0, 0.0, 0.0, 0.0};
  // (the last slab of the matrix may be short: it is fetched apart, so that the
  // loop's loads have no conditions)
  const int64_t nfull = d / kRows;
  auto products = [&](int cur, int half) {
    gram_products<NT>(gsm + cur * (kSlots * 16) + grp * (NT * 2048) + half * 1024 + lane * 16,
                      wv * TPW, tile0, acc);
  };
  int cur = 0;
  const int64_t e1 = min(s1, nfull);
  if (s0 < e1) {
    fetch(s0, true);
    put(gsm);
    fetch(min(s0 + 1, e1 - 1), true);
  }
  __syncthreads();
  for (int64_t sl = s0; sl < e1; ++sl) {
    // between the halves: the next slab, loaded since the middle of the one
    // before, goes to the other buffer and the one after it is asked for
    // (past the last one the same slab again, which is not used)
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      products(cur, half);
      if (half == 0) {
        put(gsm + (cur ^ 1) * (kSlots * 16));
        fetch(min(sl + 2, e1 - 1), true);
      }
    }
    __syncthreads();
    cur ^= 1;
  }
  if (e1 < s1) {
    fetch(e1, false);
    put(gsm + cur * (kSlots * 16));
    __syncthreads();
    products(cur, 0);
    products(cur, 1);
  }
  // packed tiles: entry r * 64 + lane of tile t
  double *P = part + ((int64_t)blockIdx.x * gs.groups + grp) * gs.ntiles * 256;
#pragma unroll
  for (int s = 0; s < TPW; ++s) {
    const int t = wv * TPW + s;
    if (t < gs.ntiles)
#pragma unroll
      for (int r = 0; r < 4; ++r) P[(int64_t)t * 256 + r * 64 + lane] = acc[s][r];
  }
}

// W = the sum of the packed partials: 64 entries of a tile per workgroup,
// sixteen waves each adding a contiguous run of the partials in order, the
// sixteen sums then added in run order.
constexpr int kGrT = 1024;
__global__ __launch_bounds__(kGrT) void k_gram_wide_reduce(int nparts, int NT, int np,
                                                           const double *__restrict__ part,
                                                           double *__restrict__ W) {
  __shared__ double sums[kGrT];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int ntiles = NT * (NT + 1) / 2;
  const int t = blockIdx.x >> 2, r = blockIdx.x & 3;
  const int p0 = nparts * w / 16, p1 = nparts * (w + 1) / 16;
  const double *p = part + (int64_t)t * 256 + r * 64 + lane;
  double s = 0.0;
#pragma unroll 8
  for (int c = p0; c < p1; ++c) s += p[(int64_t)c * ntiles * 256];
  sums[threadIdx.x] = s;
  __syncthreads();
  if (w == 0) {
    double v = sums[lane];
    for (int u = 1; u < 16; ++u) v += sums[u * 64 + lane];
    const GramTile g = gram_tile(NT, t);
    W[(int64_t)(16 * g.it + (lane >> 4) + 4 * r) * np + 16 * g.jt + (lane & 15)] = v;
  }
}

// W_XX = R1^T R1 in place by a blocked right-looking Cholesky with 64 x 64
// blocks; the right-hand sides W_XB are columns n .. n + nrhs - 1 of W and
// take part in every block row and trailing update, which leaves R1^{-T} W_XB
// in them.  W is row-major with leading dimension np (upper part read and
// overwritten).
constexpr int kCsB = 64;    // block order
constexpr int kCsL = 65;    // LDS row stride of a block
constexpr int kCsT = 256;   // threads
constexpr int kCbT = 1024;  // threads of the backward solve

__device__ __forceinline__ double rd_lane(double v, int lane) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(u & 0xffffffffLL), lane);
  const int hi = __builtin_amdgcn_readlane((int)(u >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// element (i, j) of an upper-triangular factor: R1 in W (row-major, np) or
// R0 in fact (column-major, ldf)
struct TriRef {
  const double *p;
  int64_t ld;
  bool rowmajor;
  __device__ double operator()(int i, int j) const {
    return rowmajor ? p[(int64_t)i * ld + j] : p[i + (int64_t)j * ld];
  }
};

// z (LDS, z[c * 256 + i], nrhs columns) := U^{-1} z for upper-triangular U
// of order n, by 64 x 64 blocks from the last (all kCbT threads call it; ub:
// LDS for one block, ps: LDS for kCbT partial sums).  A block's triangle is
// solved by one wave per right-hand side with an unknown per lane
// (finite_quotient(), so that the chain from one unknown to the next is short, and
// once more by divisions if an unknown is not finite); the
// rows above it are then updated by every thread, a row per thread and a
// quarter of the block's columns each.
__device__ void back_solve(const TriRef &U, int n, int nrhs, double *z, double *ub, double *ps) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = (n + kCsB - 1) / kCsB;
  for (int kb = nb - 1; kb >= 0; --kb) {
    const int r0 = kCsB * kb, m = min(kCsB, n - r0);
    for (int t = tid; t < kCsB * kCsB; t += kCbT) {
      // consecutive threads along U's storage
      const int a = t >> 6, b = t & 63;
      const int i = U.rowmajor ? a : b, j = U.rowmajor ? b : a;
      ub[i * kCsL + j] = (i < m && j < m) ? (i <= j ? U(r0 + i, r0 + j) : 0.0) : (i == j ? 1.0 : 0.0);
    }
    __syncthreads();
    if (wave < nrhs) {
      const double z0 = lane < m ? z[wave * 256 + r0 + lane] : 0.0;
      const double dg = ub[lane * kCsL + lane], rc = 1.0 / dg;
      auto solve = [&](auto divide) {
        double zi = z0;
        for (int t = m - 1; t >= 0; --t) {
          const double xt = rd_lane(divide(zi), t);   // lane t's unknown
          // (the unknowns below t are solved: zero times an infinite one must not reach them)
          zi = lane == t ? xt : lane < t ? zi - ub[lane * kCsL + t] * xt : zi;
        }
        return zi;
      };
      double zi = solve([&](double a) { return finite_quotient(a, dg, rc); });
      if (!__all(isfinite(zi))) zi = solve([&](double a) { return a / dg; });
      if (lane < m) z[wave * 256 + r0 + lane] = zi;
    }
    __syncthreads();
    if (r0 > 0) {
      const int i = tid & 255, q4 = tid >> 8;
      double u[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) u[t] = (i < r0 && 16 * q4 + t < m) ? U(i, r0 + 16 * q4 + t) : 0.0;
      for (int c = 0; c < nrhs; ++c) {
        double s = 0.0;
#pragma unroll
        for (int t = 0; t < 16; ++t)
          if (16 * q4 + t < m) s += u[t] * z[c * 256 + r0 + 16 * q4 + t];
        ps[tid] = s;
        __syncthreads();
        if (tid < r0) z[c * 256 + tid] -= ((ps[tid] + ps[256 + tid]) + ps[512 + tid]) + ps[768 + tid];
        __syncthreads();
      }
    }
  }
}

// (a) Diagonal block kb of the blocked Cholesky: one wave, lane l holding
// column l of the block's upper part; R_kk is written back in place.  A
// breakdown sets *bad (every later launch then returns at once).  Block 0
// clears *bad first.
__global__ __launch_bounds__(64) void k_chol_diag(int n, int np, int kb, double *__restrict__ W,
                                                  int *__restrict__ bad) {
  __shared__ double rb[kCsB * kCsL];
  const int lane = threadIdx.x;
  if (kb == 0) {
    if (lane == 0) *bad = 0;
  } else if (*bad) {
    return;
  }
  const int r0 = kCsB * kb, m = min(kCsB, n - r0);
  double g[kCsB];
#pragma unroll
  for (int i = 0; i < kCsB; ++i)
    g[i] = (i < m && lane < m) ? (i <= lane ? W[(int64_t)(r0 + i) * np + r0 + lane] : 0.0)
                               : (i == lane ? 1.0 : 0.0);
  bool fail = false;
#pragma unroll
  for (int j = 0; j < kCsB; ++j) {
    const double djj = rd_lane(g[j], j);
    if (!(djj > 0.0) || !isfinite(djj)) {
      fail = true;
      break;
    }
    const double rjj = sqrt(djj);
    const double rl = lane > j ? g[j] / rjj : (lane == j ? rjj : 0.0);
    g[j] = rl;
    rb[j * kCsL + lane] = rl;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
    for (int i = j + 1; i < kCsB; ++i) g[i] -= rb[j * kCsL + i] * rl;
  }
  if (fail) {
    if (lane == 0) *bad = 1;
    return;
  }
  if (lane < m)
#pragma unroll
    for (int i = 0; i < kCsB; ++i)
      if (i < m && i <= lane) W[(int64_t)(r0 + i) * np + r0 + lane] = g[i];
}

// (b) Block row kb: R_kk^T x = W[r0 : r0 + m, c] for the columns c >= r0 + m
// (those of A past the block, then the right-hand sides), one workgroup per 64
// columns, R_kk and the columns in LDS.  Sixteen rows at a time: the four
// waves subtract the rows solved before (four rows each, a column per lane),
// then one wave solves the 16 x 16 triangle (finite_quotient(); by divisions if
// something is not finite).
__global__ __launch_bounds__(kCsT) void k_chol_row(int n, int nc, int np, int kb,
                                                   double *__restrict__ W,
                                                   const int *__restrict__ bad) {
  __shared__ __align__(16) double dk[kCsB * kCsB];
  __shared__ double xs[kCsB * kCsB];
  if (*bad) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r0 = kCsB * kb, m = min(kCsB, n - r0);
  const int c = r0 + m + 64 * blockIdx.x + lane;
#pragma unroll
  for (int u = 0; u < kCsB / 4; ++u) {
    const int i = 4 * u + wave;
    dk[i * kCsB + lane] = (i < m && lane < m) ? (i <= lane ? W[(int64_t)(r0 + i) * np + r0 + lane] : 0.0)
                                              : (i == lane ? 1.0 : 0.0);
    xs[i * kCsB + lane] = (i < m && c < nc) ? W[(int64_t)(r0 + i) * np + c] : 0.0;
  }
  __syncthreads();
  for (int jb = 0; jb < kCsB; jb += 16) {
    const int j0 = jb + 4 * wave;
    double w4[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) w4[r] = xs[(j0 + r) * kCsB + lane];
#pragma unroll 8
    for (int q = 0; q < jb; ++q) {
      const double xq = xs[q * kCsB + lane];
#pragma unroll
      for (int r = 0; r < 4; ++r) w4[r] -= dk[q * kCsB + j0 + r] * xq;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) xs[(j0 + r) * kCsB + lane] = w4[r];
    __syncthreads();
    if (wave == 0) {
      double w[16];
      auto solve = [&](auto divide) {
        bool finite = true;
#pragma unroll
        for (int r = 0; r < 16; ++r) w[r] = xs[(jb + r) * kCsB + lane];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          w[i] = divide(w[i], dk[(jb + i) * kCsB + jb + i]);
          finite &= isfinite(w[i]);
#pragma unroll
          for (int r = i + 1; r < 16; ++r) w[r] -= dk[(jb + i) * kCsB + jb + r] * w[i];
        }
        return __all(finite);
      };
      if (!solve([](double a, double b) { return finite_quotient(a, b, 1.0 / b); }))
        solve([](double a, double b) { return a / b; });
#pragma unroll
      for (int r = 0; r < 16; ++r) xs[(jb + r) * kCsB + lane] = w[r];
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < kCsB / 4; ++u) {
    const int i = 4 * u + wave;
    if (c < nc && i < m) W[(int64_t)(r0 + i) * np + c] = xs[i * kCsB + lane];
  }
}

// (c) Trailing update W[i][c] -= sum_t R[r0 + t][i] R[r0 + t][c] for r0 + 64 <=
// i < n, i <= c < nc: one workgroup per 64 x 64 block (block column x, block
// row y <= x), its two panels staged in LDS, 16 x 16 x 4 products, wave w
// forming tile row w of the block.  Only whole blocks have a trailing part.
__global__ __launch_bounds__(kCsT) void k_chol_update(int n, int nc, int np, int kb,
                                                      double *__restrict__ W,
                                                      const int *__restrict__ bad) {
  __shared__ double pi[kCsB * kCsB];
  __shared__ double pc[kCsB * kCsB];
  if (blockIdx.y > blockIdx.x || *bad) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int r0 = kCsB * kb;
  const int ic = r0 + kCsB + 64 * blockIdx.y, cc = r0 + kCsB + 64 * blockIdx.x;
  for (int t = tid; t < kCsB * kCsB; t += kCsT) {
    const int tt = t >> 6, j = t & 63;
    const double *row = W + (int64_t)(r0 + tt) * np;
    pi[t] = ic + j < nc ? row[ic + j] : 0.0;
    pc[t] = cc + j < nc ? row[cc + j] : 0.0;
  }
  __syncthreads();
  v4d acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int t = 0; t < kCsB; t += 4) {
    const double a = pi[(t + lk) * kCsB + 16 * wave + li];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = mma64w(a, pc[(t + lk) * kCsB + 16 * j + li], acc[j]);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = ic + 16 * wave + lk + 4 * r, c = cc + 16 * j + li;
      if (i < n && i <= c && c < nc) W[(int64_t)i * np + c] -= acc[j][r];
    }
}

// (d) R1 x = y (y in columns n .. of W), and for rand_cholQR (fact non-null: R0
// on and above the diagonal of the k2 x n QR factors, ld ldf) x = R0^{-1} x.
// After a breakdown: X = NaN and MS_ERR_SINGULAR.
__global__ __launch_bounds__(kCbT) void k_chol_back(int n, int nrhs, int np,
                                                    const double *__restrict__ W,
                                                    const double *__restrict__ fact, int64_t ldf,
                                                    double *__restrict__ X, int64_t ldx,
                                                    const int *__restrict__ bad, int *status) {
  __shared__ double zs[16 * 256];
  __shared__ double ub[kCsB * kCsL];
  __shared__ double ps[kCbT];
  const int tid = threadIdx.x;
  if (*bad) {
    for (int t = tid; t < n * nrhs; t += kCbT) {
      const int c = t / n, i = t - c * n;
      X[i + (int64_t)c * ldx] = __longlong_as_double(0x7ff8000000000000LL);
    }
    if (tid == 0) record_status(status, MS_ERR_SINGULAR);
    return;
  }
  for (int t = tid; t < 256 * nrhs; t += kCbT) {
    const int c = t >> 8, i = t & 255;
    zs[t] = i < n ? W[(int64_t)i * np + n + c] : 0.0;
  }
  __syncthreads();
  back_solve(TriRef{W, np, true}, n, nrhs, zs, ub, ps);
  if (fact) back_solve(TriRef{fact, ldf, false}, n, nrhs, zs, ub, ps);
  for (int t = tid; t < n * nrhs; t += kCbT) {
    const int c = t / n, i = t - c * n;
    X[i + (int64_t)c * ldx] = zs[c * 256 + i];
  }
}

// Column j of the optional output R: R1, or R1 R0 for rand_cholQR, zeros below
// the diagonal (nothing after a breakdown).
__global__ void k_chol_rout(int n, int np, const double *__restrict__ W,
                            const double *__restrict__ fact, int64_t ldf,
                            double *__restrict__ Rout, int64_t ldr, const int *__restrict__ bad) {
  if (*bad) return;
  const int j = blockIdx.x;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    double v = 0.0;
    if (i <= j) {
      if (fact)
        for (int q = i; q <= j; ++q) v += W[(int64_t)i * np + q] * fact[q + (int64_t)j * ldf];
      else
        v = W[(int64_t)i * np + j];
    }
    Rout[i + (int64_t)j * ldr] = v;
  }
}

int wide_nt(int nc) { return (nc + 15) / 16; }

}  // namespace

// Workgroups of the wide Gram pass: one per compute unit, each with at least
// four slabs, so that writing and adding a workgroup's tiles (2 KB each) stays
// below the time of its products.
//
// Those partials are up to 80 MB (256 columns).  Lean: as many workgroups as
// find room in the partials of a task per wave, which workspaces that callers
// keep may have been sized for: np x np doubles for each of the chunks that
// give 2 x CUs tasks of 2 x 4 tiles, rounded up to the dies, at least 64 slabs
// of 16 rows in each (9 to 17 MB).  np x np doubles hold at least one
// workgroup's tiles, so there is always room.
int gram_wide_chunks(int64_t d, int nc, bool lean) {
  const int NT = wide_nt(nc);
  const GramShape g = gram_shape(NT);
  const int64_t nslab = (d + 16 * g.groups - 1) / (16 * g.groups);
  int64_t c = std::min<int64_t>(dev_info().cus, nslab / 4);
  if (lean) {
    const DevInfo &di = dev_info();
    const int xcds = std::max(1, di.xcds);
    int ntasks = 0;
    for (int a = 0; a < NT; a += 2) ntasks += (NT - a + 3) / 4;
    int64_t m = std::max<int64_t>(1, 2 * di.cus / ntasks);
    m = std::min<int64_t>(m, std::max<int64_t>(1, (d + 15) / 16 / 64));
    m = std::min<int64_t>((m + xcds - 1) / xcds * xcds, 4096);
    c = std::min<int64_t>(c, m * NT * NT / (g.groups * g.ntiles));
  }
  return (int)std::max<int64_t>(1, c);
}

size_t gram_wide_partial_bytes(int64_t d, int nc, bool lean) {
  const GramShape g = gram_shape(wide_nt(nc));
  return (size_t)gram_wide_chunks(d, nc, lean) * g.groups * g.ntiles * 256 * sizeof(double);
}

size_t gram_wide_w_bytes(int nc) {
  const int np = 16 * wide_nt(nc);
  return (size_t)np * np * sizeof(double);
}

template <typename TX, typename TB, int NT>
static hipError_t launch_gram_nt(int64_t d, const TX *X, int64_t ldx, const TB *B, int64_t ldb,
                                 int nx, int nc, int nchunks, double *part, hipStream_t st) {
  constexpr GramShape g = gram_shape(NT);
  static_assert(g.tpw <= 20, "accumulator registers");
  constexpr size_t lds = (size_t)2 * g.groups * NT * 2048;
  static_assert(lds <= 160 * 1024, "two slabs in LDS");
  if (lds > (size_t)dev_info().lds_per_block) return hipErrorInvalidValue;
  hipError_t e = allow_dynamic_lds((const void *)k_gram_wide<TX, TB, NT>, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_gram_wide<TX, TB, NT>), dim3((unsigned)nchunks), dim3(kGwT), lds, st, d, X,
                     ldx, B, ldb, nx, nc, nchunks, part);
  return hipGetLastError();
}

template <typename TX, typename TB>
hipError_t launch_gram_wide(int64_t d, int nx, int nc, const TX *X, int64_t ldx, const TB *B,
                            int64_t ldb, int nchunks, double *part, double *W, hipStream_t st) {
  if (nc < 1 || nc > kWideMaxCols || nx < 0 || nx > nc) return hipErrorInvalidValue;
  const int NT = wide_nt(nc), np = 16 * NT;
  const GramShape g = gram_shape(NT);
  hipError_t e = hipErrorInvalidValue;
  // (up to 64 columns the fused pass of randcholqr.hip is taken: n > 64 or
  // n + nrhs > 80 here, at least five tile columns)
  switch (NT) {
#define MS_GRAM_NT(N_) \
    case N_: e = launch_gram_nt<TX, TB, N_>(d, X, ldx, B, ldb, nx, nc, nchunks, part, st); break;
    MS_GRAM_NT(5) MS_GRAM_NT(6) MS_GRAM_NT(7) MS_GRAM_NT(8) MS_GRAM_NT(9) MS_GRAM_NT(10)
    MS_GRAM_NT(11) MS_GRAM_NT(12) MS_GRAM_NT(13) MS_GRAM_NT(14) MS_GRAM_NT(15) MS_GRAM_NT(16)
    MS_GRAM_NT(17)
#undef MS_GRAM_NT
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_gram_wide_reduce, dim3((unsigned)(4 * g.ntiles)), dim3(kGrT), 0, st,
                     nchunks * g.groups, NT, np, (const double *)part, W);
  return hipGetLastError();
}
template hipError_t launch_gram_wide<double, double>(int64_t, int, int, const double *, int64_t,
                                                     const double *, int64_t, int, double *,
                                                     double *, hipStream_t);
template hipError_t launch_gram_wide<float, float>(int64_t, int, int, const float *, int64_t,
                                                   const float *, int64_t, int, double *,
                                                   double *, hipStream_t);
template hipError_t launch_gram_wide<double, float>(int64_t, int, int, const double *, int64_t,
                                                    const float *, int64_t, int, double *,
                                                    double *, hipStream_t);

hipError_t launch_chol_solve_wide(int n, int nrhs, int nc, double *W, const double *fact,
                                  int64_t ldf, double *X, int64_t ldx, double *R, int64_t ldr,
                                  int *bad, int *status, hipStream_t st) {
  if (n < 1 || n > kSolveN || nrhs < 0 || nrhs > 16 || n + nrhs > nc) return hipErrorInvalidValue;
  const int np = 16 * wide_nt(nc);
  const int nb = (n + kCsB - 1) / kCsB, ncu = n + nrhs;
  for (int kb = 0; kb < nb; ++kb) {
    hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(64), 0, st, n, np, kb, W, bad);
    const int rest = ncu - std::min(n, kCsB * (kb + 1));   // columns past the block
    if (rest > 0)
      hipLaunchKernelGGL(k_chol_row, dim3((unsigned)((rest + 63) / 64)), dim3(kCsT), 0, st, n, ncu,
                         np, kb, W, (const int *)bad);
    if (kb + 1 < nb) {
      const unsigned xb = (unsigned)((rest + 63) / 64), yb = (unsigned)(nb - kb - 1);
      hipLaunchKernelGGL(k_chol_update, dim3(xb, yb), dim3(kCsT), 0, st, n, ncu, np, kb, W,
                         (const int *)bad);
    }
  }
  hipLaunchKernelGGL(k_chol_back, dim3(1), dim3(kCbT), 0, st, n, nrhs, np, (const double *)W, fact,
                     ldf, X, ldx, (const int *)bad, status);
  if (R)
    hipLaunchKernelGGL(k_chol_rout, dim3((unsigned)n), dim3(256), 0, st, n, np, (const double *)W,
                       fact, ldf, R, ldr, (const int *)bad);
  return hipGetLastError();
}

}  // namespace ms
