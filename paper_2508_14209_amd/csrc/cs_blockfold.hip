// cs_blockfold.hip -- the deterministic CountSketch (MS_CS_SORTED): every
// bucket sum of Y = C [A | B] (Def. 3, Eq. (2)) folded from +0.0 in ascending
// row order, bit-identical to the sequential loop over the rows of Alg. 2.
//
// Keys (one pass, per block of 4096 rows): each row of the block as the key
// bucket << 12 | row within the block | sign << 31, the block's keys sorted by
// (bucket, row) in LDS with a bitonic network and stored in that order.  A row
// whose bucket is outside [0, k) or whose sign is not +-1 is reported and
// keyed past every bucket.
//
// Fold: one workgroup per (column, bucket range) walks the blocks in order
// with its buckets' sums resident in LDS.  Per block it stages the column's
// 4096 values and the block's sorted keys in LDS (both loaded into registers
// one block ahead, with coalesced loads), and every run of equal buckets in
// the block is folded by one thread, in ascending row order, into that
// bucket's sum.  Per bucket the additions therefore happen in ascending row
// order over the whole column -- the order of the sequential loop -- while A
// is read in its stored order instead of gathered in bucket order.
//
// Where a thread can own whole buckets (32 to 16384 buckets, up to about 128
// columns) the sorted rows are stored as 16-bit entries grouped by fold thread,
// and every thread walks the entries of its own buckets with their sums in
// registers (k_bf_fold_sliced).
#include <algorithm>
#include <type_traits>

#include "ms_internal.h"

namespace ms {

namespace {

typedef uint32_t bf_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t bf_u32x2 __attribute__((ext_vector_type(2)));

constexpr int kBfRows = 4096;               // rows per block (12 bits of the key)
constexpr int kBfT = 1024;                  // threads
constexpr uint32_t kBfKeyMask = 0x7fffffffu;  // the (bucket, row) part of a key
constexpr uint32_t kBfPad = 0x7fffffffu;    // sorts last; its bucket field exceeds every k
constexpr int64_t kBfMaxK = (int64_t)1 << 19;  // bucket field: bits 12..30
constexpr int kBfMaxParts = 32;
static_assert(kBfRows == 4096 && kBfT == 1024, "the key sort (sort4096_lds) takes 4096 keys on 1024 threads");

__device__ __forceinline__ uint32_t bf_bucket(uint32_t key) { return (key & kBfKeyMask) >> 12; }

// Thread t keys rows 4t .. 4t + 3 of the block (q = row within the block):
// one 16-byte load of h and one 4-byte load of s when the four rows exist
// and the arrays are aligned for it (vec), else four guarded loads.
__device__ __forceinline__ void bf_make_keys(int64_t d, int64_t k, const int32_t *__restrict__ h,
                                             const int8_t *__restrict__ s, int64_t r0, bool vec,
                                             uint32_t (&v)[4], bool &bad) {
  const int q0 = 4 * threadIdx.x;
  const int64_t i0 = r0 + q0;
  int32_t m[4];
  int8_t sg[4];
  if (vec && i0 + 4 <= d) {
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    const i32x4 hm = gload(reinterpret_cast<const i32x4 *>(h + i0));
    const int sw = gload(reinterpret_cast<const int *>(s + i0));
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = hm[e];
#pragma unroll
    for (int e = 0; e < 4; ++e) sg[e] = (int8_t)(sw >> (8 * e));
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = i0 + e < d;
      m[e] = in ? gload(h + i0 + e) : -1;
      sg[e] = in ? gload(s + i0 + e) : (int8_t)1;
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t kv = kBfPad;
    if (i0 + e < d) {
      const bool ok = ((int64_t)(uint32_t)m[e] < k) & (m[e] >= 0) & ((sg[e] == 1) | (sg[e] == -1));
      bad |= !ok;
      if (ok) kv = ((uint32_t)m[e] << 12) | (uint32_t)(q0 + e) | (sg[e] < 0 ? kSignBit : 0u);
    }
    v[e] = kv;
  }
}

__global__ __launch_bounds__(kBfT) void k_bf_keys(int64_t d, int k, const int32_t *__restrict__ h,
                                                  const int8_t *__restrict__ s,
                                                  uint32_t *__restrict__ keys, int *status) {
  __shared__ __align__(16) uint32_t key[kBfRows];
  const int64_t r0 = (int64_t)blockIdx.x * kBfRows;
  const bool vec = (((uintptr_t)h & 15) | ((uintptr_t)s & 3)) == 0;
  bool bad = false;
  uint32_t v[4];
  bf_make_keys(d, k, h, s, r0, vec, v, bad);
  if (bad) record_status(status, MS_ERR_RANGE);
  // sort the 4096 keys by their (bucket, row) part, store them from registers
  sort4096_regs(v, key);
  *reinterpret_cast<uint4 *>(keys + r0 + 4 * threadIdx.x) = make_uint4(v[0], v[1], v[2], v[3]);
}

// The same keys for k <= kBfCountMaxK, sorted by counting instead of by a
// network: bucket counts in LDS (the padding keys counted as bucket k), an
// exclusive scan, each key placed at its bucket's next free slot (an LDS
// atomic, so equal buckets land in arrival order), then every bucket's few
// keys put in row order by one thread (insertion sort), which makes the
// result the same ascending (bucket, row) order as the network's.  A block
// with a bucket of more than kBfCountMaxRun rows falls back to the network.
constexpr int kBfCountMaxK = 16384;
constexpr int kBfCountMaxRun = 64;

// Sliced keys (cs_blockfold_sliced): the buckets in at most 4096
// slices of B consecutive buckets (B a power of two up to 4), each folded by
// one thread.  A block is stored, in the 16 KB its 32-bit keys would take, as
// 4096 16-bit entries in (bucket, row) order -- bucket within its slice |
// row << 3 | sign << 15 -- followed by the slices' end positions (16 bits each).
// A block in which one bucket has many more rows than the average keeps its 32-bit
// keys, for bf_fold_uneven, whose threads share out positions: the walk of a slice is
// a serial chain.  Bit 30 of the first word of the block's second half tells: clear in two
// end positions, set in such a block's key there (kBfPad has it set).
constexpr int kBfSlices = 4096;
constexpr int kBfSliceMinK = 32;
constexpr uint32_t kBfUneven = 0x40000000u;
constexpr int bf_slice_buckets(int64_t k) {
  return k <= kBfSlices ? 1 : k <= 2 * kBfSlices ? 2 : 4;
}
// The most rows of a bucket in a block that is walked; uniformly hashed rows exceed it in
// about one block in ten thousand.
__device__ __forceinline__ uint32_t bf_even_rows(int k) {
  return 2 * (kBfRows / k) + (k <= kBfSlices ? 14 : k <= 2 * kBfSlices ? 11 : 8);
}

size_t bf_count_lds(int64_t k) { return (size_t)(k + 1 + 3) / 4 * 16 + (size_t)kBfRows * 4; }

template <bool SLICED>
__global__ __launch_bounds__(kBfT) void k_bf_keys_count(int64_t d, int k,
                                                        const int32_t *__restrict__ h,
                                                        const int8_t *__restrict__ s,
                                                        uint32_t *__restrict__ keys, int *status,
                                                        int *uneven) {
  extern __shared__ __align__(16) uint32_t bsm[];
  __shared__ uint32_t wsum[kBfT / 64];
  __shared__ int s_long, s_uneven;
  uint32_t *cnt = bsm;                              // k + 1 counters
  uint32_t *key = bsm + (k + 1 + 3) / 4 * 4;        // kBfRows keys, 16-byte aligned
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kBfRows;
  const bool vec = (((uintptr_t)h & 15) | ((uintptr_t)s & 3)) == 0;
  for (int m = tid; m <= k; m += kBfT) cnt[m] = 0;
  if (tid == 0) s_long = s_uneven = 0;
  bool bad = false;
  uint32_t v[4];
  bf_make_keys(d, k, h, s, r0, vec, v, bad);
  if (bad) record_status(status, MS_ERR_RANGE);
  auto bucket_of = [&](uint32_t kv) { return min(bf_bucket(kv), (uint32_t)k); };
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 4; ++e) atomicAdd(&cnt[bucket_of(v[e])], 1u);
  __syncthreads();
  // exclusive scan of the k + 1 counts, thread t owning a contiguous range
  const int per = (k + 1 + kBfT - 1) / kBfT;
  uint32_t loc = 0, most = 0;
  for (int q = 0; q < per; ++q) {
    const int m = tid * per + q;
    if (m <= k) {
      const uint32_t n = cnt[m];
      loc += n;
      most = max(most, m < k ? n : 0u);
    }
  }
  if (most > (uint32_t)kBfCountMaxRun) s_long = 1;
  if (SLICED && most > bf_even_rows(k)) s_uneven = 1;
  uint32_t incl = loc;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  const bool longrun = s_long != 0;
  // thread t's sorted keys 4t .. 4t + 3, as keys or as 16-bit entries
  const int nb = SLICED ? bf_slice_buckets(k) : 1;
  const bool sliced = SLICED && !s_uneven;
  if (SLICED && !sliced && tid == 0) *uneven = 1;
  auto store = [&]() {
    if (sliced) {
      uint32_t e[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        e[q] = (bf_bucket(v[q]) & (uint32_t)(nb - 1)) | (v[q] & 0xfffu) << 3 | (v[q] >> 31) << 15;
      *reinterpret_cast<uint2 *>(keys + r0 + 2 * tid) = make_uint2(e[0] | e[1] << 16, e[2] | e[3] << 16);
    } else {
      if (SLICED && tid == kBfRows / 2 / 4) v[0] |= kBfUneven;
      *reinterpret_cast<uint4 *>(keys + r0 + 4 * tid) = make_uint4(v[0], v[1], v[2], v[3]);
    }
  };
  uint16_t *ends = reinterpret_cast<uint16_t *>(keys + r0 + kBfRows / 2);
  if (longrun && !SLICED) {
    // a bucket too long for the insertion sort: the network
    sort4096_regs(v, key);
    store();
    return;
  }
  uint32_t run = incl - loc;
  for (int u = 0; u < w; ++u) run += wsum[u];
  for (int q = 0; q < per; ++q) {
    const int m = tid * per + q;
    if (m <= k) {
      const uint32_t c = cnt[m];
      cnt[m] = run;
      run += c;
    }
  }
  __syncthreads();
  if (SLICED) {
    // a slice ends where the next one's first bucket starts (cnt[k]: the padding)
    if (sliced)
      for (int sl = tid; sl * nb < k; sl += kBfT) ends[sl] = (uint16_t)cnt[min((sl + 1) * nb, k)];
    if (longrun) {
      sort4096_regs(v, key);
      store();
      return;
    }
    __syncthreads();   // cnt is advanced below
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) key[atomicAdd(&cnt[bucket_of(v[e])], 1u)] = v[e];
  __syncthreads();
  // cnt[m] is now the end of bucket m, cnt[m - 1] its start
  for (int m = tid; m < k; m += kBfT) {
    const uint32_t b1 = cnt[m], b0 = m > 0 ? cnt[m - 1] : 0u;
    for (uint32_t i = b0 + 1; i < b1; ++i) {
      const uint32_t x = key[i];
      uint32_t j = i;
      while (j > b0 && (key[j - 1] & kBfKeyMask) > (x & kBfKeyMask)) {
        key[j] = key[j - 1];
        --j;
      }
      key[j] = x;
    }
  }
  __syncthreads();
  const uint4 sorted = *reinterpret_cast<const uint4 *>(key + 4 * tid);
  v[0] = sorted.x;
  v[1] = sorted.y;
  v[2] = sorted.z;
  v[3] = sorted.w;
  store();
}

template <typename T>
__device__ __forceinline__ const T *bf_col(const Cols<T> &c, int j) {
  return j < c.n_a ? c.A + (int64_t)j * c.lda : c.B + (int64_t)(j - c.n_a) * c.ldb;
}

// Fold buckets [m0, m1) of one column col (d rows) into acc (LDS, zero on
// entry; slot m - m0) over the blocks in order; stage and lkey: LDS for one
// block's values and keys (two blocks' when DB: the next block is staged while
// the current one is folded, one barrier per block instead of two).  Thread t loads rows 4t .. 4t + 3 of a block (its
// values and keys) into registers kBfAhead blocks before the block is folded,
// so that a block's loads are in flight while the blocks before it are
// folded.  Ends with the workgroup synchronised.
constexpr int kBfAhead = 4;

template <typename T, bool DB = false>
__device__ __forceinline__ void bf_fold_column(int64_t d, const T *__restrict__ col,
                                               const uint32_t *__restrict__ keys, uint32_t m0,
                                               uint32_t m1, T *acc, T *stage, uint32_t *lkey) {
  const int tid = threadIdx.x;
  const int64_t nblk = (d + kBfRows - 1) / kBfRows;
  typedef T T4 __attribute__((ext_vector_type(4)));
  T4 v[kBfAhead];
  bf_u32x4 kv[kBfAhead];
  // the column's 4-row groups are vector-aligned when its start is
  const bool vec = ((uintptr_t)col & (4 * sizeof(T) - 1)) == 0;
  // block b (past the last block: the last one again, never used) into set j
  auto fetch = [&](int j, int64_t b) {
    const int64_t r = min(b, nblk - 1) * kBfRows + 4 * tid;
    if (vec && r + 4 <= d) {
      v[j] = gload(reinterpret_cast<const T4 *>(col + r));
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[j][q] = gload(col + min(r + q, d - 1));   // rows past d: padding keys
    }
    kv[j] = gload(reinterpret_cast<const bf_u32x4 *>(keys + r));
  };
  auto put = [&](int j, T *sg, uint32_t *kg) {
    *reinterpret_cast<T4 *>(sg + 4 * tid) = v[j];
    *reinterpret_cast<bf_u32x4 *>(kg + 4 * tid) = kv[j];
  };
  // fold the block staged in sg (values) and kg (sorted keys)
  auto fold = [&](const T *sg, const uint32_t *kg) {
    // this thread's four positions 4t .. 4t + 3 and the key before them;
    // the reads of all four runs' sums and first values are issued
    // together, a run inside the four positions is folded in registers,
    // and a run that goes on past them continues from LDS
    const int p0 = 4 * tid;
    const bf_u32x4 k4 = *reinterpret_cast<const bf_u32x4 *>(kg + p0);
    const uint32_t kprev = p0 > 0 ? kg[p0 - 1] : kBfPad;
    uint32_t kq[5] = {kprev, k4[0], k4[1], k4[2], k4[3]};
    bool start[4];
    uint32_t mq[4];
    T a[4], x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      mq[q] = bf_bucket(kq[q + 1]);
      start[q] = mq[q] >= m0 && mq[q] < m1 && bf_bucket(kq[q]) != mq[q];
      a[q] = start[q] ? acc[mq[q] - m0] : T(0);
      x[q] = start[q] ? sg[kq[q + 1] & (kBfRows - 1)] : T(0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (!start[q]) continue;
      T s = a[q] + apply_sign(x[q], kq[q + 1]);
      // the run's next rows among this thread's positions (static indices)
      bool more = true;
#pragma unroll
      for (int r = q + 1; r < 4; ++r) {
        if (more && bf_bucket(kq[r + 1]) == mq[q])
          s = s + apply_sign(sg[kq[r + 1] & (kBfRows - 1)], kq[r + 1]);
        else
          more = false;
      }
      if (more) {   // the run may go on into the next threads' positions
        // four keys per LDS read; their values are read together once the
        // first of them is known to continue the run, then added in order
        for (int g = p0 + 4; g < kBfRows; g += 4) {
          const bf_u32x4 kn = *reinterpret_cast<const bf_u32x4 *>(kg + g);
          if (bf_bucket(kn[0]) != mq[q]) break;
          T xn[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) xn[e] = sg[kn[e] & (kBfRows - 1)];
          bool cont = true;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (cont && bf_bucket(kn[e]) == mq[q])
              s = s + apply_sign(xn[e], kn[e]);
            else
              cont = false;
          }
          if (!cont) break;
        }
      }
      acc[mq[q] - m0] = s;
    }
  };
#pragma unroll
  for (int j = 0; j < kBfAhead; ++j) fetch(j, j);
  if constexpr (DB) {
    // two staging buffers: block b + 1 is written while block b is folded,
    // one barrier per block (the folds of consecutive blocks stay ordered)
    put(0, stage, lkey);
    fetch(0, kBfAhead);
    __syncthreads();   // acc cleared, block 0 staged
    for (int64_t b0 = 0; b0 < nblk; b0 += kBfAhead) {
#pragma unroll
      for (int j = 0; j < kBfAhead; ++j) {
        const int64_t b = b0 + j;
        if (b >= nblk) break;
        const int cur = (int)(b & 1);
        if (b + 1 < nblk) {
          const int jn = (j + 1) % kBfAhead;
          put(jn, stage + (cur ^ 1) * kBfRows, lkey + (cur ^ 1) * kBfRows);
          fetch(jn, b + 1 + kBfAhead);
        }
        fold(stage + cur * kBfRows, lkey + cur * kBfRows);
        __syncthreads();   // this block folded, the next one staged
      }
    }
    return;
  }
  for (int64_t b0 = 0; b0 < nblk; b0 += kBfAhead) {
#pragma unroll
    for (int j = 0; j < kBfAhead; ++j) {
      const int64_t b = b0 + j;
      if (b >= nblk) break;
      __syncthreads();   // acc cleared, or the previous block's runs done with stage and lkey
      put(j, stage, lkey);
      __syncthreads();
      fetch(j, b + kBfAhead);   // in flight while this block and the next ones are folded
      fold(stage, lkey);
    }
  }
  __syncthreads();
}

// Workgroup (column c, part p) owns buckets [m0, m1) of column c.
template <typename T, bool DB>
__global__ __launch_bounds__(kBfT) void k_bf_fold(int64_t d, int k, Cols<T> cols, int parts,
                                                  int slots, const uint32_t *__restrict__ keys,
                                                  T *__restrict__ Y, int64_t ldy) {
  constexpr int NB = DB ? 2 : 1;   // staging buffers
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T *acc = reinterpret_cast<T *>(smem_raw);                           // slots
  T *stage = acc + slots;                                             // NB kBfRows
  uint32_t *lkey = reinterpret_cast<uint32_t *>(stage + NB * kBfRows);  // NB kBfRows
  const int tid = threadIdx.x;
  const int c = blockIdx.x / parts, part = blockIdx.x - (blockIdx.x / parts) * parts;
  const uint32_t m0 = (uint32_t)((int64_t)k * part / parts);
  const uint32_t m1 = (uint32_t)((int64_t)k * (part + 1) / parts);
  for (uint32_t i = tid; i < m1 - m0; i += kBfT) acc[i] = T(0);
  bf_fold_column<T, DB>(d, bf_col(cols, c), keys, m0, m1, acc, stage, lkey);
  for (uint32_t i = tid; i < m1 - m0; i += kBfT) Y[(m0 + i) + (int64_t)c * ldy] = acc[i];
}

// The fold of sliced keys: workgroup (column c, part p) -- the parts of a column
// on one die, whose L2 fetches the column once -- owns slices [s0, s1) of column
// c, thread t the slices s0 + t + 1024 n (n < NS) with their B sums each
// in registers.  The column's 4096 values of a block and its entries are
// staged in LDS (two buffers, one barrier per block, loads in flight kSlAhead
// blocks ahead); a thread then walks its entries, gathering each one's value
// from LDS while the entry after it is read.
// Bound by what one compute unit reads from its L2 (every part reads the whole
// column, about 30 bytes a cycle: 1.0 of the 1.4 ms below) and then by the walk,
// in which a wave takes as many steps as the longest of its 64 slices (4 to 5
// where they average one).  4,194,304 x 65 FP64, k = 8192, the keys included: 1.41 ms against
// 2.09 for bf_fold_column, whose threads own positions instead (every thread
// looks at every position of its four, reads and writes the sums in LDS).
// Uneven blocks leave that loop (their second halves in flight with the rest cost the even
// ones a tenth): they, and even ones until kSlCalm follow each other, are staged one block
// ahead and folded with the sums in LDS.  1,000,003 x 65 FP64, k = 16,384, 64 rows in a row
// to a bucket: 0.79 ms, 2.9 walked, 0.85 by bf_fold_column.  The loop looks for uneven blocks only
// where the keys' pass met one (*uneven): looking costs it 2 to 3 % (1.42 and 1.44 ms).
constexpr int kSlAhead = 4, kSlCalm = 8;

// An uneven block, staged in sg (values) and kg (sorted keys), into acc (slot m - m0 of
// buckets m0 <= m < m1): as in bf_fold_column the thread at whose position a run starts
// folds it, four rows at a time.
template <typename T>
__device__ __forceinline__ void bf_fold_uneven(const T *sg, const uint32_t *kg, uint32_t m0,
                                               uint32_t m1, T *acc) {
  const int p0 = 4 * threadIdx.x;
  uint32_t kp = p0 > 0 ? kg[p0 - 1] : kBfPad;
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
    const uint32_t kv = kg[p0 + q], m = bf_bucket(kv), before = bf_bucket(kp);
    kp = kv;
    if (m < m0 || m >= m1 || m == before) continue;
    T s = acc[m - m0] + apply_sign(sg[kv & (kBfRows - 1)], kv);
    int g = p0 + q + 1;
    auto one = [&]() {   // row g, if the run goes on
      const uint32_t kn = g < kBfRows ? kg[g] : kBfPad;
      if (bf_bucket(kn) != m) return false;
      s = s + apply_sign(sg[kn & (kBfRows - 1)], kn);
      ++g;
      return true;
    };
    bool on = true;
    while (on && (g & 3)) on = one();
    while (on && g < kBfRows) {
      const bf_u32x4 kn = *reinterpret_cast<const bf_u32x4 *>(kg + g);
      T xn[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) xn[e] = sg[kn[e] & (kBfRows - 1)];
      on = bf_bucket(kn[3]) == m;   // (sorted: then all four)
      if (!on) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) s = s + apply_sign(xn[e], kn[e]);
      g += 4;
    }
    while (one()) {
    }
    acc[m - m0] = s;
  }
}

template <typename T, int B, int NS>
__global__ __launch_bounds__(kBfT) void k_bf_fold_sliced(int64_t d, int k, Cols<T> cols, int parts,
                                                         int xcds,
                                                         const uint32_t *__restrict__ keys,
                                                         const int *__restrict__ uneven,
                                                         T *__restrict__ Y, int64_t ldy) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  // (the entries first: the one past a buffer's end is read, not used)
  uint16_t *lent = reinterpret_cast<uint16_t *>(smem_raw);   // 2 kBfRows, or one block's keys
  T *stage = reinterpret_cast<T *>(lent + 2 * kBfRows);      // 2 kBfRows
  T *lacc = stage + 2 * kBfRows;                             // NS kBfT B sums
  // thread t stages 16 bytes of values kV times, kBfT threads apart (contiguous
  // across a wave, in memory and in LDS)
  constexpr int kR = 16 / (int)sizeof(T), kV = kBfRows / kBfT / kR;
  typedef T V __attribute__((ext_vector_type(kR)));
  typedef T Va __attribute__((ext_vector_type(kR), aligned(sizeof(T))));
  const int tid = threadIdx.x;
  const int x = blockIdx.x % xcds, j0 = blockIdx.x / xcds;
  const int part = j0 % parts, c = (j0 / parts) * xcds + x;
  if (c >= cols.ncols) return;
  const int nsl = (k + B - 1) / B;
  const int s0 = (int)((int64_t)nsl * part / parts), s1 = (int)((int64_t)nsl * (part + 1) / parts);
  const T *col = bf_col(cols, c);
  const int nblk = (int)((d + kBfRows - 1) / kBfRows);
  T acc[NS][B];
  int sl[NS];
#pragma unroll
  for (int n = 0; n < NS; ++n) {
    sl[n] = min(s0 + tid + kBfT * n, s1 - 1);   // past s1: the last slice again, not stored
#pragma unroll
    for (int q = 0; q < B; ++q) acc[n][q] = T(0);
  }
  // a last block that is not whole is staged with the rows before it (the
  // last 4096 of the column), its row 0 at position `shift`: every load is
  // unconditional, so that the loads in flight can be counted exactly
  const int shift = (int)((int64_t)nblk * kBfRows - d);
  V v[kSlAhead][kV];
  bf_u32x2 ev[kSlAhead];
  uint16_t lo[kSlAhead][NS], hi[kSlAhead][NS];   // the slices' starts and ends, as loaded
  // the next block to fetch (past the last one: the last one again, not
  // used), uniform pointers advanced block by block
  const T *cb;
  const uint32_t *kb;
  int fb;
  auto values_at = [&](int b) {
    return b < nblk - 1 ? col + (int64_t)b * kBfRows : col + (d - kBfRows);
  };
  auto load_values = [&](const T *from, V (&to)[kV]) {
#pragma unroll
    for (int q = 0; q < kV; ++q)
      to[q] = *(const __attribute__((address_space(1))) Va *)(from + kR * (tid + kBfT * q));
  };
  auto put_values = [&](const V (&from)[kV], T *to) {
#pragma unroll
    for (int q = 0; q < kV; ++q) *reinterpret_cast<V *>(to + kR * (tid + kBfT * q)) = from[q];
  };
  auto fetch = [&](int j) {
    load_values(cb, v[j]);
    ev[j] = gload(reinterpret_cast<const bf_u32x2 *>(kb) + tid);
    const uint16_t *ends = reinterpret_cast<const uint16_t *>(kb + kBfRows / 2);
#pragma unroll
    for (int n = 0; n < NS; ++n) {
      lo[j][n] = gload(ends + max(sl[n] - 1, 0));
      hi[j][n] = gload(ends + sl[n]);
    }
    ++fb;
    cb = fb < nblk - 1 ? cb + kBfRows : col + (d - kBfRows);
    kb += fb < nblk ? kBfRows : 0;
  };
  auto put = [&](int j, int buf) {
    put_values(v[j], stage + buf * kBfRows);
    *reinterpret_cast<bf_u32x2 *>(lent + buf * kBfRows + 4 * tid) = ev[j];
  };
  // the entries at bytes [p, pe) of eb, added to their slice's sums; sb: the values
  auto walk = [&](const unsigned char *sb, const unsigned char *eb, uint32_t p, uint32_t pe,
                  T (&sums)[B]) {
    if (p >= pe) return;
    int e = *reinterpret_cast<const int16_t *>(eb + p);
    do {
      // this entry's value and the next entry (at the end: one not used)
      // are read together; the empty statement keeps the compiler from
      // moving the second read into the next turn, behind its use
      const uint32_t at = sizeof(T) == 8 ? (e & 0x7ff8) : ((e >> 1) & 0x3ffc);
      T xv = *reinterpret_cast<const T *>(sb + at);
      p += 2;
      int en = *reinterpret_cast<const int16_t *>(eb + p);
      asm volatile("" : "+v"(xv), "+v"(en));
      xv = apply_sign(xv, (uint32_t)e);
      // (adding +0.0 to the others keeps every bit: a sum from +0.0 is
      // never -0.0; the selects before the adds, or each waits for the one before)
      T xm[B];
#pragma unroll
      for (int m = 0; m < B; ++m) xm[m] = B == 1 || (e & (B - 1)) == m ? xv : T(0);
#pragma unroll
      for (int m = 0; m < B; ++m) sums[m] = sums[m] + xm[m];
      e = en;
    } while (p < pe);
  };
  uint16_t cl[NS], ch[NS];
  auto fold = [&](const T *sg, const uint16_t *le) {
#pragma unroll
    for (int n = 0; n < NS; ++n)
      walk(reinterpret_cast<const unsigned char *>(sg), reinterpret_cast<const unsigned char *>(le),
           sl[n] > 0 ? 2u * cl[n] : 0u, 2u * ch[n], acc[n]);
  };
  // block at's word that tells an uneven block; in lanes 0 .. 3 those of the four from at on
  auto tell = [&](int at) {
    return gload(keys + (int64_t)min(at, nblk - 1) * kBfRows + kBfRows / 2);
  };
  const int q4 = tid & 3;
  static_assert(kSlAhead == 4, "buffers and slots of the unrolled loop");
  // UNEVEN: some block of the matrix is
  auto blocks = [&](auto UNEVEN) {
    for (int b = 0; b < nblk;) {
      uint32_t word = UNEVEN ? tell(b + q4) : 0u;
      fb = b;
      cb = values_at(b);
      kb = keys + (int64_t)b * kBfRows;
#pragma unroll
      for (int j = 0; j < kSlAhead; ++j) fetch(j);
      bool odd = UNEVEN && __any(word & kBfUneven);   // one of the next four blocks
      if (!odd) {
        put(0, 0);
#pragma unroll
        for (int n = 0; n < NS; ++n) {
          cl[n] = lo[0][n];
          ch[n] = hi[0][n];
        }
        fetch(0);
        __syncthreads();
      }
      while (b < nblk && !odd) {
        if (UNEVEN) word = tell(b + kSlAhead + q4);
#pragma unroll
        for (int j = 0; j < kSlAhead; ++j) {
          if (b >= nblk) break;
          constexpr int kNext[kSlAhead] = {1, 2, 3, 0};
          const int jn = kNext[j], cur = j & 1;
          uint16_t nl[NS], nh[NS];
          put(jn, cur ^ 1);   // (after the last block: a block that is not folded)
#pragma unroll
          for (int n = 0; n < NS; ++n) {
            nl[n] = lo[jn][n];
            nh[n] = hi[jn][n];
          }
          fetch(jn);
          fold(stage + cur * kBfRows + (b + 1 < nblk ? 0 : shift), lent + cur * kBfRows);
#pragma unroll
          for (int n = 0; n < NS; ++n) {
            cl[n] = nl[n];
            ch[n] = nh[n];
          }
          __syncthreads();   // this block folded, the next one staged
          ++b;
        }
        odd = UNEVEN && __any(word & kBfUneven);
      }
      if (!UNEVEN || b >= nblk) break;
      // four blocks with an uneven one among them: the sums in LDS (slot: bucket of this part)
#pragma unroll
      for (int n = 0; n < NS; ++n)
#pragma unroll
        for (int q = 0; q < B; ++q)
          if (s0 + tid + kBfT * n < s1) lacc[(sl[n] - s0) * B + q] = acc[n][q];
      V cv[kV];
      bf_u32x4 ck;
      uint32_t ct;
      uint32_t *lkey = reinterpret_cast<uint32_t *>(lent);
      auto ahead = [&](int at) {
        ct = tell(at);
        load_values(values_at(at), cv);
        ck = gload(reinterpret_cast<const bf_u32x4 *>(keys + (int64_t)at * kBfRows) + tid);
      };
      ahead(b);
      for (int calm = 0; b < nblk && calm < kSlCalm; ++b) {
        put_values(cv, stage);
        const bool unb = (__builtin_amdgcn_readfirstlane(ct) & kBfUneven) != 0;
        if (unb && tid == kBfRows / 2 / 4 && ck[0] != kBfPad) ck[0] &= ~kBfUneven;
        *reinterpret_cast<bf_u32x4 *>(lkey + 4 * tid) = ck;
        __syncthreads();
        ahead(min(b + 1, nblk - 1));
        const T *sg = stage + (b + 1 < nblk ? 0 : shift);
        if (unb) {
          bf_fold_uneven(sg, lkey, (uint32_t)(s0 * B), (uint32_t)min(s1 * B, k), lacc);
        } else {
          const uint16_t *ends = lent + kBfRows;
#pragma unroll 1
          for (int s = s0 + tid; s < s1; s += kBfT) {
            T sums[B];
#pragma unroll
            for (int q = 0; q < B; ++q) sums[q] = lacc[(s - s0) * B + q];
            walk(reinterpret_cast<const unsigned char *>(sg),
                 reinterpret_cast<const unsigned char *>(lent), s > 0 ? 2u * ends[s - 1] : 0u,
                 2u * ends[s], sums);
#pragma unroll
            for (int q = 0; q < B; ++q) lacc[(s - s0) * B + q] = sums[q];
          }
        }
        calm = unb ? 0 : calm + 1;
        __syncthreads();
      }
#pragma unroll
      for (int n = 0; n < NS; ++n)
#pragma unroll
        for (int q = 0; q < B; ++q) acc[n][q] = lacc[(sl[n] - s0) * B + q];
    }
  };
  if (*uneven)
    blocks(std::true_type{});
  else
    blocks(std::false_type{});
#pragma unroll
  for (int n = 0; n < NS; ++n)
    if (s0 + tid + kBfT * n < s1)
#pragma unroll
      for (int q = 0; q < B; ++q) {
        const int m = sl[n] * B + q;
        if (m < k) Y[m + (int64_t)c * ldy] = acc[n][q];
      }
}

// ------------------------------------------------------------------ batched

// Persistent over every problem's key blocks: problem p's block b sorted
// into keyarea + key_off (as k_bf_keys); bad rows recorded for the problem.
__global__ __launch_bounds__(kBfT) void k_batch_bf_keys(int count, const ms_problem *__restrict__ P,
                                                        const BatchEntry *__restrict__ E,
                                                        const BatchTotals *__restrict__ tot,
                                                        unsigned char *__restrict__ keyarea,
                                                        int *pstatus, int *status) {
  __shared__ __align__(16) uint32_t key[kBfRows];
  const int tid = threadIdx.x;
  const int64_t total = tot->bk_items;
  for (int64_t it = blockIdx.x; it < total; it += gridDim.x) {
    const int p = batch_find_m<&BatchEntry::bk_start>(E, count, it);
    const ms_problem &Q = P[p];
    const BatchEntry &e = E[p];
    const int64_t r0 = (it - e.bk_start) * kBfRows;
    const int32_t *h = Q.h;
    const int8_t *s = Q.s;
    const bool vec = (((uintptr_t)h & 15) | ((uintptr_t)s & 3)) == 0;
    bool bad = false;
    uint32_t v[4];
    bf_make_keys(Q.d, Q.k, h, s, r0, vec, v, bad);
    if (bad) {
      record_status(&pstatus[p], MS_ERR_RANGE);
      record_status(status, MS_ERR_RANGE);
    }
    // the scratch is reused by the next item: the sort's first LDS phase
    // stores only each thread's own positions before its barrier
    sort4096_regs(v, key);
    uint32_t *out = reinterpret_cast<uint32_t *>(keyarea + e.key_off) + r0;
    *reinterpret_cast<uint4 *>(out + 4 * tid) = make_uint4(v[0], v[1], v[2], v[3]);
  }
}

// Persistent over fold items (problem, column, bucket part).  RES = 0:
// column c of [A | B] (data T) into the problem's Y (k x nc, T, ld k);
// RES = 1: column c of its residual r (FP64, d x nrhs, ld d) into Yr (FP64,
// k x nrhs, ld k).
template <typename T, int RES>
__global__ __launch_bounds__(kBfT) void k_batch_bf_fold(int count, const ms_problem *__restrict__ P,
                                                        const BatchEntry *__restrict__ E,
                                                        const BatchTotals *__restrict__ tot,
                                                        const unsigned char *__restrict__ keyarea,
                                                        const unsigned char *__restrict__ rarea,
                                                        unsigned char *__restrict__ out,
                                                        int slots) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T *acc = reinterpret_cast<T *>(smem_raw);
  T *stage = acc + slots;
  uint32_t *lkey = reinterpret_cast<uint32_t *>(stage + kBfRows);
  const int tid = threadIdx.x;
  const int64_t total = RES ? tot->bfr_items : tot->bf_items;
  for (int64_t it = blockIdx.x; it < total; it += gridDim.x) {
    const int p = RES ? batch_find_m<&BatchEntry::bfr_start>(E, count, it)
                      : batch_find_m<&BatchEntry::bf_start>(E, count, it);
    const ms_problem &Q = P[p];
    const BatchEntry &e = E[p];
    if (RES && !e.refine) continue;   // converged in an earlier step
    const int parts = RES ? e.rparts : e.parts;
    const int64_t local = it - (RES ? e.bfr_start : e.bf_start);
    const int c = (int)(local / parts), part = (int)(local - (local / parts) * parts);
    const uint32_t m0 = (uint32_t)(Q.k * part / parts);
    const uint32_t m1 = (uint32_t)(Q.k * (part + 1) / parts);
    const T *col;
    T *Yc;
    if (RES) {
      col = reinterpret_cast<const T *>(rarea + e.r_off) + (int64_t)c * Q.d;
      Yc = reinterpret_cast<T *>(out + e.yr_off) + (int64_t)c * Q.k;
    } else {
      col = c < Q.n ? static_cast<const T *>(Q.A) + (int64_t)c * Q.lda
                    : static_cast<const T *>(Q.B) + (int64_t)(c - Q.n) * Q.ldb;
      Yc = reinterpret_cast<T *>(out + e.y_off) + (int64_t)c * Q.k;
    }
    for (uint32_t i = tid; i < m1 - m0; i += kBfT) acc[i] = T(0);
    bf_fold_column<T>(Q.d, col, reinterpret_cast<const uint32_t *>(keyarea + e.key_off), m0, m1,
                      acc, stage, lkey);
    for (uint32_t i = tid; i < m1 - m0; i += kBfT) Yc[m0 + i] = acc[i];
    __syncthreads();   // acc is cleared by the next item
  }
}

struct BfShape {
  int parts = 0, slots = 0;
  size_t lds = 0;
};

BfShape bf_shape(int64_t k, int ncols, size_t elem, int bufs = 1) {
  BfShape s;
  if (k < 1 || k > kBfMaxK || ncols < 1) return s;
  const size_t fixed = (size_t)bufs * kBfRows * (elem + 4);
  const size_t avail = (size_t)dev_info().lds_per_block;
  if (avail <= fixed + 256 * elem) return s;
  const int64_t per = (int64_t)((avail - fixed) / elem);   // bucket sums one workgroup holds
  int parts = (int)((k + per - 1) / per);
  // spread a few columns over more workgroups (each part re-reads the column)
  const int want = std::max(1, std::min(8, 256 / std::max(1, ncols)));
  parts = std::max(parts, (int)std::min<int64_t>(want, k));
  if (parts > kBfMaxParts) return s;
  s.parts = parts;
  // a multiple of 4 slots keeps the staged keys 16-byte aligned (vector reads)
  s.slots = (int)(((k + parts - 1) / parts + 3) / 4 * 4);
  s.lds = (size_t)s.slots * elem + fixed;
  if (s.lds > avail) return BfShape{};
  return s;
}

}  // namespace

bool cs_blockfold_supported(int64_t d, int64_t k, int ncols, size_t elem) {
  return d >= 1 && d <= 0x7ffffffe && bf_shape(k, ncols, elem).parts > 0;
}

size_t cs_blockfold_key_bytes(int64_t d) {
  const int64_t nblk = (d + kBfRows - 1) / kBfRows;
  return align_up((size_t)nblk * kBfRows * 4);
}

namespace {

// Parts of a column in the fold of sliced keys (each reads all of it): as many
// as the compute units of the column's die hold at one workgroup each.
int bf_sliced_parts(int ncols) {
  const DevInfo &di = dev_info();
  const int xcds = std::max(1, di.xcds), per = std::max(1, (ncols + xcds - 1) / xcds);
  return std::max(1, std::min(16, di.cus / xcds / per));
}

// Slices of a part.
int64_t bf_sliced_own(int64_t k, int ncols) {
  const int64_t B = bf_slice_buckets(k), nsl = (k + B - 1) / B, parts = bf_sliced_parts(ncols);
  return (nsl + parts - 1) / parts;
}

}  // namespace

// Sliced keys are used where a fold thread then owns at most two slices (up
// to 128 columns, and more for few buckets): 4,194,304 x 65 FP64, k = 8192:
// 1.41 ms against 2.09 for positions; with four slices a thread (129 columns,
// k = 8192) 3.3 against 2.4.  Two slices of two or four buckets each take longer to clear,
// walk and store, and need a few blocks to make up for it: 5000 x 128, k = 16,384:
// 33.8 us against 30.7, 20,000 x 100, k = 10,000: 34 and 33, 100,003 x 128: 76 and 82; k = 8192:
// 5000 x 128 29 and 27.6, 20,000 x 128 31 and 35.  FP32 sooner: k = 16,384, 20,001 x 128 33.6 and
// 36.0, x 65 30.5 and 35.0; 5000 x 128 30.1 and 28.2.  Fewer than 32 buckets (chains of more
// than 128 rows a block) keep the keys too.
bool cs_blockfold_sliced(int64_t d, int64_t k, int64_t ncols, size_t elem) {
  if (d < kBfRows || k < kBfSliceMinK || k > kBfCountMaxK || ncols < 1 || ncols > 65535) return false;
  const int64_t B = bf_slice_buckets(k), own = bf_sliced_own(k, (int)ncols);
  return own <= kBfT || (own <= 2 * kBfT && d >= (B - 1) * (elem == 8 ? 4 : 1) * kBfRows);
}

hipError_t launch_bf_keys(int64_t d, int64_t k, const int32_t *h, const int8_t *s, uint32_t *keys,
                          bool sliced, int *status, int *uneven, hipStream_t st) {
  if (d < 1 || k < 1 || k > kBfMaxK || (sliced && k > kBfCountMaxK)) return hipErrorInvalidValue;
  const int64_t nblk = (d + kBfRows - 1) / kBfRows;
  if (k <= kBfCountMaxK) {
    const size_t lds = bf_count_lds(k);
    hipError_t e = allow_dynamic_lds(sliced ? (const void *)k_bf_keys_count<true>
                                            : (const void *)k_bf_keys_count<false>, (int)lds);
    if (e != hipSuccess) return e;
    if (sliced)
      hipLaunchKernelGGL(k_bf_keys_count<true>, dim3((unsigned)nblk), dim3(kBfT), lds, st, d,
                         (int)k, h, s, keys, status, uneven);
    else
      hipLaunchKernelGGL(k_bf_keys_count<false>, dim3((unsigned)nblk), dim3(kBfT), lds, st, d,
                         (int)k, h, s, keys, status, uneven);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_bf_keys, dim3((unsigned)nblk), dim3(kBfT), 0, st, d, (int)k, h, s, keys,
                     status);
  return hipGetLastError();
}

template <typename T, int B, int NS>
static hipError_t launch_bf_sliced(int64_t d, int64_t k, const Cols<T> &c, int parts,
                                   const uint32_t *keys, const int *uneven, T *Y, int64_t ldy,
                                   hipStream_t st) {
  constexpr size_t lds = (size_t)2 * kBfRows * (sizeof(T) + 2) + (size_t)NS * kBfT * B * sizeof(T);
  hipError_t e = allow_dynamic_lds((const void *)k_bf_fold_sliced<T, B, NS>, (int)lds);
  if (e != hipSuccess) return e;
  const int xcds = std::max(1, dev_info().xcds);
  hipLaunchKernelGGL((k_bf_fold_sliced<T, B, NS>),
                     dim3((unsigned)((c.ncols + xcds - 1) / xcds * xcds * parts)), dim3(kBfT), lds,
                     st, d, (int)k, c, parts, xcds, keys, uneven, Y, ldy);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_bf_fold(int64_t d, int64_t k, const Cols<T> &c, const uint32_t *keys,
                          bool sliced, const int *uneven, T *Y, int64_t ldy, hipStream_t st) {
  if (sliced) {
    // (the residuals' fold has fewer columns than the keys were chosen for,
    // and FP64 ones where the data may be FP32)
    if (d < kBfRows || k < kBfSliceMinK || k > kBfCountMaxK || c.ncols < 1 ||
        bf_sliced_own(k, c.ncols) > 2 * kBfT)
      return hipErrorInvalidValue;
    const int B = bf_slice_buckets(k);
    const int nsl = (int)((k + B - 1) / B);
    const int parts = std::min(bf_sliced_parts(c.ncols), nsl);
    const bool one = (nsl + parts - 1) / parts <= kBfT;   // slices per thread: 1 or 2
#define MS_SLICED(B_)                                                                          \
  if (B == B_)                                                                                 \
    return one ? launch_bf_sliced<T, B_, 1>(d, k, c, parts, keys, uneven, Y, ldy, st)          \
               : launch_bf_sliced<T, B_, 2>(d, k, c, parts, keys, uneven, Y, ldy, st);
    MS_SLICED(1) MS_SLICED(2) MS_SLICED(4)
#undef MS_SLICED
  }
  const BfShape sh = bf_shape(k, c.ncols, sizeof(T));
  if (!sh.parts) return hipErrorInvalidValue;
  // two staging buffers when they leave the same workgroup count
  const BfShape sh2 = bf_shape(k, c.ncols, sizeof(T), 2);
  const bool db = sh2.parts == sh.parts;
  const BfShape &u = db ? sh2 : sh;
  const void *fn = db ? (const void *)k_bf_fold<T, true> : (const void *)k_bf_fold<T, false>;
  hipError_t e = allow_dynamic_lds(fn, (int)u.lds);
  if (e != hipSuccess) return e;
  const int64_t grid = (int64_t)c.ncols * u.parts;
  if (db)
    hipLaunchKernelGGL((k_bf_fold<T, true>), dim3((unsigned)grid), dim3(kBfT), u.lds, st, d,
                       (int)k, c, u.parts, u.slots, keys, Y, ldy);
  else
    hipLaunchKernelGGL((k_bf_fold<T, false>), dim3((unsigned)grid), dim3(kBfT), u.lds, st, d,
                       (int)k, c, u.parts, u.slots, keys, Y, ldy);
  return hipGetLastError();
}
hipError_t launch_batch_bf_keys(int count, const ms_problem *P, const BatchEntry *E,
                                const BatchTotals *tot, unsigned char *keyarea, int *pstatus,
                                int *status, int grid, hipStream_t st) {
  hipLaunchKernelGGL(k_batch_bf_keys, dim3((unsigned)grid), dim3(kBfT), 0, st, count, P, E, tot,
                     keyarea, pstatus, status);
  return hipGetLastError();
}

template <typename T, int RES>
hipError_t launch_batch_bf_fold(int count, const ms_problem *P, const BatchEntry *E,
                                const BatchTotals *tot, const unsigned char *keyarea,
                                const unsigned char *rarea, unsigned char *out, int grid,
                                hipStream_t st) {
  const int slots = (int)batch_bf_slots((int)sizeof(T));
  const size_t lds = (size_t)slots * sizeof(T) + (size_t)kBfRows * (sizeof(T) + 4);
  if (lds > (size_t)dev_info().lds_per_block) return hipErrorInvalidValue;
  const void *fn = (const void *)k_batch_bf_fold<T, RES>;
  hipError_t e = allow_dynamic_lds(fn, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_batch_bf_fold<T, RES>), dim3((unsigned)grid), dim3(kBfT), lds, st, count,
                     P, E, tot, keyarea, rarea, out, slots);
  return hipGetLastError();
}
template hipError_t launch_batch_bf_fold<float, 0>(int, const ms_problem *, const BatchEntry *,
                                                   const BatchTotals *, const unsigned char *,
                                                   const unsigned char *, unsigned char *, int,
                                                   hipStream_t);
template hipError_t launch_batch_bf_fold<double, 0>(int, const ms_problem *, const BatchEntry *,
                                                    const BatchTotals *, const unsigned char *,
                                                    const unsigned char *, unsigned char *, int,
                                                    hipStream_t);
template hipError_t launch_batch_bf_fold<double, 1>(int, const ms_problem *, const BatchEntry *,
                                                    const BatchTotals *, const unsigned char *,
                                                    const unsigned char *, unsigned char *, int,
                                                    hipStream_t);

template hipError_t launch_bf_fold<double>(int64_t, int64_t, const Cols<double> &,
                                           const uint32_t *, bool, const int *, double *, int64_t,
                                           hipStream_t);
template hipError_t launch_bf_fold<float>(int64_t, int64_t, const Cols<float> &, const uint32_t *,
                                          bool, const int *, float *, int64_t, hipStream_t);

}  // namespace ms
