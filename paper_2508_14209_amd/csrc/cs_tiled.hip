// cs_tiled.hip -- CountSketch Y += S [A | B] (Def. 3, Eq. (2), Alg. 2) when
// the bucket partial sums of one column do not fit in one workgroup's LDS
// (k > 16384 FP64 slots), e.g. k = 32,768 or 131,072 buckets.
//
// The buckets are split into nbt tiles of ktile buckets; tile t's partial
// sums live in the LDS of the workgroups that own tile t.  A plain tiled
// scheme lets every tile's workgroup stream every row and keep the rows of
// its tile, so each row is decoded and issues a (masked) LDS atomic nbt
// times.  Here a plan, built once per call from the rows' buckets, groups
// the rows of every block of 7680 consecutive rows by tile (a stable
// counting sort inside the block): entry = row offset in the block (13 bits)
// | bucket within the tile (15 bits) | sign bit.  Tile t's workgroup then
// visits only its own entries: it reads the entry, gathers that row's value
// from the column (the rows of an entry list ascend, so a wave's gathers fall
// in a few cache lines) and adds it to LDS.  Every element is decoded and
// added once, as in Alg. 2.
//
// What bounds it: each tile's workgroup visits nearly every line of A, so a
// line goes from its die's L2 to nbt compute units, about 18 TB/s over the chip,
// and the lines must still be in L2 when the last of them comes.  So the waves
// gather several blocks ahead without conditions (list starts, entries and values each
// four blocks apart), but a barrier every four blocks keeps them near each
// other, and few waves take a block (a wave's 64 to 256 consecutive entries share
// lines).  Before, entries and gathers were waited for in turn.
//   8,388,608 x 260 FP32, k = 131,072: 5.94 -> 4.25 ms
//   4,194,304 x 257 FP64, k = 131,072: 3.99 -> 3.59 ms
//   4,194,304 x 64, k = 65,536, with the plan: FP32 0.69 -> 0.46, FP64 0.85 -> 0.70 ms
// (Without the barrier, 16 waves to a block: 5.1, 4.1, 0.49 and 0.80 ms; two
// blocks ahead for four: 4.5, 3.7 ms; whole columns staged through LDS by every
// tile: 5.1 and 4.5 ms; a line touched ahead by one of the tiles: slower by a quarter.)
//
// Schedule: one workgroup per compute unit (the partial sums of a tile take
// up to 160 KB of LDS), workgroup g on die g % 8.  On each die the
// workgroups form groups of nbt, one per tile; a group walks a contiguous
// share of the (column, row block) space, so the nbt members read the same
// cache lines of A at about the same time through their die's L2.  A
// workgroup adds its partial sums to Y (device atomics) when its share
// leaves a column.
#include <algorithm>

#include "ms_internal.h"

namespace ms {

namespace {

constexpr int kWaves = 16;                     // per workgroup
constexpr int kRowsPerThread = 8;
constexpr int kPlanThreads = 960;
constexpr int64_t kBlk = kPlanThreads * kRowsPerThread;   // 7680 rows per plan block
constexpr int kOffBits = 13;
constexpr uint32_t kOffMask = (1u << kOffBits) - 1;
constexpr int kLbShift = kOffBits;             // bucket within the tile: bits 13..27
constexpr uint32_t kLbMask = 0x7fffu;
constexpr int64_t kMaxSlots = 20480;           // FP64 partial sums in 160 KB of LDS
constexpr int kMaxTiles = 32;                  // at least one group per die of 32 CUs
constexpr int kAhead = 4;                      // of a team's blocks: gathers in flight
static_assert(kBlk <= kOffMask + 1, "row field");

struct TileShape {
  int nbt = 0;  // 0: not applicable
  int64_t ktile = 0, nblk = 0;
};

TileShape tile_shape(int64_t d, int64_t k) {
  TileShape s;
  if (d < 1 || k <= 16384) return s;
  int64_t need = (k + kMaxSlots - 1) / kMaxSlots;
  int nbt = 2;
  while (nbt < need) nbt *= 2;
  // two bucket tiles: the untiled kernel, whose two tiles each stream every
  // row, measured faster (16,777,216 x 129 FP32, k = 32,768: 2.46 vs 4.2 ms);
  // from four tiles the per-tile entry lists win (k = 131,072: 4.3 vs 7.9 ms)
  if (nbt < 4 || nbt > kMaxTiles) return s;
  s.nbt = nbt;
  s.ktile = (k + nbt - 1) / nbt;
  s.nblk = (d + kBlk - 1) / kBlk;
  return s;
}

// Per block: the valid rows' entries, tile by tile, each tile's rows
// ascending.  boff[b*(nbt+1)+t] = first entry of tile t in the block,
// boff[b*(nbt+1)+nbt] = valid rows.  A wave holds 512 rows, 64 at a time; a
// row's rank among its wave's rows of the tile comes from the ballots of the tile's
// bits and a running count in LDS, and the waves' counts are summed once per
// block (a scan over the workgroup per tile, three barriers each, took 74 us for
// 8,388,608 rows and 8 tiles; this 51 us).
// SRC as in the LDS CountSketch: stored h and s (checked here), or packed
// codes from ms_pack_sketch.
template <bool CODE>
__global__ __launch_bounds__(kPlanThreads) void k_tile_plan(
    int64_t d, int64_t k, int64_t ktile, int nbt, int64_t nblk, const uint32_t *__restrict__ code,
    const int32_t *__restrict__ h, const int8_t *__restrict__ s, uint32_t *__restrict__ ent,
    uint16_t *__restrict__ boff, int *status) {
  constexpr int kPlanWaves = kPlanThreads / 64;
  __shared__ uint32_t cnt[kPlanWaves][kMaxTiles];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // a wave's LDS operations are carried out in order; the compiler has to keep them so
  auto in_order = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  bool bad = false;
  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const int64_t r0 = blk * kBlk;
    uint32_t w[kRowsPerThread];   // entry
    uint32_t tl[kRowsPerThread], pos[kRowsPerThread];
    bool ok[kRowsPerThread];
#pragma unroll
    for (int q = 0; q < kRowsPerThread; ++q) {
      const int rb = (wave * kRowsPerThread + q) * 64 + lane;
      const int64_t r = r0 + rb;
      ok[q] = false;
      w[q] = tl[q] = 0;
      if (r < d) {
        uint32_t b;
        uint32_t sg;
        if (CODE) {
          const uint32_t e = code[r];
          b = e & kIdxMask;
          sg = e & kSignBit;
          ok[q] = (int64_t)b < k;
        } else {
          const int32_t hb = h[r];
          const int8_t sv = s[r];
          b = (uint32_t)hb;
          sg = sv < 0 ? kSignBit : 0u;
          ok[q] = ((uint32_t)hb < (uint32_t)k) & ((sv == 1) | (sv == -1));
        }
        bad |= !ok[q];
        if (ok[q]) {
          tl[q] = b / (uint32_t)ktile;
          w[q] = (uint32_t)rb | ((b - tl[q] * (uint32_t)ktile) << kLbShift) | sg;
        }
      }
    }
    if (lane < kMaxTiles) cnt[wave][lane] = 0;
    in_order();
#pragma unroll
    for (int q = 0; q < kRowsPerThread; ++q) {
      uint64_t same = __ballot(ok[q]);   // the valid rows of this row's tile
      for (uint32_t bit = 1; bit < (uint32_t)nbt; bit <<= 1) {
        const uint64_t m = __ballot((tl[q] & bit) != 0);
        same &= tl[q] & bit ? m : ~m;
      }
      pos[q] = cnt[wave][tl[q]] + __popcll(same & ((1ull << lane) - 1));
      in_order();
      if (ok[q] && (same >> lane) == 1) cnt[wave][tl[q]] = pos[q] + 1;   // its last row
      in_order();
    }
    __syncthreads();
    if (wave == 0) {
      // lane t: the tile's rows before each wave's, then where the tile starts
      uint32_t sum = 0;
      if (lane < nbt)
        for (int v = 0; v < kPlanWaves; ++v) sum += cnt[v][lane];
      uint32_t incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      if (lane < nbt) {
        uint32_t at = incl - sum;
        boff[blk * (nbt + 1) + lane] = (uint16_t)at;
        if (lane == nbt - 1) boff[blk * (nbt + 1) + nbt] = (uint16_t)incl;
        for (int v = 0; v < kPlanWaves; ++v) {
          const uint32_t c = cnt[v][lane];
          cnt[v][lane] = at;
          at += c;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kRowsPerThread; ++q)
      if (ok[q]) ent[r0 + cnt[wave][tl[q]] + pos[q]] = w[q];
    in_order();
  }
  if (bad) record_status(status, MS_ERR_RANGE);
}

template <typename T>
__device__ __forceinline__ const T *tcol(const Cols<T> &c, int j) {
  return j < c.n_a ? c.A + (int64_t)j * c.lda : c.B + (int64_t)(j - c.n_a) * c.ldb;
}

// Add the LDS partial sums of column c (buckets t*ktile + l, l < kt) to Y and
// clear them.
template <typename T>
__device__ __forceinline__ void tiled_flush(double *acc, uint32_t kt, int64_t bbase, int c,
                                            T *__restrict__ Y, int64_t ldy) {
  __syncthreads();
  for (uint32_t l = threadIdx.x; l < kt; l += blockDim.x) {
    const double v = acc[l];
    acc[l] = 0.0;
    if (v != 0.0) unsafeAtomicAdd(&Y[bbase + l + (int64_t)c * ldy], (T)v);
  }
  __syncthreads();
}

// W waves, a team, take a block's list, 64 E consecutive entries each, and the 16 / W
// teams take turns at the blocks; what is left of a longer list goes by itself.
template <typename T, int W, int E>
__global__ __launch_bounds__(64 * kWaves) void k_cs_tiled(
    int64_t d, Cols<T> cols, int64_t k, int64_t ktile, int nbt, int64_t nblk,
    const uint32_t *__restrict__ ent, const uint16_t *__restrict__ boff, int xcds, int subs,
    T *__restrict__ Y, int64_t ldy) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double *acc = reinterpret_cast<double *>(smem_raw);
  constexpr int kTeams = kWaves / W;
  typedef uint64_t U8 __attribute__((aligned(4)));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int team = wave / W, first = (wave % W) * 64 * E + lane;   // position of the first entry
  const int g = blockIdx.x;
  const int x = g % xcds, slot = g / xcds;
  if (slot >= subs * nbt) return;
  const int t = slot % nbt, sub = slot / nbt;
  const int64_t ngroups = (int64_t)subs * xcds;
  const int64_t grp = (int64_t)sub * xcds + x;
  const int64_t bbase = (int64_t)t * ktile;
  if (bbase >= k) return;
  const uint32_t kt = (uint32_t)min(ktile, k - bbase);
  for (uint32_t l = threadIdx.x; l < kt; l += blockDim.x) acc[l] = 0.0;
  __syncthreads();
  const int64_t total = (int64_t)cols.ncols * nblk;
  int64_t u = total * grp / ngroups;
  const int64_t u1 = total * (grp + 1) / ngroups;
  auto add = [&](T a, uint32_t e) {
    atomicAdd(&acc[(e >> kLbShift) & kLbMask], (double)apply_sign(a, e));
  };
  while (u < u1) {
    const int c = (int)(u / nblk);
    const int64_t b0 = u - (int64_t)c * nblk, b1 = min(nblk, b0 + (u1 - u));
    const T *col = tcol(cols, c);
    // this team's blocks: b0 + team + kTeams i, i < nb
    const int nb = (int)((b1 - b0 - team + kTeams - 1) / kTeams);
    const int steps = (int)((b1 - b0 + kTeams - 1) / kTeams);   // the same for all teams
    const int64_t bb = min(b0 + team, b1 - 1);
    // In flight: block i + j: values and their entries; block i + j + kAhead:
    // entries; block i + j + 2 kAhead: where its list starts and ends.  Past the
    // last block the last one again, its entries not used: without conditions
    // the loads stay in flight.
    const T *pv = col + bb * kBlk;
    const uint32_t *pe = ent + bb * kBlk;
    uint32_t pr = (uint32_t)(bb * (nbt + 1)) + t;   // of boff, in elements
    T v[kAhead][E];
    uint32_t e[kAhead][E], en[kAhead][E];
    uint64_t rw[kAhead];
    int len[kAhead], lenn[kAhead], an[kAhead], as[kAhead];
    auto ranges = [&](int j, int i) {
      // the two u16 are in the eight bytes from the word that holds the first
      rw[j] = *(const __attribute__((address_space(4))) U8 *)(uintptr_t)(boff + (pr & ~1u)) >>
              (16 * (pr & 1));
      pr += i < nb - 1 ? kTeams * (nbt + 1) : 0;
    };
    auto entries = [&](int j, int i) {
      const int a = (int)(rw[j] & 0xffff), z = (int)(rw[j] >> 16 & 0xffff);
      an[j] = a;
      lenn[j] = i < nb ? z - a : 0;
#pragma unroll
      for (int q = 0; q < E; ++q)
        en[j][q] = gload(pe + (uint32_t)min(a + first + 64 * q, max(z - 1, 0)));
      pe += i < nb - 1 ? kTeams * kBlk : 0;
    };
    auto values = [&](int j, int i) {
      as[j] = an[j];
      len[j] = lenn[j];
#pragma unroll
      for (int q = 0; q < E; ++q) {
        // a copy that the compiler can't put off to the loop's end, where it
        // would wait for the load that follows into en
        asm volatile("v_mov_b32 %0, %1" : "=v"(e[j][q]) : "v"(en[j][q]));
        v[j][q] = gload(pv + (first + 64 * q < len[j] ? e[j][q] & kOffMask : 0u));
      }
      pv += i < nb - 1 ? kTeams * kBlk : 0;
    };
#pragma unroll
    for (int j = 0; j < kAhead; ++j) ranges(j, j);
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      entries(j, j);
      ranges(j, j + kAhead);
      __builtin_amdgcn_sched_barrier(0);   // in this order: the next wait is for the oldest
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      values(j, j);
      entries(j, j + kAhead);
      ranges(j, j + 2 * kAhead);
      __builtin_amdgcn_sched_barrier(0);
    }
    for (int i = 0; i < steps; i += kAhead) {
      // the teams stay near each other: the lines that a die's groups read at a
      // time fit its L2
      __builtin_amdgcn_s_barrier();
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
#pragma unroll
        for (int q = 0; q < E; ++q)
          if (first + 64 * q < len[j]) add(v[j][q], e[j][q]);
        if (len[j] > 64 * W * E) {   // uniform: the rest of a long list
          const int64_t r = (bb + (int64_t)kTeams * (i + j)) * kBlk;
          for (int p = 64 * (W * E + wave % W) + lane; p < len[j]; p += 64 * W) {
            const uint32_t ep = gload(ent + r + as[j] + p);
            add(gload(col + r + (ep & kOffMask)), ep);
          }
        }
        values(j, i + j + kAhead);
        entries(j, i + j + 2 * kAhead);
        ranges(j, i + j + 3 * kAhead);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    u += b1 - b0;
    tiled_flush<T>(acc, kt, bbase, c, Y, ldy);
  }
}

// Bytes of the entries (a multiple of 8192 rows), which the u16 list starts follow;
// the kernel reads a start in eight bytes, up to four past the last one.
size_t entry_bytes(int64_t d) { return align_up((size_t)((d + 8191) / 8192) * 8192 * 4); }

}  // namespace

size_t cs_tile_plan_bytes(int64_t d, int64_t k) {
  const TileShape s = tile_shape(d, k);
  if (!s.nbt) return 0;
  return entry_bytes(d) + align_up((size_t)s.nblk * (s.nbt + 1) * 2 + 4);
}

bool cs_tiled_supported(int64_t d, int64_t k) {
  const TileShape s = tile_shape(d, k);
  if (!s.nbt) return false;
  const DevInfo &di = dev_info();
  return di.lds_per_block >= s.ktile * 8 && di.cus % di.xcds == 0 && di.cus / di.xcds >= s.nbt;
}

hipError_t launch_tile_plan(int64_t d, int64_t k, const uint32_t *code, const int32_t *h,
                            const int8_t *s, void *plan, int *status, hipStream_t st) {
  const TileShape sh = tile_shape(d, k);
  if (!sh.nbt) return hipErrorInvalidValue;
  uint32_t *ent = static_cast<uint32_t *>(plan);
  uint16_t *boff =
      reinterpret_cast<uint16_t *>(static_cast<unsigned char *>(plan) + entry_bytes(d));
  const unsigned grid = (unsigned)std::min<int64_t>(sh.nblk, 4096);
  if (code)
    hipLaunchKernelGGL(k_tile_plan<true>, dim3(grid), dim3(kPlanThreads), 0, st, d, k, sh.ktile,
                       sh.nbt, sh.nblk, code, nullptr, nullptr, ent, boff, status);
  else
    hipLaunchKernelGGL(k_tile_plan<false>, dim3(grid), dim3(kPlanThreads), 0, st, d, k, sh.ktile,
                       sh.nbt, sh.nblk, nullptr, h, s, ent, boff, status);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_cs_tiled(int64_t d, int64_t k, const Cols<T> &c, const void *plan, T *Y,
                           int64_t ldy, hipStream_t st) {
  const TileShape sh = tile_shape(d, k);
  if (!sh.nbt) return hipErrorInvalidValue;
  if (c.ncols <= 0) return hipSuccess;
  const DevInfo &di = dev_info();
  const int xcds = di.xcds;
  const int subs = di.cus / xcds / sh.nbt;
  const size_t lds = (size_t)sh.ktile * 8;
  const uint32_t *ent = static_cast<const uint32_t *>(plan);
  const uint16_t *boff = reinterpret_cast<const uint16_t *>(
      static_cast<const unsigned char *>(plan) + entry_bytes(d));
  auto go = [&](auto kern) -> hipError_t {
    const hipError_t e = allow_dynamic_lds((const void *)kern, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(xcds * subs * sh.nbt)), dim3(64 * kWaves), lds, st, d,
                       c, k, sh.ktile, sh.nbt, sh.nblk, ent, boff, xcds, subs, Y, ldy);
    return hipGetLastError();
  };
  // 64 W E entries hold a list of kBlk / nbt on average and, with 4 and 8 tiles, 3.4 and
  // 2.2 deviations; with 16 (512 for 480 and a deviation of 21) and 32 tiles (256 for 240
  // and 15) 1.5 and one: there about one list in 15 and in 7 has a remainder, which is
  // read after the rest.  The fewer waves to a block the better (8 tiles, FP32 as
  // above: 16 waves 4.7, 8 waves 4.5, 4 waves 4.3 ms), up to four entries a lane (2 waves, 8 entries: 4.5 ms;
  // with 4 tiles all measured alike)
  switch (sh.nbt) {
    case 4: return go(k_cs_tiled<T, 16, 2>);
    case 8: return go(k_cs_tiled<T, 4, 4>);
    case 16: return go(k_cs_tiled<T, 4, 2>);
    default: return go(k_cs_tiled<T, 2, 2>);
  }
}
template hipError_t launch_cs_tiled<double>(int64_t, int64_t, const Cols<double> &, const void *,
                                            double *, int64_t, hipStream_t);
template hipError_t launch_cs_tiled<float>(int64_t, int64_t, const Cols<float> &, const void *,
                                           float *, int64_t, hipStream_t);

}  // namespace ms
