// pipad_frame_build_overlap: overlap extraction for a frame of k CSR snapshots on gfx950.
//
// Section 4.1 ("Overlap-aware data transfer") regroups the topology of a snapshot group as one
// overlap part plus one exclusive part per snapshot; Section 4.3 makes this the job of a data
// preparation module that runs once.  Here it runs on the GPU over *tiles*: the entries of the
// largest snapshot (the base) are cut into runs of 512 in (row, column) order, and a tile owns, of
// every other snapshot, the contiguous stretch of entries that lies between its first entry and the
// next tile's in that order.  Whatever is in all snapshots is therefore decided inside one tile, and
// since the overlap holds the same entries in every snapshot, ONE prefix sum (the tiles' numbers of
// common entries, C) places everything: an entry of snapshot t's exclusive part goes to its own
// position in the input minus the common entries before it, row pointers likewise.
//
//   prepare  where every tile starts in every snapshot; D^-1/2; how many rows of every 256 are mid
//            and hub rows (a row's class is decided by its longest input row alone)
//   mark     a workgroup per tile, a wave per snapshot: the base's entries are in LDS, and every other
//            snapshot walks along them with its own; one bit per base entry says whether it is common,
//            and the exclusive entries of every snapshot are written out next to each other
//   scan     prefix sums over the tiles' and the row blocks' counts; with them every data-dependent
//            size is known and goes to the host
//   rows     a thread per row, while the host sizes the outputs or next to the scatter step: row pointers of all
//            parts and the work lists of the aggregation (short, mid, hub rows; very long rows cut into units)
//   scatter  a wave per tile (or four) and part writes the entries in order, with their column scales
//   fill     the entries of the hub rows a second time, grouped by column class, with their scales
//
// Frames that are not large get room for as many entries as the parts can have, so that scatter need not wait for the sizes: rows
// and scatter are one launch there.  Small frames, whose launches take longer than their work, go in two launches altogether:
// prepare and mark (a tile finds its own bounds), then the sums, rows and scatter (every workgroup makes the sums it needs).
//
// All integer work; the outputs are unique, so they are bit-exact regardless of scheduling.
#include <algorithm>
#include <cstring>

#include "pipad_internal.h"

namespace pipad {
namespace {

struct Snaps {
  const int32_t *rowptr[PIPAD_MAX_K];
  const int32_t *col[PIPAD_MAX_K];
  int32_t nnz[PIPAD_MAX_K];
};

// What the kernels of the extraction share.
struct Tiles {
  int32_t n, k;
  int32_t base;           // the snapshot that is cut into tiles: the one with most entries
  int32_t ntiles;
  int32_t tile_log2;      // base entries per tile
  int32_t *brow;          // [ntiles + 1] row of every tile's first entry; n - 1 behind the last
  int32_t *bound;         // [k][ntiles + 1] where every tile starts in snapshot t; nnz_t at the end
  uint64_t *bits;         // a bit per base entry: it is common
  uint64_t *hub_bits;     // ... it belongs to a hub row
  uint16_t *wpre;         // per word of bits: common entries of the tile in the words before
  uint2 *tile_cnt;        // [ntiles] common entries per tile, and those in hub rows
  uint2 *tile_pre;        // [ntiles + 1] the same summed up over the tiles in front
  int32_t *excl[PIPAD_MAX_K];  // [nnz_t] columns of a tile's exclusive entries, from the tile's start on
  RowCounts *row_cnt;     // [row blocks] of every 256 rows
  RowCounts *row_pre;     // [row blocks + 1] of the rows in front
  uint32_t *bad;          // set when the snapshots turn out not to be canonical
};

// ---- validation -----------------------------------------------------------------------------
// One wave per (snapshot, row): row pointer sanity, then column range / order / diagonal.
__global__ __launch_bounds__(kBlock) void k_validate(Snaps s, int32_t n, int32_t k, int *bad) {
  const int64_t unit = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  if (unit >= (int64_t)k * n) return;
  // (one unit per wave: saying so lets the snapshot's pointers come through the scalar unit)
  const int t = __builtin_amdgcn_readfirstlane((int)(unit / n));
  const int32_t i = __builtin_amdgcn_readfirstlane((int32_t)(unit % n));
  const int32_t *rp = s.rowptr[t];
  const int32_t a = rp[i], b = rp[i + 1];
  bool ok = a >= 0 && b >= a && b <= s.nnz[t];
  if (i == 0 && a != 0) ok = false;
  if (i == n - 1 && b != s.nnz[t]) ok = false;
  if (ok) {
    const int32_t *col = s.col[t];
    for (int32_t e = a + lane; e < b; e += kWave) {
      const int32_t c = col[e];
      if (c < 0 || c >= n || c == i) ok = false;
      if (e > a && col[e - 1] >= c) ok = false;
    }
  }
  if (!ok) *bad = 1;
}

// ---- bounds ---------------------------------------------------------------------------------
// First position in col[lo, hi) (ascending) that holds c or more.
__device__ inline int32_t lower_bound(const int32_t *col, int32_t lo, int32_t hi, int32_t c) {
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if (col[mid] < c) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// The same, looking outwards from position `at` first: O(log distance) steps.
__device__ inline int32_t lower_bound_near(const int32_t *col, int32_t lo, int32_t hi, int32_t at, int32_t c) {
  if (lo >= hi) return lo;
  at = min(max(at, lo), hi - 1);
  int32_t a = lo, b = hi;  // the answer lies in [a, b]
  if (col[at] < c) {
    a = at + 1;
    for (int64_t step = 8; at + step < hi; step <<= 2) {
      if (col[at + step] >= c) {
        b = (int32_t)(at + step);
        break;
      }
      a = (int32_t)(at + step + 1);
    }
  } else {
    b = at;
    for (int64_t step = 8; at - step >= lo; step <<= 2) {
      if (col[at - step] < c) {
        a = (int32_t)(at - step + 1);
        break;
      }
      b = (int32_t)(at - step);
    }
  }
  return lower_bound(col, a, b, c);
}

struct RowClasses {  // the thresholds of the row classes
  int32_t short_max, mid_max, threshold, segment;
};

// Counts of 256 rows, a thread each, by every 256 threads of the workgroup (`out`: theirs, or null).
__device__ inline void count_rows(const RowClasses &rc, bool live, int64_t L, int64_t entries, int32_t common,
                                  RowCounts *out) {
  constexpr int W = 16;  // waves of a workgroup at most
  __shared__ uint32_t w_mid[W], w_hub[W], w_units[W], w_common[W], w_short[W], w_uncoded[W];
  __shared__ uint64_t w_all[W];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int cls = row_class(L, rc.short_max, rc.mid_max);
  const uint64_t is_mid = __ballot(live && cls == 1), is_hub = __ballot(live && cls == 2);
  const bool hub = is_hub >> lane & 1ull;
  uint32_t units = 0, shared = 0;
  uint64_t all = 0;
  if (is_hub) {
    units = hub ? hub_units(L, rc.threshold, rc.segment) : 0u;
    shared = hub ? (uint32_t)common : 0u;
    all = hub ? (uint64_t)entries : 0ull;
#pragma unroll
    for (int m = kWave >> 1; m >= 1; m >>= 1) {
      units += __shfl_xor(units, m, kWave);
      shared += __shfl_xor(shared, m, kWave);
      all += __shfl_xor(all, m, kWave);
    }
  }
  const uint32_t in_short = wave_sum(live && cls == 0 ? (uint32_t)L : 0u);
  const uint64_t uncoded = __ballot(live && L >= kUncoded - 1);
  if (lane == kWave - 1) {
    w_uncoded[wave] = (uint32_t)__popcll(uncoded);
    w_short[wave] = in_short;
    w_mid[wave] = (uint32_t)__popcll(is_mid);
    w_hub[wave] = (uint32_t)__popcll(is_hub);
    w_units[wave] = units;
    w_common[wave] = shared;
    w_all[wave] = all;
  }
  __syncthreads();
  if (threadIdx.x % kBlock == 0 && out) {
    RowCounts c = {};
#pragma unroll
    for (int u = 0; u < kWavesPerBlock; ++u) {
      const int w = wave + u;
      c.short_entries += w_short[w];
      c.uncoded += w_uncoded[w];
      c.common += w_common[w];
      c.mid += w_mid[w]; c.hub += w_hub[w]; c.units += w_units[w]; c.entries += w_all[w];
    }
    *out = c;
  }
}

// G lanes per tile boundary: they find its row together (eight, a 9-way search: seven round trips to
// memory for a million rows instead of twenty), then each of them its column in some of the
// snapshots, one after the other.  Bound: that chain of round trips; so 16 lanes for more than eight snapshots, one
// for each up to 16 (whole k_prepare: N = 103k, k = 16 22.2 -> 16.1 us, R-MAT 168k, k = 12 17.3 -> 13.0; 572k, k = 16, where
// the rows take longer, 53.6 -> 52.7; 16 for up to eight snapshots 9.0 -> 9.4).
template <int G>
__device__ inline void find_bounds(const Snaps &s, const Tiles &g, int64_t wave, int lane) {
  const int sub = lane & (G - 1), group0 = lane & ~(G - 1);
  const int64_t c64 = wave * (kWave / G) + lane / G;
  const bool search = c64 < g.ntiles;
  const int32_t c = (int32_t)min(c64, (int64_t)g.ntiles);
  const int64_t ldb = (int64_t)g.ntiles + 1;
  const int32_t *rp = s.rowptr[g.base];
  const int32_t e = search ? c << g.tile_log2 : 0;
  int32_t lo = 0, hi = search ? g.n : 1;  // rp[lo] <= e < rp[hi]
  while (__any(hi - lo > 1)) {
    const int32_t step = (int32_t)(((int64_t)hi - lo + G) / (G + 1));
    const int64_t idx = lo + (int64_t)(sub + 1) * step;
    const int32_t v = rp[min(idx, (int64_t)g.n)];
    const bool below = idx < hi && v <= e;
    const int m = __popc((uint32_t)(__ballot(below) >> group0) & ((1u << G) - 1u));
    lo += m * step;
    hi = (int32_t)min((int64_t)hi, (int64_t)lo + max(step, 1));
  }
  if (c64 > g.ntiles) return;
  if (sub == 0) g.brow[c] = search ? lo : max(g.n - 1, 0);
  for (int t = sub; t < g.k; t += G) {
    int32_t at;
    if (!search) at = s.nnz[t];
    else if (c == 0) at = 0;  // entries in front of the base's first one belong to the first tile
    else if (t == g.base) at = e;
    else {
      const int32_t first = s.rowptr[t][lo];
      at = lower_bound_near(s.col[t], first, s.rowptr[t][lo + 1], first + (e - rp[lo]), s.col[g.base][e]);
    }
    g.bound[t * ldb + c] = at;
  }
}

// (1 + len)^-1/2, rounded once.  (In double throughout: k_prepare, 1M nodes, k = 8 45.6 us, so 40.5.)
__device__ __forceinline__ float node_scale(int32_t len) {
  return len >= kUncoded ? (float)(1.0 / sqrt((double)(len + 1))) : scale_of_length(scale_code(len));
}

template <class W>
__device__ __forceinline__ void put_node(W *nk, int32_t k, Quad<W> v) {
  if (k > 2) *reinterpret_cast<Quad<W> *>(nk) = v;
  else nk[0] = v.x;
  if (k == 2) nk[1] = v.y;
}

// 256 rows (block rb of them): dinv_t[i] = (1 + |row i of snapshot t|)^-1/2, rounded once, and the counts the row lists are laid
// out by.  The node-major copy for the scatter step (one line per node) holds the scales, or where `code` is given their codes,
// which go there snapshot-major as well.
__device__ __forceinline__ void prepare_rows(const Snaps &s, const Tiles &g, const RowClasses &rc, int64_t rb, float *dinv,
                                             float *dinv_nk, uint16_t *code) {
  const int64_t i64 = rb * kBlock + threadIdx.x % kBlock;
  const bool live = i64 < g.n;
  const int32_t i = (int32_t)min(i64, (int64_t)g.n - 1);
  int32_t longest = 0;
  int64_t all = 0;
  constexpr int CH = 4;  // snapshots whose row pointers are requested together
  for (int t0 = 0; t0 < g.k; t0 += CH) {
    int32_t a[CH], b[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int32_t *rp = s.rowptr[min(t0 + u, g.k - 1)];
      a[u] = rp[i];
      b[u] = rp[i + 1];
    }
    float v[CH];
    uint16_t c[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int32_t len = b[u] - a[u];
      c[u] = scale_code(len);
      v[u] = node_scale(len);
      if (t0 + u < g.k) {
        longest = max(longest, len);
        all += len;
        if (live) {
          dinv[(int64_t)(t0 + u) * g.n + i] = v[u];
          if (code) code[(int64_t)(t0 + u) * g.n + i] = c[u];
        }
      }
    }
    if (live) {  // (what lies behind the k-th value repeats it)
      const int64_t at = (int64_t)i * node_stride(g.k) + t0;
      if (code) put_node(reinterpret_cast<uint16_t *>(dinv_nk) + at, g.k, Quad<uint16_t>{c[0], c[1], c[2], c[3]});
      else put_node(dinv_nk + at, g.k, Quad<float>{v[0], v[1], v[2], v[3]});
    }
  }
  count_rows(rc, live, longest, all, 0, rb * kBlock < g.n ? g.row_cnt + rb : nullptr);
}

// The first `bound_blocks` workgroups find the tiles' bounds (they wait for memory most of the
// time), the others take 256 rows each.
template <int G>
__global__ __launch_bounds__(kBlock) void k_prepare(Snaps s, Tiles g, RowClasses rc, int32_t bound_blocks,
                                                     float *dinv, float *dinv_nk, uint16_t *code) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  if ((int32_t)blockIdx.x < bound_blocks) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *g.bad = 0;
    find_bounds<G>(s, g, (int64_t)blockIdx.x * kWavesPerBlock + wave, lane);
    return;
  }
  prepare_rows(s, g, rc, (int64_t)blockIdx.x - bound_blocks, dinv, dinv_nk, code);
}

// First position in col[lo, hi) (ascending) that holds c or more, by half a wave.
__device__ __forceinline__ int32_t half_lower_bound(const int32_t *col, int32_t lo, int32_t hi, int32_t c, int lane) {
  constexpr int H = kWave / 2;
  const int sub = lane % H, shift = lane / H * H;
  while (__any(lo < hi)) {
    const int32_t step = (int32_t)(((int64_t)hi - lo + H) / (H + 1));
    const int64_t idx = lo + (int64_t)(sub + 1) * step - 1;
    bool below = false;
    if (lo < hi && idx < hi) below = col[idx] < c;
    const int m = __popc((uint32_t)(__ballot(below) >> shift));
    if (lo < hi) {
      lo += m * step;
      if (m < H) hi = (int32_t)min((int64_t)hi, (int64_t)lo + step - 1);  // (place lo + step - 1 was looked at)
    }
  }
  return lo;
}

// ---- mark -----------------------------------------------------------------------------------
// A workgroup per tile of T base entries, a wave per snapshot (two for k > 16).  The (row, column) of an
// entry becomes ONE ascending 32-bit key: the number of the tile's base rows up to its row, times 2n + 2,
// plus the column (a row that has no base entries in the tile gets keys that no base entry has).  A wave
// finds the rows of its entries by writing, where a row starts in its stretch, what the row's keys start
// with, and running a maximum over that; the base's wave puts its keys into LDS.  A lane has 10 entries
// in a row (8 in the base), so that it looks for the first of them only and walks on from there: a look
// or two per entry, and a search where the base has more than a few entries in between.  One bit per
// snapshot and base entry says where that entry was found; who has all of them is common.
// Graphs with more nodes than these keys have room for (4.1 M; 8.3 M for k > 16) take an instance with 64-bit
// keys: the row's number and the column.  (With a row searched in memory per entry instead, as below, N = 4.3M, k = 4
// took 2215 us for the whole build and N = 8M, k = 8 7386, now 1303 and 4033.)
// A tile that owns a longer stretch, or more rows than are gone through one by one, finds every entry's row by
// search, first among samples of the row pointers in LDS, and takes 64-bit keys of row and column.  A long stretch
// goes a piece at a time; where its entries were found waits in the memory that its exclusive entries will
// take.  (A binary search in memory per entry, one after the other and twice in long stretches: whole build of frames whose
// busy nodes move, N = 200k, k = 4 500 -> 229 us, N = 1M, k = 8 5770 -> 2604; four disjoint snapshots of 200k nodes 162 -> 140.
// Going through 4096 rows at most instead of 16384: 4M nodes with 0.45M entries, k = 4 198 -> 180, 8M 375 -> 341; with a
// lookup per base entry that was 170 and 328.)
//
// Bound by instruction issue and the LDS round trips of the walk: 1M-node R-MAT frame, k = 8, 0.27 ms
// (0.13 G vector instructions, 0.22 of it), against 0.44 for a look-up of every base entry in every
// snapshot's window, four waves per tile and a look-up with a row's bounds from memory (0.235 G).
// N = 200k Chung-Lu, k = 8 87 -> 55 us; R-MAT 100k, k = 5 31 -> 21; N = 20k, k = 4 12.2 -> 8.8; N = 2k 11 -> 7; with 64-bit
// keys N = 4.3M, k = 4 399 -> 292.
// A number of entries per lane that follows the stretch (8 .. 12, in branches) was slower by 40 %.
template <int T>
struct Mark {
  static constexpr int kRun = T / kWave;           // base entries per lane
  static constexpr int kMost = kRun + kRun / 4;    // entries of another snapshot per lane
  static constexpr int kCap = kMost * kWave;       // longest stretch that is taken at once
  // base entry x lies at plane x % kRun, place x / kRun: lanes that are at neighbouring runs read
  // neighbouring addresses
  static constexpr int kPlane = 96;
  static constexpr int kNone = kWave;              // behind the last entry: plane 0, place 64
  // the next entry's place in an array of keys, in bytes: the next plane, or the first one's next place
  template <class K>
  static __device__ __forceinline__ uint32_t next(uint32_t at) {
    constexpr uint32_t B = sizeof(K);
    return min(at + kPlane * B, at + kPlane * B - (kRun * kPlane * B - B));
  }
};
constexpr uint32_t kBadTile = 1u << 21;            // in tile_cnt.y of a tile whose snapshots are not canonical (k_prepare_mark)
constexpr int32_t kMarkRows = 16384;               // most rows of a tile that are gone through one by one

// Places of base entries are in bytes of the array they are looked up in.
template <class K>
__device__ __forceinline__ K mark_at(const K *keys, uint32_t at) {
  return *reinterpret_cast<const K *>(reinterpret_cast<const char *>(keys) + at);
}

// The base's first entry that is not smaller than `key`, or the last one of a run that holds only
// smaller ones.
template <int T, class K>
__device__ __forceinline__ uint32_t mark_search(const K *keys, K key) {
  using S = Mark<T>;
  uint32_t at = 0;
#pragma unroll
  for (uint32_t s = kWave / 2; s >= 1; s >>= 1) at += mark_at(keys + s, at) <= key ? s * (uint32_t)sizeof(K) : 0u;
#pragma unroll
  for (uint32_t s = S::kRun / 2; s >= 1; s >>= 1)
    at += mark_at(keys + (s - 1) * S::kPlane, at) < key ? s * S::kPlane * (uint32_t)sizeof(K) : 0u;
  return at;
}

// N consecutive entries of a list per lane, `offset` of them behind `start` (`all`: every lane's lie inside the
// list).
template <int N>
__device__ __forceinline__ void load_run(const int32_t *col, int32_t nnz, int32_t start, int32_t offset, bool all, int32_t (&c)[N]) {
  typedef int32_t i4 __attribute__((ext_vector_type(4), aligned(4)));
  if (all) {
    const int32_t *const run = col + start + offset;
#pragma unroll
    for (int q = 0; q < N / 4; ++q) {
      const i4 v = *reinterpret_cast<const i4 *>(run + 4 * q);
      c[4 * q] = v.x; c[4 * q + 1] = v.y; c[4 * q + 2] = v.z; c[4 * q + 3] = v.w;
    }
#pragma unroll
    for (int j = N / 4 * 4; j < N; ++j) c[j] = run[j];
  } else {
#pragma unroll
    for (int j = 0; j < N; ++j) c[j] = col[place_in(start, offset + j, nnz)];
  }
}

// Where the base has the ascending keys of a lane, as places in the array of 32-bit words, noted in `present`.
// From a key to the next it is mostly one entry of the base further, or two: both are looked at side by side, without a loop (what
// lies behind the last entry is in the array and never taken).  Slides of N = 500k, k = 8 with little overlap 1092 -> 1076 us,
// R-MAT 300k, k = 8 613 -> 603, 150k, k = 16 258 -> 251, R-MAT 1M, k = 8 1113 -> 1107; three of them: as many faster as slower.
template <int T, int N, class K>
__device__ __forceinline__ void mark_walk(const K *keys, const K (&key)[N], uint32_t *present, uint32_t bit, uint32_t (&at)[N]) {
  using S = Mark<T>;
  uint32_t x = mark_search<T>(keys, key[0]);
  K v = mark_at(keys, x);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const K k0 = key[j];
    if (j > 0) {
      const uint32_t x1 = S::template next<K>(x), x2 = S::template next<K>(x1);
      const K v1 = mark_at(keys, x1), v2 = mark_at(keys, x2);
      const bool one = v < k0, two = one & (v1 < k0);
      x = two ? x2 : one ? x1 : x;
      v = two ? v2 : one ? v1 : v;
    }
    int looks = 6;
    while (__builtin_amdgcn_ballot_w64(v < k0) != 0) {
      if (v < k0) {
        x = S::template next<K>(x);
        v = mark_at(keys, x);
      }
      if (--looks == 0) {
        x = mark_search<T>(keys, k0);
        v = mark_at(keys, x);
      }
    }
    at[j] = S::kNone * 4u;
    if (v == k0) {
      at[j] = x / (sizeof(K) / 4u);
      __hip_atomic_fetch_or(present + at[j] / 4u, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
}

// The same by a search for every key, G of them side by side: where a stretch is shorter than 7/8 of the tile, some of the
// wave's lanes are more than a few entries of the base further at every key.  Whole build, N = 1M Chung-Lu, k = 4, one snapshot
// of 10M edges and three with 75 / 50 / 25 / 3 % of them 536 / 571 / 585 / 550 -> 528 / 512 / 490 / 460 us; stretches as
// long as the tile take longer (R-MAT 1M, k = 8 946 -> 980).
template <int T, int N, class K>
__device__ __forceinline__ void mark_find(const K *keys, const K (&key)[N], uint32_t *present, uint32_t bit, uint32_t (&at)[N]) {
  using S = Mark<T>;
  constexpr int G = sizeof(K) == 4 ? N : 5;  // (ten 64-bit ones take too many registers)
  static_assert(N % G == 0, "");
#pragma unroll
  for (int h = 0; h < N; h += G) {
#pragma unroll
    for (int j = h; j < h + G; ++j) at[j] = 0;
#pragma unroll
    for (uint32_t s = kWave / 2; s >= 1; s >>= 1)
#pragma unroll
      for (int j = h; j < h + G; ++j) at[j] += mark_at(keys + s, at[j]) <= key[j] ? s * (uint32_t)sizeof(K) : 0u;
#pragma unroll
    for (uint32_t s = S::kRun / 2; s >= 1; s >>= 1)
#pragma unroll
      for (int j = h; j < h + G; ++j)
        at[j] += mark_at(keys + (s - 1) * S::kPlane, at[j]) < key[j] ? s * S::kPlane * (uint32_t)sizeof(K) : 0u;
#pragma unroll
    for (int j = h; j < h + G; ++j) {
      const bool found = mark_at(keys, at[j]) == key[j];
      at[j] = found ? at[j] / (sizeof(K) / 4u) : S::kNone * 4u;
      if (found) __hip_atomic_fetch_or(present + at[j] / 4u, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
}

// What the keys of a row start with (q: number of the tile's base rows up to it), and a key.
template <class K>
__device__ __forceinline__ uint32_t mark_row(uint32_t q, bool in_base, uint32_t mult) {
  return sizeof(K) == 4 ? __umul24(q, mult) + (in_base ? 0u : mult / 2u) : 2u * q + (in_base ? 0u : 1u);
}
template <class K>
__device__ __forceinline__ K mark_key(uint32_t row, int32_t col) {
  return sizeof(K) == 4 ? (K)(row + (uint32_t)col) : (K)((uint64_t)row << 32 | (uint32_t)col);
}

// Every (1 << shift)-th row pointer of rows [lo, hi], so many that CAP words of LDS hold them; returns the shift.
template <int CAP>
__device__ __forceinline__ int sample_rows(const int32_t *rp, int32_t lo, int32_t hi, uint32_t *samples, int lane) {
  int shift = 0;
  while ((hi - lo) >> shift >= CAP) ++shift;
  const int32_t last = (hi - lo) >> shift;
  int32_t v[CAP / kWave];
#pragma unroll
  for (int q = 0; q < CAP / kWave; ++q) v[q] = rp[lo + (min(q * kWave + lane, last) << shift)];
#pragma unroll
  for (int q = 0; q < CAP / kWave; ++q) samples[q * kWave + lane] = (uint32_t)v[q];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  return shift;
}

// Rows of N entries from start + offset on (behind start + last: that one's), which lie in rows [lo, hi]: first among
// the samples, then between two of them, side by side, so that a step waits for memory once.
template <int N>
__device__ __forceinline__ void rows_of_run(const int32_t *rp, int32_t lo, int32_t hi, const uint32_t *samples, int shift,
                                            int32_t start, int32_t offset, int32_t last, int32_t (&row)[N]) {
  const int32_t last_sample = (hi - lo) >> shift;
#pragma unroll
  for (int j = 0; j < N; ++j) row[j] = 0;
  for (int32_t step = last_sample > 0 ? 1 << (31 - __builtin_clz((uint32_t)last_sample)) : 0; step >= 1; step >>= 1)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int32_t by = min(step, last_sample - row[j]);
      if ((int32_t)samples[row[j] + by] <= start + min(offset + j, last)) row[j] += by;
    }
#pragma unroll
  for (int j = 0; j < N; ++j) row[j] = lo + (row[j] << shift);
  for (int32_t step = 1 << shift >> 1; step >= 1; step >>= 1)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int32_t by = min(step, hi - row[j]);
      if (rp[row[j] + by] <= start + min(offset + j, last)) row[j] += by;
    }
}

// The base has a column twice in a row (the other snapshots' entries only ever find one of the two).
template <int T, class K>
__device__ __forceinline__ bool mark_twice(const K *keys, int32_t here, int lane) {
  using S = Mark<T>;
  bool twice = false;
#pragma unroll
  for (int j = 0; j < S::kRun; ++j)
    twice |= (lane * S::kRun + j + 1 < here) & (keys[j * S::kPlane + lane] == keys[(j + 1) % S::kRun * S::kPlane + lane + (j + 1) / S::kRun]);
  return twice;
}

// (Held to eight waves per SIMD with 32-bit keys.  k_mark<512, 1> has no spilled registers: a variant that kept 48 bytes of them in
// private memory took 1337 us for the build of the 1M-node R-MAT frame, not 948.  k_prepare_mark<512, 1>, with the searches, keeps
// two, 12 bytes per lane, and k_mark<256, 2> one.)
// SELF: the waves find where the tile starts in their snapshots themselves (k_prepare_mark).
template <int T, int L, class K, bool SELF>  // L: snapshots per wave; K: 32- or 64-bit keys
__device__ __forceinline__ void mark_tile(const Snaps &s, const Tiles &g, int32_t mid_max) {
  using S = Mark<T>;
  constexpr int R = S::kRun, E = S::kMost, PLANE = S::kPlane;
  __shared__ uint64_t key_words[R * PLANE];  // keys of either width
  __shared__ uint32_t present[R * PLANE];    // bit t: snapshot t has the entry (0 behind the last entry)
  __shared__ uint32_t hub_row[T + 2];        // by number of the base row
  __shared__ uint32_t shared_of[PIPAD_MAX_K];
  extern __shared__ uint32_t tags[];         // [k][kCap]
  K *const keys = reinterpret_cast<K *>(key_words);
  uint64_t *const key64 = key_words;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int nwaves = blockDim.x / kWave;
  // (last tile first: where the ids are sorted by degree, and in R-MAT graphs, the last tiles have the most
  // rows and take longest: R-MAT, N = 100k, k = 5 25 -> 21 us, 1M nodes 284 -> 272, Chung-Lu a tie)
  const int32_t tile = g.ntiles - 1 - (int32_t)blockIdx.x;
  const int64_t ldb = (int64_t)g.ntiles + 1;
  const int32_t *rp0 = s.rowptr[g.base];
  const int32_t e0 = tile * T;
  const int32_t here = min(T, s.nnz[g.base] - e0);
  const uint32_t all_bits = ~0u >> (32 - g.k);
  const int32_t lb = min(lane, g.k - 1);
  int32_t r0, r1, my_b0, my_b1;
  if constexpr (SELF) {
    __shared__ int2 bounds[PIPAD_MAX_K];
    const bool last = tile + 1 == g.ntiles;
    const int32_t e = lane < kWave / 2 ? e0 : min(e0 + T, s.nnz[g.base] - 1);
    const int32_t column = s.col[g.base][e], row = half_row_of_entry(rp0, g.n, e, lane);
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int t = wave + l * nwaves;
      if (t >= g.k) break;
      const int32_t nnz = s.nnz[t];
      int32_t at = e;
      if (t != g.base) {
        const int32_t first = s.rowptr[t][row], end = s.rowptr[t][row + 1];
        at = half_lower_bound(s.col[t], min(max(first, 0), nnz), min(max(end, 0), nnz), column, lane);
      }
      // (entries in front of the base's first one belong to the first tile)
      const int2 b = make_int2(tile == 0 ? 0 : __builtin_amdgcn_readlane(at, 0),
                               last ? nnz : __builtin_amdgcn_readlane(at, kWave - 1));
      if (lane == 0) {
        bounds[t] = b;
        g.bound[t * ldb + tile] = b.x;
        if (last) g.bound[t * ldb + g.ntiles] = nnz;
      }
    }
    r0 = __builtin_amdgcn_readlane(row, 0);
    r1 = last ? g.n - 1 : __builtin_amdgcn_readlane(row, kWave - 1);
    __syncthreads();
    my_b0 = bounds[lb].x;
    my_b1 = bounds[lb].y;
  } else {
    r0 = g.brow[tile];
    r1 = g.brow[tile + 1];
    my_b0 = g.bound[lb * ldb + tile];
    my_b1 = g.bound[lb * ldb + tile + 1];
  }
  const int32_t rfirst = tile == 0 ? 0 : r0;  // (the first tile owns what lies in front of the base, too)
  for (int x = threadIdx.x; x < R * PLANE; x += blockDim.x) present[x] = x % PLANE < kWave ? 1u << g.base : 0u;
  for (int x = threadIdx.x; x < T + 2; x += blockDim.x) hub_row[x] = 0;
  __syncthreads();

  // 32-bit keys of row number q (1, 2, ..) start at q * mult; those of rows without base entries behind it lie
  // between its keys and those of row number q + 1 (in any order: nothing of the base lies there)
  const uint32_t mult = 2u * (uint32_t)g.n + 2u;
  const bool wide = r1 - rfirst >= kMarkRows || __any(my_b1 - my_b0 > S::kCap);

  int32_t start[L], len[L];
  int32_t c[L][E];     // columns of this lane's entries
  K key[L][E];         // ... their keys (of the base: row numbers)
  uint32_t at[L][E];   // ... and where the base has them
  bool bad = false;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const int t = wave + l * nwaves;
    if (t >= g.k) break;
    const int32_t nnz = s.nnz[t];
    // (the clamps only act on snapshots that are not canonical)
    start[l] = min(max(__builtin_amdgcn_readlane(my_b0, t), 0), nnz);
    const int32_t end = __builtin_amdgcn_readlane(my_b1, t);
    bad |= end < start[l];
    len[l] = max(min(end, nnz) - start[l], 0);
    const int per = t == g.base ? R : E;
    if (len[l] > 0) load_run(s.col[t], nnz, start[l], lane * per, reaches(start[l], (kWave - 1) * per + E, nnz), c[l]);
  }

  if (!wide) {
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int t = wave + l * nwaves;
      if (t >= g.k) break;
      const bool base = t == g.base;
      uint32_t *const tag = tags + t * S::kCap;
#pragma unroll
      for (int j = 0; j < E; ++j) tag[j * kWave + lane] = 0;
      const int32_t *rp = s.rowptr[t];
      uint32_t rank = 0;
      constexpr int kAhead = 4;  // times 64 rows whose pointers are requested together
      struct Rows {
        int32_t a, b, a0, b0;
      };
      auto request = [&](int32_t rb) __attribute__((always_inline)) {
        const int32_t r = min(rb + lane, r1);
        return Rows{rp[r], rp[r + 1], rp0[r], rp0[r + 1]};
      };
      for (int32_t rb = rfirst; rb <= r1; rb += kAhead * kWave) {
        Rows rows[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
          if (rb + u * kWave <= r1) rows[u] = request(rb + u * kWave);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          if (rb + u * kWave > r1) break;
          const Rows row = rows[u];
          const bool live = rb + u * kWave + lane <= r1;
          const bool in_base = live & (max(row.a0, e0) < min(row.b0, e0 + here));
          const uint64_t mask = __ballot(in_base);
          const uint32_t q = rank + in_base + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
          rank += (uint32_t)__popcll(mask);
          const uint32_t p = (uint32_t)max(row.a - start[l], 0);
          if (live & ((int32_t)p < min(row.b - start[l], len[l]))) {
            if (base) tag[p % R * kWave + p / R] = q;
            else tag[p % E * kWave + p / E] = mark_row<K>(q, in_base, mult);
          }
          if (in_base & (row.b - row.a > mid_max)) hub_row[q] = 1;
        }
      }
      // what lies behind the list comes behind all of the base
      if (!base && lane == 0 && len[l] < S::kCap) tag[len[l] % E * kWave + len[l] / E] = mark_row<K>(T, false, mult);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      uint32_t most = 0, row[E];
#pragma unroll
      for (int j = 0; j < E; ++j) {
        most = max(most, tag[j * kWave + lane]);
        row[j] = most;
      }
      const uint32_t front = __shfl_up(wave_max(most), 1, kWave);
      most = lane > 0 ? front : 0u;
      if (base) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
          row[j] = max(row[j], most);
          key[l][j] = row[j];
          keys[j * PLANE + lane] = lane * R + j < here ? mark_key<K>(mark_row<K>(row[j], true, mult), c[l][j]) : ~(K)0;
        }
        if (lane == 0) keys[S::kNone] = ~(K)0;
      } else {
#pragma unroll
        for (int j = 0; j < E; ++j) key[l][j] = mark_key<K>(max(row[j], most), c[l][j]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int t = wave + l * nwaves;
      if (t >= g.k) break;
      if (t == g.base) bad |= mark_twice<T>(keys, here, lane);
      if (t == g.base || len[l] == 0) continue;
      if (8 * len[l] > 7 * here) mark_walk<T>(keys, key[l], present, 1u << t, at[l]);
      else mark_find<T>(keys, key[l], present, 1u << t, at[l]);
    }
  } else {
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int t = wave + l * nwaves;
      if (t != g.base) continue;
      int32_t row[R];
      const int shift = sample_rows<S::kCap>(rp0, r0, r1, tags + t * S::kCap, lane);
      rows_of_run(rp0, r0, r1, tags + t * S::kCap, shift, e0, lane * R, here - 1, row);
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int32_t x = lane * R + j;
        key64[j * PLANE + lane] = x < here ? mark_key<uint64_t>((uint32_t)row[j], c[l][j]) : ~0ull;
        key[l][j] = (uint32_t)x;
      }
      if (lane == 0) key64[S::kNone] = ~0ull;
    }
    int shift[L];
    constexpr int G = 5;  // (entries at a time: with all ten the kernel needs too many registers for eight waves per SIMD)
    static_assert(E % G == 0, "");
    auto find_rows = [&](int l, int t, int32_t first, int32_t left) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < E; h += G) {
        int32_t row[G];
        rows_of_run(s.rowptr[t], rfirst, r1, tags + t * S::kCap, shift[l], first, lane * E + h, left - 1, row);
#pragma unroll
        for (int j = 0; j < G; ++j) key[l][h + j] = (uint32_t)row[j];
      }
    };
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int t = wave + l * nwaves;
      if (t >= g.k) break;
      if (t == g.base || len[l] == 0) continue;
      shift[l] = sample_rows<S::kCap>(s.rowptr[t], rfirst, r1, tags + t * S::kCap, lane);
      find_rows(l, t, start[l], min(len[l], S::kCap));
    }
    __syncthreads();
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const int t = wave + l * nwaves;
      if (t >= g.k) break;
#pragma unroll
      for (int j = 0; j < R; ++j) {  // (the base's entries, by their places)
        const int32_t x = lane * R + j, row = x < here ? (int32_t)(key64[j * PLANE + lane] >> 32) : r1;
        if (s.rowptr[t][row + 1] - s.rowptr[t][row] > mid_max) hub_row[x] = 1;
      }
      if (t == g.base) bad |= mark_twice<T>(key64, here, lane);
      if (t == g.base || len[l] == 0) continue;
      // a long stretch a piece at a time; where its entries were found is kept in what `excl` has for them
      for (uint32_t done = 0; done < (uint32_t)len[l]; done += S::kCap) {
        const int32_t first = start[l] + (int32_t)done, left = min(len[l] - (int32_t)done, S::kCap);
        if (done > 0) {
          load_run(s.col[t], start[l] + len[l], first, lane * E, left == S::kCap, c[l]);
          find_rows(l, t, first, left);
        }
#pragma unroll
        for (int h = 0; h < E; h += G) {
          uint64_t wide_key[G];
          uint32_t found[G];
#pragma unroll
          for (int j = 0; j < G; ++j)  // (behind the end: behind all of the base)
            wide_key[j] = lane * E + h + j < left ? mark_key<uint64_t>((uint32_t)key[l][h + j], c[l][h + j]) : (uint64_t)~0u << 32;
          mark_walk<T>(key64, wide_key, present, 1u << t, found);
#pragma unroll
          for (int j = 0; j < G; ++j) at[l][h + j] = found[j];
        }
        if (len[l] > S::kCap)
#pragma unroll
          for (int j = 0; j < E; ++j)
            if (lane * E + j < left) g.excl[t][first + (lane * E + j)] = (int32_t)at[l][j];
      }
    }
  }
  __syncthreads();

#pragma unroll
  for (int l = 0; l < L; ++l) {
    const int t = wave + l * nwaves;
    if (t >= g.k) break;
    int32_t *const out = g.excl[t] + start[l];
    // the exclusive entries go out in order through the wave's share of `tags`: from the lanes, ten in a row
    // each, a store touched up to 40 lines (whole build, few common entries: N = 500k, k = 8 1128 -> 993 us,
    // R-MAT 342k, k = 8 251 -> 224; hardly any exclusive ones: a tie)
    uint32_t *const stage = tags + t * S::kCap;
    auto write_out = [&](int32_t *to, int count) __attribute__((always_inline)) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      for (int x = lane; x < count; x += kWave) to[x] = (int32_t)stage[x];
    };
    if (t == g.base) {
      const int32_t mine = min(here - lane * R, R);
      uint32_t common = 0, hub = 0;
#pragma unroll
      for (int j = 0; j < R; ++j)
        if (j < mine) {
          common |= (uint32_t)(present[j * PLANE + lane] == all_bits) << j;
          hub |= hub_row[key[l][j]] << j;
        }
      const uint32_t cnt = (uint32_t)__popc(common), incl = wave_sum(cnt);
      const uint32_t in_hubs = wave_sum((uint32_t)__popc(common & hub));
      const uint32_t common2 = common | __shfl_down(common, 1, kWave) << R, hub2 = hub | __shfl_down(hub, 1, kWave) << R;
      const int32_t word0 = (tile << (g.tile_log2 - 6)), word = lane * R / 64;  // of this lane's entries
      if (word * 64 < here) {
        if (lane * R % 64 == 0) g.wpre[word0 + word] = (uint16_t)(incl - cnt);
        uint8_t *const bits = reinterpret_cast<uint8_t *>(g.bits + word0), *const hubs = reinterpret_cast<uint8_t *>(g.hub_bits + word0);
        if (R == 8) {
          bits[lane] = (uint8_t)common;
          hubs[lane] = (uint8_t)hub;
        } else if ((lane & 1) == 0) {  // (four entries per lane)
          bits[lane / 2] = (uint8_t)common2;
          hubs[lane / 2] = (uint8_t)hub2;
        }
      }
      if (lane == kWave - 1) {
        if (SELF) hub_row[T + 1] = in_hubs;  // (no base row has this number)
        else g.tile_cnt[tile] = make_uint2(incl, in_hubs);
        shared_of[t] = incl;
      }
      uint32_t to = lane * R - (incl - cnt);
#pragma unroll
      for (int j = 0; j < R; ++j)
        if ((j < mine) & !(common >> j & 1u)) stage[to++] = (uint32_t)c[l][j];
      write_out(out, here - __builtin_amdgcn_readlane((int)incl, kWave - 1));
    } else {
      uint32_t kept = 0;
      for (uint32_t done = 0; done < (uint32_t)len[l]; done += S::kCap) {
        const int32_t first = start[l] + (int32_t)done, left = min(len[l] - (int32_t)done, S::kCap);
        if (len[l] > S::kCap) {  // (what has been written out lies in front of this piece)
          load_run(s.col[t], start[l] + len[l], first, lane * E, left == S::kCap, c[l]);
#pragma unroll
          for (int j = 0; j < E; ++j) at[l][j] = lane * E + j < left ? (uint32_t)g.excl[t][first + (lane * E + j)] : S::kNone * 4u;
        }
        const int32_t mine = min(max(left - lane * E, 0), E);
        uint32_t excl = 0;
#pragma unroll
        for (int j = 0; j < E; ++j) excl |= mark_at(present, at[l][j]) != all_bits ? 1u << j : 0u;
        excl &= (1u << mine) - 1u;
        const uint32_t cnt = (uint32_t)__popc(excl), incl = wave_sum(cnt);
        uint32_t to = incl - cnt;
#pragma unroll
        for (int j = 0; j < E; ++j)
          if (excl >> j & 1u) stage[to++] = (uint32_t)c[l][j];
        const uint32_t count = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
        write_out(out + kept, (int)count);
        kept += count;
      }
      if (lane == 0) shared_of[t] = (uint32_t)len[l] - kept;
    }
  }
  // In canonical snapshots every common entry is found once in each of them; anything else is
  // reported, so that what follows never writes past the sizes computed from these counts.
  __syncthreads();
  if (wave == 0 && lane < g.k) bad |= shared_of[lane] != shared_of[g.base];
  if constexpr (SELF) {
    const bool any = __syncthreads_or(bad);
    if (threadIdx.x == 0) g.tile_cnt[tile] = make_uint2(shared_of[g.base], hub_row[T + 1] | (any ? kBadTile : 0u));
  } else {
    if (bad) *g.bad = 1;
  }
}

template <int T, int L, class K>
__global__ __launch_bounds__(16 * kWave) __attribute__((amdgpu_waves_per_eu(sizeof(K) == 4 ? 8 : 6))) void k_mark(Snaps s, Tiles g, int32_t mid_max) {
  mark_tile<T, L, K, false>(s, g, mid_max);
}

// The same with what k_prepare does, in one launch: a workgroup per tile, whose waves find its bounds (a search by 32 lanes
// per bound: three or four round trips for the row, one to three for the column), then workgroups of as many threads
// for 256 rows per 256 threads.  For small frames (build_overlap), whose tiles are all under way at once: with more, the
// searches add to the time for which a tile takes up its place.
template <int T, int L>
__global__ __launch_bounds__(16 * kWave) __attribute__((amdgpu_waves_per_eu(8))) void k_prepare_mark(Snaps s, Tiles g, int32_t mid_max, RowClasses rc,
                                                                                                     float *dinv, float *dinv_nk) {
  if ((int32_t)blockIdx.x < g.ntiles) {
    mark_tile<T, L, uint32_t, true>(s, g, mid_max);
    return;
  }
  const int blocks = blockDim.x / kBlock, sub = threadIdx.x / kBlock;
  if (sub >= blocks) return;  // (a whole wave: the number of threads need not divide)
  prepare_rows(s, g, rc, (int64_t)((int32_t)blockIdx.x - g.ntiles) * blocks + sub, dinv, dinv_nk, nullptr);
}

// ---- scan over the tiles and the row blocks -----------------------------------------------------
// Exclusive prefix sums of the tiles' counts and of the row blocks' counts, the totals behind the
// last.  Every workgroup takes a run of them and adds up what lies in front of the run itself (two
// counts per 16-byte load, 20 loads per thread for the last run of 40k tiles), so that none waits for
// another; the last one knows the sizes of the frame and sends them to the host (`out` may be host
// memory: the host waits for `seq` to appear behind them).
constexpr int kTileScanBlock = 1024;
constexpr int kTileScanRun = 2 * kTileScanBlock;  // tiles a workgroup scans at a time
constexpr int kTileScanMost = 64;                 // workgroups; with more tiles each takes several such runs

// Exclusive sums over the workgroup of N values per thread, and their totals.
template <int N>
__device__ inline void sum_block(const uint32_t (&v)[N], uint32_t (&before)[N], uint32_t (&total)[N]) {
  constexpr int NW = kTileScanBlock / kWave;
  static_assert(NW == 16, "the waves' sums are scanned in one row of lanes");
  __shared__ uint32_t sums[N][NW];
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const uint32_t inc = wave_sum(v[q]);
    if (lane == kWave - 1) sums[q][wave] = inc;
    before[q] = inc - v[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const uint32_t x = wave_sum(sums[q][lane & (NW - 1)]);  // (lanes 0 .. 15 count)
    total[q] = (uint32_t)__builtin_amdgcn_readlane((int)x, NW - 1);
    if (wave > 0) before[q] += (uint32_t)__builtin_amdgcn_readlane((int)x, max(wave - 1, 0));
  }
  __syncthreads();
}

// RowCounts as 32-bit values whose sums over a workgroup do not overflow.
constexpr int kRowSums = 8;
__device__ inline void split_counts(const RowCounts &c, bool in, uint32_t (&v)[kRowSums]) {
  v[0] = in ? c.mid : 0u;
  v[1] = in ? c.hub : 0u;
  v[2] = in ? c.units : 0u;
  v[3] = in ? c.common : 0u;
  v[4] = in ? (uint32_t)(c.entries & 0xfffffu) : 0u;
  v[6] = in ? c.short_entries : 0u;
  v[7] = in ? c.uncoded : 0u;
  v[5] = in ? (uint32_t)(c.entries >> 20) : 0u;  // (a workgroup's rows hold fewer than 2^36 entries)
}
__device__ inline RowCounts join_counts(const RowCounts &front, const uint32_t (&v)[kRowSums]) {
  RowCounts c;
  c.entries = front.entries + (uint64_t)v[4] + ((uint64_t)v[5] << 20);
  c.common = front.common + v[3];
  c.short_entries = front.short_entries + v[6];
  c.uncoded = front.uncoded + v[7];
  c.mid = front.mid + v[0];
  c.hub = front.hub + v[1];
  c.units = front.units + v[2];
  return c;
}

// Blocks [b0, b1) of `cnt`, scanned into `pre`; returns the counts in front of b1.  b0 is a multiple
// of kTileScanBlock, or b1.
__device__ inline RowCounts scan_rows(const RowCounts *cnt, RowCounts *pre, int64_t b0, int64_t b1) {
  RowCounts front = {};
  for (int64_t base = 0; base < b1; base += kTileScanBlock) {
    const int64_t at = base + threadIdx.x;
    uint32_t v[kRowSums], before[kRowSums], total[kRowSums];
    split_counts(cnt[min(at, b1 - 1)], at < b1, v);
    sum_block(v, before, total);
    if (at < b1 && at >= b0) pre[at] = join_counts(front, before);
    front = join_counts(front, total);
  }
  return front;
}

// Sends the sizes of a frame to the host: `common` and `in_hubs` common entries, `exclusive` ones in hub rows.
__device__ inline void send_totals(const RowCounts &all, uint32_t common, uint64_t in_hubs, uint64_t exclusive,
                                   uint32_t bad, FrameTotals *out, uint32_t seq) {
  FrameTotals v;
  v.nnz_c = common;
  v.mid = all.mid;
  v.hub = all.hub;
  v.units = all.units;
  v.short_entries = all.short_entries;
  v.uncoded = all.uncoded;
  v.split_c = in_hubs;
  v.split_d = exclusive;
  v.bad = bad;
  v.seq = 0;
  *out = v;
  __threadfence_system();
  __hip_atomic_store(&out->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

struct ScanArgs {
  const uint2 *tile_cnt;
  uint2 *tile_pre;
  const RowCounts *row_cnt;
  RowCounts *row_pre;
  const uint32_t *bad;
  int32_t ntiles, k;
  int64_t row_blocks;
  int32_t tiles_per_block;      // a multiple of kTileScanRun
  int64_t rows_per_block;
};

__global__ __launch_bounds__(kTileScanBlock) void k_scan_counts(ScanArgs a, FrameTotals *out, uint32_t seq) {
  const int64_t t0 = min((int64_t)blockIdx.x * a.tiles_per_block, (int64_t)a.ntiles);
  const int64_t t1 = min(t0 + a.tiles_per_block, (int64_t)a.ntiles);
  uint32_t carry[2], mine[2] = {0, 0}, unused[2];
  {
    // what lies in front of the run
    constexpr int AHEAD = 4;
    for (int64_t base = 2 * (int64_t)threadIdx.x; base < t0; base += AHEAD * kTileScanRun) {
      uint4 x[AHEAD];
#pragma unroll
      for (int q = 0; q < AHEAD; ++q)
        x[q] = *reinterpret_cast<const uint4 *>(a.tile_cnt + min(base + (int64_t)q * kTileScanRun, (t0 - 1) & ~(int64_t)1));
#pragma unroll
      for (int q = 0; q < AHEAD; ++q)
        if (base + (int64_t)q * kTileScanRun < t0) {
          const bool both = base + (int64_t)q * kTileScanRun + 1 < t0;
          mine[0] += x[q].x + (both ? x[q].z : 0u);
          mine[1] += x[q].y + (both ? x[q].w : 0u);
        }
    }
    sum_block(mine, unused, carry);
  }
  for (int64_t base = t0; base < t1; base += kTileScanRun) {
    const int64_t at = base + 2 * (int64_t)threadIdx.x;
    uint4 x = *reinterpret_cast<const uint4 *>(a.tile_cnt + min(at, (t1 - 1) & ~(int64_t)1));  // (padded to a pair)
    if (at >= t1) x.x = x.y = 0;
    if (at + 1 >= t1) x.z = x.w = 0;
    const uint32_t v[2] = {x.x + x.z, x.y + x.w};
    uint32_t before[2], total[2];
    sum_block(v, before, total);
    before[0] += carry[0];
    before[1] += carry[1];
    if (at < t1) a.tile_pre[at] = make_uint2(before[0], before[1]);
    if (at + 1 < t1) a.tile_pre[at + 1] = make_uint2(before[0] + x.x, before[1] + x.y);
    carry[0] += total[0];
    carry[1] += total[1];
  }
  const int64_t b0 = min((int64_t)blockIdx.x * a.rows_per_block, a.row_blocks);
  const RowCounts all = scan_rows(a.row_cnt, a.row_pre, b0, min(b0 + a.rows_per_block, a.row_blocks));
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    a.tile_pre[a.ntiles] = make_uint2(carry[0], carry[1]);
    a.row_pre[a.row_blocks] = all;
    // (of all entries of the hub rows, what the common ones take in every snapshot is not exclusive)
    send_totals(all, carry[0], carry[1], all.entries - (uint64_t)a.k * carry[1], *a.bad, out, seq);
  }
}

// The transposed frame: the parts' row pointers are known, and with them everything but the totals.
__global__ __launch_bounds__(kTileScanBlock) void k_scan_row_counts(const RowCounts *row_cnt, RowCounts *row_pre,
                                                                     int64_t row_blocks, FrameTotals *out,
                                                                     uint32_t seq) {
  const RowCounts all = scan_rows(row_cnt, row_pre, 0, row_blocks);
  if (threadIdx.x == 0) {
    row_pre[row_blocks] = all;
    send_totals(all, 0, all.common, all.entries, 0, out, seq);
  }
}

// ---- rows ------------------------------------------------------------------------------------
// The work lists of the aggregation.
struct ListArgs {
  RowClasses rc;
  int32_t *rows_short, *rows_long, *hub_rows, *hub_item_off, *item_row, *item_v0, *item_v1, *item_c0, *item_d0;
};

// Puts row i (called by every thread of a workgroup of 256 consecutive rows, `live` where there is a
// row) on its list; `first` holds the counts in front of the workgroup's rows (as summed up from
// count_rows).  place(entries, common) gives, for a hub row, where its common and its exclusive entries
// start in the class-grouped copies, from what the hub rows in front of it hold.
template <class Place>
__device__ inline void list_row(const ListArgs &q, bool live, int32_t i, int64_t L, int32_t lc, int64_t entries,
                                const RowCounts &first, Place place) {
  __shared__ uint32_t w_mid[kWavesPerBlock], w_hub[kWavesPerBlock], w_units[kWavesPerBlock],
      w_common[kWavesPerBlock];
  __shared__ uint64_t w_all[kWavesPerBlock];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int cls = row_class(L, q.rc.short_max, q.rc.mid_max);
  const uint64_t is_mid = __ballot(live && cls == 1), is_hub = __ballot(live && cls == 2);
  const bool hub = is_hub >> lane & 1ull;
  // inclusive running sums over the wave's hub rows
  const uint32_t my_units = hub ? hub_units(L, q.rc.threshold, q.rc.segment) : 0u;
  const uint64_t my_all = hub ? (uint64_t)entries : 0ull;
  uint32_t units = my_units, shared = hub ? (uint32_t)lc : 0u;
  uint64_t all = my_all;
  if (is_hub) {
#pragma unroll
    for (int s = 1; s < kWave; s <<= 1) {
      const uint32_t u = __shfl_up(units, s, kWave), c = __shfl_up(shared, s, kWave);
      const uint64_t a = __shfl_up(all, s, kWave);
      if (lane >= s) { units += u; shared += c; all += a; }
    }
  }
  if (lane == kWave - 1) {
    w_mid[wave] = (uint32_t)__popcll(is_mid);
    w_hub[wave] = (uint32_t)__popcll(is_hub);
    w_units[wave] = units;
    w_common[wave] = shared;
    w_all[wave] = all;
  }
  __syncthreads();
  if (!live) return;
  uint32_t mid = first.mid, h = first.hub, u0 = first.units + units - my_units;
  uint32_t common = first.common + shared - (hub ? (uint32_t)lc : 0u);
  uint64_t e = first.entries + all - my_all;
  for (int w = 0; w < wave; ++w) {
    mid += w_mid[w];
    h += w_hub[w];
    u0 += w_units[w];
    common += w_common[w];
    e += w_all[w];
  }
  const uint64_t below = (1ull << lane) - 1ull;
  mid += (uint32_t)__popcll(is_mid & below);
  h += (uint32_t)__popcll(is_hub & below);
  if (cls == 0) q.rows_short[(uint32_t)i - mid - h] = i;
  if (cls == 1) q.rows_long[mid] = i;
  if (hub) {
    int32_t c0, d0;
    place(e, common, &c0, &d0);
    q.hub_rows[h] = i;
    q.hub_item_off[h] = (int32_t)u0;
    for (uint32_t u = 0; u < my_units; ++u) {
      const int64_t v0 = (int64_t)u * q.rc.segment;
      q.item_row[u0 + u] = i;
      q.item_v0[u0 + u] = my_units == 1 ? 0 : (int32_t)v0;
      q.item_v1[u0 + u] = my_units == 1 ? INT32_MAX : (int32_t)min(v0 + q.rc.segment, (int64_t)INT32_MAX);
      q.item_c0[u0 + u] = c0 + (my_units == 1 ? 0 : (int32_t)min(v0, (int64_t)lc));
      q.item_d0[u0 + u] = d0;
    }
  }
}

// Common entries of the base in front of entry e (nnz > 0 entries; no branches around the loads).
__device__ inline int32_t common_before(const Tiles &g, int32_t nnz, int32_t e) {
  const int32_t x = min(max(e, 0), nnz - 1), w = x >> 6;
  const uint64_t bits = g.bits[w];
  const uint32_t v = g.tile_pre[x >> g.tile_log2].x + g.wpre[w], all = g.tile_pre[g.ntiles].x;
  return (int32_t)(e < nnz ? v + (uint32_t)__popcll(bits & ((1ull << (x & 63)) - 1ull)) : all);
}

// ... those of them that lie in hub rows.
__device__ inline int32_t hub_common_before(const Tiles &g, int32_t nnz, int32_t e) {
  if (e >= nnz) return (int32_t)g.tile_pre[g.ntiles].y;
  const int32_t tile = e >> g.tile_log2, w = e >> 6;
  uint32_t v = g.tile_pre[tile].y;
  for (int32_t x = tile << (g.tile_log2 - 6); x < w; ++x) v += (uint32_t)__popcll(g.bits[x] & g.hub_bits[x]);
  return (int32_t)(v + (uint32_t)__popcll(g.bits[w] & g.hub_bits[w] & ((1ull << (e & 63)) - 1ull)));
}

// Sums of a few row blocks' counts, in front of block `upto` and of all, for every thread.
__device__ inline void sum_row_counts(const RowCounts *cnt, int32_t blocks, int32_t upto, RowCounts *front, RowCounts *all) {
  __shared__ uint32_t sums[2][kRowSums][kWavesPerBlock];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  uint32_t v[2][kRowSums] = {};
  for (int b = threadIdx.x; b < blocks; b += kBlock) {
    uint32_t c[kRowSums];
    split_counts(cnt[b], true, c);
#pragma unroll
    for (int x = 0; x < kRowSums; ++x) {
      v[0][x] += b < upto ? c[x] : 0u;
      v[1][x] += c[x];
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int x = 0; x < kRowSums; ++x) {
      const uint32_t sum = wave_sum(v[u][x]);
      if (lane == kWave - 1) sums[u][x][wave] = sum;
    }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int x = 0; x < kRowSums; ++x) {
      v[u][x] = 0;
#pragma unroll
      for (int w = 0; w < kWavesPerBlock; ++w) v[u][x] += sums[u][x][w];
    }
  const RowCounts none = {};
  *front = join_counts(none, v[0]);
  *all = join_counts(none, v[1]);
}

// Up to so many tiles k_rows_scatter adds up itself (2^20 base entries), and so many row blocks (262,144 rows).
constexpr int kTilesEach = 8;  // per thread
constexpr int kSumTiles = kTilesEach * kBlock;
constexpr int kSumRowBlocks = 4 * kBlock;

// The counts of tiles kTilesEach * threadIdx.x and those behind it, as they lie in memory (read two at a time).
struct TileCounts {
  uint4 pair[kTilesEach / 2];
};
__device__ __forceinline__ TileCounts request_tiles(const Tiles &g) {
  const int t0 = kTilesEach * (int)threadIdx.x;
  TileCounts x;
#pragma unroll
  for (int q = 0; q < kTilesEach; q += 2) {
    x.pair[q / 2] = make_uint4(0, 0, 0, 0);
    if (t0 + q < g.ntiles) x.pair[q / 2] = *reinterpret_cast<const uint4 *>(g.tile_cnt + t0 + q);
  }
  return x;
}
// ... without the flags; returns whether a flag is set.
__device__ __forceinline__ bool split_tiles(const Tiles &g, const TileCounts &x, uint32_t (&c)[2][kTilesEach]) {
  const int t0 = kTilesEach * (int)threadIdx.x;
  uint32_t flags = 0;
#pragma unroll
  for (int q = 0; q < kTilesEach; q += 2) {
    const uint4 v = x.pair[q / 2];
    const bool both = t0 + q + 1 < g.ntiles;
    c[0][q] = v.x;
    c[1][q] = v.y & (kBadTile - 1u);
    c[0][q + 1] = both ? v.z : 0u;
    c[1][q + 1] = both ? v.w & (kBadTile - 1u) : 0u;
    flags |= v.y | (both ? v.w : 0u);
  }
  return (flags & kBadTile) != 0;
}

// What lies in front of every tile, and of all of them, into `pre`; returns whether a tile's flag is set.
__device__ inline bool sum_tiles(const Tiles &g, const TileCounts &x, uint2 *pre) {
  __shared__ uint32_t front[2][kWavesPerBlock];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, t0 = kTilesEach * (int)threadIdx.x;
  uint32_t c[2][kTilesEach];
  const bool bad = split_tiles(g, x, c);
  uint32_t at[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < kTilesEach; ++q) mine += c[u][q];
    const uint32_t incl = wave_sum(mine);
    if (lane == kWave - 1) front[u][wave] = incl;
    at[u] = incl - mine;
  }
  __syncthreads();
  for (int w = 0; w < wave; ++w) {
    at[0] += front[0][w];
    at[1] += front[1][w];
  }
#pragma unroll
  for (int q = 0; q < kTilesEach; ++q) {
    if (t0 + q < g.ntiles) pre[t0 + q] = make_uint2(at[0], at[1]);
    at[0] += c[0][q];
    at[1] += c[1][q];
  }
  if (threadIdx.x == kBlock - 1) pre[g.ntiles] = make_uint2(at[0], at[1]);
  return __syncthreads_or(bad);
}

// Common entries in front of tile `upto` (the same for the workgroup), and of all tiles, for every thread; `bad`: a tile's flag is
// set.
__device__ inline uint32_t sum_tiles_before(const Tiles &g, int32_t upto, uint32_t *all, bool *bad) {
  __shared__ uint32_t front[kWavesPerBlock], every[kWavesPerBlock], flag[kWavesPerBlock];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, t0 = kTilesEach * (int)threadIdx.x;
  uint32_t c[2][kTilesEach], mine = 0, total = 0;
  const bool here = split_tiles(g, request_tiles(g), c);
#pragma unroll
  for (int q = 0; q < kTilesEach; ++q) {
    mine += t0 + q < upto ? c[0][q] : 0u;
    total += c[0][q];
  }
  const uint32_t incl = wave_sum(mine), incl_all = wave_sum(total);
  const uint64_t any = __ballot(here);
  if (lane == kWave - 1) {
    front[wave] = incl;
    every[wave] = incl_all;
    flag[wave] = any != 0;
  }
  __syncthreads();
  uint32_t sum = 0, flags = 0;
  *all = 0;
#pragma unroll
  for (int w = 0; w < kWavesPerBlock; ++w) {
    sum += front[w];
    *all += every[w];
    flags |= flag[w];
  }
  *bad = flags != 0;
  return sum;
}

struct RowArgs {
  int32_t *rowptr_c;
  int32_t *rowptr_d[PIPAD_MAX_K];
  float *scales_nk;  // of a frame that is to have codes: where its node-major scales go if a row is too long for one
};

// A thread per row i in [0, n].  The exclusive row pointer is the input's minus the common one; the
// longest row a class is decided by is the longest input row (its common entries are in all of
// them).
// SUM: neither the tiles' counts nor the row blocks' are summed up yet; they are few enough for every
// workgroup to do that (k_rows_scatter).
// CODES: of a frame that may be to have codes.
template <bool SUM, bool CODES>
__device__ __forceinline__ void make_rows(const Snaps &s, Tiles g, const RowArgs &o, const ListArgs &q, FrameTotals *out, uint32_t seq) {
  const int64_t i64 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int32_t i = (int32_t)min(i64, (int64_t)g.n), i1 = min(i + 1, g.n);
  const bool live = i64 < g.n;
  const int32_t nnz0 = s.nnz[g.base];
  const int32_t *rp0 = s.rowptr[g.base];
  const int32_t ea = rp0[i], eb = rp0[i1];
  RowCounts first, total;
  if constexpr (SUM) {
    __shared__ uint2 pre[kSumTiles + 1];
    const TileCounts tiles = request_tiles(g);  // (under way while the rows' counts are summed up)
    sum_row_counts(g.row_cnt, (int32_t)(((int64_t)g.n + kBlock - 1) / kBlock), (int32_t)blockIdx.x, &first, &total);
    const bool bad = sum_tiles(g, tiles, pre);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      const uint2 all = pre[g.ntiles];
      send_totals(total, all.x, all.y, total.entries - (uint64_t)g.k * all.y, bad, out, seq);
    }
    g.tile_pre = pre;
  } else {
    first = g.row_pre[blockIdx.x];
    total = g.row_pre[((int64_t)g.n + kBlock - 1) / kBlock];
  }
  int32_t before = 0, after = 0, longest = 0;
  if (nnz0 > 0) {
    before = common_before(g, nnz0, ea);
    after = common_before(g, nnz0, eb);
  }
  if (i64 <= g.n) o.rowptr_c[i] = before;
  // (the clamps only ever act on snapshots that are not canonical: whatever they hold, the row
  // pointers stay within the parts)
  const int32_t nnz_c = (int32_t)g.tile_pre[g.ntiles].x;
  // (In a launch of their own behind the host's wait: frames of 26 to 29 M entries with such a row 168 us to build, so 164, 258 and 254,
  // 300 and 288; behind this loop 166, 255, 293.)
  const bool uncoded = CODES && o.scales_nk && total.uncoded > 0;
  int64_t all = 0;
  constexpr int CH = 8;  // snapshots whose row pointers are requested together
  for (int t0 = 0; t0 < g.k; t0 += CH) {
    int32_t a[CH], b[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int32_t *rp = s.rowptr[min(t0 + u, g.k - 1)];
      a[u] = rp[i];
      b[u] = rp[i1];
    }
#pragma unroll
    for (int u = 0; u < CH; ++u)
      if (t0 + u < g.k) {
        longest = max(longest, b[u] - a[u]);
        all += b[u] - a[u];
        if (i64 <= g.n) o.rowptr_d[t0 + u][i] = min(max(a[u] - before, 0), max(s.nnz[t0 + u] - nnz_c, 0));
      }
    if (uncoded && live)
#pragma unroll
      for (int u = 0; u < CH; u += 4)
        if (t0 + u < g.k)
          put_node(o.scales_nk + (int64_t)i * node_stride(g.k) + t0 + u, g.k,
                   Quad<float>{node_scale(b[u] - a[u]), node_scale(b[u + 1] - a[u + 1]), node_scale(b[u + 2] - a[u + 2]),
                               node_scale(b[u + 3] - a[u + 3])});
  }
  if (i64 == g.n) q.hub_item_off[total.hub] = (int32_t)total.units;  // the end of the last hub row's units
  list_row(q, live, i, longest, after - before, all, first, [&](uint64_t entries, uint32_t, int32_t *c0, int32_t *d0) {
    *c0 = hub_common_before(g, nnz0, ea);
    *d0 = (int32_t)((int64_t)entries - (int64_t)g.k * *c0);
  });
}

__global__ __launch_bounds__(kBlock) void k_rows(Snaps s, Tiles g, RowArgs o, ListArgs q) {
  make_rows<false, true>(s, g, o, q, nullptr, 0);
}

// The same for a frame whose row pointers are in place (the transposed frame): the counts, then the
// lists.
struct PartRows {
  const int32_t *rowptr[PIPAD_MAX_K + 1];  // common, then the k exclusive parts
};

__device__ inline int64_t part_lengths(const PartRows &p, int32_t n, int32_t k, int32_t i, int32_t *lc, int64_t *L) {
  const int32_t i1 = min(i + 1, n);
  *lc = p.rowptr[0][i1] - p.rowptr[0][i];
  int32_t longest = 0;
  int64_t ld = 0;
  for (int t = 1; t <= k; ++t) {
    const int32_t len = p.rowptr[t][i1] - p.rowptr[t][i];
    longest = max(longest, len);
    ld += len;
  }
  *L = (int64_t)*lc + longest;
  return ld;
}

__global__ __launch_bounds__(kBlock) void k_count_rows(PartRows p, int32_t n, int32_t k, RowClasses rc, RowCounts *cnt) {
  const int64_t i64 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  int32_t lc;
  int64_t L;
  const int64_t entries = part_lengths(p, n, k, (int32_t)min(i64, (int64_t)n), &lc, &L);
  count_rows(rc, i64 < n, L, entries, lc, cnt + blockIdx.x);
}

// SUM: `cnt` holds the counts of every block, of which there are no more than a workgroup has threads, and each
// workgroup adds up what it needs (a launch less, 4 us where launches decide); else what k_scan_row_counts
// made of them.
template <bool SUM>
__global__ __launch_bounds__(kBlock) void k_list_rows(PartRows p, int32_t n, int32_t k, const RowCounts *cnt, ListArgs q,
                                                       FrameTotals *out, uint32_t seq) {
  const int64_t i64 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int32_t i = (int32_t)min(i64, (int64_t)n), row_blocks = (int32_t)(((int64_t)n + kBlock - 1) / kBlock);
  RowCounts first, total;
  if (SUM) {
    sum_row_counts(cnt, row_blocks, (int32_t)blockIdx.x, &first, &total);
    if (i64 == 0) send_totals(total, 0, total.common, total.entries, 0, out, seq);
  } else {
    first = cnt[blockIdx.x];
    total = cnt[row_blocks];
  }
  if (i64 == n) q.hub_item_off[total.hub] = (int32_t)total.units;
  int32_t lc;
  int64_t L;
  const int64_t entries = part_lengths(p, n, k, i, &lc, &L);
  list_row(q, i64 < n, i, L, lc, entries, first, [](uint64_t e, uint32_t c, int32_t *c0, int32_t *d0) {
    *c0 = (int32_t)c;
    *d0 = (int32_t)e;
  });
}

// ---- class-grouped copies of the hub rows' entries ------------------------------------------------
template <class W>
struct SplitArgs {
  int32_t n_units, k, sub_log2;
  const int32_t *item_row, *item_v0, *item_v1, *item_c0, *item_d0;
  const int32_t *rowptr[PIPAD_MAX_K + 1];  // parts: common, then exclusive
  const int32_t *col[PIPAD_MAX_K + 1];
  int32_t n;
  NodeScales<W> scales;
  int32_t *sptr, *scol_c, *scol_d;
  void *swc[PIPAD_MAX_K];
  W *swd;
  int32_t block_off[PIPAD_MAX_K + 2];      // first workgroup of every part, in their natural order
  int32_t run_off[kClasses + 1];           // first workgroup of every XCD's run of the exclusive parts
  uint64_t whole;                          // bit p: part p takes a workgroup per unit, not a wave
};

constexpr int kFillRounds = 8;                        // entries per lane and piece
constexpr int kFillPiece = kFillRounds * kBlock;      // entries a workgroup puts in class order in LDS at a time

// The k scales of UN entries of the common copy, where `live`.
template <class W, int UN>
__device__ __forceinline__ void store_scales(const SplitArgs<W> &g, const int32_t (&c)[UN], const int32_t (&to)[UN],
                                             const int32_t (&live)[UN]) {
  if (g.k > 2) {
    const int32_t stride = node_stride(g.k);
    for (int q = 0; 4 * q < g.k; ++q) {
      Quad<W> w[UN];
#pragma unroll
      for (int r = 0; r < UN; ++r) w[r] = *reinterpret_cast<const Quad<W> *>(g.scales.nk + (int64_t)c[r] * stride + 4 * q);
#pragma unroll
      for (int r = 0; r < UN; ++r)
        if (live[r]) put_scales_nt(g.swc, q, g.k, to[r], w[r]);
    }
  } else if (g.k == 2) {
    Pair<W> w[UN];
#pragma unroll
    for (int r = 0; r < UN; ++r) w[r] = reinterpret_cast<const Pair<W> *>(g.scales.nk)[c[r]];
#pragma unroll
    for (int r = 0; r < UN; ++r)
      if (live[r]) {
        __builtin_nontemporal_store(w[r].x, static_cast<W *>(g.swc[0]) + to[r]);
        __builtin_nontemporal_store(w[r].y, static_cast<W *>(g.swc[1]) + to[r]);
      }
  } else {
    W w[UN];
#pragma unroll
    for (int r = 0; r < UN; ++r) w[r] = g.scales.nk[c[r]];
#pragma unroll
    for (int r = 0; r < UN; ++r)
      if (live[r]) __builtin_nontemporal_store(w[r], static_cast<W *>(g.swc[0]) + to[r]);
  }
}

// A part's entries of one unit, stably grouped by column class, by W waves.  A piece of them (8 per
// lane) is read into registers, counted and put in class order in LDS with one ballot per class and 64
// entries, and written out in that order with the scales, so that neighbouring lanes store to
// neighbouring addresses.
template <int NC, int W, class Scale>
__device__ __forceinline__ void fill_part(const SplitArgs<Scale> &g, int32_t u, int p, int lane, int wave, int32_t *stage,
                                          int32_t (*s_cnt)[NC], int32_t *s_off) {
  constexpr int32_t piece = W * kFillRounds * kWave;  // of the team
  auto sync = [&]() __attribute__((always_inline)) {
    if (W > 1) __syncthreads();
    else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  const int32_t row = g.item_row[u], v0 = g.item_v0[u], v1 = g.item_v1[u];
  const int32_t cs = g.rowptr[0][row], lc = g.rowptr[0][row + 1] - cs;
  int32_t a, b, out;  // entries [a, b) of the part, first place in the copy
  if (p == 0) {
    a = cs + min(v0, lc);
    b = cs + min(v1, lc);
    out = g.item_c0[u];
  } else {
    int32_t ds = 0, ld = 0;
    if (lane < g.k) {
      ds = g.rowptr[1 + lane][row];
      ld = g.rowptr[1 + lane][row + 1] - ds;
    }
    int32_t before = lane < p - 1 ? ld : 0;  // the row's entries in the exclusive parts in front
#pragma unroll
    for (int m = kWave >> 1; m >= 1; m >>= 1) before += __shfl_xor(before, m, kWave);
    ds = __builtin_amdgcn_readlane(ds, p - 1);
    ld = __builtin_amdgcn_readlane(ld, p - 1);
    const int32_t q0 = min(max(v0 - lc, 0), ld), q1 = min(max(v1 - lc, 0), ld);
    a = ds + q0;
    b = ds + q1;
    out = g.item_d0[u] + before + q0;
  }
  // (from the unit's first entry on: places behind a list's end may pass 2^31, offsets in a unit of 2^30 entries do not)
  const int32_t *col = g.col[p] + a;
  b -= a;
  // of a wave: every wave has a part of a short list (with 512 entries each, one wave after the other, N = 100k R-MAT, k = 5
  // 13.9 us, now 13.0; R-MAT 1M, k = 8 243, now 240)
  const int32_t share = W == 1 ? piece : min((b + W * kWave - 1) / (W * kWave), kFillRounds) * kWave;
  int32_t cv[kFillRounds];
  int32_t cnt[NC];  // this wave's entries per class (wave-uniform)
  auto load_and_count = [&](int32_t at) __attribute__((always_inline)) {
    const int32_t first = at + wave * share, end = min(first + share, b);
#pragma unroll
    for (int r = 0; r < kFillRounds; ++r) {
      if (first + r * kWave >= end) break;
      const int32_t v = col[min(first + r * kWave + lane, b - 1)];
      cv[r] = first + r * kWave + lane < b ? v : -1;
    }
#pragma unroll
    for (int r = 0; r < kFillRounds; ++r) {
      if (first + r * kWave >= end) break;
      const uint32_t cl = cv[r] >= 0 ? column_class(cv[r], g.sub_log2) : (uint32_t)NC;
#pragma unroll
      for (int x = 0; x < NC; ++x) cnt[x] += __popcll(__ballot(cl == (uint32_t)x));
    }
  };
  // lane x < NC: entries of class x that the team and that the waves in front of this one have counted
  auto exchange = [&](int32_t *team, int32_t *front) __attribute__((always_inline)) {
    int32_t mine = 0;
#pragma unroll
    for (int x = 0; x < NC; ++x)
      if (lane == x) mine = cnt[x];
    *team = mine;
    *front = 0;
    if (W == 1) return;
    if (lane < NC) s_cnt[wave][lane] = mine;
    __syncthreads();
    *team = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const int32_t c = lane < NC ? s_cnt[w][lane] : 0;
      *team += c;
      if (w < wave) *front += c;
    }
    __syncthreads();
  };
#pragma unroll
  for (int x = 0; x < NC; ++x) cnt[x] = 0;
  for (int32_t at = 0; at < b; at += piece) load_and_count(at);
  int32_t team, front;
  exchange(&team, &front);
  // the copy's class boundaries: sptr[(p * (NC + 1) + x) * n_units + u]
  int32_t run = out + (int32_t)wave_sum((uint32_t)team) - team;  // lane x: where class x goes on
  if (wave == 0 && lane <= NC) g.sptr[((int64_t)p * (NC + 1) + lane) * g.n_units + u] = run;

  for (int32_t at = 0; at < b; at += piece) {
    if (b > piece) {
#pragma unroll
      for (int x = 0; x < NC; ++x) cnt[x] = 0;
      load_and_count(at);
      exchange(&team, &front);
    }
    const int32_t pos = (int32_t)wave_sum((uint32_t)team) - team;  // the class's first place in the piece
    if (wave == 0 && lane < NC) s_off[lane] = run - pos;           // place in the copy minus place in the piece
    run += team;
    int32_t local[NC];
#pragma unroll
    for (int x = 0; x < NC; ++x) local[x] = __builtin_amdgcn_readlane(pos + front, x);
    const int32_t first = at + wave * share, end = min(first + share, b);
#pragma unroll
    for (int r = 0; r < kFillRounds; ++r) {
      if (first + r * kWave >= end) break;
      const uint32_t cl = cv[r] >= 0 ? column_class(cv[r], g.sub_log2) : (uint32_t)NC;
      int32_t where = 0;
#pragma unroll
      for (int x = 0; x < NC; ++x) {
        const uint64_t mask = __ballot(cl == (uint32_t)x);
        if (cl == (uint32_t)x)
          where = local[x] + (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
        local[x] += (int32_t)__popcll(mask);
      }
      if (cv[r] >= 0) stage[where] = cv[r];
    }
    sync();
    const int32_t here = min(b - at, piece);
    constexpr int UN = 4;  // entries per lane whose scales are requested together
    for (int32_t j0 = wave * kWave + lane; j0 < here; j0 += UN * W * kWave) {
      int32_t c[UN], to[UN];
#pragma unroll
      for (int r = 0; r < UN; ++r) {
        const int32_t j = j0 + r * W * kWave;
        c[r] = stage[min(j, here - 1)];
        to[r] = s_off[column_class(c[r], g.sub_log2)] + j;
      }
      if (p > 0) {
        Scale w[UN];
#pragma unroll
        for (int r = 0; r < UN; ++r) w[r] = g.scales.of[(int64_t)(p - 1) * g.n + c[r]];
#pragma unroll
        for (int r = 0; r < UN; ++r)
          if (j0 + r * W * kWave < here) {
            __builtin_nontemporal_store(c[r], g.scol_d + to[r]);
            __builtin_nontemporal_store(w[r], g.swd + to[r]);
          }
      } else {
        int32_t live[UN];
#pragma unroll
        for (int r = 0; r < UN; ++r) live[r] = j0 + r * W * kWave < here;
#pragma unroll
        for (int r = 0; r < UN; ++r)
          if (live[r]) __builtin_nontemporal_store(c[r], g.scol_c + to[r]);
        store_scales<Scale, UN>(g, c, to, live);
      }
    }
    sync();
  }
}

// A workgroup per unit of the parts that most of a unit's entries are in, a wave per unit of the others
// (build_split_arrays): a wave alone goes through 2048 entries in 32 steps of memory round trips, and on
// all but the largest frames there are too few of them to hide that.  A wave per unit of every part took
// 35 us on an R-MAT frame with N = 100k, k = 5, now 14; N = 200k Chung-Lu, k = 8 28, now 21.  On the
// 1M-node R-MAT frame the same either way (0.25 ms then): most of what is fetched are lines of D^-1/2 for a few scales
// each, and 0.36 GB are written.
// Its stores go past the caches: they were in the way of the lines that scales are gathered from, and the aggregation
// reads them only after the caches hold other things.  R-MAT 1M 239 -> 216 us, N = 200k, k = 8 18.0 -> 16.8.
// An XCD takes a run of the exclusive parts' units, so that it reads one or two snapshots' D^-1/2 instead
// of all: N = 200k, k = 8 60 -> 38 MB fetched, 21 -> 18.5 us; R-MAT 1M 250 -> 242; N = 100k 14 -> 13.2.  The runs hold as
// many entries each, as far as the parts' sizes tell: with as many workgroups each, N = 1M Chung-Lu, k = 4, one snapshot of 10M
// edges and three with a quarter of them took 57 us, now 46; snapshots that double in size 73, now 62.  (The same in
// k_scatter fetches a quarter less and takes as long: the L2s' requests bound it, one per gathered scale.)  A kernel for the scales alone that
// runs every class on the XCD that gathers it later fetches a third of that but shares the lines it
// writes between XCDs, and the two together were slower (0.26 ms).
template <int NC, class Scale>
__global__ __launch_bounds__(kBlock) void k_split_fill(SplitArgs<Scale> g) {
  __shared__ int32_t stage[kFillPiece];
  __shared__ int32_t s_cnt[kWavesPerBlock][NC], s_off[kWavesPerBlock][NC];
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int p = 0;
  int32_t b = blockIdx.x;
  if (b >= align_xcd(g.block_off[1])) {
    const int32_t x = b % kClasses;
    b = g.run_off[x] + (b - align_xcd(g.block_off[1])) / kClasses;
    if (b >= g.run_off[x + 1]) return;
    while (b >= g.block_off[p + 1]) ++p;
  }
  b -= g.block_off[p];
  if (p == 0 && b >= g.block_off[1]) return;
  if (g.whole >> p & 1ull) {
    fill_part<NC, kWavesPerBlock>(g, b, p, lane, wave, stage, s_cnt, s_off[0]);
  } else {
    const int32_t u = b * kWavesPerBlock + wave;
    if (u < g.n_units) fill_part<NC, 1>(g, u, p, lane, 0, stage + wave * (kFillPiece / kWavesPerBlock), s_cnt, s_off[wave]);
  }
}

// ---- scatter ----------------------------------------------------------------------------------
// A wave per (run of TILES tiles, part); grid.y = part (0 = common, 1 + t = exclusive part of snapshot t).  The
// selected entries keep the order of the input.  Besides the column index, the column scale
// dinv_t[column] of the entry is stored: for a common entry once per snapshot (from the node-major
// copy of D^-1/2: one line per node), for an exclusive entry for its own snapshot.  The scales of a
// hub row's common entries are never read from here (the aggregation takes them from the
// class-grouped copy), so they are skipped.  On the 1M-node R-MAT frame 0.84 GB are fetched and 0.57 GB
// written in 0.31 ms: 4.5 TB/s, the rate of a plain copy.
struct OutParts {
  int32_t *col[PIPAD_MAX_K + 1];
  void *wc[PIPAD_MAX_K];
  void *wd[PIPAD_MAX_K];
};

// Parts that are written before their sizes are known share their room, so that it need hold no more than the entries of the input,
// and a scale for each: the columns of all parts lie one behind the other, snapshot t's common and exclusive scales as well.  How
// far the exclusive ones move up depends on the common entries alone: OutParts has their places without any, and
// `common` entries put exclusive part t's columns behind by cols(t), its scales by scales().  Pieces start at multiples of 256 bytes.
constexpr int32_t kRoomPiece = 64;
__host__ __device__ inline int64_t room_pieces(int64_t entries) { return (entries + kRoomPiece - 1) / kRoomPiece * kRoomPiece; }
struct RoomShift {
  int32_t common;
  __host__ __device__ int64_t scales() const { return room_pieces(common); }
  __host__ __device__ int64_t cols(int t) const { return room_pieces(common) - (int64_t)t * (common / kRoomPiece * kRoomPiece); }
};

constexpr int kScatterAhead = 4;  // words whose entries a wave has in flight

__device__ inline int running_count(uint64_t sel, int lane) {  // selected entries up to and including this word
  int incl = __popcll(sel);
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int up = __shfl_up(incl, d, kWave);
    if (lane >= d) incl += up;
  }
  return incl;
}

__device__ inline uint64_t lane_word(uint64_t x, int l) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l) |
         (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l) << 32;
}

// KV > 0: a node's k scales lie in KV 16-byte pieces, read together (FULL: k == 4 * KV); KV == 0: k <= 2, read at once (500k-node
// R-MAT frame, k = 2, 65 us one after the other, now 44; k_split_fill 31 and 25), or k > 16, a piece after the other (150k nodes,
// k = 18, 353 us a scale after the other, now 277).
// common(x): common entries in front of tile x; col_shift, scale_shift: how far the exclusive part lies behind its place in OutParts.
template <class W, int KV, bool FULL, int TILES, class Common>
__device__ __forceinline__ void scatter_tiles(const Snaps &s, const Tiles &g, const OutParts &o, NodeScales<W> scales_of, int part, int32_t tile0, Common common,
                                              int64_t col_shift = 0, int64_t scale_shift = 0) {
  constexpr int WPT = kWave / TILES;  // words of a tile a wave takes at once
  const int lane = threadIdx.x % kWave;
  const int t = part == 0 ? g.base : part - 1;
  const int32_t *bound = g.bound + t * ((int64_t)g.ntiles + 1);
  const int32_t c0 = (int32_t)common(tile0);
  const int32_t tile = tile0 + lane / WPT, j = lane % WPT;
  int32_t e0 = 0, len = 0;
  if (part == 0 && tile < g.ntiles) {
    e0 = bound[tile];
    len = bound[tile + 1] - e0;
  }
  const int32_t *col = s.col[t];
  const int32_t nnz = s.nnz[t];
  if (nnz == 0) return;
  if (part == 0) {
    uint64_t sel = 0, hub = 0;
    if (j * 64 < len) {  // (a base tile has at most WPT words)
      const int64_t at = ((int64_t)tile << (g.tile_log2 - 6)) + j;
      sel = g.bits[at];
      hub = g.hub_bits[at];
    }
    constexpr int UN = kScatterAhead;
    const int32_t first = e0 + j * 64;
    const int excl = running_count(sel, lane) - __popcll(sel);
    int32_t *const out = o.col[0];
#pragma unroll 1
    for (int w0 = 0; w0 < kWave; w0 += UN) {
      if (TILES == 1 && w0 * 64 >= __builtin_amdgcn_readfirstlane(len)) break;
      uint64_t x[UN], need[UN], any = 0, scales = 0;
#pragma unroll
      for (int r = 0; r < UN; ++r) {
        x[r] = lane_word(sel, w0 + r);
        need[r] = x[r] & ~lane_word(hub, w0 + r);
        any |= x[r];
        scales |= need[r];
      }
      if (any == 0) continue;
      int32_t c[UN], at[UN];
#pragma unroll
      for (int r = 0; r < UN; ++r) {
        c[r] = col[min(__builtin_amdgcn_readlane(first, w0 + r) + lane, nnz - 1)];
        at[r] = c0 + __builtin_amdgcn_readlane(excl, w0 + r) +
                (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(x[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)x[r], 0));
      }
      if (scales == 0) {
#pragma unroll
        for (int r = 0; r < UN; ++r)
          if (x[r] >> lane & 1ull) out[at[r]] = c[r];
      } else if (KV > 0) {
        Quad<W> v[UN][KV > 0 ? KV : 1];
#pragma unroll
        for (int r = 0; r < UN; ++r) {
          const int64_t node = need[r] >> lane & 1ull ? c[r] : 0;  // (one line for the lanes that need none)
#pragma unroll
          for (int q = 0; q < KV; ++q) v[r][q] = (reinterpret_cast<const Quad<W> *>(scales_of.nk) + node * KV)[q];
        }
#pragma unroll
        for (int r = 0; r < UN; ++r) {
          if (x[r] >> lane & 1ull) out[at[r]] = c[r];
          if (need[r] >> lane & 1ull)
#pragma unroll
            for (int q = 0; q < KV; ++q) put_scales<W, FULL>(o.wc, q, g.k, at[r], v[r][q]);
        }
      } else {
#pragma unroll
        for (int r = 0; r < UN; ++r)
          if (x[r] >> lane & 1ull) out[at[r]] = c[r];
        if (g.k > 2) {  // (more than 16)
          const int32_t pieces = node_stride(g.k) / 4;
          for (int q = 0; q < pieces; ++q) {
            Quad<W> w[UN];
#pragma unroll
            for (int r = 0; r < UN; ++r) w[r] = reinterpret_cast<const Quad<W> *>(scales_of.nk)[(int64_t)c[r] * pieces + q];
#pragma unroll
            for (int r = 0; r < UN; ++r)
              if (need[r] >> lane & 1ull) put_scales(o.wc, q, g.k, at[r], w[r]);
          }
        } else {
          Pair<W> w[UN];
#pragma unroll
          for (int r = 0; r < UN; ++r) {
            const int32_t node = need[r] >> lane & 1ull ? c[r] : 0;
            if (g.k == 2) w[r] = reinterpret_cast<const Pair<W> *>(scales_of.nk)[node];
            else w[r].x = w[r].y = scales_of.nk[node];
          }
#pragma unroll
          for (int r = 0; r < UN; ++r)
            if (need[r] >> lane & 1ull) {
              static_cast<W *>(o.wc[0])[at[r]] = w[r].x;
              if (g.k == 2) static_cast<W *>(o.wc[1])[at[r]] = w[r].y;
            }
        }
      }
    }
    return;
  }
  // exclusive part: the tiles' pieces of g.excl[t], one behind the other
  int32_t from[TILES], upto[TILES];  // piece q: output places [upto[q - 1], upto[q])
  int32_t total = 0;
#pragma unroll
  for (int q = 0; q < TILES; ++q) {
    const int32_t x = min(tile0 + q, g.ntiles), y = min(x + 1, g.ntiles);
    const int32_t start = bound[x];
    from[q] = start - total;  // input place of an output place of this piece, minus the latter
    total += (bound[y] - start) - (int32_t)(common(y) - common(x));
    upto[q] = total;
  }
  const int32_t *excl = g.excl[t];
  int32_t *const out_col = o.col[part] + (col_shift + (bound[tile0] - c0));
  W *const out_w = static_cast<W *>(o.wd[t]) + (scale_shift + (bound[tile0] - c0));
  const W *of_t = scales_of.of + (int64_t)t * g.n;
  constexpr int UN = kScatterAhead;
  for (int32_t j0 = lane; j0 - lane < total; j0 += UN * kWave) {
    int32_t c[UN];
    W d[UN];
#pragma unroll
    for (int r = 0; r < UN; ++r) {
      const int32_t j = min(j0 + r * kWave, total - 1);
      int32_t at = from[0];
#pragma unroll
      for (int q = 1; q < TILES; ++q) at = j >= upto[q - 1] ? from[q] : at;
      c[r] = excl[at + j];
    }
#pragma unroll
    for (int r = 0; r < UN; ++r) d[r] = of_t[c[r]];
#pragma unroll
    for (int r = 0; r < UN; ++r)
      if (j0 + r * kWave < total) {
        out_col[j0 + r * kWave] = c[r];
        out_w[j0 + r * kWave] = d[r];
      }
  }
}

template <class W, int KV, bool FULL, int TILES>
__global__ __launch_bounds__(kBlock) void k_scatter(Snaps s, Tiles g, OutParts o, NodeScales<W> scales) {
  const int64_t tile64 = ((int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave) * TILES;
  if (tile64 >= g.ntiles) return;
  scatter_tiles<W, KV, FULL, TILES>(s, g, o, scales, (int)blockIdx.y, __builtin_amdgcn_readfirstlane((int32_t)tile64),
                                 [&](int32_t x) __attribute__((always_inline)) { return g.tile_pre[x].x; });
}

// Rows and entries in one launch: `row_wgs` workgroups make the rows, those behind them write the entries, a wave per tile and
// part.  The outputs have room for whatever entries the parts have (RoomShift), so that nothing waits for the host; where the
// snapshots are not canonical, no entries are written.  SUM: behind k_prepare_mark, with nothing summed up yet (the first
// workgroup sends the sizes to the host).
template <int KV, bool FULL, bool SUM>
__global__ __launch_bounds__(kBlock) void k_rows_scatter(Snaps s, Tiles g, RowArgs r, ListArgs q, OutParts o, int32_t row_wgs,
                                                         NodeScales<float> scales, FrameTotals *out, uint32_t seq) {
  if ((int32_t)blockIdx.x < row_wgs) {
    make_rows<SUM, false>(s, g, r, q, out, seq);
    return;
  }
  const int32_t groups = (g.ntiles + kWavesPerBlock - 1) / kWavesPerBlock, b = (int32_t)blockIdx.x - row_wgs;
  const int part = b / groups;
  const int32_t first = (b - part * groups) * kWavesPerBlock, tile0 = first + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if constexpr (SUM) {
    uint32_t mine[kWavesPerBlock];  // of the workgroup's tiles
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) mine[w] = g.tile_cnt[min(first + w, g.ntiles - 1)].x;
    bool bad;
    uint32_t all, front = sum_tiles_before(g, first, &all, &bad);
    if (bad || tile0 >= g.ntiles) return;
    uint32_t here = mine[0];
#pragma unroll
    for (int w = 1; w < kWavesPerBlock; ++w)
      if (tile0 >= first + w) {
        front += mine[w - 1];
        here = mine[w];
      }
    const RoomShift shift{(int32_t)all};
    scatter_tiles<float, KV, FULL, 1>(s, g, o, scales, part, tile0,
                               [&](int32_t x) __attribute__((always_inline)) { return x == tile0 ? front : front + here; },
                               shift.cols(part - 1), shift.scales());
  } else {
    if (tile0 >= g.ntiles || *g.bad != 0) return;
    const RoomShift shift{(int32_t)g.tile_pre[g.ntiles].x};
    scatter_tiles<float, KV, FULL, 1>(s, g, o, scales, part, tile0, [&](int32_t x) __attribute__((always_inline)) { return g.tile_pre[x].x; },
                               shift.cols(part - 1), shift.scales());
  }
}

}  // namespace

// Pinned host memory per thread for the sizes a build reads back (allocated at the thread's first
// build, kept until the process ends); null when pinned memory cannot be had.
static FrameTotals *pinned_totals() {
  thread_local FrameTotals *buf = nullptr;
  thread_local bool tried = false;
  if (!tried) {
    tried = true;
    void *ptr = nullptr;
    if (hipHostMalloc(&ptr, sizeof(FrameTotals), hipHostMallocPortable) == hipSuccess) {
      buf = static_cast<FrameTotals *>(ptr);
      std::memset(buf, 0, sizeof(*buf));
    } else {
      (void)hipGetLastError();
    }
  }
  return buf;
}

TotalsTicket expect_totals(FrameTotals *device_totals) {
  thread_local uint32_t seq = 0;
  if (++seq == 0) ++seq;
  FrameTotals *pinned = pinned_totals();
  return pinned ? TotalsTicket{pinned, seq, true} : TotalsTicket{device_totals, seq, false};
}

int wait_totals(const TotalsTicket &ticket, hipStream_t st, FrameTotals *out) {
  if (!ticket.on_host) {
    PIPAD_HIP(hipMemcpyAsync(out, ticket.where, sizeof(*out), hipMemcpyDeviceToHost, st));
    PIPAD_HIP(hipStreamSynchronize(st));
    return PIPAD_OK;
  }
  // The kernel stored the sizes straight into the pinned words and the sequence number behind them;
  // watching for it is several microseconds shorter than a copy and an event.  Every few thousand
  // looks the stream is asked whether it is still running, so that a failed launch ends the wait.
  for (uint32_t looks = 1;; ++looks) {
    if (__atomic_load_n(&ticket.where->seq, __ATOMIC_ACQUIRE) == ticket.seq) break;
    if (looks % 4096 == 0) {
      const hipError_t e = hipStreamQuery(st);
      if (e == hipSuccess) {
        if (__atomic_load_n(&ticket.where->seq, __ATOMIC_ACQUIRE) == ticket.seq) break;
        return hip_fail(hipErrorUnknown, "the scan of the sizes");
      }
      if (e != hipErrorNotReady) return hip_fail(e, "hipStreamQuery");
      (void)hipGetLastError();  // "not ready" is no error of anyone's
    }
  }
  *out = *ticket.where;
  return PIPAD_OK;
}

// Frames whose hub rows need no column classes: up to 64k nodes with 4M entries in all snapshots together.  The
// classes spread the gathers of long rows over the eight L2s, for a launch that copies these rows and one
// that adds up their partial sums; where a matrix is not much larger than an L2 that costs more than it
// gives.  R-MAT frames, classes against a workgroup per row: N = 10k, k = 5, F = 16 aggregation 14.2 -> 10.6 us, F = 64
// 24.9 -> 20.8, with the build (F = 32) 66 -> 56; N = 32k, 20 entries per row, k = 4: F = 64 55 -> 56, with the build 92 -> 81;
// N = 60k, k = 1 64 -> 56.  Chung-Lu, N = 40k, k = 4: F = 64 58 -> 55, with the build 85 -> 73.  Past the line: R-MAT,
// N = 60k, 20 entries per row, k = 8: F = 64 167 -> 181.  (With a smaller mid_max rows that a wave does better with
// would be among them.)  Of 200 frames below the line with hub rows, in the mean: steps 6 to 14 % faster, backward passes 3 to 11,
// aggregations alone 4 to 26, the more the fewer entries, with operands in the caches and without; at worst 14 % slower
// (R-MAT, N = 62k, k = 2, F = 32, aggregation alone).
constexpr int64_t kEarlyEntries = (int64_t)1 << 25, kCodeEntries = 24000000;  // (build_overlap)
constexpr int32_t kManyTiles = 16384;  // from here on a wave of k_scatter takes four
constexpr int32_t kPlainNodes = 65536, kPlainRow = 512;
constexpr int64_t kPlainEntries = (int64_t)4 << 20;

// Longest row that one lane team walks, where the option stands at its default of 64: a frame of few
// entries has few waves, and the chain of such a row's gathers (a team of 8 lanes takes 16 rounds for 64
// entries) is most of its time.  Measured up to 0.4M entries in all snapshots together, N = 1k .. 100k, F = 2 .. 128,
// R-MAT and Chung-Lu: 32 against 64 is 10 to 13 % faster in the mean for k = 1 .. 4 (fused update 4 to 6 %), at worst
// 7 % slower; for more snapshots, which bring more waves, 5 % and at worst 14 % slower, 48 is 4 % faster and at
// worst 6 % slower.  With more entries 48 is between 19 % faster and 12 % slower, 32 up to 30 % slower
// (the fused update with F = 16, k = 4, 0.5M entries 7 %).  These with operands in the caches; of 200 frames with operands
// that no cache holds 16 to 18 % faster for k = 1 .. 4 and up to 32 columns, 5 to 10 % otherwise, at worst 6 % slower (the
// update 9 %; in the caches 13 %: R-MAT, N = 5k, k = 3, F = 64, Fo = 16).
static int64_t short_rows_up_to(int64_t option, int32_t k, int64_t entries) {
  if (option != Options().short_max || entries > (3 << 17)) return option;
  return k <= 4 ? option / 2 : option / 4 * 3;
}

void frame_take_options(pipad_frame *f, int64_t entries) {
  const int64_t lim = (int64_t)1 << 30;  // thresholds beyond any int32 row length mean "never"
  f->opt = options();
  f->short_max = (int32_t)std::clamp<int64_t>(short_rows_up_to(f->opt.short_max, f->k, entries), 0, lim);
  f->mid_max = (int32_t)std::clamp<int64_t>(f->opt.mid_max, f->short_max, lim);
  f->hub_threshold = (int32_t)std::clamp<int64_t>(f->opt.hub_threshold, 1, lim);
  f->hub_segment = (int32_t)std::clamp<int64_t>(f->opt.hub_segment, 1, lim);
  f->sub_log2 = f->opt.sub_classes >= 4 ? 2 : f->opt.sub_classes >= 2 ? 1 : 0;
  f->nclass = kClasses << f->sub_log2;
  f->plain_units = f->opt.scale_codes != 2 && f->n <= kPlainNodes && entries <= kPlainEntries && f->mid_max >= kPlainRow;
}

void want_lists(Arena &a, pipad_frame *f, int64_t entries) {
  // no more rows can be longer than a threshold than the entries of all snapshots together fill
  const int64_t n = f->n;
  const int64_t mids = std::min(n, entries / ((int64_t)f->short_max + 1));
  const int64_t hubs = std::min(n, entries / ((int64_t)f->mid_max + 1));
  const int64_t units = hubs ? hubs + entries / f->hub_segment : 0;
  a.want(&f->rows_short, (size_t)n);
  a.want(&f->rows_long, (size_t)mids);
  a.want(&f->hub_rows, (size_t)hubs);
  a.want(&f->hub_item_off, (size_t)hubs + 1);
  a.want(&f->item_row, (size_t)units);
  a.want(&f->item_v0, (size_t)units);
  a.want(&f->item_v1, (size_t)units);
  a.want(&f->item_c0, (size_t)units);
  a.want(&f->item_d0, (size_t)units);
}

static RowClasses row_classes(const pipad_frame *f) {
  return RowClasses{f->short_max, f->mid_max, f->hub_threshold, f->hub_segment};
}

static ListArgs list_args(const pipad_frame *f) {
  ListArgs q;
  q.rc = row_classes(f);
  q.rows_short = f->rows_short;
  q.rows_long = f->rows_long;
  q.hub_rows = f->hub_rows;
  q.hub_item_off = f->hub_item_off;
  q.item_row = f->item_row;
  q.item_v0 = f->item_v0;
  q.item_v1 = f->item_v1;
  q.item_c0 = f->item_c0;
  q.item_d0 = f->item_d0;
  return q;
}

size_t row_count_slots(int32_t n) { return ((size_t)n + kBlock - 1) / kBlock + 1; }

int launch_list_rows(const pipad_frame *f, RowCounts *cnt, RowCounts *pre, const TotalsTicket &ticket, hipStream_t st) {
  PartRows p;
  std::memset(&p, 0, sizeof(p));
  p.rowptr[0] = f->rowptr_c;
  for (int t = 0; t < f->k; ++t) p.rowptr[1 + t] = f->rowptr_d[t];
  const dim3 blocks = grid1(f->n, kBlock);
  hipLaunchKernelGGL(k_count_rows, blocks, dim3(kBlock), 0, st, p, f->n, f->k, row_classes(f), cnt);
  const bool sum = blocks.x <= kSumRowBlocks;
  if (!sum)
    hipLaunchKernelGGL(k_scan_row_counts, dim3(1), dim3(kTileScanBlock), 0, st, cnt, pre, (int64_t)blocks.x,
                       ticket.where, ticket.seq);
  hipLaunchKernelGGL(sum ? k_list_rows<true> : k_list_rows<false>, grid1((int64_t)f->n + 1, kBlock), dim3(kBlock), 0, st, p,
                     f->n, f->k, sum ? cnt : pre, list_args(f), ticket.where, ticket.seq);
  PIPAD_HIP(hipGetLastError());
  return PIPAD_OK;
}

int set_list_sizes(pipad_frame *f, const FrameTotals &v) {
  f->n_hub = (int32_t)v.hub;
  f->n_items = (int32_t)v.units;
  f->n_long = (int32_t)v.mid;
  f->n_short = f->n - f->n_long - f->n_hub;
  f->short_entries = (int64_t)v.short_entries;
  f->split_c = f->plain_units ? 0 : (int64_t)v.split_c;
  f->split_d = f->plain_units ? 0 : (int64_t)v.split_d;
  if (f->split_c + f->split_d >= ((int64_t)1 << 31) ||
      (int64_t)(f->k + 1) * f->n_items * (f->nclass + 1) >= ((int64_t)1 << 31))
    return PIPAD_ERR_TOO_LARGE;
  return PIPAD_OK;
}

void want_split(Arena &a, pipad_frame *f) {
  if (f->plain_units) return;
  a.want(&f->sptr, (size_t)(f->k + 1) * (f->nclass + 1) * f->n_items);
  a.want(&f->scol_c, (size_t)f->split_c);
  a.want(&f->scol_d, (size_t)f->split_d);
  for (int t = 0; t < f->k; ++t) a.want_bytes(&f->swc[t], (size_t)f->split_c * scale_bytes(f));
  a.want_bytes(&f->swd, (size_t)f->split_d * scale_bytes(f));
}

template <class W>
static int fill_split_arrays(pipad_frame *f, hipStream_t st) {
  SplitArgs<W> g;
  std::memset(&g, 0, sizeof(g));
  g.n_units = f->n_items;
  g.k = f->k;
  g.sub_log2 = f->sub_log2;
  g.item_row = f->item_row;
  g.item_v0 = f->item_v0;
  g.item_v1 = f->item_v1;
  g.item_c0 = f->item_c0;
  g.item_d0 = f->item_d0;
  g.rowptr[0] = f->rowptr_c;
  g.col[0] = f->col_c;
  g.n = f->n;
  g.scales = node_scales<W>(f);
  for (int t = 0; t < f->k; ++t) {
    g.rowptr[1 + t] = f->rowptr_d[t];
    g.col[1 + t] = f->col_d[t];
    g.swc[t] = f->swc[t];
  }
  g.sptr = f->sptr;
  g.scol_c = f->scol_c;
  g.scol_d = f->scol_d;
  g.swd = static_cast<W *>(f->swd);
  auto fill = f->sub_log2 == 0 ? k_split_fill<8, W> : f->sub_log2 == 1 ? k_split_fill<16, W> : k_split_fill<32, W>;
  // a workgroup per unit for the parts that hold more than a quarter of a snapshot's entries, a wave elsewhere
  int32_t blocks = 0;
  int64_t snapshot = f->nnz_c, longest = 0;
  for (int t = 0; t < f->k; ++t) longest = std::max<int64_t>(longest, f->nnz_d[t]);
  snapshot += longest;
  double entries = 0;  // of the exclusive parts
  for (int p = 0; p <= f->k; ++p) {
    const int64_t nnz = p == 0 ? f->nnz_c : f->nnz_d[p - 1];
    const bool whole = 4 * nnz > snapshot;
    if (whole) g.whole |= 1ull << p;
    g.block_off[p] = blocks;
    blocks += whole ? f->n_items : (f->n_items + kWavesPerBlock - 1) / kWavesPerBlock;
    if (p > 0) entries += (double)nnz;
  }
  g.block_off[f->k + 1] = blocks;
  // where every XCD's run starts: at its share of the cost, a workgroup's being that of its entries, as far as the parts'
  // sizes tell, and that of 500
  const int32_t excl = blocks - g.block_off[1];
  const double scale = entries > 0 ? (double)f->split_d / entries : 0.0, each = 500.0;
  int32_t longest_run = 0;
  double front = 0;  // of the parts that end before this run starts
  g.run_off[0] = g.block_off[1];
  for (int x = 1, p = 1; x <= kClasses; ++x) {
    const double target = (scale * entries + each * excl) * x / kClasses;
    for (;; ++p) {
      const int32_t b = g.block_off[p + 1] - g.block_off[p];
      const double part = scale * f->nnz_d[p - 1] + each * b;
      if (p == f->k || front + part >= target) {
        const double share = std::min(std::max((target - front) / part, 0.0), 1.0);
        g.run_off[x] = std::max(g.run_off[x - 1], g.block_off[p] + (int32_t)(share * b));
        break;
      }
      front += part;
    }
    if (x == kClasses) g.run_off[x] = blocks;
    longest_run = std::max(longest_run, g.run_off[x] - g.run_off[x - 1]);
  }
  if (((int64_t)align_xcd(g.block_off[1]) + (int64_t)kClasses * longest_run) * kBlock >= ((int64_t)1 << 32)) {
    // (more threads than a launch takes: as many workgroups for every XCD)
    longest_run = align_xcd(excl) / kClasses;
    for (int x = 0; x < kClasses; ++x) g.run_off[x] = g.block_off[1] + std::min(x * longest_run, excl);
  }
  hipLaunchKernelGGL(fill, dim3((unsigned)(align_xcd(g.block_off[1]) + kClasses * longest_run)), dim3(kBlock), 0, st, g);
  PIPAD_HIP(hipGetLastError());
  return PIPAD_OK;
}

int build_split_arrays(pipad_frame *f, hipStream_t st) {
  if (f->n_items == 0 || f->plain_units) return PIPAD_OK;
  return f->coded ? fill_split_arrays<uint16_t>(f, st) : fill_split_arrays<float>(f, st);
}

template <class W>
static void launch_scatter(const pipad_frame *f, const Snaps &s, const Tiles &g, const OutParts &o, int instance, hipStream_t st) {
  // A wave per tile has the shortest chain of dependent loads (0.2M nodes: 65 us against 74 with four
  // tiles per wave); with 8M entries and more per snapshot there
  // are waves enough and fewer of them do better (1M nodes, 20M entries: 313 us against 339).  (Few tiles are here in frames with codes,
  // from three snapshots on by default, and where the room for `early` was refused.)
  const int per_wave = g.ntiles < kManyTiles ? 1 : 4;
  using Scatter = void (*)(Snaps, Tiles, OutParts, NodeScales<W>);
  static const Scatter kernels[2][9] = {
      {k_scatter<W, 0, false, 1>, k_scatter<W, 1, false, 1>, k_scatter<W, 1, true, 1>, k_scatter<W, 2, false, 1>,
       k_scatter<W, 2, true, 1>, k_scatter<W, 3, false, 1>, k_scatter<W, 3, true, 1>, k_scatter<W, 4, false, 1>,
       k_scatter<W, 4, true, 1>},
      {k_scatter<W, 0, false, 4>, k_scatter<W, 1, false, 4>, k_scatter<W, 1, true, 4>, k_scatter<W, 2, false, 4>,
       k_scatter<W, 2, true, 4>, k_scatter<W, 3, false, 4>, k_scatter<W, 3, true, 4>, k_scatter<W, 4, false, 4>,
       k_scatter<W, 4, true, 4>}};
  hipLaunchKernelGGL(kernels[per_wave == 1 ? 0 : 1][instance], grid1(g.ntiles, kWavesPerBlock * per_wave, f->k + 1), dim3(kBlock), 0,
                     st, s, g, o, node_scales<W>(f));
}

int build_overlap(int32_t n, int32_t k, const pipad_csr_t *snaps, uint32_t flags,
                  pipad_alloc_fn alloc, void *alloc_ctx, hipStream_t st, pipad_frame **out) {
  Snaps s;
  std::memset(&s, 0, sizeof(s));
  int64_t entries = 0;
  int32_t base = 0;
  for (int t = 0; t < k; ++t) {
    s.rowptr[t] = snaps[t].rowptr;
    s.col[t] = snaps[t].colidx;
    s.nnz[t] = snaps[t].nnz;
    entries += s.nnz[t];
    if (s.nnz[t] > s.nnz[base]) base = t;
  }

  pipad_frame *f = new (std::nothrow) pipad_frame;
  if (!f) return PIPAD_ERR_ALLOC;
  f->n = n;
  f->k = k;
  f->own_memory = alloc == nullptr;
  frame_take_options(f, entries);
  Allocator A{alloc, alloc_ctx, f};
  f->alloc = alloc;
  f->alloc_ctx = alloc_ctx;
  void *temp = nullptr;  // temporaries: from the callback (kept by the caller) or hipMalloc'd here
  bool launched = false;  // something that uses the frame's memory may be running
  // every exit path below goes through fail() or the success return
  auto fail = [&](int code) {
    if (launched) drain(st);
    if (temp && !alloc) (void)hipFree(temp);
    release(f);
    return code;
  };
  if (hipGetDevice(&f->device) != hipSuccess) return fail(hip_fail(hipGetLastError(), "hipGetDevice"));
  {
    // set-up of pipad_frame_aggregate_static on this device: look up the fixed scratch array's
    // address now, so that the entry point itself has nothing left to initialise
    float *unused_ptr = nullptr;
    size_t unused_floats = 0;
    (void)static_scratch(&unused_ptr, &unused_floats);
  }

  // ---- sizes known up front: row pointers, D^-1/2 and row lists (persistent), all temporaries
  Tiles g;
  std::memset(&g, 0, sizeof(g));
  g.n = n;
  g.k = k;
  g.base = base;
  // k_mark takes 4 bytes of LDS per entry of all stretches (20 KB for k = 8, 41 KB for k = 16 with tiles of
  // 512 entries) and 11 KB per tile; more snapshots get smaller tiles
  g.tile_log2 = k <= 16 ? 9 : 8;
  g.ntiles = (int32_t)(((int64_t)s.nnz[base] + (1 << g.tile_log2) - 1) >> g.tile_log2);

  const int64_t row_blocks = ((int64_t)n + kBlock - 1) / kBlock;
  // Small frames take two launches instead of four (or five, with the sums in a launch of their own), and get room for their
  // parts before these are known (RoomShift: 8 bytes per input entry, 82 MB at most here) together with what is sized up front,
  // so that nothing waits for the host before it has the sizes.  Whole steps and slides: N = 2k, k = 4 55 -> 48 us, N = 20k, k =
  // 4 59 -> 50, N = 1k .. 60k 60 to 80 -> 50 to 70; R-MAT 74k, k = 2 93 -> 78, Chung-Lu 125k, k = 1 62 -> 56.  Up to 2048 tiles
  // and 20000 waves of k_prepare_mark, of which 8192 run together: N = 107k, k = 8 with 2000 tiles 190 -> 186, N = 45k, k = 12
  // with 1520 181 -> 178, but N = 113k, k = 16 with 1590 180 -> 187; with 3000 to 4000 tiles and k = 2 .. 6 3 to 13 % slower.
  bool small = g.ntiles <= kSumTiles && row_blocks <= kSumRowBlocks && (int64_t)g.ntiles * k <= 20000;
  // Frames of up to 33 M entries in all snapshots get that room as well (270 MB at most), and their rows are made next to the
  // entries, in the launch that would wait for the host otherwise: steps and slides N = 100k R-MAT, k = 5 198 -> 191 us,
  // 124k, k = 2 88 -> 77, 140k, k = 3 119 -> 111; of 40 frames past the small ones 1 to 10 % less,
  // the more the shorter.  What stays unused of it, for as long as the frame is there, are 4 (k - 1) bytes per common entry: less
  // than 4 per input entry, and than what is used.  (With room for every part at its largest it was up to twice as much.)
  bool early = small || (entries <= kEarlyEntries && g.ntiles < kManyTiles);
  // From 24 M entries on the scales are stored as codes (scale_code), unless a row turns out to be too long for one; which only entries
  // whose form is known before they are written can be.  Up to 33 M entries, where that costs the room above and a wait: 24 of 28
  // drawn steps, slides, layers and backward passes 1 to 13 % faster, 4.7 in the mean, the others the same but one; 14 to 24 M between
  // 7 % faster and 4 % slower, fewer up to 18 % slower.  So are those of fewer entries with 16384 tiles (one or two snapshots), which have
  // no such room to lose: R-MAT 800k, k = 1, 10 M entries 140 -> 130 us to build, aggregations alone of 1 to 64 columns 1 % slower to 3 % faster,
  // k = 2, 18 M 178 -> 168 and 1 % slower to 5 % faster, Chung-Lu 600k, k = 2 168 -> 151 and 1 to 12 % faster.
  const bool codes =
      f->opt.scale_codes == 2 || (f->opt.scale_codes == 1 && (entries > kCodeEntries || g.ntiles >= kManyTiles));
  if (codes) small = early = false;

  Arena keep1;
  keep1.want(&f->rowptr_c, (size_t)n + 1);
  for (int t = 0; t < k; ++t) keep1.want(&f->rowptr_d[t], (size_t)n + 1);
  keep1.want(&f->dinv, (size_t)k * n);
  keep1.want(&f->dinv_nk, (size_t)node_stride(k) * n);
  want_lists(keep1, f, entries);
  // room of the parts that are written before their sizes are known (RoomShift)
  int64_t room_at[PIPAD_MAX_K + 1] = {0};  // snapshot t's entries start here without common ones
  for (int t = 0; t < k; ++t) room_at[t + 1] = room_at[t] + room_pieces(s.nnz[t]);
  auto scales_at = [&](int t) { return room_at[t] + (int64_t)t * kRoomPiece; };
  const size_t room = (size_t)(room_at[k] + kRoomPiece + scales_at(k)) * 4;

  Arena tmp;
  FrameTotals *totals = nullptr;
  int *dflags = nullptr;
  for (int t = 0; t < k; ++t) tmp.want(&g.excl[t], (size_t)s.nnz[t]);
  const size_t base_words = ((size_t)s.nnz[base] + 63) / 64;
  tmp.want(&g.bits, base_words);
  tmp.want(&g.hub_bits, base_words);
  tmp.want(&g.wpre, base_words);
  tmp.want(&g.brow, (size_t)g.ntiles + 1);
  tmp.want(&g.bound, ((size_t)g.ntiles + 1) * k);
  tmp.want(&g.tile_cnt, (size_t)g.ntiles + 1);  // (read two at a time)
  tmp.want(&g.tile_pre, (size_t)g.ntiles + 1);
  tmp.want(&g.row_cnt, row_count_slots(n));
  tmp.want(&g.row_pre, row_count_slots(n));
  tmp.want(&g.bad, 1);
  tmp.want(&totals, 1);
  tmp.want(&dflags, (size_t)64);
  // where there is no room for the parts before they are known there may be for what they take (less than a megabyte is not worth it)
  const bool tight = !early || room > (1u << 20);
  const bool together = small && one_request(f, keep1.total + room + tmp.total, kBuildTogether);
  void *base_ptr = together ? A.get(keep1.total + room + tmp.total) : nullptr;
  const bool refused = together && !base_ptr;
  if (refused && !tight) return fail(PIPAD_ERR_ALLOC);
  if (base_ptr) {
    tmp.assign(static_cast<char *>(base_ptr) + keep1.total + room);
  } else {
    if (alloc) {
      temp = alloc(tmp.total, alloc_ctx);
      f->temp_ptr = temp;
      f->temp_bytes = temp ? tmp.total : 0;
    } else if (hipMalloc(&temp, tmp.total) != hipSuccess) {
      (void)hipGetLastError();
      temp = nullptr;
    }
    if (!temp) return fail(PIPAD_ERR_ALLOC);
    tmp.assign(temp);
    if (early && !refused) base_ptr = A.get(keep1.total + room);
  }
  if (!base_ptr && tight) {
    small = early = false;
    base_ptr = A.get(keep1.total);
  }
  if (!base_ptr) return fail(PIPAD_ERR_ALLOC);
  keep1.assign(base_ptr);
  int32_t *const room_cols = reinterpret_cast<int32_t *>(static_cast<char *>(base_ptr) + keep1.total);
  float *const room_scales = reinterpret_cast<float *>(room_cols + (room_at[k] + kRoomPiece));
  // Where the parts are in that room, with so many common entries (none: where OutParts has them).
  auto place_parts = [&](int32_t common) {
    const RoomShift shift{common};
    f->col_c = room_cols;
    for (int t = 0; t < k; ++t) {
      f->col_d[t] = room_cols + (room_at[t] + shift.cols(t));
      f->wc[t] = room_scales + scales_at(t);
      f->wd[t] = room_scales + (scales_at(t) + shift.scales());
    }
  };
  if (early) place_parts(0);

  auto hipcheck = [&](hipError_t e, const char *what) { return e == hipSuccess ? 0 : hip_fail(e, what); };
#define PIPAD_TRY(call)                                   \
  do {                                                    \
    int rc__ = hipcheck((call), #call);                   \
    if (rc__ != 0) return fail(rc__);                     \
  } while (0)

  launched = true;
  if ((flags & PIPAD_VALIDATE) && n > 0) {
    PIPAD_TRY(hipMemsetAsync(dflags, 0, 256, st));
    hipLaunchKernelGGL(k_validate, grid1((int64_t)k * n, kWavesPerBlock), dim3(kBlock), 0, st, s, n,
                       k, dflags);
    int bad = 0;
    PIPAD_TRY(hipGetLastError());
    PIPAD_TRY(hipMemcpyAsync(&bad, dflags, sizeof(int), hipMemcpyDeviceToHost, st));
    PIPAD_TRY(hipStreamSynchronize(st));
    if (bad) return fail(PIPAD_ERR_BAD_CSR);
  }

  // (514 rows and the like times 2n + 2 columns have to fit a 32-bit key)
  const bool large = n >= 0x7fffffff / ((k <= 16 ? 512 : 256) + 2);
  const int cap = k <= 16 ? Mark<512>::kCap : Mark<256>::kCap, waves = k <= 16 ? k : (k + 1) / 2;
  const size_t mark_lds = (size_t)k * cap * sizeof(uint32_t);
  const int32_t hub_min = f->plain_units ? INT32_MAX : f->mid_max;  // (the classes' copies hold the hub rows' scales)
  RowArgs rows;
  std::memset(&rows, 0, sizeof(rows));
  rows.rowptr_c = f->rowptr_c;
  for (int t = 0; t < k; ++t) rows.rowptr_d[t] = f->rowptr_d[t];
  rows.scales_nk = codes ? f->dinv_nk : nullptr;
  auto out_parts = [&]() {
    OutParts o;
    std::memset(&o, 0, sizeof(o));
    o.col[0] = f->col_c;
    for (int t = 0; t < k; ++t) {
      o.col[1 + t] = f->col_d[t];
      o.wc[t] = f->wc[t];
      o.wd[t] = f->wd[t];
    }
    return o;
  };
  const int kv = k <= 2 || k > 16 ? 0 : node_stride(k) / 2 - (k % 4 ? 1 : 0);  // the instance for k snapshots
  const TotalsTicket ticket = expect_totals(totals);
  if (small) {
    const int threads = std::max(waves * kWave, kBlock);
    const int64_t row_wgs = (row_blocks + threads / kBlock - 1) / (threads / kBlock);
    if (n > 0)
      hipLaunchKernelGGL((k <= 16 ? k_prepare_mark<512, 1> : k_prepare_mark<256, 2>), dim3((unsigned)(g.ntiles + row_wgs)),
                         dim3((unsigned)threads), mark_lds, st, s, g, hub_min, row_classes(f), f->dinv, f->dinv_nk);
  } else {
    const int per_block = kBlock / (k > 8 ? 16 : 8);  // bounds
    const int32_t bound_blocks = (int32_t)(((int64_t)g.ntiles + 1 + per_block - 1) / per_block);
    hipLaunchKernelGGL((k > 8 ? k_prepare<16> : k_prepare<8>), dim3((unsigned)(bound_blocks + row_blocks)), dim3(kBlock), 0, st,
                       s, g, row_classes(f), bound_blocks, f->dinv, f->dinv_nk,
                       codes ? codes_nk(f) + (size_t)node_stride(k) * n : nullptr);
    if (g.ntiles > 0) {
      auto mark = k <= 16 ? (large ? k_mark<512, 1, uint64_t> : k_mark<512, 1, uint32_t>)
                          : (large ? k_mark<256, 2, uint64_t> : k_mark<256, 2, uint32_t>);
      hipLaunchKernelGGL(mark, dim3((unsigned)g.ntiles), dim3((unsigned)(waves * kWave)), mark_lds, st, s, g, hub_min);
    }
    ScanArgs a;
    a.tile_cnt = g.tile_cnt;
    a.tile_pre = g.tile_pre;
    a.row_cnt = g.row_cnt;
    a.row_pre = g.row_pre;
    a.bad = g.bad;
    a.ntiles = g.ntiles;
    a.k = k;
    a.row_blocks = row_blocks;
    const int64_t runs = ((int64_t)g.ntiles + kTileScanRun - 1) / kTileScanRun;
    const int64_t row_runs = (row_blocks + kTileScanBlock - 1) / kTileScanBlock;
    const int64_t blocks = std::clamp<int64_t>(std::max(runs, row_runs), 1, kTileScanMost);
    a.tiles_per_block = (int32_t)std::min<int64_t>((runs + blocks - 1) / blocks * kTileScanRun, 1 << 30);
    a.rows_per_block = (row_runs + blocks - 1) / blocks * kTileScanBlock;
    hipLaunchKernelGGL(k_scan_counts, dim3((unsigned)blocks), dim3(kTileScanBlock), 0, st, a, ticket.where, ticket.seq);
    if (!early)
      hipLaunchKernelGGL(k_rows, grid1((int64_t)n + 1, kBlock), dim3(kBlock), 0, st, s, g, rows, list_args(f));
  }
  if (early) {
    using RowsScatter = void (*)(Snaps, Tiles, RowArgs, ListArgs, OutParts, int32_t, NodeScales<float>, FrameTotals *, uint32_t);
    static const RowsScatter kernels[2][9] = {
        {k_rows_scatter<0, false, false>, k_rows_scatter<1, false, false>, k_rows_scatter<1, true, false>,
         k_rows_scatter<2, false, false>, k_rows_scatter<2, true, false>, k_rows_scatter<3, false, false>,
         k_rows_scatter<3, true, false>, k_rows_scatter<4, false, false>, k_rows_scatter<4, true, false>},
        {k_rows_scatter<0, false, true>, k_rows_scatter<1, false, true>, k_rows_scatter<1, true, true>,
         k_rows_scatter<2, false, true>, k_rows_scatter<2, true, true>, k_rows_scatter<3, false, true>,
         k_rows_scatter<3, true, true>, k_rows_scatter<4, false, true>, k_rows_scatter<4, true, true>}};
    const int32_t row_groups = (int32_t)grid1((int64_t)n + 1, kBlock).x;
    const int32_t tile_groups = (int32_t)grid1(g.ntiles, kWavesPerBlock).x;
    hipLaunchKernelGGL(kernels[small ? 1 : 0][kv], dim3((unsigned)(row_groups + tile_groups * (k + 1))), dim3(kBlock), 0, st, s, g,
                       rows, list_args(f), out_parts(), row_groups, node_scales<float>(f), ticket.where, ticket.seq);
  }
  PIPAD_TRY(hipGetLastError());

  // ---- the one host synchronisation: sizes of the data-dependent outputs (k_rows, or k_rows_scatter, runs meanwhile)
  FrameTotals v;
  {
    const int rc = wait_totals(ticket, st, &v);
    if (rc != PIPAD_OK) return fail(rc);
  }
  if (v.bad) return fail(PIPAD_ERR_BAD_CSR);
  f->nnz_c = (int32_t)v.nnz_c;
  for (int t = 0; t < k; ++t) f->nnz_d[t] = s.nnz[t] - f->nnz_c;
  {
    const int rc = set_list_sizes(f, v);
    if (rc != 0) return fail(rc);
  }

  f->coded = codes && v.uncoded == 0;

  Arena keep2;
  if (early) {
    place_parts(f->nnz_c);
  } else {
    keep2.want(&f->col_c, (size_t)f->nnz_c);
    for (int t = 0; t < k; ++t) {
      keep2.want(&f->col_d[t], (size_t)f->nnz_d[t]);
      keep2.want_bytes(&f->wc[t], (size_t)f->nnz_c * scale_bytes(f));
      keep2.want_bytes(&f->wd[t], (size_t)f->nnz_d[t] * scale_bytes(f));
    }
  }
  want_split(keep2, f);
  if (!early || (f->n_items > 0 && !f->plain_units)) {
    void *base_ptr = A.get(keep2.total);
    if (!base_ptr) return fail(PIPAD_ERR_ALLOC);
    keep2.assign(base_ptr);
  }
  if (!early && g.ntiles > 0) {
    if (f->coded) launch_scatter<uint16_t>(f, s, g, out_parts(), kv, st);
    else launch_scatter<float>(f, s, g, out_parts(), kv, st);
    PIPAD_TRY(hipGetLastError());
  }
  {
    const int rc = build_split_arrays(f, st);
    if (rc != 0) return fail(rc);
  }
  if (!alloc) {
    PIPAD_TRY(hipStreamSynchronize(st));  // the temporaries are freed next
    (void)hipFree(temp);
    temp = nullptr;
  }
#undef PIPAD_TRY
  *out = f;
  return PIPAD_OK;
}

void destroy_frame(pipad_frame *f) { release(f); }

}  // namespace pipad
