// pipad_frame_transpose: the frame of the transposed parts with the forward normalisation.
//
// Every part (the overlap part and the k exclusive parts) is transposed on its own - the transpose
// of an intersection is the intersection of the transposes - and all 1 + k parts go through the
// same launches.  Transposing a CSR pattern is a stable sort of its entries by column: rows arrive
// in ascending order, so they leave in ascending order within every column, which makes the result
// canonical CSR again.  The sort is a least-significant-digit radix sort with two digits of up to 10
// bits for up to a million nodes (three, then four, beyond; one of up to 12 for a few thousand nodes), written for 64-lane waves:
//
//   tiles      a part is cut into tiles of 2048, 4096 or 8192 consecutive entries, a workgroup of 8
//              waves each
//   histogram  per tile and digit value
//   scan       a workgroup per part and 64 digit values (a lane each, the tiles dealt to its waves):
//              the entries with that digit in the tiles in front, and in all tiles of the part
//   scatter    every wave ranks its share of the tile, 64 entries at a time: lanes of equal digit
//              find each other with one ballot per digit bit, the lowest of them moves the wave's
//              count of that digit on.  With the waves' counts summed up the tile goes to LDS in
//              digit order and is written out in that order, neighbouring lanes to neighbouring
//              addresses (direct stores would go to 64 different places each).  The first pass
//              reads the part's columns in place and finds the entries' rows itself: where a row starts
//              goes to LDS, a running maximum gives every entry its row
//
// The sorted columns then give the row pointers (every change of the column is a row's start) in the
// kernel that writes the entries' scales.
//
// Integer work with unique results: outputs are bit-exact regardless of scheduling.
#include <cstring>

#include "pipad_internal.h"

namespace pipad {
namespace {

constexpr int kMaxDigitBits = 10;
constexpr int kMaxDigits = 1 << kMaxDigitBits;
constexpr int kSortBlock = 512;                      // threads per workgroup of the sort
constexpr int kSortWaves = kSortBlock / kWave;
constexpr int32_t kRowsWalked = 4096;                // a wave's entries find their rows by going through so many at most

// Up to so many tiles in every part a workgroup of k_radix_scatter adds up the part's counts itself, which
// takes as long as k_radix_scan but no launch: with the lists' sums made the same way (k_list_rows) N = 2k and
// 8k, k = 3 and 4, transposition and aggregation 80 -> 69 us, N = 20k R-MAT 84 -> 79; with 32 tiles at most 81.
constexpr uint32_t kFewTiles = 64;
// Up to 8 tiles it counts the part's digits itself, straight from the keys (k_radix_hist and its launch take longer than the
// four round trips), and up to 4096 nodes, with digits of up to 12 bits and 32 tiles, the whole sort is one launch instead of
// four: 5 launches for a small transposition and the aggregation behind it, not 8.  Medians of whole backward passes: N = 1100,
// k = 1 65 -> 48 us, N = 2000, k = 6 69 -> 52, N = 2341, 16 k entries in the overlap part 66 -> 50, N = 4000, 20 k 67 -> 54, 55 k
// 66 -> 57 (on a faster host 51 -> 52); two passes: N = 6000, k = 8, 13 k 72 -> 61, N = 5000, 15 k 66 -> 57.  Digits of 12 bits where 11
// do are 6 % slower.
constexpr uint32_t kCountTiles = 8, kCountTilesOnce = 32;
constexpr int kMostDigitBits = 12;
// Where k_radix_scatter has the counts of the digits from.
enum Counts {
  kScanned,  // summed up by k_radix_scan
  kTiles,    // each tile's, from k_radix_hist
  kKeys,     // counted here
};
struct SortArgs {
  int32_t nparts;                       // 1 + k
  int32_t n;
  int32_t shift, bits;                  // digit = (key >> shift) & (2^bits - 1)
  int32_t first, last;                  // first pass: keys are the parts' columns; last: values are the result
  uint32_t part_off[PIPAD_MAX_K + 2];   // first entry of every part in the concatenated arrays
  uint32_t tile_off[PIPAD_MAX_K + 2];   // first tile of every part
  const int32_t *rowptr[PIPAD_MAX_K + 1];  // source parts
  const int32_t *col[PIPAD_MAX_K + 1];
  int32_t *col_out[PIPAD_MAX_K + 1];       // transposed parts
  const int32_t *key_in, *val_in;
  int32_t *key_out, *val_out;
  uint32_t *hist;                       // [tiles][digits]
  uint32_t *total;                      // [nparts][digits] entries per digit value
  const float4 *dinv_from;              // first pass: D^-1/2, copied by workgroups behind the tiles'
  float4 *dinv_to;
  int64_t dinv_pieces;                  // of 16 bytes
};

// Part that holds position e of a concatenated array with the given part offsets.
__device__ inline int part_of(const uint32_t *off, int nparts, uint32_t e) {
  int p = 0;
  for (int step = nparts > 1 ? 1 << (31 - __builtin_clz(nparts - 1)) : 0; step >= 1; step >>= 1)
    if (p + step < nparts && e >= off[p + step]) p += step;
  return p;
}

struct TileRange {
  int p;
  uint32_t tile, tiles;  // tile number within the part, tiles of the part
  uint32_t begin, count;  // first entry within the part, entries
};

template <int R>
__device__ inline TileRange tile_range(const SortArgs &g, uint32_t t) {
  TileRange r;
  r.p = part_of(g.tile_off, g.nparts, t);
  r.tile = t - g.tile_off[r.p];
  r.tiles = g.tile_off[r.p + 1] - g.tile_off[r.p];
  r.begin = r.tile * (uint32_t)(kSortBlock * R);
  r.count = min((uint32_t)(kSortBlock * R), g.part_off[r.p + 1] - g.part_off[r.p] - r.begin);
  return r;
}

__device__ inline const int32_t *tile_keys(const SortArgs &g, const TileRange &r) {
  return (g.first ? g.col[r.p] : g.key_in + g.part_off[r.p]) + r.begin;
}

// D^-1/2 for the new frame, by workgroups behind those of the first launch (5 us as a copy of its own, there hardly any).
__device__ inline void copy_dinv(const SortArgs &g, uint32_t block, uint32_t blocks) {
  for (int64_t x = (int64_t)block * kSortBlock + threadIdx.x; x < g.dinv_pieces; x += (int64_t)blocks * kSortBlock)
    g.dinv_to[x] = g.dinv_from[x];
}

// R entries per thread; a wave's share of a tile is R * 64 consecutive entries.
template <int R>
__global__ __launch_bounds__(kSortBlock) void k_radix_hist(SortArgs g) {
  __shared__ uint32_t cnt[kMaxDigits];
  const uint32_t tiles = g.tile_off[g.nparts];
  if (blockIdx.x >= tiles) {
    copy_dinv(g, blockIdx.x - tiles, gridDim.x - tiles);
    return;
  }
  const TileRange r = tile_range<R>(g, blockIdx.x);
  const int digits = 1 << g.bits;
  for (int d = threadIdx.x; d < digits; d += kSortBlock) cnt[d] = 0;
  const int32_t *keys = tile_keys(g, r);
  uint32_t key[R];
#pragma unroll
  for (int q = 0; q < R; ++q) key[q] = (uint32_t)keys[min((uint32_t)(q * kSortBlock) + threadIdx.x, r.count - 1)];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < R; ++q)
    if ((uint32_t)(q * kSortBlock) + threadIdx.x < r.count) atomicAdd(&cnt[(key[q] >> g.shift) & (digits - 1)], 1u);
  __syncthreads();
  uint32_t *hist = g.hist + ((uint64_t)blockIdx.x << g.bits);
  for (int d = threadIdx.x; d < digits; d += kSortBlock) hist[d] = cnt[d];
}

// A lane per digit value (64 of them per workgroup, grid.y = part): its counts in the part's tiles are
// summed up over the tiles in front.  The tiles are dealt to the waves in runs: each sums up its run,
// then goes through it again from what the runs in front hold.  Bound by its round trips to memory: with the
// counts of up to 32 tiles kept in registers in between 5.6 us, loaded twice, eight at a time, 7.8 (840 tiles).
constexpr int kScanWaves = 16;
__global__ __launch_bounds__(kScanWaves * kWave) void k_radix_scan(SortArgs g) {
  __shared__ uint32_t sums[kScanWaves][kWave];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int p = blockIdx.y;
  const uint32_t digits = 1u << g.bits, d = blockIdx.x * kWave + lane, dc = min(d, digits - 1);
  const uint32_t tiles = g.tile_off[p + 1] - g.tile_off[p];
  const uint32_t run = (tiles + kScanWaves - 1) / kScanWaves;
  const uint32_t t0 = min(wave * run, tiles), t1 = min(t0 + run, tiles);
  uint32_t *hist = g.hist + ((uint64_t)g.tile_off[p] << g.bits) + dc;
  constexpr int UN = 8;      // loads in flight together
  constexpr uint32_t KEEP = 32;  // counts of the run that stay in registers between the two goes
  uint32_t sum = 0;
  uint32_t kept[KEEP];
#pragma unroll
  for (uint32_t u = 0; u < KEEP; u += UN)
    if (t0 + u < t1)
#pragma unroll
      for (uint32_t q = u; q < u + UN; ++q) kept[q] = hist[(uint64_t)min(t0 + q, t1 - 1) << g.bits];
#pragma unroll
  for (uint32_t q = 0; q < KEEP; ++q) sum += t0 + q < t1 ? kept[q] : 0u;
  for (uint32_t t = t0 + KEEP; t < t1; t += UN) {
    uint32_t c[UN];
#pragma unroll
    for (int q = 0; q < UN; ++q) c[q] = hist[(uint64_t)min(t + q, t1 - 1) << g.bits];
#pragma unroll
    for (int q = 0; q < UN; ++q) sum += t + q < t1 ? c[q] : 0u;
  }
  sums[wave][lane] = sum;
  __syncthreads();
  uint32_t at = 0, all = 0;
  for (int w = 0; w < kScanWaves; ++w) {
    const uint32_t x = sums[w][lane];
    if (w < wave) at += x;
    all += x;
  }
  if (wave == 0 && d < digits) g.total[((uint64_t)p << g.bits) + d] = all;
#pragma unroll
  for (uint32_t q = 0; q < KEEP; ++q)
    if (t0 + q < t1) {
      if (d < digits) hist[(uint64_t)(t0 + q) << g.bits] = at;
      at += kept[q];
    }
  for (uint32_t t = t0 + KEEP; t < t1; t += UN) {
    uint32_t c[UN];
#pragma unroll
    for (int q = 0; q < UN; ++q) c[q] = hist[(uint64_t)min(t + q, t1 - 1) << g.bits];
#pragma unroll
    for (int q = 0; q < UN; ++q)
      if (t + q < t1) {
        if (d < digits) hist[(uint64_t)(t + q) << g.bits] = at;
        at += c[q];
      }
  }
}

// The lanes of the wave whose digit equals this lane's, lanes with `live` false excluded.
template <int BITS>
__device__ inline uint64_t same_digit(uint32_t digit, int bits, bool live) {
  uint64_t mask = __ballot(live);
#pragma unroll
  for (int b = 0; b < BITS; ++b)
    if (b < bits) {
      const bool bit = (digit >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      mask &= bit ? bal : ~bal;
    }
  return mask;
}

// Bound by the stores of the first pass: a tile of 4096 entries has 8 of each of 512 digits, 32 bytes to a
// place.  The next tile's go right behind them, so an XCD takes a run of tiles and its L2 puts the lines
// together (3.4 M entries: 38 -> 33 us; tiles dealt to the XCDs in turn, whole lines never met).  With rows
// found by a running maximum instead of a binary search per entry 43 -> 38 us.
// (An instance for every kind of counts: as a branch those of the tiles took 24 registers more.)
// (With 16 entries per thread held to the 128 registers that two workgroups per CU allow: 150 took the transposition of 58M
// entries from 810 to 980 us.)
template <int R, Counts C = kScanned, int BITS = kMaxDigitBits>
__global__ __launch_bounds__(kSortBlock) __attribute__((amdgpu_waves_per_eu(R == 16 ? 4 : 1))) void k_radix_scatter(SortArgs g) {
  constexpr int kDigits = 1 << BITS;
  __shared__ uint16_t rank_of[kSortWaves][kDigits];  // counts, then the first place in the tile, per wave
  __shared__ int32_t stage[kSortBlock * R];          // the tile's keys, then its values, in digit order
  __shared__ uint32_t to[kDigits];                   // place in the part minus place in the tile
  __shared__ uint32_t wave_total[kSortWaves], wave_front[kSortWaves];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const uint32_t tiles = g.tile_off[g.nparts], tile = (uint32_t)xcd_run((int32_t)blockIdx.x, (int32_t)tiles);
  if (C == kKeys && (int32_t)blockIdx.x >= align_xcd((int32_t)tiles)) {
    copy_dinv(g, blockIdx.x - align_xcd((int32_t)tiles), gridDim.x - align_xcd((int32_t)tiles));
    return;
  }
  if (tile >= tiles) return;
  const TileRange r = tile_range<R>(g, tile);
  const int digits = 1 << g.bits;
  const int32_t *keys = tile_keys(g, r);
  const uint32_t first = (uint32_t)wave * (R * kWave);  // of this wave's share
  int32_t key[R], val[R];
#pragma unroll
  for (int q = 0; q < R; ++q) key[q] = keys[min(first + q * kWave + lane, r.count - 1)];
  // entries of the part in the tiles in front, and behind, by digit
  __shared__ uint32_t in_front[C == kKeys ? kDigits : 1], behind[C == kKeys ? kDigits : 1];
  if constexpr (C == kKeys) {
    for (int d = tid; d < digits; d += kSortBlock) in_front[d] = behind[d] = 0;
    __syncthreads();
    const int32_t *const part = keys - r.begin;
    const uint32_t entries = g.part_off[r.p + 1] - g.part_off[r.p];
    constexpr int AHEAD = 8;
    for (uint32_t base = tid; base < entries; base += AHEAD * kSortBlock) {
      uint32_t d[AHEAD];
#pragma unroll
      for (int q = 0; q < AHEAD; ++q) d[q] = (uint32_t)part[min(base + q * kSortBlock, entries - 1)];
#pragma unroll
      for (int q = 0; q < AHEAD; ++q) {
        const uint32_t e = base + q * kSortBlock;
        if (e < entries && e - r.begin >= r.count)  // (e < r.begin wraps)
          atomicAdd((e < r.begin ? in_front : behind) + ((d[q] >> g.shift) & (digits - 1)), 1u);
      }
    }
  }
  if (!g.first) {
#pragma unroll
    for (int q = 0; q < R; ++q)
      val[q] = g.val_in[g.part_off[r.p] + r.begin + min(first + q * kWave + lane, r.count - 1)];
  } else if (first < r.count) {
    const int32_t *rp = g.rowptr[r.p];
    const int32_t e0 = (int32_t)(r.begin + first), e1 = (int32_t)(r.begin + min(first + R * kWave, r.count)) - 1;
    const int32_t end = half_row_of_entry(rp, g.n, lane < kWave / 2 ? e0 : e1, lane);
    const int32_t r0 = __builtin_amdgcn_readlane(end, 0), r1 = __builtin_amdgcn_readlane(end, kWave - 1);
    if (r1 - r0 < kRowsWalked) {
      // where a row starts in the share goes to LDS (rows without entries start nowhere), and a running
      // maximum gives every entry its row
      int32_t *const start = stage + first;
#pragma unroll
      for (int q = 0; q < R; ++q) start[q * kWave + lane] = 0;
      constexpr int AHEAD = 4;
      for (int32_t rb = r0 + 1; rb <= r1; rb += AHEAD * kWave) {
        int32_t a[AHEAD], b[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
          const int32_t row = min(rb + u * kWave + lane, r1);
          a[u] = rp[row];
          b[u] = rp[row + 1];
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)
          if (rb + u * kWave + lane <= r1 && a[u] < b[u]) start[min(max(a[u] - e0, 0), R * kWave - 1)] = rb + u * kWave + lane;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      int32_t row = r0;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        val[q] = (int32_t)max((uint32_t)row, wave_max((uint32_t)start[q * kWave + lane]));
        row = __builtin_amdgcn_readlane(val[q], kWave - 1);
      }
    } else {
#pragma unroll
      for (int q = 0; q < R; ++q) val[q] = r0;
      constexpr int G = R < 8 ? R : 8;  // entries that are searched for side by side
      for (int32_t step = r1 > r0 ? 1 << (31 - __builtin_clz((uint32_t)(r1 - r0))) : 0; step >= 1; step >>= 1)
#pragma unroll
        for (int h = 0; h < R; h += G) {
          int32_t at[G];
#pragma unroll
          for (int q = 0; q < G; ++q) at[q] = rp[val[h + q] + min(step, r1 - val[h + q])];
          // (left to itself the compiler waited for each load before the next: parts of few entries, N = 29k, k = 16 36 -> 25 us)
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int q = h; q < h + G; ++q)
            if (at[q - h] <= min(e0 + q * kWave + lane, e1)) val[q] += min(step, r1 - val[q]);
        }
    }
  }
  for (int x = tid; x < kSortWaves * kDigits / 2; x += kSortBlock) reinterpret_cast<uint32_t *>(rank_of)[x] = 0;
  __syncthreads();
  uint16_t *const mine = rank_of[wave];
  uint32_t rank[R];  // entries of the same digit in front, within the wave
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const bool live = first + q * kWave + lane < r.count;
    const uint32_t digit = ((uint32_t)key[q] >> g.shift) & (digits - 1);
    const uint64_t mask = same_digit<BITS>(digit, g.bits, live);
    const uint64_t below = mask & ((1ull << lane) - 1ull);
    const uint32_t before = mine[digit];
    rank[q] = before + (uint32_t)__popcll(below);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // all reads before the count moves on
    if (live && below == 0) mine[digit] = (uint16_t)(before + (uint32_t)__popcll(mask));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  __syncthreads();
  {
    // places of the digits in the tile, and of the part's digits in the part: thread t takes digits
    // 2 t and 2 t + 1 (8 t and so on of 4096)
    constexpr int PER = kDigits / kSortBlock;
    const uint32_t *hist = g.hist + ((uint64_t)tile << g.bits), *total = g.total + ((uint64_t)r.p << g.bits);
    uint32_t in_tile[PER], in_part[PER], before[PER], all = 0, all_part = 0;
    if constexpr (C == kTiles) {
      // (all counts of the part, of which there are few, instead of a launch that adds them up)
#pragma unroll
      for (int q = 0; q < PER; ++q) before[q] = in_part[q] = 0;
      const uint32_t *part = hist - ((uint64_t)r.tile << g.bits);
#pragma unroll 8
      for (uint32_t t = 0; t < r.tiles; ++t)
#pragma unroll
        for (int q = 0; q < PER; ++q) {
          const uint32_t c = part[((uint64_t)t << g.bits) + min(tid * PER + q, digits - 1)];
          before[q] += t < r.tile ? c : 0u;
          in_part[q] += c;
        }
    } else if constexpr (C == kScanned) {
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        before[q] = hist[min(tid * PER + q, digits - 1)];
        in_part[q] = total[min(tid * PER + q, digits - 1)];
      }
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      in_tile[q] = 0;
      for (int w = 0; w < kSortWaves; ++w) in_tile[q] += rank_of[w][tid * PER + q];
      if constexpr (C == kKeys) {
        const int d = min(tid * PER + q, digits - 1);
        before[q] = in_front[d];
        in_part[q] = in_front[d] + in_tile[q] + behind[d];
      }
      if (tid * PER + q >= digits) in_part[q] = 0;
      all += in_tile[q];
      all_part += in_part[q];
    }
    const uint32_t incl = wave_sum(all), incl_part = wave_sum(all_part);
    if (lane == kWave - 1) {
      wave_total[wave] = incl;
      wave_front[wave] = incl_part;
    }
    __syncthreads();
    uint32_t at = incl - all, at_part = incl_part - all_part;
    for (int w = 0; w < wave; ++w) {
      at += wave_total[w];
      at_part += wave_front[w];
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int d = tid * PER + q;
      if (d < digits) to[d] = at_part + before[q] - at;  // (mod 2^32)
      at_part += in_part[q];
      for (int w = 0; w < kSortWaves; ++w) {
        const uint32_t c = rank_of[w][d];
        rank_of[w][d] = (uint16_t)at;
        at += c;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < R; ++q) {
    rank[q] += mine[((uint32_t)key[q] >> g.shift) & (digits - 1)];
    if (first + q * kWave + lane < r.count) stage[rank[q]] = key[q];
  }
  __syncthreads();
  int32_t sorted[R];
#pragma unroll
  for (int q = 0; q < R; ++q) sorted[q] = stage[q * kSortBlock + tid];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < R; ++q)
    if (first + q * kWave + lane < r.count) stage[rank[q]] = val[q];
  __syncthreads();
  int32_t *const key_out = g.key_out + g.part_off[r.p];
  int32_t *const val_out = g.last ? g.col_out[r.p] : g.val_out + g.part_off[r.p];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const uint32_t j = (uint32_t)(q * kSortBlock) + tid;
    if (j < r.count) {
      const uint32_t pos = to[((uint32_t)sorted[q] >> g.shift) & (digits - 1)] + j;
      key_out[pos] = sorted[q];
      val_out[pos] = stage[j];
    }
  }
}

// Row pointers and scales of the transposed parts (grid.y = part), a lane per entry.  The sorted
// columns change where a row of the transposed part starts: the lane behind a change writes the row
// pointers of the rows in between (many at once by the whole wave).  wc_t[e] = dinv_t[col_c[e]] for the
// overlap part (a node's k scales from the node-major copy of D^-1/2), wd_t[e] = dinv_t[col_d_t[e]] for
// the exclusive part of snapshot t.
template <class W>  // what a scale is stored as
struct FinishArgs {
  int32_t nparts, n, k;
  uint32_t block_off[PIPAD_MAX_K + 2];    // first workgroup of every part, in their natural order
  int32_t step_xcd, step_block;           // from one XCD's exclusive workgroup to the next XCD's, and to its own next
  uint32_t part_off[PIPAD_MAX_K + 2];
  const int32_t *key;                     // sorted columns of the source, part by part
  const int32_t *col[PIPAD_MAX_K + 1];    // columns of the transposed parts
  int32_t *rowptr[PIPAD_MAX_K + 1];
  NodeScales<W> scales;
  void *wc[PIPAD_MAX_K];
  void *wd[PIPAD_MAX_K];
};

// rp[lo .. hi] = v, per lane; long runs by the whole wave.
__device__ inline void fill_run(int32_t *rp, int32_t lo, int32_t hi, int32_t v, int lane) {
  constexpr int32_t kAlone = 8;
  uint64_t many = __ballot(hi - lo >= kAlone);
  if (hi - lo < kAlone)
    for (int32_t x = lo; x <= hi; ++x) rp[x] = v;
  while (many) {
    const int l = __ffsll((unsigned long long)many) - 1;
    many &= many - 1;
    const int32_t a = __builtin_amdgcn_readlane(lo, l), b = __builtin_amdgcn_readlane(hi, l),
                  w = __builtin_amdgcn_readlane(v, l);
    for (int64_t x = (int64_t)a + lane; x <= b; x += kWave) rp[x] = w;
  }
}

// KV > 0: a node's k scales lie in KV 16-byte pieces, read together (FULL: k == 4 * KV); KV == 0: k <= 2, or k > 16, a piece after
// the other.
template <class W, int KV, bool FULL>
__global__ __launch_bounds__(kBlock) void k_finish_parts(FinishArgs<W> g) {
  const int lane = threadIdx.x % kWave;
  // (an XCD takes a run of the exclusive parts, so that it reads one or two snapshots' D^-1/2; no workgroup
  // is launched for nothing where the parts differ in size: N = 200k, k = 4 27 -> 25 us; with more than eight snapshots
  // the workgroups go in turn, N = 29k, k = 16 with hardly any common entries 23 -> 18, transposition of N = 200k, k = 16 811 -> 761)
  int p = 0;
  int32_t b = blockIdx.x;
  if (b >= align_xcd(g.block_off[1])) {
    b -= align_xcd(g.block_off[1]);
    b = g.block_off[1] + b % kClasses * g.step_xcd + b / kClasses * g.step_block;
    p = part_of(g.block_off, g.nparts, (uint32_t)b);
  }
  if ((uint32_t)b >= g.block_off[p + 1]) return;
  b -= g.block_off[p];
  const int32_t nnz = (int32_t)(g.part_off[p + 1] - g.part_off[p]);
  const int64_t e64 = (int64_t)b * kBlock + threadIdx.x;
  int32_t *const rp = g.rowptr[p];
  if (nnz == 0) {  // no entries: all workgroups of the part clear its row pointers
    for (int64_t x = e64; x <= g.n; x += (int64_t)(g.block_off[p + 1] - g.block_off[p]) * kBlock) rp[x] = 0;
    return;
  }
  if (e64 - lane >= nnz) return;  // whole wave
  const bool live = e64 < nnz;
  const int32_t e = (int32_t)min(e64, (int64_t)nnz - 1);
  const int32_t *key = g.key + g.part_off[p];
  const int32_t mine = key[e], prev = e > 0 ? key[max(e - 1, 0)] : -1;
  const int32_t c = g.col[p][e];
  fill_run(rp, prev + 1, live ? mine : prev, e, lane);
  const bool end = e64 == nnz - 1;
  fill_run(rp, mine + 1, end ? g.n : mine, nnz, lane);
  if (!live) return;
  if (p == 0) {
    if (KV > 0) {
      const Quad<W> *row = reinterpret_cast<const Quad<W> *>(g.scales.nk) + (int64_t)c * KV;
      Quad<W> v[KV > 0 ? KV : 1];
#pragma unroll
      for (int q = 0; q < KV; ++q) v[q] = row[q];
#pragma unroll
      for (int q = 0; q < KV; ++q) put_scales<W, FULL>(g.wc, q, g.k, e, v[q]);
    } else if (g.k > 2) {
      const int32_t pieces = node_stride(g.k) / 4;
      const Quad<W> *row = reinterpret_cast<const Quad<W> *>(g.scales.nk) + (int64_t)c * pieces;
      for (int q = 0; q < pieces; ++q) put_scales(g.wc, q, g.k, e, row[q]);
    } else if (g.k == 2) {
      const Pair<W> v = reinterpret_cast<const Pair<W> *>(g.scales.nk)[c];
      static_cast<W *>(g.wc[0])[e] = v.x;
      static_cast<W *>(g.wc[1])[e] = v.y;
    } else {
      static_cast<W *>(g.wc[0])[e] = g.scales.nk[c];
    }
  } else {
    static_cast<W *>(g.wd[p - 1])[e] = g.scales.of[(int64_t)(p - 1) * g.n + c];
  }
}

template <class W>
void launch_finish(const pipad_frame *g, const SortArgs &s, const int32_t *sorted_keys, hipStream_t st) {
  const int32_t n = g->n, k = g->k;
  FinishArgs<W> c;
  std::memset(&c, 0, sizeof(c));
  c.nparts = k + 1;
  c.n = n;
  c.k = k;
  for (int p = 0; p <= k + 1; ++p) c.part_off[p] = s.part_off[p];
  c.key = sorted_keys;
  c.scales = node_scales<W>(g);
  for (int p = 0; p <= k; ++p) {
    c.col[p] = s.col_out[p];
    c.rowptr[p] = p == 0 ? g->rowptr_c : g->rowptr_d[p - 1];
  }
  for (int t = 0; t < k; ++t) {
    c.wc[t] = g->wc[t];
    c.wd[t] = g->wd[t];
  }
  using Finish = void (*)(FinishArgs<W>);
  static const Finish kernels[] = {k_finish_parts<W, 0, false>, k_finish_parts<W, 1, false>, k_finish_parts<W, 1, true>,
                                   k_finish_parts<W, 2, false>, k_finish_parts<W, 2, true>,  k_finish_parts<W, 3, false>,
                                   k_finish_parts<W, 3, true>,  k_finish_parts<W, 4, false>, k_finish_parts<W, 4, true>};
  auto finish = kernels[k <= 2 || k > 16 ? 0 : node_stride(k) / 2 - (k % 4 ? 1 : 0)];
  int64_t blocks = 0;
  for (int p = 0; p <= k; ++p) {
    const int64_t nnz = (int64_t)(s.part_off[p + 1] - s.part_off[p]);
    c.block_off[p] = (uint32_t)blocks;
    blocks += nnz > 0 ? (nnz + kBlock - 1) / kBlock : std::min<int64_t>((int64_t)n / kBlock + 1, 1024);
  }
  c.block_off[k + 1] = (uint32_t)blocks;
  const int32_t first_excl = align_xcd(c.block_off[1]);
  const int32_t excl_blocks = align_xcd((int32_t)blocks - c.block_off[1]);
  c.step_xcd = k <= 8 ? excl_blocks / kClasses : 1;
  c.step_block = k <= 8 ? 1 : kClasses;
  hipLaunchKernelGGL(finish, dim3((unsigned)(first_excl + excl_blocks)), dim3(kBlock), 0, st, c);
}

}  // namespace

// The frame of the transposed patterns with the SAME D^-1/2: aggregating with it multiplies by
// the transposed normalised adjacency.
int transpose_frame(const pipad_frame *f, pipad_alloc_fn alloc, void *alloc_ctx, hipStream_t st,
                    pipad_frame **out) {
  const int32_t n = f->n, k = f->k;
  pipad_frame *g = new (std::nothrow) pipad_frame;
  if (!g) return PIPAD_ERR_ALLOC;
  g->n = n;
  g->k = k;
  g->device = f->device;
  g->own_memory = alloc == nullptr;
  g->alloc = alloc;
  g->alloc_ctx = alloc_ctx;
  g->opt = f->opt;  // the transposed frame keeps the options of the frame it comes from
  g->short_max = f->short_max;
  g->mid_max = f->mid_max;
  g->hub_threshold = f->hub_threshold;
  g->hub_segment = f->hub_segment;
  g->sub_log2 = f->sub_log2;
  g->nclass = f->nclass;
  g->plain_units = f->plain_units;
  g->coded = f->coded;
  g->nnz_c = f->nnz_c;
  for (int t = 0; t < k; ++t) g->nnz_d[t] = f->nnz_d[t];
  Allocator A{alloc, alloc_ctx, g};
  void *temp = nullptr;
  bool launched = false;  // something that uses the frame's memory may be running
  auto fail = [&](int code) {
    if (launched) drain(st);
    if (temp && !alloc) (void)hipFree(temp);
    release(g);
    return code;
  };
  auto hipcheck = [&](hipError_t e, const char *what) { return e == hipSuccess ? 0 : hip_fail(e, what); };
#define PIPAD_TRY_T(call)                                 \
  do {                                                    \
    int rc__ = hipcheck((call), #call);                   \
    if (rc__ != 0) return fail(rc__);                     \
  } while (0)

  Arena keep;
  keep.want(&g->rowptr_c, (size_t)n + 1);
  for (int t = 0; t < k; ++t) keep.want(&g->rowptr_d[t], (size_t)n + 1);
  keep.want(&g->dinv, (size_t)k * n);
  keep.want(&g->dinv_nk, (size_t)node_stride(k) * n);
  keep.want(&g->col_c, (size_t)g->nnz_c);
  for (int t = 0; t < k; ++t) {
    keep.want(&g->col_d[t], (size_t)g->nnz_d[t]);
    keep.want_bytes(&g->wc[t], (size_t)g->nnz_c * scale_bytes(g));
    keep.want_bytes(&g->wd[t], (size_t)g->nnz_d[t] * scale_bytes(g));
  }
  {
    int64_t entries = g->nnz_c;  // a row's length counts its longest exclusive row only
    for (int t = 0; t < k; ++t) entries += g->nnz_d[t];
    want_lists(keep, g, entries);
  }
  if (n == 0) {
    void *base = A.get(keep.total);
    if (!base) return fail(PIPAD_ERR_ALLOC);
    keep.assign(base);
    *out = g;
    return PIPAD_OK;
  }

  // ---- the parts side by side, cut into tiles.  Long tiles make long runs of equal digits, and with
  // them long stores; short ones make enough workgroups out of few entries.
  SortArgs s;
  std::memset(&s, 0, sizeof(s));
  s.nparts = k + 1;
  s.n = n;
  int64_t total = 0, tiles = 0;
  for (int p = 0; p <= k; ++p) {
    const int32_t nnz = p == 0 ? f->nnz_c : f->nnz_d[p - 1];
    s.part_off[p] = (uint32_t)total;
    total += nnz;
    s.rowptr[p] = p == 0 ? f->rowptr_c : f->rowptr_d[p - 1];
    s.col[p] = p == 0 ? f->col_c : f->col_d[p - 1];
  }
  s.part_off[k + 1] = (uint32_t)total;
  if (total >= ((int64_t)1 << 31)) return fail(PIPAD_ERR_TOO_LARGE);
  // Measured for the whole sort (entries per thread 4 / 8 / 16): 0.24M entries 32 / 39 / 85 us, 3.4M
  // 114 / 93 / 126, 14M 595 / 446 / 498, 62M 1619 / 1118 / 982.
  const int per_thread = total < ((int64_t)1 << 20) ? 4 : total < ((int64_t)1 << 25) ? 8 : 16;
  const int64_t tile = (int64_t)kSortBlock * per_thread;
  for (int p = 0; p <= k; ++p) {
    s.tile_off[p] = (uint32_t)tiles;
    tiles += ((int64_t)(s.part_off[p + 1] - s.part_off[p]) + tile - 1) / tile;
  }
  s.tile_off[k + 1] = (uint32_t)tiles;
  uint32_t most_tiles = 0;
  for (int p = 0; p <= k; ++p) most_tiles = std::max(most_tiles, s.tile_off[p + 1] - s.tile_off[p]);
  int bits = 1;
  while (((int64_t)1 << bits) < n) ++bits;
  const bool few = per_thread == 4 && most_tiles <= kFewTiles;
  const bool keys = few && most_tiles <= (bits > kMostDigitBits ? kCountTiles : kCountTilesOnce);
  const bool wide = keys && bits > kMaxDigitBits && bits <= kMostDigitBits;  // digits of more than 10 bits
  const int passes = wide ? 1 : (bits + kMaxDigitBits - 1) / kMaxDigitBits;
  s.bits = (bits + passes - 1) / passes;

  Arena tmp;
  RowCounts *row_cnt = nullptr, *row_pre = nullptr;
  FrameTotals *totals = nullptr;
  int32_t *key_a = nullptr, *key_b = nullptr, *val_a = nullptr, *val_b = nullptr;
  tmp.want(&key_a, (size_t)total);
  tmp.want(&key_b, passes > 1 ? (size_t)total : 0);
  tmp.want(&val_a, passes > 1 ? (size_t)total : 0);
  tmp.want(&val_b, passes > 2 ? (size_t)total : 0);
  tmp.want(&s.hist, keys ? 0 : (size_t)tiles << s.bits);
  tmp.want(&s.total, few ? 0 : (size_t)s.nparts << s.bits);
  tmp.want(&row_cnt, row_count_slots(n));
  tmp.want(&row_pre, row_count_slots(n));
  tmp.want(&totals, 1);
  const bool together = one_request(g, keep.total + tmp.total, kTransposeTogether);
  void *const base_ptr = A.get(keep.total + (together ? tmp.total : 0));
  if (!base_ptr) return fail(PIPAD_ERR_ALLOC);
  keep.assign(base_ptr);
  for (int p = 0; p <= k; ++p) s.col_out[p] = p == 0 ? g->col_c : g->col_d[p - 1];
  if (together) {
    tmp.assign(static_cast<char *>(base_ptr) + keep.total);
  } else if (alloc) {
    temp = alloc(tmp.total, alloc_ctx);
    g->temp_ptr = temp;
    g->temp_bytes = temp ? tmp.total : 0;
  } else if (hipMalloc(&temp, tmp.total) != hipSuccess) {
    (void)hipGetLastError();
    temp = nullptr;
  }
  if (!together) {
    if (!temp) return fail(PIPAD_ERR_ALLOC);
    tmp.assign(temp);
  }

  launched = true;
  // The two copies of D^-1/2 lie next to each other in every frame, padded to 256 bytes.
  const size_t dinv_bytes = (size_t)((char *)f->dinv_nk - (char *)f->dinv) + sizeof(float) * (size_t)node_stride(k) * n;
  if ((char *)g->dinv_nk - (char *)g->dinv != (char *)f->dinv_nk - (char *)f->dinv) return fail(PIPAD_ERR_INVALID_ARG);
  if (total == 0) {
    PIPAD_TRY_T(hipMemcpyAsync(g->dinv, f->dinv, dinv_bytes, hipMemcpyDeviceToDevice, st));
  } else {
    s.dinv_from = reinterpret_cast<const float4 *>(f->dinv);
    s.dinv_to = reinterpret_cast<float4 *>(g->dinv);
    s.dinv_pieces = (int64_t)((dinv_bytes + 15) / 16);
  }

  // ---- stable sort of all entries by column, digit by digit
  const int32_t *sorted_keys = key_a;
  if (total > 0) {
    for (int pass = 0; pass < passes; ++pass) {
      s.first = pass == 0;
      s.last = pass == passes - 1;
      s.shift = pass * s.bits;
      // keys alternate between the two buffers; the values of the first and last pass live elsewhere
      s.key_in = pass % 2 == 0 ? key_b : key_a;
      s.key_out = pass % 2 == 0 ? key_a : key_b;
      s.val_in = pass % 2 == 0 ? val_b : val_a;
      s.val_out = pass % 2 == 0 ? val_a : val_b;
      auto hist = per_thread == 16 ? k_radix_hist<16> : per_thread == 8 ? k_radix_hist<8> : k_radix_hist<4>;
      auto scatter = per_thread == 16 ? k_radix_scatter<16> : per_thread == 8 ? k_radix_scatter<8>
                     : wide            ? (s.bits > 11 ? k_radix_scatter<4, kKeys, 12> : k_radix_scatter<4, kKeys, 11>)
                     : keys            ? k_radix_scatter<4, kKeys>
                     : few             ? k_radix_scatter<4, kTiles>
                                       : k_radix_scatter<4>;
      const int64_t copiers = pass == 0 ? std::min<int64_t>((s.dinv_pieces + kSortBlock - 1) / kSortBlock, 2048) : 0;
      if (!keys) hipLaunchKernelGGL(hist, dim3((unsigned)(tiles + copiers)), dim3(kSortBlock), 0, st, s);
      if (!few)
        hipLaunchKernelGGL(k_radix_scan, grid1(1 << s.bits, kWave, k + 1), dim3(kScanWaves * kWave), 0, st, s);
      hipLaunchKernelGGL(scatter, dim3((unsigned)(align_xcd((int32_t)tiles) + (keys ? copiers : 0))), dim3(kSortBlock), 0, st, s);
      PIPAD_TRY_T(hipGetLastError());
      sorted_keys = s.key_out;
    }
  }
  if (g->coded) launch_finish<uint16_t>(g, s, sorted_keys, st);
  else launch_finish<float>(g, s, sorted_keys, st);
  PIPAD_TRY_T(hipGetLastError());

  // ---- row classes, work lists and the class-grouped copies, as in the build
  const TotalsTicket ticket = expect_totals(totals);
  {
    const int rc = launch_list_rows(g, row_cnt, row_pre, ticket, st);
    if (rc != 0) return fail(rc);
  }
  FrameTotals v;
  {
    const int rc = wait_totals(ticket, st, &v);
    if (rc != 0) return fail(rc);
  }
  {
    const int rc = set_list_sizes(g, v);
    if (rc != 0) return fail(rc);
  }

  Arena lists;
  want_split(lists, g);
  if (g->n_items > 0 && !g->plain_units) {
    void *base = A.get(lists.total);
    if (!base) return fail(PIPAD_ERR_ALLOC);
    lists.assign(base);
  }
  {
    const int rc = build_split_arrays(g, st);
    if (rc != 0) return fail(rc);
  }
  if (!alloc) {
    PIPAD_TRY_T(hipStreamSynchronize(st));  // the temporaries are freed next
    (void)hipFree(temp);
  }
#undef PIPAD_TRY_T
  *out = g;
  return PIPAD_OK;
}

}  // namespace pipad
