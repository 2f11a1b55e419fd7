// Internal declarations shared by the translation units of libpipad (never installed).
#ifndef PIPAD_INTERNAL_H_
#define PIPAD_INTERNAL_H_

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <new>
#include <vector>

#include "pipad.h"
#include "pipad_ranges.h"

namespace pipad {

constexpr int kWave = 64;        // gfx950 wavefront width
constexpr int kBlock = 256;      // threads per workgroup used by every kernel here (4 waves)
constexpr int kWavesPerBlock = kBlock / kWave;

// Records the text of a failed HIP call for pipad_last_hip_error() and returns PIPAD_ERR_HIP.
int hip_fail(hipError_t e, const char *what);

#define PIPAD_HIP(call)                                            \
  do {                                                             \
    hipError_t e__ = (call);                                       \
    if (e__ != hipSuccess) return ::pipad::hip_fail(e__, #call);   \
  } while (0)

struct Options {
  // structure of the frame's work lists
  int64_t short_max = 64;       // rows up to this many entries are walked whole by one lane team
  int64_t mid_max = 512;        // up to here a whole wave per row; longer rows are split by column class
  int64_t hub_threshold = 2048; // rows longer than this are also cut into units of hub_segment entries
  int64_t hub_segment = 2048;
  int64_t sub_classes = 1;      // column classes per XCD for hub rows (1, 2 or 4), taken one after the other
  int64_t agg_order = 2;        // workgroup order: 0 slices side by side, 1 one slice after the other, 2 by operand size
  // kernel choices of the aggregation
  int64_t agg_nt = 1;           // bit 0: non-temporal Y stores, bit 1: non-temporal index streams
  int64_t agg_coalescent = 1;   // small-F coalescent kernel: 0 never, 1 automatic, 2 whenever possible
  int64_t slice_cols = 0;       // columns per slice (0: automatic, else at most 64)
  int64_t agg_generic = 0;      // 1: force the generic (bounds-checked, 64-bit address) kernel
  // structure of the frame's entry lists
  int64_t scale_codes = 1;      // 16-bit codes for the entries' scales: 0 never, 1 in large frames, 2 always
};
Options &options();

}  // namespace pipad

// The frame.  All pointers are device pointers on `device`.
struct pipad_frame {
  int32_t n = 0, k = 0;
  int device = 0;
  bool own_memory = true;            // buffers came from hipMalloc (freed in destroy)
  std::vector<void *> owned;         // everything to hipFree when own_memory
  pipad_alloc_fn alloc = nullptr;    // caller's allocator (also used for the aggregate scratch)
  void *alloc_ctx = nullptr;
  void *temp_ptr = nullptr;          // the build's temporaries when they came from the caller's
  size_t temp_bytes = 0;             // allocator (see pipad_frame_temporaries)

  int32_t nnz_c = 0;
  int32_t *rowptr_c = nullptr;       // [n+1]
  int32_t *col_c = nullptr;          // [nnz_c]
  int32_t nnz_d[PIPAD_MAX_K] = {};
  int32_t *rowptr_d[PIPAD_MAX_K] = {};  // each [n+1]
  int32_t *col_d[PIPAD_MAX_K] = {};     // each [nnz_d[t]]
  float *dinv = nullptr;             // [k][n]: dinv[t*n + i]
  float *dinv_nk = nullptr;          // [n][node_stride(k)]: the same values node-major (one line per node)
  // Where `coded`, that memory holds what these are computed from (scale_code): node-major [n][node_stride(k)], and
  // behind it [k][n].
  bool coded = false;
  // Column scales stored per entry, so that the aggregation streams them instead of gathering
  // them: wc[t][e] = dinv_t[col_c[e]], wd[t][e] = dinv_t[col_d[t][e]].  Floats, or where `coded` 16-bit codes.
  void *wc[PIPAD_MAX_K] = {};
  void *wd[PIPAD_MAX_K] = {};

  // Rows are binned by length L(i) = common + longest exclusive row:
  //   short  L <= short_max   walked whole by one lane team, several rows per wave
  //   mid    L <= mid_max     walked whole by one wave
  //   hub    the rest         split by column class, one wave per class part; rows longer than
  //                           hub_threshold are first cut into units of hub_segment entries
  // A *unit* is a whole hub row or one cut of a very long one (n_items of them, in row order).
  pipad::Options opt;                // the options as they stood when the frame was built
  int32_t short_max = 0, mid_max = 0, hub_threshold = 0, hub_segment = 0;
  int32_t n_short = 0, n_long = 0;
  int64_t short_entries = 0;         // lengths of the short rows together
  int32_t *rows_short = nullptr;     // [n_short] ascending
  int32_t *rows_long = nullptr;      // [n_long] the mid rows
  int32_t n_hub = 0;
  int32_t *hub_rows = nullptr;       // [n_hub] ascending
  int32_t *hub_item_off = nullptr;   // [n_hub+1] first unit of each hub row
  int32_t n_items = 0;               // hub units
  int32_t *item_row = nullptr;       // [n_items]
  int32_t *item_v0 = nullptr;        // [n_items] the unit's range [v0, v1) of the row's virtual
  int32_t *item_v1 = nullptr;        //           entry list "common entries, then exclusive entries"

  int32_t *item_c0 = nullptr;        // [n_items] where the unit's common entries start in scol_c
  int32_t *item_d0 = nullptr;        // [n_items] where the row's exclusive entries start in scol_d

  // Column classes.  Every column belongs to one of nclass = 8 * sub classes (a hash of its
  // index); classes x * sub .. x * sub + sub - 1 are gathered by the workgroups that run on XCD x
  // only, so that the 8 private L2s hold disjoint sets of feature rows, and for hub rows the sub
  // classes of an XCD are taken one after the other in time, which divides the set of rows an L2
  // has to hold at any moment once more.  For every unit the entries of each part (0 = common,
  // 1 + t = exclusive part of snapshot t) are stored again, grouped by class (ascending column
  // within a class), the common ones in scol_c, the exclusive ones in scol_d:
  //   [sptr[(p * (nclass + 1) + c) * n_items + u], sptr[(p * (nclass + 1) + c + 1) * n_items + u])
  // are the entries of class c of unit u in part p.  swc[t] holds the column scales of scol_c for
  // snapshot t, swd those of scol_d.
  int32_t sub_log2 = 0;              // log2 of the sub classes per XCD
  int32_t nclass = 8;                // 8 << sub_log2
  int64_t split_c = 0, split_d = 0;  // common entries of the hub rows, exclusive ones of all parts
  int32_t *sptr = nullptr;           // [(k + 1) * (nclass + 1) * n_items]
  int32_t *scol_c = nullptr;         // [split_c]
  int32_t *scol_d = nullptr;         // [split_d]
  void *swc[PIPAD_MAX_K] = {};       // each [split_c]
  void *swd = nullptr;               // [split_d]
  // Small frames need no classes: a workgroup walks a unit from the lists of the parts themselves, and none
  // of the arrays above is there.
  bool plain_units = false;

  // Scratch for the partial sums of the class parts: nclass per hub unit * k * F floats (plain units: one
  // per unit, none where every hub row is one unit), grown on demand.
  float *partial = nullptr;
  size_t partial_floats = 0;
  // The concatenated operand times its scales (pipad_aggregate.hip, kTable), memory of its own: one that is replaced stays until the
  // frame goes, as recorded calls may hold it, and what replaces it is twice as large or more, or as large as any.
  float *table = nullptr;
  size_t table_floats = 0;
  size_t table_refused = SIZE_MAX;  // the least that could not be had (a request that fails may empty the allocator's cache)
};

namespace pipad {
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Sub-allocates many arrays from one allocation: first every array registers its size, then
// assign() hands out 256-byte aligned pieces of the block.
struct Arena {
  struct Want { void **slot; size_t offset; };
  std::vector<Want> wants;
  size_t total = 0;
  template <class T> void want(T **slot, size_t count) { want_bytes(reinterpret_cast<void **>(slot), count * sizeof(T)); }
  void want_bytes(void **slot, size_t bytes) {
    wants.push_back({slot, total});
    total += align_up(std::max<size_t>(bytes, 1), 256);
  }
  void assign(void *base) {
    for (const Want &w : wants) *w.slot = static_cast<char *>(base) + w.offset;
  }
};

struct Allocator {
  pipad_alloc_fn fn;
  void *ctx;
  pipad_frame *frame;
  // Returns nullptr on failure.  bytes == 0 still returns a valid (tiny) buffer.
  void *get(size_t bytes) {
    bytes = std::max<size_t>(bytes, 256);
    void *ptr = nullptr;
    if (fn) {
      ptr = fn(bytes, ctx);
    } else {
      if (hipMalloc(&ptr, bytes) != hipSuccess) {
        (void)hipGetLastError();
        ptr = nullptr;
      }
      if (ptr) frame->owned.push_back(ptr);
    }
    return ptr;
  }
};

inline void release(pipad_frame *f) {
  if (!f) return;
  if (f->own_memory)
    for (void *ptr : f->owned) (void)hipFree(ptr);
  if (f->partial && f->own_memory) (void)hipFree(f->partial);
  delete f;
}

// A small frame's temporaries come with the frame's own memory, in one request to the caller's allocator, and stay as long: a
// request takes 3 us of a host whose work is most of a small frame's step (20 of 45 us), and so does handing the
// temporaries back.  In a build they are about a third of that memory.  In a transposition with two digits they take 12 bytes per
// entry next to the 8 (k = 1, or nothing in common) and more that the frame keeps: up to 60 %, 56 for 60k nodes, k = 1, 0.9 M
// entries.  So what a frame may hold that way is bounded.
inline bool one_request(const pipad_frame *f, size_t bytes, size_t most) { return f->alloc && f->plain_units && bytes <= most; }
constexpr size_t kBuildTogether = (size_t)22 << 20, kTransposeTogether = (size_t)32 << 20;  // (1.7 to 1.9 and about 1.5 M entries)

// A build that gives up hands its memory back at once (hipFree, or the caller's allocator, which may
// give it to anyone): the kernels it has enqueued must have stopped writing to it by then.
inline void drain(hipStream_t st) {
  if (hipStreamSynchronize(st) != hipSuccess) (void)hipGetLastError();
}

inline dim3 grid1(int64_t items, int per_block, int y = 1) {
  return dim3((unsigned)((items + per_block - 1) / per_block), (unsigned)y);
}


// Helpers of the build that the transposition shares (defined in pipad_build.hip).
// Counts of a run of rows: mid rows, hub rows and hub units, and what the hub rows hold: entries (of
// all snapshots; of the exclusive parts where the parts are known) and, where known, common entries.
struct RowCounts {
  uint64_t entries;
  uint32_t common, mid, hub, units;
  uint32_t short_entries;  // lengths of the short rows
  uint32_t uncoded;        // rows too long for a scale code
};
// The data-dependent sizes as the host reads them.
struct FrameTotals {
  uint64_t split_c, split_d;  // common / exclusive entries of the hub rows
  uint32_t nnz_c, mid, hub, units, short_entries, uncoded;
  uint32_t bad;               // the snapshots are not canonical
  uint32_t seq;               // which build these sizes belong to
};
// Where a kernel puts the sizes: pinned host memory of this thread, or device memory when there is
// none.
struct TotalsTicket {
  FrameTotals *where;
  uint32_t seq;
  bool on_host;
};
TotalsTicket expect_totals(FrameTotals *device_totals);
// Waits for the sizes (the one host synchronisation of a build).
int wait_totals(const TotalsTicket &ticket, hipStream_t st, FrameTotals *out);
// Registers the row lists of a frame whose snapshots hold `entries` entries together (upper bounds:
// the lists are written before their sizes are known).
void want_lists(Arena &a, pipad_frame *f, int64_t entries);
// Lists the rows of a frame whose row pointers are in place; cnt, pre: row_count_slots(n) counts each.
int launch_list_rows(const pipad_frame *f, RowCounts *cnt, RowCounts *pre, const TotalsTicket &ticket, hipStream_t st);
size_t row_count_slots(int32_t n);
// Takes the sizes; PIPAD_ERR_TOO_LARGE when an index space overflows.
int set_list_sizes(pipad_frame *f, const FrameTotals &v);
// Bytes of an entry's scale.
inline size_t scale_bytes(const pipad_frame *f) { return f->coded ? sizeof(uint16_t) : sizeof(float); }
// Registers the class-grouped arrays.
void want_split(Arena &a, pipad_frame *f);
// Row classes and unit counts are the same for a frame and its transpose: one definition.
__host__ __device__ inline int row_class(int64_t total, int32_t short_max, int32_t mid_max) {
  return total <= short_max ? 0 : total <= mid_max ? 1 : 2;  // short, mid, hub
}
__host__ __device__ inline uint32_t hub_units(int64_t total, int32_t threshold, int32_t segment) {
  return total <= threshold ? 1u : (uint32_t)((total + segment - 1) / segment);
}
// Copies the thresholds from the options into a new frame (clamped to what int32 sizes allow).
void frame_take_options(pipad_frame *f, int64_t entries);  // (of all snapshots)
// The class-grouped copies of the hub rows' entries (sptr, scol_c, scol_d, swc, swd), once the
// frame's parts, D^-1/2 and row lists are in place.
int build_split_arrays(pipad_frame *f, hipStream_t st);
// Floats per node of the node-major copy of D^-1/2: from three snapshots on a multiple of four, so that a
// node's scales are read 16 bytes at a time whatever k is (R-MAT, N = 100k, k = 5: one scale after the
// other k_split_fill took 44 us and k_scatter 34, so 35 and 20).
__host__ __device__ inline int32_t node_stride(int32_t k) { return k <= 2 ? k : (k + 3) / 4 * 4; }
// Column class of a column index: the top 3 + sub_log2 bits of a multiplicative hash, so that the
// class's XCD is class >> sub_log2.
__host__ __device__ inline uint32_t column_class(int32_t j, int sub_log2) {
  return ((uint32_t)j * 2654435769u) >> (29 - sub_log2);
}
constexpr int kClasses = 8;      // XCDs of the chip
constexpr int kMaxSubLog2 = 2;   // at most 4 sub classes per XCD

// Workgroup b of a launch runs on XCD b mod 8.  `blocks` pieces of work are launched as align_xcd(blocks)
// workgroups (from a multiple of 8 on); xcd_run gives workgroup b of them its piece so that an XCD has a
// run of consecutive pieces, and with them a share of what the pieces read in common (pieces from `blocks` on
// do not exist).
__host__ __device__ inline int32_t align_xcd(int32_t blocks) { return (blocks + kClasses - 1) / kClasses * kClasses; }
__device__ inline int32_t xcd_run(int32_t b, int32_t blocks) {
  return b % kClasses * (align_xcd(blocks) / kClasses) + b / kClasses;
}

// The rows of two entries by a whole wave, half of it each (e: the half's entry, which exists): 32 places are looked at in one
// round trip.  Returns the half's own answer.
__device__ __forceinline__ int32_t half_row_of_entry(const int32_t *rp, int32_t n, int32_t e, int lane) {
  constexpr int H = kWave / 2;
  const int sub = lane % H, shift = lane / H * H;
  int32_t lo = 0, hi = n;  // rp[lo] <= e < rp[hi]
  while (__any(hi - lo > 1)) {
    const int32_t step = (int32_t)(((int64_t)hi - lo + H) / (H + 1));
    const int64_t idx = lo + (int64_t)(sub + 1) * step;
    const int32_t v = rp[min(idx, (int64_t)n)];
    const int m = __popc((uint32_t)(__ballot(idx < hi && v <= e) >> shift));
    lo += m * step;
    hi = (int32_t)min((int64_t)hi, (int64_t)lo + max(step, 1));
  }
  return lo;
}

// A scale as a code: 1 + the length of the node's row, in 16 bits (0: no entry, scale 0).  In frames of many entries the scales
// are most of what a build stores, and an aggregation reads as many bytes of them as of column indices: half as many this
// way, for eight instructions per entry that make the float again, bit for bit.  A frame with a row of kUncoded - 1 entries or more
// keeps floats.  R-MAT 1M, k = 8: k_scatter 311 -> 246 us, k_split_fill 216 -> 182, aggregation with F = 64 3875 -> 3844 (5058 -> 4990
// for Chung-Lu 500k, F = 128); of 30 drawn frames of more than 33 M entries in all snapshots together, whole calls 0 to 13 % faster,
// 5.6 in the mean.  Aggregations alone, seven frames of 25 to 80 M entries: 1 to 100 columns the same (R-MAT 200k, k = 8, F = 1) to 22 % faster
// (60k, k = 16, F = 4 234 -> 195 us); concatenated, where most calls read no scales, 1.4 % slower to 8 % faster.  With fewer entries, which lie
// in the caches, there is little to gain: R-MAT 147k, k = 6, 8.4 M entries F = 2 73.5 -> 73.9, to build 84 -> 87.
constexpr int32_t kUncoded = 65535;
__device__ __forceinline__ uint16_t scale_code(int32_t row_length) { return (uint16_t)min((uint32_t)row_length + 1u, 65535u); }
// x^-1/2 rounded to the nearest float, 1 <= x < 65536: the reciprocal square root of the hardware (an ulp off at most) and a
// Newton step on its exact residual.  The same bits as (float)(1.0 / sqrt((double)x)) for every such x and any
// start within three ulps.  (NaN for 0.)
__device__ __forceinline__ float scale_of_length(uint32_t x) {
  const float xf = (float)x, r = __builtin_amdgcn_rsqf(xf);
  const float h = r * r, l = fmaf(r, r, -h);
  return fmaf(-0.5f * r, fmaf(xf, l, fmaf(xf, h, -1.f)), r);
}
// (The clamp rides on the last operation and makes 0 of a NaN.  With a test for 0 instead, which became a branch, R-MAT 500k, k = 12,
// F = 16 847 us, so 810.)
__device__ __forceinline__ float scale_of(uint32_t code) { return __builtin_amdgcn_fmed3f(scale_of_length(code), 0.f, 1.f); }

// Two and four scales (float) or codes (uint16_t) next to each other.
template <class W> struct alignas(2 * sizeof(W)) Pair { W x, y; };
template <class W> struct alignas(4 * sizeof(W)) Quad { W x, y, z, w; };

// A node's scales of snapshots 4 q .. 4 q + 3 (of k; FULL: all four exist) into place `at` of their streams.
template <class W, bool FULL = false>
__device__ __forceinline__ void put_scales(void *const (&w)[PIPAD_MAX_K], int q, int32_t k, int32_t at, Quad<W> v) {
  static_cast<W *>(w[4 * q])[at] = v.x;
  if (FULL || 4 * q + 1 < k) static_cast<W *>(w[4 * q + 1])[at] = v.y;
  if (FULL || 4 * q + 2 < k) static_cast<W *>(w[4 * q + 2])[at] = v.z;
  if (FULL || 4 * q + 3 < k) static_cast<W *>(w[4 * q + 3])[at] = v.w;
}
// The same past the caches.
template <class W>
__device__ __forceinline__ void put_scales_nt(void *const (&w)[PIPAD_MAX_K], int q, int32_t k, int32_t at, Quad<W> v) {
  __builtin_nontemporal_store(v.x, static_cast<W *>(w[4 * q]) + at);
  if (4 * q + 1 < k) __builtin_nontemporal_store(v.y, static_cast<W *>(w[4 * q + 1]) + at);
  if (4 * q + 2 < k) __builtin_nontemporal_store(v.z, static_cast<W *>(w[4 * q + 2]) + at);
  if (4 * q + 3 < k) __builtin_nontemporal_store(v.w, static_cast<W *>(w[4 * q + 3]) + at);
}

// The two tables that a frame's scales (W: float) or their codes (uint16_t) are gathered from.
template <class W> struct NodeScales {
  const W *of, *nk;  // [k][n], [n][node_stride(k)]
};
// Of a frame's memory (pipad_frame): codes lie in the place of dinv_nk.
inline uint16_t *codes_nk(const pipad_frame *f) { return reinterpret_cast<uint16_t *>(f->dinv_nk); }
template <class W> NodeScales<W> node_scales(const pipad_frame *f) {
  if constexpr (sizeof(W) == sizeof(float)) return {f->dinv, f->dinv_nk};
  else return {codes_nk(f) + (size_t)node_stride(f->k) * f->n, codes_nk(f)};
}

// Inclusive sum over the lanes up to this one: within rows of 16 lanes, then across the rows.
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return x;
}

// The same for the maximum.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false));  // row_shr:1
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false));  // row_shr:2
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false));  // row_shr:4
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false));  // row_shr:8
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false));  // row_bcast:15
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false));  // row_bcast:31
  return x;
}

// The update that may follow the aggregation: H_t = Y_t W + bias.
struct UpdateSpec {
  const float *W;     // [F][Fo], row stride ldw
  int64_t ldw;
  const float *bias;  // [Fo] or null
  int32_t Fo;
  float *const *H;    // k device pointers, row stride ldh
  int64_t ldh;
};
// Where the partial sums of a call go: a buffer and its capacity in floats.  With a frame it is the
// frame's own buffer, which the call may replace by a larger one (through the frame's allocator);
// else it cannot grow (the call then allocates nothing and fails with PIPAD_ERR_SCRATCH when the
// partial sums do not fit).
struct ScratchRef {
  float **ptr;
  size_t *floats;
  pipad_frame *frame;  // it grows, and gets a table next to it, through this frame's allocator; null: a fixed array
};
// Y may be null when `update` is given and the shape allows the fused kernel.  The frame itself
// is only read.
// `subset` (nsubset distinct snapshot numbers): only these snapshots are aggregated; X[t] and Y[t]
// of the others may be null.
int aggregate_launch(const pipad_frame *f, int32_t F, const float *const *X, int64_t ldx,
                     float *const *Y, int64_t ldy, hipStream_t stream, ScratchRef scratch,
                     const UpdateSpec *update = nullptr, const int32_t *subset = nullptr,
                     int32_t nsubset = 0);

// Address, on the current device, of the library's fixed scratch array (resolved once per device).
int static_scratch(float **ptr, size_t *floats);
}

#endif  // PIPAD_INTERNAL_H_
