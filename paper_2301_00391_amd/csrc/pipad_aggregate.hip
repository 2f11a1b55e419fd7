// pipad_frame_aggregate: frame-parallel GCN neighbour aggregation on gfx950.
//
// Section 4.2 ("Dimension-aware parallel GNN"): the aggregation of a snapshot group is split into
// the parallel aggregation of the overlap adjacency with the features of ALL snapshots of the
// group (the coalescent features) and the per-snapshot aggregations of the exclusive parts.  Here
// both parts and the self-loop term of Eq. 1 are fused into one pass per destination row, so every
// output element is stored exactly once and no floating-point atomics are needed:
//
//   Y_t[i,:] = dinv_t[i] * ( sum_{e in common(i)}  wc_t[e] X_t[col_c[e],:]
//                          + sum_{e in delta_t(i)} wd_t[e] X_t[col_d_t[e],:]
//                          + dinv_t[i] X_t[i,:] )                            (self-loop)
//
// with wc_t[e] = dinv_t[col_c[e]], wd_t[e] = dinv_t[col_d_t[e]] stored per entry by the build, so
// the per-snapshot normalisation D_t^-1/2 (A_t + I) D_t^-1/2 costs a streamed float per entry
// instead of a gathered cache line.  The memory path is the bound (sparse row gathers, no dense
// contraction), so there is no MFMA.
//
// How one launch covers the frame.  The coalescent feature row of a node (k snapshots x F
// columns) is cut into *slices* of at most 64 columns of one snapshot (rows of 65 to 128 columns in
// one slice where that is better), and the launch goes through the slices one after the other
// (workgroups are dispatched in index order; small matrices side by side instead): the whole chip works
// on one snapshot's matrix at a time, so the caches see one matrix instead of k.
//
// Column classes.  The chip has 8 XCDs, each with a private 4 MB L2; workgroup b runs on XCD
// b mod 8.  A feature row that all 8 L2s cache occupies 8 times its size, and the gathered rows of
// a power-law graph do not fit one L2.  So every column belongs to one of 8 classes (a hash of its
// index), the entries of the long ("hub") rows are stored a second time, grouped by class, and
// the part of a row that falls into class x is walked by a workgroup whose index is x mod 8: XCD x
// only ever gathers class x, and the 8 L2s together act as one cache of 32 MB.  The price is that
// such a row is summed in 8 parts; the partial sums go through a scratch buffer and a second small
// kernel adds them in a fixed order, applies the self-loop term and the row scale, and stores the
// row.  Measured, the 8 partial sums (written and read back through memory) only pay for rows of
// several hundred entries, so the other rows - most rows, and on graphs of moderate skew most
// entries - are walked whole.
//
// Work items of a slice, by row length L = common + longest exclusive row (binned by the build):
//   hub rows    split by class; a wave per class part, the 64/LS lane teams take different
//               entries and are summed with cross-lane shuffles.  Rows beyond hub_threshold
//               entries are first cut into units (the role the paper's sliced CSR plays for load
//               balance, Section 4.1).  In small frames (plain_units) a workgroup walks a unit whole.
//   mid rows    walked whole by a wave, the same way; self-loop, row scale and store at once.
//   short rows  walked whole: a team of LS lanes (LS * VEC = slice width) per row, 64/LS rows
//               side by side, row metadata for a whole batch loaded in one go.
// Entries are fetched a team-wide chunk at a time (one coalesced load of indices and scales),
// turned into 32-bit row offsets and handed to the lane teams through LDS, so the inner loop
// issues only the 16-byte row gathers (the "vector memory instruction" of Section 4.2), four of
// them in flight per lane; the next chunk and the next row's first chunk are requested early.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "pipad_internal.h"

#ifndef PIPAD_ORDER_BYTES
#define PIPAD_ORDER_BYTES (28 << 20)
#endif
#ifndef PIPAD_ROW_ORDER_A
#define PIPAD_ROW_ORDER_A 3  // short rows of a batch are taken longest first when 2 * longest > A * mean + B
#define PIPAD_ROW_ORDER_B 2  // (in gather rounds per row)
#endif
#ifndef PIPAD_PARTIAL_NT
#define PIPAD_PARTIAL_NT 0
#endif

namespace pipad {
namespace {

// Most rows a wave takes one after the other (lane l holds the metadata of row l of the batch).
// The launch lowers these for small frames, so that the chip still gets enough waves.
constexpr int kShortRowsPerWave = 64;  // short rows, a lane team per row
constexpr int kLongRowsPerWave = 8;    // mid rows, a wave per row
#ifndef PIPAD_WIDE_BATCH
#define PIPAD_WIDE_BATCH 4
#endif
constexpr int kWideUnitsPerWave = PIPAD_WIDE_BATCH;   // class parts of hub units, a wave per part

// x / by for x < 2^31 by a multiplication (a quotient that is at most one too small, and a look at what is left).
struct Divisor {
  uint32_t by, inverse;
};
inline Divisor divisor(int64_t by) { return Divisor{(uint32_t)by, UINT32_MAX / (uint32_t)std::max<int64_t>(by, 1)}; }
__device__ __forceinline__ uint32_t divide(uint32_t x, Divisor d) {
  const uint32_t q = __umulhi(x, d.inverse);
  return x - q * d.by >= d.by ? q + 1 : q;
}

struct AggArgs {
  int32_t n, k, F;
  int32_t ls_log2;    // log2 of the lanes per slice row
  int32_t fchunks;    // slices per snapshot = ceil(F / (LS * VEC))
  int32_t nslices;    // k * fchunks
  int32_t nsel;       // snapshots this call aggregates (k, or fewer for a subset call)
  uint64_t sel[4];    // their numbers, one byte each, in the order they are taken
  int32_t n_short, n_long, n_items, n_hub;
  // workgroups of one slice ("phase"): for every sub class in turn 8 * blocks_wide for the hub
  // units (workgroup r of them takes XCD r mod 8's class), then blocks_mid for the mid rows, then
  // blocks_short (padded so that every phase starts at a multiple of 8 and the XCD a workgroup is
  // meant for is the one it runs on)
  int32_t blocks_wide, blocks_mid, blocks_short;
  int32_t team_log2;      // log2 of the lanes that walk a short row: those of a slice, or more (short_row_team)
  int32_t uneven;         // ... lanes by the length of the row (uneven_rows)
  int32_t batch_short, batch_mid, batch_wide;  // rows / class parts per wave
  int64_t blocks_per_phase;
  Divisor per_phase, per_row;  // workgroups per phase, slices
  int32_t order;      // 1: one slice after the other; else hub class parts so and the rows of all slices side by
                      // side, 0: in turn, 2: in a run of slices per XCD
  int32_t sub_log2;   // log2 of the sub classes per XCD
  int32_t nclass;     // 8 << sub_log2
  int64_t nvp;        // partial sums per slice: nclass per hub unit
  int32_t nt;         // non-temporal hints (bit 0: Y stores, bit 1: index streams)
  int32_t sg;         // coalescent kernel: snapshots per lane team (slices are snapshot groups)
  int32_t products;   // ... the sums are those of kTable
  int32_t longest_first;  // ... a wave's short rows in order of their common entries where those differ a lot
  int32_t share;        // ... the lanes of a quad fetch common entries for each other (walk_front)
  int32_t whole_units;  // coalescent kernel: one partial sum per hub unit, not one per class part
  int32_t plain;        // hub units are walked by a workgroup each, from the lists of the parts (nclass is 1 then)
  int32_t direct;       // ... and every hub row is one unit: the row is finished there, no partial sums
  int64_t ldx, ldy;
  const int32_t *rowptr_c, *col_c;
  const float *dinv;
  const int32_t *rows_short, *rows_long;
  const int32_t *item_row, *item_v0, *item_v1, *hub_rows, *hub_item_off;
  const int32_t *sptr;    // class parts of the hub rows: see pipad_frame
  const int32_t *scol_c, *scol_d;
  const void *swd;
  float *partial;
  const int32_t *rowptr_d[PIPAD_MAX_K];
  const int32_t *col_d[PIPAD_MAX_K];
  const void *wc[PIPAD_MAX_K];  // the scales: floats, or codes where `coded`
  const void *wd[PIPAD_MAX_K];
  const void *swc[PIPAD_MAX_K];
  int32_t coded;
  const float *table;     // coalescent kernel: the rows times their scales, row stride ldt (k_scale_rows)
  int64_t ldt;
  const void *nk;         // the scales node-major, or their codes where `coded`
  const float *X[PIPAD_MAX_K];
  float *Y[PIPAD_MAX_K];   // aggregation results (optional when the update is fused in)
  // fused update: H_t = Y_t W + bias
  const float *W;          // [F][Fo], row stride ldw
  const float *bias;       // [Fo] or null
  int32_t Fo;
  int64_t ldw, ldh;
  float *H[PIPAD_MAX_K];
};

// w * x, rounded whatever is done with it (never part of a fused multiply-add).
__device__ __forceinline__ float rounded(float w, float x) {
#pragma clang fp contract(off)
  float p = w * x;
  asm volatile("" : "+v"(p));
  return p;
}

// d * (a + d * x) in 64 bits, rounded to 32 at the end.
__device__ __forceinline__ float done(float d, float x, float a) {
  return (float)((double)d * ((double)a + (double)d * (double)x));
}

template <int VEC> struct V;
template <> struct V<4> {
  using T = float4;
  // 16 bytes at any multiple of 4: the global memory instructions do not ask for more
  typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
  static __device__ inline T zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
  static __device__ inline T load(const float *p) {
    const f4 q = *reinterpret_cast<const f4 *>(p);
    return make_float4(q.x, q.y, q.z, q.w);
  }
  static __device__ inline void store(float *p, T v, bool nt) {
    const f4 q = {v.x, v.y, v.z, v.w};
    if (nt) {
      // (the empty statements keep the two stores apart: merged into one they lose the hint)
      asm volatile("");
      __builtin_nontemporal_store(q, reinterpret_cast<f4 *>(p));
      asm volatile("");
    } else {
      *reinterpret_cast<f4 *>(p) = q;
    }
  }
  static __device__ inline void fma(T &a, float w, T x) {
    a.x = fmaf(w, x.x, a.x); a.y = fmaf(w, x.y, a.y); a.z = fmaf(w, x.z, a.z); a.w = fmaf(w, x.w, a.w);
  }
  static __device__ inline void add(T &a, T b) { a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w; }
  static __device__ inline T scale(float w, T a) { return make_float4(w * a.x, w * a.y, w * a.z, w * a.w); }
  static __device__ inline T product(float w, T a) { return make_float4(rounded(w, a.x), rounded(w, a.y), rounded(w, a.z), rounded(w, a.w)); }
  static __device__ inline T finish(float d, T x, T a) { return make_float4(done(d, x.x, a.x), done(d, x.y, a.y), done(d, x.z, a.z), done(d, x.w, a.w)); }
  static __device__ inline T shfl_xor(T v, int m) {
    return make_float4(__shfl_xor(v.x, m, kWave), __shfl_xor(v.y, m, kWave),
                       __shfl_xor(v.z, m, kWave), __shfl_xor(v.w, m, kWave));
  }
};
template <> struct V<2> {
  using T = float2;
  static __device__ inline T zero() { return make_float2(0.f, 0.f); }
  typedef float f2 __attribute__((ext_vector_type(2), aligned(4)));
  static __device__ inline T load(const float *p) {
    const f2 q = *reinterpret_cast<const f2 *>(p);
    return make_float2(q.x, q.y);
  }
  static __device__ inline void store(float *p, T v, bool) {
    const f2 q = {v.x, v.y};
    *reinterpret_cast<f2 *>(p) = q;
  }
  static __device__ inline void fma(T &a, float w, T x) { a.x = fmaf(w, x.x, a.x); a.y = fmaf(w, x.y, a.y); }
  static __device__ inline void add(T &a, T b) { a.x += b.x; a.y += b.y; }
  static __device__ inline T scale(float w, T a) { return make_float2(w * a.x, w * a.y); }
  static __device__ inline T product(float w, T a) { return make_float2(rounded(w, a.x), rounded(w, a.y)); }
  static __device__ inline T finish(float d, T x, T a) { return make_float2(done(d, x.x, a.x), done(d, x.y, a.y)); }
  static __device__ inline T shfl_xor(T v, int m) {
    return make_float2(__shfl_xor(v.x, m, kWave), __shfl_xor(v.y, m, kWave));
  }
};
template <> struct V<1> {
  using T = float;
  static __device__ inline T zero() { return 0.f; }
  static __device__ inline T load(const float *p) { return *p; }
  static __device__ inline void store(float *p, T v, bool nt) {
    if (nt) {
      asm volatile("");
      __builtin_nontemporal_store(v, p);
      asm volatile("");
    } else {
      *p = v;
    }
  }
  static __device__ inline void fma(T &a, float w, T x) { a = fmaf(w, x, a); }
  static __device__ inline void add(T &a, T b) { a += b; }
  static __device__ inline T scale(float w, T a) { return w * a; }
  static __device__ inline T product(float w, T a) { return rounded(w, a); }
  static __device__ inline T finish(float d, T x, T a) { return done(d, x, a); }
  static __device__ inline T shfl_xor(T v, int m) { return __shfl_xor(v, m, kWave); }
};

// What a lane needs to know about its slice.
struct Slice {
  int t;                    // snapshot
  const float *xt;          // X_t (the same for the whole workgroup)
  const float *xb;          // X_t + feature column of this lane
  float *yb;                // Y_t + feature column of this lane (null: not wanted)
  float *ht;                // H_t (fused update only)
  const float *dv;          // dinv_t
  const void *wc, *wd;      // per-entry column scales of the common / exclusive part (short rows)
  const int32_t *rpd, *cd;  // exclusive CSR of snapshot t (short rows)
  const void *swc;          // column scales of the common region of the class-grouped entries
  int fcol;
  bool fvalid;              // the lane's columns exist (F need not fill the last slice)
};

// Of snapshot t and its fc-th chunk of columns.
__device__ __forceinline__ Slice slice_setup(const AggArgs &a, int t, int fc, int fl, int vec) {
  Slice s;
  // (the slice is the same for the whole workgroup: saying so lets the per-snapshot pointers come
  // from the kernel arguments through the scalar unit)
  t = __builtin_amdgcn_readfirstlane(t);
  fc = __builtin_amdgcn_readfirstlane(fc);
  s.t = t;
  s.fcol = (fc << a.ls_log2) * vec + fl * vec;
  s.fvalid = s.fcol < a.F;
  // F need not be a multiple of vec: the lane whose columns would go past the row's end takes the
  // last vec columns (it computes and stores some of its neighbour's again, with the same bits)
  s.fcol = min(s.fcol, max(a.F - vec, 0));
  // (idle lanes read the row's last columns as well, and never store: lines that the slice's other lanes touch.
  // Reading column 0 instead brought another line of every gathered row into the last slice: N = 200k,
  // k = 4, F = 96 783 -> 605 us, F = 100 993 -> 798.)
  s.xt = a.X[t];
  s.xb = a.X[t] + s.fcol;
  s.yb = a.Y[t] ? a.Y[t] + s.fcol : nullptr;
  s.ht = a.H[t];
  s.dv = a.dinv + (int64_t)t * a.n;
  s.wc = a.wc[t];
  s.wd = a.wd[t];
  s.rpd = a.rowptr_d[t];
  s.cd = a.col_d[t];
  s.swc = a.swc[t];
  return s;
}

// One entry as fetched (column index, and the column scale's bits or code) ...
struct Raw {
  int32_t c;
  uint32_t w;
};
// ... and as staged in LDS for the lane groups: where its feature row starts, and the scale.
struct Staged {
  uint32_t off;  // FAST: byte offset of row c within the slice's matrix; else c itself
  float w;
};

// A row's two entry lists, walked as one: the common entries, then the exclusive ones.
struct Lists {
  const int32_t *colc, *cold;  // (the same for the whole wave)
  const void *wc, *wd;
};

// Where the column scales of a row's entries come from.
enum Scales {
  kStreams,   // out of the lists of scales, each product added in one operation
  kTable,     // the gathered rows hold the products (k_scale_rows); four of them are added up, then to the sum
  kProducts,  // out of the lists, with the products and sums of kTable: the same bits
  kCodes, kCodeProducts  // as kStreams and kProducts, out of lists of codes (scale_code)
};
constexpr bool coded(Scales s) { return s == kCodes || s == kCodeProducts; }

// Entry `pos` of a row whose lists start at cs / ds and hold clen / total - clen entries, or (own row,
// weight 0) past their end: such a filler may be gathered harmlessly, which lets the FAST inner loop
// run without bounds checks.
template <Scales S>
__device__ __forceinline__ Raw fetch_entry(const Lists &l, int32_t cs, int32_t clen, int32_t ds, int32_t total,
                                           int32_t pos, int32_t self, bool nt) {
  Raw r;
  r.c = self;
  r.w = 0;
  if (pos < total) {
    const bool common = pos < clen;
    const int32_t at = common ? cs + pos : ds + (pos - clen);
    const int32_t *pc = (common ? l.colc : l.cold) + at;
    using W = std::conditional_t<coded(S), uint16_t, uint32_t>;
    const W *pw = static_cast<const W *>(common ? l.wc : l.wd) + at;
    if (nt) {
      r.c = __builtin_nontemporal_load(pc);
      r.w = __builtin_nontemporal_load(pw);
    } else {
      r.c = *pc;
      r.w = *pw;
    }
  }
  return r;
}

// The same without the scale: column -1 past the end, so that no weight takes a register.
__device__ __forceinline__ Raw fetch_index(const Lists &l, int32_t cs, int32_t clen, int32_t ds, int32_t total, int32_t pos) {
  Raw r;
  r.c = -1;
  r.w = 0;
  if (pos < total) {
    const bool common = pos < clen;
    r.c = (common ? l.colc : l.cold)[common ? cs + pos : ds + (pos - clen)];
  }
  return r;
}
template <Scales S>
__device__ __forceinline__ Raw fetch(const Lists &l, int32_t cs, int32_t clen, int32_t ds, int32_t total, int32_t pos,
                                     int32_t self, bool nt) {
  return S == kTable ? fetch_index(l, cs, clen, ds, total, pos) : fetch_entry<S>(l, cs, clen, ds, total, pos, self, nt);
}

template <Scales S>
__device__ __forceinline__ uint32_t entry_column(const Raw &r) { return (uint32_t)(S == kTable ? max(r.c, 0) : r.c); }
template <Scales S>
__device__ __forceinline__ float entry_weight(const Raw &r) {
  return S == kTable ? (r.c >= 0 ? 1.f : 0.f) : coded(S) ? scale_of(r.w) : __uint_as_float(r.w);
}

// Adds the (up to) four gathered rows of one step to the sum.
template <int VEC, Scales S, int N>
__device__ __forceinline__ void add_step(const float (&w)[N], const typename V<VEC>::T (&x)[N], typename V<VEC>::T &acc) {
  using VT = V<VEC>;
  if constexpr (S == kStreams || S == kCodes) {
#pragma unroll
    for (int j = 0; j < N; ++j) VT::fma(acc, w[j], x[j]);
  } else {
    static_assert(N == 4, "");
    typename VT::T p[N];
#pragma unroll
    for (int j = 0; j < N; ++j) p[j] = w[j] == 0.f ? VT::zero() : S != kTable ? VT::product(w[j], x[j]) : x[j];  // (a filler may be infinite)
    VT::add(p[0], p[1]);
    VT::add(p[2], p[3]);
    VT::add(p[0], p[2]);
    VT::add(acc, p[0]);
  }
}

// Adds sum_e w[e] * X[col[e], :] over a row's entries (see fetch_entry) to acc.
//   first      entries q, q + team_lanes, ... of the row's first chunk, already fetched by the caller
//   team_base  first lane of the team; team_lanes lanes fetch a chunk of entries together
//   q          this lane's index within the team
//   slot/nslots  the team's lane groups take entries slot, slot + nslots, ... of each chunk
//   lds        this wave's 64 * EPL staging slots
// A chunk - EPL entries per lane of the team, so that a team of one or two lanes has eight to go on
// with, too - is fetched with coalesced loads of indices and scales (the next chunk is requested
// before the current chunk's gathers), turned into row offsets once per entry, and parked in LDS;
// every lane group then picks its entry up with a single 8-byte LDS read, so the inner loop is
// one LDS read, one add, one 16-byte gather and VEC fused multiply-adds per entry.
// (One walk over both lists instead of one each: most rows have only a few exclusive entries, and a
// walk of their own cost them a whole round of gathers.)
// The FAST inner loop needs nslots * UNR to divide team_lanes * EPL.
// BLOCKS: a lane group takes UNR entries next to each other at a time and leaves out a block that lies past the end, so that no
// more of the row is filled up than by one group alone.
// ALONE: a lane takes exactly the entries that it fetches (one lane per row and snapshot, so that the lane
// groups are the lanes of the team): nothing goes through LDS, whose bank conflicts took a third of the
// coalescent kernel's time.  Same order of the sum.  N = 200k, k = 8, concatenated, F = 1 / 2 / 4 102 / 107 /
// 111 -> 97 / 102 / 107 us; R-MAT 60k, k = 5 29 / 32.5 / 33.8 -> 27.7 / 30.8 / 32.4, 1M, k = 8 534 / 588 / 627 ->
// 532 / 576 / 619.
template <int VEC, int UNR, bool FAST, int EPL, bool ALONE = false, Scales S = kStreams, bool BLOCKS = false>
__device__ __forceinline__ void walk(const Lists &l, int32_t cs, int32_t clen, int32_t ds, int32_t len,
                            const Raw (&first)[EPL],
                            int team_base, int team_lanes,
                            int q, int slot, int nslots, const Slice &s, int64_t ldx, int32_t self,
                            bool nt, Staged *lds, typename V<VEC>::T &acc) {
  using VT = V<VEC>;
  if (len <= 0) return;
  const uint32_t row_bytes = (uint32_t)ldx * 4u;
  // FAST addressing: wave-uniform matrix base + 32-bit (row offset + this lane's column offset)
  const char *xbytes = reinterpret_cast<const char *>(s.xt);
  const uint32_t lane_bytes = (uint32_t)s.fcol * 4u;
  const float *xcol = s.xb;
  const int chunk = team_lanes * EPL;
  Staged *const mine_lds = lds + team_base * EPL;
  Raw mine[EPL], next[EPL];
#pragma unroll
  for (int j = 0; j < EPL; ++j) mine[j] = next[j] = first[j];
  // Codes: the next chunk's become scales while the rows of this one are on their way, so that a row of many chunks does not wait
  // for that in each: R-MAT 500k, k = 12, F = 10 848 -> 768 us, F = 16 810 -> 777, 200k, k = 8, F = 1 152 -> 147, concatenated, F = 12 246 ->
  // 223.  (Not by row length in lanes of one column: 76 registers, a wave fewer per SIMD, 500k, F = 1 492 -> 512.)
  constexpr bool AHEAD = coded(S) && (VEC == 4 || !BLOCKS) && FAST && !ALONE;
  auto decode = [](Raw (&r)[EPL]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < EPL; ++j) r[j].w = __float_as_uint(scale_of(r[j].w));
  };
  if (AHEAD) decode(mine);
  for (int32_t base = 0; base < len; base += chunk) {
    const int32_t cnt = min(chunk, len - base);
    const bool more = base + chunk < len;
    if (more)
#pragma unroll
      for (int j = 0; j < EPL; ++j)
        next[j] = fetch<S>(l, cs, clen, ds, len, base + chunk + j * team_lanes + q, self, nt);
    if constexpr (ALONE) {
      static_assert(FAST, "");
      typename VT::T x[EPL];
      float w[EPL];
#pragma unroll
      for (int j = 0; j < EPL; ++j) {
        w[j] = entry_weight<S>(mine[j]);
#ifdef PIPAD_NO_GATHER
        x[j] = VT::zero();
#else
        x[j] = VT::load(reinterpret_cast<const float *>(xbytes + (entry_column<S>(mine[j]) * row_bytes + lane_bytes)));
#endif
      }
      add_step<VEC, S>(w, x, acc);
#pragma unroll
      for (int j = 0; j < EPL; ++j) mine[j] = next[j];
      continue;
    }
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      Staged st;
      st.off = FAST ? entry_column<S>(mine[j]) * row_bytes : entry_column<S>(mine[j]);
      st.w = AHEAD ? __uint_as_float(mine[j].w) : entry_weight<S>(mine[j]);
      mine_lds[j * team_lanes + q] = st;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    static_assert(FAST || !BLOCKS, "");
    for (int32_t e0 = BLOCKS ? slot * UNR : 0; e0 < cnt; e0 += nslots * UNR) {
      Staged en[UNR];
      typename VT::T x[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        int32_t e = BLOCKS ? e0 + u : e0 + u * nslots + slot;
        if (!FAST) e = min(e, chunk - 1);
        en[u] = mine_lds[e];
        if (!FAST && e0 + u * nslots + slot >= cnt) en[u].w = 0.f;
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
#ifdef PIPAD_NO_GATHER  // measurement builds: everything but the row gathers (wrong results)
        x[u] = VT::zero();
#else
        if (FAST)
          x[u] = VT::load(reinterpret_cast<const float *>(xbytes + (en[u].off + lane_bytes)));
        else
          x[u] = VT::load(xcol + (int64_t)en[u].off * ldx);
#endif
      }
      if (AHEAD && more && e0 == (BLOCKS ? slot * UNR : 0)) decode(next);  // (a chunk with one behind it is full: every lane group has some of it)
      float w[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) w[u] = en[u].w;
      add_step<VEC, S>(w, x, acc);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int j = 0; j < EPL; ++j) mine[j] = next[j];
  }
}

// ---- fused update (one GCN layer: the fully connected update applied to the aggregation result,
// Eq. 1; the weights stay on chip for every row of every snapshot a workgroup meets: the
// weight reuse of Section 4.2) ----------------------------------------------------------------
// A wave parks finished rows (the slice is the whole row of one snapshot here, K = 4 * LS columns)
// in a 16-row LDS tile and multiplies a full tile by W with fp32 MFMA 16x16x4 instructions:
//   A operand  lane (m = lane % 16, g = lane / 16) supplies tile[m][g * KS + ks] at step ks
//   B operand  the same lane supplies W[g * KS + ks][16 * nt + m]
// (the instruction sums its four k values over g; KS = K / 4 steps cover every k once), and the
// result comes back as D[4 * g + r][m] in register r.
constexpr int kTileRows = 16;
constexpr int kTileStride = 68;  // floats per tile row: 64 + 4, keeps 16-byte alignment

// Copies rows [0, rows) of W (zeros from row F on) and, as row `rows`, the bias, for columns col0 ..
// col0 + cols - 1 (zeros from Fo on); four elements per thread are requested together (one after
// the other they cost a round trip to the L2 each).
__device__ __forceinline__ void stage_weights(const AggArgs &a, float *lds, int rows, int cols, int col0, int ws) {
  constexpr int B = 4;
  const int total = rows * cols;
  for (int base = threadIdx.x; base < total; base += B * kBlock) {
    float v[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int idx = min(base + u * kBlock, total - 1), kk = idx / cols;
      v[u] = a.W[(int64_t)min(kk, a.F - 1) * a.ldw + min(col0 + idx - kk * cols, a.Fo - 1)];
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int idx = base + u * kBlock, kk = idx / cols, o = idx - kk * cols;
      if (idx < total) lds[kk * ws + o] = kk < a.F && col0 + o < a.Fo ? v[u] : 0.f;
    }
  }
  for (int o = threadIdx.x; o < cols; o += kBlock)
    lds[rows * ws + o] = a.bias && col0 + o < a.Fo ? a.bias[col0 + o] : 0.f;
}

struct Sink {
  float *tile;        // this wave's [kTileRows][kTileStride]
  int32_t *rows;      // this wave's [kTileRows] row ids
  const float *wl;    // the workgroup's W in LDS: [K][Fo + 1], then the bias as row K
  int cnt;            // rows parked (wave-uniform)
};

typedef float mfma_f4 __attribute__((ext_vector_type(4)));

template <int KS>  // k values per lane group = lanes per row
__device__ __forceinline__ void sink_flush_ks(const AggArgs &a, const Slice &s, Sink &k, int lane) {
  const int m = lane & 15, g = lane >> 4;
  float av[KS];
#pragma unroll
  for (int q = 0; q < KS / 4; ++q) {
    const float4 v = *reinterpret_cast<const float4 *>(k.tile + m * kTileStride + g * KS + 4 * q);
    av[4 * q + 0] = v.x; av[4 * q + 1] = v.y; av[4 * q + 2] = v.z; av[4 * q + 3] = v.w;
  }
  const int ws = a.Fo + 1;
  for (int nt = 0; nt * 16 < a.Fo; ++nt) {  // (what lies behind the last column is never stored)
    const float *wcol = k.wl + (g * KS) * ws + 16 * nt + m;
    const float b = k.wl[(4 * KS) * ws + 16 * nt + m];  // the bias sits behind W's last row
    mfma_f4 d = {0.f, 0.f, 0.f, 0.f};
    constexpr int KB = KS < 8 ? KS : 8;  // operand reads issued together (more would spill)
#pragma unroll
    for (int k0 = 0; k0 < KS; k0 += KB) {
      float bv[KB];
#pragma unroll
      for (int ks = 0; ks < KB; ++ks) bv[ks] = wcol[(k0 + ks) * ws];
#pragma unroll
      for (int ks = 0; ks < KB; ++ks)
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(av[k0 + ks], bv[ks], d, 0, 0, 0);
    }
    // (the tile's rows are in registers: their place takes the product)
#pragma unroll
    for (int r = 0; r < 4; ++r) k.tile[(4 * g + r) * kTileStride + 16 * nt + m] = d[r] + b;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const int quads = (a.Fo + 3) / 4;  // 16-byte pieces of a row of H, the last one maybe shorter
  for (int x = lane; x < k.cnt * quads; x += kWave) {
    const int row = x / quads, q = x - row * quads;
    const float4 h = *reinterpret_cast<const float4 *>(k.tile + row * kTileStride + 4 * q);
    float *out = s.ht + (int64_t)k.rows[row] * a.ldh + 4 * q;
    if (4 * q + 4 <= a.Fo) {
      V<4>::store(out, h, a.nt & 1);
    } else {
      out[0] = h.x;
      if (4 * q + 1 < a.Fo) out[1] = h.y;
      if (4 * q + 2 < a.Fo) out[2] = h.z;
    }
  }
}

__device__ __forceinline__ void sink_flush(const AggArgs &a, const Slice &s, Sink &k, int lane) {
  if (k.cnt == 0) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  switch (a.ls_log2) {
    case 2: sink_flush_ks<4>(a, s, k, lane); break;
    case 3: sink_flush_ks<8>(a, s, k, lane); break;
    default: sink_flush_ks<16>(a, s, k, lane); break;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  k.cnt = 0;
}

// Self-loop term and row scale; the row goes to the tile (and to Y_t when that is wanted).
__device__ __forceinline__ void finish_row_to_sink(const AggArgs &a, const Slice &s, Sink &k, int slot, int fl,
                                          int32_t i, float di, float4 xi, float4 acc) {
  using VT = V<4>;
  VT::fma(acc, di, xi);
  float4 y = VT::scale(di, acc);
  if (!s.fvalid) y = make_float4(0.f, 0.f, 0.f, 0.f);  // columns past F pad K with zeros
  else if (s.yb) VT::store(s.yb + (int64_t)i * a.ldy, y, a.nt & 1);
  *reinterpret_cast<float4 *>(k.tile + slot * kTileStride + fl * 4) = y;
  if (fl == 0) k.rows[slot] = i;
}

// Self-loop term, row scale, store.
template <int VEC>
__device__ __forceinline__ void finish_row(const AggArgs &a, const Slice &s, int32_t i, float di,
                                  typename V<VEC>::T xi, typename V<VEC>::T acc) {
  using VT = V<VEC>;
  VT::fma(acc, di, xi);
  VT::store(s.yb + (int64_t)i * a.ldy, VT::scale(di, acc), a.nt & 1);
}

template <int VEC>
__device__ __forceinline__ void reduce_slots(int ls_log2, typename V<VEC>::T &acc) {
  for (int m = kWave >> 1; m >= (1 << ls_log2); m >>= 1) V<VEC>::add(acc, V<VEC>::shfl_xor(acc, m));
}

constexpr bool kPartialNt = PIPAD_PARTIAL_NT;  // non-temporal stores for the partial sums

// The t_seq-th snapshot this call aggregates (all four words are read before one is chosen, so
// that the kernel arguments are only read at constant offsets).
__device__ __forceinline__ int selected_snapshot(const AggArgs &a, int t_seq) {
  const uint64_t w0 = a.sel[0], w1 = a.sel[1], w2 = a.sel[2], w3 = a.sel[3];
  const uint64_t w = t_seq < 8 ? w0 : t_seq < 16 ? w1 : t_seq < 24 ? w2 : w3;
  return (int)((w >> ((t_seq & 7) * 8)) & 0xffu);
}

// Where partial sum `slot` (= hub unit * nclass + class) of the slice_seq-th slice of the call
// goes: all partial sums of one slice are contiguous, so a phase writes and the finishing kernel
// reads dense memory, and a call over some of the snapshots needs room for those only.
__device__ __forceinline__ float *partial_slot(const AggArgs &a, int slice_seq, int64_t slot, int fl, int vec) {
  return a.partial + (((int64_t)slice_seq * a.nvp + slot) << a.ls_log2) * vec + fl * vec;
}

// Short rows: as many as there are lane teams are walked side by side and a step lasts as long as its longest
// row.  Where the lengths within a batch differ a lot (skewed graphs: the longest row takes more
// than 1.5 times the mean number of gather rounds plus one) the wave takes its rows in order of
// decreasing work: a stable 5-bit radix sort over the lanes, ballots and one cross-lane move per
// bit.  Returns the index within the batch of the row taken as number `lane`; which rows a wave
// works on does not change.  Not for batches of similar rows, where the natural order keeps the
// rows of a step next to each other in memory (R-MAT frames, k = 8, F = 64: N = 200k 610 -> 585 us,
// 1M 3926 -> 3865; Chung-Lu frames, where it is not triggered, 1 % slower when applied regardless).
__device__ __forceinline__ int longest_first(int rounds, int rows_here, int lane) {
  int order = lane;
#ifndef PIPAD_NO_ROW_ORDER
  int mx = rounds, sm = rounds;
#pragma unroll
  for (int m = kWave >> 1; m >= 1; m >>= 1) {
    mx = max(mx, __shfl_xor(mx, m, kWave));
    sm += __shfl_xor(sm, m, kWave);
  }
  if (2 * mx * rows_here > PIPAD_ROW_ORDER_A * sm + PIPAD_ROW_ORDER_B * rows_here) {  // wave-uniform
    int packed = (min(rounds, 31) << 8) | lane;
#pragma unroll
    for (int bit = 8; bit < 13; ++bit) {
      const bool one = (packed >> bit) & 1;
      const uint64_t ones = __ballot(one);
      const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(ones >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ones, 0));
      const int dest = one ? below : __popcll(ones) + (lane - below);
      packed = __builtin_amdgcn_ds_permute(dest << 2, packed);
    }
    order = packed & 0xff;
  }
#endif
  return order;
}

#ifndef PIPAD_AGG_DEPTH
#define PIPAD_AGG_DEPTH 4  // row gathers in flight per lane
#endif
// A wave-wide team has 64 / LS lane groups and a chunk of 64 * EPL entries, EPL >= 4 / LS (launch()).
static_assert(PIPAD_AGG_DEPTH <= 4, "more gathers in flight than a chunk holds");

// What a wave of a workgroup walks of a plain hub unit: a quarter of the unit's range of the row's two
// lists, taken as one.
struct Piece {
  int32_t i, cs, clen, ds, len;
};
__device__ __forceinline__ Piece unit_piece(const AggArgs &a, int64_t unit, const int32_t *rpd, int wave) {
  Piece p;
  p.i = a.item_row[unit];
  const int32_t v0 = a.item_v0[unit], v1 = a.item_v1[unit];
  p.cs = a.rowptr_c[p.i];
  p.clen = a.rowptr_c[p.i + 1] - p.cs;
  p.ds = rpd[p.i];
  const int32_t end = min(v1, p.clen + rpd[p.i + 1] - p.ds);
  const int32_t quarter = (max(end - v0, 0) + kWavesPerBlock - 1) / kWavesPerBlock;
  const int32_t at = min(v0 + wave * quarter, end), skip = min(at, p.clen);
  p.len = min(quarter, end - at);
  p.cs += skip;
  p.clen -= skip;
  p.ds += at - skip;
  return p;
}

// Lane groups that walk a short row.
enum Teams {
  kOneGroup,
  kSeveral,   // the same number for every row (short_row_team)
  kByLength,  // up to 8 entries one, up to 32 four, from there on eight (uneven_rows)
};

// Lanes of a mask below this one.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// PLAIN: hub units as they are in a frame with plain_units.
template <int VEC, bool FAST, int EPL, bool UPD, bool PLAIN, bool ALONE = false, Scales S = kStreams, Teams TEAMS = kOneGroup>
__device__ __forceinline__ void aggregate_body(const AggArgs &a) {
  using VT = V<VEC>;
  static_assert(TEAMS == kOneGroup || (FAST && !ALONE), "");
  static_assert(TEAMS != kByLength || !UPD, "");
  static_assert(!UPD || (VEC == 4 && FAST), "the fused update rides on the fast float4 path");
  extern __shared__ __align__(16) float upd_lds[];  // UPD: W [K][Fo + 1], then the waves' tiles and row ids
  Sink sink;
  // Row gathers in flight per lane.  Measured on MI355X (N = 1M R-MAT frame): 4 beats 2 and 8;
  // deeper bursts only queue up in front of the L1's miss slots.
  constexpr int U = FAST ? PIPAD_AGG_DEPTH : 1;
  __shared__ Staged staging[kWavesPerBlock][kWave * EPL];
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  Staged *lds = staging[wave];
  const int ls = 1 << a.ls_log2;
  const int fl = lane & (ls - 1);
  const int team = lane >> a.ls_log2;  // lane group index within the wave
  const int nteams = kWave >> a.ls_log2;

  // Workgroups are dispatched in index order and dealt round-robin to the XCDs: the launch goes
  // through the slices (snapshot-major) one after the other, and within a slice's class parts the
  // class of a workgroup is its index mod 8.
  // (A wave of a small frame takes 8 to 16 rows, and half of its 660 instructions were about which: so 32-bit numbers, there are fewer
  // than 2^31 workgroups, divisions by a multiplication, the wave's number known to be one, and no order for rows that are all
  // taken at once.  N = 20k, k = 4, F = 32 15.8 -> 14.3 us, 37k, k = 8, F = 16 26.6 -> 23.0, R-MAT 8k, k = 5, F = 16 12.7 -> 10.8.)
  const uint32_t b = blockIdx.x;
  const uint32_t wide_blocks = kClasses * a.blocks_wide;  // per sub class
  const uint32_t split_blocks = PLAIN ? a.n_items : wide_blocks << a.sub_log2;
  uint32_t slice_seq;
  uint32_t w;  // workgroup index within the slice's phase: class parts, mid rows, short rows
  if (a.order == 1) {
    slice_seq = divide(b, a.per_phase);
    w = b - slice_seq * a.per_phase.by;
  } else {
    // Side by side: neighbouring workgroups take the same rows in different slices, so the
    // entry lists they share (the overlap part's indices, the row pointers) are fetched once for
    // all of them - what pays while the operand is small next to the index streams.  The class
    // parts keep their slice-after-slice order in front (their class is the workgroup index mod 8).
    const uint32_t nsl = a.per_row.by;
    const uint32_t hub_total = split_blocks * nsl;
    if (b < hub_total) {
      slice_seq = b / split_blocks;
      w = b - slice_seq * split_blocks;
    } else {
      const uint32_t r = b - hub_total;
      if (a.order == 0) {
        const uint32_t q = divide(r, a.per_row);
        slice_seq = r - q * nsl;
        w = split_blocks + q;
      } else {
        // The workgroups of a slice's mid rows, dealt into 8 parts, make 8 * nsl parts in slice order, of
        // which XCD x takes nsl in a row: it only ever reads two or three of the matrices.  All mid
        // rows first, then the short ones the same way.
        const uint32_t x = r & (kClasses - 1);
        uint32_t i = r / kClasses, part = a.blocks_mid / kClasses, start = 0;
        if (i >= part * nsl) {
          i -= part * nsl;
          start = a.blocks_mid;
          part = (a.per_phase.by - split_blocks - start) / kClasses;
        }
        const uint32_t q = i / part, share = nsl * x + q;
        slice_seq = share / kClasses;
        w = split_blocks + start + (i - q * part) * kClasses + share % kClasses;
      }
    }
  }
  const int t_seq = a.fchunks == 1 ? slice_seq : slice_seq / a.fchunks;
  const Slice s = slice_setup(a, selected_snapshot(a, t_seq), slice_seq - t_seq * a.fchunks, fl, VEC);
  const bool ntl = a.nt & 2;

  if (UPD && w < split_blocks && !a.direct) {
    sink.cnt = 0;  // (class parts of hub units end in partial sums: no use for W)
  } else if (UPD) {
    const int K = 4 << a.ls_log2, ws = a.Fo + 1;
    // (row K: the bias; a load from global memory inside the flush would make the wave wait for every gather
    // it has in flight)
    stage_weights(a, upd_lds, K, a.Fo, 0, ws);
    const int w_floats = ((K + 1) * ws + 3) & ~3;
    float *tiles = upd_lds + w_floats;
    sink.wl = upd_lds;
    sink.tile = tiles + (threadIdx.x / kWave) * kTileRows * kTileStride;
    sink.rows = reinterpret_cast<int32_t *>(tiles + kWavesPerBlock * kTileRows * kTileStride) +
                (threadIdx.x / kWave) * kTileRows;
    sink.cnt = 0;
    __syncthreads();  // before any wave leaves
  }

  if (PLAIN && w < split_blocks) {
    // ---- a hub unit by the whole workgroup, a quarter of its entries per wave, the waves' sums added in
    //      order: a row of 2048 entries has 32 rounds of gathers one after the other (F = 64), as a mid row
    //      of 512, and is finished here unless it is cut
    __shared__ typename VT::T sums[kWavesPerBlock][kWave / 2];
    const Piece p = unit_piece(a, w, s.rpd, wave);
    Lists l;
    l.colc = a.col_c;
    l.wc = s.wc;
    l.cold = s.cd;
    l.wd = s.wd;
    Raw head[EPL];
#pragma unroll
    for (int j = 0; j < EPL; ++j) head[j] = fetch_entry<S>(l, p.cs, p.clen, p.ds, p.len, j * kWave + lane, p.i, ntl);
    const typename VT::T xi = VT::load(s.xb + (int64_t)p.i * a.ldx);
    const float di = s.dv[p.i];
    typename VT::T acc = VT::zero();
    walk<VEC, U, FAST, EPL, ALONE, S>(l, p.cs, p.clen, p.ds, p.len, head, 0, kWave, lane, team, nteams, s, a.ldx, p.i, ntl, lds,
                                   acc);
    reduce_slots<VEC>(a.ls_log2, acc);
    if (team == 0) sums[wave][fl] = acc;
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int x = 1; x < kWavesPerBlock; ++x) VT::add(acc, sums[x][fl]);
    if (!a.direct) {
      if (team == 0 && s.fvalid) VT::store(partial_slot(a, slice_seq, w, fl, VEC), acc, kPartialNt);
    } else if constexpr (UPD) {
      if (team == 0) finish_row_to_sink(a, s, sink, 0, fl, p.i, di, xi, acc);
      sink.cnt = 1;
      sink_flush(a, s, sink, lane);
    } else {
      if (team == 0 && s.fvalid) finish_row<VEC>(a, s, p.i, di, xi, acc);
    }
    return;
  }

  // ---- what this wave works on: a batch of consecutive list elements.  Class parts of hub units
  //      (from the class-grouped copies, ending in a partial sum) and whole mid rows: the whole
  //      wave on one list at a time, its lane groups taking different entries.  Short rows: one
  //      lane group each, nteams side by side.  The metadata of the whole batch is loaded up front
  //      (lane l holds element l of the batch), and while one element is being gathered the first
  //      chunk of entries (and, for whole rows, the self-loop row) of the next one are already on
  //      their way.
  // (every field is read into a local before the control flow that chooses among them, so that
  // the kernel arguments are only ever read at constant offsets)
  const int32_t *const p_items = a.item_row, *const p_mid = a.rows_long, *const p_short = a.rows_short;
  const int32_t n_items = a.n_items, n_mid = a.n_long, n_short = a.n_short;
  const int b_wide = a.batch_wide, b_mid = a.batch_mid, b_short = a.batch_short;
  const bool split = !PLAIN && w < split_blocks;        // class parts of hub units
  const bool wide = w < split_blocks + a.blocks_mid;    // ... or whole mid rows: a wave per list
  int cls = 0;  // column class of this wave's class parts
  if (split) {
    const int sub = (int)(w / wide_blocks);  // the sub classes come one after the other in time
    w -= sub * wide_blocks;
    cls = ((int)(w & (kClasses - 1)) << a.sub_log2) + sub;
    w >>= 3;
  } else if (wide) {
    w -= split_blocks;
  } else {
    w -= split_blocks + a.blocks_mid;
  }
  const int32_t *list = split ? p_items : wide ? p_mid : p_short;
  const int32_t list_len = split ? n_items : wide ? n_mid : n_short;
  const int batch = split ? b_wide : wide ? b_mid : b_short;
  const int64_t first64 = ((int64_t)w * kWavesPerBlock + wave) * batch;
  if (first64 >= list_len) return;
  const int32_t first = (int32_t)first64;
#ifdef PIPAD_PARTS_MASK  // measurement builds only: which kinds of work items run (results incomplete)
  if (!((PIPAD_PARTS_MASK) & (split ? 1 : wide ? 2 : 4))) return;
#endif
  const int rows_here = min(batch, list_len - first);
  // entry lists: the class-grouped copies for hub units, the frame's CSRs for whole rows
  Lists lists;
  lists.colc = split ? a.scol_c : a.col_c;
  lists.wc = split ? s.swc : s.wc;
  lists.cold = split ? a.scol_d : s.cd;
  lists.wd = split ? a.swd : s.wd;
  // hub units only: first partial sum; nclass of them per unit
  const int64_t v_first = (int64_t)first * a.nclass + cls;
  int32_t r = 0, mc0 = 0, mc1 = 0, md0 = 0, md1 = 0;
  float mdi = 0.f;
  if (lane < rows_here) {
    r = list[first + lane];
    if (split) {
      const int32_t *sp = a.sptr + (int64_t)cls * n_items + first + lane;
      mc0 = sp[0];
      mc1 = sp[n_items];
      sp += (int64_t)(1 + s.t) * (a.nclass + 1) * n_items;
      md0 = sp[0];
      md1 = sp[n_items];
    } else {
      mc0 = a.rowptr_c[r]; mc1 = a.rowptr_c[r + 1];
      md0 = s.rpd[r]; md1 = s.rpd[r + 1];
      mdi = s.dv[r];
    }
  }
  const int team_log2 = TEAMS == kSeveral ? a.team_log2 : a.ls_log2;  // of a short row (kByLength: at least)
  const int per_step = wide ? 1 : kWave >> team_log2;     // elements worked on side by side
  int order = lane;
  int n8 = 0, n4 = 0;  // kByLength: rows of eight and of four lane groups, which come first
  if constexpr (TEAMS == kByLength) {
    if (!wide) {
      const int len = lane < rows_here ? mc1 - mc0 + md1 - md0 : 0;
      const uint64_t eight = __ballot(len > 32), four = __ballot(len > 8) & ~eight;
      n8 = __popcll(eight);
      n4 = __popcll(four);
      if (n8 + n4 > 0) {
        const bool in8 = eight >> lane & 1ull, in4 = four >> lane & 1ull;
        const int at = lanes_below(in8 ? eight : in4 ? four : ~(eight | four)) + (in8 ? 0 : in4 ? n8 : n8 + n4);
        order = __builtin_amdgcn_ds_permute(at << 2, lane);
      }
    }
  } else if (!wide && rows_here > per_step && ((VEC * 4) << a.ls_log2) >= 128) {
    // (not for slices narrower than a cache line, where neighbouring rows share lines, and not for rows that are all taken at once)
    order = longest_first(lane < rows_here ? (mc1 - mc0 + md1 - md0 + U - 1) / U : 0, rows_here, lane);
  }
  // (kByLength alone: the compiler cannot know that the quotients are 0 elsewhere)
  const int steps8 = TEAMS == kByLength ? (8 * n8 + nteams - 1) / nteams : 0;
  const int steps4 = TEAMS == kByLength ? (4 * n4 + nteams - 1) / nteams : 0;

  // What a step takes: elements at, at + 1, ... in front of `end`, each by a team of 1 << log2 lanes.
  struct Shape {
    int at, end, log2;
  };
  auto shape = [&](int step) __attribute__((always_inline)) {
    Shape h = {step * per_step, rows_here, wide ? 6 : team_log2};
    if constexpr (TEAMS == kByLength) {
      if (step < steps8) {
        h = {step * (nteams / 8), n8, team_log2 + 3};
      } else if (step < steps8 + steps4) {
        h = {n8 + (step - steps8) * (nteams / 4), n8 + n4, team_log2 + 2};
      } else {
        h.at = n8 + n4 + (step - steps8 - steps4) * per_step;
      }
    }
    return h;
  };
  // This lane's place in its team, the same in every step but for kByLength.
  struct Place {
    int team, base, lanes, q, slot, nslots;
  };
  Place same;
  same.team = wide ? 0 : TEAMS == kOneGroup ? team : lane >> team_log2;
  same.base = wide ? 0 : same.team << team_log2;
  same.lanes = wide ? kWave : 1 << team_log2;
  same.q = wide ? lane : TEAMS == kOneGroup ? fl : lane - same.base;
  same.slot = wide ? team : TEAMS == kOneGroup ? 0 : same.q >> a.ls_log2;
  same.nslots = wide ? nteams : TEAMS == kOneGroup ? 1 : same.lanes >> a.ls_log2;
  auto place = [&](const Shape &h) __attribute__((always_inline)) {
    Place p = same;
    if (TEAMS == kByLength && !wide) {
      p.team = lane >> h.log2;
      p.base = p.team << h.log2;
      p.lanes = 1 << h.log2;
      p.q = lane - p.base;
      p.slot = p.q >> a.ls_log2;
      p.nslots = p.lanes >> a.ls_log2;
    }
    return p;
  };

  struct Item {
    int32_t i, cs, clen, ds, len;  // len: both lists together
    float di;
    bool have;
    Raw first[EPL];
    typename VT::T xi;
  };
  auto prefetch = [&](int step) __attribute__((always_inline)) {
    Item it;
    const Shape h = shape(step);
    const Place p = place(h);
    const int li = h.at + p.team;
    it.have = li < h.end;
    const int src = __shfl(order, it.have ? li : 0, kWave);
    it.i = __shfl(r, src, kWave);
    it.cs = __shfl(mc0, src, kWave);
    it.clen = __shfl(mc1, src, kWave) - it.cs;
    it.ds = __shfl(md0, src, kWave);
    it.len = it.clen + __shfl(md1, src, kWave) - it.ds;
    it.di = __shfl(mdi, src, kWave);
    if (!it.have) { it.clen = 0; it.len = 0; }
#pragma unroll
    for (int j = 0; j < EPL; ++j)
      it.first[j] = fetch_entry<S>(lists, it.cs, it.clen, it.ds, it.len, j * p.lanes + p.q, it.i, ntl);
    it.xi = VT::zero();
    if (!split) it.xi = VT::load(s.xb + (int64_t)it.i * a.ldx);
    return it;
  };
  const int nsteps = steps8 + steps4 + (rows_here - n8 - n4 + per_step - 1) / per_step;
  Item nxt = prefetch(0);
  for (int step = 0; step < nsteps; ++step) {
    const Item cur = nxt;
    const int rows_now = wide ? 1 : min(per_step, rows_here - step * per_step);
    if constexpr (UPD) {
      // Make room in the tile before the next rows' loads are requested: the multiplication then
      // runs while nothing but this step's (already needed) data is in flight, and its registers
      // do not compete with the prefetched rows.
      if (!split && sink.cnt + rows_now > kTileRows) sink_flush(a, s, sink, lane);
    }
    if (step + 1 < nsteps) nxt = prefetch(step + 1);
    typename VT::T acc = VT::zero();
    if (wide) {
      walk<VEC, U, FAST, EPL, ALONE, S>(lists, cur.cs, cur.clen, cur.ds, cur.len, cur.first, same.base, same.lanes, same.q, same.slot,
                          same.nslots, s, a.ldx, cur.i, ntl, lds, acc);
      reduce_slots<VEC>(a.ls_log2, acc);
      if (split) {
        if (team == 0 && s.fvalid)
          VT::store(partial_slot(a, slice_seq, v_first + (int64_t)step * a.nclass, fl, VEC), acc, kPartialNt);
      } else if constexpr (UPD) {
        if (team == 0) finish_row_to_sink(a, s, sink, sink.cnt, fl, cur.i, cur.di, cur.xi, acc);
        sink.cnt += 1;
      } else {
        if (team == 0 && s.fvalid) finish_row<VEC>(a, s, cur.i, cur.di, cur.xi, acc);
      }
    } else {
      const Place p = place(shape(step));
      constexpr bool ONE = TEAMS == kOneGroup && (VEC == 4 || !coded(S));
      if (cur.have)
        // (one group: said to the compiler, which gets a step's entries with two accesses to LDS then, not four.  With that and no
        // divisions above R-MAT 100k, k = 5, F = 30 97.7 -> 96.2 us, 200k, k = 8, F = 1 145.2 -> 144.2; but 145.1 -> 149.3 with codes)
        walk<VEC, U, FAST, EPL, ALONE, S, TEAMS != kOneGroup>(lists, cur.cs, cur.clen, cur.ds, cur.len, cur.first, p.base, p.lanes, p.q,
                            ONE ? 0 : p.slot, ONE ? 1 : p.nslots, s, a.ldx, cur.i, ntl, lds, acc);
      if constexpr (TEAMS != kOneGroup)
        for (int m = p.lanes >> 1; m >= ls; m >>= 1) VT::add(acc, VT::shfl_xor(acc, m));
      if constexpr (UPD) {
        if (cur.have && (TEAMS == kOneGroup || p.slot == 0)) finish_row_to_sink(a, s, sink, sink.cnt + p.team, fl, cur.i, cur.di, cur.xi, acc);
        sink.cnt += rows_now;  // teams 0 .. rows_now - 1 had a row
      } else {
        if (cur.have && (TEAMS == kOneGroup || p.slot == 0) && s.fvalid) finish_row<VEC>(a, s, cur.i, cur.di, cur.xi, acc);
      }
    }
  }
  if constexpr (UPD) sink_flush(a, s, sink, lane);
}

#ifndef PIPAD_AGG_WAVES
#define PIPAD_AGG_WAVES 1  // lower bound on waves per SIMD the register allocation must allow
#endif

// EPL: entries per lane and chunk; teams of 8 lanes and more get on with 1.  (Teams of 1 and 2 lanes with
// one entry per lane, fetched and gathered one after the other: N = 500k, k = 4, F = 4 486 us, with 4
// entries 375; 8 entries take too many registers.)
template <int VEC, bool FAST, int EPL, bool PLAIN, bool ALONE = false, Scales S = kStreams, Teams TEAMS = kOneGroup>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(PIPAD_AGG_WAVES)))
void k_aggregate(const AggArgs a) {
  aggregate_body<VEC, FAST, EPL, false, PLAIN, ALONE, S, TEAMS>(a);
}

// The same walk with the update fused in, held to the four waves per SIMD that its 120 registers allow
// (left to the compiler: 853 us against 851 on N = 200k, k = 8, F = Fo = 64).
template <bool PLAIN, Scales S = kStreams, Teams TEAMS = kOneGroup>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_aggregate_update(const AggArgs a) {
  aggregate_body<4, true, 1, true, PLAIN, false, S, TEAMS>(a);
}

// Adds the partial sums of every hub row in a fixed order and finishes the row.  One wave per
// (hub row, slice), slice-major so that consecutive waves read consecutive partial sums; the lane
// teams stride over the row's class parts.
// UPD: the slice is the whole row; these rows are multiplied by W with plain FMAs, which give the bits that they would have inside
// the aggregation (sink_flush), so that H does not depend on whether a row is summed in parts, nor (k_update_resident,
// LIKE_INSIDE) on whether its sums are kept: a step of the matrix instruction is four FMAs in the order of the lane groups, the
// same bits in 314 million sums of ordinary and of denormal numbers, overflows, zeros and infinities, NaNs among the results.
// Bound: the chain row id - partial sums - row - weights, so the weights come 16 at a time: R-MAT 1M, k = 8, F = Fo = 64 75.7 -> 67.4 us,
// Chung-Lu 200k 10.6 -> 9.3 (with the instruction itself, 4 or 16 rows of a workgroup in a tile, which wait for one another, 82 to 88 and 12).
template <int VEC, bool UPD = false>
__global__ __launch_bounds__(kBlock) void k_split_finish(const AggArgs a) {
  using VT = V<VEC>;
  __shared__ __align__(16) float yrow[UPD ? kWavesPerBlock : 1][UPD ? kWave : 1];
  const int lane = threadIdx.x % kWave;
  const int wave = threadIdx.x / kWave;
  const int ls = 1 << a.ls_log2;
  const int fl = lane & (ls - 1);
  const int team = lane >> a.ls_log2;
  const int nteams = kWave >> a.ls_log2;
  const int64_t row_blocks = ((int64_t)a.n_hub + kWavesPerBlock - 1) / kWavesPerBlock;
  const int64_t b = blockIdx.x;
  const int slice_seq = (int)(b / row_blocks);
  const int t_seq = slice_seq / a.fchunks;
  const int64_t sr = (b - slice_seq * row_blocks) * kWavesPerBlock + wave;
  if (sr >= a.n_hub) return;
  const Slice s = slice_setup(a, selected_snapshot(a, t_seq), slice_seq - t_seq * a.fchunks, fl, VEC);
  const int32_t i = a.hub_rows[sr];
  const int64_t v0 = (int64_t)a.hub_item_off[sr] * a.nclass;  // the row's partial sums
  const int64_t v1 = (int64_t)a.hub_item_off[sr + 1] * a.nclass;
  typename VT::T acc = VT::zero();
  if (s.fvalid)
    for (int64_t v = v0 + team; v < v1; v += nteams)
      VT::add(acc, VT::load(partial_slot(a, slice_seq, v, fl, VEC)));
  reduce_slots<VEC>(a.ls_log2, acc);
  if constexpr (UPD) {
    if (team == 0) {
      const float di = s.dv[i];
      VT::fma(acc, di, VT::load(s.xb + (int64_t)i * a.ldx));
      typename VT::T y = VT::scale(di, acc);
      if (!s.fvalid) y = VT::zero();
      else if (s.yb) VT::store(s.yb + (int64_t)i * a.ldy, y, a.nt & 1);
      *reinterpret_cast<typename VT::T *>(&yrow[wave][fl * VEC]) = y;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    auto multiply = [&](uint32_t o, auto whole) __attribute__((always_inline)) {
      float h = 0.f;
      for (int step = 0; step < ls; step += 4) {  // step takes columns step, ls + step, 2 ls + step and 3 ls + step
        float y[4][4], w[4][4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 v = *reinterpret_cast<const float4 *>(&yrow[wave][g * ls + step]);
          y[g][0] = v.x; y[g][1] = v.y; y[g][2] = v.z; y[g][3] = v.w;
          w[g][0] = w[g][1] = w[g][2] = w[g][3] = 0.f;
          if (whole.value || g * ls + step < a.F)  // (F is a multiple of 4)
#pragma unroll
            for (int j = 0; j < 4; ++j) w[g][j] = (a.W + (int64_t)(g * ls + step + j) * a.ldw)[o];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) h = fmaf(y[g][j], w[g][j], h);
      }
      s.ht[(int64_t)i * a.ldh + o] = h + (a.bias ? a.bias[o] : 0.f);
    };
    if (lane < a.Fo) {  // (64 columns at most)
      if (a.F == 4 * ls) multiply(lane, std::true_type());
      else multiply(lane, std::false_type());
    }
  } else {
    if (team == 0 && s.fvalid)
      finish_row<VEC>(a, s, i, s.dv[i], VT::load(s.xb + (int64_t)i * a.ldx), acc);
  }
}

// Update alone, for shapes the fused kernel does not take: H_t = Y_t W + bias from the stored
// aggregation results.  A wave owns 16 rows of one snapshot; fp32 MFMA 16x16x4 with the usual
// operand layout (lane (m, g): A[m][k0 + g], B[k0 + g][16 nt + m]; D[4 g + r][m] in register r).
__global__ __launch_bounds__(kBlock) void k_update(const AggArgs a) {
  const int lane = threadIdx.x % kWave;
  const int64_t tiles = ((int64_t)a.n + 15) / 16;
  const int64_t id = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
  if (id >= tiles * a.k) return;
  const int t = __builtin_amdgcn_readfirstlane((int)(id / tiles));  // one snapshot per wave
  float *ht = a.H[t];
  const int64_t row0 = (id - t * tiles) * 16;
  const int m = lane & 15, g = lane >> 4;
  const int64_t row = row0 + m;
  const float *arow = a.Y[t] + min(row, (int64_t)a.n - 1) * a.ldy;
  for (int nt = 0; nt * 16 < a.Fo; ++nt) {
    const int col = 16 * nt + m;
    mfma_f4 d = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < a.F; k0 += 4) {
      const int kk = k0 + g;
      const float av = (kk < a.F && row < a.n) ? arow[kk] : 0.f;
      const float bv = (kk < a.F && col < a.Fo) ? a.W[(int64_t)kk * a.ldw + col] : 0.f;
      d = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, d, 0, 0, 0);
    }
    const float bias = (a.bias && col < a.Fo) ? a.bias[col] : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t orow = row0 + 4 * g + r;
      if (orow < a.n && col < a.Fo) ht[orow * a.ldh + col] = d[r] + bias;
    }
  }
}

// The same multiplication with the weights resident in LDS: a workgroup copies W's rows (all K of
// them, zero-padded to a multiple of 4) for the `cbw` output columns of its column block (blockIdx.y)
// once and its waves then take per_wave row tiles each.  The product is formed transposed, W^T Y_t^T:
// lane (m, g) supplies row m of the tile with four consecutive columns per 16-byte load (step j of a
// block of 16 columns multiplies k = 4 g + j; what is left of K past the last block goes one column per
// lane, k = 4 j + g), the next 64 columns on their way meanwhile, and gets back four consecutive columns
// of H for one 16-byte store per accumulator tile.
// Bound: the stream of Y and H.  (Rows of Y staged through an LDS tile 64 columns at a time, K padded to
// a multiple of 64, dword stores, W copied one element after the other and 8 tiles per wave whatever
// their number: N = 150k, k = 3, F = 128, Fo = 40 123 us, now 77 (3.9 TB/s); 39k, k = 8, F = 2, Fo = 128
// 106, now 45; 1.7k, k = 4, F = 64, Fo = 10 18, now 6.)  An instance for every number of accumulator
// tiles: with a test per tile instead the compiler hoists the operands of all of them (256 registers and
// more), and without the fence below it takes W into registers ahead of the loop.
constexpr int kUpdTiles = 8;       // row tiles per wave at most
constexpr int kUpdMaxCols = 128;   // output columns per column block (8 accumulator tiles)
constexpr int kUpdPad = 4;         // floats behind an LDS row of W: the lane groups' rows lie 16 banks apart

// LIKE_INSIDE: rows of 33 to 64 columns are summed up in the order of the multiplication inside the aggregation (sink_flush: step j
// takes columns j, 16 + j, 32 + j and 48 + j), for calls that without A go there: H has the same bits with A and without.  A lane
// group takes 16 consecutive columns then, and rows of W lie a word further apart, so that those of the groups are 16 banks apart.
// (Against the order of the other instances -2 to 1 % of aggregation and update, with 40 columns, which take as many steps as 64,
// 30.9 -> 32.2 us for N = 15k, k = 3, Fo = 64.)
template <int NT, bool LIKE_INSIDE = false>  // 16-column accumulator tiles a wave keeps
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_update_resident(const AggArgs a, int kpad, int per_wave) {
  constexpr int cbw = 16 * NT;
  constexpr int GROUP = LIKE_INSIDE ? 16 : 4, BLOCK = LIKE_INSIDE ? 4 : 16;  // columns from a lane group, a block, to the next
  using VT = V<4>;
  extern __shared__ __align__(16) float upd_lds[];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int m = lane & 15, g = lane >> 4;
  const int ws = cbw + (LIKE_INSIDE ? 1 : kUpdPad);
  const int col0 = blockIdx.y * cbw;
  stage_weights(a, upd_lds, kpad, cbw, col0, ws);
  __syncthreads();
  const int64_t tiles = ((int64_t)a.n + 15) / 16;
  const int64_t first = ((int64_t)blockIdx.x * kWavesPerBlock + wave) * per_wave;
  const int64_t last = min(first + per_wave, tiles * a.k);
  const int blocks = LIKE_INSIDE ? 4 : a.F / 16;    // whole blocks of 16 columns
  const int tail = LIKE_INSIDE ? 0 : (a.F - 16 * blocks + 3) / 4;  // steps behind them
  const int chunks = max((blocks + 3) / 4, 1);
  // four blocks of this lane's row (those past the last whole one repeat it; without a whole one they
  // are not there) and, with the last chunk, the tail
  auto request = [&](int64_t id, int chunk, float4 (&v)[4], float (&tv)[4]) __attribute__((always_inline)) {
    const int t = __builtin_amdgcn_readfirstlane((int)(id / tiles));
    const float *src = a.Y[t] + min((id - t * tiles) * 16 + m, (int64_t)a.n - 1) * a.ldy;
    if (blocks > 0)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int col = BLOCK * min(4 * chunk + b, blocks - 1) + GROUP * g;
        v[b] = VT::load(src + (LIKE_INSIDE ? min(col, a.F - 4) : col));
      }
    if (tail > 0 && chunk == chunks - 1)
#pragma unroll
      for (int j = 0; j < 4; ++j) tv[j] = src[min(16 * blocks + 4 * j + g, a.F - 1)];
  };
  float4 nxt[4] = {};
  float nxt_tail[4] = {};
  if (first < last) request(first, 0, nxt, nxt_tail);
  for (int64_t id = first; id < last; ++id) {
    const int t = __builtin_amdgcn_readfirstlane((int)(id / tiles));
    const int64_t row = (id - t * tiles) * 16 + m;
    asm volatile("" ::: "memory");
    mfma_f4 d[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) d[nt] = mfma_f4{0.f, 0.f, 0.f, 0.f};
    for (int chunk = 0; chunk < chunks; ++chunk) {
      float4 cur[4];
      float cur_tail[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        cur[b] = nxt[b];
        cur_tail[b] = nxt_tail[b];
      }
      if (chunk + 1 < chunks) request(id, chunk + 1, nxt, nxt_tail);
      else if (id + 1 < last) request(id + 1, 0, nxt, nxt_tail);
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        __builtin_amdgcn_sched_barrier(0);  // (all blocks' operands at once would take too many registers)
        if (4 * chunk + b >= blocks) break;
        const int col = BLOCK * (4 * chunk + b) + GROUP * g;
        if (LIKE_INSIDE && col >= a.F) cur[b] = VT::zero();
        const float y[4] = {cur[b].x, cur[b].y, cur[b].z, cur[b].w};
        const float *w = upd_lds + col * ws + m;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            d[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[j * ws + 16 * nt], y[j], d[nt], 0, 0, 0);
      }
      if (chunk == chunks - 1)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (j >= tail) break;
          const int kk = 16 * blocks + 4 * j + g;
          const float y = kk < a.F ? cur_tail[j] : 0.f;
          const float *w = upd_lds + kk * ws + m;
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            d[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[16 * nt], y, d[nt], 0, 0, 0);
        }
    }
    float *out = a.H[t] + row * a.ldh + col0 + 4 * g;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const float *b = upd_lds + kpad * ws + 16 * nt + 4 * g;
      const float4 h = make_float4(d[nt][0] + b[0], d[nt][1] + b[1], d[nt][2] + b[2], d[nt][3] + b[3]);
      const int left = a.Fo - (col0 + 16 * nt + 4 * g);  // columns from here on
      if (row >= a.n) continue;
      if (left >= 4) {
        VT::store(out + 16 * nt, h, false);
      } else {
        if (left > 0) out[16 * nt] = h.x;
        if (left > 1) out[16 * nt + 1] = h.y;
        if (left > 2) out[16 * nt + 2] = h.z;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Small feature widths (F < 32): the coalescent kernel.
//
// When the k feature matrices are handed over as ONE concatenated operand (X[t] = X[0] + t*F, row
// stride >= k*F: the paper's "coalescent features", Section 4.2) and F is small, one snapshot's row
// is only a few bytes, which is the "bandwidth unsaturation" case of Section 3.2.  Here a lane team
// covers the rows of SG consecutive snapshots side by side (SG*F <= 64 columns), so one decoded
// column index of the overlap part drives ONE contiguous gather for SG snapshots -- the paper's
// parallel aggregation as it stands, with 64-lane waves: LPS = ceil(F/VEC) lanes per snapshot, LS
// lanes (SG * LPS, rounded up to a power of two) per row, 64/LS rows (short rows) or entries (mid
// rows and class parts) side by side per wave.  Snapshot groups play the role of slices.
// The exclusive entries differ per snapshot, so the lanes of a snapshot walk a list of their own: the
// common entries, then that snapshot's exclusive ones, in the same loop as in k_aggregate (walk), with
// those lanes as its team.  Hub units go by column class, each on the XCD that holds the class.
// Bound: with many entries the loads of scales - 4 bytes per entry and snapshot out of k arrays, where a lane that
// fetches for itself (F <= 4 in short rows) loads a dword at a time and an instruction touches up to 64 lines.  So
// the rows are multiplied by their scales first (kTable; aggregate_launch says when): N = 1M R-MAT, k = 8, F = 2
// 572 -> 368 us, of which 26 for the products; hub units 185 -> 101, mid rows 203 -> 123, short rows 265 -> 153 (each
// alone), everything but the row gathers 339 -> 152.  Scales gathered from the node-major D^-1/2 next to the rows instead: 525 us, and
// slower with few snapshots (k = 4 113 -> 150).  What is left is bound by the gathers of half lines (64 bytes) and, in the
// exclusive parts, of 8 bytes of a line.  For small frames the chain index - row pointers - entries - rows, which is
// therefore requested two steps ahead.  Measured (wide operand; before: entries staged for all snapshots
// of a team one load after the other, hub units whole, VEC from F's divisors): N = 1M R-MAT, k = 8, F = 2
// 617 -> 585 us; 300k, k = 8, F = 6 467 -> 352; 300k, k = 16, F = 3 846 -> 510; 50k, k = 12, F = 9 468 ->
// 139; 5k, k = 16, F = 5 74 -> 19; 200k, k = 8, F = 16 173 -> 175.
struct CoalItem {
  int32_t i, cs, clen, ds, len;  // len: both lists together (0: this lane has nothing to do)
  int32_t front;                 // common entries in front of these, for walk_front
};

// The value of lane J of the quad.
template <int J>
__device__ __forceinline__ uint32_t of_quad(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, J * 0x55, 0xf, 0xf, true);
}

// Adds `front` common entries of a row, a multiple of the chunk of 4 * team_lanes: where the lanes of a team are one snapshot
// each, they all take the same ones, and a lane of a quad fetches one and turns it into an offset for all four, where it
// fetched four for itself (walk).  at: the place of this lane's first one in colc, of which `c` is the column.
// The same sums as walk's.
template <int VEC>
__device__ __forceinline__ void walk_front(const int32_t *colc, int32_t at, int32_t c, int32_t front, int32_t chunk, const float *table,
                                           uint32_t row_bytes, uint32_t lane_bytes, typename V<VEC>::T &acc) {
  using VT = V<VEC>;
  const char *const bytes = reinterpret_cast<const char *>(table);
  const float w[4] = {1.f, 1.f, 1.f, 1.f};
  auto row = [&](uint32_t off) __attribute__((always_inline)) { return VT::load(reinterpret_cast<const float *>(bytes + (off + lane_bytes))); };
  for (int32_t left = front; left > 0; left -= chunk) {
    const uint32_t off = (uint32_t)c * row_bytes;
    at += chunk;
    if (left > chunk) c = colc[at];
    const typename VT::T x[4] = {row(of_quad<0>(off)), row(of_quad<1>(off)), row(of_quad<2>(off)), row(of_quad<3>(off))};
    add_step<VEC, kTable>(w, x, acc);
  }
}

// Where snapshot group g's partial sums of class part `cls` of a hub unit (of the whole unit, where that
// is summed at once) start, as the place of column 0 of the wide row: the groups one after the other, in
// each the columns of its snapshots side by side without gaps.  All of them take k * F floats per part,
// which is no more than a call with the same F and one matrix per snapshot needs: what one call has
// sized the scratch for, the other can do with.
__device__ __forceinline__ float *unit_partial(const AggArgs &a, int g, int64_t unit, int cls) {
  const int64_t parts = a.whole_units ? 1 : a.nclass;
  const int64_t col0 = (int64_t)g * a.sg * a.F;  // the group's first column
  const int width = min(a.sg, a.k - g * a.sg) * a.F;
  return a.partial + col0 * (a.n_items * parts) + (unit * parts + cls) * width - col0;
}

// Self-loop term, row scale, store.  (With the products of kTable in 64 bits up to the store, which saves more than their own
// roundings cost: of seven R-MAT and Chung-Lu frames, k = 4 .. 16, F = 1 .. 12, rows of up to 64 entries have 0.74 to 0.92 of the
// error of kStreams against 64 bits, of up to 512 0.67 to 0.94, longer ones, which are summed up in parts, 0.75 to 0.97.)
template <int VEC, Scales S>
__device__ __forceinline__ void finish_coalescent(float *y, float di, typename V<VEC>::T xi, typename V<VEC>::T acc, bool nt) {
  using VT = V<VEC>;
  if constexpr (S == kStreams || S == kCodes) {
    VT::fma(acc, di, xi);
    VT::store(y, VT::scale(di, acc), nt);
  } else {
    VT::store(y, VT::finish(di, xi, acc), nt);
  }
}

template <int VEC, int EPL, bool PLAIN, bool ALONE, Scales S>
__global__ __launch_bounds__(kBlock) void k_aggregate_coalescent(const AggArgs a) {
  using VT = V<VEC>;
  constexpr int U = 4;  // row gathers in flight per lane
  __shared__ Staged staging[kWavesPerBlock][kWave * EPL];
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  Staged *lds = staging[wave];
  const int fl = lane & ((1 << a.ls_log2) - 1);
  const int team = lane >> a.ls_log2;
  const int nteams = kWave >> a.ls_log2;

  // Class parts first, one snapshot group after the other (the class's XCD is the workgroup index
  // mod 8); then the whole rows, the groups side by side: they share the entry lists.
  // (32-bit numbers, a scalar for the wave and no division by one group: with 64-bit ones the instances for four columns without
  // products took 100 registers, four waves per SIMD; now 94 to 96, five.  F = 16, concatenated: Chung-Lu 36k, k = 16 64.4 -> 57.8 us, 70k,
  // k = 8 56.1 -> 50.0, 51k, k = 4 23.7 -> 21.8, R-MAT 759k, k = 2 190 -> 167, 201k, k = 12 399 -> 373; F = 2 and 5 0 to 1 %; 12k, k = 6,
  // F = 15 19.1 -> 19.4.  Divisions by a multiplication, as in k_aggregate, are 1 to 3 % slower here.)
  const uint32_t b = blockIdx.x;
  const uint32_t wide_blocks = kClasses * a.blocks_wide;  // per sub class
  const uint32_t split_blocks = PLAIN ? a.n_items : a.whole_units ? a.blocks_wide : wide_blocks << a.sub_log2;
  const uint32_t unit_blocks = split_blocks * a.nslices;
  const bool unit = b < unit_blocks;
  const bool split = !PLAIN && unit;
  int g = 0;  // snapshot group
  uint32_t w;
  if (unit) {
    if (a.nslices > 1) g = b / split_blocks;
    w = b - g * split_blocks;
  } else {
    const uint32_t r0 = b - unit_blocks;
    w = r0;
    if (a.nslices > 1) {
      w = r0 / (uint32_t)a.nslices;
      g = r0 - w * a.nslices;
    }
  }

  // this lane's place in the group's row: VEC columns of snapshot t (F need not be a multiple of
  // VEC: a snapshot's last lane takes its last VEC columns)
  const int lps = (a.F + VEC - 1) / VEC;
  int u = fl / lps;
  int t = g * a.sg + u;
  const bool valid = u < a.sg && t < a.k;
  if (!valid) { u = 0; t = g * a.sg; }
  const int lane_col = t * a.F + (valid ? min((fl - u * lps) * VEC, a.F - VEC) : 0);  // within the wide row
  float *ylane = a.Y[0] + lane_col;
  const float *dv = a.dinv + (int64_t)t * a.n;
  const int32_t *rpd = a.rowptr_d[t];
  const uint32_t row_bytes = (uint32_t)a.ldx * 4u;
  const char *xbytes = reinterpret_cast<const char *>(a.X[0]);
  const uint32_t lane_bytes = (uint32_t)lane_col * 4u;

  // For the walk a team is the lanes of one snapshot, of one row or, wave-wide, of all lane groups:
  // they fetch that snapshot's entries together (the next smaller power of two of them, so that a
  // chunk is a multiple of U entries; the others do the same again).
  const int fetchers = lps >= 8 ? 8 : lps >= 4 ? 4 : lps >= 2 ? 2 : 1;
  Slice s;
  s.xt = S == kTable ? a.table : a.X[0];  // what is gathered
  s.fcol = lane_col;
  s.fvalid = true;
  s.xb = s.xt + lane_col;
  const int64_t ldg = S == kTable ? a.ldt : a.ldx;

  if (PLAIN && unit) {
    // a hub unit by the whole workgroup, as in k_aggregate
    __shared__ typename VT::T sums[kWavesPerBlock][kWave];
    Piece p = unit_piece(a, w, rpd, wave);
    if (!valid) p.len = 0;
    Lists l;
    l.colc = a.col_c;
    l.wc = a.wc[t];
    l.cold = a.col_d[t];
    l.wd = a.wd[t];
    const int team_lanes = nteams * fetchers, q = team * fetchers + ((fl - u * lps) & (fetchers - 1));
    Raw head[EPL];
#pragma unroll
    for (int v = 0; v < EPL; ++v)
      head[v] = fetch<S>(l, p.cs, p.clen, p.ds, p.len, v * team_lanes + q, p.i, false);
    typename VT::T acc = VT::zero();
    walk<VEC, U, true, EPL, ALONE, S>(l, p.cs, p.clen, p.ds, p.len, head, u * nteams * fetchers, team_lanes, q, team, nteams, s,
                                      ldg, p.i, false, lds, acc);
    reduce_slots<VEC>(a.ls_log2, acc);
    if (team == 0) sums[wave][fl] = acc;
    __syncthreads();
    if (wave > 0 || team > 0 || !valid) return;
#pragma unroll
    for (int x = 1; x < kWavesPerBlock; ++x) VT::add(acc, sums[x][fl]);
    if (a.direct) {
      finish_coalescent<VEC, S>(ylane + (int64_t)p.i * a.ldy, dv[p.i],
                                VT::load(reinterpret_cast<const float *>(xbytes + ((uint32_t)p.i * row_bytes + lane_bytes))), acc, a.nt & 1);
    } else {
      VT::store(unit_partial(a, g, w, 0) + lane_col, acc, false);
    }
    return;
  }

  const int32_t *const p_items = a.item_row, *const p_mid = a.rows_long, *const p_short = a.rows_short;
  const int32_t n_items = a.n_items, n_mid = a.n_long, n_short = a.n_short;
  const int b_wide = a.batch_wide, b_mid = a.batch_mid, b_short = a.batch_short;
  const bool wide = split || w < (uint32_t)a.blocks_mid;  // the whole wave on one list
  int cls = 0;
  if (split && !a.whole_units) {
    const int sub = a.sub_log2 == 0 ? 0 : (int)(w / wide_blocks);
    w -= sub * wide_blocks;
    cls = ((int)(w & (kClasses - 1)) << a.sub_log2) + sub;
    w >>= 3;
  } else if (!wide) {
    w -= a.blocks_mid;
  }
  const int32_t *list = split ? p_items : wide ? p_mid : p_short;
  const int32_t list_len = split ? n_items : wide ? n_mid : n_short;
  const int batch = split ? b_wide : wide ? b_mid : b_short;
  const int64_t first64 = ((int64_t)w * kWavesPerBlock + wave) * batch;
  if (first64 >= list_len) return;
  const int32_t first = (int32_t)first64;
  const int rows_here = min(batch, list_len - first);

  // entry lists: the class-grouped copies for hub units, the frame's CSRs for whole rows
  Lists lists;
  {
    const void *w_plain = a.wc[t], *w_grouped = a.swc[t];
    const int32_t *d_plain = a.col_d[t];
    const void *wd_plain = a.wd[t];
    lists.colc = split ? a.scol_c : a.col_c;
    lists.cold = split ? a.scol_d : d_plain;
    lists.wc = split ? w_grouped : w_plain;
    lists.wd = split ? a.swd : wd_plain;
  }
  // metadata of the batch: lane l holds element l (the exclusive lists are per snapshot and read one
  // step ahead)
  int32_t r = 0, mc0 = 0, mc1 = 0;
  if (lane < rows_here) {
    r = list[first + lane];
    const int32_t *pc = split ? a.sptr + ((int64_t)cls * n_items + first + lane) : a.rowptr_c + r;
    mc0 = pc[0];
    mc1 = pc[split ? n_items : 1];
  }
  int order = lane;
  if (!wide && a.longest_first && rows_here > nteams)
    order = longest_first(lane < rows_here ? (mc1 - mc0 + U - 1) / U : 0, rows_here, lane);  // (by the common entries)
  const int per_step = wide ? 1 : nteams;
  const int team_lanes = wide ? nteams * fetchers : fetchers;
  const int q = (wide ? team * fetchers : 0) + ((fl - u * lps) & (fetchers - 1));
  const int team_base = (wide ? u * nteams : team * a.sg + u) * fetchers;
  const int slot = wide ? team : 0;
  const int nslots = wide ? nteams : 1;
  const bool share = ALONE && S == kTable && a.share;
  const int32_t chunk = 4 * team_lanes, place = (fl & 3) * team_lanes + q;
  auto meta = [&](int step, int part) __attribute__((always_inline)) {
    CoalItem it;
    const int li = step * per_step + (wide ? 0 : team);
    const bool have = li < rows_here;
    const int src = __shfl(order, have ? li : 0, kWave);
    it.i = __shfl(r, src, kWave);
    it.cs = __shfl(mc0, src, kWave);
    it.clen = __shfl(mc1, src, kWave) - it.cs;
    it.front = share && have ? it.clen & -chunk : 0;  // (the lanes without columns take part)
    it.cs += it.front;
    it.clen -= it.front;
    int64_t stride = 1;
    const int32_t *pd = rpd + it.i;
    if (split) {
      stride = n_items;
      pd = a.sptr + ((int64_t)(1 + t) * (a.nclass + 1) + cls + part) * n_items + first + src;
    }
    it.ds = pd[0];
    it.len = it.clen + pd[stride] - it.ds;
    if (!have || !valid) it.len = 0;
    return it;
  };
  struct Fetched {
    Raw e[EPL];
    int32_t c;  // of walk_front
  };
  auto fetch = [&](const CoalItem &it) __attribute__((always_inline)) {
    Fetched f;
    f.c = 0;
    if constexpr (ALONE && S == kTable)
      if (it.front > 0) f.c = lists.colc[it.cs - it.front + place];
#pragma unroll
    for (int v = 0; v < EPL; ++v)
      f.e[v] = pipad::fetch<S>(lists, it.cs, it.clen, it.ds, it.len, v * team_lanes + q, it.i, false);
    return f;
  };
  auto walk_item = [&](const CoalItem &it, const Fetched &f) __attribute__((always_inline)) {
    typename VT::T acc = VT::zero();
    if constexpr (ALONE && S == kTable)
      walk_front<VEC>(lists.colc, it.cs - it.front + place, f.c, it.front, chunk, s.xt, (uint32_t)ldg * 4u, lane_bytes, acc);
    walk<VEC, U, true, EPL, ALONE, S>(lists, it.cs, it.clen, it.ds, it.len, f.e, team_base, team_lanes, q, slot, nslots, s,
                                      ldg, it.i, false, lds, acc);
    return acc;
  };

  const int nsteps = (rows_here + per_step - 1) / per_step;
  CoalItem m = meta(0, 0);
  Fetched f = fetch(m);
  CoalItem m_next = meta(1, 0);
  for (int step = 0; step < nsteps; ++step) {
    const CoalItem cur = m;
    const Fetched cur_f = f;
    const bool have = step * per_step + (wide ? 0 : team) < rows_here;
    typename VT::T xi = VT::zero();
    float di = 0.f;
    if (!split) {
      xi = VT::load(reinterpret_cast<const float *>(xbytes + ((uint32_t)cur.i * row_bytes + lane_bytes)));
      di = dv[cur.i];
    }
    if (step + 1 < nsteps) {
      m = m_next;
      f = fetch(m);
      m_next = meta(step + 2, 0);
    }
    typename VT::T acc = walk_item(cur, cur_f);
    if (wide) reduce_slots<VEC>(a.ls_log2, acc);
    if (split) {
      if (a.whole_units) {
        // no room for a partial sum per class part: the parts one after the other, added in the
        // order in which k_hub_finish_coalescent adds them
        for (int part = 1; part < a.nclass; ++part) {
          CoalItem it = meta(step, part);
          const int64_t c0 = a.sptr[(int64_t)part * n_items + first + step];
          const int64_t c1 = a.sptr[(int64_t)(part + 1) * n_items + first + step];
          const int32_t dlen = it.len - it.clen;
          it.front = 0;
          it.cs = (int32_t)c0;
          it.clen = (int32_t)(c1 - c0);
          it.len = valid ? it.clen + dlen : 0;
          typename VT::T more = walk_item(it, fetch(it));
          reduce_slots<VEC>(a.ls_log2, more);
          VT::add(acc, more);
        }
      }
      if (team == 0 && valid) VT::store(unit_partial(a, g, first + step, cls) + lane_col, acc, false);
    } else if (have && valid && (!wide || team == 0)) {
      finish_coalescent<VEC, S>(ylane + (int64_t)cur.i * a.ldy, di, xi, acc, a.nt & 1);
    }
  }
}

// Hub rows of the coalescent kernel: adds a unit's class parts in class order, then the units in a
// fixed order.
template <int VEC>
__global__ __launch_bounds__(kBlock) void k_hub_finish_coalescent(const AggArgs a) {
  using VT = V<VEC>;
  const int lane = threadIdx.x % kWave;
  const int wave = threadIdx.x / kWave;
  const int fl = lane & ((1 << a.ls_log2) - 1);
  const int team = lane >> a.ls_log2;
  const int nteams = kWave >> a.ls_log2;
  const int64_t b = blockIdx.x;
  const int g = (int)(b % a.nslices);
  const int64_t hr = (b / a.nslices) * kWavesPerBlock + wave;
  if (hr >= a.n_hub) return;
  const int lps = (a.F + VEC - 1) / VEC;
  const int u = fl / lps;
  const int t = g * a.sg + u;
  const bool valid = u < a.sg && t < a.k;
  const int32_t i = a.hub_rows[hr];
  const int32_t it0 = a.hub_item_off[hr], it1 = a.hub_item_off[hr + 1];
  const int parts = a.whole_units ? 1 : a.nclass;
  const int stride = min(a.sg, a.k - g * a.sg) * a.F;  // (see unit_partial)
  const int lane_col = t * a.F + min((fl - u * lps) * VEC, a.F - VEC);
  typename VT::T acc = VT::zero();
  if (valid)
    for (int32_t it = it0 + team; it < it1; it += nteams) {
      const float *p = unit_partial(a, g, it, 0) + lane_col;
      typename VT::T sum = VT::load(p);
      if (parts > 1) {
        for (int q = 0; q < parts; q += 8) {  // (a unit has 8, 16 or 32 class parts)
          typename VT::T x[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) x[j] = VT::load(p + (q + j) * stride);
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (q + j > 0) VT::add(sum, x[j]);
        }
      }
      VT::add(acc, sum);
    }
  reduce_slots<VEC>(a.ls_log2, acc);
  if (team == 0 && valid) {
    const float di = a.dinv[(int64_t)t * a.n + i];
    const typename VT::T xi = VT::load(a.X[0] + lane_col + (int64_t)i * a.ldx);
    float *const y = a.Y[0] + lane_col + (int64_t)i * a.ldy;
    if (a.products) finish_coalescent<VEC, kProducts>(y, di, xi, acc, a.nt & 1);
    else finish_coalescent<VEC, kStreams>(y, di, xi, acc, a.nt & 1);
  }
}

// Every row of the concatenated operand times its column scales, dinv_t[i] X_t[i], rounded: what kTable gathers.  A thread takes
// four columns of a node, 16 bytes at a time where the rows allow it (VECTOR), and gets its scales (W), or their codes, from one line
// (k streams instead: R-MAT 200k, k = 8, F = 9 223 -> 232 us in all, 60k, k = 16 241 -> 249).  Bound: the stream of X and of the table.
template <class W, bool VECTOR>
__global__ __launch_bounds__(kBlock) void k_scale_rows(const AggArgs a, float *table) {
  const uint32_t cols = (uint32_t)(a.k * a.F), quads = (cols + 3) / 4;
  const int64_t x = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (x >= (int64_t)a.n * quads) return;
  const int32_t i = (int32_t)(x / quads);
  const uint32_t c = 4 * (uint32_t)(x - (int64_t)i * quads);
  const W *scales = static_cast<const W *>(a.nk) + (int64_t)i * node_stride(a.k);
  const float *row = a.X[0] + (int64_t)i * a.ldx;
  float v[4], w[4];
  if (VECTOR) {
    const float4 q = V<4>::load(row + c);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t at = min(c + j, cols - 1);
    if (!VECTOR) v[j] = row[at];
    if constexpr (sizeof(W) == sizeof(float)) w[j] = scales[at / (uint32_t)a.F];
    else w[j] = scale_of_length(scales[at / (uint32_t)a.F]);
  }
  // (the table's rows are padded to 16 bytes)
  *reinterpret_cast<float4 *>(table + (int64_t)i * a.ldt + c) =
      make_float4(rounded(w[0], v[0]), rounded(w[1], v[1]), rounded(w[2], v[2]), rounded(w[3], v[3]));
}

inline int ceil_log2(int64_t x) {
  int l = 0;
  while (((int64_t)1 << l) < x) ++l;
  return l;
}

// LDS of the fused-update kernel: W [K][Fo + 1] and the bias, one tile and 16 row ids per wave.
inline size_t update_lds_bytes(const AggArgs &a) {
  const size_t K = (size_t)4 << a.ls_log2;
  const size_t w_floats = ((K + 1) * (a.Fo + 1) + 3) & ~(size_t)3;  // W and, as row K, the bias
  return (w_floats + (size_t)kWavesPerBlock * kTileRows * kTileStride) * sizeof(float) +
         (size_t)kWavesPerBlock * kTileRows * sizeof(int32_t);
}

// The instance for teams of 1 << ls_log2 lanes (rows of one column at a time have at most four columns).
template <int VEC, bool PLAIN, Scales S = kStreams>
void (*aggregate_kernel(bool fast, int ls_log2))(AggArgs) {
  if (!fast) return k_aggregate<VEC, false, 1, PLAIN, false, S>;
  if constexpr (VEC > 1)
    if (ls_log2 >= 3) return k_aggregate<VEC, true, 1, PLAIN, false, S>;
  return ls_log2 >= 2 ? k_aggregate<VEC, true, 2, PLAIN, false, S>
         : ls_log2 == 1 ? k_aggregate<VEC, true, 4, PLAIN, false, S> : k_aggregate<VEC, true, 4, PLAIN, true, S>;
}

// The same with several lane groups per short row, for slices of up to eight lanes.
template <int VEC>
void (*teams_kernel(int ls_log2))(AggArgs) {
  if constexpr (VEC > 1)
    if (ls_log2 >= 3) return k_aggregate<VEC, true, 1, true, false, kStreams, kSeveral>;
  return ls_log2 == 2 ? k_aggregate<VEC, true, 2, true, false, kStreams, kSeveral> : k_aggregate<VEC, true, 4, true, false, kStreams, kSeveral>;
}
// The same with lane groups by the length of the row, for slices of two and four lanes.
template <int VEC, Scales S>
void (*uneven_kernel(int ls_log2))(AggArgs) {
  return ls_log2 == 2 ? k_aggregate<VEC, true, 2, false, false, S, kByLength> : k_aggregate<VEC, true, 4, false, false, S, kByLength>;
}

// Whether lane groups go by the length of a short row.  A wave of narrow slices takes 16 or 32 rows side by side and as long as the
// longest of them; in skewed frames, whose short rows hold the smaller part of the entries, most of the lanes wait for a few.
// There the rows of a batch with more than 32 entries come first, by eight lane groups each, then those with more than 8 by four, then
// the others: each is one chunk.  More sums and up to three part-filled steps, which take a batch of rows that differ and rows enough: with
// two lanes per slice (5 to 8 columns) of 17 R-MAT frames of 1 to 6 M rows in all snapshots 14 1 to 8 % faster, the others the same but one, 1.5 %
// slower; with four lanes 10 of 1 to 1.6 M rows 5 % slower to 4 % faster (300k, k = 4, 16 entries per row, F = 4 5 %), 7 of 1.8 to 6 M up to 8 %
// faster, at worst 0.8 % slower.  500k, k = 12, F = 5 721 -> 694 us, 120k, k = 16, F = 2 8 %, 700k, k = 8, F = 4 4 %; frames of fewer rows up to 8 %
// slower, Chung-Lu frames, whose short rows are alike, 7 % (369k, k = 16, F = 3 709 -> 760).  Not from 16 columns on, where the update would
// have to add up in the same order (R-MAT 700k, k = 8, F = 16 657 -> 614).  Like short_row_team it looks at the whole frame.
bool uneven_rows(const pipad_frame *f, int ls_log2, int32_t F, int64_t entries) {
  return !f->plain_units && F < 16 && (ls_log2 == 1 || ls_log2 == 2) && 2 * f->short_entries < entries &&
         (int64_t)f->n_short * f->k > (ls_log2 == 1 ? 1000000 : 1750000);
}

// log2 of the lanes that walk a short row.  A small frame of few columns has few waves: 64 / LS rows each where a slice takes LS
// lanes (so short rows by one lane group), and a wave takes as long as the longest of them, a chain of up to 16 gathers that the chip
// waits for.  So there several lane groups walk a row, four entries each at a time, and their sums are added up in a fixed order:
// more waves, and shorter chains.  GPU time per call (calls recorded one behind the other), one group against the rule: Chung-Lu 1083
// nodes, k = 8, F = 16 7.1 -> 4.8 us, 2985, k = 5, F = 5 8.4 -> 5.1, 9127, k = 5, F = 7 9.0 -> 6.6, R-MAT 3683, k = 8, F = 16 7.2 -> 6.4;
// the update, 1623, k = 5, F = 16, Fo = 32 9.3 -> 7.0.  Once the waves fill the chip the sums are only more work.  Two groups pay up
// to 4096 waves, as many as run together at four per SIMD, and with more than four snapshots up to 8192 (9216 nodes, k = 6, F = 4
// 8.3 -> 6.9 us; with fewer 14,119, k = 3, F = 16 7.6 -> 8.0; past it 15,639, k = 8, F = 16 11.3 -> 13.8); more groups up to 3072 (1656, k = 4,
// F = 16: two 4.8 us, four 4.2, eight 4.7).  From 16 columns on, where the update may do the same sums in its own kernel, whose
// waves take 16 rows, two groups stop at 3072 as well (3223, k = 8, F = Fo = 16 11.3 -> 11.8, 4302, k = 6, F = 32, Fo = 64 12.8 -> 18.2).
// It looks at the whole frame, so that a row's sum is the same whichever snapshots a call takes and with the update or without;
// slices of 16 lanes and more, whose waves hold four rows at most, gain nothing (7121, k = 3, F = 58 11.5 -> 12.2).
int short_row_team(const pipad_frame *f, int ls_log2, int32_t F, int fchunks) {
  int log2 = ls_log2;
  const int64_t rows = (int64_t)f->n_short * f->k * fchunks;
  if (f->plain_units && ls_log2 > 0 && ls_log2 <= 3)
    while (log2 < ls_log2 + 3 && (rows << (log2 + 1)) / kWave <= (log2 > ls_log2 || F >= 16 ? 3072 : f->k > 4 ? 8192 : 4096)) ++log2;
  return log2;
}

template <int VEC>
int launch(const AggArgs &a, bool fast, hipStream_t st, bool fused_update = false) {
  const int64_t phases = (int64_t)a.nsel * a.fchunks;
  const int64_t blocks = a.blocks_per_phase * phases;
  if (blocks >= ((int64_t)1 << 31)) return PIPAD_ERR_TOO_LARGE;
  const int64_t fin = a.direct ? 0 : ((int64_t)a.n_hub + kWavesPerBlock - 1) / kWavesPerBlock * phases;
  if (fin >= ((int64_t)1 << 31)) return PIPAD_ERR_TOO_LARGE;
  const dim3 grid((unsigned)blocks), block(kBlock);
  if constexpr (VEC == 4) {
    if (fused_update) {
      if (!fast || a.ls_log2 < 2) return PIPAD_ERR_INVALID_ARG;  // the caller checked the shape
      auto kern = a.team_log2 > a.ls_log2 ? k_aggregate_update<true, kStreams, kSeveral>
                  : a.plain ? k_aggregate_update<true> : a.coded ? k_aggregate_update<false, kCodes> : k_aggregate_update<false>;
      if (blocks > 0) hipLaunchKernelGGL(kern, grid, block, update_lds_bytes(a), st, a);
      if (fin > 0)
        hipLaunchKernelGGL((k_split_finish<4, true>), dim3((unsigned)fin), dim3(kBlock), 0, st, a);
      PIPAD_HIP(hipGetLastError());
      return PIPAD_OK;
    }
  }
  auto kern = a.team_log2 > a.ls_log2 ? teams_kernel<VEC>(a.ls_log2)
              : a.uneven && a.coded ? uneven_kernel<VEC, kCodes>(a.ls_log2)
              : a.uneven ? uneven_kernel<VEC, kStreams>(a.ls_log2)
              : a.plain ? aggregate_kernel<VEC, true>(fast, a.ls_log2)
              : a.coded ? aggregate_kernel<VEC, false, kCodes>(fast, a.ls_log2) : aggregate_kernel<VEC, false>(fast, a.ls_log2);
  if (blocks > 0) hipLaunchKernelGGL(kern, grid, block, 0, st, a);
  if (fin > 0) hipLaunchKernelGGL((k_split_finish<VEC>), dim3((unsigned)fin), dim3(kBlock), 0, st, a);
  PIPAD_HIP(hipGetLastError());
  return PIPAD_OK;
}

// The update behind the aggregation, from the stored results of all snapshots (like_inside: of 36 to 64 columns in whole 16-byte
// pieces, up to 64 columns of H in whole tiles).
int launch_update(const AggArgs &a, bool like_inside, hipStream_t st) {
  const int64_t tiles = ((int64_t)a.n + 15) / 16 * a.k;
  // Weights resident in LDS, in as few blocks of columns of the same width as fit (every block reads all of Y), else
  // straight from memory.  64 KB of LDS, for two workgroups per CU, where Y is past the memory-side cache (256 MB): with
  // at most 40 KB, for four, N = 200k, k = 4, F = 128, Fo = 80 277 -> 200 us, F = 80, Fo = 128 314 -> 217; N = 150k, k = 3, F = 200,
  // Fo = 128 337 -> 272.  Where that cache holds Y, blocks of more than 32 columns get 53 KB, for three workgroups: N = 60k, k = 2, F = 128,
  // Fo = 112 with 64 KB 79 us, now 55, F = 160, Fo = 96 87 and 61, F = 200, Fo = 64 72 and 49.  And 40 KB where there are fewer than
  // 1024 workgroups for a block of columns, or 512 of longer rows: N = 3000, k = 1, F = 128, Fo = 112 15 and 11, N = 12k, k = 2 24 and 19, F = 200,
  // Fo = 200 56 and 39, F = 384, Fo = 64 39 and 34; N = 30k, k = 2, F = 112, Fo = 96 38 and 31, but F = 384, Fo = 128 98 and 122.
  const int kpad = like_inside ? 64 : (a.F + 3) / 4 * 4;
  const size_t two = 64u << 10, three = 53u << 10, four = 40u << 10;  // workgroups per CU
  const bool far = (int64_t)a.n * a.k * a.F * 4 > (256 << 20), few = !far && tiles < (a.F < 256 ? 4096 : 2048);
  int64_t col_blocks = 0;
  int cbw = 0;
  size_t lds = 0;
  do {
    ++col_blocks;
    cbw = (int)((a.Fo + 16 * col_blocks - 1) / (16 * col_blocks)) * 16;
    lds = (size_t)(kpad + 1) * (cbw + kUpdPad) * 4;
  } while (cbw > 16 && (cbw > kUpdMaxCols || lds > (few ? four : far || cbw <= 32 ? two : three)));
  if (lds <= two) {
    // as many tiles per wave as leave 16 waves for every CU
    const int per_wave = (int)std::clamp<int64_t>(tiles * col_blocks / 4096, 1, kUpdTiles);
    const int64_t per_block = (int64_t)kWavesPerBlock * per_wave;
    const dim3 grid((unsigned)((tiles + per_block - 1) / per_block), (unsigned)col_blocks);
    void (*const kern[])(AggArgs, int, int) = {k_update_resident<1>, k_update_resident<2>, k_update_resident<3>,
                                               k_update_resident<4>, k_update_resident<5>, k_update_resident<6>,
                                               k_update_resident<7>, k_update_resident<8>};
    void (*const like[])(AggArgs, int, int) = {k_update_resident<1, true>, k_update_resident<2, true>, k_update_resident<3, true>,
                                               k_update_resident<4, true>};
    hipLaunchKernelGGL((like_inside ? like : kern)[cbw / 16 - 1], grid, dim3(kBlock), lds, st, a, kpad, per_wave);
  } else {
    hipLaunchKernelGGL(k_update, dim3((unsigned)((tiles + kWavesPerBlock - 1) / kWavesPerBlock)),
                       dim3(kBlock), 0, st, a);
  }
  PIPAD_HIP(hipGetLastError());
  return PIPAD_OK;
}

// Entries per fetching lane, so that a chunk holds U = 4 and more for every lane group: 4 for one or
// two lanes per snapshot (F <= 4), 2 for two and more; F == VEC is one lane per snapshot.
template <int VEC, Scales S>
void (*coalescent_kernel(const AggArgs &a))(AggArgs) {
  constexpr bool PLAIN = !coded(S);  // (a frame of plain units has no codes)
  if constexpr (VEC > 1) {  // (VEC is F up to two columns, two for three, and four)
    constexpr int EPL = VEC == 4 ? 2 : 4;
    if (a.F > VEC) {
      return a.plain ? k_aggregate_coalescent<VEC, EPL, PLAIN, false, S> : k_aggregate_coalescent<VEC, EPL, false, false, S>;
    }
  }
  return a.plain ? k_aggregate_coalescent<VEC, 4, PLAIN, true, S> : k_aggregate_coalescent<VEC, 4, false, true, S>;
}

template <int VEC>
int launch_coalescent(const AggArgs &a, hipStream_t st) {
  const int64_t wide = a.plain ? a.n_items : a.whole_units ? a.blocks_wide : (int64_t)a.blocks_wide * a.nclass;
  const int64_t blocks = (wide + a.blocks_mid + a.blocks_short) * a.nslices;
  if (blocks >= ((int64_t)1 << 31)) return PIPAD_ERR_TOO_LARGE;
  void (*kern)(AggArgs) = nullptr;
  if (a.table) {
    const int64_t threads = (int64_t)a.n * ((a.k * a.F + 3) / 4);
    const bool vector = a.k * a.F % 4 == 0;
    auto scale = a.coded ? (vector ? k_scale_rows<uint16_t, true> : k_scale_rows<uint16_t, false>)
                         : (vector ? k_scale_rows<float, true> : k_scale_rows<float, false>);
    hipLaunchKernelGGL(scale, grid1(threads, kBlock), dim3(kBlock), 0, st, a, const_cast<float *>(a.table));
    kern = coalescent_kernel<VEC, kTable>(a);
  } else {
    kern = a.coded ? (a.products ? coalescent_kernel<VEC, kCodeProducts> : coalescent_kernel<VEC, kCodes>)(a)
                   : (a.products ? coalescent_kernel<VEC, kProducts> : coalescent_kernel<VEC, kStreams>)(a);
  }
  if (blocks > 0) hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kBlock), 0, st, a);
  if (a.n_hub > 0 && !a.direct) {
    const int64_t hb = ((int64_t)a.n_hub + kWavesPerBlock - 1) / kWavesPerBlock * a.nslices;
    hipLaunchKernelGGL((k_hub_finish_coalescent<VEC>), dim3((unsigned)hb), dim3(kBlock), 0, st, a);
  }
  PIPAD_HIP(hipGetLastError());
  return PIPAD_OK;
}

}  // namespace

// ---- the fixed scratch array of pipad_frame_aggregate_static -----------------------------------
// One array per GPU (every device that loads the library's code holds its own copy until the
// process ends).  The array's name is only a handle in host code: its device address is looked up
// once per device, with that device current, and only that address is ever handed to a kernel.
constexpr size_t kStaticScratchBytes = PIPAD_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void *g_scratch_ptr[kMaxDevices] = {};

int static_scratch(float **ptr, size_t *floats) {
  int dev = -1;
  PIPAD_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return PIPAD_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    PIPAD_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return PIPAD_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *ptr = static_cast<float *>(g_scratch_ptr[dev]);
  *floats = kStaticScratchBytes / sizeof(float);
  return PIPAD_OK;
}

constexpr int64_t kTableFloats = (int64_t)1 << 28;  // of kTable's table: 1 GiB at most
// It starts so far into its memory: allocations start at multiples of 2 MB, and with a row of the products at the same place in
// them as the operand's R-MAT 1M, k = 8, F = 4 takes 435 us, not 417, F = 2 347 and 341 (3 MB in 1 more), 900k, k = 6, F = 2 289 and
// 287; Chung-Lu 200k to 1M, k = 4 and 8, and R-MAT 262k and 300k with F = 2 and 4 the same within 0.5 %.
constexpr size_t kTableSkip = 16384 + 448;

int aggregate_launch(const pipad_frame *f, int32_t F, const float *const *X, int64_t ldx,
                     float *const *Y, int64_t ldy, hipStream_t st, ScratchRef scratch,
                     const UpdateSpec *upd, const int32_t *subset, int32_t nsubset) {
  if (f->n == 0 || (subset && nsubset == 0)) return PIPAD_OK;
  const Options &opt = f->opt;  // as they stood when the frame was built
  AggArgs a;
  std::memset(&a, 0, sizeof(a));
  a.n = f->n;
  a.k = f->k;
  a.F = F;
  a.ldx = ldx;
  a.ldy = ldy;
  a.rowptr_c = f->rowptr_c;
  a.col_c = f->col_c;
  a.dinv = f->dinv;
  a.coded = f->coded;
  a.nk = f->dinv_nk;
  a.rows_short = f->rows_short;
  a.rows_long = f->rows_long;
  a.item_row = f->item_row;
  a.hub_rows = f->hub_rows;
  a.hub_item_off = f->hub_item_off;
  a.sptr = f->sptr;
  a.scol_c = f->scol_c;
  a.scol_d = f->scol_d;
  a.swd = f->swd;
  a.item_v0 = f->item_v0;
  a.item_v1 = f->item_v1;
  a.plain = f->plain_units && f->n_items > 0;  // (without hub rows both kernels do the same; the other has fewer registers)
  a.direct = a.plain && f->n_items == f->n_hub;
  a.sub_log2 = f->plain_units ? 0 : f->sub_log2;
  a.nclass = f->plain_units ? 1 : f->nclass;
  a.nvp = a.direct ? 0 : (int64_t)f->n_items * a.nclass;
  a.n_short = f->n_short;
  a.n_long = f->n_long;
  a.n_items = f->n_items;
  a.n_hub = f->n_hub;
  a.nt = (int32_t)opt.agg_nt;
  // Workgroup order.  One slice after the other keeps one snapshot's matrix in the caches at a
  // time; side by side shares the index streams between the slices, which wins while a slice's matrix
  // (N rows of the slice's width) is smaller than the eight L2s together; from PIPAD_ORDER_BYTES on the
  // slices go one after the other.  Measured, k = 8, the other order against the one taken: N = 100k,
  // F = 64 328 us against 317, N = 200k, F = 32 364 against 348, F = 16 252 against 256; and beyond the
  // line N = 200k, F = 64 724 against 714, R-MAT 1M 3910 against 3865, low-overlap 5735 against 5049.
  // (Which of the two ways of side by side: below.)
  a.order = opt.agg_order >= 2 ? -1 : (int32_t)opt.agg_order;
  a.nsel = subset ? nsubset : f->k;
  for (int q = 0; q < a.nsel; ++q)
    a.sel[q >> 3] |= (uint64_t)(subset ? subset[q] : q) << ((q & 7) * 8);
  bool aligned = F % 4 == 0 && ldx % 4 == 0 && ldy % 4 == 0;
  for (int t = 0; t < f->k; ++t) {
    a.rowptr_d[t] = f->rowptr_d[t];
    a.col_d[t] = f->col_d[t];
    a.wc[t] = f->wc[t];
    a.wd[t] = f->wd[t];
    a.swc[t] = f->swc[t];
    a.X[t] = X[t];  // (null for a snapshot a subset call leaves out: never touched)
    a.Y[t] = Y ? Y[t] : nullptr;
    if ((reinterpret_cast<uintptr_t>(X[t]) | reinterpret_cast<uintptr_t>(a.Y[t])) & 15u) aligned = false;
  }
  // (four columns: four lanes of one each; a lane alone walked a row of 64 entries in 16 rounds, and 64 such rows
  // waited for the longest.  N = 20k, k = 4 20.4 -> 10.9 us, 200k 126 -> 98, R-MAT 200k, k = 8 190 -> 167)
  const bool vec4 = F > 4;
  // the fast path needs 32-bit byte offsets into a snapshot's matrix
  const bool fast = (int64_t)f->n * ldx * 4 < ((int64_t)1 << 32) && !opt.agg_generic;
  // The update rides inside the aggregation kernel when a slice is a whole row of one snapshot
  // (F <= 64 in float4 pieces), W fits next to the row tiles in LDS and the fast addressing
  // applies; other shapes aggregate into Y first and multiply afterwards.
  bool fused = false, like_inside = false;
  if (upd) {
    a.W = upd->W;
    a.bias = upd->bias;
    a.Fo = upd->Fo;
    a.ldw = upd->ldw;
    a.ldh = upd->ldh;
    for (int t = 0; t < f->k; ++t) a.H[t] = upd->H[t];
    // (Widths of H that are no multiples of 16 as well, where the aggregation is wanted too; without A they are
    // refused.  What the update adds to the aggregation, behind it and inside: N = 200k, k = 4, F = 64, Fo = 8 / 20 / 40 51 / 61
    // / 78 -> 29 / 35 / 47 us, F = 16 25 / 39 / 59 -> 10 / 17 / 28; R-MAT 60k, k = 8, F = 64 58 / 62 / 79 -> 33 / 43 / 55.  From
    // 400k rows of all snapshots together on where a slice has more than 32 columns: with fewer, a wave's 16 rows four at
    // a time take up to 1.5 times as long as rows of their own and a second launch; 32 and less are 4 to 30 % faster, but for
    // R-MAT frames with N = 300k .. 450k, k = 4 and 8, F = 16, Fo <= 24: with fresh operands up to 8 % slower.)
    const bool tiles = upd->Fo >= 16 && upd->Fo % 16 == 0;
    // Widths that are multiples of 16 go inside, with the aggregation wanted and more than 32 columns but for two kinds of frames.
    // A wave inside takes 16 rows where that makes 2048 waves, those of mid and hub rows among them (`min_short` below; 32768 rows
    // where all are short), else 4.  With 16 there are too few such waves (3600 at 58000 rows) to hide what the longest of its
    // rows costs: with many entries, rows of their own and a second launch are faster.  With 4 it still multiplies 16: more than a
    // second launch costs with more than 32 columns of H.  The lines are those of the frames that were measured, in rows and
    // entries: 24000 rows with more than 500000 entries, which have long rows, mostly make the 2048 waves.  Of 1500 random frames
    // and widths of both kinds, 1 to 16 snapshots, Chung-Lu and R-MAT, 1 to 40 % churn, behind is 1.25x as fast in the mean (0.94x
    // to 1.65x; 98 in 100 gain; 2200 others the same): F = Fo = 64, n = 2k, k = 8, R-MAT of degree 16 26.0 -> 18.1 us, 24k, k = 2
    // 48.3 -> 38.8, 36k, k = 1 43.2 -> 33.5.  With fewer rows behind is 0.8 to 1.1x, with half the entries (24k, k = 2, degree 6)
    // 26.4 -> 27.7, from 58k rows on 0.85 to 1.3x without a rule that tells which, from 300k on 0.75 to 1.1x.
    const int64_t all_rows = (int64_t)f->n * f->k;
    int64_t all_entries = (int64_t)f->nnz_c * f->k;
    for (int t = 0; t < f->k; ++t) all_entries += f->nnz_d[t];
    const bool few_tiles = Y && F > 32 &&
                           (all_rows >= 24000 ? all_rows < 58000 && all_entries > 500000
                                              : all_rows >= 14500 && f->k > 1 && f->n >= 1500 && upd->Fo > 32);
    const bool inside = tiles ? !few_tiles : Y && (F <= 32 || all_rows >= 400000);
    const bool fusable = aligned && F >= 16 && F <= 64 && upd->Fo <= 64 && fast;
    fused = fusable && inside;
    like_inside = fusable && tiles && few_tiles;
    if (!fused && !Y) return PIPAD_ERR_INVALID_ARG;  // the two-step form needs Y as its workspace
  }
  int64_t entries = f->nnz_c;  // of a snapshot
  for (int t = 0; t < f->k; ++t) entries += f->nnz_d[t] / f->k;
  // Small F handed over as one concatenated operand: the coalescent kernel (snapshot groups).
  // Measured at F = 1 .. 27, k = 3 .. 16: on that operand it beats the per-snapshot slices by 1.03 to
  // 3.8x (a slice would use 4*F bytes of every k*F-float row it touches); on R-MAT frames with
  // F >= 16 it is up to 8 % slower (fewer hot rows fit in an L2); operands of a few hundred KB
  // are a tie.
  const int64_t mode = opt.agg_coalescent;  // 0 never, 1 automatic, 2 whenever possible
  const bool wanted = mode >= 2 || (mode == 1 && (int64_t)f->n * f->k * F * 4 >= ((int64_t)1 << 20));
  bool coalescent = wanted && !upd && !subset && F < 32 && f->k > 1 && ldx >= (int64_t)f->k * F &&
                    ldy >= (int64_t)f->k * F && (int64_t)f->n * ldx * 4 < ((int64_t)1 << 32);
  for (int t = 1; t < f->k && coalescent; ++t)
    coalescent = X[t] == X[0] + (int64_t)t * F && Y[t] == Y[0] + (int64_t)t * F;
  int cvec = 1;
  if (coalescent) {
    cvec = F >= 4 ? 4 : F >= 2 ? 2 : 1;  // (any 4-byte alignment: see V)
    // Snapshots side by side in a team: up to 64 columns, the groups as even as they get, and of
    // those splits the one that costs least by a sum of lanes (idle ones included) and 12 per cache
    // line that an entry's row is expected to touch.  Measured with 64, 48, 32 and 16 columns at most:
    // k = 12, F = 9 154, 139, 162, 172 us; k = 5, F = 16 910, 910, 832, 930; k = 3, F = 16 518, 518, 644,
    // 707; k = 8, F = 16 179, 225, 176, 246; k = 8, F = 6 351, 351, 356, 453; k = 3, F = 27 775, 863.
    const int lps = (F + cvec - 1) / cvec;
    int64_t best = INT64_MAX;
    for (int groups = (int)((f->k * F + 63) / 64); groups <= f->k; ++groups) {
      const int sg = (f->k + groups - 1) / groups;
      if (sg * F > 64 || (f->k + sg - 1) / sg != groups) continue;
      const int lanes_log2 = ceil_log2(sg * lps);
      const uint64_t starts = (uint64_t)ldx * 4 | reinterpret_cast<uintptr_t>(X[0]) | (uint64_t)sg * F * 4 | 128u;
      const int64_t align = (int64_t)(starts & (~starts + 1));
      const int64_t touched = (int64_t)f->k * F * 4 + groups * (128 - align);
      const int64_t cost = ((int64_t)groups << lanes_log2) * 128 + 12 * touched;
      if (cost > best) continue;
      best = cost;
      a.nslices = groups;  // snapshot groups
      a.sg = sg;
      a.ls_log2 = lanes_log2;  // lanes per team (<= 64)
    }
    a.fchunks = 1;
    // Short rows longest first where the common entries tell the lengths and rows are not narrow: 28 bytes of a team's row per
    // entry of a snapshot's that is common.  R-MAT 1M, k = 8, F = 1 / 2 / 4 / 8 / 16 310 / 366 / 476 / 788 / 1540 -> 294 / 348 / 447 /
    // 728 / 1444 us, 61k, k = 16, F = 3 68.7 -> 62, Chung-Lu 162k, k = 8, F = 3 92 -> 85; on the other side of it Chung-Lu 89k, k = 3,
    // F = 2 34 -> 36.4, 150k, k = 8, F = 2, churn 0.3 71 -> 74.
    a.longest_first = (int64_t)a.sg * F * 4 * f->nnz_c >= 28 * entries;
    // Common entries fetched once for the lanes of a quad (which lies within a team then) from 10 common entries per row on: R-MAT 1M,
    // k = 8, F = 1 / 2 / 4 290 / 350 / 442 -> 281 / 341 / 431 us, 300k, F = 2 116 -> 109, 700k, k = 3 177 -> 168, Chung-Lu 217k, k = 4,
    // F = 2 57.8 -> 55.0; 147k, k = 6, F = 1 50.2 -> 49.9.  With fewer, whose rows end soon after the common entries that make up whole
    // chunks, between 3 % faster and 3 % slower (Chung-Lu 260k, k = 8, F = 2 64.8 -> 66.5, 118k, k = 12, 70.8 -> 71.9).
    a.share = a.ls_log2 >= 2 && (int64_t)f->nnz_c >= 10 * (int64_t)f->n;
    // The gathered rows multiplied by their scales first (k_scale_rows), so that a walk only reads indices: one pass over the
    // operand against 4 bytes per entry and snapshot, of which an instruction of the walk touched up to 64 lines.  Measured,
    // that saves 1.5 us per million entries of all snapshots, whatever F is, and the pass takes 5 us and its bytes at 4.4 TB/s:
    // the rule asks for a little more.  Of 60 frames on the one side of it 0.57 to 0.97 of the time, at worst 1.00; on the
    // other 0.92 to 1.7: R-MAT 1M, k = 8, 20 entries per row, F = 1 / 2 / 4 / 8 / 12 534 / 578 / 629 / 915 / 1495 ->
    // 311 / 365 / 478 / 790 / 1355 us; 300k, F = 2 220 -> 127; Chung-Lu 200k, k = 8 101 -> 69; 500k, k = 4, F = 4 126 -> 118; and
    // 20k, k = 4, F = 16 12.6 -> 22, 1M, k = 2, 4 entries per row, F = 8 111 -> 123.
    const int64_t cols = (int64_t)f->k * F;
    // row stride: up to a cache line so that hardly any row lies on two, else whole 16 bytes
    a.ldt = cols > 32 ? (cols + 3) / 4 * 4 : cols > 8 && cols <= 12 ? 12 : (int64_t)4 << ceil_log2((cols + 3) / 4);
    a.products = 3 * f->k * entries > 10000000 + (int64_t)f->k * f->n * (4 * F + 1) && f->n * a.ldt <= kTableFloats;
  }
  // slice geometry: LS lanes of VEC columns each, 64 columns per slice (a gathered piece of a row is then
  // at most 256 bytes: two cache lines) or 128.  Rows of 65 to 128 columns go in one slice where
  // that touches fewer lines or there would be a half-empty second one: if they do not start at
  // lines, so that two slices both fetch the line where they meet, or are no longer than three.  Two
  // slices against one, k = 4, N = 200k Chung-Lu / 50k R-MAT / 500k Chung-Lu: dense rows, F = 66 751 / 139 / 1079 -> 550 /
  // 114 / 827 us, F = 100 984 / 153 / 1398 -> 802 / 136 / 1111, F = 127 1238 / 186 / 1789 -> 1063 / 170 / 1456; rows on
  // lines, F = 66 773 / 131 / 1122 -> 608 / 121 / 892, F = 80 603 / 124 / 919 -> 609 / 120 / 895, but F = 112
  // 791 / 134 / 1157 -> 848 / 145 / 1206: two.
  // The sums of a row depend on its slices, and a snapshot gets the same bits whichever others a call
  // takes and wherever its matrix lies: so the strides alone decide, not the pointers.  Rows are taken to
  // start at lines where ldx is a whole number of them, unless the snapshots lie side by side in a row that k
  // times F columns fit in and F is no whole number of lines (two slices against one, N = 200k, k = 4, F = 112 / 120
  // 794 / 945 -> 747 / 857 us; 50k R-MAT, k = 8 307 / 352 -> 268 / 308).  Matrices with whole lines from row to row that
  // start off a line are taken for ones that do (F = 112 882 us, in one slice 749).
  // Frames of few rows take two slices all the same: they have too few waves, and in one slice there are half as many
  // with half as many lane groups for a long row each.  Of 500 frames with F = 66 .. 127 and N = 1k .. 300k, operands in the caches
  // and not: two slices up to 1.5 times as fast for k = 1 .. 3 below the line (N = 12k Chung-Lu, k = 1 15.6 against 10.8 us; N = 10k
  // R-MAT, k = 2 22.1, 16.2; N = 15k, k = 2 30.2, 23.5), 5 to 25 % for k >= 4 (N = 1875 R-MAT, k = 4); past it one slice, up to
  // 25 % (N = 43k, k = 2 34.8 against 44.1; N = 10k, k = 8 33.8, 41.0).  Over all of them 6 % better than one
  // slice always, 0.5 % from the best of both; at worst 26 % slower than the other (N = 50 .. 58k Chung-Lu, k = 1).
  const int vec = coalescent ? cvec : vec4 ? 4 : 1;
  const bool side_by_side = f->k > 1 && ldx >= (int64_t)f->k * F;
  const bool on_lines = ldx % 32 == 0 && !(side_by_side && F % 32 != 0);
  const bool few_rows = (int64_t)f->n * f->k < (f->k == 1 ? 60000 : f->k <= 3 ? 50000 : 10000);
  int max_cols = !fused && !few_rows && F <= (on_lines ? 96 : 128) ? 128 : 64;
  if (opt.slice_cols > 0 && !fused) max_cols = (int)std::min<int64_t>(64, opt.slice_cols);
  const int cols = std::min(F, max_cols);
  if (!coalescent) {
    a.ls_log2 = ceil_log2((cols + vec - 1) / vec);
    // One or two columns: a team of four lanes as well, idle ones among them, that fetch entries together (F = 1,
    // N = 20k, k = 4 18.7 -> 10.4 us, 200k 102 -> 78, R-MAT 1M 579 -> 564; F = 2 13.9 -> 10.7, 88 -> 82, 606 -> 595).  Their
    // partial sums, where there are any, take the room of four columns: only where every call with k
    // snapshots needs that much, and the fixed scratch array holds it.
    if (F <= 2 && opt.slice_cols == 0 &&
        (a.nvp == 0 || (f->k >= 4 && a.nvp * 16 <= (int64_t)PIPAD_STATIC_SCRATCH_BYTES)))
      a.ls_log2 = 2;
    a.fchunks = (F + ((1 << a.ls_log2) * vec) - 1) / ((1 << a.ls_log2) * vec);
    a.nslices = f->k * a.fchunks;
  }
  const int sw = (1 << a.ls_log2) * vec;
  a.team_log2 = coalescent || !fast ? a.ls_log2 : short_row_team(f, a.ls_log2, F, a.fchunks);
  a.uneven = !coalescent && fast && !fused && uneven_rows(f, a.ls_log2, F, entries);
  const int nteams = kWave >> a.team_log2;
  if (a.order < 0) {
    const int64_t matrix = (int64_t)f->n * sw * 4, slices = (int64_t)a.nsel * a.fchunks;
    a.order = matrix >= (int64_t)PIPAD_ORDER_BYTES ? 1 : 0;
    // Side by side, in turn: workgroup b, on XCD b mod 8, takes slice b mod `slices`, so that an XCD keeps to
    // one or a few slices where their number divides 8, and goes through most of them otherwise, with
    // more matrices in its L2 than that can hold.  Then an XCD gets a run of slices instead (order 2).
    // Measured, k = 3 .. 16, 6 to 16 entries per row, R-MAT and Chung-Lu frames: 5 MiB matrices
    // and more, 8 entries per row and more 5 to 26 % faster in the mean of each number of slices (N = 100k,
    // k = 5, F = 30 132 -> 98 us; N = 120k, k = 12, F = 16 258 -> 180), 3 % slower at worst; with 6 entries
    // per row it is the slices' parity that decides: odd numbers 5 to 13 % faster from 10 MiB on, others
    // between 7 % faster and 4 % slower; smaller matrices and numbers that divide 8 up to 30 % slower.
    // (All with operands in the caches as far as they fit.  Of 80 frames inside the rule 15 % faster in the mean so, at worst
    // 8 % slower; with operands that no cache holds 5 % faster, from 12 entries per row on 9 to 15 %, with 8 to 10 entries
    // and matrices of less than 12 MiB 5 to 7 % slower, at worst 13.)
    if (a.order == 0 && !coalescent && !fused && kClasses % slices != 0 && matrix >= (5 << 20) &&
        (entries >= 8 * (int64_t)f->n || (slices % 2 == 1 && matrix >= (10 << 20))))
      a.order = 2;
  }

  // Rows per wave: the full batches amortise the per-wave set-up (and let a wave request its next
  // row while it gathers the current one) on big frames; smaller ones get shorter batches, until what
  // runs together - one slice, or all of them when they go side by side - has about 44 waves for
  // every CU, and a lane team does not walk too many entries one after the other: some 50 where the
  // short rows hold most of the entries, 70 elsewhere.  Twice to four times as many waves were slower
  // by 4 to 27 % (N = 20k .. 200k), half as many by as much.  Chains of 70, 50 and 35 (N = 60k .. 1M,
  // k = 4 and 8): 50 against 70 is 0 to 5 % faster on Chung-Lu frames (N = 500k, k = 8, F = 128, hardly
  // any overlap: 5233 -> 5042 us; longer than 70: 5284), where the short rows hold 51 to 74 % of the
  // entries; on R-MAT frames, where they hold 24 to 28 %, it is a tie but for one loss of 3 % (N = 60k,
  // F = 64), and 35 is up to 5 % slower than 70.
  {
    a.batch_short = kShortRowsPerWave;
    a.batch_mid = kLongRowsPerWave;
    a.batch_wide = kWideUnitsPerWave;
    const int64_t slices_run = coalescent ? a.nslices : a.order == 1 ? 1 : (int64_t)a.nsel * a.fchunks;
    auto waves = [&]() {
      return ((int64_t)(f->n_short + a.batch_short - 1) / a.batch_short +
              (int64_t)(f->n_long + a.batch_mid - 1) / a.batch_mid +
              (a.plain ? (int64_t)f->n_items * kWavesPerBlock
                       : (int64_t)(f->n_items + a.batch_wide - 1) / a.batch_wide * f->nclass)) * slices_run;
    };
    // With the update fused in, a workgroup first copies W to LDS and a wave multiplies 16 rows at a
    // time, so batches stay longer (N = 200k, F = Fo = 64: 4 to 8 rows per wave take 1.36 ms, 32 take
    // 0.90, 64 take 0.95), and shorter than a tile only where there would be hardly any waves.
    const int64_t enough = fused ? 8192 : coalescent ? 64 * 1024 : 11 * 1024;
    int min_short = fused ? std::max(nteams, kTileRows) : nteams;
    // entries that a lane team walks one after the other in a batch of short rows
    auto chain = [&]() {
      return fused || coalescent || f->n_short == 0 ? 0 : f->short_entries * a.batch_short / nteams / f->n_short;
    };
    const int64_t longest_chain = 2 * f->short_entries > entries ? 50 : 70;
    if (a.order == 2) {
      // Runs of slices: 22000 waves of short rows and 2000 of mid ones in all; chains of 20 entries where
      // the short rows hold most of them, of 70 elsewhere; two rows per lane team at least, so that there
      // is something to put in order, where a team has 8 lanes and more.  (Of 360 frames the best of all
      // batches is 2.4 % faster in the mean; the rule of the other orders is 4 % slower.)
      a.batch_short = std::min(kShortRowsPerWave, 8 * nteams);
      const int at_least = nteams <= 8 ? 2 * nteams : nteams;
      const int64_t chain_max = 2 * f->short_entries > entries ? 20 : 70;
      while (a.batch_short > at_least && (f->n_short * slices_run / a.batch_short < 22000 || chain() > chain_max))
        a.batch_short >>= 1;
      a.batch_mid = 4;
      while (a.batch_mid > 1 && f->n_long * slices_run / a.batch_mid < 2000) a.batch_mid >>= 1;
      while (a.batch_wide > 1 && (int64_t)f->n_items * f->nclass * slices_run / a.batch_wide < 2000) a.batch_wide >>= 1;
    }
    while (a.order != 2 && ((waves() < enough && (a.batch_short > min_short || a.batch_mid > 1 || a.batch_wide > 1)) ||
           (chain() > longest_chain && a.batch_short > min_short))) {
      if (a.batch_short > min_short) a.batch_short >>= 1;
      if (a.batch_mid > 1) a.batch_mid >>= 1;
      if (a.batch_wide > 1) a.batch_wide >>= 1;
      if (a.batch_short <= min_short && fused && waves() < 2048) min_short = nteams;
    }
    a.batch_short = std::max(a.batch_short, nteams);
    auto blocks_for = [](int64_t items, int per_wave) {
      return (int32_t)((items + (int64_t)kWavesPerBlock * per_wave - 1) / ((int64_t)kWavesPerBlock * per_wave));
    };
    a.blocks_wide = a.plain ? 0 : blocks_for(f->n_items, a.batch_wide);
    a.blocks_mid = blocks_for(f->n_long, a.batch_mid);
    a.blocks_short = blocks_for(f->n_short, a.batch_short);
    if (!coalescent) {
      // phases start at multiples of 8 workgroups, with runs of slices the short rows as well
      if (a.order == 2) a.blocks_mid = align_xcd(a.blocks_mid);
      a.blocks_short += (kClasses - (a.blocks_mid + a.blocks_short) % kClasses) % kClasses;
      const int64_t hub_blocks = a.plain ? f->n_items : (int64_t)kClasses * a.blocks_wide << f->sub_log2;
      a.blocks_per_phase = hub_blocks + a.blocks_mid + a.blocks_short;
      a.per_phase = divisor(a.blocks_per_phase);
      a.per_row = divisor((int64_t)a.nsel * a.fchunks);
    }
  }

  // scratch for the partial sums: one slice-wide vector per class part and slice; k * F floats per class
  // part for the coalescent kernel
  const size_t per_snapshot = coalescent ? (size_t)a.nvp * (size_t)F : (size_t)a.nvp * (size_t)a.fchunks * (size_t)sw;
  size_t need = per_snapshot * (size_t)a.nsel;
  const size_t sums = align_up(need, 64), table = a.products ? (size_t)f->n * (size_t)a.ldt : 0;
  // It cannot grow where it is the fixed array, and not while the stream is being captured into a graph:
  // growing means allocating.  Captured, a call with a larger k * F than all before is refused; with
  // no larger one it is only the padding of its slices that can be missing.
  bool fixed = !scratch.frame;
  if (!fixed && (need > *scratch.floats || table > f->table_floats)) {
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &capturing) != hipSuccess) (void)hipGetLastError();
    fixed = capturing != hipStreamCaptureStatusNone;
    if (fixed && (size_t)a.nvp * (size_t)a.nsel * (size_t)F > *scratch.floats) return PIPAD_ERR_SCRATCH;
  }
  if (need > *scratch.floats && fixed) {
    if (coalescent) {
      // one partial sum per hub unit then, the same sums
      a.whole_units = 1;
      need /= (size_t)a.nclass;
      if (need > *scratch.floats) return PIPAD_ERR_SCRATCH;
    } else {
      // The snapshots in groups that fit, one launch after the other on the stream (a snapshot's
      // result does not depend on what runs beside it, so the bits are the same); there must be room
      // for one snapshot's partial sums.
      const size_t group = *scratch.floats / per_snapshot;
      if (group == 0) return PIPAD_ERR_SCRATCH;
      int32_t list[PIPAD_MAX_K];
      for (int q = 0; q < a.nsel; ++q) list[q] = subset ? subset[q] : q;
      for (int start = 0; start < a.nsel; start += (int)group) {
        const int rc = aggregate_launch(f, F, X, ldx, Y, ldy, st, scratch, fused ? upd : nullptr, list + start,
                                        std::min<int>((int)group, a.nsel - start));
        if (rc != PIPAD_OK) return rc;
      }
      return upd && !fused ? launch_update(a, like_inside, st) : PIPAD_OK;
    }
  }
  if (need > *scratch.floats) {
    // (the fused update takes slices of up to 64 columns also where the option asks for narrower ones)
    if (opt.slice_cols > 0) need = std::max(need, (size_t)a.nvp * (size_t)a.nsel * 64);
    void *ptr = nullptr;
    if (f->alloc) {
      // the caller's allocator owns the memory; a smaller buffer from before stays with it
      ptr = f->alloc(need * sizeof(float), f->alloc_ctx);
      if (!ptr) return PIPAD_ERR_ALLOC;
    } else {
      // the old buffer may still be in use by earlier aggregations of this frame
      if (*scratch.ptr) {
        PIPAD_HIP(hipDeviceSynchronize());
        (void)hipFree(*scratch.ptr);
      }
      *scratch.ptr = nullptr;
      *scratch.floats = 0;
      if (hipMalloc(&ptr, need * sizeof(float)) != hipSuccess) {
        (void)hipGetLastError();
        return PIPAD_ERR_ALLOC;
      }
    }
    *scratch.ptr = static_cast<float *>(ptr);
    *scratch.floats = need;
  }
  a.partial = *scratch.ptr;
  // The table goes behind the sums in the fixed array, into memory of its own otherwise (asked for last, and not again where as
  // much was refused before).  Without room for it the kernel makes its products itself, with the same bits; so it does in a
  // call that has no sums to put into the fixed array, and does not touch what all calls share, and with one sum per unit.
  if (table && !a.whole_units) {
    if (pipad_frame *const to = scratch.frame) {
      if (table > to->table_floats && table < to->table_refused && !fixed) {
        const size_t floats = std::max(table, std::min<size_t>(2 * to->table_floats, kTableFloats));
        if (void *ptr = Allocator{to->alloc, to->alloc_ctx, to}.get((kTableSkip + floats) * sizeof(float))) {
          to->table = static_cast<float *>(ptr) + kTableSkip;
          to->table_floats = floats;
        } else {
          to->table_refused = table;
        }
      }
      if (table <= to->table_floats) a.table = to->table;
    } else if (need > 0 && sums + table <= *scratch.floats) {
      a.table = *scratch.ptr + sums;
    }
  }
  if (coalescent)
    return cvec == 4 ? launch_coalescent<4>(a, st)
                     : cvec == 2 ? launch_coalescent<2>(a, st) : launch_coalescent<1>(a, st);
  if (fused) return launch<4>(a, fast, st, true);
  const int rc = vec4 ? launch<4>(a, fast, st) : launch<1>(a, fast, st);
  if (rc != PIPAD_OK || !upd) return rc;
  return launch_update(a, like_inside, st);
}

}  // namespace pipad
