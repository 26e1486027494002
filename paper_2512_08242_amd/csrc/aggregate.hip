// chopper_aggregate: metric aggregation at every granularity (paper Section
// III-C; granularities of Section I; duration and launch overhead as sums of
// kernel durations and bubbles, caption of Fig. end_to_end).
//
// Records are visited in (gpu, kind, start') order.  At marker level l the
// group of a record is identified by its deepest non-NONE marker among
// levels 0..l (or its GPU when all are NONE) and its kind; for nested
// markers that marker determines the whole path.  Rows are numbered in order
// of each group's first record.  Where every group is one run of the order,
// a count of the runs of every wave tile numbers the rows; where groups have
// several runs, or a filter leaves records out, an election over the pieces
// of the wave tiles does; both use the same wave-tile reduction (below).
// Markers that are not nested, whose groups need exact ids, more pieces to
// add than the overflow list holds, and markers out of range or beyond 2^30
// take the element-wise path:
//   1. election: atomicMin of the record position into a per-level owner
//      table keyed by group (only at positions where the key changes);
//   2. owners are counted per tile and one exclusive scan over the
//      level-major table of tile counts yields final row numbers, level
//      offsets included;
//   3. owners write the row header (path, gpu, kind, first record);
//   4. segmented reductions: tiles of 2048 items, eight consecutive items
//      per thread, a thread-local pass plus one block-wide segmented scan per
//      field.  The piece holding a row's first item stores the row; other
//      pieces of the same row (rare: the group's records are not
//      consecutive) go through a small overflow list applied with atomics.
// The finest level reads the records (counters exactly once); each coarser
// level reads the rows of the level below.  GPU and workload rows, which
// are few, accumulate with atomics.
#include <type_traits>

#include "sort.h"
#include "wave.h"

namespace chopper {

bool validate_records(const chopper_records* r);
bool validate_markers(const chopper_markers* m);

constexpr int kAggIpt = 8;
constexpr int kAggTile = kBlock * kAggIpt;
constexpr int kMaxLevels = 10;            // depth <= 8, + GPU + workload
constexpr int kMaxFields = 6 + 16;        // n dur gap ovl tmin tmax ctr[16]

struct FilterDev {
  uint64_t gpu_mask[4];
  uint32_t class_mask;
  uint32_t use_iter;
  uint32_t iter_lo, iter_hi;
  uint32_t active;
};

struct RecSrc {
  int64_t n;
  int D;
  int64_t M;
  const uint32_t* korder;
  const uint8_t* gpu;
  const uint8_t* cls;
  const int64_t* start;
  const int64_t* end;
  const uint32_t* idx;
  const int64_t* gap;
  const int64_t* ovl;
  const uint64_t* ctr;
  int nc;
  const uint32_t* mlabel;
  FilterDev f;
  // exact group ids of the marker levels ([D][n] by korder position), or
  // null: groups by the deepest marker (exact for nested markers)
  const uint32_t* gk;
  // the general path's items gathered once in korder position order (or
  // null: gathered through korder where used): marker path [D][n] and
  // gpu * 2 + kind (0xFFFF: left out by the filter)
  const uint32_t* ipath;
  const uint16_t* igk;
};

struct RowsDev {
  int64_t cap;
  uint32_t* path;
  uint8_t* gpu;
  uint8_t* kind;
  uint64_t* n;
  int64_t* dur;
  int64_t* gap;
  int64_t* ovl;
  int64_t* tmin;
  int64_t* tmax;
  uint32_t* first;
  uint64_t* ctr;
  uint32_t* firstpos;   // scratch: korder position of each row's first record
  int D;
  int nc;
};

// key space of a level
__host__ __device__ inline int64_t key_space(int li, int D, int64_t M) {
  if (li < D) return 2 * (M + 256);
  if (li == D) return 512;
  return 2;
}

__device__ inline bool rec_pass(const RecSrc& S, uint32_t r) {
  if (!S.f.active) return true;
  const uint32_t g = S.gpu[r], c = S.cls[r];
  if (!((S.f.gpu_mask[g >> 6] >> (g & 63)) & 1ull)) return false;
  if (c >= 32 || !((S.f.class_mask >> c) & 1u)) return false;
  if (S.f.use_iter) {
    if (S.D < 1) return false;
    const uint32_t m0 = S.idx[r];
    if (m0 == kNone || (int64_t)m0 >= S.M) return false;
    const uint32_t lab = S.mlabel[m0];
    if (lab < S.f.iter_lo || lab > S.f.iter_hi) return false;
  }
  return true;
}

// group key of a record with path p at level li (kNone: not aggregated)
__device__ inline uint32_t group_key(const uint32_t* p, int D, int64_t M,
                                     int li, uint32_t g, uint32_t kind) {
  if (li < D) {
    uint32_t slot = kNone;
    for (int l = 0; l <= li; ++l)
      if (p[l] != kNone) slot = p[l];
    if (slot == kNone) return (uint32_t)((M + g) * 2 + kind);
    if ((int64_t)slot >= M) return kNone;
    return slot * 2u + kind;
  }
  if (li == D) return g * 2u + kind;
  return kind;
}

// key of an item at level li: its exact group id at the marker levels when
// those are given (fpos = korder position of the item, or of the first
// record of a row), else the deepest-marker key
__device__ inline uint32_t item_key(const uint32_t* gk, int64_t nrec,
                                    const uint32_t* p, int D, int64_t M,
                                    int li, uint32_t g, uint32_t kind,
                                    uint32_t fpos) {
  if (gk && li < D) return gk[(int64_t)li * nrec + fpos];
  return group_key(p, D, M, li, g, kind);
}

// One record position: its record, pass flag, gpu, kind and path.
struct RecItem {
  uint32_t r;
  bool ok;
  uint32_t g, kind;
  uint32_t p[8];
};

__device__ inline void load_item(const RecSrc& S, int64_t pos, RecItem& it) {
  it.r = S.korder[pos];
  if (S.igk) {
    const uint32_t v = S.igk[pos];
    it.ok = v != 0xFFFFu;
    it.g = (v >> 1) & 255u;
    it.kind = v & 1u;
    for (int l = 0; l < S.D; ++l) it.p[l] = S.ipath[(int64_t)l * S.n + pos];
    return;
  }
  it.g = S.gpu[it.r];
  it.kind = (uint32_t)kind_of(S.cls[it.r]);
  it.ok = rec_pass(S, it.r);
  for (int l = 0; l < S.D; ++l) it.p[l] = S.idx[(int64_t)l * S.n + it.r];
}

// The general path's items in korder position order, gathered once.
__global__ __launch_bounds__(kBlock) void k_agg_items(RecSrc S, uint32_t* ipath,
                                                      uint16_t* igk) {
  const int64_t pos = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (pos >= S.n) return;
  const uint32_t r = S.korder[pos];
  const uint32_t g = S.gpu[r];
  const uint32_t kind = (uint32_t)kind_of(S.cls[r]);
  igk[pos] = rec_pass(S, r) ? (uint16_t)(g * 2u + kind) : (uint16_t)0xFFFFu;
  for (int l = 0; l < S.D; ++l)
    ipath[(int64_t)l * S.n + pos] = S.idx[(int64_t)l * S.n + r];
}

// ---------------------------------------------------- records in no order
// Reading a column through korder fetches a cache line per value where the
// order jumps (27 ms for the 20 columns of 50M records, and 8 ms for their
// markers and GPUs).  Such input goes through rows instead: a pass in input
// order puts several columns of a record side by side in one row, and the
// pass in korder order fetches that row -- one line, not one a column.
// Markers, GPU and kind (32 or 64 bytes) are written back in korder order,
// for the passes that read them several times; the fields go four columns at
// a time (32 bytes) straight into the reduction, one launch a group, so that
// the scratch is 32 bytes a record in the element-wise path's space.  50M
// records, depth 6, 16 counters: items 0.5 + 1.5 ms, each of the five groups
// 0.6 + 2.2 (with eight columns a group written back in korder order for one
// reduction, 160 bytes a record: 15.0 ms in place of 14.0).
constexpr int kRowCols = 4;
constexpr int64_t kStageMin = (int64_t)1 << 20;   // below, columns stay cached

// Do the records lie far from korder?  Positions spread over all of it are
// sampled by one block: *far = steps of more than 4,096 records among them.
__global__ __launch_bounds__(kBlock) void k_sample_jumps(const uint32_t* korder,
                                                         int64_t n,
                                                         uint32_t* far) {
  const int64_t p = (n - 1) * (int64_t)threadIdx.x / kBlock;
  const int64_t d = (int64_t)korder[p + 1] - (int64_t)korder[p];
  uint32_t tot;
  block_exclusive(d > 4096 || d < -4096 ? 1u : 0u, OpAdd(), 0u, &tot);
  if (threadIdx.x == 0) *far = tot;
}

// Items in rows of W words: the path in words 0 .. D - 1 (D < W) and, in the
// last word, gpu * 2 + kind (0xFFFF: left out).
template <int W>
__global__ __launch_bounds__(kBlock) void k_stage_items(RecSrc S, uint4* rows) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= S.n) return;
  uint32_t v[W];
#pragma unroll
  for (int l = 0; l < W; ++l)
    v[l] = l < S.D && l < W - 1 ? S.idx[(int64_t)l * S.n + i] : kNone;
  const uint32_t gk = (uint32_t)S.gpu[i] * 2u + (uint32_t)kind_of(S.cls[i]);
  v[W - 1] = rec_pass(S, (uint32_t)i) ? gk : 0xFFFFu;
#pragma unroll
  for (int q = 0; q < W / 4; ++q)
    rows[i * (W / 4) + q] =
        make_uint4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
}

template <int W>
__global__ __launch_bounds__(kBlock) void k_unstage_items(
    const uint32_t* korder, int64_t n, int D, const uint4* rows,
    uint32_t* ipath, uint16_t* igk) {
  const int64_t pos = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (pos >= n) return;
  const int64_t r = korder[pos];
  uint32_t v[W];
#pragma unroll
  for (int q = 0; q < W / 4; ++q) {
    const uint4 x = rows[r * (W / 4) + q];
    v[4 * q] = x.x;
    v[4 * q + 1] = x.y;
    v[4 * q + 2] = x.z;
    v[4 * q + 3] = x.w;
  }
#pragma unroll
  for (int l = 0; l < W - 1; ++l)
    if (l < D) ipath[(int64_t)l * n + pos] = v[l];
  igk[pos] = (uint16_t)v[W - 1];
}

// kRowCols columns (fewer: the rest of the row is not written)
struct StageCols {
  const uint64_t* in[kRowCols];
};

__global__ __launch_bounds__(kBlock) void k_stage_columns(StageCols C,
                                                          int64_t n,
                                                          ulonglong2* rows) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  uint64_t v[kRowCols];
#pragma unroll
  for (int c = 0; c < kRowCols; ++c) v[c] = C.in[c] ? C.in[c][i] : 0ull;
#pragma unroll
  for (int q = 0; q < kRowCols / 2; ++q)
    if (C.in[2 * q])
      rows[i * (kRowCols / 2) + q] = make_ulonglong2(v[2 * q], v[2 * q + 1]);
}

// ------------------------------------------------------------------ election
__global__ __launch_bounds__(kBlock) void k_agg_elect(RecSrc S, uint32_t act,
                                                      uint32_t** own) {
  __shared__ uint32_t s_last[kBlock];
  const int64_t base = (int64_t)blockIdx.x * kAggTile;
  RecItem it[kAggIpt];
  bool valid[kAggIpt];
  for (int j = 0; j < kAggIpt; ++j) {
    const int64_t pos = base + (int64_t)threadIdx.x * kAggIpt + j;
    valid[j] = pos < S.n;
    if (valid[j]) load_item(S, pos, it[j]);
  }
  for (int li = 0; li < S.D + 2; ++li) {
    if (!((act >> li) & 1u)) continue;
    uint32_t key[kAggIpt];
    for (int j = 0; j < kAggIpt; ++j) {
      const int64_t pos = base + (int64_t)threadIdx.x * kAggIpt + j;
      key[j] = (valid[j] && it[j].ok)
                   ? item_key(S.gk, S.n, it[j].p, S.D, S.M, li, it[j].g,
                              it[j].kind, (uint32_t)pos)
                   : kNone;
    }
    s_last[threadIdx.x] = key[kAggIpt - 1];
    __syncthreads();
    uint32_t prev = threadIdx.x > 0 ? s_last[threadIdx.x - 1] : kNone;
    for (int j = 0; j < kAggIpt; ++j) {
      const bool head = (threadIdx.x == 0 && j == 0) || key[j] != prev;
      if (key[j] != kNone && head) {
        const int64_t pos = base + (int64_t)threadIdx.x * kAggIpt + j;
        atomicMin(&own[li][key[j]], (uint32_t)pos);
      }
      prev = key[j];
    }
    __syncthreads();
  }
}

// owners per tile and level: position pos owns its key at level li
__global__ __launch_bounds__(kBlock) void k_agg_count(RecSrc S, uint32_t act,
                                                      uint32_t** own,
                                                      int64_t ntiles,
                                                      uint32_t* tilecnt) {
  const int64_t base = (int64_t)blockIdx.x * kAggTile;
  RecItem it[kAggIpt];
  bool valid[kAggIpt];
  for (int j = 0; j < kAggIpt; ++j) {
    const int64_t pos = base + (int64_t)threadIdx.x * kAggIpt + j;
    valid[j] = pos < S.n;
    if (valid[j]) load_item(S, pos, it[j]);
  }
  for (int li = 0; li < S.D + 2; ++li) {
    uint32_t c = 0;
    if ((act >> li) & 1u) {
      for (int j = 0; j < kAggIpt; ++j) {
        if (!valid[j] || !it[j].ok) continue;
        const int64_t pos = base + (int64_t)threadIdx.x * kAggIpt + j;
        const uint32_t key = item_key(S.gk, S.n, it[j].p, S.D, S.M, li,
                                      it[j].g, it[j].kind, (uint32_t)pos);
        if (key != kNone && own[li][key] == (uint32_t)pos) ++c;
      }
    }
    uint32_t tot;
    block_exclusive(c, OpAdd(), 0u, &tot);
    if (threadIdx.x == 0) tilecnt[(int64_t)li * ntiles + blockIdx.x] = tot;
  }
}

__global__ void k_agg_offsets_all(int L, int64_t ntiles, const uint32_t* tilebase,
                              const uint32_t* total, int64_t cap,
                              int64_t* level_offset, uint32_t* status) {
  const int li = threadIdx.x;
  if (li < L) level_offset[li] = ntiles > 0 ? tilebase[(int64_t)li * ntiles] : 0;
  if (li == L) {
    level_offset[L] = *total;
    if ((int64_t)*total > cap) atomicOr(status, (uint32_t)CHOPPER_ST_ROWS_OVERFLOW);
  }
}

// owners take their row: rowof[key] = row, header fields, and (atomic levels)
// initial sums
__global__ __launch_bounds__(kBlock) void k_agg_assign(
    RecSrc S, uint32_t act, uint32_t atomic_levels, uint32_t** own,
    uint32_t** rowof, int64_t ntiles, const uint32_t* tilebase, RowsDev R) {
  const int64_t base = (int64_t)blockIdx.x * kAggTile;
  RecItem it[kAggIpt];
  bool valid[kAggIpt];
  for (int j = 0; j < kAggIpt; ++j) {
    const int64_t pos = base + (int64_t)threadIdx.x * kAggIpt + j;
    valid[j] = pos < S.n;
    if (valid[j]) load_item(S, pos, it[j]);
  }
  for (int li = 0; li < S.D + 2; ++li) {
    if (!((act >> li) & 1u)) continue;   // uniform across the block
    uint32_t key[kAggIpt];
    bool mine[kAggIpt];
    uint32_t c = 0;
    for (int j = 0; j < kAggIpt; ++j) {
      const int64_t pos = base + (int64_t)threadIdx.x * kAggIpt + j;
      key[j] = (valid[j] && it[j].ok)
                   ? item_key(S.gk, S.n, it[j].p, S.D, S.M, li, it[j].g,
                              it[j].kind, (uint32_t)pos)
                   : kNone;
      mine[j] = key[j] != kNone && own[li][key[j]] == (uint32_t)pos;
      c += mine[j] ? 1u : 0u;
    }
    uint32_t tot;
    uint32_t row = block_exclusive(c, OpAdd(), 0u, &tot) +
                   tilebase[(int64_t)li * ntiles + blockIdx.x];
    for (int j = 0; j < kAggIpt; ++j) {
      if (!mine[j]) continue;
      const int64_t pos = base + (int64_t)threadIdx.x * kAggIpt + j;
      if (li == S.D + 1) {
        // workload rows span GPUs: ordered by kind alone
        row = tilebase[(int64_t)li * ntiles] +
              ((it[j].kind == 1u && own[li][0] != kNone) ? 1u : 0u);
      }
      rowof[li][key[j]] = row;
      if ((int64_t)row < R.cap) {
        for (int l = 0; l < S.D; ++l)
          R.path[(int64_t)l * R.cap + row] =
              (li < S.D && l <= li) ? it[j].p[l] : kNone;
        R.gpu[row] = (li == S.D + 1) ? (uint8_t)0xFF : (uint8_t)it[j].g;
        R.kind[row] = (uint8_t)it[j].kind;
        // workload rows: fixed after the reduction (k_agg_workload_first)
        R.first[row] = (li == S.D + 1) ? kNone : it[j].r;
        R.firstpos[row] = (uint32_t)pos;
        if ((atomic_levels >> li) & 1u) {
          R.n[row] = 0;
          R.dur[row] = 0;
          R.gap[row] = 0;
          R.ovl[row] = 0;
          R.tmin[row] = kI64Max;
          R.tmax[row] = kI64Min;
          for (int q = 0; q < R.nc; ++q) R.ctr[(int64_t)q * R.cap + row] = 0;
        }
      }
      ++row;
    }
  }
}

// ------------------------------------------------------------------ reduction
template <typename T>
struct FV {
  uint32_t f;
  T v;
};
template <typename T>
__device__ inline FV<T> shfl_up(FV<T> x, int d) {
  FV<T> r;
  r.f = __shfl_up(x.f, d, kWave);
  r.v = __shfl_up(x.v, d, kWave);
  return r;
}

struct CombAdd {
  __device__ uint64_t operator()(uint64_t a, uint64_t b) const { return a + b; }
};
struct CombMin {
  __device__ uint64_t operator()(uint64_t a, uint64_t b) const {
    return (int64_t)a < (int64_t)b ? a : b;
  }
};
struct CombMax {
  __device__ uint64_t operator()(uint64_t a, uint64_t b) const {
    return (int64_t)a > (int64_t)b ? a : b;
  }
};
struct CombLeft {
  __device__ uint64_t operator()(uint64_t a, uint64_t) const { return a; }
};

template <typename Comb>
struct OpSeg {
  Comb c;
  __device__ FV<uint64_t> operator()(FV<uint64_t> a, FV<uint64_t> b) const {
    return FV<uint64_t>{a.f | b.f, b.f ? b.v : c(a.v, b.v)};
  }
};

// Segmented inclusive scan over the tile; items are blocked (thread t owns
// items t*kAggIpt ..).  head[j] starts a new segment.
template <typename Comb>
__device__ inline void seg_scan(const bool (&head)[kAggIpt],
                                uint64_t (&x)[kAggIpt], uint64_t identity,
                                Comb comb) {
  FV<uint64_t> acc{0u, identity};
  for (int j = 0; j < kAggIpt; ++j) {
    if (head[j]) acc = FV<uint64_t>{1u, x[j]};
    else acc.v = comb(acc.v, x[j]);
    x[j] = acc.v;
  }
  FV<uint64_t> tot;
  FV<uint64_t> pre = block_exclusive(acc, OpSeg<Comb>{comb},
                                     FV<uint64_t>{0u, identity}, &tot);
  bool seen = false;
  for (int j = 0; j < kAggIpt; ++j) {
    seen = seen || head[j];
    if (!seen) x[j] = comb(pre.v, x[j]);
  }
}

struct FieldRef {
  const uint64_t* a;
  const uint64_t* b;
  int mode;
  __device__ uint64_t get(uint32_t r) const {
    if (mode == 0) return 1ull;
    if (mode == 1) return a[r] - b[r];
    return a[r];
  }
};

// column of row field f (same bits for the signed columns)
__device__ inline uint64_t* row_column(const RowsDev& R, int f) {
  switch (f) {
    case 0: return R.n;
    case 1: return (uint64_t*)R.dur;
    case 2: return (uint64_t*)R.gap;
    case 3: return (uint64_t*)R.ovl;
    case 4: return (uint64_t*)R.tmin;
    case 5: return (uint64_t*)R.tmax;
    default: return R.ctr + (int64_t)(f - 6) * R.cap;
  }
}

// Item sources for the reduction: records in korder, or rows of a finer
// level.  Fields: 0 n, 1 dur, 2 gap, 3 ovl, 4 tmin, 5 tmax, 6.. counters.
struct FromRecords {
  static constexpr bool kRecords = true;
  RecSrc S;
  // columns of the fast reduction: start and end give n (no load), dur,
  // tmin and tmax; the plain sums are gap, ovl and the counters
  __device__ const int64_t* start_col() const { return S.start; }
  __device__ const int64_t* end_col() const { return S.end; }
  __device__ int nsum() const { return 2 + S.nc; }
  __device__ const uint64_t* sum_col(int i) const {
    if (i == 0) return (const uint64_t*)S.gap;
    if (i == 1) return (const uint64_t*)S.ovl;
    return S.ctr + (int64_t)(i - 2) * S.n;
  }
  __device__ int sum_dst(int i) const { return i < 2 ? 2 + i : 6 + (i - 2); }
  __device__ int64_t count() const { return S.n; }
  __device__ void load(int64_t i, uint32_t& r, bool& ok, uint32_t* p,
                       uint32_t& g, uint32_t& kind, uint32_t& fpos) const {
    RecItem it;
    load_item(S, i, it);
    r = it.r;
    g = it.g;
    kind = it.kind;
    ok = it.ok;
    for (int l = 0; l < S.D; ++l) p[l] = it.p[l];
    fpos = (uint32_t)i;
  }
  __device__ uint32_t first_of(uint32_t r) const { return r; }
  __device__ uint32_t index(int64_t i) const { return S.korder[i]; }
  __device__ bool ok(uint32_t r) const { return rec_pass(S, r); }
  __device__ uint32_t pathv(uint32_t r, int l) const {
    return S.idx[(int64_t)l * S.n + r];
  }
  __device__ uint32_t gpuv(uint32_t r) const { return S.gpu[r]; }
  __device__ uint32_t kindv(uint32_t r) const {
    return (uint32_t)kind_of(S.cls[r]);
  }
  __device__ uint32_t keyof(uint32_t r, int li) const {
    if (!rec_pass(S, r)) return kNone;
    uint32_t p[8];
    for (int l = 0; l < S.D; ++l) p[l] = pathv(r, l);
    return group_key(p, S.D, S.M, li, gpuv(r), kindv(r));
  }
  __device__ uint32_t key_at(int li, const uint32_t* p, uint32_t g,
                             uint32_t kind, uint32_t fpos) const {
    return item_key(S.gk, S.n, p, S.D, S.M, li, g, kind, fpos);
  }
  // column of field f, resolved once per field: mode 0 constant 1,
  // 1 a[r] - b[r], 2 a[r]
  __device__ FieldRef fref(int f) const {
    switch (f) {
      case 0: return FieldRef{nullptr, nullptr, 0};
      case 1: return FieldRef{(const uint64_t*)S.end, (const uint64_t*)S.start, 1};
      case 2: return FieldRef{(const uint64_t*)S.gap, nullptr, 2};
      case 3: return FieldRef{(const uint64_t*)S.ovl, nullptr, 2};
      case 4: return FieldRef{(const uint64_t*)S.start, nullptr, 2};
      case 5: return FieldRef{(const uint64_t*)S.end, nullptr, 2};
      default: return FieldRef{S.ctr + (int64_t)(f - 6) * S.n, nullptr, 2};
    }
  }
  __device__ uint64_t field(int f, uint32_t r) const {
    switch (f) {
      case 0: return 1ull;
      case 1: return (uint64_t)(S.end[r] - S.start[r]);
      case 2: return (uint64_t)S.gap[r];
      case 3: return (uint64_t)S.ovl[r];
      case 4: return (uint64_t)S.start[r];
      case 5: return (uint64_t)S.end[r];
      default: return S.ctr[(int64_t)(f - 6) * S.n + r];
    }
  }
};

struct FromRows {
  static constexpr bool kRecords = false;
  RowsDev R;
  int64_t M;        // number of markers (key space)
  const int64_t* level_offset;
  int lo_slot;      // level_offset index of the finer level
  const uint32_t* gk = nullptr;   // exact group ids (RecSrc::gk) or null
  int64_t nrec = 0;               // records (row stride of gk)
  // columns of the fast reduction: tmin and tmax, then the plain sums
  // n, dur, gap, ovl and the counters
  __device__ const int64_t* start_col() const { return R.tmin; }
  __device__ const int64_t* end_col() const { return R.tmax; }
  __device__ int nsum() const { return 4 + R.nc; }
  __device__ const uint64_t* sum_col(int i) const {
    if (i < 4) return (const uint64_t*)row_column(R, i);
    return R.ctr + (int64_t)(i - 4) * R.cap;
  }
  __device__ int sum_dst(int i) const { return i < 4 ? i : 6 + (i - 4); }
  __device__ int64_t count() const {
    int64_t a = level_offset[lo_slot], b = level_offset[lo_slot + 1];
    if (b > R.cap) b = R.cap;
    return b > a ? b - a : 0;
  }
  __device__ void load(int64_t i, uint32_t& r, bool& ok, uint32_t* p,
                       uint32_t& g, uint32_t& kind, uint32_t& fpos) const {
    r = (uint32_t)(level_offset[lo_slot] + i);
    g = R.gpu[r];
    kind = R.kind[r];
    ok = true;
    for (int l = 0; l < R.D; ++l) p[l] = R.path[(int64_t)l * R.cap + r];
    fpos = R.firstpos[r];
  }
  __device__ uint32_t first_of(uint32_t r) const { return R.first[r]; }
  __device__ uint32_t index(int64_t i) const {
    return (uint32_t)(level_offset[lo_slot] + i);
  }
  __device__ bool ok(uint32_t) const { return true; }
  __device__ uint32_t pathv(uint32_t r, int l) const {
    return R.path[(int64_t)l * R.cap + r];
  }
  __device__ uint32_t gpuv(uint32_t r) const { return R.gpu[r]; }
  __device__ uint32_t kindv(uint32_t r) const { return R.kind[r]; }
  __device__ uint32_t keyof(uint32_t r, int li) const {
    uint32_t p[8];
    for (int l = 0; l < R.D; ++l) p[l] = pathv(r, l);
    return group_key(p, R.D, M, li, gpuv(r), kindv(r));
  }
  __device__ uint32_t key_at(int li, const uint32_t* p, uint32_t g,
                             uint32_t kind, uint32_t fpos) const {
    return item_key(gk, nrec, p, R.D, M, li, g, kind, fpos);
  }
  __device__ FieldRef fref(int f) const {
    return FieldRef{(const uint64_t*)row_column(R, f), nullptr, 2};
  }
  __device__ uint64_t field(int f, uint32_t r) const {
    switch (f) {
      case 0: return R.n[r];
      case 1: return (uint64_t)R.dur[r];
      case 2: return (uint64_t)R.gap[r];
      case 3: return (uint64_t)R.ovl[r];
      case 4: return (uint64_t)R.tmin[r];
      case 5: return (uint64_t)R.tmax[r];
      default: return R.ctr[(int64_t)(f - 6) * R.cap + r];
    }
  }
};

struct Overflow {
  uint32_t* count;   // entries requested
  uint32_t* lost;    // sticky: set when an entry did not fit
  uint32_t* row;
  uint64_t* val;     // [kMaxFields][cap]
  int64_t cap;
};

__device__ inline void store_field(RowsDev& R, int f, uint32_t row,
                                   uint64_t v) {
  switch (f) {
    case 0: R.n[row] = v; break;
    case 1: R.dur[row] = (int64_t)v; break;
    case 2: R.gap[row] = (int64_t)v; break;
    case 3: R.ovl[row] = (int64_t)v; break;
    case 4: R.tmin[row] = (int64_t)v; break;
    case 5: R.tmax[row] = (int64_t)v; break;
    default: R.ctr[(int64_t)(f - 6) * R.cap + row] = v; break;
  }
}

__device__ inline void atomic_field(RowsDev& R, int f, uint32_t row,
                                    uint64_t v) {
  switch (f) {
    case 0: atomicAdd((unsigned long long*)&R.n[row], (unsigned long long)v); break;
    case 1: atomicAdd((unsigned long long*)&R.dur[row], (unsigned long long)v); break;
    case 2: atomicAdd((unsigned long long*)&R.gap[row], (unsigned long long)v); break;
    case 3: atomicAdd((unsigned long long*)&R.ovl[row], (unsigned long long)v); break;
    case 4: atomicMin((long long*)&R.tmin[row], (long long)v); break;
    case 5: atomicMax((long long*)&R.tmax[row], (long long)v); break;
    default:
      atomicAdd((unsigned long long*)&R.ctr[(int64_t)(f - 6) * R.cap + row],
                (unsigned long long)v);
      break;
  }
}

template <typename Src>
__global__ __launch_bounds__(kBlock) void k_agg_reduce(
    Src src, int li, int D, int64_t M, bool atomic_mode, const uint32_t* own,
    const uint32_t* rowof, RowsDev R, Overflow ovf, int nfields,
    uint32_t* status, uint32_t* cflag) {
  __shared__ uint32_t s_last[kBlock];
  __shared__ uint32_t s_head0[kBlock];
  const int64_t cnt = src.count();
  const int64_t base = (int64_t)blockIdx.x * kAggTile;
  if (base >= cnt) return;   // uniform: whole block
  uint32_t rid[kAggIpt], tgt[kAggIpt];
  bool head[kAggIpt], last[kAggIpt], valid[kAggIpt];
  uint64_t ownbit[kAggIpt];
  bool conflict = false;
  for (int j = 0; j < kAggIpt; ++j) {
    const int64_t i = base + (int64_t)threadIdx.x * kAggIpt + j;
    valid[j] = i < cnt;
    tgt[j] = kNone;
    ownbit[j] = 0;
    rid[j] = 0;
    if (!valid[j]) continue;
    uint32_t p[8], g, kind, fpos;
    bool ok;
    src.load(i, rid[j], ok, p, g, kind, fpos);
    if (!ok) continue;
    const uint32_t key = src.key_at(li, p, g, kind, fpos);
    if (key == kNone) continue;
    const uint32_t row = rowof[key];
    tgt[j] = row;
    ownbit[j] = (!atomic_mode && own[key] == fpos) ? 1ull : 0ull;
    // the row holds its first item's path: another path here means a
    // marker shared by different paths (markers not nested); past the
    // capacity the first item is read instead
    if (li < D) {
      if ((int64_t)row < R.cap) {
        for (int l = 0; l <= li; ++l)
          if (R.path[(int64_t)l * R.cap + row] != p[l]) conflict = true;
      } else if constexpr (Src::kRecords) {
        // (rows of a coarser level always precede those of a finer one, so
        // only the records' level has items past the capacity)
        const uint32_t ro = src.S.korder[own[key]];
        for (int l = 0; l <= li; ++l)
          if (src.S.idx[(int64_t)l * src.S.n + ro] != p[l]) conflict = true;
      }
    }
  }
  wave_flag_or(status, conflict, (uint32_t)CHOPPER_ST_PATH_CONFLICT);
  wave_flag_or(cflag, conflict, 1u);
  // piece boundaries
  s_last[threadIdx.x] = tgt[kAggIpt - 1];
  __syncthreads();
  uint32_t prev = threadIdx.x > 0 ? s_last[threadIdx.x - 1] : kNone;
  for (int j = 0; j < kAggIpt; ++j) {
    head[j] = (threadIdx.x == 0 && j == 0) || !valid[j] || tgt[j] != prev;
    prev = tgt[j];
  }
  s_head0[threadIdx.x] = head[0] ? 1u : 0u;
  __syncthreads();
  for (int j = 0; j < kAggIpt; ++j) {
    bool next_head;
    if (j + 1 < kAggIpt) next_head = head[j + 1];
    else next_head = threadIdx.x + 1 < kBlock ? s_head0[threadIdx.x + 1] != 0 : true;
    last[j] = valid[j] && tgt[j] != kNone && next_head;
  }
  // is the piece the first piece of its row? (propagated from the head)
  seg_scan(head, ownbit, 0ull, CombLeft());
  // overflow slots for non-first pieces
  uint32_t slot[kAggIpt];
  for (int j = 0; j < kAggIpt; ++j) {
    slot[j] = kNone;
    if (last[j] && !atomic_mode && ownbit[j] == 0 && (int64_t)tgt[j] < R.cap) {
      uint32_t e = atomicAdd(ovf.count, 1u);
      if ((int64_t)e < ovf.cap) {
        slot[j] = e;
        ovf.row[e] = tgt[j];
      } else {
        atomicOr(ovf.lost, 1u);
      }
    }
  }
  for (int f = 0; f < nfields; ++f) {
    uint64_t x[kAggIpt];
    for (int j = 0; j < kAggIpt; ++j) {
      const bool use = valid[j] && tgt[j] != kNone;
      if (f == 4) x[j] = use ? src.field(f, rid[j]) : (uint64_t)kI64Max;
      else if (f == 5) x[j] = use ? src.field(f, rid[j]) : (uint64_t)kI64Min;
      else x[j] = use ? src.field(f, rid[j]) : 0ull;
    }
    if (f == 4) seg_scan(head, x, (uint64_t)kI64Max, CombMin());
    else if (f == 5) seg_scan(head, x, (uint64_t)kI64Min, CombMax());
    else seg_scan(head, x, 0ull, CombAdd());
    for (int j = 0; j < kAggIpt; ++j) {
      if (!last[j] || (int64_t)tgt[j] >= R.cap) continue;
      if (atomic_mode) atomic_field(R, f, tgt[j], x[j]);
      else if (ownbit[j]) store_field(R, f, tgt[j], x[j]);
      else if (slot[j] != kNone) ovf.val[(int64_t)f * ovf.cap + slot[j]] = x[j];
    }
  }
}

// ------------------------------------------------------------------ fast path
// When every group is one run of consecutive items -- the keys met at piece
// boundaries strictly increase inside each (gpu, kind) segment, which holds
// when markers are numbered in the order they open -- rows are simply the
// pieces in item order: no owner tables, rows numbered by counting piece
// heads.  Each wavefront works alone on a tile of kWaveTile consecutive
// items (eight per lane); nothing is shared between the waves of a block.
// The fast path runs only without a record filter; what it refuses goes to
// the election on wave tiles (k_gen_elect below).
static_assert(kAggIpt == kTileIpt, "wave tiles hold eight items per lane");

// group key from the deepest non-NONE slot
__device__ inline uint32_t slot_key(uint32_t slot, int64_t M, uint32_t gk) {
  if (slot == kNone) return (uint32_t)((M + (gk >> 1)) * 2 + (gk & 1u));
  if ((int64_t)slot >= M) return kNone;
  return slot * 2u + (gk & 1u);
}

// Marker counts below which the natural-tile heads pass compares slots.
constexpr uint32_t kSlotFastM = 1u << 30;

// The same as selects: m2 = (uint32_t)(2 M) and mlim = min(M, 2^32 - 1)
// (so that slot >= mlim iff slot >= M for every slot below kNone).
struct SlotKeys {
  uint32_t m2, mlim;
  __device__ explicit SlotKeys(int64_t M)
      : m2((uint32_t)(2 * M)),
        mlim(M >= (int64_t)kNone ? kNone : (uint32_t)M) {}
  __device__ uint32_t operator()(uint32_t slot, uint32_t gk) const {
    const uint32_t kval = slot >= mlim ? kNone : slot * 2u + (gk & 1u);
    return slot == kNone ? m2 + gk : kval;
  }
};

// key of an item at level li (marker levels, then the GPU level)
template <int MaxD>
__device__ inline uint32_t level_key(const uint32_t (&p)[MaxD], uint32_t gk,
                                     int li, int D, int64_t M) {
  if (li >= D) return gk;
  uint32_t slot = kNone;
#pragma unroll
  for (int l = 0; l < MaxD; ++l)
    if (l <= li && p[l] != kNone) slot = p[l];
  return slot_key(slot, M, gk);
}

// One item's source index, gpu * 2 + kind and path (levels >= D are NONE),
// loaded without branches so that all loads of a tile are in flight at once.
template <int MaxD, typename Src>
__device__ inline void gather_item(const Src& src, int64_t i, int D,
                                   uint32_t& r, uint32_t& gk,
                                   uint32_t (&p)[MaxD]) {
  r = src.index(i);
  gk = src.gpuv(r) * 2u + src.kindv(r);
  if (D > 0) {        // uniform; without levels there is no path column
#pragma unroll
    for (int l = 0; l < MaxD; ++l) {
      const uint32_t v = src.pathv(r, l < D ? l : D - 1);
      p[l] = l < D ? v : kNone;
    }
  } else {
#pragma unroll
    for (int l = 0; l < MaxD; ++l) p[l] = kNone;
  }
}

// Per wave tile: number of piece heads at every level in [lv0, lv1] whose
// bit is set in `act` (tilecnt[(li - lv0) * nwt + tile]); flags[0] |= 1 when
// a key does not increase inside its segment, flags[1] |= 1 << kind for the
// kinds present; PATH_CONFLICT when two neighbours share a key but not the
// path.  Items are striped (item j * 64 + lane of the tile in lane `lane`);
// the previous item comes from the lane below by a DPP rotate.
template <int MaxD, typename Src>
__device__ inline void agg_heads(
    const Src& src, uint32_t act, int lv0, int lv1, int D, int64_t M,
    int64_t nwt, uint32_t* tilecnt, uint32_t* flags, uint32_t* status) {
  const int lane = lane_id();
  const int64_t w =
      (int64_t)blockIdx.x * kWavesPerBlock + (int64_t)(threadIdx.x / kWave);
  if (w >= nwt) return;
  // groups already known not to be runs: the counts are not used
  if (__builtin_amdgcn_readfirstlane((int)flag_read(&flags[0])) & 1) return;
  const int64_t cnt = src.count();
  const int64_t base = w * kWaveTile;
  if (base >= cnt) {
    if (lane <= lv1 - lv0) tilecnt[(int64_t)lane * nwt + w] = 0;
    return;
  }
  const int tile_n =
      (int)((cnt - base) < kWaveTile ? (cnt - base) : (int64_t)kWaveTile);
  uint32_t r[kAggIpt], gk[kAggIpt], p[kAggIpt][MaxD];
  uint32_t cr, cgk, cp[MaxD];      // the item before the tile
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const int q = j * kWave + lane;
    gather_item<MaxD>(src, base + (q < tile_n ? q : 0), D, r[j], gk[j], p[j]);
  }
  gather_item<MaxD>(src, base > 0 ? base - 1 : 0, D, cr, cgk, cp);
  (void)cr;
  bool cvalid = base > 0;          // lane 0's previous item exists
  uint64_t cpk = 0;                // 4-bit head counts per level, packed
  bool notinc = false, conflict = false;
  uint32_t kinds = 0;
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    // previous item: lane below; lane 0 the last lane of the previous row
    uint32_t pp[MaxD], pgk;
#pragma unroll
    for (int l = 0; l < MaxD; ++l) {
      const uint32_t x = wave_ror1_u32(p[j][l]);
      pp[l] = lane == 0 ? cp[l] : x;
      cp[l] = x;
    }
    {
      const uint32_t x = wave_ror1_u32(gk[j]);
      pgk = lane == 0 ? cgk : x;
      cgk = x;
    }
    const bool pvalid = lane != 0 || cvalid;
    cvalid = true;
    const bool valid = j * kWave + lane < tile_n;
    uint32_t slot = kNone, pslot = kNone;
    bool eq = true;
#pragma unroll
    for (int li = 0; li < MaxD; ++li) {
      slot = p[j][li] != kNone ? p[j][li] : slot;
      pslot = pp[li] != kNone ? pp[li] : pslot;
      eq = eq && p[j][li] == pp[li];
      if (li >= D || li < lv0 || li > lv1 || !((act >> li) & 1u)) continue;
      const uint32_t key = slot_key(slot, M, gk[j]);
      const uint32_t pkey = pvalid ? slot_key(pslot, M, pgk) : kNone;
      if (valid && key == kNone) notinc = true;   // unkeyed item: general path
      if (key != pkey && key != kNone) {
        cpk += (valid ? 1ull : 0ull) << (4 * li);
        // inside a segment the no-marker group may only come first, so it
        // orders before every marker key in this test
        const int64_t ok = key >= 2 * M ? -1 : (int64_t)key;
        const int64_t opk = pkey >= 2 * M ? -1 : (int64_t)pkey;
        if (valid && pvalid && pgk == gk[j] && ok <= opk) notinc = true;
      } else if (valid && pvalid && key == pkey && key != kNone && !eq) {
        conflict = true;
      }
    }
    if (valid && D >= lv0 && D <= lv1 && ((act >> D) & 1u) &&
        (!pvalid || gk[j] != pgk)) {
      cpk += 1ull << (4 * D);
      kinds |= 1u << (gk[j] & 1u);
    }
  }
  // wave totals from bit planes of the per-lane counts (each at most 8)
  for (int li = lv0; li <= lv1; ++li) {
    const uint32_t c = (uint32_t)(cpk >> (4 * li)) & 15u;
    uint32_t tot = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      tot += (uint32_t)__popcll(__ballot((c >> b) & 1u)) << b;
    if (lane == 0) tilecnt[(int64_t)(li - lv0) * nwt + w] = tot;
  }
  wave_flag_or(&flags[0], notinc, 1u);
  // a conflict sends the call to the general path, which groups by the
  // whole path
  if (__ballot(conflict) != 0 && lane == 0) {
    atomicOr(&flags[0], 2u);
    atomicOr(status, (uint32_t)CHOPPER_ST_PATH_CONFLICT);
  }
  // kinds present: the shared word is zeroed before the launch and only
  // gains bits, so a bit read as set here was set by this launch
  const uint32_t kk = (__ballot(kinds & 1u) != 0 ? 1u : 0u) |
                      (__ballot(kinds & 2u) != 0 ? 2u : 0u);
  if (lane == 0 && kk &&
      (__atomic_load_n(&flags[1], __ATOMIC_RELAXED) & kk) != kk)
    atomicOr(&flags[1], kk);
}

// Level offsets and what the host reads: the level-major scan of the head
// counts gives every level but the workload level, whose rows are the kinds
// present.  `stage`, and `host` (a read-back slot or null) beside it,
// receive the three flags, the L + 1 offsets and, with `interior`, L more
// counts.  The last block of a heads pass does this itself for a small table
// (it scans it first), else one wave of its own.
struct StageOut {
  int L;
  int64_t stride;          // counts per level
  uint32_t* tilecnt;
  uint32_t* tilebase;      // scanned
  uint32_t* total;
  const uint32_t* interior;
  bool nat;                // flags[2] rules the counts out
  bool workload;
  int64_t cap;
  int64_t* level_offset;
  int64_t* stage;
  uint32_t* host;
  uint32_t* status;
  uint32_t* count;         // of the blocks that are done; null: not here
};

__device__ inline void stage_out(const StageOut& O, const uint32_t* flags,
                                 uint32_t total) {
  const int t = (int)threadIdx.x;
  const uint32_t f0 = flag_read(&flags[0]), f1 = flag_read(&flags[1]),
                 f2 = flag_read(&flags[2]);
  const int64_t tot =
      (int64_t)total + (O.workload ? __popc(f1 & 3u) : 0);
  auto put = [&](int i, int64_t v) {
    O.stage[i] = v;
    store_host(O.host, i, v);
  };
  if (t <= O.L) {
    const int64_t v =
        t == O.L ? tot : (int64_t)O.tilebase[(int64_t)t * O.stride];
    O.level_offset[t] = v;
    put(3 + t, v);
  }
  if (O.interior && t < O.L)
    put(3 + O.L + 1 + t, (int64_t)flag_read(&O.interior[t]));
  if (t < 3) put(t, (int64_t)(t == 0 ? f0 : t == 1 ? f1 : f2));
  // the counts are the row counts only when the path applies (and, for the
  // natural tiles, when the input order qualified)
  if (t == 0 && f0 == 0 && !(O.nat && f2) && tot > O.cap)
    atomicOr(O.status, (uint32_t)CHOPPER_ST_ROWS_OVERFLOW);
}

__global__ void k_agg_offsets(StageOut O, const uint32_t* flags) {
  stage_out(O, flags, *O.total);
}

// the end of a heads pass over `blocks` blocks: see StageOut
__device__ inline void heads_end(const StageOut& O, const uint32_t* flags,
                                 uint32_t blocks) {
  if (!O.count || !last_block(O.count, blocks)) return;
  const uint32_t tot =
      block_scan_array(O.tilecnt, O.tilebase, (int64_t)O.L * O.stride);
  if (threadIdx.x == 0) *O.total = tot;
  __syncthreads();
  stage_out(O, flags, tot);
}

template <int MaxD>
__global__ __launch_bounds__(kBlock) void k_agg_heads(
    FromRecords src, uint32_t act, int lv0, int lv1, int D, int64_t M,
    int64_t nwt, uint32_t* tilecnt, uint32_t* flags, uint32_t* status,
    StageOut O) {
  agg_heads<MaxD>(src, act, lv0, lv1, D, M, nwt, tilecnt, flags, status);
  heads_end(O, flags, gridDim.x);
}

// ------------------------------------------------------------ input order
// A profiler writes each GPU's records together and in start order.  For
// such input the (gpu, kind, start') order is the input order with every
// GPU's communication records moved after its compute records, so the fast
// path can read all columns in input order instead of through korder, where
// each sparse communication record would pull a whole cache line of every
// column.  A wave tile then covers consecutive input positions of one GPU
// and regroups its items by kind in LDS (compute first, order kept), which
// yields per (gpu, kind) exactly the item sequence of the korder tiles.
//
// Tiles: the natural tiles of kWaveTile positions, cut at GPU boundaries;
// GPU g owns tiles tb[g] .. tb[g + 1] - 1.  Head counts of a level are laid
// out as (gpu, kind, tile), so one exclusive scan numbers the rows in
// (gpu, kind, first record) order, as on the korder tiles.
struct NatGeom {
  const uint32_t* tb;   // [G + 1] first tile of every GPU; tb[G] = tiles
  const uint8_t* tg;    // [tiles] GPU of every tile
  const uint32_t* gs;   // [G] first input position of the GPU, kNone: none
  const uint32_t* ge;   // [G] one past its last position
  const int32_t* lp;    // [2][lps] last kind-k position before natural
                        // tile t, -1 if none
  const uint32_t* bad;  // nonzero: the input order does not qualify
  int64_t nnt;          // natural tiles
  int64_t lps;          // row stride of lp (nnt rounded up to kLpIpt)
  int G;
  // the fast-path flags, for a launch queued before the host has read them:
  // it does nothing unless flags[0] and flags[2] are both zero
  const uint32_t* fflags = nullptr;
};

struct NatTile {
  uint32_t g;
  int64_t base;
  int tile_n;
  int64_t prev[2];      // last kind-k position of the GPU before the tile
  uint32_t tbg, cg, tl; // GPU's first tile, its tile count, tile - tbg
};

// Geometry of tile tt; false past the last tile.
__device__ inline bool nat_tile(const NatGeom& N, int64_t tt, NatTile& T) {
  if (tt >= (int64_t)N.tb[N.G]) return false;
  const uint32_t g = N.tg[tt];
  const int64_t gs = N.gs[g], ge = N.ge[g];
  T.g = g;
  T.tbg = N.tb[g];
  T.cg = N.tb[g + 1] - T.tbg;
  T.tl = (uint32_t)(tt - T.tbg);
  const int64_t nt = gs / kWaveTile + T.tl;
  const int64_t a = nt * kWaveTile;
  T.base = a > gs ? a : gs;
  const int64_t e = a + kWaveTile < ge ? a + kWaveTile : ge;
  T.tile_n = (int)(e - T.base);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    int64_t pv = -1;
    if (T.base > gs) {
      pv = N.lp[(int64_t)k * N.lps + nt];
      if (pv < gs) pv = -1;
    }
    T.prev[k] = pv;
  }
  return true;
}

// Kind regrouping of a tile: item q (striped) goes to LDS slot dst[j]
// (padded), compute items first; n0 = compute items.
__device__ inline void nat_regroup(const bool (&valid)[kAggIpt],
                                   const uint32_t (&kind)[kAggIpt], int lane,
                                   uint32_t (&dst)[kAggIpt], int* n0_out) {
  uint64_t m0[kAggIpt], m1[kAggIpt];
  uint32_t n0 = 0;
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    m0[j] = __ballot(valid[j] && kind[j] == 0u);
    m1[j] = __ballot(valid[j] && kind[j] != 0u);
    n0 += (uint32_t)__popcll(m0[j]);
  }
  uint32_t c0 = 0, c1 = n0;
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    uint32_t d = (uint32_t)(j * kWave + lane);
    if (valid[j]) d = kind[j] == 0u ? c0 + lanes_below(m0[j])
                                    : c1 + lanes_below(m1[j]);
    dst[j] = (uint32_t)pad8((int)d);
    c0 += (uint32_t)__popcll(m0[j]);
    c1 += (uint32_t)__popcll(m1[j]);
  }
  *n0_out = (int)n0;
}

template <typename T>
__device__ inline void wave_regroup_to_blocked(T* slice, T (&v)[kAggIpt],
                                               const uint32_t (&dst)[kAggIpt],
                                               int lane) {
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) slice[dst[j]] = v[j];
  wave_sync();
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) v[j] = slice[pad8(lane * kAggIpt + j)];
  wave_sync();
}

template <typename T>
__device__ inline void wave_blocked_to_regrouped(
    T* slice, T (&v)[kAggIpt], const uint32_t (&dst)[kAggIpt], int lane) {
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) slice[pad8(lane * kAggIpt + j)] = v[j];
  wave_sync();
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) v[j] = slice[dst[j]];
  wave_sync();
}

// Per natural tile: last position of each kind, the first position of every
// GPU, and whether the order qualifies (GPU ids never decrease, start'
// never decreases inside a GPU, every id below G).  Lane l reads positions
// 8l .. 8l + 7 of the tile, with vector loads when the columns allow.
__global__ __launch_bounds__(kBlock) void k_nat_pre(
    int64_t n, int G, const uint8_t* gpu, const uint8_t* cls,
    const int64_t* start, int64_t nnt, int64_t lps, int32_t* lpraw,
    uint32_t* gs, uint32_t* bad) {
  const int lane = lane_id();
  const int64_t nt =
      (int64_t)blockIdx.x * kWavesPerBlock + (int64_t)(threadIdx.x / kWave);
  if (nt >= nnt) return;
  // (the order is already known not to qualify: nothing here is used)
  if (__builtin_amdgcn_readfirstlane((int)flag_read(bad)) != 0) return;
  const int64_t base = nt * kWaveTile;
  const int64_t p0 = base + (int64_t)lane * kAggIpt;
  uint32_t g[kAggIpt], k[kAggIpt];
  int64_t s[kAggIpt];
  const bool vec = base + kWaveTile <= n && ((uintptr_t)gpu & 7) == 0 &&
                   ((uintptr_t)cls & 7) == 0 && ((uintptr_t)start & 15) == 0;
  if (vec) {
    const uint64_t gw = *(const uint64_t*)(gpu + p0);
    const uint64_t cw = *(const uint64_t*)(cls + p0);
#pragma unroll
    for (int j = 0; j < kAggIpt; j += 2) {
      const longlong2 v = *(const longlong2*)(start + p0 + j);
      s[j] = v.x;
      s[j + 1] = v.y;
    }
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      g[j] = (uint32_t)(gw >> (8 * j)) & 0xFFu;
      k[j] = (uint32_t)kind_of((uint32_t)(cw >> (8 * j)) & 0xFFu);
    }
  } else {
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      const int64_t p = p0 + j;
      g[j] = p < n ? (uint32_t)gpu[p] : 0u;
      k[j] = p < n ? (uint32_t)kind_of(cls[p]) : 0u;
      s[j] = p < n ? start[p] : 0;
    }
  }
  // the item before each lane's first: the lane below, or the tile's
  // predecessor for lane 0
  uint32_t pg = wave_shr1_u32(0u, g[kAggIpt - 1]);
  int64_t ps = dpp_any<kDppWaveShr1, 0xF>((int64_t)0, s[kAggIpt - 1]);
  if (lane == 0 && base > 0) {
    pg = gpu[base - 1];
    ps = start[base - 1];
  }
  bool wrong = false;
  int32_t last[2] = {-1, -1};
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const int64_t p = p0 + j;
    if (p < n) {
      if (g[j] >= (uint32_t)G) wrong = true;
      if (p > 0 && (g[j] < pg || (g[j] == pg && s[j] < ps))) wrong = true;
      if ((p == 0 || g[j] != pg) && g[j] < (uint32_t)G) gs[g[j]] = (uint32_t)p;
      last[k[j] ? 1 : 0] = (int32_t)p;
    }
    pg = g[j];
    ps = s[j];
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const uint64_t m = __ballot(last[q] >= 0);
    const int32_t v =
        m ? __builtin_amdgcn_readlane(last[q], 63 - __clzll((long long)m))
          : -1;
    if (lane == 0) lpraw[(int64_t)q * lps + nt] = v;
  }
  wave_flag_or(bad, wrong, 1u);
}

// Block 0: GPU ranges, tile offsets and the GPU of every tile.  Blocks
// 1 ..: the exclusive running maximum of the last-position table over
// kLpSpan entries of each kind, each block taking the maximum of the entries
// before its span itself.
constexpr int kLpIpt = 4;                      // entries per thread and kind
constexpr int64_t kLpSpan = 1024 * kLpIpt;     // entries per block and kind
__global__ __launch_bounds__(1024) void k_nat_tiles(
    int64_t n, int G, int64_t nnt, int64_t lps, const int32_t* lpraw,
    int32_t* lp, const uint32_t* gs, uint32_t* ge, uint32_t* tb, uint8_t* tg,
    const uint32_t* bad) {
  if (*bad) return;
  __shared__ uint32_t s_c[256];
  __shared__ uint32_t s_tb[257];
  __shared__ int32_t s_w[2][1024 / kWave];
  __shared__ int32_t s_p[2][1024 / kWave];
  const int t = (int)threadIdx.x, lane = lane_id(), w = t / kWave;
  if (blockIdx.x == 0) {
    if (t < G) {
      const uint32_t a = gs[t];
      uint32_t e = (uint32_t)n;
      if (a != kNone) {
        for (int h = t + 1; h < G; ++h) {
          const uint32_t b = gs[h];
          if (b != kNone) {
            e = b;
            break;
          }
        }
      }
      ge[t] = a == kNone ? kNone : e;
      s_c[t] = a == kNone ? 0u
                          : (e - 1u) / (uint32_t)kWaveTile -
                                a / (uint32_t)kWaveTile + 1u;
    }
    __syncthreads();
    if (w == 0) {
      uint32_t carry = 0;
      for (int b0 = 0; b0 < G; b0 += kWave) {
        const uint32_t v = b0 + lane < G ? s_c[b0 + lane] : 0u;
        const uint32_t incl = wave_incl(v, OpAdd(), 0u);
        if (b0 + lane < G) {
          tb[b0 + lane] = carry + incl - v;
          s_tb[b0 + lane] = carry + incl - v;
        }
        carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
      }
      if (lane == 0) {
        tb[G] = carry;
        s_tb[G] = carry;
      }
    }
    __syncthreads();
    for (int g = 0; g < G; ++g)
      for (uint32_t i = s_tb[g] + (uint32_t)t; i < s_tb[g + 1]; i += 1024)
        tg[i] = (uint8_t)g;
    return;
  }
  OpMax op;
  const int64_t b0 = (int64_t)(blockIdx.x - 1) * kLpSpan;
  const int64_t i0 = b0 + (int64_t)t * kLpIpt;
  int32_t pre[2] = {-1, -1}, v[2][kLpIpt], acc[2] = {-1, -1};
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int32_t* row = lpraw + (int64_t)q * lps;
    for (int64_t i = (int64_t)t * kLpIpt; i < b0; i += kLpSpan) {
      const int4 x = *(const int4*)(row + i);
      pre[q] = op(pre[q], op(op(x.x, x.y), op(x.z, x.w)));
    }
    int4 x = make_int4(-1, -1, -1, -1);
    if (i0 < nnt) x = *(const int4*)(row + i0);
    v[q][0] = x.x;
    v[q][1] = i0 + 1 < nnt ? x.y : -1;
    v[q][2] = i0 + 2 < nnt ? x.z : -1;
    v[q][3] = i0 + 3 < nnt ? x.w : -1;
#pragma unroll
    for (int j = 0; j < kLpIpt; ++j) acc[q] = op(acc[q], v[q][j]);
  }
  int32_t incl[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    incl[q] = wave_incl(acc[q], op, (int32_t)-1);
    const int32_t pw = lane63(wave_incl(pre[q], op, (int32_t)-1));
    if (lane == kWave - 1) {
      s_w[q][w] = incl[q];
      s_p[q][w] = pw;
    }
  }
  __syncthreads();
  if (i0 >= nnt) return;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    int32_t p = -1;
    for (int r = 0; r < 1024 / kWave; ++r) {
      p = op(p, s_p[q][r]);
      if (r < w) p = op(p, s_w[q][r]);
    }
    p = op(p, wave_shr1_any((int32_t)-1, incl[q]));
    int4 x;
    x.x = p;
    p = op(p, v[q][0]);
    x.y = p;
    p = op(p, v[q][1]);
    x.z = p;
    p = op(p, v[q][2]);
    x.w = p;
    *(int4*)(lp + (int64_t)q * lps + i0) = x;
  }
}

// Item of the natural tiles: gpu * 2 + kind and path of input position i.
template <int MaxD>
__device__ inline void nat_item(const RecSrc& S, int64_t i, uint32_t g, int D,
                                uint32_t& gk, uint32_t (&p)[MaxD]) {
  gk = g * 2u + (uint32_t)kind_of(S.cls[i]);
#pragma unroll
  for (int l = 0; l < MaxD; ++l) {
    const int ll = l < D ? l : (D > 0 ? D - 1 : 0);
    const uint32_t v = D > 0 ? S.idx[(int64_t)ll * S.n + i] : kNone;
    p[l] = l < D ? v : kNone;
  }
}

// Heads pass over the natural tiles: per level and kind the groups that
// start in the tile, at tilecnt[(li - lv0) * stride + 2 * tbg + k * cg + tl];
// entries past the last tile are zeroed.  Flags as in k_agg_heads.
template <int MaxD>
__device__ inline void agg_heads_nat(
    const RecSrc& S, const NatGeom& N, uint32_t act, int lv0, int lv1, int D,
    int64_t M, int64_t stride, uint32_t* tilecnt, uint32_t* flags,
    uint32_t* status) {
  __shared__ uint32_t s_k[kWavesPerBlock][kSlice];
  if (*N.bad) return;
  const int lane = lane_id();
  const int wv = (int)(threadIdx.x / kWave);
  const int64_t tt = (int64_t)blockIdx.x * kWavesPerBlock + wv;
  if (tt >= N.nnt + N.G) return;
  if (__builtin_amdgcn_readfirstlane((int)flag_read(&flags[0])) & 1) return;
  NatTile T;
  if (!nat_tile(N, tt, T)) {
    if (lane <= lv1 - lv0) {
      tilecnt[(int64_t)lane * stride + 2 * tt] = 0;
      tilecnt[(int64_t)lane * stride + 2 * tt + 1] = 0;
    }
    return;
  }
  uint32_t* sk = s_k[wv];
  uint32_t gk[kAggIpt], p[kAggIpt][MaxD], kind[kAggIpt], dst[kAggIpt];
  bool valid[kAggIpt];
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const int q = j * kWave + lane;
    valid[j] = q < T.tile_n;
    nat_item<MaxD>(S, T.base + (valid[j] ? q : 0), T.g, D, gk[j], p[j]);
    kind[j] = gk[j] & 1u;
  }
  int n0;
  nat_regroup(valid, kind, lane, dst, &n0);
  wave_regroup_to_blocked(sk, gk, dst, lane);
#pragma unroll
  for (int l = 0; l < MaxD; ++l) {
    uint32_t x[kAggIpt];
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) x[j] = p[j][l];
    wave_regroup_to_blocked(sk, x, dst, lane);
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) p[j][l] = x[j];
  }
  // the items before the tile, one per kind (same GPU)
  uint32_t qgk[2], qp[2][MaxD];
  bool qv[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    qv[k] = T.prev[k] >= 0;
    nat_item<MaxD>(S, qv[k] ? T.prev[k] : T.base, T.g, D, qgk[k], qp[k]);
  }
  // 4-bit head counts per level (the GPU level D included), per kind
  using Cnt = typename std::conditional<(MaxD + 1) * 4 <= 32, uint32_t,
                                        uint64_t>::type;
  // Every item of a run of the tile, and the item before the run, has the
  // tile's GPU and the run's kind, so the keys of two consecutive items
  // compare as their slots: equal iff the slots are, ordered as slot + 1
  // modulo 2^32 (which puts items with no marker first, as their keys are),
  // a slot at or above M giving no key.  That holds while keys of distinct
  // slots differ, M < 2^30; beyond, the call takes the general path.
  const uint32_t mlim = (uint32_t)(M < (int64_t)kSlotFastM ? M : 0);
  Cnt cpk[2] = {0, 0};
  bool notinc = M >= (int64_t)kSlotFastM, conflict = false;
  uint32_t kinds = 0;
  // previous item in the regrouped order: lane below for j == 0
  uint32_t cp[MaxD];
#pragma unroll
  for (int l = 0; l < MaxD; ++l) cp[l] = wave_shr1_u32(0u, p[kAggIpt - 1][l]);
  // (selects rather than branches: the conditions differ between lanes)
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const int v = lane * kAggIpt + j;
    const bool vv = v < T.tile_n;
    const bool comm = v >= n0;
    // the first item of a kind takes the item before the tile of its kind
    const bool first = v == n0 || v == 0;
    const bool fk = v == n0;
    const bool pvalid = first ? (fk ? qv[1] : qv[0]) : true;
    uint32_t pp[MaxD];
#pragma unroll
    for (int l = 0; l < MaxD; ++l)
      pp[l] = first ? (fk ? qp[1][l] : qp[0][l]) : cp[l];
#pragma unroll
    for (int l = 0; l < MaxD; ++l) cp[l] = p[j][l];
    Cnt inc = 0;
    uint32_t slot = kNone, pslot = kNone;
    bool eq = true;
#pragma unroll
    for (int li = 0; li < MaxD; ++li) {
      slot = p[j][li] != kNone ? p[j][li] : slot;
      pslot = pp[li] != kNone ? pp[li] : pslot;
      eq = eq & (p[j][li] == pp[li]);
      if (li >= D || li < lv0 || li > lv1 || !((act >> li) & 1u)) continue;
      const uint32_t s1 = slot + 1u, ps1 = pslot + 1u;
      const bool bad = s1 > mlim;        // no key
      const bool same = slot == pslot;
      const bool head = !bad & (!pvalid | !same);
      notinc = notinc | (vv & bad);
      inc += (vv & head) ? (Cnt)1 << (4 * li) : (Cnt)0;
      notinc = notinc | (vv & head & pvalid & (s1 <= ps1));
      // equal keys over different paths: the groups are not the runs
      conflict = conflict | (vv & pvalid & !bad & same & !eq);
    }
    if (D >= lv0 && D <= lv1 && ((act >> D) & 1u)) {
      const bool g = vv & !pvalid;
      inc += g ? (Cnt)1 << (4 * D) : (Cnt)0;
      kinds |= g ? (comm ? 2u : 1u) : 0u;
    }
    cpk[0] += comm ? (Cnt)0 : inc;
    cpk[1] += comm ? inc : (Cnt)0;
  }
  for (int li = lv0; li <= lv1; ++li) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const uint32_t c = (uint32_t)(cpk[k] >> (4 * li)) & 15u;
      uint32_t tot = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        tot += (uint32_t)__popcll(__ballot((c >> b) & 1u)) << b;
      if (lane == 0)
        tilecnt[(int64_t)(li - lv0) * stride + 2 * (int64_t)T.tbg +
                (int64_t)k * T.cg + T.tl] = tot;
    }
  }
  wave_flag_or(&flags[0], notinc, 1u);
  // a conflict sends the call to the general path, which groups by the
  // whole path
  if (__ballot(conflict) != 0 && lane == 0) {
    atomicOr(&flags[0], 2u);
    atomicOr(status, (uint32_t)CHOPPER_ST_PATH_CONFLICT);
  }
  const uint32_t kk = (__ballot(kinds & 1u) != 0 ? 1u : 0u) |
                      (__ballot(kinds & 2u) != 0 ? 2u : 0u);
  if (lane == 0 && kk &&
      (__atomic_load_n(&flags[1], __ATOMIC_RELAXED) & kk) != kk)
    atomicOr(&flags[1], kk);
}

template <int MaxD>
__global__ __launch_bounds__(kBlock) void k_agg_heads_nat(
    RecSrc S, NatGeom N, uint32_t act, int lv0, int lv1, int D, int64_t M,
    int64_t stride, uint32_t* tilecnt, uint32_t* flags, uint32_t* status,
    StageOut O) {
  agg_heads_nat<MaxD>(S, N, act, lv0, lv1, D, M, stride, tilecnt, flags,
                      status);
  heads_end(O, flags, gridDim.x);
}

// ---------------------------------------------------- groups of several runs
// With a filter, or when groups are not runs (a marker that was lost leaves
// its records to the marker around it, whose group then comes back after
// every marker inside it; markers numbered out of order), rows are numbered
// by election: every piece (run of equal keys within a wave tile) puts the
// smallest position of its group into the group's entry of its level's
// table, and the piece whose first item is that position owns the row.  The
// passes share the tiles, the LDS regrouping and the reduction kernel of the
// fast path; items left out by the filter are regrouped behind the tile's
// last item.  Positions are input positions on natural tiles (a group never
// spans GPUs or kinds, inside which input order is (start', index) order)
// and korder positions otherwise.
//   k_gen_elect  keys of all levels, one atomicMin per piece (none where the
//                entry already holds a smaller position)
//   k_gen_count  owners per tile and level, each lane's owners as a byte of
//                a mask (so that no later pass reads the tables again), and
//                whether pieces of one key hold different paths
//   reduction    rows of the owners; other pieces go to the overflow list
//                with their key, owners leave their row in the table, and
//                k_gen_apply adds the list to the rows
// Against the element-wise passes further up (eight consecutive items per
// thread, uncoalesced, four passes over the tables), which still take what
// this path hands back: 2.46M records with 16 counters, two compute streams
// and one marker in a hundred lost, the whole call 2.62 -> 0.90 ms; a
// selection of 90 of 100 iterations 1.69 -> 0.54 ms, of which the election
// is 0.034, the count 0.058 (waiting on the table entries), the records
// reduction 0.228 (0.187 where groups are runs) and the lists 0.042.
struct GenTab {
  uint32_t* own[kMaxLevels];   // by group key; the row, after the reduction
  int64_t ks[kMaxLevels];
};

// Largest marker count of this path: keys below 2^31 leave the top bit of an
// overflow entry to tell the reduction's two levels apart.
constexpr int64_t kGenMaxM = ((int64_t)1 << 30) - 512;

// Tables to "no position", counters to zero.
__global__ __launch_bounds__(kBlock) void k_gen_fill(GenTab tab, uint32_t act,
                                                     uint32_t* flags,
                                                     uint32_t* interior,
                                                     uint32_t* ovf_count) {
  const int li = (int)blockIdx.y;
  if (blockIdx.x == 0 && li == 0) {
    if (threadIdx.x < 2) flags[threadIdx.x] = 0;
    // (the counter of finished blocks after the levels)
    if (threadIdx.x <= kMaxLevels) interior[threadIdx.x] = 0;
    if (threadIdx.x == 0) *ovf_count = 0;
  }
  if (!((act >> li) & 1u)) return;
  uint32_t* p = tab.own[li];
  const int64_t n4 = tab.ks[li] >> 2;
  const int64_t step = (int64_t)gridDim.x * kBlock;
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < (tab.ks[li] & 3)) p[4 * n4 + i] = kNone;
  for (; i < n4; i += step)
    ((uint4*)p)[i] = make_uint4(kNone, kNone, kNone, kNone);
}

// Does the filter keep a record with gpu * 2 + kind gk, class c and level-0
// marker m0?
__device__ inline bool filter_keeps(const RecSrc& S, uint32_t gk, uint32_t c,
                                    uint32_t m0) {
  const uint32_t g = gk >> 1;
  if (!((S.f.gpu_mask[g >> 6] >> (g & 63)) & 1ull)) return false;
  if (c >= 32 || !((S.f.class_mask >> c) & 1u)) return false;
  if (S.f.use_iter) {
    if (S.D < 1) return false;
    if (m0 == kNone || (int64_t)m0 >= S.M) return false;
    const uint32_t lab = S.mlabel[m0];
    if (lab < S.f.iter_lo || lab > S.f.iter_hi) return false;
  }
  return true;
}

// As nat_regroup, with valid items anywhere in the tile: n0 valid items of
// run 0 first, then those of run 1, then the rest.  nv = valid items.
__device__ inline void gen_regroup(const bool (&valid)[kAggIpt],
                                   const uint32_t (&run)[kAggIpt], int lane,
                                   uint32_t (&dst)[kAggIpt], int* n0_out,
                                   int* nv_out) {
  uint64_t m0[kAggIpt], m1[kAggIpt];
  uint32_t n0 = 0, n1 = 0;
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    m0[j] = __ballot(valid[j] && run[j] == 0u);
    m1[j] = __ballot(valid[j] && run[j] != 0u);
    n0 += (uint32_t)__popcll(m0[j]);
    n1 += (uint32_t)__popcll(m1[j]);
  }
  uint32_t c0 = 0, c1 = n0, c2 = n0 + n1;
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const uint64_t mx = ~(m0[j] | m1[j]);
    const uint64_t mine = valid[j] ? (run[j] == 0u ? m0[j] : m1[j]) : mx;
    const uint32_t c = valid[j] ? (run[j] == 0u ? c0 : c1) : c2;
    dst[j] = (uint32_t)pad8((int)(c + lanes_below(mine)));
    c0 += (uint32_t)__popcll(m0[j]);
    c1 += (uint32_t)__popcll(m1[j]);
    c2 += (uint32_t)__popcll(mx);
  }
  *n0_out = (int)n0;
  *nv_out = (int)(n0 + n1);
}

// A wave tile of this path, items striped: records of a natural tile
// (kNat), records in korder (the items gathered by k_agg_items), or rows of
// a finer level.
template <int MaxD>
struct GenTile {
  uint32_t rs[kAggIpt];       // record or row
  uint32_t id[kAggIpt];       // position the election compares
  uint32_t gk[kAggIpt];
  uint32_t p[kAggIpt][MaxD];
  uint32_t dst[kAggIpt];
  int n0, nv;                 // items of run 0, items of both
  int64_t e0, e1;             // entries of the runs' counts in a level
  int64_t prev[2];            // position before each run, -1: none
};

// False past the last tile (e0, e1 are then entries to clear).
template <int MaxD, bool kNat>
__device__ inline bool gen_load(const FromRecords& src, const NatGeom& N,
                                int64_t w, int D, int lane,
                                GenTile<MaxD>& X) {
  const RecSrc& S = src.S;
  bool valid[kAggIpt];
  uint32_t run[kAggIpt];
  if constexpr (kNat) {
    NatTile T;
    if (!nat_tile(N, w, T)) {
      X.e0 = 2 * w;
      X.e1 = 2 * w + 1;
      return false;
    }
    X.e0 = 2 * (int64_t)T.tbg + T.tl;
    X.e1 = X.e0 + T.cg;
    X.prev[0] = T.prev[0];
    X.prev[1] = T.prev[1];
    uint32_t c[kAggIpt];
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      const int q = j * kWave + lane;
      valid[j] = q < T.tile_n;
      const int64_t i = T.base + (valid[j] ? q : 0);
      X.rs[j] = (uint32_t)i;
      X.id[j] = (uint32_t)i;
      c[j] = S.cls[i];
      X.gk[j] = T.g * 2u + (uint32_t)kind_of(c[j]);
      run[j] = X.gk[j] & 1u;
#pragma unroll
      for (int l = 0; l < MaxD; ++l) {
        const int ll = l < D ? l : (D > 0 ? D - 1 : 0);
        const uint32_t v = D > 0 ? S.idx[(int64_t)ll * S.n + i] : kNone;
        X.p[j][l] = l < D ? v : kNone;
      }
    }
    if (S.f.active) {
#pragma unroll
      for (int j = 0; j < kAggIpt; ++j)
        valid[j] = valid[j] && filter_keeps(S, X.gk[j], c[j], X.p[j][0]);
    }
  } else {
    X.e0 = w;
    X.e1 = w;
    const int64_t base = w * kWaveTile;
    X.prev[0] = X.prev[1] = base - 1;
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      const int64_t i = base + j * kWave + lane;
      const bool in = i < S.n;
      const int64_t pos = in ? i : base;
      const uint32_t v = S.igk[pos];
      valid[j] = in && v != 0xFFFFu;
      X.rs[j] = S.korder[pos];
      X.id[j] = (uint32_t)pos;
      X.gk[j] = v & 511u;
      run[j] = 0;
#pragma unroll
      for (int l = 0; l < MaxD; ++l) {
        const int ll = l < D ? l : (D > 0 ? D - 1 : 0);
        const uint32_t u = D > 0 ? S.ipath[(int64_t)ll * S.n + pos] : kNone;
        X.p[j][l] = l < D ? u : kNone;
      }
    }
  }
  gen_regroup(valid, run, lane, X.dst, &X.n0, &X.nv);
  return true;
}

template <int MaxD, bool kNat>
__device__ inline bool gen_load(const FromRows& src, const NatGeom&,
                                int64_t w, int D, int lane,
                                GenTile<MaxD>& X) {
  X.e0 = w;
  X.e1 = w;
  const int64_t cnt = src.count();
  const int64_t base = w * kWaveTile;
  if (base >= cnt) return false;
  const int n =
      (int)((cnt - base) < kWaveTile ? (cnt - base) : (int64_t)kWaveTile);
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const int q = j * kWave + lane;
    gather_item<MaxD>(src, base + (q < n ? q : 0), D, X.rs[j], X.gk[j],
                      X.p[j]);
    X.id[j] = src.R.firstpos[X.rs[j]];
    X.dst[j] = (uint32_t)pad8(q);
  }
  X.n0 = n;
  X.nv = n;
  return true;
}

// The tile's items to the blocked arrangement (lane holds 8 lane + j).
template <int MaxD>
__device__ inline void gen_block(GenTile<MaxD>& X, uint32_t* sk, int lane) {
  wave_regroup_to_blocked(sk, X.id, X.dst, lane);
  wave_regroup_to_blocked(sk, X.gk, X.dst, lane);
#pragma unroll
  for (int l = 0; l < MaxD; ++l) {
    uint32_t x[kAggIpt];
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) x[j] = X.p[j][l];
    wave_regroup_to_blocked(sk, x, X.dst, lane);
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) X.p[j][l] = x[j];
  }
}

// Bit j: item j of the lane starts a piece (valid items only).
__device__ inline uint32_t gen_heads(const uint32_t (&key)[kAggIpt], int n0,
                                     int nv, int lane) {
  uint32_t prev = wave_shr1_u32(0u, key[kAggIpt - 1]);
  uint32_t m = 0;
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const int v = lane * kAggIpt + j;
    if (v < nv && (v == 0 || v == n0 || key[j] != prev)) m |= 1u << j;
    prev = key[j];
  }
  return m;
}

// The kept item before each of a tile's two runs, if there is one.
template <int MaxD>
struct GenPrev {
  uint32_t p[2][MaxD], gk[2];
  uint32_t slot[2];           // deepest marker of the levels met so far
  bool kept[2];
};

template <int MaxD, bool kNat>
__device__ inline void gen_prev(const FromRecords& src,
                                const GenTile<MaxD>& X, int D,
                                GenPrev<MaxD>& Q) {
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int64_t i = X.prev[k];
    Q.slot[k] = kNone;
    Q.kept[k] = i >= 0;
    const int64_t ii = Q.kept[k] ? i : 0;
    if constexpr (kNat) {
      const uint32_t c = src.S.cls[ii];
      nat_item<MaxD>(src.S, ii, src.S.gpu[ii], D, Q.gk[k], Q.p[k]);
      if (src.S.f.active)
        Q.kept[k] = Q.kept[k] && filter_keeps(src.S, Q.gk[k], c, Q.p[k][0]);
    } else {
      const uint32_t v = src.S.igk[ii];
      Q.kept[k] = Q.kept[k] && v != 0xFFFFu;
      Q.gk[k] = v & 511u;
#pragma unroll
      for (int l = 0; l < MaxD; ++l)
        Q.p[k][l] = l < D ? src.S.ipath[(int64_t)l * src.S.n + ii] : kNone;
    }
  }
}

template <int MaxD>
__device__ inline void gen_prev_level(GenPrev<MaxD>& Q, int li) {
#pragma unroll
  for (int k = 0; k < 2; ++k)
    Q.slot[k] = Q.p[k][li] != kNone ? Q.p[k][li] : Q.slot[k];
}

// Bit j: item j of the lane is the first of its run in the tile and belongs
// to the group of the kept item before the run.
template <int MaxD, bool kNat>
__device__ inline uint32_t gen_goes_on(const GenTile<MaxD>& X,
                                       const GenPrev<MaxD>& Q,
                                       const uint32_t (&key)[kAggIpt],
                                       bool marker, int64_t M, int lane) {
  uint32_t m = 0;
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const int v = lane * kAggIpt + j;
    if (v != 0 && v != X.n0) continue;
    const int k = kNat && v == X.n0 ? 1 : 0;
    const uint32_t g = k ? Q.gk[1] : Q.gk[0];
    const uint32_t qk =
        marker ? slot_key(k ? Q.slot[1] : Q.slot[0], M, g) : g;
    if ((k ? Q.kept[1] : Q.kept[0]) && key[j] == qk) m |= 1u << j;
  }
  return m;
}

template <int MaxD, bool kNat>
__global__ __launch_bounds__(kBlock) void k_gen_elect(
    FromRecords src, NatGeom N, uint32_t act, int D, int64_t M, int64_t nwt,
    GenTab tab, uint32_t* flags) {
  __shared__ uint32_t s_k[kWavesPerBlock][kSlice];
  if constexpr (kNat) {
    if (*N.bad) return;
  }
  const int lane = lane_id();
  const int wv = (int)(threadIdx.x / kWave);
  const int64_t w = (int64_t)blockIdx.x * kWavesPerBlock + wv;
  if (w >= nwt) return;
  GenTile<MaxD> X;
  if (!gen_load<MaxD, kNat>(src, N, w, D, lane, X)) return;
  gen_block(X, s_k[wv], lane);
  // a piece that goes on with its group has nothing to elect (without this
  // every tile would meet at the entries of the coarse levels: 0.097 instead
  // of 0.034 ms on 2.46M records)
  GenPrev<MaxD> Q;
  gen_prev<MaxD, kNat>(src, X, D, Q);
  uint32_t slot[kAggIpt], key[kAggIpt];
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) slot[j] = kNone;
  bool unkeyed = false;
  auto elect = [&](uint32_t* own, bool marker) {
    uint32_t m = gen_heads(key, X.n0, X.nv, lane);
    m &= ~gen_goes_on<MaxD, kNat>(X, Q, key, marker, M, lane);
    uint32_t cur[kAggIpt];
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j)
      cur[j] = (m >> j) & 1u && key[j] != kNone ? flag_read(own + key[j]) : 0u;
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j)
      if (cur[j] > X.id[j]) atomicMin(own + key[j], X.id[j]);
  };
#pragma unroll
  for (int li = 0; li < MaxD; ++li) {
    if (li >= D) continue;
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j)
      slot[j] = X.p[j][li] != kNone ? X.p[j][li] : slot[j];
    gen_prev_level(Q, li);
    if (!((act >> li) & 1u)) continue;
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      key[j] = slot_key(slot[j], M, X.gk[j]);
      if (lane * kAggIpt + j < X.nv && key[j] == kNone) unkeyed = true;
    }
    elect(tab.own[li], true);
  }
  if ((act >> D) & 1u) {
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) key[j] = X.gk[j];
    elect(tab.own[D], false);
  }
  // (an item whose marker is out of range: left to the element-wise path)
  wave_flag_or(&flags[0], unkeyed, 1u);
}

// Owners of levels [lv0, lv1] per tile: tilecnt[(li - lv0) * stride + entry]
// and omask[(li - lv0) * mstride + 64 w + lane].  From records also: the
// kinds present (flags[1]), the groups that come back (interior[li]: pieces
// that do not own their row and are not the rest of a piece of the tile
// before), and PATH_CONFLICT when two items of a key hold different paths.
template <int MaxD, typename Src, bool kNat>
__device__ inline void gen_count(
    const Src& src, const NatGeom& N, uint32_t act, int lv0, int lv1, int D,
    int64_t M, int64_t nwt, int64_t stride, const GenTab& tab,
    uint32_t* tilecnt, uint8_t* omask, int64_t mstride, uint32_t* flags,
    uint32_t* interior, uint32_t* status) {
  __shared__ uint32_t s_k[kWavesPerBlock][kSlice];
  if constexpr (kNat) {
    if (*N.bad) return;
  }
  const int lane = lane_id();
  const int wv = (int)(threadIdx.x / kWave);
  const int64_t w = (int64_t)blockIdx.x * kWavesPerBlock + wv;
  if (w >= nwt) return;
  GenTile<MaxD> X;
  if (!gen_load<MaxD, kNat>(src, N, w, D, lane, X)) {
    if (lane <= lv1 - lv0) {
      tilecnt[(int64_t)lane * stride + X.e0] = 0;
      tilecnt[(int64_t)lane * stride + X.e1] = 0;
    }
    return;
  }
  gen_block(X, s_k[wv], lane);
  uint32_t slot[kAggIpt], key[kAggIpt];
  bool eq[kAggIpt];            // path equal to the item before, so far
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    slot[j] = kNone;
    eq[j] = true;
  }
  bool conflict = false;
  GenPrev<MaxD> Q;
  if constexpr (Src::kRecords) gen_prev<MaxD, kNat>(src, X, D, Q);
  // items of the lane before position n0
  const int b0 = X.n0 - lane * kAggIpt;
  const uint32_t m_run0 = b0 <= 0 ? 0u : (b0 >= kAggIpt ? 0xFFu
                                                        : (1u << b0) - 1u);
  auto wave_total = [&](uint32_t c) {
    uint32_t t = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
      t += (uint32_t)__popcll(__ballot((c >> b) & 1u)) << b;
    return t;
  };
  auto level = [&](int li) {
    const uint32_t m = gen_heads(key, X.n0, X.nv, lane);
    const uint32_t* own = tab.own[li];
    uint32_t o[kAggIpt];
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j)
      o[j] = (m >> j) & 1u && key[j] != kNone ? own[key[j]] : kNone;
    uint32_t mine = 0, other = 0;
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      const bool h = (m >> j) & 1u && key[j] != kNone;
      mine |= h && o[j] == X.id[j] ? 1u << j : 0u;
      other |= h && o[j] != X.id[j] ? 1u << j : 0u;
    }
    if constexpr (Src::kRecords) {
      if (li < D) {
        // inside a piece, then the piece against its group's first item
#pragma unroll
        for (int j = 0; j < kAggIpt; ++j) {
          const int v = lane * kAggIpt + j;
          conflict |= v < X.nv && !((m >> j) & 1u) && key[j] != kNone &&
                      !eq[j];
          if ((other >> j) & 1u) {
#pragma unroll
            for (int l = 0; l < MaxD; ++l) {
              if (l > li) continue;
              const uint32_t* col = kNat ? src.S.idx : src.S.ipath;
              conflict |= col[(int64_t)l * src.S.n + o[j]] != X.p[j][l];
            }
          }
        }
      }
      const uint32_t back =
          other & ~gen_goes_on<MaxD, kNat>(X, Q, key, li < D, M, lane);
      const uint32_t t = wave_total((uint32_t)__popc(back));
      if (lane == 0 && t) atomicAdd(&interior[li], t);
    }
    omask[(int64_t)(li - lv0) * mstride + w * kWave + lane] = (uint8_t)mine;
    const uint32_t t0 = wave_total((uint32_t)__popc(mine & m_run0));
    uint32_t* tc = tilecnt + (int64_t)(li - lv0) * stride;
    if constexpr (kNat) {
      const uint32_t t1 = wave_total((uint32_t)__popc(mine & ~m_run0));
      if (lane == 0) tc[X.e1] = t1;
    }
    if (lane == 0) tc[X.e0] = t0;
  };
#pragma unroll
  for (int li = 0; li < MaxD; ++li) {
    if (li >= D) continue;
    if constexpr (Src::kRecords) {
      uint32_t prev = wave_shr1_u32(0u, X.p[kAggIpt - 1][li]);
#pragma unroll
      for (int j = 0; j < kAggIpt; ++j) {
        eq[j] = eq[j] && X.p[j][li] == prev;
        prev = X.p[j][li];
      }
      gen_prev_level(Q, li);
    }
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j)
      slot[j] = X.p[j][li] != kNone ? X.p[j][li] : slot[j];
    if (li < lv0 || li > lv1) continue;
    if (!((act >> li) & 1u)) {
      if (lane == 0) {
        tilecnt[(int64_t)(li - lv0) * stride + X.e0] = 0;
        tilecnt[(int64_t)(li - lv0) * stride + X.e1] = 0;
      }
      continue;
    }
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j)
      key[j] = slot_key(slot[j], M, X.gk[j]);
    level(li);
  }
  if (D <= lv1) {
    if ((act >> D) & 1u) {
#pragma unroll
      for (int j = 0; j < kAggIpt; ++j) key[j] = X.gk[j];
      level(D);
    } else if (lane == 0) {
      tilecnt[(int64_t)(D - lv0) * stride + X.e0] = 0;
      tilecnt[(int64_t)(D - lv0) * stride + X.e1] = 0;
    }
  }
  for (int li = D + 1; li <= lv1; ++li)
    if (lane == 0) {
      tilecnt[(int64_t)(li - lv0) * stride + X.e0] = 0;
      tilecnt[(int64_t)(li - lv0) * stride + X.e1] = 0;
    }
  if constexpr (Src::kRecords) {
    if (__ballot(conflict) != 0 && lane == 0) {
      atomicOr(&flags[0], 2u);
      atomicOr(status, (uint32_t)CHOPPER_ST_PATH_CONFLICT);
    }
    uint32_t kinds = 0;
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j)
      if (lane * kAggIpt + j < X.nv) kinds |= 1u << (X.gk[j] & 1u);
    const uint32_t kk = (__ballot(kinds & 1u) != 0 ? 1u : 0u) |
                        (__ballot(kinds & 2u) != 0 ? 2u : 0u);
    if (lane == 0 && kk && (flag_read(&flags[1]) & kk) != kk)
      atomicOr(&flags[1], kk);
  }
}

template <int MaxD, bool kNat>
__global__ __launch_bounds__(kBlock) void k_gen_count(
    FromRecords src, NatGeom N, uint32_t act, int lv0, int lv1, int D,
    int64_t M, int64_t nwt, int64_t stride, GenTab tab, uint32_t* tilecnt,
    uint8_t* omask, int64_t mstride, uint32_t* flags, uint32_t* interior,
    uint32_t* status, StageOut O) {
  gen_count<MaxD, FromRecords, kNat>(src, N, act, lv0, lv1, D, M, nwt, stride,
                                     tab, tilecnt, omask, mstride, flags,
                                     interior, status);
  heads_end(O, flags, gridDim.x);
}

// over rows (the overflow list of the level below has been applied); the
// last block scans a table of at most kTailScan counts
template <int MaxD>
__global__ __launch_bounds__(kBlock) void k_gen_count_rows(
    FromRows src, uint32_t act, int lv0, int lv1, int D, int64_t M,
    int64_t nwt, GenTab tab, uint32_t* tilecnt, uint32_t* tilebase,
    uint8_t* omask, int64_t mstride, uint32_t* count, uint32_t* ovf_count) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *ovf_count = 0;
  const NatGeom none{};
  gen_count<MaxD, FromRows, false>(src, none, act, lv0, lv1, D, M, nwt, nwt,
                                   tab, tilecnt, omask, mstride, nullptr,
                                   nullptr, nullptr);
  if (!count || !last_block(count, gridDim.x)) return;
  block_scan_array(tilecnt, tilebase, (int64_t)(lv1 - lv0 + 1) * nwt);
}

// What the reduction needs of this path: the owner masks and tables of the
// level and the next coarser one.  kStaged: the rows of columns
// [c0, c0 + nc) of start, end, gap, ovl and the counters; the first group's
// launch has the headers and leaves every tile's first overflow slot of
// either level in `slots`, so that the others put their pieces' values beside
// its own.
struct GenRed {
  const uint8_t* mask = nullptr;
  const uint8_t* mask2 = nullptr;
  uint32_t* own = nullptr;
  uint32_t* own2 = nullptr;
  const ulonglong2* rows = nullptr;
  int c0 = 0, nc = 0;
  uint32_t* slots = nullptr;
};

// Overflow entries (group keys; top bit: the reduction's second level) to
// their rows, which the owners left in the tables.
__global__ __launch_bounds__(kBlock) void k_gen_apply(
    Overflow ovf, RowsDev R, int nfields, const uint32_t* own,
    const uint32_t* own2) {
  int64_t cnt = (int64_t)*ovf.count;
  if (cnt > ovf.cap) cnt = ovf.cap;
  const int64_t step = (int64_t)gridDim.x * kBlock;
  for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < cnt;
       e += step) {
    const uint32_t k = ovf.row[e];
    const uint32_t row = k >> 31 ? own2[k & 0x7FFFFFFFu] : own[k];
    if ((int64_t)row >= R.cap) continue;
    for (int f = 0; f < nfields; ++f)
      atomic_field(R, f, row, ovf.val[(int64_t)f * ovf.cap + e]);
  }
}

// Piece structure of one level over a wave tile (blocked arrangement: lane
// holds items lane * 8 + j).  Pieces are maximal runs of equal keys.  Items
// [0, n0) and [n0, tile_n) are two separate runs of rows (the two kinds of
// a natural tile; n0 = tile_n on korder tiles): rows r0 + i for the pieces
// of the first, r1 + i for the second.  The first piece of each may continue
// a row of an earlier tile (c0, c1).
struct LevelTile {
  uint32_t m_head;    // item starts a piece (tile start and invalid items too)
  uint32_t m_hv;      // ... and is valid
  uint32_t m_last;    // valid item ends a piece
  uint32_t m_real;    // valid item starts a group (key differs from previous)
  uint32_t pfx;       // pieces started in the lanes below
  uint32_t NP;        // pieces in the tile
  uint32_t NP0;       // pieces of the first run
  uint32_t c0, c1;    // the run's first piece continues an earlier row
  int64_t r0, r1;     // row of the run's first new group
  uint32_t before;    // items of the lane before its first piece head
  WaveSegMasks masks; // lane segment flags for wave scans
};

// slot[j]: LDS slot of item j's value -- its piece index when it ends a
// piece, else a junk slot of its own lane.  prev0 / prev1: keys of the items
// before each run (kNone: none).
__device__ inline void level_tile(const uint32_t (&key)[kAggIpt],
                                  uint32_t prev0, uint32_t prev1, int n0,
                                  int tile_n, int lane, int64_t r0, int64_t r1,
                                  LevelTile& T, uint32_t (&slot)[kAggIpt]) {
  uint32_t m_valid = 0, m_real = 0, m_head = 0;
  uint32_t prev = wave_shr1_u32(prev0, key[kAggIpt - 1]);
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const int q = lane * kAggIpt + j;
    const bool valid = q < tile_n;
    const uint32_t k = key[j];
    if (q == n0) prev = prev1;
    if (valid) m_valid |= 1u << j;
    if (valid && k != prev) m_real |= 1u << j;
    if (!valid || q == 0 || q == n0 || k != prev) m_head |= 1u << j;
    prev = k;
  }
  const uint64_t h0 = __ballot(m_head & 1u);
  const uint32_t next0 =
      lane == kWave - 1 ? 1u : (uint32_t)((h0 >> (lane + 1)) & 1u);
  T.m_head = m_head;
  T.m_hv = m_head & m_valid;
  T.m_real = m_real;
  T.m_last = m_valid & ((m_head >> 1) | (next0 << (kAggIpt - 1)));
  const uint32_t hc = (uint32_t)__popc(T.m_hv);
  T.pfx = wave_prefix_small<4>(hc);
  T.NP = (uint32_t)__builtin_amdgcn_readlane((int)(T.pfx + hc), kWave - 1);
  if (n0 >= tile_n) {
    T.NP0 = T.NP;
    T.c1 = 0;
  } else {
    // pieces that start below position n0, and whether the item there is
    // a new group
    const int ln = n0 / kAggIpt, jn = n0 % kAggIpt;
    const uint32_t below =
        T.pfx + (uint32_t)__popc(T.m_hv & ((1u << jn) - 1u));
    T.NP0 = (uint32_t)__builtin_amdgcn_readlane((int)below, ln);
    const uint32_t real_n =
        (uint32_t)__builtin_amdgcn_readlane((int)((m_real >> jn) & 1u), ln);
    T.c1 = real_n ? 0u : 1u;
  }
  T.c0 = n0 > 0 && __ballot(lane == 0 && !(m_real & 1u)) != 0 ? 1u : 0u;
  T.r0 = r0;
  T.r1 = r1;
  T.before = m_head ? (uint32_t)(__ffs(m_head) - 1) : (uint32_t)kAggIpt;
  T.masks = wave_seg_masks(m_head != 0);
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const uint32_t idx =
        T.pfx + (uint32_t)__popc(T.m_hv & ((2u << j) - 1u)) - 1u;
    slot[j] = ((T.m_last >> j) & 1u) ? idx : (uint32_t)(kWaveTile + lane);
  }
}

// Row of piece q, or -1 when it continues a row of an earlier tile.
__device__ inline int64_t piece_row(const LevelTile& T, uint32_t q) {
  const bool second = q >= T.NP0;
  const uint32_t qi = second ? q - T.NP0 : q;
  const uint32_t cc = second ? T.c1 : T.c0;
  if (qi < cc) return -1;
  return (second ? T.r1 : T.r0) + (int64_t)(qi - cc);
}

// Reduction of one level -- with kTwo also the next coarser one -- when
// groups are runs.  Within a wave tile, rows are numbered from the tile's
// head count (level-major exclusive scan of the heads pass).  Every field
// goes striped -> blocked through the wave's LDS slice; sums take one plain
// prefix sum over the tile and a piece's total is the difference of the
// prefix at its last item and at the previous piece's last item (exact
// modulo 2^64), for both levels from the same prefix; tmin and tmax take a
// segmented scan per level.  Piece values are written to LDS at the piece's
// index, so that the stores of consecutive lanes go to consecutive rows.  A
// run's first piece may continue a row of an earlier tile: it goes to the
// tile's overflow slot of its level (korder tiles: slot w of level li,
// nwt + w of level li - 1; natural tiles: 2w + kind and 2nwt + 2w + kind).
// Every valid item has a key here (the heads pass sends traces with unkeyed
// items to the general path).  kNat: the natural tiles, items read in input
// order and regrouped by kind on the way to the blocked arrangement.
// Where there are fewer tiles than wave slots, blockIdx.y splits a tile's
// fields over several waves, each of which finds the tile's pieces again
// (kSplit; reduce_parts below).
// kGen: groups of several runs (above): every piece is a head here, the
// owners' rows are numbered by rank, and a piece's row -- or, top bit set,
// its overflow slot -- is kept per piece in LDS.  kStaged: the columns come
// from rows, four a launch (see k_stage_columns).
constexpr int kSpecial = 5;
constexpr int64_t kReduceWaves = 3072;
template <int MaxD, typename Src, bool kTwo, bool kNat, bool kGen, bool kSplit,
          bool kStaged = false>
__global__ __launch_bounds__(kBlock) void k_agg_fast_reduce(
    Src src, NatGeom N, int li, int D, int64_t M, const uint32_t* tilebase,
    const uint32_t* tilebase2, const int64_t* row0, RowsDev R, Overflow ovf,
    int64_t nwt, GenRed GR) {
  __shared__ uint64_t s_v[kWavesPerBlock][kSlice];
  __shared__ uint32_t s_row[kGen ? kWavesPerBlock : 1][kGen && kTwo ? 2 : 1]
                           [kGen ? kWaveTile : 1];
  const int lane = lane_id();
  const int wv = (int)(threadIdx.x / kWave);
  const int64_t w = (int64_t)blockIdx.x * kWavesPerBlock + wv;
  if (w >= nwt) return;
  if constexpr (kNat) {
    if (N.fflags && __builtin_amdgcn_readfirstlane(
                        (int)(N.fflags[0] | N.fflags[2])) != 0)
      return;
  }
  int64_t base;
  int tile_n;
  NatTile NT;
  if constexpr (kGen) {
    base = 0;
    tile_n = 0;
  } else if constexpr (kNat) {
    if (!nat_tile(N, w, NT)) {
      if (lane < 2) {
        ovf.row[2 * w + lane] = kNone;
        if (kTwo) ovf.row[2 * nwt + 2 * w + lane] = kNone;
      }
      return;
    }
    base = NT.base;
    tile_n = NT.tile_n;
  } else {
    const int64_t cnt = src.count();
    base = w * kWaveTile;
    if (base >= cnt) {
      if (lane == 0) {
        ovf.row[w] = kNone;
        if (kTwo) ovf.row[nwt + w] = kNone;
      }
      return;
    }
    tile_n =
        (int)((cnt - base) < kWaveTile ? (cnt - base) : (int64_t)kWaveTile);
  }
  const int li2 = li - 1;
  uint64_t* sv = s_v[wv];
  uint32_t* sk = (uint32_t*)sv;
  // striped items: source index, gpu * 2 + kind, path, keys
  uint32_t rs[kAggIpt], gk[kAggIpt], p[kAggIpt][MaxD];
  uint32_t key[kAggIpt], key2[kAggIpt], dst[kAggIpt];
  uint32_t tprev[2] = {kNone, kNone}, tprev2[2] = {kNone, kNone};
  int n0 = tile_n;
  int64_t r0 = 0, r1 = 0, q0 = 0, q1 = 0;
  uint32_t id[kAggIpt];            // (kGen) election positions
  if constexpr (kGen) {
    GenTile<MaxD> X;
    if (!gen_load<MaxD, kNat>(src, N, w, D, lane, X)) return;
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      rs[j] = X.rs[j];
      id[j] = X.id[j];
      gk[j] = X.gk[j];
      dst[j] = X.dst[j];
#pragma unroll
      for (int l = 0; l < MaxD; ++l) p[j][l] = X.p[j][l];
    }
    n0 = X.n0;
    tile_n = X.nv;
    // (row0: the scan covers the rows' levels only, see below)
    r0 = (row0 ? row0[0] - (int64_t)tilebase[0] : 0) + (int64_t)tilebase[X.e0];
    r1 = kNat ? (int64_t)tilebase[X.e1] : r0;
    if (kTwo) {
      q0 = (row0 ? row0[-1] - (int64_t)tilebase2[0] : 0) +
           (int64_t)tilebase2[X.e0];
      q1 = kNat ? (int64_t)tilebase2[X.e1] : q0;
    }
  } else if constexpr (kNat) {
    bool valid[kAggIpt];
    uint32_t kind[kAggIpt];
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      const int q = j * kWave + lane;
      valid[j] = q < tile_n;
      rs[j] = (uint32_t)(base + (valid[j] ? q : 0));
      nat_item<MaxD>(src.S, rs[j], NT.g, D, gk[j], p[j]);
      kind[j] = gk[j] & 1u;
    }
    nat_regroup(valid, kind, lane, dst, &n0);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (NT.prev[k] < 0) continue;
      uint32_t cgk, cp[MaxD];
      nat_item<MaxD>(src.S, NT.prev[k], NT.g, D, cgk, cp);
      tprev[k] = level_key<MaxD>(cp, cgk, li, D, M);
      if (kTwo) tprev2[k] = level_key<MaxD>(cp, cgk, li2, D, M);
    }
    const int64_t e0 = 2 * (int64_t)NT.tbg + NT.tl;
    const int64_t e1 = e0 + NT.cg;
    r0 = tilebase[e0];
    r1 = tilebase[e1];
    if (kTwo) {
      q0 = tilebase2[e0];
      q1 = tilebase2[e1];
    }
  } else {
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      const int q = j * kWave + lane;
      gather_item<MaxD>(src, base + (q < tile_n ? q : 0), D, rs[j], gk[j],
                        p[j]);
      dst[j] = 0;
    }
    uint32_t cr, cgk, cp[MaxD];
    gather_item<MaxD>(src, base > 0 ? base - 1 : 0, D, cr, cgk, cp);
    tprev[0] = base > 0 ? level_key<MaxD>(cp, cgk, li, D, M) : kNone;
    if (kTwo)
      tprev2[0] = base > 0 ? level_key<MaxD>(cp, cgk, li2, D, M) : kNone;
    // rows: the level offset (row0, when the scan covers this level only)
    // plus the scanned head count; row0[-1] is the second level's offset
    r0 = (row0 ? row0[0] - (int64_t)tilebase[0] : 0) + (int64_t)tilebase[w];
    if (kTwo)
      q0 = (row0 ? row0[-1] - (int64_t)tilebase2[0] : 0) +
           (int64_t)tilebase2[w];
  }
  // (with kGen the items past tile_n, which the regrouping put there, have
  // keys too; level_tile looks at the first tile_n only)
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) {
    const int q = j * kWave + lane;
    key[j] = kGen || q < tile_n ? level_key<MaxD>(p[j], gk[j], li, D, M)
                                : kNone;
    key2[j] = kTwo && (kGen || q < tile_n)
                  ? level_key<MaxD>(p[j], gk[j], li2, D, M) : kNone;
  }
  auto blk32 = [&](uint32_t (&x)[kAggIpt]) {
    if constexpr (kNat || kGen) wave_regroup_to_blocked(sk, x, dst, lane);
    else wave_to_blocked(sk, x, lane);
  };
  auto blk64 = [&](uint64_t (&x)[kAggIpt]) {
    if constexpr (kNat || kGen) wave_regroup_to_blocked(sv, x, dst, lane);
    else wave_to_blocked(sv, x, lane);
  };
  blk32(key);
  if (kTwo) blk32(key2);
  LevelTile T1, T2;
  uint32_t slot[kAggIpt], slot2[kAggIpt];
  level_tile(key, tprev[0], tprev[1], n0, tile_n, lane, r0, r1, T1, slot);
  if (kTwo)
    level_tile(key2, tprev2[0], tprev2[1], n0, tile_n, lane, q0, q1, T2,
               slot2);
  // the launch, or the part, with the headers
  const bool first = kSplit ? blockIdx.y == 0 : !kStaged || GR.c0 == 0;
  // (kGen) rows of the pieces: owners by rank, the others an overflow slot
  uint32_t m_own = 0, m_own2 = 0, own_row[kAggIpt], own_row2[kAggIpt];
  auto piece_rows = [&](const LevelTile& T, const uint32_t (&k)[kAggIpt],
                        uint32_t mine, int which, uint32_t (&orow)[kAggIpt]) {
    const uint32_t other = T.m_hv & ~mine;
    const int b0 = n0 - lane * kAggIpt;
    const uint32_t m0 = b0 <= 0 ? 0u : (b0 >= kAggIpt ? 0xFFu
                                                      : (1u << b0) - 1u);
    const uint32_t c0 = (uint32_t)__popc(mine & m0);
    const uint32_t c1 = (uint32_t)__popc(mine & ~m0);
    const uint32_t x0 = wave_prefix_small<4>(c0);
    const uint32_t x1 = wave_prefix_small<4>(c1);
    const uint32_t co = (uint32_t)__popc(other);
    const uint32_t xo = wave_prefix_small<4>(co);
    const uint32_t no =
        (uint32_t)__builtin_amdgcn_readlane((int)(xo + co), kWave - 1);
    uint32_t ob = 0;
    if (no) {                      // uniform
      if (lane == 0) {
        ob = first ? atomicAdd(ovf.count, no) : GR.slots[2 * w + which];
        if (kStaged && first) GR.slots[2 * w + which] = ob;
      }
      ob = (uint32_t)__builtin_amdgcn_readlane((int)ob, 0);
    }
    uint32_t* srow = s_row[wv][which];
    const int64_t a0 = which ? q0 : r0, a1 = which ? q1 : r1;
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      const uint32_t below = (1u << j) - 1u;
      orow[j] = kNone;
      if (!((T.m_hv >> j) & 1u)) continue;
      const uint32_t q = T.pfx + (uint32_t)__popc(T.m_hv & below);
      uint32_t v = kNone;
      if ((mine >> j) & 1u) {
        const int64_t row =
            (m0 >> j) & 1u ? a0 + x0 + __popc(mine & m0 & below)
                           : a1 + x1 + __popc(mine & ~m0 & below);
        if (row < R.cap) v = (uint32_t)row;
        orow[j] = v;
      } else {
        const uint32_t e = ob + xo + (uint32_t)__popc(other & below);
        if ((int64_t)e < ovf.cap) {
          if (first) ovf.row[e] = k[j] | ((uint32_t)which << 31);
          v = e | 0x80000000u;
        }
      }
      srow[q] = v;
    }
  };
  if constexpr (kGen) {
    m_own = GR.mask[w * kWave + lane];
    piece_rows(T1, key, m_own, 0, own_row);
    if (kTwo) {
      m_own2 = GR.mask2[w * kWave + lane];
      piece_rows(T2, key2, m_own2, 1, own_row2);
    }
  }

  // headers of the rows that start here, written from the striped items:
  // the row of every group head goes back through LDS
  auto headers = [&](const LevelTile& T, int lv,
                     const uint32_t (&orow)[kAggIpt], uint32_t* own) {
    uint32_t rw[kAggIpt];
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      if constexpr (kGen) {
        rw[j] = orow[j];
        continue;
      }
      const uint32_t idx =
          T.pfx + (uint32_t)__popc(T.m_hv & ((2u << j) - 1u)) - 1u;
      const int64_t row = piece_row(T, idx);
      rw[j] = ((T.m_real >> j) & 1u) && row >= 0 && row < R.cap
                  ? (uint32_t)row : kNone;
    }
    if constexpr (kNat || kGen) wave_blocked_to_regrouped(sk, rw, dst, lane);
    else wave_to_striped(sk, rw, lane);
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) {
      const uint32_t wr = rw[j];
      if (wr == kNone) continue;
#pragma unroll
      for (int l = 0; l < MaxD; ++l)
        if (l < D)
          R.path[(int64_t)l * R.cap + wr] =
              (lv < D && l <= lv) ? p[j][l] : kNone;
      R.gpu[wr] = (uint8_t)(gk[j] >> 1);
      R.kind[wr] = (uint8_t)(gk[j] & 1u);
      R.first[wr] = src.first_of(rs[j]);
      if constexpr (kGen) {
        R.firstpos[wr] = id[j];
        own[level_key<MaxD>(p[j], gk[j], lv, D, M)] = wr;
      }
    }
  };
  if (first) {
    headers(T1, li, own_row, GR.own);
    if (kTwo) headers(T2, li2, own_row2, GR.own2);
  }
  auto cont_row = [&](uint32_t c, int64_t r) -> uint32_t {
    return c && r >= 1 && r - 1 < R.cap ? (uint32_t)(r - 1) : kNone;
  };
  if (!kGen && first && lane == 0) {
    if constexpr (kNat) {
      ovf.row[2 * w] = cont_row(T1.c0, T1.r0);
      ovf.row[2 * w + 1] = cont_row(T1.c1, T1.r1);
      if (kTwo) {
        ovf.row[2 * nwt + 2 * w] = cont_row(T2.c0, T2.r0);
        ovf.row[2 * nwt + 2 * w + 1] = cont_row(T2.c1, T2.r1);
      }
    } else {
      ovf.row[w] = cont_row(T1.c0, T1.r0);
      if (kTwo) ovf.row[nwt + w] = cont_row(T2.c0, T2.r0);
    }
  }
  // byte offsets of the striped items (sizes are below 2^29 here)
  uint32_t off[kAggIpt];
#pragma unroll
  for (int j = 0; j < kAggIpt; ++j) off[j] = rs[j] << 3;

  // piece values at the slots -> rows (and the overflow slots)
  auto store_pieces = [&](const LevelTile& T, int64_t obase, int f,
                          bool diff) {
    uint64_t* col = row_column(R, f);
    uint64_t* oslot = ovf.val + (int64_t)f * ovf.cap +
                      (kGen ? 0 : obase + (kNat ? 2 * w : w));
    wave_sync();
    for (uint32_t q = lane; q < T.NP; q += kWave) {
      uint64_t v = sv[q];
      if (diff && q > 0) v -= sv[q - 1];
      if constexpr (kGen) {
        const uint32_t r = s_row[wv][obase][q];
        if (!(r >> 31)) col[r] = v;
        else if (r != kNone) oslot[r & 0x7FFFFFFFu] = v;
        continue;
      }
      const int64_t row = piece_row(T, q);
      if (row < 0) {
        oslot[q >= T.NP0 ? 1 : 0] = v;
      } else if (row < R.cap) {
        col[row] = v;
      }
    }
    wave_sync();
  };
  auto put = [&](const uint32_t (&sl)[kAggIpt], const uint64_t (&x)[kAggIpt]) {
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) sv[sl[j]] = x[j];
  };
  const int64_t ob2 = kGen ? 1 : kNat ? 2 * nwt : nwt;   // (kGen: s_row's)
  auto do_sum = [&](const uint64_t (&v)[kAggIpt], int f) {
    uint64_t x[kAggIpt];
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) x[j] = v[j];
    blk64(x);
#pragma unroll
    for (int j = 1; j < kAggIpt; ++j) x[j] += x[j - 1];
    const uint64_t incl = wave_incl(x[kAggIpt - 1], OpAdd(), (uint64_t)0);
    const uint64_t carry = wave_shr1(0ull, incl);
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) x[j] += carry;
    put(slot, x);
    store_pieces(T1, 0, f, true);
    if (kTwo) {
      put(slot2, x);
      store_pieces(T2, ob2, f, true);
    }
  };
  auto seg_pass = [&](const LevelTile& T, const uint32_t (&sl)[kAggIpt],
                      const uint64_t (&xin)[kAggIpt], int64_t obase, int f,
                      auto cmb) {
    using C = decltype(cmb);
    uint64_t x[kAggIpt];
    uint64_t acc = xin[0];
    x[0] = acc;
#pragma unroll
    for (int j = 1; j < kAggIpt; ++j) {
      acc = ((T.m_head >> j) & 1u) ? xin[j] : cmb(acc, xin[j]);
      x[j] = acc;
    }
    const uint64_t incl = wave_seg_incl<C>(T.masks, acc);
    const uint64_t carry = wave_shr1(C::ident, incl);
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j)
      sv[sl[j]] = (uint32_t)j < T.before ? cmb(carry, x[j]) : x[j];
    store_pieces(T, obase, f, false);
  };
  auto do_seg = [&](const uint64_t (&v)[kAggIpt], int f, auto cmb) {
    uint64_t x[kAggIpt];
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j) x[j] = v[j];
    blk64(x);
    seg_pass(T1, slot, x, 0, f, cmb);
    if (kTwo) seg_pass(T2, slot2, x, ob2, f, cmb);
  };
  auto load = [&](const uint64_t* col, uint64_t (&v)[kAggIpt]) {
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j)
      v[j] = *(const uint64_t*)((const char*)col + off[j]);
  };

  if constexpr (kStaged) {
    uint64_t c[kRowCols][kAggIpt];
#pragma unroll
    for (int j = 0; j < kAggIpt; ++j)
#pragma unroll
      for (int q = 0; q < kRowCols / 2; ++q) {
        const ulonglong2 v = GR.rows[(int64_t)rs[j] * (kRowCols / 2) + q];
        c[2 * q][j] = v.x;
        c[2 * q + 1][j] = v.y;
      }
    if (first) {                   // start, end, gap, ovl
      uint64_t x[kAggIpt];
#pragma unroll
      for (int j = 0; j < kAggIpt; ++j)
        x[j] = (uint64_t)(lane * kAggIpt + j + 1);
      put(slot, x);
      store_pieces(T1, 0, 0, true);
      if (kTwo) {
        put(slot2, x);
        store_pieces(T2, ob2, 0, true);
      }
#pragma unroll
      for (int j = 0; j < kAggIpt; ++j) x[j] = c[1][j] - c[0][j];
      do_sum(x, 1);
      do_seg(c[0], 4, CMin());
      do_seg(c[1], 5, CMax());
      do_sum(c[2], 2);
      do_sum(c[3], 3);
    } else {
#pragma unroll
      for (int q = 0; q < kRowCols; ++q)
        if (q < GR.nc) do_sum(c[q], GR.c0 + q + 2);
    }
    return;
  }

  // this part's plain sums: is .. ns - 1 (the special fields, which come to
  // about kSpecial sums, are the first part's)
  int is = 0, ns = src.nsum();
  if constexpr (kSplit) {
    const int units = kSpecial + ns, P = (int)gridDim.y, q = (int)blockIdx.y;
    const int u0 = units * q / P - kSpecial;
    const int u1 = units * (q + 1) / P - kSpecial;
    is = u0 > 0 ? u0 : 0;
    ns = u1 > 0 ? u1 : 0;
  }
  // three plain-sum columns in flight: each is loaded three fields ahead of
  // its use (the first ones staggered between the special fields)
  uint64_t va[kAggIpt], vb[kAggIpt], vc[kAggIpt];
  if (kSplit && !first) {
    if (ns > is) load(src.sum_col(is), va);
    if (ns > is + 1) load(src.sum_col(is + 1), vb);
    if (ns > is + 2) load(src.sum_col(is + 2), vc);
  } else {
    uint64_t ts[kAggIpt], te[kAggIpt];
    load((const uint64_t*)src.start_col(), ts);
    load((const uint64_t*)src.end_col(), te);
    if (ns > 0) load(src.sum_col(0), va);
    if constexpr (Src::kRecords) {
      // n: the prefix of ones at a piece's last item is its position + 1
      uint64_t pos[kAggIpt];
#pragma unroll
      for (int j = 0; j < kAggIpt; ++j)
        pos[j] = (uint64_t)(lane * kAggIpt + j + 1);
      put(slot, pos);
      store_pieces(T1, 0, 0, true);
      if (kTwo) {
        put(slot2, pos);
        store_pieces(T2, ob2, 0, true);
      }
      uint64_t du[kAggIpt];
#pragma unroll
      for (int j = 0; j < kAggIpt; ++j) du[j] = te[j] - ts[j];
      if (ns > 1) load(src.sum_col(1), vb);
      do_sum(du, 1);
    } else {
      if (ns > 1) load(src.sum_col(1), vb);
    }
    do_seg(ts, 4, CMin());
    if (ns > 2) load(src.sum_col(2), vc);
    do_seg(te, 5, CMax());
  }
  for (int i = is; i < ns; i += 3) {
    do_sum(va, src.sum_dst(i));
    if (i + 3 < ns) load(src.sum_col(i + 3), va);
    if (i + 1 < ns) {
      do_sum(vb, src.sum_dst(i + 1));
      if (i + 4 < ns) load(src.sum_col(i + 4), vb);
    }
    if (i + 2 < ns) {
      do_sum(vc, src.sum_dst(i + 2));
      if (i + 5 < ns) load(src.sum_col(i + 5), vc);
    }
  }
}

// GPU rows from the level-0 rows (with no marker level, the GPU rows
// themselves): the level-0 rows of one (gpu, kind) are consecutive and
// ordered by (tmin, first), and every record is in exactly one of them.
// Block b sums the rows of the pair gpu * 2 + kind = b into slot b of
// `pair` (fields, then tmin, first and a presence flag); a single block
// then numbers the pairs present, writes the GPU rows and adds them up into
// the workload rows (one per kind present, kind 0 first).
constexpr int kPairW = kMaxFields + 3;

// First row in [a0, a1) whose pair is >= k, for every thread of the block:
// a search with kBlock probes per round.
__device__ inline int64_t block_pair_lower(const RowsDev& R, int64_t a0,
                                           int64_t a1, uint32_t k,
                                           uint32_t* s_cnt) {
  int64_t lo = a0, hi = a1;           // answer in [lo, hi]
  while (hi > lo) {
    const int64_t step = (hi - lo + kBlock - 1) / kBlock;
    const int64_t p = lo + (int64_t)threadIdx.x * step;
    const bool below =
        p < hi && (uint32_t)R.gpu[p] * 2u + R.kind[p] < k;
    const uint64_t m = __ballot(below);
    __syncthreads();
    if (lane_id() == 0) s_cnt[threadIdx.x / kWave] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t c = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) c += s_cnt[i];
    // probes 0 .. c - 1 are below k (rows are sorted by pair)
    if (c == 0) return lo;
    const int64_t nlo = lo + (int64_t)(c - 1) * step + 1;
    const int64_t nhi = lo + (int64_t)c * step;
    lo = nlo;
    hi = nhi < hi ? nhi : hi;
  }
  return lo;
}

__device__ inline void agg_gpu_sums(const int64_t* level_offset,
                                    const RowsDev& R, int nfields,
                                    uint64_t* pair) {
  __shared__ uint32_t s_cnt[kWavesPerBlock];
  __shared__ uint64_t s_f[kWavesPerBlock][kMaxFields];
  const uint32_t b = blockIdx.x;
  uint64_t* slot = pair + (int64_t)b * kPairW;
  int64_t a0 = level_offset[0], a1 = level_offset[1];
  if (a1 > R.cap) a1 = R.cap;
  if (a0 > a1) a0 = a1;
  const int64_t lo = block_pair_lower(R, a0, a1, b, s_cnt);
  const int64_t hi = block_pair_lower(R, lo, a1, b + 1, s_cnt);
  if (lo >= hi) {
    if (threadIdx.x == 0) slot[kMaxFields + 2] = 0;
    return;
  }
  uint64_t acc[kMaxFields];
#pragma unroll
  for (int f = 0; f < kMaxFields; ++f)
    acc[f] = f == 5 ? (uint64_t)kI64Min : 0ull;
  for (int64_t r = lo + threadIdx.x; r < hi; r += kBlock) {
#pragma unroll
    for (int f = 0; f < kMaxFields; ++f) {
      if (f == 4 || f >= nfields) continue;
      const uint64_t x = row_column(R, f)[r];
      acc[f] = f == 5 ? ((int64_t)x > (int64_t)acc[f] ? x : acc[f])
                      : acc[f] + x;
    }
  }
  // (lane moves without LDS; the fields that are there)
#pragma unroll
  for (int f = 0; f < kMaxFields; ++f) {
    if (f == 4 || f >= nfields) continue;
    const uint64_t v =
        f == 5 ? (uint64_t)lane63(wave_incl((int64_t)acc[f], OpMax(), kI64Min))
               : lane63(wave_incl(acc[f], OpAdd(), (uint64_t)0));
    if (lane_id() == 0) s_f[threadIdx.x / kWave][f] = v;
  }
  __syncthreads();
  const int f = (int)threadIdx.x;
  if (f < nfields && f != 4) {
    uint64_t t = s_f[0][f];
    for (int i = 1; i < kWavesPerBlock; ++i)
      t = f == 5 ? ((int64_t)s_f[i][f] > (int64_t)t ? s_f[i][f] : t)
                 : t + s_f[i][f];
    slot[f] = t;
  }
  if (f == 0) {
    // the pair's first row has the smallest (tmin, first)
    slot[4] = (uint64_t)R.tmin[lo];
    slot[kMaxFields] = (uint64_t)R.tmin[lo];
    slot[kMaxFields + 1] = R.first[lo];
    slot[kMaxFields + 2] = 1;
  }
}

// (one block of kBlock threads)
__device__ inline void agg_gpu_finish(const int64_t* level_offset, int D,
                                      const RowsDev& R, int nfields,
                                      int npairs, const uint64_t* pair) {
  __shared__ uint32_t s_rank[513];
  const int t = (int)threadIdx.x;
  {
    // two consecutive pairs a thread (at most 512)
    const int q0 = 2 * t;
    uint32_t p0 = 0, p1 = 0, tot;
    if (q0 < npairs)
      p0 = (uint32_t)pair[(int64_t)q0 * kPairW + kMaxFields + 2];
    if (q0 + 1 < npairs)
      p1 = (uint32_t)pair[(int64_t)(q0 + 1) * kPairW + kMaxFields + 2];
    const uint32_t pre = block_exclusive(p0 + p1, OpAdd(), 0u, &tot);
    s_rank[q0] = pre;
    s_rank[q0 + 1] = pre + p0;
    if (t == 0) s_rank[512] = tot;
  }
  __syncthreads();
  const int64_t g0 = level_offset[D];
  // GPU rows: one thread per (pair, field) of the pairs present
  for (int i = t; i < npairs * kPairW; i += kBlock) {
    const int q = i / kPairW, f = i % kPairW;
    const uint64_t* slot = pair + (int64_t)q * kPairW;
    if (!slot[kMaxFields + 2]) continue;
    const int64_t row = g0 + s_rank[q];
    if (row >= R.cap) continue;
    if (f < nfields) {
      row_column(R, f)[row] = slot[f];
    } else if (f == kMaxFields) {
      R.first[row] = (uint32_t)slot[kMaxFields + 1];
      R.gpu[row] = (uint8_t)(q >> 1);
      R.kind[row] = (uint8_t)(q & 1);
      for (int l = 0; l < D; ++l) R.path[(int64_t)l * R.cap + row] = kNone;
    }
  }
  // workload rows: kind 0 first when present
  const int64_t w0 = level_offset[D + 1], w1 = level_offset[D + 2];
  for (int i = t; i < 2 * kPairW; i += kBlock) {
    const uint32_t kd = (uint32_t)(i / kPairW);
    const int f = i % kPairW;
    bool any = false;
    uint64_t acc = f == 5 ? (uint64_t)kI64Min : 0ull;
    int64_t bt = kI64Max;
    uint32_t bf = kNone;
    for (int q = (int)kd; q < npairs; q += 2) {
      const uint64_t* slot = pair + (int64_t)q * kPairW;
      if (!slot[kMaxFields + 2]) continue;
      any = true;
      const uint64_t x = slot[f < kMaxFields ? f : 0];
      acc = f == 5 ? ((int64_t)x > (int64_t)acc ? x : acc) : acc + x;
      const int64_t tq = (int64_t)slot[kMaxFields];
      const uint32_t fq = (uint32_t)slot[kMaxFields + 1];
      if (tq < bt || (tq == bt && fq < bf)) {
        bt = tq;
        bf = fq;
      }
    }
    if (!any) continue;
    const int64_t w = w0 + (w1 - w0 == 2 ? (int64_t)kd : 0);
    if (w >= w1 || w >= R.cap) continue;
    if (f < nfields && f != 4) {
      row_column(R, f)[w] = acc;
    } else if (f == 4) {
      R.tmin[w] = bt;
    } else if (f == kMaxFields) {
      R.first[w] = bf;
      R.gpu[w] = 0xFF;
      R.kind[w] = (uint8_t)kd;
      for (int l = 0; l < D; ++l) R.path[(int64_t)l * R.cap + w] = kNone;
    }
  }
}

// GPU rows, then the workload rows by the last block.
__global__ __launch_bounds__(kBlock) void k_agg_gpu_rows(
    const int64_t* level_offset, int D, RowsDev R, int nfields, int npairs,
    uint64_t* pair, uint32_t* count) {
  agg_gpu_sums(level_offset, R, nfields, pair);
  if (last_block(count, gridDim.x))
    agg_gpu_finish(level_offset, D, R, nfields, npairs, pair);
}

// first record of a workload row: the smallest input index among the records
// (or GPU rows) whose start equals the row's tmin
template <typename Src>
__global__ __launch_bounds__(kBlock) void k_agg_workload_first(
    Src src, int D, int64_t M, const uint32_t* rowof, RowsDev R) {
  const int64_t cnt = src.count();
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= cnt) return;
  uint32_t r, p[8], g, kind, fpos;
  bool ok;
  src.load(i, r, ok, p, g, kind, fpos);
  if (!ok) return;
  const uint32_t row = rowof[kind];
  if ((int64_t)row >= R.cap) return;
  if ((int64_t)src.field(4, r) == R.tmin[row])
    atomicMin(&R.first[row], src.first_of(r));
}

// Entry e of [0, nslots), or of [0, *count) when nslots < 0; a slot holding
// kNone is empty.
__device__ inline void apply_overflow(const Overflow& ovf, RowsDev R,
                                      int nfields, int64_t nslots, int64_t e) {
  int64_t cnt = nslots >= 0 ? nslots : (int64_t)*ovf.count;
  if (cnt > ovf.cap) cnt = ovf.cap;
  if (e >= cnt) return;
  const uint32_t row = ovf.row[e];
  if (row == kNone || (int64_t)row >= R.cap) return;
  for (int f = 0; f < nfields; ++f)
    atomic_field(R, f, row, ovf.val[(int64_t)f * ovf.cap + e]);
}

__global__ __launch_bounds__(kBlock) void k_agg_apply_overflow(
    Overflow ovf, RowsDev R, int nfields, int64_t nslots) {
  apply_overflow(ovf, R, nfields, nslots,
                 (int64_t)blockIdx.x * kBlock + threadIdx.x);
}

// The heads pass over rows (its first `hblocks` blocks; it reads headers
// only) and beside it the finer levels' overflow slots (the blocks after
// them, null ovf.row: none).  The last heads block scans a table of at most
// kTailScan counts.
template <int MaxD>
__global__ __launch_bounds__(kBlock) void k_agg_heads_rows(
    FromRows src, uint32_t act, int lv0, int lv1, int D, int64_t M,
    int64_t nwt, uint32_t* tilecnt, uint32_t* tilebase, uint32_t* flags,
    uint32_t* status, uint32_t* count, uint32_t hblocks, Overflow ovf,
    RowsDev R, int nfields, int64_t nslots) {
  if (blockIdx.x >= hblocks) {
    apply_overflow(ovf, R, nfields, nslots,
                   (int64_t)(blockIdx.x - hblocks) * kBlock + threadIdx.x);
    return;
  }
  agg_heads<MaxD>(src, act, lv0, lv1, D, M, nwt, tilecnt, flags, status);
  if (!count || !last_block(count, hblocks)) return;
  block_scan_array(tilecnt, tilebase, (int64_t)(lv1 - lv0 + 1) * nwt);
}

// zero the sums of rows [level_offset[a], level_offset[b]) (atomic re-run)
__global__ __launch_bounds__(kBlock) void k_agg_zero_rows(
    const int64_t* level_offset, int a, int b, RowsDev R) {
  int64_t lo = level_offset[a], hi = level_offset[b];
  if (hi > R.cap) hi = R.cap;
  for (int64_t row = lo + (int64_t)blockIdx.x * kBlock + threadIdx.x; row < hi;
       row += (int64_t)gridDim.x * kBlock) {
    R.n[row] = 0;
    R.dur[row] = 0;
    R.gap[row] = 0;
    R.ovl[row] = 0;
    R.tmin[row] = kI64Max;
    R.tmax[row] = kI64Min;
    for (int q = 0; q < R.nc; ++q) R.ctr[(int64_t)q * R.cap + row] = 0;
  }
}

// ------------------------------------------------------- exact group ids
// Exact group ids, level by level from the outermost: the key of korder
// position p at marker level l is (its group id at level l - 1, or
// gpu * 2 + kind at l = 0) * (M + 2) + (its level-l marker, M + 1 for
// NONE), so that equal keys are equal paths; records left out by the filter
// get kfilt, above every key.  After a stable sort by key the group id of a
// position is the position of its group's first record.
__global__ __launch_bounds__(kBlock) void k_xk_keys(RecSrc S, int l,
                                                    const uint32_t* gprev,
                                                    uint64_t kfilt,
                                                    uint64_t* key,
                                                    uint32_t* val) {
  const int64_t pos = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (pos >= S.n) return;
  const uint32_t r = S.korder[pos];
  uint64_t k = kfilt;
  if (rec_pass(S, r)) {
    const uint64_t parent =
        l == 0 ? (uint64_t)S.gpu[r] * 2u + (uint64_t)kind_of(S.cls[r])
               : (uint64_t)gprev[pos];
    const uint32_t m = S.idx[(int64_t)l * S.n + r];
    const uint64_t mi = m == kNone ? (uint64_t)S.M + 1
                                   : ((int64_t)m >= S.M ? (uint64_t)S.M : m);
    k = parent * ((uint64_t)S.M + 2) + mi;
  }
  key[pos] = k;
  val[pos] = (uint32_t)pos;
}

__global__ __launch_bounds__(kBlock) void k_xk_heads(int64_t n,
                                                     const uint64_t* skey,
                                                     uint32_t* head) {
  const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (q < n) head[q] = (q == 0 || skey[q] != skey[q - 1]) ? 1u : 0u;
}

// first[run] = position of the run's first item (the smallest: the sort is
// stable over ascending positions)
__global__ __launch_bounds__(kBlock) void k_xk_first(int64_t n,
                                                     const uint32_t* head,
                                                     const uint32_t* runx,
                                                     const uint32_t* sval,
                                                     uint32_t* first) {
  const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (q < n && head[q]) first[runx[q]] = sval[q];
}

__global__ __launch_bounds__(kBlock) void k_xk_assign(
    int64_t n, const uint64_t* skey, uint64_t kfilt, const uint32_t* head,
    const uint32_t* runx, const uint32_t* sval, const uint32_t* first,
    uint32_t* gid) {
  const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (q >= n) return;
  gid[sval[q]] = skey[q] == kfilt ? kNone : first[runx[q] + head[q] - 1u];
}

__global__ void k_fill_u32_many(uint32_t** p, const int64_t* counts, int L,
                                uint32_t act) {
  const int li = blockIdx.y;
  if (li >= L || !((act >> li) & 1u)) return;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
       i < counts[li]; i += (int64_t)gridDim.x * blockDim.x)
    p[li][i] = 0xFFFFFFFFu;
}

// Counters of finished blocks (last_block), one per launch of a call that
// uses one: the heads passes, the GPU rows, the row passes.
constexpr int kDoneHeads = 0, kDoneHeads2 = 1, kDoneGpu = 2, kDoneRows = 3,
              kDone = kDoneRows + kMaxLevels;

// flags, the counters of finished blocks and the GPUs' first positions
__global__ void k_nat_init(uint32_t* flags, uint32_t* flags2, uint32_t* done,
                           uint32_t* gs, int G) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < 3) flags[i] = flags2[i] = 0;
  if (i < kDone) done[i] = 0;
  if (i < G) gs[i] = kNone;
}

__global__ void k_zero_u32(uint32_t* p, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------------------
// words read back by the host: flags, level offsets, interior pieces
constexpr int kStageWords = 3 + kMaxLevels + 1 + kMaxLevels;
static_assert(kStageWords * sizeof(int64_t) <= kReadBackMax, "one read-back");

struct AggLayout {
  int L;
  int64_t ntiles;
  uint32_t* own[kMaxLevels];
  uint32_t* rowof[kMaxLevels];
  int64_t ks[kMaxLevels];
  uint32_t** own_tab;     // device copies of the pointer tables
  uint32_t** rowof_tab;
  int64_t* ks_dev;
  uint32_t* tilecnt;
  uint32_t* tilebase;
  uint32_t* scantmp;
  uint32_t* total;
  uint32_t* firstpos;
  uint32_t* ovf_count;    // [2]: count, lost
  uint32_t* ovf_row;
  uint64_t* ovf_val;
  int64_t ovf_cap;
  // fast path: head counts per wave tile of kWaveTile items
  int64_t ntiles_h;
  uint32_t* htc;          // [L][ntiles_h]
  uint32_t* htb;
  uint32_t* hscan;
  uint32_t* htotal;
  uint32_t* hflags;       // [0] keys not increasing, [1] kinds present,
                          // [2] input order unfit for the natural tiles
  uint32_t* htc2;         // one or two levels over rows
  uint32_t* htb2;
  uint32_t* hflags2;
  uint32_t* done;         // [kDone] counters of finished blocks
  // natural tiles
  int G;
  int64_t nstride;        // 2 * (natural tiles + G): counts per level
  uint32_t* ntc;          // [L][nstride]
  uint32_t* ntb;
  uint32_t* nscan;
  int64_t lps;            // ntiles_h rounded up to kLpIpt
  int32_t* lpraw;         // [2][lps]
  int32_t* lp;
  uint8_t* tg;            // [ntiles_h + G]
  uint64_t* pair;         // [2G][kPairW] GPU row sums
  int64_t* stage;         // flags and level offsets for the host
  uint32_t* gs;           // [G]
  uint32_t* ge;
  uint32_t* gtb;          // [G + 1]
  // exact group ids (markers not nested)
  uint32_t* gk;           // [D][n]
  uint32_t* xflag;
  uint64_t* xskey;        // sorted keys
  uint32_t* xsval;        // positions in key order
  uint32_t* xhead;
  uint32_t* xrunx;
  uint32_t* xfirst;
  uint32_t* xtot;
  uint32_t* xscan;        // scan temporaries over n items
  ClassSortLayout xsort;
  uint32_t* ipath;        // [D][n] general-path items by korder position
  uint16_t* igk;          // [n]
  // records in no order, null below kStageMin of them
  char* srow;             // a row per record
  uint32_t* slots;        // [2 * tiles] first overflow slot of either level
  // groups of several runs
  uint8_t* omask;         // [L][mstride] owners of every lane
  int64_t mstride;        // 64 * (natural tiles + G)
  uint32_t* interior;     // [kMaxLevels] and a counter of finished blocks
};

static AggLayout agg_layout(Scratch& sc, int64_t n, int D, int64_t M,
                            int64_t cap, uint32_t act, int G) {
  AggLayout L;
  L.L = D + 2;
  L.ntiles = ceil_div(n, kAggTile);
  for (int li = 0; li < L.L; ++li) {
    // (exact group ids at the marker levels are korder positions < n)
    int64_t ks = key_space(li, D, M);
    if (li < D && n > ks) ks = n;
    L.ks[li] = ((act >> li) & 1u) ? ks : 1;
    L.own[li] = sc.take<uint32_t>(L.ks[li]);
  }
  L.own_tab = sc.take<uint32_t*>(kMaxLevels);
  L.rowof_tab = sc.take<uint32_t*>(kMaxLevels);
  L.ks_dev = sc.take<int64_t>(kMaxLevels);
  L.firstpos = sc.take<uint32_t>(cap);
  L.ntiles_h = ceil_div(n, kWaveTile);
  L.nstride = 2 * (L.ntiles_h + G);
  L.ovf_cap = n / 64 > 65536 ? n / 64 : 65536;
  if (L.ovf_cap < 2 * L.nstride) L.ovf_cap = 2 * L.nstride;
  L.ovf_count = sc.take<uint32_t>(2);
  L.ovf_row = sc.take<uint32_t>(L.ovf_cap);
  L.ovf_val = sc.take<uint64_t>((int64_t)kMaxFields * L.ovf_cap);
  L.htc = sc.take<uint32_t>((int64_t)L.L * L.ntiles_h);
  L.htb = sc.take<uint32_t>((int64_t)L.L * L.ntiles_h);
  L.hscan = sc.take<uint32_t>(scan_scratch_elems((int64_t)L.L * L.ntiles_h));
  L.htotal = sc.take<uint32_t>(2);
  L.hflags = sc.take<uint32_t>(3);
  L.htc2 = sc.take<uint32_t>(2 * L.ntiles_h);
  L.htb2 = sc.take<uint32_t>(2 * L.ntiles_h);
  L.hflags2 = sc.take<uint32_t>(3);
  L.done = sc.take<uint32_t>(kDone);
  L.G = G;
  L.ntc = sc.take<uint32_t>((int64_t)L.L * L.nstride);
  L.ntb = sc.take<uint32_t>((int64_t)L.L * L.nstride);
  L.nscan = sc.take<uint32_t>(scan_scratch_elems((int64_t)L.L * L.nstride));
  L.lps = ceil_div(L.ntiles_h, (int64_t)kLpIpt) * kLpIpt;
  L.lpraw = sc.take<int32_t>(2 * L.lps);
  L.lp = sc.take<int32_t>(2 * L.lps);
  L.tg = sc.take<uint8_t>(L.ntiles_h + G);
  L.pair = sc.take<uint64_t>((int64_t)2 * G * kPairW);
  L.stage = sc.take<int64_t>(kStageWords);
  L.gs = sc.take<uint32_t>(G);
  L.ge = sc.take<uint32_t>(G);
  L.gtb = sc.take<uint32_t>(G + 1);
  L.xflag = sc.take<uint32_t>(1);
  // the element-wise path's own, and in the same space what only the tiles
  // of groups of several runs use
  Scratch gen = sc;
  for (int li = 0; li < L.L; ++li) L.rowof[li] = sc.take<uint32_t>(L.ks[li]);
  L.tilecnt = sc.take<uint32_t>((int64_t)L.L * L.ntiles);
  L.tilebase = sc.take<uint32_t>((int64_t)L.L * L.ntiles);
  L.scantmp = sc.take<uint32_t>(scan_scratch_elems((int64_t)L.L * L.ntiles));
  L.total = sc.take<uint32_t>(1);
  L.gk = sc.take<uint32_t>((int64_t)(D > 0 ? D : 1) * n);
  L.xskey = sc.take<uint64_t>(n);
  L.xsval = sc.take<uint32_t>(n);
  L.xhead = sc.take<uint32_t>(n);
  L.xrunx = sc.take<uint32_t>(n);
  L.xfirst = sc.take<uint32_t>(n);
  L.xtot = sc.take<uint32_t>(1);
  L.xscan = sc.take<uint32_t>(scan_scratch_elems(n));
  L.xsort = class_sort_layout(sc, n, 256);
  L.interior = gen.take<uint32_t>(kMaxLevels + 1);
  L.mstride = (int64_t)kWave * (L.ntiles_h + G);
  L.omask = gen.take<uint8_t>((int64_t)L.L * L.mstride);
  L.srow = nullptr;
  L.slots = nullptr;
  if (n >= kStageMin) {
    // (items, then a group of columns)
    static_assert(kRowCols * sizeof(uint64_t) <= 32, "rows of 32 bytes");
    L.srow = gen.take<char>((D < 8 ? 32 : 64) * n);
    L.slots = gen.take<uint32_t>(2 * L.ntiles_h);
  }
  if (gen.used > sc.used) sc.used = gen.used;
  L.ipath = sc.take<uint32_t>((int64_t)(D > 0 ? D : 1) * n);
  L.igk = sc.take<uint16_t>(n);
  return L;
}

static int bitlen_of(uint64_t x) {
  int b = 0;
  while (x) { ++b; x >>= 1; }
  return b;
}

// Exact group ids of the marker levels 0 .. lmax into L.gk (see k_xk_keys).
static int exact_group_ids(const AggLayout& L, const RecSrc& S, int lmax,
                           hipStream_t s) {
  const int64_t n = S.n;
  const dim3 g = grid_for(n, kBlock);
  for (int l = 0; l <= lmax; ++l) {
    // keys below kfilt = (parents) * (M + 2); parents: 512 (gpu, kind) ids
    // at level 0, positions below n after
    const unsigned __int128 kf =
        (unsigned __int128)(l == 0 ? 512u : (uint64_t)n) *
        (unsigned __int128)((uint64_t)S.M + 2);
    if (kf >> 63) return CHOPPER_EINVAL;
    const uint64_t kfilt = (uint64_t)kf;
    CHOPPER_HIP(launch("agg_exact_keys", k_xk_keys, g, dim3(kBlock), s, S, l,
                       (const uint32_t*)(l > 0 ? L.gk + (int64_t)(l - 1) * n
                                               : nullptr),
                       kfilt, L.xsort.key0, L.xsort.val0));
    int rc = radix_sort_pairs(L.xsort, bitlen_of(kfilt), L.xsval, L.xskey,
                              s);
    if (rc != CHOPPER_OK) return rc;
    CHOPPER_HIP(launch("agg_exact_keys", k_xk_heads, g, dim3(kBlock), s, n,
                       (const uint64_t*)L.xskey, L.xhead));
    CHOPPER_HIP(exclusive_scan<uint32_t>(L.xhead, L.xrunx, n, L.xscan,
                                         L.xtot, s));
    CHOPPER_HIP(launch("agg_exact_keys", k_xk_first, g, dim3(kBlock), s, n,
                       (const uint32_t*)L.xhead, (const uint32_t*)L.xrunx,
                       (const uint32_t*)L.xsval, L.xfirst));
    CHOPPER_HIP(launch("agg_exact_keys", k_xk_assign, g, dim3(kBlock), s, n,
                       (const uint64_t*)L.xskey, kfilt,
                       (const uint32_t*)L.xhead, (const uint32_t*)L.xrunx,
                       (const uint32_t*)L.xsval, (const uint32_t*)L.xfirst,
                       L.gk + (int64_t)l * n));
  }
  return CHOPPER_OK;
}

}  // namespace chopper

using namespace chopper;

// Parts of the reduction's fields.  A wave takes about 1 us a field, and the
// chip holds 3,072 of them, so that below as many tiles most of it would
// idle: 262 tiles of 134,000 rows with 16 counters 43 to 23 us, the 480 of
// 245,760 records without counters 27 to 24.  Above, finding the pieces again
// costs what the fuller chip gives (4,808 tiles in two parts: no change, in
// three 5 % slower).
static unsigned reduce_parts(int64_t tiles, int nsum) {
  const int64_t most = (kSpecial + nsum) / 3;
  int64_t p = ceil_div(kReduceWaves, tiles > 0 ? tiles : 1);
  if (p > most) p = most;
  return (unsigned)(p > 0 ? p : 1);
}

// Geometry of the natural tiles (flag 2 set when the order does not qualify).
static int nat_geometry(const AggLayout& L, const RecSrc& S, hipStream_t s) {
  const int64_t Th = L.ntiles_h;
  CHOPPER_HIP(launch("agg_nat_init", k_nat_init, dim3(1), dim3(kBlock), s,
                     L.hflags, L.hflags2, L.done, L.gs, L.G));
  CHOPPER_HIP(launch("agg_nat_pre", k_nat_pre,
                     dim3((unsigned)ceil_div(Th, (int64_t)kWavesPerBlock)),
                     dim3(kBlock), s, S.n, L.G, S.gpu, S.cls, S.start, Th,
                     L.lps, L.lpraw, L.gs, L.hflags + 2));
  CHOPPER_HIP(launch("agg_nat_tiles", k_nat_tiles,
                     dim3((unsigned)(1 + ceil_div(Th, kLpSpan))), dim3(1024), s,
                     S.n, L.G, Th, L.lps, (const int32_t*)L.lpraw, L.lp,
                     (const uint32_t*)L.gs, L.ge, L.gtb, L.tg,
                     (const uint32_t*)(L.hflags + 2)));
  return CHOPPER_OK;
}

// GPU rows and the workload rows from the level-0 rows.
static int gpu_rows(const AggLayout& L, const RowsDev& R, int D, int nfields,
                    const int64_t* level_offset, hipStream_t s) {
  CHOPPER_HIP(launch("agg_gpu_rows", k_agg_gpu_rows,
                     dim3((unsigned)(2 * L.G)), dim3(kBlock), s, level_offset,
                     D, R, nfields, 2 * L.G, L.pair, L.done + kDoneGpu));
  return CHOPPER_OK;
}

// Fast path over all requested levels (MaxD >= depth); returns 1 when the
// groups are not runs and the general path must be used.  The natural tiles
// are tried first; when the input order does not qualify, the korder tiles
// count the heads again.
template <int kMD>
static int agg_fast(const AggLayout& L, const RecSrc& S, const RowsDev& R,
                    const Overflow& ovf, int64_t T, int Lv, uint32_t act,
                    int D, int64_t M, int nfields, chopper_rows* rows,
                    int level, bool want_workload, uint32_t* status,
                    hipEvent_t ready, hipStream_t s, int* nat_out,
                    bool* conflict) {
  int rc = CHOPPER_OK;
  const int64_t Th = L.ntiles_h;
  const int G = L.G;
  const int64_t NW = Th + G;          // natural tile slots
  FromRecords fr{S};
  const NatGeom N{L.gtb, L.tg, L.gs, L.ge, L.lp, L.hflags + 2, Th, L.lps, G};
  const NatGeom none{};
  // the records reduction on the natural tiles: level li and, with `two`,
  // li - 1
  auto nat_records = [&](const NatGeom& NG, int li, bool two) -> int {
    const uint32_t* tb = L.ntb + (int64_t)li * L.nstride;
    const unsigned parts = reduce_parts(NW, fr.S.nc + 2);
    const dim3 grid((unsigned)ceil_div(NW, (int64_t)kWavesPerBlock), parts);
    if (two)
      CHOPPER_HIP(launch("agg_fast_reduce_records",
                         parts > 1 ? k_agg_fast_reduce<kMD, FromRecords, true, true, false, true>
                                   : k_agg_fast_reduce<kMD, FromRecords, true, true, false, false>,
                         grid, dim3(kBlock), s, fr, NG, li, D, M, tb,
                         (const uint32_t*)(tb - L.nstride),
                         (const int64_t*)nullptr, R, ovf, NW, GenRed{}));
    else
      CHOPPER_HIP(launch("agg_fast_reduce_records",
                         parts > 1 ? k_agg_fast_reduce<kMD, FromRecords, false, true, false, true>
                                   : k_agg_fast_reduce<kMD, FromRecords, false, true, false, false>,
                         grid, dim3(kBlock), s, fr, NG, li, D, M, tb,
                         (const uint32_t*)nullptr, (const int64_t*)nullptr,
                         R, ovf, NW, GenRed{}));
    return CHOPPER_OK;
  };
  // the level the records reduce to (with li0 - 1 when two0)
  const int li0 = level == CHOPPER_LEVEL_ALL
                      ? (D > 0 ? D - 1 : D)
                      : (level == CHOPPER_LEVEL_GPU ? D : level);
  const bool two0 = level == CHOPPER_LEVEL_ALL && D >= 2;
  bool spec = false;   // the natural-tile records reduction is queued
  // the fast-path flags and the level offsets (row counts per level size
  // the launches of the coarser levels); with `speculate` the natural-tile
  // records reduction, which needs none of them, is queued before the wait
  // and exits on the device unless the flags let it run
  uint32_t hf[3] = {1u, 0u, 1u};
  int64_t lo_h[kMaxLevels + 1];
  // opened before the kernel that stores the words, finished here
  ReadBack rb;
  auto stage_of = [&](int64_t stride, uint32_t* tc, uint32_t* tb, bool isnat,
                      int done) -> StageOut {
    StageOut O;
    O.L = Lv;
    O.stride = stride;
    O.tilecnt = tc;
    O.tilebase = tb;
    O.total = L.htotal;
    O.interior = nullptr;
    O.nat = isnat;
    O.workload = want_workload;
    O.cap = rows->cap;
    O.level_offset = rows->level_offset;
    O.stage = L.stage;
    O.host = read_back_open(sizeof(int64_t) * (size_t)(3 + Lv + 1), &rb);
    O.status = status;
    O.count = (int64_t)Lv * stride <= kTailScan ? L.done + done : nullptr;
    return O;
  };
  auto scan_of = [&](const StageOut& O, uint32_t* tmp) -> int {
    if (O.count) return CHOPPER_OK;       // done by the heads pass
    CHOPPER_HIP(exclusive_scan<uint32_t>(O.tilecnt, O.tilebase,
                                         (int64_t)Lv * O.stride, tmp, O.total,
                                         s));
    CHOPPER_HIP(launch("agg_offsets", k_agg_offsets, dim3(1), dim3(64), s, O,
                       (const uint32_t*)L.hflags));
    return CHOPPER_OK;
  };
  auto fetch_stage = [&](bool speculate) -> int {
    int64_t st[3 + kMaxLevels + 1];
    CHOPPER_HIP(read_back_close(L.stage, s, &rb));
    // gap and ovl are read from here on: the caller's event first (the
    // read-back above does not wait for it)
    if (ready) CHOPPER_HIP(hipStreamWaitEvent(s, ready, 0));
    if (speculate) {
      NatGeom NS = N;
      NS.fflags = L.hflags;
      const int r = nat_records(NS, li0, two0);
      if (r != CHOPPER_OK) return r;
      spec = true;
    }
    CHOPPER_HIP(read_back_finish(&rb, st));
    for (int i = 0; i < 3; ++i) hf[i] = (uint32_t)st[i];
    for (int i = 0; i <= Lv; ++i) lo_h[i] = st[3 + i];
    return CHOPPER_OK;
  };
  rc = nat_geometry(L, S, s);
  if (rc != CHOPPER_OK) return rc;
  {
    const StageOut O = stage_of(L.nstride, L.ntc, L.ntb, true, kDoneHeads);
    CHOPPER_HIP(launch("agg_heads_nat", k_agg_heads_nat<kMD>,
                       dim3((unsigned)ceil_div(NW, (int64_t)kWavesPerBlock)),
                       dim3(kBlock), s, S, N, act, 0, Lv - 1, D, M, L.nstride,
                       L.ntc, L.hflags, status, O));
    rc = scan_of(O, L.nscan);
    if (rc != CHOPPER_OK) return rc;
  }
  rc = fetch_stage(true);
  if (rc != CHOPPER_OK) return rc;
  const bool nat = hf[2] == 0;
  *nat_out = nat ? 1 : 0;
  if (!nat) {
    CHOPPER_HIP(launch("agg_zero", k_zero_u32, dim3(1), dim3(64), s,
                       L.hflags, 3));
    const StageOut O = stage_of(Th, L.htc, L.htb, false, kDoneHeads2);
    CHOPPER_HIP(launch("agg_heads_records", k_agg_heads<kMD>,
                       dim3((unsigned)ceil_div(Th, (int64_t)kWavesPerBlock)),
                       dim3(kBlock), s, fr, act, 0, Lv - 1, D, M, Th, L.htc,
                       L.hflags, status, O));
    rc = scan_of(O, L.hscan);
    if (rc != CHOPPER_OK) return rc;
    rc = fetch_stage(false);
    if (rc != CHOPPER_OK) return rc;
  }
  auto level_rows = [&](int li) -> int64_t {
    int64_t a = lo_h[li], b = lo_h[li + 1];
    if (b > rows->cap) b = rows->cap;
    return b > a ? b - a : 0;
  };
  if (hf[0] & 2u) *conflict = true;
  if (hf[0] != 0) return 1;
  // overflow slots of the pass before, applied beside the next heads pass
  // over rows (which reads headers only) or, after the last pass, alone
  int64_t slots = 0;
  auto apply = [&]() -> int {
    if (slots == 0) return CHOPPER_OK;
    CHOPPER_HIP(launch("agg_apply_overflow", k_agg_apply_overflow,
                       grid_for(slots, kBlock), dim3(kBlock), s, ovf, R,
                       nfields, slots));
    slots = 0;
    return CHOPPER_OK;
  };
  // finer < 0: from the records (two levels, li and li - 1, when `two`)
  auto fast_level = [&](int li, int finer, bool two) -> int {
    if (finer < 0) {
      if (nat) {
        // (queued before the flags were read, when they allowed it)
        if (!(spec && li == li0 && two == two0)) {
          const int r = nat_records(N, li, two);
          if (r != CHOPPER_OK) return r;
        }
        slots = (two ? 4 : 2) * NW;
      } else {
        const uint32_t* tb = L.htb + (int64_t)li * Th;
        const unsigned parts = reduce_parts(Th, fr.S.nc + 2);
        if (two)
          CHOPPER_HIP(launch("agg_fast_reduce_records",
                             parts > 1 ? k_agg_fast_reduce<kMD, FromRecords, true, false, false, true>
                                       : k_agg_fast_reduce<kMD, FromRecords, true, false, false, false>,
                             dim3((unsigned)T, parts),
                             dim3(kBlock), s, fr, none, li,
                             D, M, tb, (const uint32_t*)(tb - Th),
                             (const int64_t*)nullptr, R, ovf, Th, GenRed{}));
        else
          CHOPPER_HIP(launch("agg_fast_reduce_records",
                             parts > 1 ? k_agg_fast_reduce<kMD, FromRecords, false, false, false, true>
                                       : k_agg_fast_reduce<kMD, FromRecords, false, false, false, false>,
                             dim3((unsigned)T, parts),
                             dim3(kBlock), s, fr, none, li,
                             D, M, tb, (const uint32_t*)nullptr,
                             (const int64_t*)nullptr, R, ovf, Th, GenRed{}));
        slots = two ? 2 * Th : Th;
      }
    } else {
      // launches sized by the finer level's row count; with `two` also the
      // level li - 1 (heads of li - 1 first in the table, then li)
      const int64_t cnt = level_rows(finer);
      if (cnt == 0) return apply();
      const int64_t nw = ceil_div(cnt, (int64_t)kWaveTile);
      const unsigned gr = (unsigned)ceil_div(nw, (int64_t)kWavesPerBlock);
      FromRows src{R, M, rows->level_offset, finer};
      const int lv0 = two ? li - 1 : li;
      const uint32_t lact = two ? (3u << (li - 1)) : (1u << li);
      const int64_t tab = (two ? 2 : 1) * nw;
      uint32_t* done = tab <= kTailScan ? L.done + kDoneRows + li : nullptr;
      CHOPPER_HIP(launch("agg_heads_rows", k_agg_heads_rows<kMD>,
                         dim3(gr + (unsigned)ceil_div(slots, (int64_t)kBlock)),
                         dim3(kBlock), s, src, lact, lv0, li, D, M, nw,
                         L.htc2, L.htb2, L.hflags2, status, done, gr, ovf, R,
                         nfields, slots));
      if (!done)
        CHOPPER_HIP(exclusive_scan<uint32_t>(L.htc2, L.htb2, tab, L.hscan,
                                             L.htotal + 1, s));
      const int64_t* r0 = rows->level_offset + li;
      const unsigned parts = reduce_parts(nw, R.nc + 4);
      if (two)
        CHOPPER_HIP(launch("agg_fast_reduce_rows",
                           parts > 1 ? k_agg_fast_reduce<kMD, FromRows, true, false, false, true>
                                     : k_agg_fast_reduce<kMD, FromRows, true, false, false, false>,
                           dim3(gr, parts), dim3(kBlock), s,
                           src, none, li, D, M,
                           (const uint32_t*)(L.htb2 + nw),
                           (const uint32_t*)L.htb2, r0, R, ovf, nw,
                           GenRed{}));
      else
        CHOPPER_HIP(launch("agg_fast_reduce_rows",
                           parts > 1 ? k_agg_fast_reduce<kMD, FromRows, false, false, false, true>
                                     : k_agg_fast_reduce<kMD, FromRows, false, false, false, false>,
                           dim3(gr, parts), dim3(kBlock), s,
                           src, none, li, D, M,
                           (const uint32_t*)L.htb2, (const uint32_t*)nullptr,
                           r0, R, ovf, nw, GenRed{}));
      slots = tab;
    }
    return CHOPPER_OK;
  };
  if (level == CHOPPER_LEVEL_ALL) {
    // the records give the two finest levels, coarser marker levels come
    // in pairs from the rows of the level below, the GPU rows from the
    // level-0 rows
    const bool two = D >= 2;
    rc = fast_level(D > 0 ? D - 1 : D, -1, two);
    if (rc != CHOPPER_OK) return rc;
    for (int li = D - (two ? 3 : 2); li >= 0; li -= 2) {
      rc = fast_level(li, li + 1, li >= 1);
      if (rc != CHOPPER_OK) return rc;
    }
    rc = apply();
    if (rc != CHOPPER_OK) return rc;
    rc = gpu_rows(L, R, D, nfields, rows->level_offset, s);
    if (rc != CHOPPER_OK) return rc;
  } else {
    rc = fast_level(level == CHOPPER_LEVEL_GPU ? D : level, -1, false);
    if (rc != CHOPPER_OK) return rc;
    rc = apply();
    if (rc != CHOPPER_OK) return rc;
  }
  return CHOPPER_OK;
}

// Groups of several runs (k_gen_elect above) over all requested levels.
// nat: 1 natural tiles, 0 korder tiles, -1 not known yet (the natural
// geometry is made here, and the korder tiles taken when the order does not
// qualify).  Returns 1 when the call must take the element-wise path: an
// item whose marker is out of range, more pieces to add than the overflow
// list holds, or (with *conflict set) markers that are not nested.
template <int kMD, bool kNat>
static int agg_gen_tiles(const AggLayout& L, RecSrc S, const RowsDev& R,
                         const Overflow& ovf, int Lv, uint32_t act, int D,
                         int64_t M, int nfields, chopper_rows* rows, int level,
                         bool want_workload, uint32_t* status,
                         hipEvent_t ready, hipStream_t s, bool* conflict,
                         bool* bad_order) {
  const int64_t Th = L.ntiles_h;
  const int64_t nwt = kNat ? Th + L.G : Th;
  const int64_t stride = kNat ? L.nstride : Th;
  uint32_t* tc = kNat ? L.ntc : L.htc;
  uint32_t* tb = kNat ? L.ntb : L.htb;
  const NatGeom N{L.gtb, L.tg, L.gs, L.ge, L.lp, L.hflags + 2, Th, L.lps, L.G};
  const dim3 grid((unsigned)ceil_div(nwt, (int64_t)kWavesPerBlock));
  GenTab tab;
  int64_t maxks = 1;
  for (int li = 0; li < kMaxLevels; ++li) {
    tab.own[li] = li < Lv ? L.own[li] : nullptr;
    tab.ks[li] = li < Lv && ((act >> li) & 1u) ? key_space(li, D, M) : 0;
    if (tab.ks[li] > maxks) maxks = tab.ks[li];
  }
  // one table entry in sixteen bytes a thread, at most 2,048 blocks a level
  unsigned fx = (unsigned)ceil_div(maxks, (int64_t)4 * kBlock);
  if (fx > 2048) fx = 2048;
  FromRecords fr{S};
  int64_t st[kStageWords];
  bool far = false;            // records in no order: through rows
  if (!kNat) {
    const dim3 gi = grid_for(S.n, kBlock);
    if (L.srow) {
      uint32_t jumps = 0;
      CHOPPER_HIP(launch("agg_stage", k_sample_jumps, dim3(1), dim3(kBlock), s,
                         S.korder, S.n, L.xflag));
      CHOPPER_HIP(read_back(L.xflag, &jumps, sizeof(jumps), s));
      far = jumps > kBlock / 2;
    }
    uint4* rows4 = reinterpret_cast<uint4*>(L.srow);
    if (far && D < 8) {
      CHOPPER_HIP(launch("agg_stage", k_stage_items<8>, gi, dim3(kBlock), s, S,
                         rows4));
      CHOPPER_HIP(launch("agg_stage", k_unstage_items<8>, gi, dim3(kBlock), s,
                         S.korder, S.n, D, (const uint4*)rows4, L.ipath,
                         L.igk));
    } else if (far) {
      CHOPPER_HIP(launch("agg_stage", k_stage_items<16>, gi, dim3(kBlock), s,
                         S, rows4));
      CHOPPER_HIP(launch("agg_stage", k_unstage_items<16>, gi, dim3(kBlock),
                         s, S.korder, S.n, D, (const uint4*)rows4, L.ipath,
                         L.igk));
    } else {
      CHOPPER_HIP(launch("agg_items", k_agg_items, gi, dim3(kBlock), s, S,
                         L.ipath, L.igk));
    }
    fr.S.ipath = L.ipath;
    fr.S.igk = L.igk;
  }
  CHOPPER_HIP(launch("agg_gen_fill", k_gen_fill, dim3(fx, (unsigned)(D + 1)),
                     dim3(kBlock), s, tab, act, L.hflags, L.interior,
                     L.ovf_count));
  CHOPPER_HIP(launch("agg_gen_elect", k_gen_elect<kMD, kNat>, grid,
                     dim3(kBlock), s, fr, N, act, D, M, nwt, tab, L.hflags));
  ReadBack rb;
  StageOut O;
  O.L = Lv;
  O.stride = stride;
  O.tilecnt = tc;
  O.tilebase = tb;
  O.total = L.htotal;
  O.interior = L.interior;
  O.nat = kNat;
  O.workload = want_workload;
  O.cap = rows->cap;
  O.level_offset = rows->level_offset;
  O.stage = L.stage;
  O.host = read_back_open(sizeof(int64_t) * (size_t)(3 + Lv + 1 + Lv), &rb);
  O.status = status;
  O.count = (int64_t)Lv * stride <= kTailScan ? L.interior + kMaxLevels
                                              : nullptr;
  CHOPPER_HIP(launch("agg_gen_count", k_gen_count<kMD, kNat>, grid,
                     dim3(kBlock), s, fr, N, act, 0, Lv - 1, D, M, nwt,
                     stride, tab, tc, L.omask, L.mstride, L.hflags,
                     L.interior, status, O));
  if (!O.count) {
    CHOPPER_HIP(exclusive_scan<uint32_t>(tc, tb, (int64_t)Lv * stride,
                                         kNat ? L.nscan : L.hscan,
                                         L.htotal, s));
    CHOPPER_HIP(launch("agg_offsets", k_agg_offsets, dim3(1), dim3(64), s,
                       O, (const uint32_t*)L.hflags));
  }
  CHOPPER_HIP(read_back_close(L.stage, s, &rb));
  if (ready) CHOPPER_HIP(hipStreamWaitEvent(s, ready, 0));
  CHOPPER_HIP(read_back_finish(&rb, st));
  if (kNat && st[2] != 0) {
    *bad_order = true;
    return 1;
  }
  const int64_t* lo_h = st + 3;
  const int64_t* inner = st + 3 + Lv + 1;
  if (st[0] & 2) *conflict = true;
  if (st[0] != 0) return 1;
  if (lo_h[Lv] > rows->cap) return CHOPPER_OK;     // (ROWS_OVERFLOW is set)
  // the levels in the order they are reduced: (level, source, with the next)
  struct Pass { int li; bool records, two; };
  Pass ps[kMaxLevels];
  int np = 0;
  if (level == CHOPPER_LEVEL_ALL) {
    ps[np++] = Pass{D > 0 ? D - 1 : D, true, D >= 2};
    for (int li = D - (D >= 2 ? 3 : 2); li >= 0; li -= 2)
      ps[np++] = Pass{li, false, li >= 1};
  } else {
    ps[np++] = Pass{level == CHOPPER_LEVEL_GPU ? D : level, true, false};
  }
  // Pieces a pass may leave to the overflow list, of either level: the groups
  // that come back, and the first piece of every run of a tile.  Records: the
  // tiles the count was made on.  Rows, in order of their groups' first
  // records: where a group comes back at row b, the row before it belongs to
  // another group whose first record lies between that group's first record
  // and b's, so b's first record is in a stretch of the records in which the
  // group came back too, and in no other such row's stretch: rows come back
  // at most as often as records, and their own tiles' first pieces are added.
  // (The stretch may start on a record tile, so the count has to know the
  // item before it: rows that came back there were once missing.)
  auto left = [&](const Pass& q) {
    const int64_t runs =
        q.records ? (kNat ? 2 : 1) * nwt
                  : ceil_div(lo_h[q.li + 2] - lo_h[q.li + 1],
                             (int64_t)kWaveTile);
    return inner[q.li] + runs + (q.two ? inner[q.li - 1] + runs : 0);
  };
  for (int i = 0; i < np; ++i)
    if (left(ps[i]) > ovf.cap) return 1;
  // columns c0 .. c0 + kRowCols - 1 of start, end, gap, ovl and the counters
  // side by side (gap and ovl are complete here: the event above)
  const int cols = 4 + S.nc;
  auto stage = [&](int c0) -> int {
    StageCols C;
    for (int i = 0; i < kRowCols; ++i) {
      const int c = c0 + i;
      C.in[i] = c == 0    ? (const uint64_t*)S.start
                : c == 1  ? (const uint64_t*)S.end
                : c == 2  ? (const uint64_t*)S.gap
                : c == 3  ? (const uint64_t*)S.ovl
                : c < cols ? S.ctr + (int64_t)(c - 4) * S.n : nullptr;
    }
    CHOPPER_HIP(launch("agg_stage", k_stage_columns, grid_for(S.n, kBlock),
                       dim3(kBlock), s, C, S.n,
                       reinterpret_cast<ulonglong2*>(L.srow)));
    return CHOPPER_OK;
  };
  for (int i = 0; i < np; ++i) {
    const Pass& q = ps[i];
    const int li = q.li;
    GenRed GR;
    GR.own = tab.own[li];
    GR.own2 = q.two ? tab.own[li - 1] : tab.own[li];
    if (q.records) {
      const uint32_t* tbl = tb + (int64_t)li * stride;
      GR.mask = L.omask + (int64_t)li * L.mstride;
      GR.mask2 = q.two ? GR.mask - L.mstride : nullptr;
      if constexpr (!kNat) {
        GR.rows = reinterpret_cast<const ulonglong2*>(L.srow);
        GR.slots = L.slots;
        for (int c0 = 0; far && c0 < cols; c0 += kRowCols) {
          const int r = stage(c0);
          if (r != CHOPPER_OK) return r;
          GR.c0 = c0;
          GR.nc = cols - c0 < kRowCols ? cols - c0 : kRowCols;
          CHOPPER_HIP(launch("agg_gen_reduce_columns",
                             q.two ? k_agg_fast_reduce<kMD, FromRecords, true, false, true, false, true>
                                   : k_agg_fast_reduce<kMD, FromRecords, false, false, true, false, true>,
                             grid, dim3(kBlock), s, fr, N, li, D, M, tbl,
                             tbl - (q.two ? stride : 0),
                             (const int64_t*)nullptr, R, ovf, nwt, GR));
        }
      }
      if (!far)
        CHOPPER_HIP(launch("agg_gen_reduce_records",
                           q.two ? k_agg_fast_reduce<kMD, FromRecords, true, kNat, true, false>
                                 : k_agg_fast_reduce<kMD, FromRecords, false, kNat, true, false>,
                           grid, dim3(kBlock), s, fr, N, li, D, M, tbl,
                           tbl - (q.two ? stride : 0),
                           (const int64_t*)nullptr, R, ovf, nwt, GR));
    } else {
      const int64_t cnt = lo_h[li + 2] - lo_h[li + 1];
      if (cnt == 0) break;
      const int64_t nw = ceil_div(cnt, (int64_t)kWaveTile);
      const dim3 gr((unsigned)ceil_div(nw, (int64_t)kWavesPerBlock));
      FromRows src{R, M, rows->level_offset, li + 1};
      const int lv0 = q.two ? li - 1 : li;
      const uint32_t lact = q.two ? (3u << (li - 1)) : (1u << li);
      const int64_t tab_n = (q.two ? 2 : 1) * nw;
      uint32_t* done = tab_n <= kTailScan ? L.done + kDoneRows + li : nullptr;
      CHOPPER_HIP(launch("agg_gen_count_rows", k_gen_count_rows<kMD>, gr,
                         dim3(kBlock), s, src, lact, lv0, li, D, M, nw, tab,
                         L.htc2, L.htb2, L.omask, L.mstride, done,
                         L.ovf_count));
      if (!done)
        CHOPPER_HIP(exclusive_scan<uint32_t>(L.htc2, L.htb2, tab_n, L.hscan,
                                             L.htotal + 1, s));
      GR.mask = L.omask + (q.two ? L.mstride : 0);
      GR.mask2 = L.omask;
      const int64_t* r0 = rows->level_offset + li;
      if (q.two)
        CHOPPER_HIP(launch("agg_gen_reduce_rows",
                           k_agg_fast_reduce<kMD, FromRows, true, false, true, false>,
                           gr, dim3(kBlock), s, src, NatGeom{}, li, D, M,
                           (const uint32_t*)(L.htb2 + nw),
                           (const uint32_t*)L.htb2, r0, R, ovf, nw, GR));
      else
        CHOPPER_HIP(launch("agg_gen_reduce_rows",
                           k_agg_fast_reduce<kMD, FromRows, false, false, true, false>,
                           gr, dim3(kBlock), s, src, NatGeom{}, li, D, M,
                           (const uint32_t*)L.htb2, (const uint32_t*)nullptr,
                           r0, R, ovf, nw, GR));
    }
    CHOPPER_HIP(launch("agg_gen_apply", k_gen_apply,
                       grid_for(left(q), kBlock), dim3(kBlock), s, ovf, R,
                       nfields, (const uint32_t*)GR.own,
                       (const uint32_t*)GR.own2));
  }
  if (level == CHOPPER_LEVEL_ALL)
    return gpu_rows(L, R, D, nfields, rows->level_offset, s);
  return CHOPPER_OK;
}

template <int kMD>
static int agg_gen(const AggLayout& L, const RecSrc& S, const RowsDev& R,
                   const Overflow& ovf, int Lv, uint32_t act, int D,
                   int64_t M, int nfields, chopper_rows* rows, int level,
                   bool want_workload, uint32_t* status, hipEvent_t ready,
                   hipStream_t s, int nat, bool* conflict) {
  if (nat < 0) {
    const int rc = nat_geometry(L, S, s);
    if (rc != CHOPPER_OK) return rc;
  }
  if (nat != 0) {
    bool bad = false;
    const int rc = agg_gen_tiles<kMD, true>(
        L, S, R, ovf, Lv, act, D, M, nfields, rows, level, want_workload,
        status, ready, s, conflict, &bad);
    if (!bad) return rc;
  }
  bool bad = false;
  return agg_gen_tiles<kMD, false>(L, S, R, ovf, Lv, act, D, M, nfields, rows,
                                   level, want_workload, status, ready, s,
                                   conflict, &bad);
}

extern "C" int chopper_aggregate(const chopper_records* rec,
                                 const int64_t* start_al,
                                 const int64_t* end_al, const uint32_t* korder,
                                 const uint32_t* idx, int32_t depth,
                                 const int64_t* gap, const int64_t* ovl,
                                 const chopper_markers* mk, int32_t level,
                                 const chopper_filter* filter,
                                 chopper_rows* rows, void* scratch,
                                 size_t* scratch_bytes, uint32_t* status,
                                 void* ready, void* stream) {
  if (!validate_records(rec) || !validate_markers(mk) || !rows ||
      !scratch_bytes)
    return CHOPPER_EINVAL;
  const int64_t n = rec->n;
  const int D = depth;
  if (D < 0 || D > 8) return CHOPPER_EINVAL;
  if (mk && mk->depth != D) return CHOPPER_EINVAL;
  const int64_t M = mk ? mk->n : 0;
  if (filter && filter->use_iter && (!mk || (M > 0 && !mk->label)))
    return CHOPPER_EINVAL;
  if (n > 0 && (!start_al || !end_al || !korder || !gap || !ovl ||
                (D > 0 && !idx)))
    return CHOPPER_EINVAL;
  if (rows->cap < 0 || !rows->level_offset) return CHOPPER_EINVAL;
  if (rows->cap > 0 && (!rows->gpu || !rows->kind || !rows->n || !rows->dur ||
                        !rows->gap || !rows->ovl || !rows->tmin ||
                        !rows->tmax || !rows->first ||
                        (D > 0 && !rows->path) ||
                        (rec->n_counters > 0 && !rows->ctr)))
    return CHOPPER_EINVAL;
  uint32_t act = 0;
  if (level == CHOPPER_LEVEL_ALL) act = (1u << (D + 2)) - 1u;
  else if (level >= 0 && level < D) act = 1u << level;
  else if (level == CHOPPER_LEVEL_GPU) act = 1u << D;
  else if (level == CHOPPER_LEVEL_WORKLOAD) act = 1u << (D + 1);
  else return CHOPPER_EINVAL;

  Scratch probe(nullptr);
  agg_layout(probe, n, D, M, rows->cap, act, rec->n_gpus);
  int rc = scratch_check(scratch, scratch_bytes, probe.used);
  if (rc != 0) return rc > 0 ? CHOPPER_OK : rc;
  if (!status) return CHOPPER_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  Scratch sc(scratch);
  AggLayout L = agg_layout(sc, n, D, M, rows->cap, act, rec->n_gpus);
  const int Lv = L.L;
  const int64_t T = L.ntiles;
  const int nc = rec->n_counters;
  const int nfields = 6 + nc;

  RecSrc S;
  S.n = n;
  S.D = D;
  S.M = M;
  S.korder = korder;
  S.gpu = rec->gpu;
  S.cls = rec->cls;
  S.start = start_al;
  S.end = end_al;
  S.idx = idx;
  S.gap = gap;
  S.ovl = ovl;
  S.ctr = rec->counters;
  S.nc = nc;
  S.mlabel = mk ? mk->label : nullptr;
  memset(&S.f, 0, sizeof(S.f));
  S.gk = nullptr;
  S.ipath = nullptr;
  S.igk = nullptr;
  if (filter) {
    for (int q = 0; q < 4; ++q) S.f.gpu_mask[q] = filter->gpu_mask[q];
    S.f.class_mask = filter->class_mask;
    S.f.use_iter = filter->use_iter;
    S.f.iter_lo = filter->iter_lo;
    S.f.iter_hi = filter->iter_hi;
    S.f.active = 1;
  }
  RowsDev R;
  R.cap = rows->cap;
  R.path = rows->path;
  R.gpu = rows->gpu;
  R.kind = rows->kind;
  R.n = rows->n;
  R.dur = rows->dur;
  R.gap = rows->gap;
  R.ovl = rows->ovl;
  R.tmin = rows->tmin;
  R.tmax = rows->tmax;
  R.first = rows->first;
  R.ctr = rows->ctr;
  R.firstpos = L.firstpos;
  R.D = D;
  R.nc = nc;

  Overflow ovf{L.ovf_count, L.ovf_count + 1, L.ovf_row, L.ovf_val, L.ovf_cap};
  const bool want_workload = (act >> (D + 1)) & 1u;

  // ---- fast path: every group is one run of consecutive records
  // (the fast path addresses columns with 32-bit byte offsets)
  const bool tiles = n > 0 && level != CHOPPER_LEVEL_WORKLOAD &&
                     n < ((int64_t)1 << 29) && rows->cap < ((int64_t)1 << 29);
  const hipEvent_t rdy = (hipEvent_t)ready;
  int nat = -1;
  bool conflict = false;
  if (tiles && !filter) {
    rc = D <= 4 ? agg_fast<4>(L, S, R, ovf, T, Lv, act, D, M, nfields, rows,
                              level, want_workload, status, rdy, s, &nat,
                              &conflict)
       : D <= 6 ? agg_fast<6>(L, S, R, ovf, T, Lv, act, D, M, nfields, rows,
                              level, want_workload, status, rdy, s, &nat,
                              &conflict)
                : agg_fast<8>(L, S, R, ovf, T, Lv, act, D, M, nfields, rows,
                              level, want_workload, status, rdy, s, &nat,
                              &conflict);
    if (rc != 1) return rc;
  }
  // ---- groups of several runs, and selections
  if (tiles && M < kGenMaxM && !conflict) {
    rc = D <= 4 ? agg_gen<4>(L, S, R, ovf, Lv, act, D, M, nfields, rows,
                             level, want_workload, status, rdy, s, nat,
                             &conflict)
       : D <= 6 ? agg_gen<6>(L, S, R, ovf, Lv, act, D, M, nfields, rows,
                             level, want_workload, status, rdy, s, nat,
                             &conflict)
                : agg_gen<8>(L, S, R, ovf, Lv, act, D, M, nfields, rows,
                             level, want_workload, status, rdy, s, nat,
                             &conflict);
    if (rc != 1) return rc;
  }

  // ---- general path: per-level owner election (it reads gap and ovl)
  if (ready) CHOPPER_HIP(hipStreamWaitEvent(s, (hipEvent_t)ready, 0));
  // pointer tables for the per-level owner / row maps
  CHOPPER_HIP(hipMemcpyAsync(L.own_tab, L.own, sizeof(L.own),
                             hipMemcpyHostToDevice, s));
  CHOPPER_HIP(hipMemcpyAsync(L.rowof_tab, L.rowof, sizeof(L.rowof),
                             hipMemcpyHostToDevice, s));
  CHOPPER_HIP(hipMemcpyAsync(L.ks_dev, L.ks, sizeof(L.ks),
                             hipMemcpyHostToDevice, s));
  int64_t maxks = 1;
  for (int li = 0; li < Lv; ++li) maxks = L.ks[li] > maxks ? L.ks[li] : maxks;
  unsigned fx = (unsigned)ceil_div(maxks, kBlock);
  if (fx > 4096) fx = 4096;
  const uint32_t atomic_levels = (1u << D) | (1u << (D + 1));
  if (n > 0) {
    // the items once, in korder order, for the passes below
    CHOPPER_HIP(launch("agg_items", k_agg_items, grid_for(n, kBlock),
                       dim3(kBlock), s, S, L.ipath, L.igk));
    S.ipath = L.ipath;
    S.igk = L.igk;
  }

  // order of work: finest marker level from records, coarser marker levels
  // from the rows below, GPU rows from level-0 rows, workload from GPU rows
  auto run_level = [&](int li, bool atomic_mode) -> int {
    int finer = -1;                       // level whose rows feed this one
    if (level == CHOPPER_LEVEL_ALL) {
      if (li < D - 1) finer = li + 1;
      else if (li == D && D > 0) finer = 0;
      else if (li == D + 1) finer = D;
    }
    if (!atomic_mode)
      CHOPPER_HIP(launch("agg_zero", k_zero_u32, dim3(1), dim3(64), s,
                         L.ovf_count, 1));
    if (finer < 0) {
      FromRecords src{S};
      CHOPPER_HIP(launch("agg_reduce_records", k_agg_reduce<FromRecords>,
                         dim3((unsigned)T), dim3(kBlock), s, src, li, D, M,
                         atomic_mode, (const uint32_t*)L.own[li],
                         (const uint32_t*)L.rowof[li], R, ovf, nfields,
                         status, L.xflag));
    } else {
      FromRows src{R, M, rows->level_offset, finer, S.gk, n};
      // rows of the finer level never outnumber the records
      CHOPPER_HIP(launch("agg_reduce_rows", k_agg_reduce<FromRows>,
                         dim3((unsigned)T), dim3(kBlock), s, src, li, D, M,
                         atomic_mode, (const uint32_t*)L.own[li],
                         (const uint32_t*)L.rowof[li], R, ovf, nfields,
                         status, L.xflag));
    }
    if (!atomic_mode)
      CHOPPER_HIP(launch("agg_apply_overflow", k_agg_apply_overflow,
                         grid_for(L.ovf_cap, kBlock), dim3(kBlock), s, ovf, R,
                         nfields, (int64_t)-1));
    if (li == D + 1) {
      if (finer < 0) {
        FromRecords src{S};
        CHOPPER_HIP(launch("agg_workload_first",
                           k_agg_workload_first<FromRecords>,
                           grid_for(n, kBlock), dim3(kBlock), s, src, D, M,
                           (const uint32_t*)L.rowof[li], R));
      } else {
        FromRows src{R, M, rows->level_offset, finer, S.gk, n};
        CHOPPER_HIP(launch("agg_workload_first", k_agg_workload_first<FromRows>,
                           grid_for(n, kBlock), dim3(kBlock), s, src, D, M,
                           (const uint32_t*)L.rowof[li], R));
      }
    }
    return CHOPPER_OK;
  };
  int order_levels[kMaxLevels];
  int nl = 0;
  for (int li = D - 1; li >= 0; --li)
    if ((act >> li) & 1u) order_levels[nl++] = li;
  if ((act >> D) & 1u) order_levels[nl++] = D;
  if ((act >> (D + 1)) & 1u) order_levels[nl++] = D + 1;
  auto run_all = [&]() -> int {
    CHOPPER_HIP(launch("agg_fill_owner", k_fill_u32_many, dim3(fx, Lv),
                       dim3(kBlock), s, L.own_tab, (const int64_t*)L.ks_dev,
                       Lv, act));
    if (n > 0) {
      CHOPPER_HIP(launch("agg_elect", k_agg_elect, dim3((unsigned)T),
                         dim3(kBlock), s, S, act, L.own_tab));
      CHOPPER_HIP(launch("agg_count", k_agg_count, dim3((unsigned)T),
                         dim3(kBlock), s, S, act, L.own_tab, T, L.tilecnt));
    }
    CHOPPER_HIP(exclusive_scan<uint32_t>(L.tilecnt, L.tilebase,
                                         (int64_t)Lv * T, L.scantmp, L.total,
                                         s));
    CHOPPER_HIP(launch("agg_offsets", k_agg_offsets_all, dim3(1), dim3(64), s,
                       Lv, T, (const uint32_t*)L.tilebase,
                       (const uint32_t*)L.total, rows->cap,
                       rows->level_offset, status));
    if (n == 0) return CHOPPER_OK;
    CHOPPER_HIP(launch("agg_assign", k_agg_assign, dim3((unsigned)T),
                       dim3(kBlock), s, S, act, atomic_levels, L.own_tab,
                       L.rowof_tab, T, (const uint32_t*)L.tilebase, R));
    CHOPPER_HIP(launch("agg_zero", k_zero_u32, dim3(1), dim3(64), s,
                       L.ovf_count, 2));
    for (int q = 0; q < nl; ++q) {
      const int li = order_levels[q];
      const int r = run_level(li, (atomic_levels >> li) & 1u);
      if (r != CHOPPER_OK) return r;
    }
    return CHOPPER_OK;
  };
  // markers not nested (a record's path differs from its row's): grouped by
  // the whole path, with exact group ids -- at once when the tiles above
  // met it, else after the deepest-marker pass that does
  int lmax = -1;
  for (int li = 0; li < D; ++li)
    if ((act >> li) & 1u) lmax = li;
  if (n > 0)
    CHOPPER_HIP(launch("agg_zero", k_zero_u32, dim3(1), dim3(64), s, L.xflag,
                       1));
  if (!conflict) {
    rc = run_all();
    if (rc != CHOPPER_OK || n == 0) return rc;
    uint32_t met = 0;
    CHOPPER_HIP(read_back(L.xflag, &met, sizeof(uint32_t), s));
    conflict = met != 0;
  }
  if (conflict && lmax >= 0) {
    rc = exact_group_ids(L, S, lmax, s);
    if (rc != CHOPPER_OK) return rc;
    S.gk = L.gk;
    rc = run_all();
    if (rc != CHOPPER_OK) return rc;
  }
  // an overflow list that did not fit: redo the marker levels with atomics
  uint32_t lost = 0;
  CHOPPER_HIP(read_back(L.ovf_count + 1, &lost, sizeof(uint32_t), s));
  if (lost) {
    for (int q = 0; q < nl; ++q) {
      const int li = order_levels[q];
      CHOPPER_HIP(launch("agg_zero_rows", k_agg_zero_rows, dim3(1024),
                         dim3(kBlock), s, (const int64_t*)rows->level_offset,
                         li, li + 1, R));
      rc = run_level(li, true);
      if (rc != CHOPPER_OK) return rc;
    }
  }
  return CHOPPER_OK;
}
