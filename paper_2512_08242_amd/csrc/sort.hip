// Stable sorts of items by (class, time) for gfx950.
//
// Fast path: a stable counting-sort pass by class (class ids are dense, at
// most 256) followed by a check that every class run of the output is
// non-decreasing in time.  When the input already lists each class in time
// order -- what a profiler emits per GPU and stream -- that single pass is
// the complete stable sort.
//
// General path: LSD radix sort of packed 64-bit keys (class << T | time -
// tmin) with 8-bit digits.  Every pass: per-tile digit histograms in LDS, a
// device-wide exclusive scan of the digit-major histogram table, then a
// stable scatter whose in-tile ranks come from wave64 ballots (eight
// __ballot calls match lanes with equal digits, popcount of the lower lanes
// gives the rank) and per-wave digit counts in LDS.  Each tile is first
// reordered in LDS so that the global writes of one digit bucket are
// contiguous.
#include <type_traits>

#include "sort.h"
#include "wave.h"

namespace chopper {

constexpr int kSortIpt = 8;
constexpr int kSortTile = kBlock * kSortIpt;

int64_t sort_tiles(int64_t n) { return ceil_div(n, kSortTile); }

// ---------------------------------------------------------------------------
// In-tile stable ranking of up to 256 digit values.
// Every wave takes kWaveTile consecutive positions of the tile, a row of 64
// at a time (item j of a lane is tile position tile_pos(j)).  A row counts
// its digits with `nbits` ballots (lanes with equal digits find each other);
// an item's rank is the wave's count of its digit so far, kept in LDS, plus
// the equal lanes below it, and the lowest of them moves the count on: no
// barrier until the four waves' counts are put in order.  (The partition is
// bound by what a block keeps in flight; with one count per row and wave,
// cleared and scanned, 16 KB of LDS a block and four more barriers, the
// partition of seven passes of 9.83M entries took 182 us, now 130.)
// On return count[d] = number of valid items with digit d in the tile,
// start[d] = exclusive prefix of count, rank[j] = stable position of the
// item among equal digits.
// ---------------------------------------------------------------------------
struct RankShared {
  uint32_t cell[kWavesPerBlock][256];   // counts, then prefixes over waves
  uint32_t start[256];
};
static_assert(kSortIpt == kTileIpt, "a wave's share of a tile");

__device__ inline int tile_pos(int j) {
  return (int)(threadIdx.x / kWave) * kWaveTile + j * kWave + lane_id();
}

__device__ inline void tile_rank(const uint32_t (&dig)[kSortIpt],
                                 const bool (&valid)[kSortIpt],
                                 uint32_t (&rank)[kSortIpt], RankShared& sh,
                                 int nbits) {
  const int t = threadIdx.x;
  const int lane = t & (kWave - 1);
  const int w = t / kWave;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t* cell = sh.cell[w];
  reinterpret_cast<uint4*>(cell)[lane] = make_uint4(0u, 0u, 0u, 0u);
  wave_sync();
#pragma unroll
  for (int j = 0; j < kSortIpt; ++j) {
    const uint32_t d = dig[j];
    const bool v = valid[j];
    const uint64_t peers = digit_peers(d, v, nbits);
    const uint32_t before = (uint32_t)__popcll(peers & lt);
    const uint32_t base = v ? cell[d] : 0u;
    rank[j] = base + before;
    wave_sync();
    if (v && before == 0) cell[d] = base + (uint32_t)__popcll(peers);
    wave_sync();
  }
  __syncthreads();
  // digit t: exclusive prefix over the waves
  uint32_t acc = 0;
#pragma unroll
  for (int q = 0; q < kWavesPerBlock; ++q) {
    const uint32_t c = sh.cell[q][t];
    sh.cell[q][t] = acc;
    acc += c;
  }
  uint32_t tot;
  sh.start[t] = block_exclusive(acc, OpAdd(), 0u, &tot);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSortIpt; ++j)
    if (valid[j]) rank[j] += cell[dig[j]];
}

// ---------------------------------------------------------------------------
// Class-partition fast path
// ---------------------------------------------------------------------------
// Class ids of the tile in the arrangement the ranking needs: loaded eight
// consecutive items per lane and turned around inside the wave through
// `s_tmp` (kSortTile bytes; class ids are below 256).
template <typename Acc>
__device__ inline void striped_classes(const Acc& acc, int64_t base,
                                       int64_t n, uint8_t* s_tmp,
                                       uint32_t (&dig)[kSortIpt],
                                       bool (&valid)[kSortIpt]) {
  uint32_t d[kSortIpt];
  bool v[kSortIpt];
  cls_block(acc, base + (int64_t)threadIdx.x * kSortIpt, n, d, v);
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    lo |= d[j] << (8 * j);
    hi |= d[j + 4] << (8 * j);
  }
  reinterpret_cast<uint2*>(s_tmp)[threadIdx.x] = make_uint2(lo, hi);
  wave_sync();
#pragma unroll
  for (int j = 0; j < kSortIpt; ++j) {
    const int q = tile_pos(j);
    valid[j] = base + q < n;
    dig[j] = valid[j] ? (uint32_t)s_tmp[q] : 0u;
  }
  wave_sync();
}

// With `unsorted`, also a cheap sufficient test of sortedness on the same
// items, while they are at hand: is the input ordered by (major, time)?
template <typename Acc>
__device__ inline void class_hist(const Acc& acc, uint32_t block, int64_t n,
                                  int64_t ntiles, uint32_t* tilehist,
                                  uint32_t* unsorted) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int nbits = class_bits(acc.nclass());
  const int lane = threadIdx.x & (kWave - 1);
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int64_t base = (int64_t)block * kSortTile;
  // (counts need no order: eight consecutive items per lane, vector loads)
  uint32_t d[kSortIpt];
  bool v[kSortIpt];
  cls_block(acc, base + (int64_t)threadIdx.x * kSortIpt, n, d, v);
  // one LDS add per distinct class of every wave-row
#pragma unroll
  for (int j = 0; j < kSortIpt; ++j) {
    const uint64_t peers = digit_peers(d[j], v[j], nbits);
    if (v[j] && __popcll(peers & lt) == 0)
      atomicAdd(&h[d[j]], (uint32_t)__popcll(peers));
  }
  if (unsorted) {
    // eight consecutive items and the next one per lane
    const int64_t i0 = base + (int64_t)threadIdx.x * kSortIpt;
    bool bad = false;
    if (i0 < n) {
      uint32_t m[9];
      int64_t t[9];
      bool w[9];
      major_time_block(acc, i0, n, m, t, w);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (w[j + 1])
          bad = bad || m[j] > m[j + 1] || (m[j] == m[j + 1] && t[j + 1] < t[j]);
    }
    wave_flag_or(unsorted, bad, 1u);
  }
  __syncthreads();
  if ((int)threadIdx.x < acc.nclass())
    tilehist[(int64_t)threadIdx.x * ntiles + block] = h[threadIdx.x];
}

template <typename Acc>
__global__ __launch_bounds__(kBlock) void k_class_hist(Acc acc, int64_t n,
                                                       int64_t ntiles,
                                                       uint32_t* tilehist,
                                                       uint32_t* unsorted) {
  class_hist(acc, blockIdx.x, n, ntiles, tilehist, unsorted);
}

// Block 0 also writes the class start offsets: coff[c] = first position of
// class c (the scanned table's first tile), coff[C] = n.  `sub`: what the
// scan had counted before this table.
template <typename Acc, typename Cols>
__device__ inline void class_partition(
    const Acc& acc, uint32_t block, int64_t n, int64_t ntiles,
    const uint32_t* tileoff, uint32_t sub, uint32_t* out, uint32_t* coff,
    const Cols& cols) {
  if (block == 0) {
    const int C = acc.nclass();
    for (int c = threadIdx.x; c <= C; c += kBlock)
      coff[c] = c < C ? tileoff[(int64_t)c * ntiles] - sub : (uint32_t)n;
  }
  __shared__ RankShared sh;
  __shared__ uint32_t s_val[kSortTile];
  __shared__ __attribute__((aligned(8))) uint8_t s_dig[kSortTile];
  __shared__ uint32_t s_gbase[256];
  const int64_t base = (int64_t)block * kSortTile;
  uint32_t dig[kSortIpt], rank[kSortIpt];
  bool valid[kSortIpt];
  striped_classes(acc, base, n, s_dig, dig, valid);
  tile_rank(dig, valid, rank, sh, class_bits(acc.nclass()));
  if ((int)threadIdx.x < acc.nclass())
    s_gbase[threadIdx.x] =
        tileoff[(int64_t)threadIdx.x * ntiles + block] - sub;
  for (int j = 0; j < kSortIpt; ++j) {
    if (!valid[j]) continue;
    uint32_t lp = sh.start[dig[j]] + rank[j];
    s_val[lp] = (uint32_t)(base + tile_pos(j));
    s_dig[lp] = (uint8_t)dig[j];
  }
  __syncthreads();
  const int64_t tile_n = (n - base) < kSortTile ? (n - base) : kSortTile;
  for (int j = 0; j < kSortIpt; ++j) {
    int q = j * kBlock + threadIdx.x;
    if (q >= tile_n) continue;
    uint32_t d = s_dig[q];
    const int64_t pos = (int64_t)s_gbase[d] + (q - sh.start[d]);
    out[pos] = s_val[q];
    cols.put(pos, s_val[q], d);
  }
}

template <typename Acc, typename Cols>
__global__ __launch_bounds__(kBlock) void k_class_partition(
    Acc acc, int64_t n, int64_t ntiles, const uint32_t* tileoff,
    uint32_t* out, uint32_t* coff, Cols cols) {
  class_partition(acc, blockIdx.x, n, ntiles, tileoff, 0u, out, coff, cols);
}

// the same for several item lists, one per blockIdx.y
__global__ __launch_bounds__(kBlock) void k_class_hist_lists(ClassLists B,
                                                             uint32_t* tilehist) {
  const ClassList& P = B.l[blockIdx.y];
  const int64_t T = (P.n + kSortTile - 1) / kSortTile;
  if ((int64_t)blockIdx.x >= T) return;                    // whole block
  class_hist(P.key, blockIdx.x, P.n, T, tilehist + P.tab, nullptr);
}

__global__ __launch_bounds__(kBlock) void k_class_partition_lists(
    ClassLists B, const uint32_t* tileoff) {
  const ClassList& P = B.l[blockIdx.y];
  const int64_t T = (P.n + kSortTile - 1) / kSortTile;
  if ((int64_t)blockIdx.x >= T) return;                    // whole block
  class_partition(P.key, blockIdx.x, P.n, T, tileoff + P.tab, P.sub, P.out,
                  P.coff, NoColumns());
}

// (stops reading once some wave has found the answer)
template <typename Acc>
__global__ __launch_bounds__(kBlock) void k_class_verify(Acc acc, int64_t n,
                                                         const uint32_t* perm,
                                                         uint32_t* unsorted) {
  if (__builtin_amdgcn_readfirstlane((int)flag_read(unsorted)) != 0) return;
  int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  bool bad = false;
  if (p + 1 < n) {
    uint32_t a = perm[p], b = perm[p + 1];
    bad = acc.cls(a) == acc.cls(b) && acc.time(b) < acc.time(a);
  }
  wave_flag_or(unsorted, bad, 1u);
}

// ---------------------------------------------------------------------------
// General path: packed keys + LSD radix passes
// ---------------------------------------------------------------------------
template <typename Acc>
__global__ __launch_bounds__(kBlock) void k_time_minmax(Acc acc, int64_t n,
                                                        int64_t* mm) {
  int64_t lo = kI64Max, hi = kI64Min;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kBlock) {
    int64_t t = acc.time(i);
    lo = t < lo ? t : lo;
    hi = t > hi ? t : hi;
  }
  for (int d = kWave / 2; d > 0; d >>= 1) {
    int64_t a = __shfl_xor(lo, d, kWave), b = __shfl_xor(hi, d, kWave);
    lo = a < lo ? a : lo;
    hi = b > hi ? b : hi;
  }
  if ((threadIdx.x & (kWave - 1)) == 0) {
    atomicMin((long long*)&mm[0], (long long)lo);
    atomicMax((long long*)&mm[1], (long long)hi);
  }
}

__global__ void k_init_minmax(int64_t* mm) {
  mm[0] = kI64Max;
  mm[1] = kI64Min;
}

template <typename Acc>
__global__ __launch_bounds__(kBlock) void k_make_keys(Acc acc, int64_t n,
                                                      const int64_t* mm,
                                                      int tbits, uint64_t* key,
                                                      uint32_t* val) {
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  uint64_t t = (uint64_t)(acc.time(i) - mm[0]);
  uint64_t c = acc.cls(i);
  key[i] = (tbits >= 64 ? 0ull : (c << tbits)) | t;
  val[i] = (uint32_t)i;
}

__global__ __launch_bounds__(kBlock) void k_digit_hist(const uint64_t* key,
                                                       int64_t n, int shift,
                                                       int64_t ntiles,
                                                       uint32_t* tilehist) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
  for (int j = 0; j < kSortIpt; ++j) {
    int64_t i = base + (int64_t)j * kBlock + threadIdx.x;
    if (i < n) atomicAdd(&h[(uint32_t)(key[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  tilehist[(int64_t)threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

__global__ __launch_bounds__(kBlock) void k_digit_scatter(
    const uint64_t* key_in, const uint32_t* val_in, int64_t n, int shift,
    int64_t ntiles, const uint32_t* tileoff, uint64_t* key_out,
    uint32_t* val_out) {
  __shared__ RankShared sh;
  __shared__ uint64_t s_key[kSortTile];
  __shared__ uint32_t s_val[kSortTile];
  __shared__ uint32_t s_gbase[256];
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
  uint32_t dig[kSortIpt], rank[kSortIpt];
  bool valid[kSortIpt];
  uint64_t k[kSortIpt];
  uint32_t v[kSortIpt];
  for (int j = 0; j < kSortIpt; ++j) {
    int64_t i = base + tile_pos(j);
    valid[j] = i < n;
    k[j] = valid[j] ? key_in[i] : 0ull;
    v[j] = valid[j] ? val_in[i] : 0u;
    dig[j] = (uint32_t)(k[j] >> shift) & 255u;
  }
  tile_rank(dig, valid, rank, sh, 8);
  s_gbase[threadIdx.x] = tileoff[(int64_t)threadIdx.x * ntiles + blockIdx.x];
  for (int j = 0; j < kSortIpt; ++j) {
    if (!valid[j]) continue;
    uint32_t lp = sh.start[dig[j]] + rank[j];
    s_key[lp] = k[j];
    s_val[lp] = v[j];
  }
  __syncthreads();
  const int64_t tile_n = (n - base) < kSortTile ? (n - base) : kSortTile;
  for (int j = 0; j < kSortIpt; ++j) {
    int q = j * kBlock + threadIdx.x;
    if (q >= tile_n) continue;
    uint64_t kk = s_key[q];
    uint32_t d = (uint32_t)(kk >> shift) & 255u;
    int64_t pos = (int64_t)s_gbase[d] + (q - sh.start[d]);
    if (key_out) key_out[pos] = kk;
    val_out[pos] = s_val[q];
  }
}

// class histogram for more than 256 classes (general path only)
template <typename Acc>
__global__ __launch_bounds__(kBlock) void k_class_count_global(
    Acc acc, int64_t n, uint32_t* counts) {
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) atomicAdd(&counts[acc.cls(i)], 1u);
}

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_status_set(uint32_t bits, uint32_t* status) {
  atomicOr(status, bits);
}

// ---------------------------------------------------------------------------
// Host driver
// ---------------------------------------------------------------------------
static int bitlen_u64(uint64_t x) {
  int b = 0;
  while (x) { ++b; x >>= 1; }
  return b;
}

ClassSortLayout class_sort_layout(Scratch& sc, int64_t n, int C) {
  ClassSortLayout L;
  L.n = n;
  L.C = C;   // maximum number of classes the tables are sized for
  L.ntiles = sort_tiles(n);
  int64_t hist_elems = (int64_t)(C > 256 ? 256 : C) * L.ntiles;
  int64_t radix_elems = 256 * L.ntiles;
  int64_t tab = hist_elems > radix_elems ? hist_elems : radix_elems;
  if (C > 256 && C > tab) tab = C;
  L.tilehist = sc.take<uint32_t>(tab);
  L.tileoff = sc.take<uint32_t>(tab);
  L.scantmp = sc.take<uint32_t>(scan_scratch_elems(tab));
  L.total = sc.take<uint32_t>(4);
  L.flag = sc.take<uint32_t>(4);
  L.mm = sc.take<int64_t>(2);
  L.key0 = sc.take<uint64_t>(n);
  L.key1 = sc.take<uint64_t>(n);
  L.val0 = sc.take<uint32_t>(n);
  L.val1 = sc.take<uint32_t>(n);
  return L;
}

template <typename Acc, typename Cols>
int class_sort(const Acc& acc, const ClassSortLayout& L, uint32_t* out,
               uint32_t* coff, bool* range_error, hipStream_t s,
               int known_sorted, const Cols& cols, bool* cols_done) {
  if (cols_done) *cols_done = false;
  const int64_t n = L.n;
  const int C = acc.nclass();
  const int64_t T = L.ntiles;
  if (C > L.C) return CHOPPER_EINVAL;
  *range_error = false;
  if (n == 0) {
    CHOPPER_HIP(launch("sort_fill", k_fill_u32, dim3(1), dim3(kBlock), s,
                       coff, (int64_t)(C + 1), 0u));
    return CHOPPER_OK;
  }
  bool sorted = false;
  if (C <= 256) {
    // cheap sufficient test on the input, ordered by (major, time), made
    // by the histogram pass; its read-back is waited for after the
    // partition is queued, which runs either way
    ReadBack rb;
    if (known_sorted < 0)
      CHOPPER_HIP(launch("sort_fill", k_fill_u32, dim3(1), dim3(kBlock), s,
                         L.flag, (int64_t)1, 0u));
    CHOPPER_HIP(launch("sort_class_hist", k_class_hist<Acc>, dim3((unsigned)T),
                       dim3(kBlock), s, acc, n, T, L.tilehist,
                       known_sorted < 0 ? L.flag : (uint32_t*)nullptr));
    if (known_sorted < 0)
      CHOPPER_HIP(read_back_start(L.flag, sizeof(uint32_t), s, &rb));
    CHOPPER_HIP(exclusive_scan<uint32_t>(L.tilehist, L.tileoff, (int64_t)C * T,
                                         L.scantmp, L.total, s));
    // The markers' partition may run beside the overlap call on another
    // stream, whose union runs decide when the step goes on: 12 KB of LDS
    // that it does not use keep it at five blocks a CU.  (At full occupancy
    // it takes the union runs' slots: a step of 19.66M records 3224 us
    // against 3196 with the LDS.  Where there is nothing beside it, or fewer
    // blocks than that, it makes no difference: steps of 2,000, 245,760 and
    // 2.46M records 220, 299 and 633 us against 219, 299 and 637, 50M
    // shuffled ones 86.4 ms against 86.5, within what two runs differ.)
    constexpr size_t kSpare = std::is_same<Cols, MarkerColumns>::value ? 12288 : 0;
    CHOPPER_HIP(launch_shm("sort_class_partition",
                           k_class_partition<Acc, Cols>, dim3((unsigned)T),
                           dim3(kBlock), kSpare, s, acc, n, T,
                           (const uint32_t*)L.tileoff, out, coff, cols));
    if (known_sorted < 0) {
      uint32_t unsorted = 1;
      CHOPPER_HIP(read_back_finish(&rb, &unsorted));
      if (unsorted == 0) known_sorted = 1;
    }
    if (known_sorted == 1) {
      sorted = true;
    } else {
      // the partition may still be the sorted order (e.g. input already in
      // class order): verify the class runs of the output
      CHOPPER_HIP(launch("sort_fill", k_fill_u32, dim3(1), dim3(kBlock), s,
                         L.flag, (int64_t)1, 0u));
      CHOPPER_HIP(launch("sort_class_verify", k_class_verify<Acc>,
                         grid_for(n, kBlock), dim3(kBlock), s, acc, n,
                         (const uint32_t*)out, L.flag));
      uint32_t unsorted = 1;
      CHOPPER_HIP(read_back(L.flag, &unsorted, sizeof(uint32_t), s));
      sorted = (unsorted == 0);
    }
  } else {
    CHOPPER_HIP(launch("sort_fill", k_fill_u32, grid_for(C, kBlock),
                       dim3(kBlock), s, L.tilehist, (int64_t)C, 0u));
    CHOPPER_HIP(launch("sort_class_count", k_class_count_global<Acc>,
                       grid_for(n, kBlock), dim3(kBlock), s, acc, n,
                       L.tilehist));
    CHOPPER_HIP(exclusive_scan<uint32_t>(L.tilehist, coff, (int64_t)C,
                                         L.scantmp, coff + C, s));
  }
  if (sorted) {
    if (cols_done) *cols_done = true;
    return CHOPPER_OK;
  }

  // general path
  CHOPPER_HIP(launch("sort_init_minmax", k_init_minmax, dim3(1), dim3(1), s,
                     L.mm));
  CHOPPER_HIP(launch("sort_time_minmax", k_time_minmax<Acc>,
                     dim3((unsigned)(T < 1024 ? T : 1024)), dim3(kBlock), s,
                     acc, n, L.mm));
  int64_t mm[2];
  CHOPPER_HIP(read_back(L.mm, mm, sizeof(mm), s));
  const int tbits = bitlen_u64((uint64_t)(mm[1] - mm[0]));
  const int cbits = bitlen_u64((uint64_t)(C > 1 ? C - 1 : 0));
  if (tbits + cbits > 64) {
    *range_error = true;
    return CHOPPER_OK;
  }
  CHOPPER_HIP(launch("sort_make_keys", k_make_keys<Acc>, grid_for(n, kBlock),
                     dim3(kBlock), s, acc, n, (const int64_t*)L.mm, tbits,
                     L.key0, L.val0));
  return radix_sort_pairs(L, tbits + cbits, out, nullptr, s);
}

int class_partition_lists(ClassLists& B, const ClassSortLayout& L,
                          hipStream_t s) {
  int64_t tab = 0, tmax = 0;
  uint32_t sub = 0;
  for (int p = 0; p < B.count; ++p) {
    ClassList& P = B.l[p];
    const int64_t T = sort_tiles(P.n);
    P.tab = tab;
    P.sub = sub;
    tab += T * P.key.nclass();
    sub += (uint32_t)P.n;
    tmax = T > tmax ? T : tmax;
  }
  if (tab > 256 * L.ntiles) return CHOPPER_EINVAL;
  if (tmax == 0) return CHOPPER_OK;
  const dim3 g((unsigned)tmax, (unsigned)B.count);
  CHOPPER_HIP(launch("sort_class_hist", k_class_hist_lists, g, dim3(kBlock), s,
                     B, L.tilehist));
  CHOPPER_HIP(exclusive_scan<uint32_t>(L.tilehist, L.tileoff, tab, L.scantmp,
                                       L.total, s));
  CHOPPER_HIP(launch("sort_class_partition", k_class_partition_lists, g,
                     dim3(kBlock), s, B, (const uint32_t*)L.tileoff));
  return CHOPPER_OK;
}

int radix_sort_pairs(const ClassSortLayout& L, int bits, uint32_t* out,
                     uint64_t* keys_out, hipStream_t s) {
  const int64_t n = L.n;
  const int64_t T = L.ntiles;
  if (n == 0) return CHOPPER_OK;
  const int passes = bits <= 0 ? 0 : (bits + 7) / 8;
  uint64_t* kin = L.key0;
  uint64_t* kout = L.key1;
  uint32_t* vin = L.val0;
  uint32_t* vout = L.val1;
  for (int p = 0; p < passes; ++p) {
    const int shift = 8 * p;
    const bool last = (p == passes - 1);
    CHOPPER_HIP(launch("sort_digit_hist", k_digit_hist, dim3((unsigned)T),
                       dim3(kBlock), s, (const uint64_t*)kin, n, shift, T,
                       L.tilehist));
    CHOPPER_HIP(exclusive_scan<uint32_t>(L.tilehist, L.tileoff, 256 * T,
                                         L.scantmp, L.total, s));
    CHOPPER_HIP(launch("sort_digit_scatter", k_digit_scatter,
                       dim3((unsigned)T), dim3(kBlock), s,
                       (const uint64_t*)kin, (const uint32_t*)vin, n, shift, T,
                       (const uint32_t*)L.tileoff, last ? keys_out : kout,
                       last ? out : vout));
    uint64_t* tk = kin; kin = kout; kout = tk;
    uint32_t* tv = vin; vin = vout; vout = tv;
  }
  if (passes == 0) {
    CHOPPER_HIP(hipMemcpyAsync(out, L.val0, sizeof(uint32_t) * n,
                               hipMemcpyDeviceToDevice, s));
    if (keys_out)
      CHOPPER_HIP(hipMemcpyAsync(keys_out, L.key0, sizeof(uint64_t) * n,
                                 hipMemcpyDeviceToDevice, s));
  }
  return CHOPPER_OK;
}

// ---------------------------------------------------------------------------
// Two class partitions of the same items, for input already ordered by
// (major, time): one histogram pass fills both tables (A's classes, then
// B's), one scan covers both, one pass writes both permutations.
// ---------------------------------------------------------------------------
template <typename AccA, typename AccB>
__global__ __launch_bounds__(kBlock) void k_class_hist2(
    AccA a, AccB b, int64_t n, int64_t ntiles, const WaveClasses* wcls,
    uint32_t* tilehist) {
  __shared__ uint32_t h[2][256];
  h[0][threadIdx.x] = 0;
  h[1][threadIdx.x] = 0;
  __syncthreads();
  static_assert(kSortTile == kWavesPerBlock * kWaveTile,
                "a sort tile is four wave tiles");
  if (wcls) {
    // the tile's wave tiles, when each holds at most two classes per key
    // (the same decision in every thread)
    const int64_t w0 = (int64_t)blockIdx.x * kWavesPerBlock;
    const int64_t nw = ceil_div(n, (int64_t)kWaveTile);
    bool few = true;
    for (int q = 0; q < kWavesPerBlock; ++q)
      if (w0 + q < nw)
        few = few && wcls[w0 + q].a1 != kManyClasses &&
              wcls[w0 + q].b1 != kManyClasses;
    if (few) {
      // thread q * 4 + k: wave q, key k / 2, class k % 2
      const int q = (int)threadIdx.x >> 2, k = (int)threadIdx.x & 3;
      if (q < kWavesPerBlock && w0 + q < nw) {
        const WaveClasses& c = wcls[w0 + q];
        const uint32_t raw = k == 0 ? c.a0 : k == 1 ? c.a1 : k == 2 ? c.b0 : c.b1;
        const uint32_t cnt =
            k == 0 ? c.na0 : k == 1 ? c.na1 : k == 2 ? c.nb0 : c.nb1;
        if (cnt > 0)
          atomicAdd(&h[k >> 1][k < 2 ? a.cls_of_raw(raw) : b.cls_of_raw(raw)],
                    cnt);
      }
      __syncthreads();
      const int CA = a.nclass();
      if ((int)threadIdx.x < CA)
        tilehist[(int64_t)threadIdx.x * ntiles + blockIdx.x] = h[0][threadIdx.x];
      if ((int)threadIdx.x < b.nclass())
        tilehist[(int64_t)(CA + threadIdx.x) * ntiles + blockIdx.x] =
            h[1][threadIdx.x];
      return;
    }
  }
  const int lane = threadIdx.x & (kWave - 1);
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
  const int nb[2] = {class_bits(a.nclass()), class_bits(b.nclass())};
  // every class id of the tile first (eight consecutive items per lane,
  // vector loads; counts need no order), then the counts
  uint32_t d[2][kSortIpt];
  bool v[kSortIpt];
  cls_block(a, base + (int64_t)threadIdx.x * kSortIpt, n, d[0], v);
  cls_block(b, base + (int64_t)threadIdx.x * kSortIpt, n, d[1], v);
#pragma unroll
  for (int j = 0; j < kSortIpt; ++j) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const uint64_t peers = digit_peers(d[q][j], v[j], nb[q]);
      if (v[j] && __popcll(peers & lt) == 0)
        atomicAdd(&h[q][d[q][j]], (uint32_t)__popcll(peers));
    }
  }
  __syncthreads();
  const int CA = a.nclass();
  if ((int)threadIdx.x < CA)
    tilehist[(int64_t)threadIdx.x * ntiles + blockIdx.x] = h[0][threadIdx.x];
  if ((int)threadIdx.x < b.nclass())
    tilehist[(int64_t)(CA + threadIdx.x) * ntiles + blockIdx.x] =
        h[1][threadIdx.x];
}

// Tiles of at most two classes per key -- nearly every tile of records in
// (gpu, start') order: one GPU's compute and communication streams -- are
// partitioned by a pass of their own: the tile's classes c0 (its first
// item's) and c1 come from its waves' class records; every thread takes
// eight consecutive items and compares their raw codes with c1; one block
// scan of the class-c1 counts of both keys (packed in one word) ranks every
// item; both permutations are laid out in LDS in output order, so that the
// stores are coalesced.  It flags the other tiles, and the general pass
// below (the LDS ranking) does only those.
template <typename AccA, typename AccB>
__global__ __launch_bounds__(kBlock) void k_class_partition2_two(
    AccA a, AccB b, int64_t n, int64_t ntiles, const uint32_t* tileoff,
    const WaveClasses* wcls, uint32_t* outA, uint32_t* outB,
    uint8_t* general) {
  __shared__ uint32_t s_out[2][kSortTile];
  __shared__ uint32_t s_w[kWavesPerBlock];
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
  const int tile_n =
      (int)((n - base) < kSortTile ? (n - base) : (int64_t)kSortTile);
  // the tile's classes per key (the same in every thread): wave 0's first
  // class is the tile's first item's
  const int64_t w0 = (int64_t)blockIdx.x * kWavesPerBlock;
  const int64_t nw = ceil_div(n, (int64_t)kWaveTile);
  uint32_t A[2] = {kNone, kNone}, B[2] = {kNone, kNone};
  bool ok = true;
  auto add = [&](uint32_t (&C)[2], uint32_t c, uint32_t cnt) {
    if (c == kManyClasses) ok = false;
    if (!ok || cnt == 0) return;
    if (C[0] == kNone || C[0] == c) C[0] = c;
    else if (C[1] == kNone || C[1] == c) C[1] = c;
    else ok = false;
  };
  for (int q = 0; q < kWavesPerBlock; ++q) {
    if (w0 + q >= nw) break;
    const WaveClasses c = wcls[w0 + q];
    add(A, c.a0, c.na0);
    add(A, c.a1, c.na1);
    add(B, c.b0, c.nb0);
    add(B, c.b1, c.nb1);
  }
  if (threadIdx.x == 0) general[blockIdx.x] = ok ? 0 : 1;
  if (!ok) return;   // (block-uniform)
  const int t = (int)threadIdx.x, lane = t & (kWave - 1), wv = t / kWave;
  uint32_t ra[kSortIpt], rb[kSortIpt];
  a.raw8(base + (int64_t)t * kSortIpt, n, ra);
  b.raw8(base + (int64_t)t * kSortIpt, n, rb);
  uint32_t ma = 0, mb = 0;   // the thread's class-c1 items
#pragma unroll
  for (int j = 0; j < kSortIpt; ++j) {
    const bool v = t * kSortIpt + j < tile_n;
    if (v && ra[j] == A[1]) ma |= 1u << j;
    if (v && rb[j] == B[1]) mb |= 1u << j;
  }
  // class-c1 items before the thread, both keys in one word (at most
  // kSortTile each)
  const uint32_t cnt = ((uint32_t)__popc(ma) << 16) | (uint32_t)__popc(mb);
  const uint32_t incl = wave_incl(cnt, OpAdd(), 0u);
  if (lane == kWave - 1) s_w[wv] = incl;
  __syncthreads();
  uint32_t pre = incl - cnt, tot = 0;
#pragma unroll
  for (int q = 0; q < kWavesPerBlock; ++q) {
    if (q < wv) pre += s_w[q];
    tot += s_w[q];
  }
  const uint32_t n1a = tot >> 16, n1b = tot & 0xFFFFu;
  const uint32_t n0a = (uint32_t)tile_n - n1a, n0b = (uint32_t)tile_n - n1b;
  // output order in LDS: class c0 first, then class c1, each by rank
#pragma unroll
  for (int j = 0; j < kSortIpt; ++j) {
    const uint32_t pos = (uint32_t)(t * kSortIpt + j);
    if ((int)pos >= tile_n) continue;
    const uint32_t lo = (1u << j) - 1u;
    const uint32_t r1a = (pre >> 16) + (uint32_t)__popc(ma & lo);
    const uint32_t r1b = (pre & 0xFFFFu) + (uint32_t)__popc(mb & lo);
    s_out[0][((ma >> j) & 1u) ? n0a + r1a : pos - r1a] = (uint32_t)base + pos;
    s_out[1][((mb >> j) & 1u) ? n0b + r1b : pos - r1b] = (uint32_t)base + pos;
  }
  // B's rows of the table follow A's; its scanned values include A's n
  const int64_t CA = a.nclass();
  const uint32_t ga0 =
      tileoff[(int64_t)a.cls_of_raw(A[0]) * ntiles + blockIdx.x];
  const uint32_t ga1 =
      A[1] != kNone ? tileoff[(int64_t)a.cls_of_raw(A[1]) * ntiles +
                              blockIdx.x]
                    : 0u;
  const uint32_t gb0 =
      tileoff[(CA + b.cls_of_raw(B[0])) * ntiles + blockIdx.x] - (uint32_t)n;
  const uint32_t gb1 =
      B[1] != kNone
          ? tileoff[(CA + b.cls_of_raw(B[1])) * ntiles + blockIdx.x] -
                (uint32_t)n
          : 0u;
  __syncthreads();
  for (int k = t; k < tile_n; k += kBlock) {
    const uint32_t uk = (uint32_t)k;
    outA[(int64_t)(uk < n0a ? ga0 + uk : ga1 + (uk - n0a))] = s_out[0][k];
    outB[(int64_t)(uk < n0b ? gb0 + uk : gb1 + (uk - n0b))] = s_out[1][k];
  }
}

template <typename AccA, typename AccB>
__global__ __launch_bounds__(kBlock) void k_class_partition2(
    AccA a, AccB b, int64_t n, int64_t ntiles, const uint32_t* tileoff,
    uint32_t* outA, uint32_t* outB, uint32_t* coffA, uint32_t* coffB,
    const uint8_t* general) {
  if (blockIdx.x == 0) {
    // class start offsets of both sorts (B's scanned values include A's n)
    const int CA = a.nclass(), CB = b.nclass();
    for (int c = threadIdx.x; c <= CA; c += kBlock)
      coffA[c] = c < CA ? tileoff[(int64_t)c * ntiles] : (uint32_t)n;
    for (int c = threadIdx.x; c <= CB; c += kBlock)
      coffB[c] = c < CB ? tileoff[(int64_t)(CA + c) * ntiles] - (uint32_t)n
                        : (uint32_t)n;
  }
  if (!general[blockIdx.x]) return;   // done by the two-class pass
  __shared__ RankShared sh;
  __shared__ uint32_t s_val[kSortTile];
  __shared__ __attribute__((aligned(8))) uint8_t s_dig[kSortTile];
  __shared__ uint32_t s_gbase[256];
  const int64_t base = (int64_t)blockIdx.x * kSortTile;
  const int64_t tile_n = (n - base) < kSortTile ? (n - base) : kSortTile;
  uint32_t da[kSortIpt], db[kSortIpt], rank[kSortIpt];
  bool valid[kSortIpt];
  striped_classes(a, base, n, s_dig, da, valid);
  striped_classes(b, base, n, s_dig, db, valid);
  const int CA = a.nclass();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const uint32_t(&dig)[kSortIpt] = q == 0 ? da : db;
    const int C = q == 0 ? CA : b.nclass();
    tile_rank(dig, valid, rank, sh, class_bits(C));
    // B's rows of the table follow A's; its scanned values include A's n
    const int64_t row0 = q == 0 ? 0 : CA;
    const uint32_t sub = q == 0 ? 0u : (uint32_t)n;
    if ((int)threadIdx.x < C)
      s_gbase[threadIdx.x] =
          tileoff[(row0 + threadIdx.x) * ntiles + blockIdx.x] - sub;
    for (int j = 0; j < kSortIpt; ++j) {
      if (!valid[j]) continue;
      const uint32_t lp = sh.start[dig[j]] + rank[j];
      s_val[lp] = (uint32_t)(base + tile_pos(j));
      s_dig[lp] = (uint8_t)dig[j];
    }
    __syncthreads();
    uint32_t* out = q == 0 ? outA : outB;
    for (int j = 0; j < kSortIpt; ++j) {
      const int qq = j * kBlock + threadIdx.x;
      if (qq >= tile_n) continue;
      const uint32_t d = s_dig[qq];
      out[(int64_t)s_gbase[d] + (qq - sh.start[d])] = s_val[qq];
    }
    __syncthreads();
  }
}

template <typename AccA, typename AccB>
int class_sort2(const AccA& a, const AccB& b, const ClassSortLayout& L,
                uint32_t* outA, uint32_t* coffA, uint32_t* outB,
                uint32_t* coffB, hipStream_t s, const WaveClasses* wcls) {
  const int64_t n = L.n;
  const int CA = a.nclass(), CB = b.nclass();
  const int64_t T = L.ntiles;
  if (n == 0 || CA > 256 || CB > 256 || CA + CB > 256 || !wcls)
    return CHOPPER_EINVAL;
  CHOPPER_HIP(launch("sort_class_hist", k_class_hist2<AccA, AccB>,
                     dim3((unsigned)T), dim3(kBlock), s, a, b, n, T, wcls,
                     L.tilehist));
  CHOPPER_HIP(exclusive_scan<uint32_t>(L.tilehist, L.tileoff,
                                       (int64_t)(CA + CB) * T, L.scantmp,
                                       L.total, s));
  // (a byte per tile: the radix keys' space is free on this path)
  uint8_t* general = reinterpret_cast<uint8_t*>(L.key0);
  CHOPPER_HIP(launch("sort_class_partition",
                     k_class_partition2_two<AccA, AccB>, dim3((unsigned)T),
                     dim3(kBlock), s, a, b, n, T, (const uint32_t*)L.tileoff,
                     wcls, outA, outB, general));
  CHOPPER_HIP(launch("sort_class_partition", k_class_partition2<AccA, AccB>,
                     dim3((unsigned)T), dim3(kBlock), s, a, b, n, T,
                     (const uint32_t*)L.tileoff, outA, outB, coffA, coffB,
                     (const uint8_t*)general));
  return CHOPPER_OK;
}

template <typename AccA, typename AccB>
__global__ __launch_bounds__(kBlock) void k_class_verify2(
    AccA a, AccB b, int64_t n, const uint32_t* pa, const uint32_t* pb,
    uint32_t* unsorted) {
  // (stops reading once some wave has found the answer)
  if (__builtin_amdgcn_readfirstlane((int)flag_read(unsorted)) != 0) return;
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  bool bad = false;
  if (p + 1 < n) {
    const uint32_t x = pa[p], y = pa[p + 1], u = pb[p], v = pb[p + 1];
    bad = (a.cls(x) == a.cls(y) && a.time(y) < a.time(x)) ||
          (b.cls(u) == b.cls(v) && b.time(v) < b.time(u));
  }
  wave_flag_or(unsorted, bad, 1u);
}

template <typename AccA, typename AccB>
int class_verify2(const AccA& a, const AccB& b, const ClassSortLayout& L,
                  const uint32_t* outA, const uint32_t* outB, bool* sorted,
                  hipStream_t s) {
  CHOPPER_HIP(launch("sort_fill", k_fill_u32, dim3(1), dim3(kBlock), s, L.flag,
                     (int64_t)1, 0u));
  CHOPPER_HIP(launch("sort_class_verify", k_class_verify2<AccA, AccB>,
                     grid_for(L.n, kBlock), dim3(kBlock), s, a, b, L.n, outA,
                     outB, L.flag));
  uint32_t unsorted = 1;
  CHOPPER_HIP(read_back(L.flag, &unsorted, sizeof(uint32_t), s));
  *sorted = unsorted == 0;
  return CHOPPER_OK;
}

// time - tmin in the low bits, A's class at bit `tbits`, B's above it
template <typename AccA, typename AccB>
__global__ __launch_bounds__(kBlock) void k_make_keys2(
    AccA a, AccB b, int64_t n, const int64_t* mm, int tbits, uint64_t* key,
    uint32_t* val) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  key[i] = (uint64_t)(a.time(i) - mm[0]) | (uint64_t)a.cls(i) << tbits |
           (uint64_t)b.cls(i) << (tbits + 8);
  val[i] = (uint32_t)i;
}

template <typename AccA, typename AccB>
int time_sort2(const AccA& a, const AccB& b, const ClassSortLayout& L,
               uint32_t* outA, uint32_t* outB, bool* fits, hipStream_t s) {
  const int64_t n = L.n, T = L.ntiles;
  *fits = false;
  if (n == 0 || a.nclass() > 256 || b.nclass() > 256) return CHOPPER_OK;
  CHOPPER_HIP(launch("sort_init_minmax", k_init_minmax, dim3(1), dim3(1), s,
                     L.mm));
  CHOPPER_HIP(launch("sort_time_minmax", k_time_minmax<AccA>,
                     dim3((unsigned)(T < 1024 ? T : 1024)), dim3(kBlock), s,
                     a, n, L.mm));
  int64_t mm[2];
  CHOPPER_HIP(read_back(L.mm, mm, sizeof(mm), s));
  const int passes = (bitlen_u64((uint64_t)mm[1] - (uint64_t)mm[0]) + 7) / 8;
  if (passes > 6) return CHOPPER_OK;
  *fits = true;
  const int tbits = 8 * passes;
  CHOPPER_HIP(launch("sort_make_keys", k_make_keys2<AccA, AccB>,
                     grid_for(n, kBlock), dim3(kBlock), s, a, b, n,
                     (const int64_t*)L.mm, tbits, L.key0, L.val0));
  uint64_t *kin = L.key0, *kout = L.key1;
  uint32_t *vin = L.val0, *vout = L.val1;
  auto pass = [&](int shift, uint64_t* ko, uint32_t* vo) -> int {
    CHOPPER_HIP(launch("sort_digit_hist", k_digit_hist, dim3((unsigned)T),
                       dim3(kBlock), s, (const uint64_t*)kin, n, shift, T,
                       L.tilehist));
    CHOPPER_HIP(exclusive_scan<uint32_t>(L.tilehist, L.tileoff, 256 * T,
                                         L.scantmp, L.total, s));
    CHOPPER_HIP(launch("sort_digit_scatter", k_digit_scatter,
                       dim3((unsigned)T), dim3(kBlock), s,
                       (const uint64_t*)kin, (const uint32_t*)vin, n, shift, T,
                       (const uint32_t*)L.tileoff, ko, vo));
    return CHOPPER_OK;
  };
  for (int p = 0; p < passes; ++p) {
    const int rc = pass(8 * p, kout, vout);
    if (rc != CHOPPER_OK) return rc;
    uint64_t* tk = kin; kin = kout; kout = tk;
    uint32_t* tv = vin; vin = vout; vout = tv;
  }
  int rc = pass(tbits, nullptr, outA);
  if (rc == CHOPPER_OK) rc = pass(tbits + 8, nullptr, outB);
  return rc;
}

template int class_verify2<KeyRecStream, KeyRecKind>(
    const KeyRecStream&, const KeyRecKind&, const ClassSortLayout&,
    const uint32_t*, const uint32_t*, bool*, hipStream_t);
template int time_sort2<KeyRecStream, KeyRecKind>(
    const KeyRecStream&, const KeyRecKind&, const ClassSortLayout&, uint32_t*,
    uint32_t*, bool*, hipStream_t);
template int class_sort2<KeyRecStream, KeyRecKind>(
    const KeyRecStream&, const KeyRecKind&, const ClassSortLayout&, uint32_t*,
    uint32_t*, uint32_t*, uint32_t*, hipStream_t, const WaveClasses*);

template int class_sort<KeyRecStream, NoColumns>(
    const KeyRecStream&, const ClassSortLayout&, uint32_t*, uint32_t*, bool*,
    hipStream_t, int, const NoColumns&, bool*);
template int class_sort<KeyRecKind, NoColumns>(
    const KeyRecKind&, const ClassSortLayout&, uint32_t*, uint32_t*, bool*,
    hipStream_t, int, const NoColumns&, bool*);
template int class_sort<KeyMarker, MarkerColumns>(
    const KeyMarker&, const ClassSortLayout&, uint32_t*, uint32_t*, bool*,
    hipStream_t, int, const MarkerColumns&, bool*);
template int class_sort<KeySeqLabel, NoColumns>(
    const KeySeqLabel&, const ClassSortLayout&, uint32_t*, uint32_t*, bool*,
    hipStream_t, int, const NoColumns&, bool*);

}  // namespace chopper
