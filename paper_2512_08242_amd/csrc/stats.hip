// chopper_op_stats: overlap statistics and overhead breakdown of operations
// (Fig. gemm_overlap: overlap ratio against operation duration, their
// correlation, 25-75 % and min-max fills; Section VI duration breakdown,
// eqs. 6-10).
//
// The instances (compute rows of the operation level) are put in order of
// (phase, operation) group, row order kept inside a group, as compact columns
// of the overlap ratio (Q30), the time and the GPU: a counting pass writes
// every block's instances per group, which one scan turns into every block's
// first slot of each group, and a second pass writes the columns.  (The
// counting pass adds the three counters of every group in LDS on the way.)
// Blocks of 8192 instances of one group then add the exact moments in 64-bit
// words (halves of the products that would overflow) -- integer sums do not
// depend on their order, so the derived doubles are the same IEEE operations
// on the same values as anywhere else -- and build the histograms of a radix
// selection of six order statistics of the ratio per group, eleven bits and
// then ten per pass, all groups at once.  The rows of a GPU follow each
// other, so the instances of a group on one GPU are a stretch of the group's
// column; one wave, one block or the passes' blocks select that CDF's order
// statistics from it, by its length.
#include "common.h"
#include "sort.h"
#include "wave.h"

namespace chopper {

bool validate_markers(const chopper_markers* m);

namespace {

constexpr int kMaxGroups = 16 * 128;
constexpr int kStatT = 1024;
constexpr int kStatIpt = 8;
// rows per block of the two row passes: eight waves, whose 16-bit counts of
// up to 2,048 groups take 32 KB of LDS
constexpr int kRowT = 512;
constexpr int kRowSpan = kRowT * kStatIpt;
constexpr int kChunk = kStatT * kStatIpt;     // instances per block
constexpr int kRanks = 6;                     // order statistics per group
constexpr int kSums = 8;                      // exact moment words per group
constexpr int kTies = 3;                      // ranks whose times are wanted
constexpr int kTopBits = 11;                  // digits of a ratio (31 bits)
constexpr int kLowBits = 10;
constexpr int kTopBins = 1 << kTopBits;
constexpr int kLowBins = 1 << kLowBits;
constexpr int kHistW = kRanks * kLowBins;     // histogram words of a group
// Counter sums are kept in this many copies, by block: every block adds to
// every group's words, and one copy would queue them all on a few lines.
constexpr int kCopies = 32;
constexpr uint16_t kNoGroup = 0xFFFFu;
static_assert(kHistW >= kTopBins, "the first pass has one histogram");
static_assert(kMaxGroups < kNoGroup, "group numbers are 16-bit");
constexpr int kStats = 17;
typedef __int128 i128;
typedef unsigned __int128 u128;

struct StatArgs {
  const int64_t* level_offset;
  const uint32_t* path;
  const uint8_t* kind;
  const int64_t* dur;
  const int64_t* gap;
  const int64_t* ovl;
  const uint64_t* ctr;
  int64_t cap;
  int nc;
  int lv_phase, lv_op;
  const uint32_t* label;
  int64_t nm;
  int P, O;
};

__device__ inline void level_range(const StatArgs& A, int64_t& lo,
                                   int64_t& hi) {
  lo = A.level_offset[A.lv_op];
  hi = A.level_offset[A.lv_op + 1];
  if (hi > A.cap) hi = A.cap;
  if (lo > hi) lo = hi;
}

// nearest double to a 128-bit integer (round half to even): a magnitude
// below 2^63 converts directly; else its top 64 bits with every lower bit
// folded into the last one (below the double's precision there) convert
// and are scaled back exactly
__device__ inline double i128_to_double(i128 v) {
  const bool neg = v < 0;
  const u128 a = neg ? (u128)0 - (u128)v : (u128)v;
  double d;
  if ((a >> 63) == 0) {
    d = (double)(uint64_t)a;
  } else {
    const uint64_t hi64 = (uint64_t)(a >> 64);
    const int len = hi64 ? 128 - __clzll((long long)hi64) : 64;
    const int sh = len - 64;
    uint64_t top = (uint64_t)(a >> sh);
    if (sh > 0 && (a & (((u128)1 << sh) - 1)) != 0) top |= 1u;
    d = ldexp((double)top, sh);
  }
  return neg ? -d : d;
}

// add 1 for every active lane to h[bin]: one LDS add for the lanes that share
// the first one's bin, then one per lane
__device__ inline void lds_count(uint32_t* h, uint32_t bin, bool act) {
  const uint64_t m = __ballot(act);
  if (m == 0) return;
  const int ld = __ffsll((long long)m) - 1;
  const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)bin, ld);
  const uint64_t same = __ballot(act && bin == b0);
  if (lane_id() == ld) atomicAdd(&h[b0], (uint32_t)__popcll(same));
  if (act && bin != b0) atomicAdd(&h[bin], 1u);
}

// No overlap and full overlap: between them most instances, whose adds to
// their two bins would queue.  A wave counts them by ballots instead and
// adds its counts once (their digits below the first are 0).
constexpr uint32_t kFull = 1u << 30;
struct Ends {
  uint32_t none = 0, full = 0;              // (the same in every lane)
  // counts x's two, returns whether it is another instance
  __device__ bool count(uint32_t x, bool ok) {
    none += (uint32_t)__popcll(__ballot(ok && x == 0u));
    full += (uint32_t)__popcll(__ballot(ok && x == kFull));
    return ok && x != 0u && x != kFull;
  }
  __device__ void add_top(uint32_t* h) const {
    if (lane_id() == 0 && none) atomicAdd(&h[0], none);
    if (lane_id() == 1 && full) atomicAdd(&h[kFull >> (2 * kLowBits)], full);
  }
  __device__ void add_low(uint32_t* h, const uint32_t (&pre)[kRanks],
                          uint32_t own, int sh) const {
    const int hs = sh + kLowBits;
#pragma unroll
    for (int r = 0; r < kRanks; ++r) {
      if (!((own >> r) & 1u) || lane_id() != 0) continue;
      const uint32_t n = (pre[r] >> hs) == 0u             ? none
                         : (pre[r] >> hs) == (kFull >> hs) ? full : 0u;
      if (n) atomicAdd(&h[r * kLowBins], n);
    }
  }
};

// Ranks that still have the same prefix share the histogram of the first of
// them (ranks are in ascending order, so they are neighbours): bit r of the
// result is set for the ranks that have one of their own.
__device__ inline uint32_t own_hist(const uint32_t (&pre)[kRanks]) {
  uint32_t m = 1u;
#pragma unroll
  for (int r = 1; r < kRanks; ++r)
    if (pre[r] != pre[r - 1]) m |= 1u << r;
  return m;
}

// the rank whose histogram rank w uses
__device__ inline int hist_of(const uint32_t (&pre)[kRanks], int w) {
  const uint32_t m = own_hist(pre) & ((2u << w) - 1u);
  return 31 - __clz((int)m);
}

// the candidates' digits of one instance into the ranks' histograms
__device__ inline void count_digit(uint32_t* h, const uint32_t (&pre)[kRanks],
                                   uint32_t own, uint32_t x, int sh, bool ok) {
  const int hs = sh + kLowBits;
  const uint32_t dig = (x >> sh) & (uint32_t)(kLowBins - 1);
  uint32_t m = 0;
#pragma unroll
  for (int r = 0; r < kRanks; ++r)
    m |= ok && (x >> hs) == (pre[r] >> hs) ? 1u << r : 0u;
  m &= own;
  if (__ballot(m != 0) == 0) return;
#pragma unroll
  for (int r = 0; r < kRanks; ++r)
    if ((m >> r) & 1u) atomicAdd(&h[r * kLowBins + dig], 1u);
}

// CDF groups: instances, first slot and one past the last slot.
struct Cells {
  uint32_t* cnt;
  uint32_t* beg;
  uint32_t* end;
};

// A CDF group is selected by one wave, by one block or in parts by many
// blocks, by the length of its stretch and the instances in it: one wave up
// to kFewCell slots, or up to kWaveCell where there are more than kManyCells
// groups longer than kFewCell (a wave takes longer than a block, but a CU
// holds sixteen of them and one block); parts of about kPart instances above
// kLongCell instances (both sides measured: see k_cdf_cells).
constexpr int kWaveCell = 1024;
constexpr int kFewCell = 128;
constexpr uint32_t kManyCells = 512;
constexpr int kCountCopies = 16;
constexpr int64_t kLongCell = 32768;
constexpr int64_t kPart = kChunk;
constexpr int64_t kPartBlocks = 256;        // for parts, in every pass

// a CDF group in parts
struct LongCell {
  uint32_t c;
  uint32_t part0, parts;      // its parts, numbered over all of these groups
  unsigned long long ymin;
};

// the groups in parts (in no order: every group is on its own)
struct CellLists {
  unsigned long long* n_long; // number << 32 | their parts
  LongCell* lng;
  uint32_t* n_cells;          // [kCountCopies] longer than kFewCell, by block
  uint32_t* of_part;          // a part's group in parts
  uint32_t* ties;             // [3] a part
};

// ranks 0, (m-1)/4, (m-1)/2, m/2, 3(m-1)/4 and m-1
__device__ inline int64_t rank_of(int64_t m, int r) {
  return r == 0 ? 0 : r == 1 ? (m - 1) / 4 : r == 2 ? (m - 1) / 2
       : r == 3 ? m / 2 : r == 4 ? 3 * (m - 1) / 4 : m - 1;
}

// rank of tie k: 0, 2 and 3
__device__ inline int tie_rank(int k) { return k == 0 ? 0 : k + 1; }

// part `q`: its group in parts, GPU, slots [lo, hi), and are they all the
// group's?
struct Part {
  uint32_t i, h;
  bool all;
  int64_t lo, hi;
  __device__ Part(const Cells& C, const CellLists& Q, int NG, uint32_t q) {
    i = Q.of_part[q];
    const LongCell L = Q.lng[i];
    const int64_t beg = C.beg[L.c], len = (int64_t)C.end[L.c] - beg;
    const int64_t p = q - L.part0;
    h = L.c % (uint32_t)NG;
    all = len == (int64_t)C.cnt[L.c];
    lo = beg + len * p / L.parts;
    hi = beg + len * (p + 1) / L.parts;
  }
};

__global__ void k_stats_clear(int G, uint32_t* hist, int64_t nh,
                              uint64_t* csum, Cells C, int64_t NGG,
                              CellLists Q) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i0 == 0) *Q.n_long = 0;
  if (i0 < kCountCopies) Q.n_cells[i0] = 0;
  for (int64_t i = i0; i < nh; i += step) hist[i] = 0;
  for (int64_t i = i0; i < 3 * (int64_t)G * kCopies; i += step) csum[i] = 0;
  for (int64_t i = i0; i < NGG; i += step) {
    C.cnt[i] = 0;
    C.beg[i] = 0xFFFFFFFFu;
    C.end[i] = 0;
  }
}

// Group of every row of the operation level (kNoGroup when it is no
// instance: not a compute row, zero length, or a label out of range) and the
// instances per group of every block, hist[g * blocks + b].  Every column of
// a thread's eight rows is requested before the labels are looked up, the
// counters among them, so a thread waits twice, not eight times (0.103 to
// 0.064 ms on 6.1M rows with counters, 0.25 GB).
__global__ __launch_bounds__(kRowT) void k_stats_keys(StatArgs A,
                                                       uint16_t* key,
                                                       uint32_t* hist,
                                                       uint64_t* csum) {
  extern __shared__ uint64_t s_cs[];        // [3][G] counter sums, then [G]
  const int G = A.P * A.O;
  uint32_t* s_h = reinterpret_cast<uint32_t*>(s_cs + 3 * G);
  const bool ctr = A.nc >= 16;
  for (int g = threadIdx.x; g < G; g += kRowT) {
    s_h[g] = 0;
    s_cs[g] = s_cs[G + g] = s_cs[2 * G + g] = 0;
  }
  __syncthreads();
  int64_t lo, hi;
  level_range(A, lo, hi);
  const int64_t r0 = lo + (int64_t)blockIdx.x * kRowSpan + threadIdx.x;
  uint8_t kd[kStatIpt];
  int64_t du[kStatIpt];
  uint32_t mp[kStatIpt], mo[kStatIpt];
  uint64_t c0[kStatIpt], c1[kStatIpt], c2[kStatIpt];
#pragma unroll
  for (int k = 0; k < kStatIpt; ++k) {
    const int64_t r = r0 + (int64_t)k * kRowT;
    const bool ok = r < hi;
    kd[k] = ok ? A.kind[r] : (uint8_t)1;
    du[k] = ok ? A.dur[r] : 0;
    mp[k] = ok ? A.path[(int64_t)A.lv_phase * A.cap + r] : kNone;
    mo[k] = ok ? A.path[(int64_t)A.lv_op * A.cap + r] : kNone;
  }
#pragma unroll
  for (int k = 0; k < kStatIpt; ++k) {
    // GPU cycles, MFMA-busy cycles and FLOPs of the row (eqs. 7, 8, 10)
    const int64_t r = r0 + (int64_t)k * kRowT;
    const bool ok = ctr && r < hi;
    c0[k] = ok ? A.ctr[0 * A.cap + r] : 0;
    c1[k] = ok ? A.ctr[1 * A.cap + r] : 0;
    c2[k] = ok ? A.ctr[11 * A.cap + r] : 0;
  }
  uint32_t lp[kStatIpt], lo_[kStatIpt];
  bool ok[kStatIpt];
#pragma unroll
  for (int k = 0; k < kStatIpt; ++k) {
    ok[k] = kd[k] == 0 && du[k] > 0 && (int64_t)mp[k] < A.nm &&
            (int64_t)mo[k] < A.nm;
    lp[k] = ok[k] ? A.label[mp[k]] : 0u;
    lo_[k] = ok[k] ? A.label[mo[k]] : 0u;
  }
#pragma unroll
  for (int k = 0; k < kStatIpt; ++k) {
    const int64_t r = r0 + (int64_t)k * kRowT;
    ok[k] = ok[k] && lp[k] < (uint32_t)A.P && lo_[k] < (uint32_t)A.O;
    const uint32_t g = ok[k] ? lp[k] * (uint32_t)A.O + lo_[k] : 0u;
    if (r < hi) key[r - lo] = ok[k] ? (uint16_t)g : kNoGroup;
    lds_count(s_h, g, ok[k]);
    if (ctr && ok[k]) {
      atomicAdd((unsigned long long*)&s_cs[g], (unsigned long long)c0[k]);
      atomicAdd((unsigned long long*)&s_cs[G + g], (unsigned long long)c1[k]);
      atomicAdd((unsigned long long*)&s_cs[2 * G + g],
                (unsigned long long)c2[k]);
    }
  }
  __syncthreads();
  for (int g = threadIdx.x; g < G; g += kRowT) {
    hist[(int64_t)g * gridDim.x + blockIdx.x] = s_h[g];
    if (ctr && s_h[g])
      for (int f = 0; f < 3; ++f)
        atomicAdd((unsigned long long*)&csum[(blockIdx.x % kCopies * 3 + f) *
                                                 (int64_t)G + g],
                  (unsigned long long)s_cs[f * G + g]);
  }
}

// group offsets and counts from the scanned table, chunk offsets and the
// ranks to select (one block)
__device__ inline void stats_offsets(
    const uint32_t* tab, int64_t nb, const uint32_t* total, int G,
    uint32_t* cnt, uint32_t* off, uint32_t* coff, uint32_t* spre,
    int64_t* srank) {
  __shared__ uint32_t s_w[kBlock / kWave];
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  uint32_t ccarry = 0;
  for (int b0 = 0; b0 < G; b0 += kBlock) {
    const int g = b0 + t;
    uint32_t v = 0;
    if (g < G) {
      const uint32_t a = tab[(int64_t)g * nb];
      v = (g + 1 < G ? tab[(int64_t)(g + 1) * nb] : *total) - a;
      off[g] = a;
      cnt[g] = v;
    }
    const uint32_t c = (uint32_t)ceil_div(v, kChunk);
    const uint32_t cincl = wave_incl(c, OpAdd(), 0u);
    if (lane == kWave - 1) s_w[w] = cincl;
    __syncthreads();
    uint32_t cpre = ccarry, ctot = ccarry;
    for (int q = 0; q < kBlock / kWave; ++q) {
      if (q < w) cpre += s_w[q];
      ctot += s_w[q];
    }
    if (g < G) {
      coff[g] = cpre + cincl - c;
#pragma unroll
      for (int r = 0; r < kRanks; ++r) {
        spre[g * kRanks + r] = 0;
        srank[g * kRanks + r] = rank_of(v, r);
      }
    }
    ccarry = ctot;
    __syncthreads();
  }
  if (t == 0) {
    off[G] = *total;
    coff[G] = ccarry;
  }
}

// Every instance into its slot of its group, row order kept, with its ratio
// x (Q30), its time y and its GPU.  A wave takes 512 consecutive rows and
// ranks them row by row (lanes of equal groups find each other by ballots;
// the wave's running counts are in LDS); the block's table entry and the
// waves before give the slot.  A block whose rows are all on one GPU --
// every block but the few where one GPU's rows end -- notes the GPU, and the
// CDF groups get its instances from the table; another block adds them, one
// lane for the others of a row and CDF group.
__global__ __launch_bounds__(kRowT) void k_stats_scatter(
    StatArgs A, const uint8_t* gpu, int NG, const uint16_t* key,
    const uint32_t* tab, uint32_t* xs, uint64_t* ys, uint8_t* hs,
    uint16_t* bgpu, Cells C, uint32_t* status) {
  extern __shared__ uint32_t s_base[];      // [G], then u16 [waves][G]
  constexpr int kWaves = kRowT / kWave;
  const int G = A.P * A.O;
  uint16_t* s_cnt = reinterpret_cast<uint16_t*>(s_base + G);
  for (int g = threadIdx.x; g < kWaves * G; g += kRowT) s_cnt[g] = 0;
  int64_t lo, hi;
  level_range(A, lo, hi);
  const int lane = lane_id(), w = (int)(threadIdx.x / kWave);
  const int64_t b0 = lo + (int64_t)blockIdx.x * kRowSpan;
  const int64_t r0 = b0 + (int64_t)w * (kStatIpt * kWave) + lane;
  uint32_t g[kStatIpt], rank[kStatIpt], h[kStatIpt];
  int64_t du[kStatIpt], ol[kStatIpt], gp[kStatIpt];
#pragma unroll
  for (int k = 0; k < kStatIpt; ++k) {
    const int64_t r = r0 + (int64_t)k * kWave;
    const bool ok = r < hi;
    g[k] = ok ? key[r - lo] : kNoGroup;
    h[k] = ok ? gpu[r] : 0u;
    du[k] = ok ? A.dur[r] : 1;
    ol[k] = ok ? A.ovl[r] : 0;
    gp[k] = ok ? A.gap[r] : 0;
  }
  const uint32_t h0 = b0 < hi ? (uint32_t)gpu[b0] : 0u;
  __syncthreads();
  uint16_t* mine = s_cnt + w * G;
  const int nbits = 11;                     // (kMaxGroups = 2^11)
  bool other = false;
#pragma unroll
  for (int k = 0; k < kStatIpt; ++k) {
    const bool v = g[k] != kNoGroup;
    const uint64_t peers = digit_peers(g[k], v, nbits);
    const uint32_t below = lanes_below(peers);
    const uint32_t c = v ? mine[g[k]] : 0u;
    wave_sync();
    if (v && below == 0) mine[g[k]] = (uint16_t)(c + __popcll(peers));
    wave_sync();
    rank[k] = c + below;
    other = other || (v && h[k] != h0);
  }
  const bool mixed = __syncthreads_or(other);
  for (int q = threadIdx.x; q < G; q += kRowT) {
    uint32_t acc = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
      const uint32_t c = s_cnt[i * G + q];
      s_cnt[i * G + q] = (uint16_t)acc;
      acc += c;
    }
    s_base[q] = tab[(int64_t)q * gridDim.x + blockIdx.x];
  }
  if (threadIdx.x == 0) bgpu[blockIdx.x] = mixed ? kNoGroup : (uint16_t)h0;
  __syncthreads();
  bool big = false;
#pragma unroll
  for (int k = 0; k < kStatIpt; ++k) {
    if (g[k] == kNoGroup) continue;
    const uint64_t d = (uint64_t)du[k];
    const uint64_t ov = (uint64_t)ol[k];
    const uint64_t y = d + (uint64_t)gp[k];
    const uint64_t x = (ov << 30) / d;
    if ((y >> 34) != 0 || x > (1ull << 30)) big = true;
    const uint32_t pos = s_base[g[k]] + mine[g[k]] + rank[k];
    xs[pos] = x > 0x7FFFFFFFull ? 0x7FFFFFFFu : (uint32_t)x;
    ys[pos] = y;
    hs[pos] = (uint8_t)h[k];
  }
  // (by one lane for the others of a row and CDF group: instance by instance
  // a block where one GPU of one group ends took 0.3 ms)
#pragma unroll 1
  for (int k = 0; mixed && k < kStatIpt; ++k) {
    const bool v = g[k] != kNoGroup && (int)h[k] < NG;
    const uint64_t m = digit_peers(g[k], v, nbits) & digit_peers(h[k], v, 8);
    if (!v) continue;
    const int64_t c = (int64_t)g[k] * NG + h[k];
    const uint32_t pos = s_base[g[k]] + mine[g[k]] + rank[k];
    if (lanes_below(m) == 0) {
      atomicAdd(&C.cnt[c], (uint32_t)__popcll(m));
      atomicMin(&C.beg[c], pos);
    }
    if (lane == 63 - __clzll((long long)m)) atomicMax(&C.end[c], pos + 1);
  }
  if (__ballot(big) != 0 && lane == 0) atomicOr(status, CHOPPER_ST_RANGE);
}

// The CDF groups of a (phase, operation) from the blocks of rows on one GPU,
// in row order (the other blocks have added theirs); those to be selected in
// parts are listed, and those without instances get their results.  (Before
// the passes, so that those take the groups in parts along.)  One more block
// finds the offsets.
__global__ __launch_bounds__(kBlock) void k_stats_cells(
    uint32_t* cnt, uint32_t* off, uint32_t* coff, const uint32_t* total,
    int G, const uint32_t* hist, const uint32_t* tab, int64_t nb,
    const uint16_t* bgpu, int NG, Cells C, CellLists Q, uint32_t* ghist,
    uint32_t* spre, int64_t* srank, double* gout, int64_t* gcnt_out) {
  if (blockIdx.x == 0) {
    stats_offsets(tab, nb, total, G, cnt, off, coff, spre, srank);
    return;
  }
  __shared__ uint32_t s_n[256], s_b[256], s_e[256];
  __shared__ uint32_t s_nl, s_nc, s_long[256];
  static_assert(kBlock >= 256, "a thread a GPU");
  const int g = (int)blockIdx.x - 1, t = threadIdx.x;
  const int64_t c = (int64_t)g * NG + t, NGG = (int64_t)G * NG;
  const bool any = (g + 1 < G ? tab[(int64_t)(g + 1) * nb] : *total) !=
                   tab[(int64_t)g * nb];    // (uniform)
  if (t == 0) s_nl = s_nc = 0;
  if (t < NG) {
    s_n[t] = any ? C.cnt[c] : 0u;
    s_b[t] = any ? C.beg[c] : 0u;
    s_e[t] = any ? C.end[c] : 0u;
  }
  __syncthreads();
  for (int64_t b = t; any && b < nb; b += kBlock) {
    const uint32_t h = bgpu[b], n = hist[(int64_t)g * nb + b];
    if (n == 0 || h >= (uint32_t)NG) continue;
    const uint32_t at = tab[(int64_t)g * nb + b];
    atomicAdd(&s_n[h], n);
    atomicMin(&s_b[h], at);
    atomicMax(&s_e[h], at + n);
  }
  __syncthreads();
  if (t < NG && s_n[t] == 0) {
    for (int k = 0; k < 9; ++k) gout[k * NGG + c] = __builtin_nan("");
    gcnt_out[c] = 0;
  } else if (t < NG) {
    const int64_t m = s_n[t];
    C.cnt[c] = s_n[t];
    C.beg[c] = s_b[t];
    C.end[c] = s_e[t];
    if (m > kLongCell) {
      const uint32_t parts = (uint32_t)ceil_div(m, kPart);
      const unsigned long long q =
          atomicAdd(Q.n_long, 1ull << 32 | (unsigned long long)parts);
      const uint32_t i = (uint32_t)(q >> 32);
      Q.lng[i] = LongCell{(uint32_t)c, (uint32_t)q, parts, ~0ull};
      for (int r = 0; r < kRanks; ++r) {
        spre[(int64_t)(G + i) * kRanks + r] = 0;
        srank[(int64_t)(G + i) * kRanks + r] = rank_of(m, r);
      }
      s_long[atomicAdd(&s_nl, 1u)] = i;
    } else if (s_e[t] - s_b[t] > (uint32_t)kFewCell) {
      atomicAdd(&s_nc, 1u);
    }
  }
  __syncthreads();
  if (t == 0 && s_nc) atomicAdd(&Q.n_cells[blockIdx.x % kCountCopies], s_nc);
  for (uint32_t k = 0; k < s_nl; ++k) {
    const uint32_t i = s_long[k];
    const LongCell L = Q.lng[i];
    for (uint32_t q = t; q < L.parts; q += kBlock) Q.of_part[L.part0 + q] = i;
    for (int q = t; q < kHistW; q += kBlock)
      ghist[(int64_t)(G + i) * kHistW + q] = 0;
  }
}

// the group and slots of chunk c (false past the last chunk)
__device__ inline bool chunk_of(const uint32_t* coff, const uint32_t* off,
                                int G, uint32_t c, int64_t& b, int64_t& e,
                                int& g) {
  if (c >= coff[G]) return false;
  int lo = 0, hi = G;        // the last g with coff[g] <= c
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (coff[mid] <= c) lo = mid;
    else hi = mid;
  }
  g = lo;
  b = (int64_t)off[g] + (int64_t)(c - coff[g]) * kChunk;
  e = b + kChunk;
  if (e > (int64_t)off[g + 1]) e = off[g + 1];
  return true;
}

// sum of v over the block into s_part (kSums words), exact in 64 bits
__device__ inline void block_sums(uint64_t (&v)[kSums],
                                  uint64_t (*s_w)[kSums], uint64_t* dst) {
  const int w = threadIdx.x / kWave;
#pragma unroll
  for (int k = 0; k < kSums; ++k) {
    const uint64_t s = lane63(wave_incl(v[k], OpAdd(), (uint64_t)0));
    if (lane_id() == 0) s_w[w][k] = s;
  }
  __syncthreads();
  if (threadIdx.x < kSums) {
    uint64_t s = 0;
    for (int q = 0; q < (int)(blockDim.x / kWave); ++q)
      s += s_w[q][threadIdx.x];
    dst[threadIdx.x] = s;
  }
}

// One radix pass over a chunk of one group: the histogram of the digit at
// `sh` of the candidates of every rank (those whose higher digits equal the
// rank's selected prefix) into the group's global histograms.  The first
// pass has one histogram (no prefix yet) and also writes the chunk's sums of
// x, y, x^2, y^2, xy (in 32-bit halves where they would overflow); the
// counter sums come from the grouping pass.  After the eleven bits of the
// first pass few instances are candidates but for those that share one
// value (no overlap at all), which one LDS add per wave counts.
//
// The blocks after the groups' do the same for the parts of CDF groups, whose
// histograms follow the groups'; instead of the sums they keep the smallest y.
// (Code of their own: the checks a part needs, in the groups' loop, took the
// pass over 6.1M instances from 23 to 32 us.)
struct PassShared {
  uint32_t h[kHistW];
  uint64_t w[kStatT / kWave][kSums];
};
template <bool First, bool Whole>
__device__ inline void stats_pass(int64_t b, int64_t e, bool all, uint32_t h,
                                  const uint32_t* xs, const uint64_t* ys,
                                  const uint8_t* hs, const uint32_t* spre,
                                  int sh, uint32_t* gh, uint64_t* part,
                                  unsigned long long* ymin, PassShared& S) {
  constexpr int kBins = First ? kTopBins : kHistW;
  const int t = threadIdx.x;
  uint32_t x[kStatIpt];
  uint64_t y[kStatIpt];
  bool on[kStatIpt];
  auto load = [&](int64_t b0) {
#pragma unroll
    for (int k = 0; k < kStatIpt; ++k) {
      const int64_t i = b0 + (int64_t)k * kStatT + t;
      on[k] = i < e;
      x[k] = i < e ? xs[i] : 0u;
      if (First) y[k] = i < e ? ys[i] : 0ull;
    }
    if (!Whole && !all) {
#pragma unroll
      for (int k = 0; k < kStatIpt; ++k)
        on[k] = on[k] && (uint32_t)hs[b0 + (int64_t)k * kStatT + t] == h;
    }
  };
  load(b);
  for (int q = t; q < kBins; q += kStatT) S.h[q] = 0;
  uint32_t pre[kRanks];
#pragma unroll
  for (int r = 0; r < kRanks; ++r) pre[r] = First ? 0u : spre[r];
  const uint32_t own = own_hist(pre);
  __syncthreads();
  uint64_t acc[kSums], low = ~0ull;
  Ends ends;
#pragma unroll
  for (int k = 0; k < kSums; ++k) acc[k] = 0;
  auto count = [&]() {
#pragma unroll
    for (int k = 0; k < kStatIpt; ++k) {
      if (First) {
        lds_count(S.h, x[k] >> sh, ends.count(x[k], on[k]));
        if (Whole && on[k]) {
          const uint64_t xx = (uint64_t)x[k] * x[k];
          const u128 yy = (u128)y[k] * y[k];
          const uint64_t xy = (uint64_t)x[k] * y[k];
          acc[0] += x[k];
          acc[1] += y[k];
          acc[2] += xx & 0xFFFFFFFFull;
          acc[3] += xx >> 32;
          acc[4] += (uint64_t)yy & 0xFFFFFFFFull;
          acc[5] += (uint64_t)(yy >> 32);
          acc[6] += xy & 0xFFFFFFFFull;
          acc[7] += xy >> 32;
        }
        if (!Whole && on[k]) low = y[k] < low ? y[k] : low;
      } else {
        count_digit(S.h, pre, own, x[k], sh, ends.count(x[k], on[k]));
      }
    }
  };
  count();
  // (a part with other GPUs' slots between may be longer than a chunk)
  for (int64_t b0 = b + kChunk; !Whole && b0 < e; b0 += kChunk) {
    load(b0);
    count();
  }
  if (First) ends.add_top(S.h);
  else ends.add_low(S.h, pre, own, sh);
  if (First && Whole) block_sums(acc, S.w, part);
  if (First && !Whole) {
    low = lane63(wave_incl(low, OpMin(), (uint64_t)~0ull));
    if (lane_id() == 0) atomicMin(ymin, (unsigned long long)low);
  }
  __syncthreads();
  for (int q = t; q < kBins; q += kStatT)
    if (S.h[q]) atomicAdd(&gh[q], S.h[q]);
}

// (eight waves a SIMD, two blocks a CU: the scalar registers of both ways
// would leave one)
template <bool First>
__global__ __launch_bounds__(kStatT, 8) void k_stats_pass(
    const uint32_t* off, const uint32_t* coff, int G, const uint32_t* xs,
    const uint64_t* ys, const uint8_t* hs, int NG, Cells C, CellLists Q,
    uint32_t nchunk, const uint32_t* spre, int sh, uint32_t* ghist,
    uint64_t* part) {
  __shared__ PassShared S;
  if (blockIdx.x < nchunk) {
    int64_t b, e;
    int g;
    if (!chunk_of(coff, off, G, blockIdx.x, b, e, g)) return;
    stats_pass<First, true>(b, e, true, 0u, xs, ys, hs,
                            spre + (int64_t)g * kRanks, sh,
                            ghist + (int64_t)g * kHistW,
                            part + (int64_t)blockIdx.x * kSums, nullptr, S);
    return;
  }
  const uint32_t parts = (uint32_t)*Q.n_long;
  for (uint32_t q = blockIdx.x - nchunk; q < parts; q += gridDim.x - nchunk) {
    const Part X(C, Q, NG, q);
    stats_pass<First, false>(X.lo, X.hi, X.all, X.h, xs, ys, hs,
                             spre + (int64_t)(G + X.i) * kRanks, sh,
                             ghist + (int64_t)(G + X.i) * kHistW, nullptr,
                             &Q.lng[X.i].ymin, S);
    __syncthreads();                        // (S is used again)
  }
}

// The bin of a histogram of kPer * 64 counts in which rank `rank` falls and
// the counts before it, found by one wave (the same in every lane).
template <int kPer>
__device__ inline void wave_find(const uint32_t* hist, int64_t rank,
                                 uint32_t* bin, int64_t* under) {
  const int lane = lane_id();
  uint32_t h[kPer], sum = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    h[q] = hist[lane * kPer + q];
    sum += h[q];
  }
  const uint32_t incl = wave_incl(sum, OpAdd(), 0u);
  const uint64_t past = __ballot((int64_t)incl > rank);
  const int ln = past ? __ffsll((long long)past) - 1 : kWave - 1;
  int64_t u = (int64_t)incl - sum;
  uint32_t d = (uint32_t)(lane * kPer + kPer - 1);
  bool found = false;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const bool here = !found && u + (int64_t)h[q] > rank;
    if (here) d = (uint32_t)(lane * kPer + q);
    found = found || here;
    if (!found && q + 1 < kPer) u += h[q];
  }
  *bin = (uint32_t)__builtin_amdgcn_readlane((int)d, ln);
  *under = readlane64(u, ln);
}

// the digit of every rank of a group from its histogram; the prefix and
// the rank within the remaining candidates move on, and the histograms are
// cleared for the next pass (the blocks after the groups': CDF groups in
// parts)
template <bool First>
__global__ __launch_bounds__(kRanks * kWave) void k_stats_select(
    const uint32_t* cnt, int G, const unsigned long long* n_long, int sh,
    uint32_t* ghist, uint32_t* spre, int64_t* srank) {
  const int g = blockIdx.x, w = threadIdx.x / kWave, lane = lane_id();
  if (g < G ? cnt[g] == 0 : (uint32_t)(g - G) >= (uint32_t)(*n_long >> 32))
    return;
  uint32_t* gh = ghist + (int64_t)g * kHistW;
  uint32_t bin, pre[kRanks];
  int64_t under;
#pragma unroll
  for (int r = 0; r < kRanks; ++r) pre[r] = spre[g * kRanks + r];
  const int64_t rank = srank[g * kRanks + w];
  if (First) wave_find<kTopBins / kWave>(gh, rank, &bin, &under);
  else
    wave_find<kLowBins / kWave>(gh + hist_of(pre, w) * kLowBins, rank, &bin,
                                &under);
  __syncthreads();
  if (lane == 0) {
    spre[g * kRanks + w] |= bin << sh;
    srank[g * kRanks + w] = rank - under;
  }
  for (int q = threadIdx.x; q < (First ? kTopBins : kHistW);
       q += kRanks * kWave)
    gh[q] = 0;
}

struct StatOut {
  double* out;
  int64_t* cnt;
  double freq_peak, tpt_peak;
  int have_f;
  double f_gemm[128];
};

// instances of part X that tie with the ratios of the wanted ranks
__device__ inline void part_ties(const Part& X, const uint32_t* pre,
                                 const uint32_t* xs, const uint8_t* hs,
                                 uint32_t* ties) {
  __shared__ uint32_t s_n[kTies];
  if (threadIdx.x < kTies) s_n[threadIdx.x] = 0;
  __syncthreads();
  uint32_t tx[kTies], n[kTies] = {0, 0, 0};
#pragma unroll
  for (int k = 0; k < kTies; ++k)
    tx[k] = pre[(int64_t)X.i * kRanks + tie_rank(k)];
#pragma unroll 8
  for (int64_t i = X.lo + threadIdx.x; i < X.hi; i += kBlock) {
    const bool ok = X.all || (uint32_t)hs[i] == X.h;
    const uint32_t x = xs[i];
#pragma unroll
    for (int k = 0; k < kTies; ++k) n[k] += ok && x == tx[k] ? 1u : 0u;
  }
#pragma unroll
  for (int k = 0; k < kTies; ++k) {
    const uint32_t sum = lane63(wave_incl(n[k], OpAdd(), 0u));
    if (lane_id() == 0 && sum) atomicAdd(&s_n[k], sum);
  }
  __syncthreads();
  if (threadIdx.x < kTies) ties[threadIdx.x] = s_n[threadIdx.x];
  __syncthreads();                          // (s_n is used again)
}

// the exact sums of a group from its chunks and the derived values, in the
// same IEEE operations as their definition; the blocks after them count the
// wanted ties of the parts of CDF groups
__global__ __launch_bounds__(kBlock) void k_stats_final(
    const uint32_t* cnt, const uint32_t* coff, int G, int O, int nc,
    const uint64_t* part, const uint64_t* csum, const uint32_t* spre,
    int NG, Cells C, CellLists Q, const uint32_t* xs, const uint8_t* hs,
    StatOut S) {
  if ((int)blockIdx.x >= G) {
    const uint32_t parts = (uint32_t)*Q.n_long;
    for (uint32_t q = blockIdx.x - G; q < parts; q += gridDim.x - G)
      part_ties(Part(C, Q, NG, q), spre + (int64_t)G * kRanks, xs, hs,
                Q.ties + (int64_t)q * kTies);
    return;
  }
  __shared__ uint64_t s_cs[3];
  __shared__ uint64_t s_w[kBlock / kWave][kSums];
  __shared__ uint64_t s_tot[kSums];
  const int g = blockIdx.x, t = threadIdx.x;
  const int64_t m = cnt[g];
  const double nan = __builtin_nan("");
  double* o = S.out;
  if (m == 0) {
    if (t < kStats) o[(int64_t)t * G + g] = nan;
    if (t == 0) S.cnt[g] = 0;
    return;
  }
  uint64_t acc[kSums];
#pragma unroll
  for (int k = 0; k < kSums; ++k) acc[k] = 0;
  for (uint32_t c = coff[g] + t; c < coff[g + 1]; c += kBlock)
#pragma unroll
    for (int k = 0; k < kSums; ++k) acc[k] += part[(int64_t)c * kSums + k];
  block_sums(acc, s_w, s_tot);
  // counter sums: a wave a word
  const int wv = t / kWave;
  if (wv < 3) {
    const uint64_t v =
        lane_id() < kCopies
            ? csum[(lane_id() * 3 + wv) * (int64_t)G + g] : 0ull;
    const uint64_t sum = lane63(wave_incl(v, OpAdd(), (uint64_t)0));
    if (lane_id() == 0) s_cs[wv] = sum;
  }
  __syncthreads();
  if (t != 0) return;
  for (int k = 0; k < kStats; ++k) o[(int64_t)k * G + g] = nan;
  S.cnt[g] = m;
  const i128 sx = (i128)s_tot[0], sy = (i128)s_tot[1];
  const i128 sxx = ((i128)s_tot[3] << 32) + (i128)s_tot[2];
  const i128 syy = ((i128)s_tot[5] << 32) + (i128)s_tot[4];
  const i128 sxy = ((i128)s_tot[7] << 32) + (i128)s_tot[6];
  const uint64_t cyc = s_cs[0], busy = s_cs[1], flops = s_cs[2];
  const i128 im = (i128)m;
  const i128 cov = im * sxy - sx * sy;
  const i128 vx = im * sxx - sx * sx;
  const i128 vy = im * syy - sy * sy;
  const double dm = (double)m;
  if (m >= 2 && vx != 0 && vy != 0)
    o[0 * G + g] = i128_to_double(cov) /
                   sqrt(i128_to_double(vx) * i128_to_double(vy));
  double slope = nan, a = nan;
  if (vx != 0) {
    slope = i128_to_double(cov) / i128_to_double(vx);
    a = (i128_to_double(sy) - slope * i128_to_double(sx)) / dm;
  }
  o[1 * G + g] = slope;
  o[2 * G + g] = a;
  const double d0 = a, d50 = a + slope * 536870912.0;
  o[3 * G + g] = d0;
  o[4 * G + g] = d50;
  const uint32_t* v = spre + g * kRanks;
  const double q = 1.0 / 1073741824.0;
  o[5 * G + g] = (double)v[0] * q;
  o[6 * G + g] = (double)v[1] * q;
  o[7 * G + g] = ((double)v[2] + (double)v[3]) / 2.0 * q;
  o[8 * G + g] = (double)v[4] * q;
  o[9 * G + g] = (double)v[5] * q;
  const double dact = i128_to_double(sy) / dm;
  o[10 * G + g] = dact;
  const double ovr_ov = d50 / d0;
  o[14 * G + g] = ovr_ov;
  const double fg = S.have_f ? S.f_gemm[g % O] : nan;
  if (nc >= 16) {
    const double dpeak = (double)cyc * 1000.0 / S.freq_peak / dm;
    o[11 * G + g] = dpeak;
    o[12 * G + g] = 1.0 / ((double)busy / (double)cyc);
    o[13 * G + g] = ((double)flops / dm) / fg;
    o[15 * G + g] = dact / dpeak / ovr_ov;
  }
  o[16 * G + g] = fg / S.tpt_peak;
}

// ------------------------------------------------------ per-GPU overlap CDF
// Instances of (phase, operation) group g on GPU h form CDF group
// c = g * NG + h, in CDF order: ascending x, equal x in row order (time
// order on a GPU).  They lie in slots beg .. end - 1 of the group's column,
// in row order, alone there when the rows of a GPU follow each other as
// chopper_aggregate writes them; where they do not, those of the other GPUs
// are passed over.
//
// The six order statistics come from the radix selection of the pooled ones
// with its histograms in LDS; then, for the three whose times are wanted, the
// slot of the tie the rank falls on (each wave counts the ties of its part of
// the stretch in order).  One block does this for a group, reading the
// stretch about six times, from cache.  It is bound by its own latency and
// one CU's reads, so long groups go in parts beside the pooled passes, like a
// (phase, operation) of their own, and only their ties are found here; short
// ones, where a block's clears and barriers are most of it, go to a wave.
// The whole call, us, with one block for any group, with the ways below, and
// with a stable radix sort of every instance before either:  6.1M rows in 1
// group 8175, 480, 661; in 28 517, 364, 743; in 672 361, 359, 848; in 16,384
// 1745, 764, 1290; in 131,072 8936, 1005, 1853; 2.46M rows in 8,192 of 300
// 919, 460, 676; in 4,096 of 700 675, 483, 716.  Between the block and the
// parts: 46 groups of 64,000 241 and 203, 224 of 27,000 340 and 366.  Between
// the wave and the block: 128 groups of 450 109 and 100, 512 124 and 133, 1,024
// 137 and 183; of 900 134 and 104, 151 and 141, 167 and 193; of 100 84 and 88.
constexpr int kWaves = kStatT / kWave;

struct CdfArgs {
  int NG;
  int64_t NGG;
  Cells C;
  CellLists Q;
  const uint32_t* xs;
  const uint64_t* ys;
  const uint8_t* hs;
  const uint32_t* lpre;       // ratios and ranks among their ties of the
  const int64_t* lrank;       // groups in parts
  double* gout;
  int64_t* gcnt_out;
};

// Slots lo .. hi - 1 as a block walks them: wave w takes the w-th part, a
// lane four slots a round (aligned down), the next round's requested before
// this one is looked at.
struct Stretch {
  const uint32_t* xs;
  const uint8_t* hs;
  uint32_t h;
  bool all;                   // no other GPU's slots between
  int64_t lo, w0, w1;
  struct Four {
    uint32_t x[4], hw;
  };
  __device__ Stretch(const CdfArgs& A, uint32_t c, int64_t l, int64_t hi)
      : xs(A.xs), hs(A.hs), h(c % (uint32_t)A.NG),
        all(A.C.end[c] - A.C.beg[c] == A.C.cnt[c]), lo(l) {
    const int64_t a = lo & ~(int64_t)3;
    const int64_t part = ceil_div(ceil_div(hi - a, (int64_t)4), kWaves) * 4;
    w0 = a + (int64_t)(threadIdx.x / kWave) * part;
    w1 = w0 + part < hi ? w0 + part : hi;
  }
  __device__ void load(int64_t i, Four& F) const {
    F.hw = 0;
    if (i + 4 <= w1) {
      const uint4 v = *reinterpret_cast<const uint4*>(xs + i);
      F.x[0] = v.x;
      F.x[1] = v.y;
      F.x[2] = v.z;
      F.x[3] = v.w;
      if (!all) F.hw = *reinterpret_cast<const uint32_t*>(hs + i);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        F.x[q] = i + q < w1 ? xs[i + q] : 0u;
        if (!all && i + q < w1) F.hw |= (uint32_t)hs[i + q] << (8 * q);
      }
    }
  }
  // f(first slot of the lane, x, mask of the slots that count)
  template <typename F>
  __device__ void visit(F f) const {
    if (w0 >= w1) return;                              // (uniform)
    const int lane = lane_id();
    Four cur, next;
    load(w0 + 4 * lane, cur);
#pragma unroll 1
    for (int64_t c = w0; c < w1; c += 4 * kWave) {     // (uniform)
      const int64_t i = c + 4 * lane;
      load(i + 4 * kWave, next);
      uint32_t ok = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        ok |= i + q >= lo && i + q < w1 &&
                      (all || ((cur.hw >> (8 * q)) & 255u) == h)
                  ? 1u << q : 0u;
      f(i, cur.x, ok);
      cur = next;
    }
  }
  // the first pass: histogram of the top digit; returns the lane's smallest
  // time
  __device__ uint64_t count_top(const uint64_t* ys, uint32_t* hist,
                                Ends& ends) const {
    uint64_t low = ~0ull;
    visit([&](int64_t i, const uint32_t (&v)[4], uint32_t ok) {
      uint64_t y[4];
      if (i + 4 <= w1) {
        const ulonglong2 y0 = *reinterpret_cast<const ulonglong2*>(ys + i);
        const ulonglong2 y1 = *reinterpret_cast<const ulonglong2*>(ys + i + 2);
        y[0] = y0.x;
        y[1] = y0.y;
        y[2] = y1.x;
        y[3] = y1.y;
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) y[q] = i + q < w1 ? ys[i + q] : 0ull;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        lds_count(hist, v[q] >> (2 * kLowBits),
                  ends.count(v[q], (ok >> q) & 1u));
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if ((ok >> q) & 1u) low = y[q] < low ? y[q] : low;
    });
    ends.add_top(hist);
    return low;
  }
  // a later one, `ends` counted by the first
  __device__ void count_low(const uint32_t (&pre)[kRanks], int sh,
                            uint32_t* hist, const Ends& ends) const {
    const uint32_t own = own_hist(pre);
    visit([&](int64_t, const uint32_t (&v)[4], uint32_t ok) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        count_digit(hist, pre, own, v[q], sh,
                    (ok >> q) & 1u && v[q] != 0u && v[q] != kFull);
    });
    ends.add_low(hist, pre, own, sh);
  }
  __device__ void count_ties(const uint32_t (&tx)[kTies],
                             uint32_t (&n)[kTies]) const {
#pragma unroll
    for (int k = 0; k < kTies; ++k) n[k] = 0;
    visit([&](int64_t, const uint32_t (&v)[4], uint32_t ok) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int k = 0; k < kTies; ++k)
          n[k] += (ok >> q) & 1u && v[q] == tx[k] ? 1u : 0u;
    });
#pragma unroll
    for (int k = 0; k < kTies; ++k)
      n[k] = lane63(wave_incl(n[k], OpAdd(), 0u));
  }
  // The times of the ties of rank tr[k] among the block's: s_tie has every
  // wave's ties.
  __device__ void find_ties(const uint64_t* ys, const uint32_t (&tx)[kTies],
                            int64_t (&tr)[kTies],
                            const uint32_t (*s_tie)[kWaves],
                            double* s_y) const {
    const int w = (int)(threadIdx.x / kWave);
    bool here = false;
#pragma unroll
    for (int k = 0; k < kTies; ++k) {
      for (int q = 0; q < w; ++q) tr[k] -= s_tie[k][q];
      here = here || (tr[k] >= 0 && tr[k] < (int64_t)s_tie[k][w]);
    }
    if (!here) return;                                 // (uniform)
    // tr[k]: rank among the ties from here on (negative: passed)
    visit([&](int64_t i, const uint32_t (&v)[4], uint32_t ok) {
#pragma unroll
      for (int k = 0; k < kTies; ++k) {
        uint32_t tie = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          tie |= v[q] == tx[k] ? ok & (1u << q) : 0u;
        if (__ballot(tie != 0) == 0) continue;
        const uint32_t c = (uint32_t)__popc(tie);
        const uint32_t incl = wave_incl(c, OpAdd(), 0u);
        const int64_t at = tr[k] - (int64_t)(incl - c);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (((tie >> q) & 1u) &&
              at == (int64_t)__popc(tie & ((1u << q) - 1u)))
            s_y[k] = (double)ys[i + q];
        tr[k] -= lane63(incl);
      }
    });
  }
};

// results of a CDF group from its six ratios, smallest time and the times of
// ranks 0, 2 and 3, in the same IEEE operations as their definition
__device__ inline void cdf_out(const CdfArgs& A, int64_t c, const uint32_t* x,
                               uint64_t ymin, const double* y) {
  const int64_t NGG = A.NGG;
  double* gout = A.gout;
  auto xq = [&](int r) { return (double)x[r]; };
  const double q = 1.0 / 1073741824.0, dy = (double)ymin;
  A.gcnt_out[c] = A.C.cnt[c];
  gout[0 * NGG + c] = xq(0) * q;
  gout[1 * NGG + c] = xq(1) * q;
  gout[2 * NGG + c] = (xq(2) + xq(3)) / 2.0 * q;
  gout[3 * NGG + c] = xq(4) * q;
  gout[4 * NGG + c] = xq(5) * q;
  gout[5 * NGG + c] = dy;
  const double c0 = y[0] / dy;
  const double c50 = (y[1] / dy + y[2] / dy) / 2.0;
  gout[6 * NGG + c] = c0;
  gout[7 * NGG + c] = c50;
  gout[8 * NGG + c] = c50 / c0;
}

struct CellShared {
  uint32_t pre[kRanks];
  int64_t rank[kRanks];
  uint32_t tie[kTies][kWaves];
  uint64_t low[kWaves];
  double y[kTies];
  uint32_t part[kTies];
};

// one block, one CDF group
__device__ inline void cdf_block(const CdfArgs& A, uint32_t c, uint32_t* s_h,
                                 CellShared& S) {
  const int t = (int)threadIdx.x, lane = lane_id(), w = t / kWave;
  const int64_t m = A.C.cnt[c];
  const Stretch X(A, c, A.C.beg[c], A.C.end[c]);
  if (t < kRanks) {
    S.pre[t] = 0;
    S.rank[t] = rank_of(m, t);
  }
  uint64_t low = ~0ull;
  Ends ends;
  for (int pass = 0; pass < 3; ++pass) {
    const int sh = pass == 0 ? 2 * kLowBits : pass == 1 ? kLowBits : 0;
    for (int q = t; q < (pass == 0 ? kTopBins : kHistW); q += kStatT)
      s_h[q] = 0;
    __syncthreads();
    uint32_t pre[kRanks];
#pragma unroll
    for (int r = 0; r < kRanks; ++r) pre[r] = S.pre[r];
    // (the smallest time on the way)
    if (pass == 0) low = X.count_top(A.ys, s_h, ends);
    else X.count_low(pre, sh, s_h, ends);
    __syncthreads();
    if (w < kRanks) {
      uint32_t bin;
      int64_t under;
      const int64_t rank = S.rank[w];
      if (pass == 0) wave_find<kTopBins / kWave>(s_h, rank, &bin, &under);
      else
        wave_find<kLowBins / kWave>(s_h + hist_of(pre, w) * kLowBins, rank,
                                    &bin, &under);
      if (lane == 0) {
        S.pre[w] |= bin << sh;
        S.rank[w] = rank - under;
      }
    }
    __syncthreads();
  }
  // the ties of every wave, then the wanted one of each
  uint32_t tx[kTies], n[kTies];
  int64_t tr[kTies];
#pragma unroll
  for (int k = 0; k < kTies; ++k) {
    tx[k] = S.pre[tie_rank(k)];
    tr[k] = S.rank[tie_rank(k)];
  }
  X.count_ties(tx, n);
  low = lane63(wave_incl(low, OpMin(), (uint64_t)~0ull));
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < kTies; ++k) S.tie[k][w] = n[k];
    S.low[w] = low;
  }
  __syncthreads();
  X.find_ties(A.ys, tx, tr, S.tie, S.y);
  __syncthreads();
  if (t == 0) {
    uint64_t ymin = ~0ull;
    for (int q = 0; q < kWaves; ++q) ymin = S.low[q] < ymin ? S.low[q] : ymin;
    cdf_out(A, c, S.pre, ymin, S.y);
  }
  __syncthreads();                          // (S is used again)
}

// One wave, one CDF group of at most R * 64 slots, held in registers.  The
// least and the largest ratio come from the lanes' own; the others bit by
// bit, a ratio of rank k being the largest t with at most k instances below
// it, which ballots count.  (Ranking every instance against every other one
// took a call on 128 groups of 500 172 us, this 107.)
template <int R>
__device__ inline void cdf_wave(const CdfArgs& A, uint32_t c) {
  const int lane = lane_id();
  auto uni = [](uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
  };
  const uint32_t m = uni(A.C.cnt[c]), b = uni(A.C.beg[c]);
  const uint32_t len = uni(A.C.end[c]) - b;
  const uint32_t h = c % (uint32_t)A.NG;
  const bool all = len == m;
  uint32_t x[R], lo = kNone, hi = 0;
  uint64_t low = ~0ull;
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const uint32_t i = (uint32_t)(j * kWave + lane);
    const bool ok = i < len && (all || (uint32_t)A.hs[(int64_t)b + i] == h);
    x[j] = ok ? A.xs[(int64_t)b + i] : kNone;          // (above every ratio)
    const uint64_t y = ok ? A.ys[(int64_t)b + i] : ~0ull;
    low = y < low ? y : low;
    lo = x[j] < lo ? x[j] : lo;
    hi = ok && x[j] > hi ? x[j] : hi;
  }
  low = lane63(wave_incl(low, OpMin(), (uint64_t)~0ull));
  lo = lane63(wave_incl(lo, OpMin(), kNone));
  hi = lane63(wave_incl(hi, OpMax(), 0u));
  auto below = [&](uint32_t v) {
    uint32_t n = 0;
#pragma unroll
    for (int j = 0; j < R; ++j) n += (uint32_t)__popcll(__ballot(x[j] < v));
    return n;
  };
  uint32_t val[kRanks];
  const int top = 31 - __clz((int)(lo ^ hi));          // (-1: all the same)
#pragma unroll
  for (int r = 0; r < kRanks; ++r)
    val[r] = top < 0 ? lo : lo & ~(uint32_t)((2ull << top) - 1u);
  for (int bit = top; bit >= 0; --bit) {
    uint32_t t = kNone, n = 0;
#pragma unroll
    for (int r = 1; r < kRanks - 1; ++r) {
      // (ranks are ascending: equal ones so far are neighbours)
      const uint32_t v = val[r] | 1u << bit;
      if (v != t) n = below(v);
      t = v;
      if (n <= (uint32_t)rank_of(m, r)) val[r] = v;
    }
  }
  val[0] = lo;
  val[kRanks - 1] = hi;
  double y[kTies];
#pragma unroll
  for (int k = 0; k < kTies; ++k) {
    const uint32_t v = val[tie_rank(k)];
    uint32_t r = (uint32_t)rank_of(m, tie_rank(k)) - below(v);
    uint64_t at = 0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const uint64_t tie = __ballot(x[j] == v);
      const uint32_t n = (uint32_t)__popcll(tie);
      const bool here = x[j] == v && lanes_below(tie) == r;
      const uint64_t one = __ballot(here);
      if (one) {
        at = (uint64_t)b + (uint32_t)(j * kWave) + (uint32_t)__ffsll((long long)one) - 1u;
        r = kNone;                                     // (found)
      } else if (r != kNone) {
        r -= n;
      }
    }
    y[k] = (double)A.ys[at];
  }
  if (lane == 0) cdf_out(A, c, val, low, y);
}

// one block, one CDF group in parts, whose ties are counted: wave k finds the
// part with the wanted tie k and its rank there, then the block the tie
__device__ inline void cdf_long(const CdfArgs& A, uint32_t i, CellShared& S) {
  const int lane = lane_id(), w = (int)(threadIdx.x / kWave);
  const LongCell L = A.Q.lng[i];
  const uint32_t* pre = A.lpre + (int64_t)i * kRanks;
  if (w < kTies) {
    const uint32_t* ties = A.Q.ties + (int64_t)L.part0 * kTies + w;
    int64_t rank = A.lrank[(int64_t)i * kRanks + tie_rank(w)], at = -1;
    for (int64_t p0 = 0; p0 < L.parts && at < 0; p0 += kWave) {
      const int64_t p = p0 + lane;
      const uint32_t v = p < L.parts ? ties[p * kTies] : 0u;
      const uint32_t incl = wave_incl(v, OpAdd(), 0u);
      const uint64_t past = __ballot((int64_t)incl > rank);
      if (past) {
        const int ln = __ffsll((long long)past) - 1;
        at = p0 + ln;
        rank -= readlane64((int64_t)(incl - v), ln);
      } else {
        rank -= lane63(incl);
      }
    }
    if (lane == 0) {
      S.part[w] = (uint32_t)(at < 0 ? 0 : at);
      S.rank[w] = rank;
    }
  }
  __syncthreads();
  uint32_t tx[kTies], n[kTies];
#pragma unroll
  for (int k = 0; k < kTies; ++k) tx[k] = pre[tie_rank(k)];
  for (int k = 0; k < kTies; ++k) {
    const Part P(A.C, A.Q, A.NG, L.part0 + S.part[k]);
    const Stretch X(A, L.c, P.lo, P.hi);
    // (the other two are beyond any part)
    int64_t tr[kTies];
#pragma unroll
    for (int j = 0; j < kTies; ++j)
      tr[j] = j == k ? S.rank[k] : (int64_t)1 << 62;
    X.count_ties(tx, n);
    if (lane == 0)
#pragma unroll
      for (int j = 0; j < kTies; ++j) S.tie[j][w] = n[j];
    __syncthreads();
    X.find_ties(A.ys, tx, tr, S.tie, S.y);
    __syncthreads();
  }
  if (threadIdx.x == 0) cdf_out(A, L.c, pre, L.ymin, S.y);
  __syncthreads();                          // (S is used again)
}

// The first `long_blocks` blocks take the groups in parts, the next
// `cell_blocks` those of a block, the others those of a wave.
__global__ __launch_bounds__(kStatT) void k_cdf_cells(CdfArgs A,
                                                      uint32_t long_blocks,
                                                      uint32_t cell_blocks) {
  __shared__ uint32_t s_h[kHistW];
  __shared__ CellShared S;
  __shared__ uint32_t s_list[kStatT], s_n;
  uint32_t b = blockIdx.x;
  if (b < long_blocks) {
    const uint32_t n = (uint32_t)(*A.Q.n_long >> 32);
    for (uint32_t i = b; i < n; i += long_blocks) cdf_long(A, i, S);
    return;
  }
  b -= long_blocks;
  // a block's groups: every `step`-th, those of its way listed first
  const bool by_block = b < cell_blocks;
  uint32_t step = cell_blocks;
  if (!by_block) {
    b -= cell_blocks;
    step = gridDim.x - long_blocks - cell_blocks;
  }
  const int64_t c = b + (int64_t)threadIdx.x * step;
  const bool on = c < A.NGG;
  const int64_t m = on ? A.C.cnt[c] : 0;
  const int64_t len = on ? (int64_t)A.C.end[c] - (int64_t)A.C.beg[c] : 0;
  const uint32_t some = lane_id() < kCountCopies ? A.Q.n_cells[lane_id()] : 0u;
  const int64_t most = lane63(wave_incl(some, OpAdd(), 0u)) > kManyCells
                           ? kWaveCell : kFewCell;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  if (m > 0 && m <= kLongCell && (len > most) == by_block)
    s_list[atomicAdd(&s_n, 1u)] = (uint32_t)c;
  __syncthreads();
  const int n = (int)s_n;
  if (by_block) {
    for (int i = 0; i < n; ++i) cdf_block(A, s_list[i], s_h, S);
    return;
  }
  const int w = (int)(threadIdx.x / kWave);
  for (int i = w; i < n; i += kWaves) {
    const uint32_t c1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_list[i]);
    const uint32_t len = A.C.end[c1] - A.C.beg[c1];
    if (len <= kFewCell) cdf_wave<kFewCell / kWave>(A, c1);
    else if (len <= 8 * kWave) cdf_wave<8>(A, c1);
    else cdf_wave<kWaveCell / kWave>(A, c1);
  }
}

// eq. 9 per (phase, operation), one wave each: the median over its GPUs with
// instances of their D_50% / D_0%; eq. 10 divides by it (overwrites columns
// 14 and 15 of k_stats_final).  Lanes hold four GPUs each; a value's place
// in ascending order is the number of values below it, or equal and before.
__global__ __launch_bounds__(kWave) void k_cdf_pool(int G, int NG, int nc,
                                                    const int64_t* gcnt,
                                                    const double* gout,
                                                    int64_t NGG, double* out) {
  __shared__ double s_v[256];
  __shared__ double s_mid[2];
  const int g = (int)blockIdx.x, lane = lane_id();
  const int64_t c0 = (int64_t)g * NG;
  int k = 0;
  for (int h0 = 0; h0 < NG; h0 += kWave) {
    const int h = h0 + lane;
    const bool on = h < NG && gcnt[c0 + h] != 0;
    const uint64_t m = __ballot(on);
    if (on) s_v[k + (int)lanes_below(m)] = gout[8 * NGG + c0 + h];
    k += (int)__popcll(m);
  }
  if (lane < 2) s_mid[lane] = __builtin_nan("");
  __syncthreads();
  for (int i = lane; i < k; i += kWave) {
    const double x = s_v[i];
    int at = 0;
    for (int j = 0; j < k; ++j) {
      const double y = s_v[j];
      at += y < x || (y == x && j < i) ? 1 : 0;
    }
    if (at == (k - 1) / 2) s_mid[0] = x;
    if (at == k / 2) s_mid[1] = x;
  }
  __syncthreads();
  if (lane != 0) return;
  const double ovr = k > 0 ? (s_mid[0] + s_mid[1]) / 2.0 : __builtin_nan("");
  out[14 * (int64_t)G + g] = ovr;
  if (nc >= 16)
    out[15 * (int64_t)G + g] =
        out[10 * (int64_t)G + g] / out[11 * (int64_t)G + g] / ovr;
}

}  // namespace

extern "C" int chopper_op_stats(const chopper_rows* rows, int32_t depth,
                                int32_t n_counters,
                                const chopper_markers* mk,
                                const chopper_stats_spec* spec, double* out,
                                int64_t* cnt, double* gpu_out,
                                int64_t* gpu_cnt, void* scratch,
                                size_t* scratch_bytes, uint32_t* status,
                                void* stream) {
  if (!rows || !spec || !mk || !validate_markers(mk) || !scratch_bytes ||
      !out || !cnt)
    return CHOPPER_EINVAL;
  const int P = spec->n_phases, O = spec->n_ops, NG = spec->n_gpus;
  if (NG < 1 || NG > 256) return CHOPPER_EINVAL;
  if (depth < 1 || depth > mk->depth || spec->phase_level < 0 ||
      spec->phase_level >= depth || spec->op_level < 0 ||
      spec->op_level >= depth || P < 1 || P > 16 || O < 1 || O > 128 ||
      n_counters < 0 || n_counters > 16 || rows->cap < 0 ||
      rows->cap >= (int64_t)0xFFFFFFFF || !rows->level_offset)
    return CHOPPER_EINVAL;
  if (rows->cap > 0 && (!rows->path || !rows->kind || !rows->dur ||
                        !rows->gap || !rows->ovl || !rows->gpu ||
                        (n_counters > 0 && !rows->ctr)))
    return CHOPPER_EINVAL;
  if (mk->n > 0 && !mk->label) return CHOPPER_EINVAL;
  const int G = P * O;
  const int64_t cap = rows->cap;
  const int64_t nchunk = ceil_div(cap, kChunk) + G;
  const int64_t nh = (int64_t)G * kHistW;
  const int64_t NGG = (int64_t)G * NG;      // CDF groups
  const int64_t nb = ceil_div(cap > 0 ? cap : 1, (int64_t)kRowSpan);
  // CDF groups in parts, and their parts, at most
  const int64_t max_long = cap / (kLongCell + 1);
  const int64_t max_parts = max_long > 0 ? cap / kPart + max_long : 0;
  struct Bufs {
    uint16_t* key;
    uint8_t* hs;
    uint16_t* bgpu;
    uint32_t *gcnt, *off, *coff, *xs, *ghist, *spre, *hist, *tab, *scan, *tot;
    uint64_t *ys, *csum, *part;
    int64_t* srank;
    Cells cells;
    CellLists lists;
    double* gout;
    int64_t* gcnt_out;
  } B;
  auto layout = [&](Scratch& sc) {
    B.key = sc.take<uint16_t>(cap);
    B.hs = sc.take<uint8_t>(cap);
    B.bgpu = sc.take<uint16_t>(nb);
    B.gcnt = sc.take<uint32_t>(G);
    B.off = sc.take<uint32_t>(G + 1);
    B.coff = sc.take<uint32_t>(G + 1);
    B.xs = sc.take<uint32_t>(cap);
    B.ys = sc.take<uint64_t>(cap);
    B.csum = sc.take<uint64_t>(3 * (int64_t)G * kCopies);
    B.part = sc.take<uint64_t>(nchunk * kSums);
    B.ghist = sc.take<uint32_t>(nh + max_long * kHistW);
    B.spre = sc.take<uint32_t>((G + max_long) * kRanks);
    B.srank = sc.take<int64_t>((G + max_long) * kRanks);
    B.hist = sc.take<uint32_t>(G * nb);
    B.tab = sc.take<uint32_t>(G * nb);
    B.scan = sc.take<uint32_t>(scan_scratch_elems(G * nb));
    B.tot = sc.take<uint32_t>(1);
    B.cells.cnt = sc.take<uint32_t>(NGG);
    B.cells.beg = sc.take<uint32_t>(NGG);
    B.cells.end = sc.take<uint32_t>(NGG);
    B.lists.n_long = sc.take<unsigned long long>(1);
    B.lists.n_cells = sc.take<uint32_t>(kCountCopies);
    B.lists.lng = sc.take<LongCell>(max_long);
    B.lists.of_part = sc.take<uint32_t>(max_parts);
    B.lists.ties = sc.take<uint32_t>(max_parts * kTies);
    // (per-GPU results in scratch when the caller passes no arrays)
    B.gout = gpu_out ? gpu_out : sc.take<double>(9 * NGG);
    B.gcnt_out = gpu_cnt ? gpu_cnt : sc.take<int64_t>(NGG);
  };
  Scratch probe(nullptr);
  layout(probe);
  int rc = scratch_check(scratch, scratch_bytes, probe.used);
  if (rc != 0) return rc > 0 ? CHOPPER_OK : rc;
  if (!status) return CHOPPER_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  Scratch sc(scratch);
  layout(sc);
  StatArgs A{rows->level_offset, rows->path, rows->kind, rows->dur,
             rows->gap, rows->ovl, rows->ctr, cap, n_counters,
             spec->phase_level, spec->op_level, mk->label, mk->n, P, O};
  StatOut S{out, cnt, spec->freq_peak_mhz, spec->tpt_peak,
            spec->f_gemm != nullptr, {0}};
  for (int o = 0; o < O && spec->f_gemm; ++o) S.f_gemm[o] = spec->f_gemm[o];
  int64_t nclear = nh > NGG ? nh : NGG;
  if (nclear > (int64_t)4096 * kBlock) nclear = (int64_t)4096 * kBlock;
  CHOPPER_HIP(launch("stats_clear", k_stats_clear, grid_for(nclear, kBlock),
                     dim3(kBlock), s, G, B.ghist, nh, B.csum, B.cells, NGG,
                     B.lists));
  const dim3 rb((unsigned)nb);
  CHOPPER_HIP(launch_shm("stats_keys", k_stats_keys, rb, dim3(kRowT),
                         (size_t)G * 28, s, A, B.key, B.hist, B.csum));
  CHOPPER_HIP(exclusive_scan<uint32_t>(B.hist, B.tab, G * nb, B.scan, B.tot,
                                       s));
  const size_t lds = (size_t)G * 4 + (size_t)G * 2 * (kRowT / kWave);
  CHOPPER_HIP(launch_shm("stats_scatter", k_stats_scatter, rb, dim3(kRowT),
                         lds, s, A, rows->gpu, NG, (const uint16_t*)B.key,
                         (const uint32_t*)B.tab, B.xs, B.ys, B.hs, B.bgpu,
                         B.cells, status));
  CHOPPER_HIP(launch("stats_cells", k_stats_cells, dim3((unsigned)G + 1),
                     dim3(kBlock), s, B.gcnt, B.off, B.coff,
                     (const uint32_t*)B.tot, G,
                     (const uint32_t*)B.hist, (const uint32_t*)B.tab, nb,
                     (const uint16_t*)B.bgpu, NG, B.cells, B.lists, B.ghist,
                     B.spre, B.srank, B.gout, B.gcnt_out));
  auto at_most = [](int64_t n, int64_t most) {
    return (unsigned)(n < most ? n : most);
  };
  // (blocks for parts that there are not cost their launch: 1,100 of them
  // 5 us a pass)
  const unsigned parts = at_most(max_parts, kPartBlocks);
  for (int pass = 0; pass < 3; ++pass) {
    const int sh = pass == 0 ? 2 * kLowBits : pass == 1 ? kLowBits : 0;
    CHOPPER_HIP(launch("stats_pass",
                       pass == 0 ? k_stats_pass<true> : k_stats_pass<false>,
                       dim3(parts + (unsigned)nchunk), dim3(kStatT), s,
                       (const uint32_t*)B.off, (const uint32_t*)B.coff, G,
                       (const uint32_t*)B.xs, (const uint64_t*)B.ys,
                       (const uint8_t*)B.hs, NG, B.cells, B.lists,
                       (uint32_t)nchunk,
                       (const uint32_t*)B.spre, sh, B.ghist, B.part));
    CHOPPER_HIP(launch("stats_select",
                       pass == 0 ? k_stats_select<true>
                                 : k_stats_select<false>,
                       dim3((unsigned)(G + max_long)), dim3(kRanks * kWave),
                       s, (const uint32_t*)B.gcnt, G,
                       (const unsigned long long*)B.lists.n_long, sh, B.ghist,
                       B.spre, B.srank));
  }
  CHOPPER_HIP(launch("stats_final", k_stats_final, dim3((unsigned)G + parts),
                     dim3(kBlock), s, (const uint32_t*)B.gcnt,
                     (const uint32_t*)B.coff, G, O, n_counters,
                     (const uint64_t*)B.part, (const uint64_t*)B.csum,
                     (const uint32_t*)B.spre, NG, B.cells, B.lists,
                     (const uint32_t*)B.xs, (const uint8_t*)B.hs, S));
  // per-GPU overlap CDFs, and eq. 9 / eq. 10 from them
  const CdfArgs K{NG, NGG, B.cells, B.lists, B.xs, B.ys, B.hs,
                  B.spre + (int64_t)G * kRanks, B.srank + (int64_t)G * kRanks,
                  B.gout, B.gcnt_out};
  const unsigned long_blocks = at_most(max_long, 256);
  // (a thread lists a group: 1,024 blocks of either kind take the largest
  // call's 2^19)
  static_assert((int64_t)kMaxGroups * 256 <= 1024 * kStatT, "groups a block");
  const unsigned cell_blocks = at_most(NGG, 1024);
  const unsigned wave_blocks = at_most(ceil_div(NGG, (int64_t)kWaves), 1024);
  CHOPPER_HIP(launch("stats_cdf", k_cdf_cells,
                     dim3(long_blocks + cell_blocks + wave_blocks),
                     dim3(kStatT), s, K, long_blocks, cell_blocks));
  CHOPPER_HIP(launch("stats_cdf", k_cdf_pool, dim3((unsigned)G), dim3(kWave),
                     s, G, NG, n_counters, (const int64_t*)B.gcnt_out,
                     (const double*)B.gout, NGG, out));
  return CHOPPER_OK;
}

}  // namespace chopper
