// Shared device primitives and host plumbing of libchopper (gfx950).
//
// Wave64 scans are built on __shfl_up (DPP / ds_bpermute underneath); block
// scans combine the per-wave totals through LDS.  All integer work, so every
// reduction is order-independent and exact.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include "../../include/chopper.h"

namespace chopper {

constexpr int kWave = 64;
constexpr int kBlock = 256;               // threads per block, 4 waves
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr int64_t kI64Max = INT64_MAX;
constexpr int64_t kI64Min = INT64_MIN;

__host__ __device__ inline int kind_of(uint32_t cls) {
  return (cls == 5u || cls == 6u) ? 1 : 0;
}

__host__ __device__ inline int64_t ceil_div(int64_t a, int64_t b) {
  return (a + b - 1) / b;
}

// ---------------------------------------------------------------------------
// Wave and block scans
// ---------------------------------------------------------------------------
struct OpAdd {
  template <typename T>
  __device__ T operator()(T a, T b) const { return a + b; }
};
struct OpMin {
  template <typename T>
  __device__ T operator()(T a, T b) const { return a < b ? a : b; }
};
struct OpMax {
  template <typename T>
  __device__ T operator()(T a, T b) const { return a > b ? a : b; }
};

template <typename T>
__device__ inline T shfl_up(T v, int d) {
  return __shfl_up(v, d, kWave);
}

// Inclusive scan across the 64 lanes of a wave.
template <typename T, typename Op>
__device__ inline T wave_inclusive(T v, Op op) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    T u = shfl_up(v, d);
    if (lane >= d) v = op(u, v);
  }
  return v;
}

// Block-wide exclusive scan (kBlock threads).  `identity` is the value of the
// empty prefix; returns the exclusive value and writes the block total.
template <typename T, typename Op>
__device__ inline T block_exclusive(T v, Op op, T identity, T* total) {
  __shared__ T wave_tot[kWavesPerBlock];
  const int lane = threadIdx.x & (kWave - 1);
  const int w = threadIdx.x / kWave;
  T inc = wave_inclusive(v, op);
  if (lane == kWave - 1) wave_tot[w] = inc;
  __syncthreads();
  T pre = identity;
  T tot = identity;
#pragma unroll
  for (int i = 0; i < kWavesPerBlock; ++i) {
    if (i < w) pre = op(pre, wave_tot[i]);
    tot = op(tot, wave_tot[i]);
  }
  T prev = shfl_up(inc, 1);                // inclusive value of lane - 1
  T exc = (lane == 0) ? pre : op(pre, prev);
  __syncthreads();
  if (total) *total = tot;
  return exc;
}

// Pair scanned lexicographically by (seg, val) with max: the running maximum
// restricted to the last segment seen, since segment ids never decrease along
// a scan.
struct SegMax {
  uint32_t seg;
  int64_t val;
};
struct OpSegMax {
  __device__ SegMax operator()(SegMax a, SegMax b) const {
    if (a.seg != b.seg) return a.seg > b.seg ? a : b;
    return a.val >= b.val ? a : b;
  }
};
template <>
__device__ inline SegMax shfl_up<SegMax>(SegMax v, int d) {
  SegMax r;
  r.seg = __shfl_up(v.seg, d, kWave);
  r.val = __shfl_up(v.val, d, kWave);
  return r;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
#define CHOPPER_HIP(x)                      \
  do {                                      \
    hipError_t e_ = (x);                    \
    if (e_ != hipSuccess) return CHOPPER_EHIP; \
  } while (0)

// Carves 256-byte-aligned sub-buffers out of the caller's scratch.  With a
// null base it only measures.
struct Scratch {
  char* base;
  size_t used = 0;
  explicit Scratch(void* b) : base(static_cast<char*>(b)) {}
  template <typename T>
  T* take(int64_t count) {
    size_t bytes = (size_t)(count > 0 ? count : 1) * sizeof(T);
    size_t off = (used + 255) & ~(size_t)255;
    used = off + bytes;
    return base ? reinterpret_cast<T*>(base + off) : nullptr;
  }
};

// Scratch protocol shared by all entry points: returns 1 when the call was a
// size query (already answered), 0 when the caller's buffer is large enough,
// or a negative code.
inline int scratch_check(void* scratch, size_t* scratch_bytes, size_t need) {
  if (!scratch_bytes) return CHOPPER_EINVAL;
  if (!scratch) { *scratch_bytes = need; return 1; }
  if (*scratch_bytes < need) return CHOPPER_ESCRATCH;
  if (((uintptr_t)scratch & 255) != 0) return CHOPPER_EINVAL;
  return 0;
}

// Kernel timing hook (chopper_time_kernel).
struct TimerHook {
  const char* name = nullptr;
  hipEvent_t start = nullptr, stop = nullptr;
};
TimerHook& timer_hook();

template <typename Kern, typename... Args>
inline hipError_t launch(const char* name, Kern kern, dim3 grid, dim3 block,
                         hipStream_t s, Args... args) {
  if (grid.x == 0 || grid.y == 0 || grid.z == 0) return hipSuccess;
  TimerHook& h = timer_hook();
  bool timed = h.name && strcmp(h.name, name) == 0;
  if (timed) (void)hipEventRecord(h.start, s);
  hipLaunchKernelGGL(kern, grid, block, 0, s, args...);
  hipError_t e = hipGetLastError();
  if (timed) (void)hipEventRecord(h.stop, s);
  return e;
}

// Copies `bytes` of device memory at `dev` to `host` once the work queued
// on `s` before it is done, and returns when they are there (polling, not
// the runtime's blocking wait).
hipError_t read_back(const void* dev, void* host, size_t bytes, hipStream_t s);

// The same in two halves: read_back_start queues the copy (at most
// kReadBackMax bytes) into pinned memory that the library keeps and records
// an event after it; work queued on `s` afterwards runs while the host
// waits in read_back_finish, which polls that event only and then copies
// the value to `host`.  Every start is followed by one finish on the same
// host thread.  Without a free pinned slot the copy is done at once by
// read_back_start (the stream drained), and the finish only hands it over.
// A read-back left unfinished (an early error return) waits for its copy
// and frees its slot when it goes out of scope.
constexpr size_t kReadBackMax = 256;
struct ReadBack {
  void* slot = nullptr;
  size_t bytes = 0;
  hipError_t err = hipSuccess;
  alignas(8) unsigned char now[kReadBackMax];
  ReadBack() = default;
  ReadBack(const ReadBack&) = delete;
  ReadBack& operator=(const ReadBack&) = delete;
  ~ReadBack();
};
hipError_t read_back_start(const void* dev, size_t bytes, hipStream_t s,
                           ReadBack* rb);
hipError_t read_back_finish(ReadBack* rb, void* host);
// The first half without a launch of its own, for a kernel that stores the
// words itself: read_back_open hands out the slot's device address (null
// when there is none), which the kernel writes beside `dev` (store_host
// below); read_back_close after the launch records the event, or reads
// `dev` at once when there was no slot.
uint32_t* read_back_open(size_t bytes, ReadBack* rb);
hipError_t read_back_close(const void* dev, hipStream_t s, ReadBack* rb);

// One word of a read-back into the slot (host memory), visible to the host
// before the kernel, and the event after it, ends.
__device__ inline void store_host(uint32_t* slot, int i, uint32_t v) {
  if (slot) {
    slot[i] = v;
    __threadfence_system();
  }
}
__device__ inline void store_host(uint32_t* slot, int i, int64_t v) {
  if (slot) {
    reinterpret_cast<int64_t*>(slot)[i] = v;
    __threadfence_system();
  }
}

// Is this the last block of a launch of `blocks` blocks to get here (the
// same in every thread)?  Everything the other blocks stored before is then
// visible.  `count` is zero before the launch.  A kernel whose blocks each
// leave a small result ends this way with the steps that combine them,
// which saves a launch or more.  It costs the fence, 3 us beside 120 blocks,
// so it pays where it stands for two launches, not for one.
// Every thread of every block comes here.
__device__ inline bool last_block(uint32_t* count, uint32_t blocks) {
  __shared__ uint32_t s_last;
  // (every wave's stores have reached the L2 before one wave writes it back)
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    s_last = atomicAdd(count, 1u) == blocks - 1u;
  }
  __syncthreads();
  const bool last = s_last != 0;
  if (last) __threadfence();
  return last;
}

// Exclusive prefix sums of in[0 .. n) by one block of kBlock threads, for
// small n (16-byte loads and stores; in and out 16-byte aligned and readable
// and writable up to a multiple of four); returns the total in every thread.
__device__ inline uint32_t block_scan_array(const uint32_t* in, uint32_t* out,
                                            int64_t n) {
  constexpr int kQ = 4;
  uint32_t carry = 0;
  for (int64_t b = 0; b < n; b += (int64_t)kBlock * kQ * 4) {
    const int64_t i0 = b + (int64_t)threadIdx.x * (kQ * 4);
    uint32_t v[kQ * 4], acc = 0;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      uint4 x = make_uint4(0u, 0u, 0u, 0u);
      if (i0 + 4 * q < n) x = *reinterpret_cast<const uint4*>(in + i0 + 4 * q);
      v[4 * q] = x.x;
      v[4 * q + 1] = i0 + 4 * q + 1 < n ? x.y : 0u;
      v[4 * q + 2] = i0 + 4 * q + 2 < n ? x.z : 0u;
      v[4 * q + 3] = i0 + 4 * q + 3 < n ? x.w : 0u;
    }
#pragma unroll
    for (int q = 0; q < kQ * 4; ++q) {
      const uint32_t x = v[q];
      v[q] = acc;
      acc += x;
    }
    uint32_t tot;
    const uint32_t pre = block_exclusive(acc, OpAdd(), 0u, &tot) + carry;
#pragma unroll
    for (int q = 0; q < kQ; ++q)
      if (i0 + 4 * q < n)
        *reinterpret_cast<uint4*>(out + i0 + 4 * q) =
            make_uint4(pre + v[4 * q], pre + v[4 * q + 1], pre + v[4 * q + 2],
                       pre + v[4 * q + 3]);
    carry += tot;
  }
  return carry;
}
// the largest table a kernel's last block scans itself: three rounds of the
// loop above, which is what the scan's launches take
constexpr int64_t kTailScan = 12288;

// the same as launch() with `shm` bytes of dynamic LDS
template <typename Kern, typename... Args>
inline hipError_t launch_shm(const char* name, Kern kern, dim3 grid,
                             dim3 block, size_t shm, hipStream_t s,
                             Args... args) {
  if (grid.x == 0 || grid.y == 0 || grid.z == 0) return hipSuccess;
  TimerHook& h = timer_hook();
  bool timed = h.name && strcmp(h.name, name) == 0;
  if (timed) (void)hipEventRecord(h.start, s);
  hipLaunchKernelGGL(kern, grid, block, shm, s, args...);
  hipError_t e = hipGetLastError();
  if (timed) (void)hipEventRecord(h.stop, s);
  return e;
}

inline dim3 grid_for(int64_t items, int per_block) {
  int64_t b = ceil_div(items, per_block);
  return dim3((unsigned)(b > 0 ? b : 0));
}

// ---------------------------------------------------------------------------
// Device-wide exclusive scans (three passes: tile totals, scan of totals in
// one block, rescan of each tile with its prefix).
// ---------------------------------------------------------------------------
int64_t scan_scratch_elems(int64_t n);   // number of T slots needed
template <typename T>
hipError_t exclusive_scan(const T* in, T* out, int64_t n, T* tmp, T* total,
                          hipStream_t s);
// the same over the first min(n, *n_dev) elements (n_dev on the device)
template <typename T>
hipError_t exclusive_scan(const T* in, T* out, int64_t n, const uint32_t* n_dev,
                          T* tmp, T* total, hipStream_t s);

// Sorts (key u64) stably and writes the permutation of 0..n-1.
// Implemented in sort.hip.
struct SortPlan;

}  // namespace chopper
