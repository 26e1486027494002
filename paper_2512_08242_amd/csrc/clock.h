// Per-GPU clock transform on the device (Section III-B alignment): shared by
// the alignment of records and markers and of kernel dispatch times.
#pragma once

#include "common.h"

namespace chopper {

struct ClockDev {
  int64_t x0, c, d;
};

// The clock table of a launch: up to kArgClocks GPUs travel with the kernel's
// arguments (a copy into device memory before it took 2 us of device time
// and twice that on the host, a quarter of a launch split of 100,000
// records), more come from device memory.  Kernels put it into LDS first.
constexpr int kArgClocks = 64;
constexpr int kMaxClocks = 256;
struct ClockArgs {
  ClockDev c[kArgClocks];
  const ClockDev* tab;        // null: c
};

// Arguments of G <= kMaxClocks clocks; `dev` (room for G) is used when they
// are more than travel with the launch.
inline hipError_t clock_args(const chopper_clock* clocks, int G, ClockDev* dev,
                             hipStream_t s, ClockArgs* A) {
  memset(A, 0, sizeof(*A));
  if (G <= kArgClocks) {
    for (int g = 0; g < G; ++g)
      A->c[g] = ClockDev{clocks[g].x0, clocks[g].c, clocks[g].d_q48};
    return hipSuccess;
  }
  ClockDev all[kMaxClocks];
  for (int g = 0; g < G; ++g)
    all[g] = ClockDev{clocks[g].x0, clocks[g].c, clocks[g].d_q48};
  A->tab = dev;
  // (a copy from pageable memory is staged before the call returns)
  return hipMemcpyAsync(dev, all, sizeof(ClockDev) * G, hipMemcpyHostToDevice,
                        s);
}

// table[g] for g < G, by the whole block (with its barrier)
__device__ inline void clocks_to_lds(const ClockArgs& A, int G,
                                     ClockDev* table) {
  for (int g = (int)threadIdx.x; g < G; g += (int)blockDim.x)
    table[g] = A.tab ? A.tab[g] : A.c[g & (kArgClocks - 1)];
  __syncthreads();
}

// t + c + floor((t - x0) * d / 2^48): the signed 128-bit product is formed
// from __mul64hi and the low 64-bit product; the floor division by 2^48 is
// the arithmetic shift of that 128-bit value.
__device__ inline int64_t align_time(int64_t t, ClockDev k) {
  const int64_t u = t - k.x0;
  const int64_t hi = __mul64hi(u, k.d);
  const uint64_t lo = (uint64_t)u * (uint64_t)k.d;
  const int64_t q = (int64_t)(((uint64_t)hi << 16) | (lo >> 48));
  return t + k.c + q;
}

__device__ inline bool out_of_range(int64_t t) {
  const int64_t lim = (int64_t)1 << 62;
  return t >= lim || t <= -lim;
}

}  // namespace chopper
