// Host read-back of small device values (flags and counts that size later
// launches), in two halves so that the caller can queue more work on the
// stream before it waits: a one-wave kernel on the stream stores the words
// into a slot of pinned host memory (mapped for the device; a runtime copy
// there would go through the copy engine, which later kernels of the stream
// wait for), an event is recorded after it, and the wait polls that event.
// The slots (a few per device, each with its event) are created on first
// use and kept for the life of the process; when none is free, or pinned
// memory cannot be had, the read-back is done at once into the caller's
// memory, waiting for the whole stream.
#include <chrono>
#include <cstring>
#include <mutex>

#include "common.h"

namespace chopper {

namespace {

// a stream that has not drained after this long is reported as an error
constexpr double kReadBackLimitSeconds = 120.0;
constexpr int kRbDevices = 64;
constexpr int kRbSlots = 4;
static_assert(kReadBackMax / 4 <= kWave, "one word per lane");

struct RbSlot {
  void* pin = nullptr;
  uint32_t* dpin = nullptr;   // its device address
  hipEvent_t ev = nullptr;
  bool busy = false;
  bool failed = false;   // creation failed: never used
};

std::mutex g_rb_mu;
RbSlot g_rb[kRbDevices][kRbSlots];

// Polls until `done` stops returning hipErrorNotReady, within the limit.
template <typename F>
hipError_t poll(F done) {
  hipError_t e;
  const auto t0 = std::chrono::steady_clock::now();
  while ((e = done()) == hipErrorNotReady) {
    const std::chrono::duration<double> dt =
        std::chrono::steady_clock::now() - t0;
    if (dt.count() > kReadBackLimitSeconds) return hipErrorLaunchTimeOut;
  }
  return e;
}

// the synchronous read-back: the copy, then the whole stream drained
hipError_t read_now(const void* dev, void* host, size_t bytes, hipStream_t s) {
  hipError_t e = hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  return poll([&] { return hipStreamQuery(s); });
}

// a free slot of the current device (created on first use), or null
RbSlot* take_slot() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kRbDevices)
    return nullptr;
  std::lock_guard<std::mutex> lk(g_rb_mu);
  for (int i = 0; i < kRbSlots; ++i) {
    RbSlot& q = g_rb[dev][i];
    if (q.busy || q.failed) continue;
    if (!q.pin) {
      if (hipHostMalloc(&q.pin, kReadBackMax, hipHostMallocDefault) !=
          hipSuccess) {
        q.pin = nullptr;
        q.failed = true;
        continue;
      }
      void* dp = nullptr;
      if (hipHostGetDevicePointer(&dp, q.pin, 0) != hipSuccess ||
          hipEventCreateWithFlags(&q.ev, hipEventDisableTiming) !=
              hipSuccess) {
        (void)hipHostFree(q.pin);
        q.pin = nullptr;
        q.ev = nullptr;
        q.failed = true;
        continue;
      }
      q.dpin = static_cast<uint32_t*>(dp);
    }
    q.busy = true;
    return &q;
  }
  return nullptr;
}

void give_slot(RbSlot* q) {
  std::lock_guard<std::mutex> lk(g_rb_mu);
  q->busy = false;
}

// the words of a read-back, one per lane, into the pinned slot
__global__ __launch_bounds__(kWave) void k_put_host(const uint32_t* src,
                                                    uint32_t* dst, int nw) {
  const int i = (int)threadIdx.x;
  if (i < nw) dst[i] = src[i];
  // visible to the host before the kernel (and the event after it) ends
  __threadfence_system();
}

}  // namespace

uint32_t* read_back_open(size_t bytes, ReadBack* rb) {
  rb->bytes = bytes;
  rb->err = hipSuccess;
  // whole words only (every caller's case)
  RbSlot* q = bytes > 0 && bytes <= kReadBackMax && bytes % 4 == 0
                  ? take_slot() : nullptr;
  rb->slot = q;
  return q ? q->dpin : nullptr;
}

hipError_t read_back_close(const void* dev, hipStream_t s, ReadBack* rb) {
  if (rb->bytes == 0) return hipSuccess;
  RbSlot* q = static_cast<RbSlot*>(rb->slot);
  if (!q) {
    // no slot: read now into the inline buffer
    rb->err = rb->bytes > kReadBackMax ? hipErrorInvalidValue
                                       : read_now(dev, rb->now, rb->bytes, s);
    return rb->err;
  }
  const hipError_t e = hipEventRecord(q->ev, s);
  if (e != hipSuccess) {
    // (the kernel before may still store into the slot)
    (void)poll([&] { return hipStreamQuery(s); });
    rb->slot = nullptr;
    give_slot(q);
  }
  return e;
}

hipError_t read_back_start(const void* dev, size_t bytes, hipStream_t s,
                           ReadBack* rb) {
  if (bytes > kReadBackMax) return hipErrorInvalidValue;
  uint32_t* slot = ((uintptr_t)dev & 3) == 0 ? read_back_open(bytes, rb)
                                             : nullptr;
  if (!slot) {
    rb->slot = nullptr;
    rb->bytes = bytes;
    return read_back_close(dev, s, rb);
  }
  const hipError_t e = launch("read_back", k_put_host, dim3(1), dim3(kWave),
                              s, static_cast<const uint32_t*>(dev), slot,
                              (int)(bytes / 4));
  if (e != hipSuccess) {
    give_slot(static_cast<RbSlot*>(rb->slot));
    rb->slot = nullptr;
    return e;
  }
  return read_back_close(dev, s, rb);
}

hipError_t read_back_finish(ReadBack* rb, void* host) {
  if (rb->bytes == 0) return hipSuccess;
  RbSlot* q = static_cast<RbSlot*>(rb->slot);
  if (!q) {
    if (rb->err == hipSuccess) std::memcpy(host, rb->now, rb->bytes);
    return rb->err;
  }
  const hipError_t e = poll([&] { return hipEventQuery(q->ev); });
  if (e == hipSuccess) std::memcpy(host, q->pin, rb->bytes);
  rb->slot = nullptr;
  give_slot(q);
  return e;
}

ReadBack::~ReadBack() {
  if (!slot) return;
  RbSlot* q = static_cast<RbSlot*>(slot);
  // the copy into the slot may still be queued: wait for it before the
  // slot can be taken again (a slot that was opened and not closed, its
  // launch having failed, has only its earlier event, already past)
  (void)poll([&] { return hipEventQuery(q->ev); });
  give_slot(q);
}

hipError_t read_back(const void* dev, void* host, size_t bytes,
                     hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  if (bytes > kReadBackMax) return read_now(dev, host, bytes, s);
  ReadBack rb;
  hipError_t e = read_back_start(dev, bytes, s, &rb);
  if (e != hipSuccess) return e;
  return read_back_finish(&rb, host);
}

}  // namespace chopper
