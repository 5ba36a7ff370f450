// workspace.h -- the per-call workspaces of the entry points: a stream-ordered memory pool of the
// library's own per device, and a few kept pieces of it for small calls.  Host code on the HIP
// runtime's C functions only, so that a test can compile it against a stand-in for them.
#pragma once
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstddef>
#include <cstdint>
#include <mutex>

namespace afno {

constexpr int kMaxDevices = 64;

// Per-call workspaces come from a stream-ordered memory pool of the library's own, one per
// device, that keeps freed memory for the next call instead of returning it to the device
// (release threshold: unbounded), so that a call's allocation and free cost only the pool's
// bookkeeping (measured: the 90 x 180 x 768 bf16 call takes 2.5 us less than from the
// device's default pool).  The pool holds the largest workspaces in use at once until the
// process ends.
inline std::mutex g_pool_mu;
inline hipMemPool_t g_pool[kMaxDevices] = {};

inline hipError_t ws_alloc(void** p, size_t bytes, hipStream_t stream) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipMallocAsync(p, bytes, stream);
  hipMemPool_t pool = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_pool_mu);
    if (!g_pool[dev]) {
      hipMemPoolProps props = {};
      props.allocType = hipMemAllocationTypePinned;
      props.location.type = hipMemLocationTypeDevice;
      props.location.id = dev;
      e = hipMemPoolCreate(&pool, &props);
      if (e != hipSuccess) return e;
      uint64_t keep = UINT64_MAX;
      e = hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep);
      if (e != hipSuccess) {
        (void)hipMemPoolDestroy(pool);
        return e;
      }
      g_pool[dev] = pool;
    }
    pool = g_pool[dev];
  }
  return hipMallocFromPoolAsync(p, bytes, pool, stream);
}

// Small workspaces (up to kSlotBytes) come from slots of that pool's memory that the library
// keeps, at most kSlots (256 MB) a device: a pool allocation and free cost the host 14 to 17 us a
// call, more than the three kernels of a small filter take (16 x 32 x 64 fp32, 200 calls in a row
// on a stream: 31 to 34 us a call from the pool, 17 from a slot; the kernels 11).
//
// One call holds a slot while it enqueues, and records the slot's event behind its work.  The next
// holder first makes its stream wait for that event, whatever its handle is: one handle can name
// another stream by then (hipStreamPerThread in another thread, a destroyed and recreated stream).
// Which slot a call takes:
//  1. the one its own stream handle used last;
//  2. the least recently used one of another handle if that one's work has ended (asked of that
//     one slot alone: no stream is made to wait for another's work, and as many slots are
//     allocated as calls overlap in time, not one per stream that ever called);
//  3. one that is not allocated yet;
//  4. none: the pool, as larger workspaces and streams under capture (whose graph must own its
//     memory) always do.  If the device has no memory left for that, the slots that no call holds
//     are freed and the pool trimmed, once.
constexpr size_t kSlotBytes = (size_t)32 << 20;
constexpr int kSlots = 8;
struct Slot {
  void* ptr = nullptr;
  hipEvent_t done = nullptr;
  hipStream_t last = nullptr;
  uint64_t used = 0;  // g_slot_clock when it was taken last
  bool held = false;
};
inline std::mutex g_slot_mu;
inline Slot g_slots[kMaxDevices][kSlots];
inline uint64_t g_slot_clock = 0;
inline std::atomic<int64_t> g_slot_calls{0};  // calls that ran in a slot (the tests read it)

// Whether the slot's last work has ended.  A capture that another thread (or this one, on another
// stream) has under way in the global mode forbids queries; a relaxed thread may make them.
inline bool slot_idle(const Slot& s) {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  const bool idle = hipEventQuery(s.done) == hipSuccess;
  if (!idle) (void)hipGetLastError();  // not ready
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  return idle;
}

// The memory of the slots that no call holds, given back to the device (a call whose workspace did
// not fit): freed behind their last work, in order on `stream`.  True if there was any.
inline bool free_idle_slots(int dev, hipStream_t stream) {
  {
    std::lock_guard<std::mutex> lk(g_slot_mu);
    bool any = false;
    for (Slot& s : g_slots[dev]) {
      if (s.held || !s.ptr || hipStreamWaitEvent(stream, s.done, 0) != hipSuccess ||
          hipFreeAsync(s.ptr, stream) != hipSuccess)
        continue;
      (void)hipEventDestroy(s.done);
      s.ptr = nullptr;
      any = true;
    }
    if (!any) return false;
  }
  if (hipStreamSynchronize(stream) != hipSuccess) return false;
  std::lock_guard<std::mutex> lk(g_pool_mu);
  return g_pool[dev] && hipMemPoolTrimTo(g_pool[dev], 0) == hipSuccess;
}

// One call's workspace.
struct Workspace {
  void* ptr = nullptr;
  Slot* slot = nullptr;
  hipStream_t stream = nullptr;

  hipError_t acquire(size_t bytes, hipStream_t st) {
    stream = st;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    int dev = -1;
    if (bytes <= kSlotBytes && hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices &&
        hipStreamIsCapturing(st, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone &&
        take_slot(dev))
      return hipSuccess;
    (void)hipGetLastError();
    hipError_t e = ws_alloc(&ptr, bytes, st);
    if (e == hipErrorOutOfMemory && hipGetDevice(&dev) == hipSuccess && dev >= 0 &&
        dev < kMaxDevices && hipStreamIsCapturing(st, &cap) == hipSuccess &&
        cap == hipStreamCaptureStatusNone && free_idle_slots(dev, st)) {
      (void)hipGetLastError();
      e = ws_alloc(&ptr, bytes, st);
    }
    return e;
  }
  // after the call's last launch
  hipError_t release() {
    if (!slot) return hipFreeAsync(ptr, stream);
    hipError_t e = hipEventRecord(slot->done, stream);
    if (e != hipSuccess) e = hipStreamSynchronize(stream);  // nothing may still use the slot
    std::lock_guard<std::mutex> lk(g_slot_mu);
    slot->held = false;
    return e;
  }

 private:
  bool take_slot(int dev) {
    Slot* got = nullptr;
    {
      std::lock_guard<std::mutex> lk(g_slot_mu);
      Slot *fresh = nullptr, *oldest = nullptr;
      for (Slot& s : g_slots[dev]) {
        if (s.held) continue;
        if (!s.ptr) {
          if (!fresh) fresh = &s;
        } else if (s.last == stream) {
          got = &s;
          break;
        } else if (!oldest || s.used < oldest->used) {
          oldest = &s;
        }
      }
      if (!got && oldest && slot_idle(*oldest)) got = oldest;
      if (!got) got = fresh;
      if (!got) return false;
      got->held = true;
      got->last = stream;
      got->used = ++g_slot_clock;
    }
    bool ok;
    if (got->ptr) {
      ok = hipStreamWaitEvent(stream, got->done, 0) == hipSuccess;
    } else {
      ok = hipEventCreateWithFlags(&got->done, hipEventDisableTiming) == hipSuccess;
      if (ok && ws_alloc(&got->ptr, kSlotBytes, stream) != hipSuccess) {
        (void)hipEventDestroy(got->done);
        got->ptr = nullptr;
        ok = false;
      }
    }
    if (!ok) {
      std::lock_guard<std::mutex> lk(g_slot_mu);
      got->held = false;
      return false;
    }
    slot = got;
    ptr = got->ptr;
    g_slot_calls.fetch_add(1, std::memory_order_relaxed);
    return true;
  }
};

}  // namespace afno
