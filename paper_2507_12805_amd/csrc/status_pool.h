// Status words of the calls that take no workspace (the encoder's error flag,
// the coder export's bit count and error flag): a fixed pool in device memory,
// 32 bytes per call in flight on a device, so that no call allocates.
#pragma once
#include <hip/hip_runtime.h>

#include <condition_variable>
#include <cstdint>
#include <mutex>

namespace pmklc {

constexpr int kStatusSlots = 64;

// one device's pool
struct StatusPool {
  std::mutex mu;
  std::condition_variable cv;
  unsigned long long *base = nullptr;   // the device's words, 4 per slot, zero at first
  uint64_t busy = 0;                    // bit i: slot i in use
  uint64_t dirty = 0;                   // bit i: slot i was released without being cleared
};

// One slot of the pool on the current device for the length of a call; a
// call waits while all slots are taken.  A slot's words are zero when it is
// acquired: the call that found them so after its stream drained says so
// (clean), any other release clears them and drains the stream, so that no
// kernel can still write a released slot.  Where that fails (a stream that is
// captured or in error) the slot is marked, taken again only when no other is
// free, and cleared then, behind everything on the device, before it is used.
struct StatusSlot {
  StatusPool *pool = nullptr;
  hipStream_t st = nullptr;
  int idx = -1;
  unsigned long long *ptr = nullptr;   // 4 words of device memory
  bool clean = false;                  // the stream has drained and the words are zero
  // base(&p): the pool's words, asked for once
  template <class Base>
  hipError_t acquire(StatusPool &from, hipStream_t stream, Base base) {
    constexpr uint64_t kAll = ~0ull >> (64 - kStatusSlots);
    std::unique_lock<std::mutex> lk(from.mu);
    if (!from.base) {
      void *p = nullptr;
      const hipError_t e = base(&p);
      if (e != hipSuccess) return e;
      from.base = static_cast<unsigned long long *>(p);
    }
    from.cv.wait(lk, [&] { return from.busy != kAll; });
    const uint64_t free_slots = kAll & ~from.busy, zero = free_slots & ~from.dirty;
    idx = __builtin_ctzll(zero ? zero : free_slots);
    from.busy |= 1ull << idx;
    const bool was_dirty = !zero;
    lk.unlock();
    pool = &from;
    ptr = from.base + 4 * idx;
    st = stream;
    if (!was_dirty) return hipSuccess;
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = clear();
    if (e == hipSuccess) {
      lk.lock();
      from.dirty &= ~(1ull << idx);
    }
    return e;
  }
  ~StatusSlot() {
    if (idx < 0) return;
    const bool zero = clean || clear() == hipSuccess;
    {
      std::lock_guard<std::mutex> lk(pool->mu);
      pool->busy &= ~(1ull << idx);
      if (!zero) pool->dirty |= 1ull << idx;
    }
    pool->cv.notify_one();
  }

 private:
  hipError_t clear() {
    const hipError_t e = hipMemsetAsync(ptr, 0, 32, st), f = hipStreamSynchronize(st);
    return e != hipSuccess ? e : f;
  }
};

}  // namespace pmklc
