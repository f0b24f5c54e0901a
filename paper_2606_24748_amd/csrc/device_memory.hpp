// Device memory of the library: the caller's allocator, the blocks kept between setups, and
// the owning buffer.  Host code only (no kernel), over the HIP calls of hip_runtime_api.h.
#pragma once

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <exception>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <utility>

#include "errors.hpp"

namespace blk {

// ---------------------------------------------------------------------------
// Device allocator: hipMalloc/hipFree, or the caller's pair of routines
// ---------------------------------------------------------------------------
struct DeviceAllocator {
  blkamg_alloc_fn alloc_fn = nullptr;  // NULL: hipMalloc / hipFree
  blkamg_free_fn free_fn = nullptr;
  void* ctx = nullptr;
};
inline std::mutex& allocator_mutex() {
  static std::mutex m;
  return m;
}
inline DeviceAllocator& allocator_slot() {
  static DeviceAllocator a;
  return a;
}
inline DeviceAllocator current_allocator() {
  std::lock_guard<std::mutex> g(allocator_mutex());
  return allocator_slot();
}
constexpr uintptr_t kDevAlign = 256;

// Waits for all work of a device, current or not; false where that is not possible (capture).
inline bool wait_for_device(int dev) {
  int cur = dev;
  (void)hipGetDevice(&cur);
  if (cur != dev) (void)hipSetDevice(dev);
  const bool ok = hipDeviceSynchronize() == hipSuccess;
  if (!ok) (void)hipGetLastError();
  if (cur != dev) (void)hipSetDevice(cur);
  return ok;
}

// Freed blocks, kept for the allocations that come next.  A setup makes and frees some 200
// buffers; hipMalloc and hipFree take microseconds for a small one and 0.3 - 0.7 ms for 50 -
// 130 MB.  Setup and destruction of a hierarchy without kept blocks -> with them, 40^3
// elements: FP64 11.4 + 5.0 -> 7.4 + 0.2 ms, FP32 18 + 4.9 -> 11.1 + 0.3; 64^3: FP64 27.3 + 8.8
// -> 19.5 + 0.3, FP32 62 + 10.7 -> 47 + 1.8.
// Bounded per device by kHeld (1 GiB was too little for 64^3) and a 64th of its memory.
// Given back when the last buffer of the library is freed, when hipMalloc or the caller's
// allocator has no memory left, when the caller sets an allocator, and by blkamg_trim.  A block
// is handed out after its device has been idle once since it came back, as it is after a
// hipFree: no stream, copy or host write can meet its former use.  An AllocScope (calls that
// wait for their stream anyway, so never under capture) waits for that; other calls take kept
// blocks only when there is nothing to wait for, so that what they free does not pile up.  A
// block serves requests of at least 7/8 of its size (any up to 64 KB).
class BlockCache {
 public:
  static BlockCache& get() {
    static BlockCache* c = new BlockCache;  // outlives every buffer
    return *c;
  }
  // NULL when there is no memory; may_wait: in an AllocScope; cap: the size to hand back
  void* make(size_t bytes, bool may_wait, int& dev, size_t& cap) {
    (void)hipGetDevice(&dev);
    std::lock_guard<std::mutex> g(m_);
    if (may_wait || !at_[dev].unsynced) {
      const auto it = free_.lower_bound({dev, bytes});
      if (it != free_.end() && it->first.first == dev &&
          (it->first.second <= kAny || it->first.second - it->first.second / 8 <= bytes) &&
          synced(dev)) {
        void* p = it->second;
        cap = it->first.second;
        at_[dev].held -= cap;
        ++live_;
        free_.erase(it);
        return p;
      }
    }
    void* p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) {
      (void)hipGetLastError();
      if (!flush()) return nullptr;
      if (hipMalloc(&p, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
      }
    }
    cap = bytes;
    ++live_;
    return p;
  }
  // waited: no queued work uses the block any more
  void give(void* p, int dev, size_t cap, bool waited) noexcept {
    std::lock_guard<std::mutex> g(m_);
    --live_;
    bool kept = false;
    try {
      if (live_ > 0 && cap <= room(dev)) {
        free_.emplace(std::make_pair(dev, cap), p);
        kept = true;
        at_[dev].held += cap;
        if (!waited) at_[dev].unsynced = true;
      }
    } catch (...) {
    }
    if (!kept) (void)hipFree(p);
    if (live_ == 0) flush();
  }
  // The end of an AllocScope: what it gave back may be handed out from now on (failed: the
  // caller's arrays are out of use too).
  void settle(bool failed) noexcept {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    std::lock_guard<std::mutex> g(m_);
    const auto d = at_.find(dev);
    const bool unsynced = d != at_.end() && d->second.unsynced;
    if ((failed || unsynced) && wait_for_device(dev) && unsynced) d->second.unsynced = false;
  }
  // Gives the kept blocks back; false if there were none.
  bool trim() noexcept {
    std::lock_guard<std::mutex> g(m_);
    return flush();
  }

 private:
  static constexpr size_t kAny = 64 * 1024, kHeld = size_t{4} << 30;
  struct Device {
    size_t held = 0, most = 0;
    bool unsynced = false;  // blocks came back since the last wait
  };
  size_t room(int dev) {
    Device& d = at_[dev];
    size_t total = 0;
    if (d.most == 0 && hipDeviceTotalMem(&total, dev) == hipSuccess) d.most = std::min(kHeld, total / 64);
    return d.most - std::min(d.held, d.most);
  }
  bool flush() noexcept {
    if (free_.empty()) return false;
    for (const auto& f : free_) (void)hipFree(f.second);
    free_.clear();
    for (auto& d : at_) d.second.held = 0;
    return true;
  }
  // the current device `dev` has been idle since its last block came back
  bool synced(int dev) {
    Device& d = at_[dev];
    if (d.unsynced) d.unsynced = !wait_for_device(dev);
    return !d.unsynced;
  }
  std::mutex m_;
  std::multimap<std::pair<int, size_t>, void*> free_;  // by device and size
  std::map<int, Device> at_;
  size_t live_ = 0;
};

// While one is open, this thread's allocations may wait for kept blocks, and released buffers
// go back without a wait: for calls that wait for their stream before they return.  At its end
// it waits once for the device if any came back, and when it is left by an exception, so that a
// call that failed has nothing queued on the caller's arrays.
class AllocScope {
 public:
  AllocScope() : thrown_(std::uncaught_exceptions()) { ++depth(); }
  ~AllocScope() {
    if (--depth() == 0) BlockCache::get().settle(std::uncaught_exceptions() > thrown_);
  }
  AllocScope(const AllocScope&) = delete;
  AllocScope& operator=(const AllocScope&) = delete;
  static int& depth() {
    thread_local int d = 0;
    return d;
  }

 private:
  int thrown_;
};

// A buffer released outside an AllocScope waits for its device, as hipFree does: callers free
// borrowed arrays once the handle is gone.  While a FreeScope is open, this thread does so at
// the first buffer of a device only (the destruction of a handle, which queues nothing).
class FreeScope {
 public:
  FreeScope() { if (depth()++ == 0) waited() = -1; }
  ~FreeScope() { --depth(); }
  FreeScope(const FreeScope&) = delete;
  FreeScope& operator=(const FreeScope&) = delete;
  static bool wait(int dev) {
    if (depth() == 0) return AllocScope::depth() == 0 && wait_for_device(dev);
    if (waited() != dev && wait_for_device(dev)) waited() = dev;
    return waited() == dev;
  }

 private:
  static int& depth() {
    thread_local int d = 0;
    return d;
  }
  static int& waited() {
    thread_local int d = -1;
    return d;
  }
};

// ---------------------------------------------------------------------------
// Device buffer (owning, freed on destruction by the routine that allocated it)
// ---------------------------------------------------------------------------
template <class T>
struct DevBuf {
  T* p = nullptr;
  size_t n = 0;
  DeviceAllocator by;
  int dev = 0;     // hipMalloc: device and size of the block
  size_t cap = 0;
  DevBuf() = default;
  explicit DevBuf(size_t count) { alloc(count); }
  DevBuf(const DevBuf&) = delete;
  DevBuf& operator=(const DevBuf&) = delete;
  DevBuf(DevBuf&& o) noexcept : p(o.p), n(o.n), by(o.by), dev(o.dev), cap(o.cap) { o.p = nullptr; o.n = 0; }
  DevBuf& operator=(DevBuf&& o) noexcept {
    if (this != &o) { release(); p = o.p; n = o.n; by = o.by; dev = o.dev; cap = o.cap; o.p = nullptr; o.n = 0; }
    return *this;
  }
  ~DevBuf() { release(); }
  void alloc(size_t count) {
    release();
    if (count == 0) return;
    const size_t bytes = count * sizeof(T);
    const DeviceAllocator a = current_allocator();
    void* q = nullptr;
    if (a.alloc_fn) {
      q = a.alloc_fn(bytes, a.ctx);
      if (q == nullptr && BlockCache::get().trim()) q = a.alloc_fn(bytes, a.ctx);
      if (q == nullptr) fail(BLKAMG_ENOMEM, "the caller's allocator returned NULL for " + std::to_string(bytes) + " bytes");
      if (reinterpret_cast<uintptr_t>(q) % kDevAlign != 0) {
        a.free_fn(q, bytes, a.ctx);
        fail(BLKAMG_EINVAL, "the caller's allocator returned a pointer not aligned to 256 bytes");
      }
    } else {
      q = BlockCache::get().make(bytes, AllocScope::depth() > 0, dev, cap);
      if (q == nullptr) fail(BLKAMG_ENOMEM, "hipMalloc of " + std::to_string(bytes) + " bytes failed");
    }
    p = static_cast<T*>(q);
    n = count;
    by = a;
  }
  void release() {
    if (p) {
      if (by.free_fn) {
        // as hipFree does: nothing queued may still use the buffer when it is handed back
        (void)hipDeviceSynchronize();
        by.free_fn(p, n * sizeof(T), by.ctx);
      } else {
        BlockCache::get().give(p, dev, cap, FreeScope::wait(dev));
      }
    }
    p = nullptr;
    n = 0;
  }
  size_t bytes() const { return n * sizeof(T); }
};

}  // namespace blk
