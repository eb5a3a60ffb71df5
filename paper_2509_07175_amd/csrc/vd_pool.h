// vd_pool.h -- device (and pinned host) blocks of grid and clip handles, kept for
// the next handle when one is freed.
//
// A program that makes a handle per call (an autograd function, a loop with
// local handles) pays about 50 allocations and as many frees for each, most of
// the time of a small diagram.  Here a freed handle's blocks are kept and handed
// to the next one of about the same size: forward and backward of 4,000 sites
// through the autograd function 8.9 -> 2.5 ms when it came (0.8 now).
//
// Bounds: at most kPoolBytes are kept.  Where they do not suffice, blocks that
// kStale handles ended without taking make room (a program that changes its sizes
// is not left with blocks that fit no more: Lloyd calls of 140,000 sites after
// smaller ones 73 against 10 ms), and else the new ones are given back; nothing of
// a handle larger than that is kept.  Nothing is when no handle of the library is
// left; an allocation of the library that fails gives all of it back and tries
// again, and vd_release_memory does for the program's own.  A block
// enters the pool only after one block of its handle went through hipFree, which
// waits for the device: whatever ran on any stream with the handle's memory is
// over.  When that call fails (a capture is running) or another device is
// current, every block takes the way of that first one.
#pragma once
#include <hip/hip_runtime.h>

#include <initializer_list>
#include <map>
#include <mutex>
#include <new>
#include <unordered_map>
#include <utility>

class BlockPool {
 public:
  static constexpr size_t kPoolBytes = 4ull << 30;  // 1.4 % of the card's memory
  static constexpr unsigned long long kStale = 8;
  static BlockPool &get() {
    static BlockPool *p = new BlockPool;  // (outlives handles that are freed at exit)
    return *p;
  }

  // (std::bad_alloc of the tables is reported like the device's)
  hipError_t alloc(void **out, size_t bytes, bool host = false) try {
    *out = nullptr;
    bytes = (bytes + 255) & ~size_t(255);
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    {
      std::lock_guard<std::mutex> lk(mu_);
      auto &m = free_[{dev, host}];
      auto it = m.lower_bound(bytes);
      if (it != m.end() && it->first <= bytes + bytes / 4 + 4096) {
        void *p = it->second.p;
        live_[p] = {it->first, dev, host};
        kept_ -= it->first;
        m.erase(it);
        *out = p;
        return hipSuccess;
      }
    }
    hipError_t e = raw_alloc(out, bytes, host);
    if (e == hipErrorOutOfMemory && drain()) e = raw_alloc(out, bytes, host);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(mu_);
    live_[*out] = {bytes, dev, host};
    return hipSuccess;
  } catch (const std::bad_alloc &) {
    if (*out) (void)(host ? hipHostFree(*out) : hipFree(*out));
    *out = nullptr;
    return hipErrorOutOfMemory;
  }

  // a device block that is not pooled
  hipError_t alloc_apart(void **out, size_t bytes) {
    hipError_t e = raw_alloc(out, bytes, false);
    if (e == hipErrorOutOfMemory && drain()) e = raw_alloc(out, bytes, false);
    return e;
  }

  // gives one block back to the device
  hipError_t free_now(void *p) {
    if (!p) return hipSuccess;
    bool host = false;
    {
      std::lock_guard<std::mutex> lk(mu_);
      auto it = live_.find(p);
      if (it != live_.end()) {
        host = it->second.host;
        live_.erase(it);
      }
    }
    return host ? hipHostFree(p) : hipFree(p);
  }

  // the blocks of a handle that ends (`blocks`: device blocks first)
  void release(std::initializer_list<void *> blocks) {
    const bool small = begin_release(blocks);
    bool idle = false;  // the device has been waited for
    for (void *p : blocks) {
      if (!p) continue;
      if (!idle || !small || !keep(p)) {
        const bool mine = on_current_device(p);
        const hipError_t e = free_now(p);
        idle = idle || (mine && e == hipSuccess);
      }
    }
  }

  void handle_made() {
    std::lock_guard<std::mutex> lk(mu_);
    handles_++;
  }
  void handle_gone() {
    bool last;
    {
      std::lock_guard<std::mutex> lk(mu_);
      last = --handles_ == 0;
    }
    if (last) drain();
  }

  // gives everything that is kept back; false: there was nothing
  bool drain() {
    Free out;
    {
      std::lock_guard<std::mutex> lk(mu_);
      out.swap(free_);
      kept_ = 0;
    }
    bool any = false;
    for (auto &m : out)
      for (auto &b : m.second) {
        any = true;
        give_back(b.second.p, m.first.second);
      }
    return any;
  }

 private:
  struct Block {
    size_t bytes;
    int dev;
    bool host;
  };
  struct Kept {
    void *p;
    unsigned long long age;  // handles that had ended when it was kept
  };
  using Free = std::map<std::pair<int, bool>, std::multimap<size_t, Kept>>;  // by device and kind, then size

  static hipError_t raw_alloc(void **out, size_t bytes, bool host) {
    const hipError_t e = host ? hipHostMalloc(out, bytes, hipHostMallocDefault) : hipMalloc(out, bytes);
    if (e != hipSuccess) {
      *out = nullptr;
      (void)hipGetLastError();  // (returned here: no later call is to find it)
    }
    return e;
  }
  bool on_current_device(void *p) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    std::lock_guard<std::mutex> lk(mu_);
    auto it = live_.find(p);
    return it != live_.end() && it->second.dev == dev && !it->second.host;
  }
  static void give_back(void *p, bool host) { (void)(host ? hipHostFree(p) : hipFree(p)); }
  // counts the handle; false: it is too large to be kept
  bool begin_release(std::initializer_list<void *> blocks) {
    std::lock_guard<std::mutex> lk(mu_);
    clock_++;
    size_t sum = 0;
    for (void *p : blocks) {
      auto it = live_.find(p);
      if (it != live_.end()) sum += it->second.bytes;
    }
    return sum <= kPoolBytes;
  }
  bool keep(void *p) try {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    std::unique_lock<std::mutex> lk(mu_);
    auto it = live_.find(p);
    if (it == live_.end() || it->second.dev != dev) return false;
    const size_t bytes = it->second.bytes;
    const bool host = it->second.host;
    while (kept_ + bytes > kPoolBytes) {
      // the oldest stale one (few blocks are ever kept: a search is enough)
      Free::mapped_type *from = nullptr;
      Free::mapped_type::iterator old;
      bool old_host = false;
      for (auto &m : free_)
        for (auto b = m.second.begin(); b != m.second.end(); ++b)
          if (b->second.age + kStale <= clock_ && (!from || b->second.age < old->second.age)) {
            from = &m.second;
            old = b;
            old_host = m.first.second;
          }
      if (!from) return false;
      void *q = old->second.p;
      kept_ -= old->first;
      from->erase(old);
      lk.unlock();
      give_back(q, old_host);
      lk.lock();
    }
    free_[{dev, host}].insert({bytes, Kept{p, clock_}});
    kept_ += bytes;
    live_.erase(p);
    return true;
  } catch (const std::bad_alloc &) {
    return false;
  }

  std::mutex mu_;
  Free free_;
  std::unordered_map<void *, Block> live_;
  size_t kept_ = 0;
  unsigned long long clock_ = 0;
  long long handles_ = 0;
};
