// A bounded store of released device blocks (devmem.hip says why there is one).
#pragma once

#include <chrono>
#include <condition_variable>
#include <cstddef>
#include <mutex>

namespace ls {

struct StoreLimits {
  size_t min_block;                    // smaller blocks are not held
  size_t max_held;                     // bytes held over all devices
  std::chrono::milliseconds idle;      // a block not taken again within this goes back
};

// Dev: bool current(int* dev), void* alloc(size_t), void free(void*), bool wait(int dev) (true once
// nothing runs on device dev and it is the current one).  Nothing here allocates host memory: give()
// is called from destructors.
template <class Dev>
class BlockStore {
 public:
  BlockStore(Dev dev, StoreLimits lim) : dev_(dev), lim_(lim) {}

  // At least `bytes` on the current device: a held block of at most 5/4 of that, the smallest that
  // fits, or a new one.  When none can be had, every held block goes back, what other threads are
  // giving back is waited for, and it is tried once more.
  void* take(size_t bytes, size_t* got, int* dev) {
    if (!dev_.current(dev)) return nullptr;
    void* p = nullptr;
    Gone out;
    if (bytes >= lim_.min_block) {
      std::lock_guard<std::mutex> lock(mu_);
      int best = -1;
      for (int i = 0; i < n_; ++i) {
        const Block& b = held_[i];
        if (b.dev == *dev && b.bytes >= bytes && b.bytes - b.bytes / 5 <= bytes &&
            (best < 0 || b.bytes < held_[best].bytes))
          best = i;
      }
      if (best >= 0) {
        p = held_[best].p;
        *got = held_[best].bytes;
        drop(best);
      }
      expired(out);
    }
    free_all(out);
    if (p) return p;
    *got = bytes;
    p = dev_.alloc(bytes);
    if (p) return p;
    {
      std::lock_guard<std::mutex> lock(mu_);
      while (n_) oldest_to(out);
    }
    free_all(out);
    {
      std::unique_lock<std::mutex> lock(mu_);
      freed_.wait(lock, [this] { return freeing_ == 0; });
    }
    return dev_.alloc(bytes);
  }

  // A block from take(): held, or freed where it is too small, too large or in use on another device.
  void give(void* p, size_t bytes, int dev) {
    if (bytes < lim_.min_block || bytes > lim_.max_held || !dev_.wait(dev)) {
      dev_.free(p);
      return;
    }
    Gone out;
    {
      std::lock_guard<std::mutex> lock(mu_);
      expired(out);
      while (n_ == kSlots || (n_ && bytes_ + bytes > lim_.max_held)) oldest_to(out);
      held_[n_++] = Block{p, bytes, dev, Clock::now()};
      bytes_ += bytes;
    }
    free_all(out);
  }

 private:
  using Clock = std::chrono::steady_clock;
  static constexpr int kSlots = 64;
  struct Block {
    void* p;
    size_t bytes;
    int dev;
    Clock::time_point since;
  };
  // blocks that leave the store, freed outside the lock
  struct Gone {
    void* p[kSlots];
    int n = 0;
  };

  void drop(int i) {
    bytes_ -= held_[i].bytes;
    for (--n_; i < n_; ++i) held_[i] = held_[i + 1];
  }
  void oldest_to(Gone& out) {
    out.p[out.n++] = held_[0].p;
    drop(0);
    ++freeing_;
  }
  void expired(Gone& out) {
    const auto now = Clock::now();
    while (n_ && now - held_[0].since > lim_.idle) oldest_to(out);
  }
  void free_all(Gone& out) {
    if (!out.n) return;
    for (int i = 0; i < out.n; ++i) dev_.free(out.p[i]);
    std::lock_guard<std::mutex> lock(mu_);
    freeing_ -= out.n;
    out.n = 0;
    freed_.notify_all();
  }

  Dev dev_;
  const StoreLimits lim_;
  std::mutex mu_;
  Block held_[kSlots];                 // oldest first
  int n_ = 0;
  size_t bytes_ = 0;
  int freeing_ = 0;                    // blocks taken out of the store and not yet freed
  std::condition_variable freed_;
};

}  // namespace ls
