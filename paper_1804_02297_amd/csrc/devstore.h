// A bounded store of released device blocks (devmem.hip says why there is one).
#pragma once

#include <pthread.h>
#include <signal.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstddef>
#include <cstdlib>
#include <mutex>
#include <thread>

namespace ls {

struct StoreLimits {
  size_t min_block;                    // smaller blocks are not held
  size_t max_held;                     // bytes held over all devices, at most,
  int part;                            // and of the memory that is free on the device: one part-th,
  std::chrono::milliseconds fresh;     // as it was at most this long ago
  std::chrono::milliseconds idle;      // a block not taken again within this goes back
};

// Dev: bool current(int* dev), void* alloc(size_t), void free(void*), bool wait(int dev) (true once
// nothing runs on device dev and it is the current one) and size_t spare() (bytes free on the current
// device); alloc and free on any thread.
//
// Blocks that stay too long are freed by a thread of the store, which the first take() starts, so they
// come back without any further call.  give() allocates no host memory: destructors call it.
template <class Dev>
class BlockStore {
 public:
  BlockStore(Dev dev, StoreLimits lim) : dev_(dev), lim_(lim) {}
  ~BlockStore() { stop(); }

  // At least `bytes` on the current device: a held block of at most 5/4 of that, the smallest that
  // fits, or a new one.  When none can be had, every held block goes back, what other threads are
  // giving back is waited for, and it is tried once more.
  void* take(size_t bytes, size_t* got, int* dev) {
    if (!dev_.current(dev)) return nullptr;
    void* p = nullptr;
    if (bytes >= lim_.min_block && bytes <= lim_.max_held) {
      std::lock_guard<std::mutex> lock(mu_);
      start();
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
    }
    if (p) return p;
    *got = bytes;
    p = dev_.alloc(bytes);
    if (p) return p;
    release();
    return dev_.alloc(bytes);
  }

  // A block from take(): held, or freed where it is too small, too large or in use on another device.
  void give(void* p, size_t bytes, int dev) {
    Gone out;
    bool held = false;
    if (bytes >= lim_.min_block && bytes <= lim_.max_held && dev_.wait(dev)) {
      std::lock_guard<std::mutex> lock(mu_);
      const auto now = Clock::now();
      if (dev != spare_dev_ || now - spare_at_ >= lim_.fresh) {
        spare_ = dev_.spare();
        spare_dev_ = dev;
        spare_at_ = now;
      }
      const size_t most = std::min(lim_.max_held, spare_ / lim_.part);
      if (started_ && !stop_ && bytes <= most) {
        while (n_ == kSlots || (n_ && bytes_ + bytes > most)) oldest_to(out);
        held_[n_++] = Block{p, bytes, dev, now};
        bytes_ += bytes;
        held = true;
        if (asleep_) wake_.notify_one();         // else the thread waits for an older block's time
      }
    }
    if (!held) dev_.free(p);
    free_all(out);
  }

  // Every held block goes back; on return none is on its way either.
  void release() {
    Gone out;
    {
      std::lock_guard<std::mutex> lock(mu_);
      while (n_) oldest_to(out);
    }
    free_all(out);
    std::unique_lock<std::mutex> lock(mu_);
    freed_.wait(lock, [this] { return freeing_ == 0; });
  }

  // Ends the thread; blocks given from now on are freed at once.
  void stop() {
    {
      std::lock_guard<std::mutex> lock(mu_);
      stop_ = true;
      wake_.notify_one();
    }
    if (thread_.joinable()) thread_.join();
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
  void free_all(Gone& out) {
    if (!out.n) return;
    for (int i = 0; i < out.n; ++i) dev_.free(out.p[i]);
    std::lock_guard<std::mutex> lock(mu_);
    freeing_ -= out.n;
    out.n = 0;
    freed_.notify_all();
  }

  // The thread that frees blocks held for longer than idle.  It takes no signals, and where it
  // cannot be started nothing is held.
  void start() {
    if (started_ || stop_) return;
    sigset_t all, old;
    sigfillset(&all);
    if (pthread_sigmask(SIG_SETMASK, &all, &old) != 0) return;
    try {
      thread_ = std::thread([this] { watch(); });
      started_ = true;
    } catch (...) {
    }
    (void)pthread_sigmask(SIG_SETMASK, &old, nullptr);
  }
  void watch() {
    std::unique_lock<std::mutex> lock(mu_);
    while (!stop_) {
      if (!n_) {
        asleep_ = true;
        wake_.wait(lock);
        asleep_ = false;
        continue;
      }
      const auto due = held_[0].since + lim_.idle;
      if (Clock::now() < due) {
        wake_.wait_until(lock, due);
        continue;
      }
      Gone out;
      oldest_to(out);
      lock.unlock();
      free_all(out);
      lock.lock();
    }
  }

  Dev dev_;
  const StoreLimits lim_;
  std::mutex mu_;
  Block held_[kSlots];                 // oldest first
  int n_ = 0;
  size_t bytes_ = 0;
  size_t spare_ = 0;                   // bytes free on spare_dev_ at spare_at_
  int spare_dev_ = -1;
  Clock::time_point spare_at_;
  int freeing_ = 0;                    // blocks taken out of the store and not yet freed
  std::condition_variable freed_, wake_;
  std::thread thread_;
  bool started_ = false, stop_ = false, asleep_ = false;
};

// The process's one store of Dev, never destroyed (buffers may be released after the statics are
// gone).  Its thread ends when the process exits normally; a forked child, where that thread does not
// run, gets a store that holds nothing.
template <class Dev>
class ProcessStore {
 public:
  static BlockStore<Dev>& get(Dev dev, StoreLimits lim) {
    static const bool made = [&] {
      at() = new BlockStore<Dev>(dev, lim);
      in_child() = new BlockStore<Dev>(dev, StoreLimits{lim.min_block, 0, 1, lim.fresh, lim.idle});
      if (std::atexit([] { at().load()->stop(); }) != 0 ||
          pthread_atfork(nullptr, nullptr, [] { at() = in_child().load(); }) != 0)
        at() = in_child().load();
      return true;
    }();
    (void)made;
    return *at().load();
  }

 private:
  static std::atomic<BlockStore<Dev>*>& at() {
    static std::atomic<BlockStore<Dev>*> s{nullptr};
    return s;
  }
  static std::atomic<BlockStore<Dev>*>& in_child() {
    static std::atomic<BlockStore<Dev>*> s{nullptr};
    return s;
  }
};

}  // namespace ls
