// Device-memory bookkeeping of the library on a pretended device (host memory that can run out).
#include <sys/wait.h>
#include <unistd.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <initializer_list>
#include <mutex>
#include <new>
#include <set>
#include <thread>
#include <vector>

#include "buffers.h"
#include "devstore.h"

// host memory that can be made to run out (ThreadSanitizer brings its own operator new)
static thread_local bool host_memory = true;
#if !__has_feature(thread_sanitizer)
void* operator new(size_t n) {
  void* p = host_memory ? std::malloc(n) : nullptr;
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
#endif

namespace {

std::atomic<int> failures{0};
void check(bool ok, const char* what) {
  if (!ok) std::printf("FAILED: %s\n", what);
  failures += !ok;
}

// ---- buffers that belong together ----------------------------------------------------------------

int allocations_left = 1 << 30;   // how many more succeed

struct HostBuf {
  void* p = nullptr;
  size_t bytes = 0;
  HostBuf() = default;
  HostBuf(const HostBuf&) = delete;
  ~HostBuf() { std::free(p); }
  void release() {
    std::free(p);
    p = nullptr;
    bytes = 0;
  }
  ls_status alloc(size_t b) {
    release();
    if (allocations_left-- <= 0) return LS_ENOMEM;
    p = std::malloc(b);
    bytes = b;
    return LS_OK;
  }
};

// A group whose fail-th allocation fails leaves no buffer, as a caller that looks at any one of them has to find it.
void group_is_all_or_nothing(int fail) {
  HostBuf a, b, c;
  const auto group = [&](size_t n) { return ls::alloc_all<HostBuf>({{&a, n}, {&b, 2 * n}, {&c, 3 * n}}); };
  allocations_left = 1 << 30;
  check(group(8) == LS_OK && a.bytes == 8 && b.bytes == 16 && c.bytes == 24, "a group that fits");
  allocations_left = fail;
  check(group(16) == LS_ENOMEM && !a.p && !b.p && !c.p, "a group that does not: nothing held");
}

// After a growth whose fail-th allocation fails, a smaller request (which the old buffers
// would have held) either finds all three buffers large enough or is refused.
void solve_work_after_a_failed_growth(int fail) {
  ls::SolveWork<HostBuf> w;
  allocations_left = 1 << 30;
  const size_t vec = 96, upd = 40;
  check(w.reserve(4, vec, upd) == LS_OK, "first growth");
  allocations_left = fail;
  check(w.reserve(16, vec, upd) == LS_ENOMEM, "growth that does not fit is refused");
  const auto holds = [&](int n) { return w.X.bytes >= vec * n && w.Z.bytes >= vec * n && w.U.bytes >= upd * n; };
  allocations_left = 0;
  for (int n : {1, 4}) check(w.reserve(n, vec, upd) != LS_OK || holds(n), "no memory left: refused, or all three there");
  allocations_left = 1 << 30;
  for (int n : {4, 1, 16}) check(w.reserve(n, vec, upd) == LS_OK && holds(n), "memory again: all three there");
}

// ---- the store of released blocks ------------------------------------------------

// A pretended card of `room` bytes.
struct Card {
  size_t room = 1 << 20, spare = 1 << 20;   // in all; what the card says is free
  std::atomic<size_t> used{0};
  std::atomic<int> refused{0};          // allocations that did not fit
  std::set<void*> live;
  std::mutex mu;
  std::function<void()> on_free;        // runs before a block goes
  ~Card() {
    for (void* p : live) std::free(p);
  }
};
struct CardDev {
  Card* card;
  int dev = 0;
  bool current(int* d) const { return *d = dev, true; }
  void* alloc(size_t n) {
    std::lock_guard<std::mutex> lock(card->mu);
    if (card->used + n > card->room) return ++card->refused, nullptr;
    size_t* p = static_cast<size_t*>(std::malloc(sizeof(size_t) + n));
    *p = n;
    card->used += n;
    card->live.insert(p);
    return p;
  }
  void free(void* q) {
    size_t* p = static_cast<size_t*>(q);
    if (card->on_free) card->on_free();
    std::lock_guard<std::mutex> lock(card->mu);
    check(card->live.erase(p) == 1, "freed once");
    card->used -= *p;
    std::free(p);
  }
  bool wait(int d) const { return d == dev; }
  size_t spare() const { return card->spare; }
};
using Store = ls::BlockStore<CardDev>;
constexpr std::chrono::milliseconds kNow(0), kLong(60000);

// A destructor gives a buffer back: that works, and throws nothing, without host memory.
void give_without_host_memory() {
  Card card;
  Store s(CardDev{&card}, ls::StoreLimits{16, 4096, 1, kNow, kLong});
  size_t got[100];
  int dev;
  void* p[100];                         // (the first take starts the store's thread)
  for (int i = 0; i < 100; ++i) p[i] = s.take(40, &got[i], &dev);
  host_memory = false;
  for (int i = 0; i < 100; ++i) [&]() noexcept { s.give(p[i], got[i], dev); }();
  host_memory = true;
  check(card.used <= 4096 && card.used >= 40, "blocks held within the bound");
  for (int i = 0; i < 200; ++i) p[0] = s.take(4 + i % 60, &got[0], &dev), s.give(p[0], got[0], dev);
  check(card.used <= 4096, "within the bound after many sizes");
}

// The oldest go first, a block serves requests of at least 4/5 of its size, and an allocation
// that fails has everything held given back.
void bounds_of_the_store() {
  Card card;
  Store s(CardDev{&card}, ls::StoreLimits{16, 1000, 1, kNow, kLong});
  size_t got;
  int dev;
  void* a = s.take(400, &got, &dev);
  void* b = s.take(500, &got, &dev);
  void* c = s.take(300, &got, &dev);
  void* d = s.take(1001, &got, &dev);
  void* e = s.take(15, &got, &dev);
  s.give(a, 400, 0);
  s.give(b, 500, 0);
  check(card.used == 2216, "two held");
  s.give(c, 300, 0);
  check(card.used == 1816, "the oldest is freed past the bound");
  s.give(d, 1001, 0);
  s.give(e, 15, 0);
  check(card.used == 800, "too large and too small ones are not held");
  void* x = s.take(399, &got, &dev);
  check(x != b && got == 399 && card.used == 1199, "a block of more than 5/4 does not serve");
  void* y = s.take(400, &got, &dev);
  check(y == b && got == 500, "one of 5/4 does");
  s.give(y, got, 1);
  check(card.used == 699, "not held while another device is current");
  s.give(x, 399, 0);
  check(card.used == 699, "held again");
  void* z = s.take(card.room, &got, &dev);
  check(z && card.used == card.room, "an allocation that failed had the store drained");
  check(!s.take(16, &got, &dev), "no memory");
  s.give(z, card.room, 0);
}

bool comes_true(const std::function<bool()>& f) {
  for (int i = 0; i < 2000; ++i) {
    if (f()) return true;
    std::this_thread::sleep_for(std::chrono::milliseconds(5));
  }
  return false;
}

// An allocation that fails while another thread is giving the held blocks back waits for them.
void allocation_during_a_drain() {
  Card card;
  card.room = 1000;
  Store s(CardDev{&card}, ls::StoreLimits{16, 1000, 1, kNow, kLong});
  size_t got, got2;
  int dev, dev2;
  s.give(s.take(900, &got, &dev), got, dev);
  std::atomic<bool> draining{false};
  card.on_free = [&] {
    draining = true;
    comes_true([&] { return card.refused >= 2; });              // the other thread was refused
    std::this_thread::sleep_for(std::chrono::milliseconds(50));
  };
  void* a = nullptr;
  std::thread t([&] { a = s.take(600, &got, &dev); });
  check(comes_true([&] { return draining.load(); }), "the first thread drains the store");
  void* b = s.take(200, &got2, &dev2);
  t.join();
  card.on_free = nullptr;
  check(a && b && card.used == 800, "both threads have their blocks");
}

// A block that nobody takes again goes back without any further call, and one that is taken in time stays.
void given_back_when_idle() {
  Card card;
  Store s(CardDev{&card}, ls::StoreLimits{16, 4096, 1, kNow, std::chrono::milliseconds(200)});
  size_t got, got2;
  int dev;
  void *p = s.take(1000, &got, &dev), *q = s.take(500, &got2, &dev);
  s.give(p, got, dev);
  s.give(q, got2, dev);
  check(card.used == 1500, "held at first");
  check(comes_true([&] { return card.used == 0; }), "given back with no call");
  p = s.take(1000, &got, &dev);
  s.give(p, got, dev);
  for (int i = 0; i < 10; ++i) {
    void* r = s.take(1000, &got, &dev);
    check(r == p, "reused");
    std::this_thread::sleep_for(std::chrono::milliseconds(50));
    s.give(r, got, dev);
  }
  check(comes_true([&] { return card.used == 0; }), "given back again");
}

// What is held leaves most of a nearly full card to others; release() and stop() leave nothing.
void given_back_on_request() {
  Card card;
  Store s(CardDev{&card}, ls::StoreLimits{16, 4096, 4, kNow, kLong});
  size_t got;
  int dev;
  void* a = s.take(1000, &got, &dev);
  void* b = s.take(1000, &got, &dev);
  card.spare = 3999;
  s.give(a, 1000, 0);
  check(card.used == 1000, "more than a quarter of what is free: not held");
  card.spare = 4000;
  s.give(b, 1000, 0);
  check(card.used == 1000, "a quarter: held");
  s.release();
  check(card.used == 0, "release");
  b = s.take(1000, &got, &dev);
  s.stop();
  s.give(b, got, 0);
  check(card.used == 0, "nothing held after stop");
}

// The free memory is asked for again once the answer is old, and not before.
void free_memory_is_asked_for_again() {
  Card card;
  Store s(CardDev{&card}, ls::StoreLimits{16, 4096, 4, std::chrono::milliseconds(100), kLong});
  size_t got;
  int dev;
  void *a = s.take(1000, &got, &dev), *b = s.take(900, &got, &dev);
  card.spare = 8000;
  s.give(a, 1000, 0);
  card.spare = 40;
  s.give(b, 900, 0);
  check(card.used == 1900, "both held by the first answer");
  std::this_thread::sleep_for(std::chrono::milliseconds(150));
  s.give(s.take(1000, &got, &dev), 1000, 0);
  check(card.used == 900, "not held by the second");
}

// A forked child, which has no thread to free blocks, holds none and ends as usual.
void forked_child() {
#if !__has_feature(thread_sanitizer)
  static Card card;
  const auto get = []() -> Store& {
    return ls::ProcessStore<CardDev>::get(CardDev{&card}, ls::StoreLimits{16, 4096, 1, kNow, kLong});
  };
  size_t got, got2;
  int dev;
  void* p = get().take(100, &got, &dev);
  void* q = get().take(200, &got2, &dev);
  get().give(p, got, dev);
  check(card.used == 300, "held in the parent");
  std::fflush(stdout);
  const pid_t pid = fork();
  if (pid == 0) {
    failures = 0;
    get().give(q, got2, dev);
    check(card.used == 100, "not held in the child");
    get().give(get().take(300, &got, &dev), got, dev);
    check(card.used == 100, "nor later");
    get().release();
    std::exit(failures ? 1 : 0);         // runs the exit handlers
  }
  int st = -1;
  check(waitpid(pid, &st, 0) == pid && WIFEXITED(st) && WEXITSTATUS(st) == 0, "the child ends as usual");
  get().give(q, got2, dev);
  check(card.used == 300, "held in the parent after the fork");
  get().release();
  check(card.used == 0, "released in the parent");
#endif
}

// Threads that take and give at once: every block is one thread's alone.
void many_threads() {
  Card card;
  Store s(CardDev{&card}, ls::StoreLimits{16, 3000, 1, kNow, kLong});
  std::vector<std::thread> ts;
  for (int t = 0; t < 4; ++t)
    ts.emplace_back([&s, t] {
      for (int i = 0; i < 2000; ++i) {
        size_t got;
        int dev;
        unsigned char* p = static_cast<unsigned char*>(s.take(8 + 37 * (i % 29), &got, &dev)) + sizeof(size_t);
        p[0] = p[7] = (unsigned char)t;
        std::this_thread::yield();
        check(p[0] == t && p[7] == t, "nobody else writes to a block");
        s.give(p - sizeof(size_t), got, dev);
      }
    });
  for (auto& t : ts) t.join();
  check(card.used <= 3000, "within the bound");
}

}  // namespace

int main() {
  allocation_during_a_drain();
  given_back_when_idle();
  given_back_on_request();
  free_memory_is_asked_for_again();
  forked_child();
  many_threads();
  give_without_host_memory();
  bounds_of_the_store();
  for (int fail = 0; fail < 3; ++fail) {
    group_is_all_or_nothing(fail);
    solve_work_after_a_failed_growth(fail);
  }
  std::printf(failures ? "FAILED %d\n" : "ALL OK\n", failures.load());
  return failures ? 1 : 0;
}
