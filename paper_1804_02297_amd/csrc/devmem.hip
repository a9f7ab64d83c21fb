// Device memory of DevBuf: hipMalloc, with a bounded store of released blocks.
//
// A factorisation allocates and frees gigabytes (fronts, factor, maps).  The
// driver clears freed memory in the background, and once a process has gone
// through the card's memory, every further hipMalloc or hipFree of that size
// waits for it: 28 + 13 ms per 2.4 GB, where the calls take 0.2 + 0.6 ms at
// first.  Blocks of at least kMinBlock are therefore kept after release and
// handed out again:
//   * at most kMaxHeld bytes are held over all devices; the oldest go first;
//   * a block not reused within kIdle is given back at the next call here,
//     and all of them when an allocation fails (which is then tried again);
//   * a block serves only requests of at least 4/5 of its size, on its own
//     device;
//   * a release waits for the device first, as hipFree does, so a block is
//     idle on every stream before anyone can have it.
// The contents of a fresh buffer are undefined, as hipMalloc's are.
#include <chrono>
#include <list>
#include <mutex>

#include "common.h"

namespace ls {
namespace {

constexpr size_t kMinBlock = 1ull << 20;
constexpr size_t kMaxHeld = 8ull << 30;
constexpr std::chrono::seconds kIdle(20);

struct Block {
  void* p;
  size_t bytes;
  int dev;
  std::chrono::steady_clock::time_point since;
};

// Never destroyed: the process may end after the HIP runtime has.
struct Store {
  std::mutex mu;
  std::list<Block> blocks;   // oldest first
  size_t held = 0;
};
Store& store() {
  static Store* s = new Store();
  return *s;
}

// Blocks that leave the store, freed by the caller outside the lock.
void take_out(Store& s, std::list<Block>::iterator it, std::list<Block>& out) {
  s.held -= it->bytes;
  out.splice(out.end(), s.blocks, it);
}
void expired(Store& s, std::list<Block>& out) {
  const auto now = std::chrono::steady_clock::now();
  while (!s.blocks.empty() && now - s.blocks.front().since > kIdle) take_out(s, s.blocks.begin(), out);
}
void free_all(const std::list<Block>& l) {
  for (const Block& b : l) (void)hipFree(b.p);
}

}  // namespace

void* device_take(size_t bytes, size_t* got, int* dev) {
  if (hipGetDevice(dev) != hipSuccess) return nullptr;
  Store& s = store();
  void* p = nullptr;
  std::list<Block> out;
  if (bytes >= kMinBlock) {
    std::lock_guard<std::mutex> lock(s.mu);
    auto best = s.blocks.end();
    for (auto it = s.blocks.begin(); it != s.blocks.end(); ++it)
      if (it->dev == *dev && it->bytes >= bytes && it->bytes - it->bytes / 5 <= bytes &&
          (best == s.blocks.end() || it->bytes < best->bytes))
        best = it;
    if (best != s.blocks.end()) {
      p = best->p;
      *got = best->bytes;
      s.held -= best->bytes;
      s.blocks.erase(best);
    }
    expired(s, out);
  }
  free_all(out);
  if (p) return p;
  *got = bytes;
  if (hipMalloc(&p, bytes) == hipSuccess) return p;
  (void)hipGetLastError();
  out.clear();
  {
    std::lock_guard<std::mutex> lock(s.mu);
    while (!s.blocks.empty()) take_out(s, s.blocks.begin(), out);
  }
  if (out.empty()) return nullptr;
  free_all(out);
  if (hipMalloc(&p, bytes) == hipSuccess) return p;
  (void)hipGetLastError();
  return nullptr;
}

void device_give(void* p, size_t bytes, int dev) {
  int cur = -1;
  if (bytes < kMinBlock || bytes > kMaxHeld || hipGetDevice(&cur) != hipSuccess || cur != dev ||
      hipDeviceSynchronize() != hipSuccess) {
    (void)hipFree(p);
    return;
  }
  Store& s = store();
  std::list<Block> out;
  {
    std::lock_guard<std::mutex> lock(s.mu);
    expired(s, out);
    while (s.held + bytes > kMaxHeld && !s.blocks.empty()) take_out(s, s.blocks.begin(), out);
    s.blocks.push_back(Block{p, bytes, dev, std::chrono::steady_clock::now()});
    s.held += bytes;
  }
  free_all(out);
}

}  // namespace ls
