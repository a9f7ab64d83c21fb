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
#include "common.h"
#include "devstore.h"

namespace ls {
namespace {

constexpr size_t kMinBlock = 1ull << 20;
constexpr size_t kMaxHeld = 8ull << 30;
constexpr std::chrono::seconds kIdle(20);

struct HipDev {
  static bool current(int* dev) { return hipGetDevice(dev) == hipSuccess; }
  static void* alloc(size_t bytes) {
    void* p = nullptr;
    if (hipMalloc(&p, bytes) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
  }
  static void free(void* p) { (void)hipFree(p); }
  static bool wait(int dev) {
    int cur = -1;
    return current(&cur) && cur == dev && hipDeviceSynchronize() == hipSuccess;
  }
};

// Never destroyed: the process may end after the HIP runtime has.
BlockStore<HipDev>& store() {
  static auto* s = new BlockStore<HipDev>(HipDev(), StoreLimits{kMinBlock, kMaxHeld, kIdle});
  return *s;
}

}  // namespace

void* device_take(size_t bytes, size_t* got, int* dev) { return store().take(bytes, got, dev); }
void device_give(void* p, size_t bytes, int dev) { store().give(p, bytes, dev); }

}  // namespace ls
