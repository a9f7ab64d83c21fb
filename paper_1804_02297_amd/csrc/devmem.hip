// Device memory of DevBuf: hipMalloc, with a bounded store of released blocks.
//
// A factorisation allocates and frees gigabytes (fronts, factor, maps).  The
// driver clears freed memory in the background, and once a process has gone
// through the card's memory, every further hipMalloc or hipFree of that size
// waits for it: 28 + 13 ms per 2.4 GB, where the calls take 0.2 + 0.6 ms at
// first.  Blocks of at least kMinBlock are therefore kept after release and
// handed out again:
//   * at most kMaxHeld bytes are held over all devices, and no more than a
//     1/kPart of what is free on the card, so that a process that needs the
//     whole card is not kept from it; the oldest go first;
//   * a block not reused within kIdle is given back by the store's own
//     thread, without any further call;
//   * all of them are given back when an allocation here fails (which is then
//     tried again), and by ls_release_memory;
//   * a block serves only requests of at least 4/5 of its size, on its own
//     device;
//   * a release waits for the device first, as hipFree does, so a block is
//     idle on every stream before anyone can have it.
// The contents of a fresh buffer are undefined, as hipMalloc's are.
// Set-ups one after another, each on a new plan (n = 29, complex128): 50 ms
// each; without the store 54 at the median, one in ten above 140 ms and the
// slowest 0.7 to 4 s (n = 48, complex64: 277 against 281, 0.8 and 1.8 s).
#include "common.h"
#include "devstore.h"

namespace ls {
namespace {

constexpr size_t kMinBlock = 1ull << 20;
constexpr size_t kMaxHeld = 8ull << 30;
constexpr int kPart = 16;
constexpr std::chrono::milliseconds kFresh(100);   // the query takes 5 us, a set-up releases some 30 blocks
constexpr std::chrono::seconds kIdle(5);   // a factor of the next medium, its stencils and the solves before it

struct HipDev {
  static bool current(int* dev) { return hipGetDevice(dev) == hipSuccess; }
  static void* alloc(size_t bytes) {
    void* p = nullptr;
    if (hipMalloc(&p, bytes) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
  }
  // also while this or another thread captures a graph, where hipFree is refused otherwise and the
  // block would be lost
  static void free(void* p) {
    hipStreamCaptureMode m = hipStreamCaptureModeRelaxed;
    const bool set = hipThreadExchangeStreamCaptureMode(&m) == hipSuccess;
    (void)hipFree(p);
    if (set) (void)hipThreadExchangeStreamCaptureMode(&m);
  }
  static bool wait(int dev) {
    int cur = -1;
    if (!current(&cur) || cur != dev) return false;
    if (hipDeviceSynchronize() == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
  }
  static size_t spare() {
    size_t bytes = 0, total = 0;
    if (hipMemGetInfo(&bytes, &total) == hipSuccess) return bytes;
    (void)hipGetLastError();
    return 0;
  }
};

BlockStore<HipDev>& store() {
  return ProcessStore<HipDev>::get(HipDev(), StoreLimits{kMinBlock, kMaxHeld, kPart, kFresh, kIdle});
}

}  // namespace

void* device_take(size_t bytes, size_t* got, int* dev) { return store().take(bytes, got, dev); }
void device_give(void* p, size_t bytes, int dev) { store().give(p, bytes, dev); }

}  // namespace ls

extern "C" void ls_release_memory(void) { ls::store().release(); }
