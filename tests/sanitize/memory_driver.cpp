// Device-memory bookkeeping of the library on a pretended device (host memory that can run out).
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "buffers.h"

namespace {

int failures = 0;
void check(bool ok, const char* what) {
  std::printf("%s: %s\n", ok ? "ok" : "FAILED", what);
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

}  // namespace

int main() {
  for (int fail = 0; fail < 3; ++fail) {
    group_is_all_or_nothing(fail);
    solve_work_after_a_failed_growth(fail);
  }
  std::printf(failures ? "FAILED %d\n" : "ALL OK\n", failures);
  return failures ? 1 : 0;
}
