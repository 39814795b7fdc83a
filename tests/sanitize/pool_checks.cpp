// The blocks of freed indexes (csrc/index_pool.cpp) on the CPU under AddressSanitizer
// and UBSan, with malloc in the device's place, built by tests/test_pair_host.py.
// Exits 0 and prints "ok" when every check holds.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#include "sd_internal.h"

namespace {
std::mutex m;
int freed = 0, current = 0;
}  // namespace

extern "C" {
hipError_t hipFree(void* p) {
  std::lock_guard<std::mutex> g(m);
  std::free(p);
  ++freed;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  std::lock_guard<std::mutex> g(m);
  current = d;
  return hipSuccess;
}
hipError_t hipDeviceTotalMem(size_t* n, hipDevice_t) {
  *n = 32 << 20;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

namespace {

int failures = 0;
void check(bool ok, const char* what) {
  std::printf("%-66s %s\n", what, ok ? "ok" : "FAILED");
  failures += !ok;
}

bool keep(sd::IndexPool& p, size_t size) {
  void* b = std::malloc(8);
  const bool kept = p.put(&b, &size, 1);
  if (!kept) std::free(b);
  return kept;
}

}  // namespace

int main() {
  auto a = sd::make_index_pool(0), b = sd::make_index_pool(0), other = sd::make_index_pool(1);
  check(a->limit == 1 << 20, "a pool keeps a 32nd of the device's memory");
  check(!keep(*a, (1 << 20) + 1) && keep(*a, 600000) && keep(*a, 400000), "no more than that");
  check(keep(*a, 500000) && freed == 2 && a->held == 500000, "the newest blocks stay");
  size_t got = 0;
  check(!a->take(440000, &got) && !a->take(500001, &got), "no block far too large, or too small");
  void* p = a->take(450000, &got);
  check(p && got == 500000 && a->held == 0, "a block that fits");
  std::free(p);
  keep(*a, 100000);
  keep(*b, 200000);
  keep(*b, 300000);
  keep(*other, 400000);
  freed = 0;
  sd::release_index_pools(0);
  check(freed == 3 && a->held == 0 && b->held == 0 && other->held == 400000,
        "a failed allocation gets every context's blocks on its device");
  b.reset();
  sd::release_index_pools(0);
  check(freed == 3, "a pool that is gone");
  // contexts that come, free, fail and go on several threads
  std::vector<std::thread> threads;
  for (int t = 0; t < 6; ++t)
    threads.emplace_back([&, t] {
      for (int x = 0; x < 300; ++x) {
        auto mine = sd::make_index_pool(0);
        keep(*mine, 1000 + t);
        keep(*a, 2000 + x);
        size_t n = 0;
        if (void* q = a->take(2000 + x / 2, &n)) hipFree(q);
        if (x % 7 == t) sd::release_index_pools(0);
      }
    });
  for (auto& t : threads) t.join();
  other.reset();
  a.reset();
  std::printf(failures ? "%d checks failed\n" : "ok\n", failures);
  return failures ? 1 : 0;
}
