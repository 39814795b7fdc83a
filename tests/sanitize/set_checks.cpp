// Which sequences of a device set the packing kernel reads (csrc/set_check.h), for
// offsets changed in up to three places, built by tests/test_pair_host.py. Exits 0
// and prints "ok" when every check holds.
#include "set_check.h"

#include <algorithm>
#include <cstdio>
#include <vector>

int main() {
  uint64_t state = 0x9E3779B97F4A7C15ull;
  auto draw = [&](uint64_t m) {
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state % m;
  };
  int failures = 0;
  auto check = [&](bool ok, const char* what) {
    if (!ok && ++failures < 20) std::printf("%s FAILED\n", what);
  };
  for (int t = 0; t < 200000; ++t) {
    const size_t n = 1 + draw(100);
    std::vector<int64_t> offs{0};
    for (size_t x = 0; x < n; ++x) offs.push_back(offs.back() + 1 + (int64_t)draw(24));
    const int64_t size = offs[n];  // of the codes
    const int64_t odd[] = {-9, 0, 3, size, size + 1, (int64_t)1 << 40, -((int64_t)1 << 62), 1400, 1410};
    for (int x = (int)draw(4); x > 0; --x)  // any offset but the last, which says how many codes there are
      offs[draw(n)] = draw(2) ? odd[draw(9)] : (int64_t)draw((uint64_t)size + 40);
    bool valid = offs[0] == 0, all = true;
    for (size_t x = 0; x < n; ++x) {
      valid = valid && offs[x] <= offs[x + 1];
      const bool in = sd::inside_set(x, offs[x], offs[x + 1], offs[n]);
      check(!in || (offs[x] >= 0 && offs[x + 1] <= size && offs[x] <= offs[x + 1]),
            "a sequence that is read lies in the codes");
      all = all && in;
    }
    check(valid == all, "sets are refused if and only if their offsets are");
  }
  std::printf(failures ? "%d checks failed\n" : "ok\n", failures);
  return failures ? 1 : 0;
}
