// The layout of the partitions (csrc/part_plan.h) over every input size the
// searches and index builds give it, built by tests/test_pair_host.py. Exits 0
// and prints "ok" when every check holds.
#include "part_plan.h"

#include <cstdio>
#include <cstdlib>

namespace {

int failures = 0;
void check(bool ok, const char* what, unsigned long long nk) {
  if (ok) return;
  std::printf("%s: %llu variants FAILED\n", what, nk);
  if (++failures > 20) std::exit(1);
}

template <class F>
void sizes(uint64_t end, F&& f) {
  for (uint64_t nk = 1; nk < 5000; ++nk) f(nk);
  for (uint64_t nk = 5000; nk < end; nk += nk / 5000) f(nk);
  // around the multiples at which a plan takes more bins
  for (uint64_t mean : {512ull, 3200ull, 10240ull, 51200ull})
    for (int lb = 0; lb < 24; ++lb)
      for (int d = -2; d <= 2; ++d) {
        const uint64_t nk = (mean << lb) + (1ull << lb) + (uint64_t)d;
        if (nk < end) f(nk);
      }
  f(end - 1);
}

}  // namespace

int main() {
  using namespace sd;
  sizes(3000000000ull, [](uint64_t nk) {
    const PartPlan p = search_plan(nk);
    check(plan_fits(p, nk, nk / 16 + 65536), "search: the kernels take the plan", nk);
    check(p.lb <= 18 && p.lb - p.lb1 <= PART_MAX_SPLIT, "search: bits of a split", nk);
    check(nk < PART_BIG_KEYS || (nk >> p.lb) <= 51200, "search: elements of a bin", nk);
  });
  // a search sized by an estimate: regions for 1.2 times the most variants
  sizes(1ull << 20, [](uint64_t nk) {
    const PartPlan p = search_plan(nk);
    check(part_fits(nk * 3, p.lb1, p.nxl, nk / 16 + 65536) && p.lb == p.lb1, "search: an estimate", nk);
  });
  sizes(1ull << 31, [](uint64_t nk) {
    const PartPlan p = sort_plan(nk);
    check(plan_fits(p, nk, nk / 16 + 65536), "index: the kernels take the plan", nk);
    check((nk >> p.lb) <= SORT_BIN_MEAN, "index: elements of a bin", nk);
  });
  // a join's bins
  sizes(3000000000ull, [](uint64_t nk) {
    for (int lb = 1; lb <= PART_MAX_LB; ++lb)
      check(part_fits(nk, lb, nk >= (2u << 20) ? 3 : 0, nk / 4 + 65536), "join: positions", nk);
  });
  // the bits below the bins' never reach the id
  for (int idbits : {24, 32})
    for (int top = 1; top <= 24; ++top)
      for (int bits = 9; bits <= 17; ++bits) {
        const int s = hash_shift(top, bits, idbits);
        check(s >= idbits && s < 64 && (s == idbits || s == 64 - top - bits), "hash bits", top);
      }
  std::printf(failures ? "%d checks failed\n" : "ok\n", failures);
  return failures ? 1 : 0;
}
