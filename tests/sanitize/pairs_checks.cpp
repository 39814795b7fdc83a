// The host side of the binned candidate pairs (csrc/pairs.cpp) on the CPU under
// AddressSanitizer and UBSan, built by tests/test_pair_host.py. The launches
// are counted and otherwise do nothing, device blocks come from malloc, and
// each read-back answers with the next of a list of states: what the search
// makes of them is checked. Exits 0 and prints "ok" when every check holds.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "sd_host.h"

namespace {

int pending = 0;  // launches since the stream was waited for
std::vector<sd::PairState> answers;
size_t answered = 0;
std::vector<std::string> log_;  // launches, in order
std::vector<uint64_t> looks;    // candidates in the lists at each early look
int looked = 0;
unsigned long long sent[128];
std::vector<uint32_t> rooms;    // of what each producer was given
int allocations = 0;            // the last of them fails (0: none does)

void launched(const char* what) {
  ++pending;
  log_.push_back(what);
}
int launches(const char* what) {
  int n = 0;
  for (const auto& x : log_) n += x == what;
  return n;
}

}  // namespace

namespace sd {
void* dalloc(sd_ctx*, size_t bytes) {
  if (--allocations == 0) throw Error{SD_E_NOMEM, "no memory"};
  return std::malloc(bytes < 4096 ? bytes : 4096);
}
void dfree(sd_ctx*, void* p) { std::free(p); }
void hip_check(hipError_t e, const char* what) {
  if (e != hipSuccess) throw Error{SD_E_HIP, what};
}
void* readback(sd_ctx*, const void*, size_t bytes, hipStream_t) {
  pending = 0;
  if (bytes == 1024) {  // an early look: the lists' counters, then the call's
    static uint32_t zeros[256];
    if (++looked % 2 == 0) return zeros;
    std::memset(sent, 0, sizeof(sent));
    for (int x = 0; x < 8; ++x) sent[16 * x] = looks.at((size_t)looked / 2) / 8;
    return sent;
  }
  if (answered >= answers.size()) throw Error{SD_E_STATE, "one read-back too many"};
  if (bytes != sizeof(PairState)) throw Error{SD_E_STATE, "a read-back of another size"};
  return &answers[answered++];
}
StageTimer::StageTimer(sd_ctx* ctx, hipStream_t st) : c(ctx), s(st), on(false) {}
void StageTimer::mark(const char*, double, int) {}
void launch_zero(std::initializer_list<ZeroRange>, hipStream_t) { launched("zero"); }
void launch_fill_u32(uint32_t*, uint32_t, uint64_t, hipStream_t) { launched("fill"); }
void launch_pair_split(const PairBins&, const PairBins&, PairState*, hipStream_t) {
  launched("split");
}
uint32_t pair_set_max(bool large) { return (large ? 8192u : 2048u) / 8 * 7; }
void launch_pair_verify(const PairBins&, bool, const PairSeqs&, const PairBufs&, hipStream_t) {
  launched("verify");
}
uint64_t pair_tiles(uint64_t na) { return (na + 4095) / 4096; }
void launch_pair_scan(const PairBufs&, uint64_t, hipStream_t) { launched("scan"); }
void launch_pair_place(const PairBins&, const PairBufs&, hipStream_t) { launched("place"); }
void launch_pair_order(const PairBufs&, uint64_t, uint32_t*, uint32_t*, uint8_t*, uint64_t,
                       const uint32_t*, hipStream_t) {
  launched("order");
}
}  // namespace sd

extern "C" {
hipError_t hipStreamSynchronize(hipStream_t) {
  pending = 0;
  return hipSuccess;
}
}

namespace {

int failures = 0;
void check(bool ok, const char* what) {
  std::printf("%-66s %s\n", what, ok ? "ok" : "FAILED");
  failures += !ok;
}

// a read-back: pairs kept, candidates put, flags, the call's error word
sd::PairState answer(uint64_t kept, uint64_t raw, uint32_t flags = 0, uint32_t err = 0) {
  sd::PairState s;
  std::memset(&s, 0, sizeof(s));
  s.count = kept;
  s.flags = flags;
  s.raw[3] = raw / 2;
  s.raw[40] = raw - raw / 2;
  s.counters[sd::CNT_LBERR] = err;
  return s;
}

struct Outcome {
  bool found = false;
  int code = SD_OK;
  sd::TileOut out;
  int produced = 0, checked = 0, appended = 0;
};

// one search of nkeys variants, k = 2, answered by `a` in turn; `next` is what
// its check says each time (done when it has run out)
Outcome search(uint64_t nkeys, std::vector<sd::PairState> a,
               std::vector<sd::PairNext> next = {}, sd_ctx* ctx = nullptr) {
  static sd_ctx fresh;
  sd_ctx* c = ctx ? ctx : &fresh;
  if (!ctx) c->out_hint.clear();
  answers = std::move(a);
  answered = 0;
  log_.clear();
  rooms.clear();
  looked = 0;
  pending = 0;
  Outcome o;
  uint32_t counters[sd::CNT_TOTAL] = {};
  sd::Scratch sc(c);
  sd::StageTimer tm(c, nullptr);
  sd::Call cl{c, nullptr, sc, tm, counters};
  const sd::PairSeqs q{nullptr, nullptr, nullptr, 1000, 1000, 2, 4, 1, nullptr, 0, 0};
  try {
    o.found = sd::binned_pairs(
        cl, "pairs/test", nkeys, 0, q,
        [&](const sd::PairBins& b) {
          ++o.produced;
          rooms.push_back(b.region);
          launched("produce");
        },
        [&](const sd::PairBins&) {
          ++o.appended;
          launched("append");
        },
        [&](const uint32_t*, uint64_t* more) {
          const size_t x = (size_t)o.checked++;
          if (x < next.size() && next[x] == sd::PairNext::add) *more = 100000;
          return x < next.size() ? next[x] : sd::PairNext::done;
        },
        [&](uint64_t*, uint64_t m) {
          sd::TileOut t;
          t.n = m;
          return t;
        },
        "group", &o.out);
  } catch (const sd::Error& e) {
    o.code = e.code;
  }
  if (o.found) {
    for (void* p : {(void*)o.out.i, (void*)o.out.j, (void*)o.out.d}) sd::dfree(c, p);
  }
  return o;
}

}  // namespace

int main() {
  {
    const Outcome o = search(100000, {answer(500, 3000)});
    check(o.found && o.out.n == 500 && o.out.ncand == 3000 && o.produced == 1 && pending == 0,
          "a search that fits runs once");
  }
  {
    // 100,000 / 22 + 1,024 candidates were expected: the bins held the 9,000 that
    // came, the result arrays did not
    const Outcome o = search(100000, {answer(9000, 9000)});
    check(o.found && o.out.n == 9000 && launches("order") == 2, "larger result arrays: ordered again");
    check(pending == 0, "larger result arrays: nothing in flight at the return");
  }
  {
    // a list keeps what it has room for, however many it was sent
    constexpr uint64_t past = (1ull << 32) + 5;
    static_assert(sd::list_room(0, 10, 100) == 10 && sd::list_room(95, 10, 100) == 5 &&
                      sd::list_room(100, 10, 100) == 0 && sd::list_room(past, 10, 100) == 0 &&
                      sd::list_room(past, 10, ~0u) == 0 && sd::list_room(~0u - 3ull, 10, ~0u) == 3,
                  "places past a list's room");
    static_assert(sizeof(*sd::PairBins{}.lists) == 8, "64-bit counts");
    const uint64_t limit = 0xFFFFFFFFull;
    Outcome o = search(100000000, {answer(0, limit, sd::PF_OVERFLOW)});
    check(!o.found && o.code == SD_OK && o.produced == 1 && o.checked == 0,
          "2^32 - 1 candidates: left to the path that counts each once");
    o = search(100000000, {answer(0, (9ull << 32) + 77, sd::PF_OVERFLOW)});
    check(!o.found && o.code == SD_OK && o.produced == 1, "far more than 2^32 candidates: the same");
    o = search(100000000, {answer(0, sd::PAIR_MOST, sd::PF_OVERFLOW)});
    check(!o.found && o.code == SD_OK && o.checked == 1, "as many as the bins take, without room");
    // and the next search of as many variants knows; a smaller one is not affected
    sd_ctx ctx;
    o = search(100000000, {answer(0, sd::PAIR_MOST + 1, sd::PF_OVERFLOW)}, {}, &ctx);
    check(!o.found && o.produced == 1 && sd::pairs_expected(&ctx, "pairs/test", 100000000, 2) > sd::PAIR_MOST,
          "more than the bins take: expected from now on");
    check(sd::pairs_expected(&ctx, "pairs/test", 1000, 2) < 20000, "not of a smaller search");
    sd::pairs_found(&ctx, "pairs/test", 100000000, 5000);
    check(sd::pairs_expected(&ctx, "pairs/test", 100000000, 2) == 100000000 / 22,
          "until the path that sorts found fewer");
  }
  for (const uint32_t bit : {SD_ERRBIT_LOOKBACK, SD_ERRBIT_PLACEMENT, SD_ERRBIT_INDEX}) {
    // an error of the sorts that `check` ran shows in the read-back after them
    Outcome o = search(100000, {answer(5, 3000), answer(5, 3500, 0, bit)}, {sd::PairNext::again});
    check(!o.found && o.code == SD_E_HIP && o.produced == 2, "an error bit fails the search");
    // only ids out of range are what an overflow leaves behind
    o = search(100000, {answer(5, 30000, sd::PF_OVERFLOW, bit), answer(5, 30000)});
    if (bit == SD_ERRBIT_INDEX)
      check(o.found && o.produced == 2 && launches("fill") == 1, "an overflow's ids are forgotten");
    else
      check(!o.found && o.code == SD_E_HIP && o.produced == 1, "an error bit beside an overflow too");
  }
  {
    // memory that ends anywhere in the first attempt: nothing has run
    int at = 0;
    bool idle = true;
    Outcome o;
    do {
      allocations = ++at;
      o = search(40000000, {answer(500, 3000)});
      idle = idle && (o.found || (o.code == SD_E_NOMEM && log_.empty()));
    } while (!o.found && at < 100);
    allocations = 0;
    check(o.found && at > 12 && idle, "all memory is taken before the first launch");
  }
  {
    // a large search: lists, two levels of bins after them
    Outcome o = search(100000000, {answer(500, 4000000)});
    check(o.found && o.produced == 1 && launches("split") == 2, "lists are split in two levels");
    // a later level was full: the lists are split again, not produced
    o = search(100000000, {answer(500, 4000000, sd::PF_OVERFLOW), answer(500, 4000000)});
    check(o.found && o.produced == 1 && launches("split") == 4, "full bins: the lists are split again");
    o = search(100000000, {answer(500, 9000000, sd::PF_OVERFLOW), answer(500, 9000000)});
    check(o.found && o.produced == 1 && launches("split") == 4, "the same with more than expected");
    // a list was full: produced again, with room for what the fullest was sent
    const uint32_t full = sd::PF_OVERFLOW | sd::PF_LISTS;
    sd::PairState one = answer(500, 4000000, full);
    one.lists[5] = 3900000;
    o = search(100000000, {one, answer(500, 4000000)});
    check(o.found && o.produced == 2 && rooms.back() == 3900000 + 16384, "a full list: more room");
    // and both in turn
    o = search(100000000, {one, answer(500, 4000000, sd::PF_OVERFLOW), answer(500, 4000000)});
    check(o.found && o.produced == 2 && launches("split") == 6, "a full list, then full bins");
    // more candidates come: produced again even if the bins were full too
    o = search(100000000, {answer(500, 4000000, sd::PF_OVERFLOW), answer(500, 4000000)},
               {sd::PairNext::again});
    check(o.found && o.produced == 2, "more candidates: produced again");
  }
  {
    // workgroups that only counted: their candidates go to lists, now and as long as
    // there are such workgroups
    sd_ctx ctx;
    sd::PairState few = answer(500, 2000), counted = answer(500, 90000);
    few.missed = 70000;
    counted.missed = 3;
    Outcome o = search(100000, {few, counted}, {}, &ctx);
    check(o.found && o.produced == 2 && launches("split") == 2 && o.out.ncand == 90000,
          "counted only: lists take them");
    o = search(100000, {counted}, {}, &ctx);
    check(o.found && o.produced == 1 && launches("split") == 2, "lists from the start");
    counted.missed = 0;
    o = search(100000, {counted}, {}, &ctx);
    check(o.found && launches("split") == 2, "lists once more");
    o = search(100000, {answer(500, 2000)}, {}, &ctx);
    check(o.found && launches("split") == 0, "bins again");
  }
  {
    // more candidates for lists that hold the rest: only they are put
    Outcome o = search(100000000, {answer(500, 4000000), answer(500, 4100000)}, {sd::PairNext::add});
    check(o.found && o.produced == 1 && o.appended == 1 && launches("split") == 4,
          "more candidates: appended, split again");
    sd::PairState near = answer(500, 4000000);
    near.lists[2] = 990000;  // of about a million
    o = search(100000000, {near, answer(500, 4100000)}, {sd::PairNext::add});
    check(o.found && o.produced == 2 && o.appended == 0 && rooms[1] == 990000 + 100000 / 8 + 16384,
          "no room for them: produced again, with room");
    o = search(100000, {answer(500, 3000), answer(500, 103000)}, {sd::PairNext::add});
    check(o.found && o.produced == 2 && o.appended == 0, "no lists: produced again");
    // a very large search looks at its lists first
    const uint64_t nk = 22ull << 27;
    looks = {90000000};
    o = search(nk, {answer(500, 90000000)});
    check(o.found && o.produced == 1 && o.checked == 2 && launches("split") == 2 && looked == 2,
          "an early look: the levels once");
    o = search(nk, {answer(500, 90100000)}, {sd::PairNext::add});
    check(o.found && o.produced == 1 && o.appended == 1 && launches("split") == 2,
          "an early look: more candidates before the levels");
    looks = {400000000, 400000000};
    o = search(nk, {answer(500, 400000000)});
    check(o.found && o.produced == 2 && launches("split") == 2 && rooms[1] == 50000000 + 16384,
          "an early look: full lists, produced again with room");
    looks = {sd::PAIR_MOST + 8};
    o = search(nk, {});
    check(!o.found && o.code == SD_OK && launches("split") == 0, "an early look: too many");
  }
  std::printf(failures ? "%d checks failed\n" : "ok\n", failures);
  return failures ? 1 : 0;
}
