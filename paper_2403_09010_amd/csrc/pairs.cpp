// Host side of the binned candidate pairs (pairs.hip): sizes, buffers and the
// one read-back of a search, and what happens when a guess was too small.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>

#include "sd_host.h"

namespace sd {

namespace {

// Bins for an expected number of candidates. A bin's hash set lies in LDS:
// 2,048 slots for a mean of up to 768 candidates; from 2^20 candidates on, and
// with three deletions (a pair can repeat 2,325 times), 8,192 slots for a mean
// of up to 4,096. Regions hold the mean, a quarter more and room for its
// deviation: bins are as even as the pair hash, but a pair comes with all its
// repeats, about 9 on average, 120 (k = 3: 500) for equal sequences, an eighth of them
// from each XCD. So the variance is taken as that many times the mean, where a
// first attempt that overflows costs the producer's work again, and as 32 times where
// it does not; and regions have four to eight hash sets' room where that is little
// memory. A set is bounded by the distinct candidates only. spread > 0, after a
// bin overflowed all the same: more room, then half as many candidates per bin
// each time.
//
// Few candidates go straight to their bins. More would leave the L2 as partial
// lines, ten times their bytes at 4M (85M candidates into 2^15 bins from the
// grouping kernel: 2.2 ms); they are appended to one list per XCD and split in
// two levels instead, a coalesced read and write each (0.65 ms). Whole searches,
// straight / split: 1.3M candidates 0.51 / 0.49 ms, 3.6M 1.10 / 1.04, 1.3M of
// weighted queries 1.41 / 1.24; below 1M the two launches cost what they save,
// unless a few workgroups put most of the candidates (`lists`). A
// list may get more than its share, since all pairs of a group of equal
// variants come from one XCD: the next attempt gives each what the fullest was sent.
struct Shape {
  PairBins b{};           // the final bins
  PairBins l1{};          // split: the first level
  bool wide = false;      // 8,192 slots
  bool split = false;
  bool fits = true;       // positions fit 32 bits
  uint64_t slots = 0;
};

// Bins of one level (2^lb bins, 2^nxl regions each).
PairBins level(uint64_t guess, int lb, int nxl, double var, uint32_t most) {
  PairBins b{};
  b.lb = lb;
  b.nbins = 1u << lb;
  b.nxl = nxl;
  const double mean = (double)guess / (double)((uint64_t)b.nbins << nxl);
  b.region =
      (uint32_t)std::min<double>(most, mean * 1.25 + 6.0 * std::sqrt(var * mean) + 32);
  // (one region per bin: counted by single atomics, which queue for their line, so
  // few bins have a line each)
  if (!nxl) b.pad = lb <= 9 ? 5 : lb <= 12 ? 2 : 0;
  return b;
}

uint64_t slots(const PairBins& b) { return ((uint64_t)b.nbins << b.nxl) * b.region; }

void take(Scratch& sc, PairBins& b) {
  if (b.lb)
    b.cursor = sc.get<uint32_t>((uint64_t)b.nbins << b.nxl << b.pad);
  else
    b.lists = sc.get<unsigned long long>((uint64_t)PAIR_LIST_STRIDE << b.nxl);
  b.base = sc.get<uint64_t>(slots(b));
}

ZeroRange cursors(const PairBins& b) {
  if (b.lists) return {reinterpret_cast<uint32_t*>(b.lists), (uint64_t)(2 * PAIR_LIST_STRIDE) << b.nxl};
  return {b.cursor, (uint64_t)b.nbins << b.nxl << b.pad};
}

Shape shape(uint64_t guess, int k, int spread, bool uneven, bool lists) {
  Shape sh;
  sh.split = lists || guess >= (1ull << 20);
  sh.wide = sh.split || k >= 3;
  const uint64_t mean_max = (sh.wide ? 4096u : 768u) >> std::max(spread - 1, 0);
  int lb = 6;
  while ((guess >> lb) > mean_max) ++lb;
  const uint32_t most = pair_set_max(sh.wide) >> (sh.split ? 3 : 0);
  if (sh.split)
    sh.b = level(guess, lb, 3, spread ? 64 : 32, spread ? 3 * most : most);
  else
    sh.b = level(guess, lb, 0, k >= 3 ? 512 : 128, k >= 3 || spread ? 3 * most : 2 * most);
  sh.slots = slots(sh.b);
  sh.fits = sh.slots < 0xFFFFFFFFull && guess <= PAIR_MOST && lb <= 18;
  if (sh.fits && sh.split)
    sh.l1 = level(guess, (lb + 1) / 2, 3, uneven ? 16384 : 1024, (uint32_t)guess);
  return sh;
}

// Searches that expect at least so many candidates read the lists' counts before the
// levels: two waits, 60 us, where the levels and the verification take 3 ms or more
// (10M sequences, k = 2, 120M expected, no copies: 13.74 ms with it, 13.65 without).
constexpr uint64_t EARLY_LOOK = 1ull << 27;

// Room for a few more candidates than were found: the same for another attempt and for
// the next search, whose blocks are then the same (560M candidates of equal sequences:
// 38 GB more at the second search where they were not).
uint64_t with_slack(uint64_t found) { return found + found / (found >= EARLY_LOOK ? 16 : 10); }

}  // namespace

uint64_t pairs_expected(const sd_ctx* c, const char* hint, uint64_t nkeys, int k) {
  constexpr double first[4] = {1.0 / 64, 1.0 / 48, 1.0 / 22, 1.0 / 9};
  double expect = (double)nkeys * first[k & 3];
  auto raw = c->out_hint.find(hint), keys = c->out_hint.find(std::string(hint) + "/variants");
  if (raw != c->out_hint.end() && keys != c->out_hint.end()) {
    const double scale = (double)nkeys / std::max((double)keys->second, 1.0);
    expect = std::max(expect, (double)with_slack(raw->second) * std::min(1.0, scale));
  }
  return (uint64_t)expect;
}

void pairs_found(sd_ctx* c, const char* hint, uint64_t nkeys, uint64_t raw) {
  c->out_hint[hint] = raw;
  c->out_hint[std::string(hint) + "/variants"] = nkeys;
}

bool binned_pairs(Call& cl0, const char* hint, uint64_t nkeys, uint64_t least,
                  const PairSeqs& q,
                  const std::function<void(const PairBins&)>& produce,
                  const std::function<void(const PairBins&)>& append,
                  const std::function<PairNext(const uint32_t*, uint64_t*)>& check,
                  const std::function<TileOut(uint64_t*, uint64_t)>& sort_pairs,
                  const char* stage, TileOut* out) {
  sd_ctx* c = cl0.c;
  hipStream_t s = cl0.s;
  const std::string hint_lists = std::string(hint) + "/lists";
  uint64_t guess = std::max(pairs_expected(c, hint, nkeys, q.k), least) + 1024;
  uint64_t cap = guess;
  int spread = 0;
  bool uneven = false;  // the level between overflowed
  auto crowded = c->out_hint.find(hint_lists);
  bool to_lists = crowded != c->out_hint.end() && crowded->second;
  // the lists that a large search's producer appends to; while they hold every
  // candidate, an attempt begins with the levels after them
  Scratch lists_sc(c);
  PairBins lists{};
  uint64_t list_room = 0;  // 0: from the guess
  bool held = false, adding = false;  // (adding: before the levels, to the lists)
  // what a list needs for what the fullest was sent and its part of `more`
  auto needs = [](const unsigned long long* sent, uint64_t more) {
    const uint64_t most = *std::max_element(sent, sent + 8);
    return std::min<uint64_t>(most + more / 8 + 16384, 0xFFFFFFFFull);
  };
  for (int attempt = 0; attempt < 8; ++attempt) {
    Scratch sc(c);
    Call cl{c, s, sc, cl0.tm, cl0.counters};
    Shape sh = shape(guess, q.k, spread, uneven, to_lists);
    if (!sh.fits) return false;
    if (sh.split && !held) {
      while (!lists_sc.blocks.empty()) lists_sc.release(lists_sc.blocks.back());
      lists = level(guess, 0, 3, 4096, (uint32_t)guess);
      if (list_room) lists.region = (uint32_t)list_room;
      take(lists_sc, lists);
    }
    const bool run = !sh.split || !held;
    PairBufs b{};
    const uint64_t tiles = pair_tiles(q.na), groups = (tiles + PAIR_GROUP - 1) / PAIR_GROUP;
    b.long_cap = (uint32_t)std::min<uint64_t>(sh.slots / 64 + 1, q.na);
    take(sc, sh.b);
    if (sh.split) take(sc, sh.l1);
    // (the pairs are placed where the level between was: no more than went through it)
    const uint64_t placed = sh.split ? std::min(sh.slots, slots(sh.l1)) : sh.slots;
    b.t = sh.split ? sh.l1.base : sc.get<uint64_t>(placed);
    b.td = sc.get<uint8_t>(placed);
    b.rank = sc.get<uint32_t>(sh.slots);
    b.kd = sc.get<uint8_t>(sh.slots);
    b.kept = sc.get<uint32_t>(sh.b.nbins);
    b.icnt = sc.get<uint32_t>(q.na);
    b.sums = sc.get<uint32_t>(tiles);
    b.groups = sc.get<uint32_t>(groups);
    b.off = sc.get<uint32_t>(q.na + 1);
    b.longs = sc.get<uint32_t>(b.long_cap);
    b.state = sc.get<PairState>(1);
    b.missed = sc.get<unsigned long long>(1);
    b.err = cl.lb_err();
    Scratch res(c);  // the result arrays, handed over at the end
    uint32_t* oi = res.get<uint32_t>(cap);
    uint32_t* oj = res.get<uint32_t>(cap);
    uint8_t* od = res.get<uint8_t>(cap);
    // (everything is taken before anything runs: where the memory does not suffice,
    // no work was for nothing)
    launch_zero({{b.icnt, q.na},
                 {b.groups, groups},
                 {reinterpret_cast<uint32_t*>(b.state), sizeof(PairState) / 4},
                 {reinterpret_cast<uint32_t*>(b.missed), 2},
                 cursors(sh.b),
                 sh.split && run ? cursors(lists) : ZeroRange{},
                 cursors(sh.l1)},
                s);
    if (run) {
      PairBins& to = sh.split ? lists : sh.b;
      to.expect = (uint32_t)std::min<uint64_t>(guess, 0xFFFFFFFFull);
      to.missed = b.missed;
      produce(to);
      cl.tm.mark(stage, (double)nkeys * 8 + (double)guess * 8, 1);
    } else if (adding) {
      append(lists);
      cl.tm.mark("append", (double)guess * 8, 1);
    }
    adding = false;
    if (run && sh.split && guess >= EARLY_LOOK) {
      // the levels take milliseconds: first look whether the lists are complete
      unsigned long long sent[8];
      const auto* l = static_cast<const unsigned long long*>(
          readback(c, lists.lists, 8 * PAIR_LIST_STRIDE * 8, s));
      for (int x = 0; x < 8; ++x) sent[x] = l[x * PAIR_LIST_STRIDE];
      uint64_t raw = 0, more = 0;
      for (unsigned long long n : sent) raw += n;
      if (raw > PAIR_MOST) {
        pairs_found(c, hint, nkeys, raw);
        return false;
      }
      const PairNext next =
          check(static_cast<const uint32_t*>(readback(c, cl.counters, CNT_TOTAL * 4, s)), &more);
      if (next == PairNext::give_up) return false;
      if (raw + more > PAIR_MOST) {
        pairs_found(c, hint, nkeys, raw + more);
        return false;
      }
      const bool full = *std::max_element(sent, sent + 8) > lists.region;
      if (full || next == PairNext::again ||
          (next == PairNext::add && needs(sent, more) > lists.region)) {
        list_room = next == PairNext::done || more ? needs(sent, more) : 0;
        guess = std::max(guess, with_slack(raw + more) + 1024);
        cap = guess;
        continue;
      }
      if (next == PairNext::add) {
        append(lists);
        cl.tm.mark("append", (double)more * 16, 1);
      }
    }
    if (sh.split) {
      launch_pair_split(lists, sh.l1, b.state, s);
      launch_pair_split(sh.l1, sh.b, b.state, s);
      cl.tm.mark("pair_split", (double)guess * 32, 2);
    }
    launch_pair_verify(sh.b, sh.wide, q, b, s);
    cl.tm.mark("pair_verify", (double)guess * (8 + 32), 1);
    launch_pair_scan(b, q.na, s);
    launch_pair_place(sh.b, b, s);
    launch_pair_order(b, q.na, oi, oj, od, cap, cl.counters, s);
    cl.tm.mark("pair_order", (double)q.na * 20, 4);
    PairState st;
    std::memcpy(&st, readback(c, b.state, sizeof(st), s), sizeof(st));
    uint64_t raw = 0, more = 0;
    for (uint64_t x : st.raw) raw += x;
    const uint64_t kept = st.count;
    const bool missed = !sh.split && st.missed;
    if (missed) raw += st.missed;
    const bool overflow = (st.flags & PF_OVERFLOW) || missed;
    if (run) to_lists = st.missed != 0;
    // (the sorts of `check` report here too, in the read-back after them)
    const uint32_t err = st.counters[CNT_LBERR];
    if (err & SD_ERRBIT_LOOKBACK) throw Error{SD_E_HIP, "internal error: a look-back wait timed out"};
    if (err & SD_ERRBIT_PLACEMENT) throw Error{SD_E_HIP, "internal error: a counted pass misplaced"};
    if (overflow)  // (a split reads slots that lost candidates never filled: ids out of range)
      launch_fill_u32(cl.lb_err(), 0, 1, s);
    else if (err & SD_ERRBIT_INDEX)
      throw Error{SD_E_HIP, "internal error: a candidate id out of range"};
    // more candidates than a search answers, or than it would without the repeats
    // of a bin that was grouped twice: the path that counts them once decides
    if (raw > PAIR_MOST) {
      pairs_found(c, hint, nkeys, raw);
      return false;
    }
    const PairNext next = check(st.counters, &more);
    if (next == PairNext::give_up || raw + more >= 0xFFFFFFFFull) return false;
    if (overflow || next != PairNext::done) {
      // more room: what was counted and what comes; where the room was there
      // but pairs have very many repeats, fewer of them per bin
      const uint64_t want = with_slack(raw + more) + 1024;
      const bool full = st.flags & PF_LISTS;
      held = sh.split && !full &&
             (next == PairNext::done ||
              (next == PairNext::add && needs(st.lists, more) <= lists.region));
      adding = held && next == PairNext::add;
      const bool mid = st.flags & PF_MID;
      if (overflow && !full && !missed && want <= guess) {
        uneven = uneven || mid;
        if (!mid) ++spread;
      }
      // (what a producer sends each list does not change; `more` is shared out in
      // chunks)
      list_room = sh.split && (more || next == PairNext::done) ? needs(st.lists, more) : 0;
      guess = std::max(guess, want);
      cap = guess;
      continue;
    }
    pairs_found(c, hint, nkeys, raw);
    c->out_hint[hint_lists] = to_lists;
    out->ncand = raw;
    if (st.flags & PF_LONG) {
      // a first id with thousands of pairs: the kept pairs take the radix sort
      *out = sort_pairs(b.t, kept);
      out->ncand = raw;
      return true;
    }
    if (kept > cap) {  // the guess held the candidates but not the pairs
      for (void* p : res.blocks) dfree(c, p);
      res.blocks.clear();
      oi = res.get<uint32_t>(kept);
      oj = res.get<uint32_t>(kept);
      od = res.get<uint8_t>(kept);
      launch_pair_order(b, q.na, oi, oj, od, kept, cl.counters, s);
      // (a call returns after its work)
      hip_check(hipStreamSynchronize(s), "synchronise");
    }
    res.blocks.clear();
    out->i = oi;
    out->j = oj;
    out->d = od;
    out->n = kept;
    return true;
  }
  return false;
}

}  // namespace sd
