// Query-versus-reference search (paper Section II A lookup with the variant
// map built once for the reference; Section IV database lookups; Section
// III D weighted rescoring after the Levenshtein prefilter).
//
// Index build (once per reference set R and radius k):
//   pack, scan, every <= k-deletion variant of R as [hash | ref id], sorted by
//   the full hash, repeated elements removed, and a directory of 2^B hash
//   segments. The index owns its device memory and is shared read-only.
// Query (per tile of query sequences, one or many sets concatenated):
//   query_tile_binned: query variants looked up as they are generated, or in bins
//   joined with the index; id pairs through the pair bins (pairs.cpp).
//   The general tile, where that does not apply: pack, scan, query variants as
//   [hash | query id], LSD passes over the same top B hash bits, query segment
//   table, a segment-wise join against the index, pair sort, exact verification
//   (or weighted rescoring). For a batch of sets the sorted result is split into
//   per-set slices.
#include <hip/hip_runtime.h>

#include <chrono>
#include <cstdio>
#include <cstdlib>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "sd_host.h"

namespace sd {

namespace {

void pack(Call& cl, const DevSeqs& in, int k, bool distinct, u128* seq, u128* planes,
          uint32_t* vcnt, unsigned long long* sums) {
  if (in.sets)
    launch_pack_sets(in.sets, in.nsets, in.n, k, distinct, seq, planes, vcnt, cl.counters + CNT_ERR,
                     cl.s, sums);
  else
    launch_pack(in.codes, in.offs, in.n, k, distinct, seq, planes, vcnt, cl.counters + CNT_ERR,
                cl.s, sums);
}

// bad offsets come first, as in sets that are checked on the host
void raise_packed(const DevSeqs& in, uint32_t err) {
  if (in.sets && (err & SD_ERRBIT_OFFSETS)) err = SD_ERRBIT_OFFSETS;
  raise_validation(err);
}

}  // namespace

Packed pack_and_count(Call& cl, const DevSeqs& in, int k, bool distinct) {
  Packed p;
  p.seq = cl.sc.get<u128>(in.n);
  p.planes = cl.sc.get<u128>(in.n);
  uint32_t* vcnt = cl.sc.get<uint32_t>(in.n);
  p.voff = cl.sc.get<uint64_t>(in.n + 1);
  launch_fill_u32(cl.counters + CNT_ERR, 0, 1, cl.s);
  pack(cl, in, k, distinct, p.seq, p.planes, vcnt, nullptr);
  const uint64_t tiles = (in.n + scan_tile() - 1) / scan_tile();
  const uint32_t epoch = next_epoch(cl.c, tiles, cl.s);
  launch_scan_excl(vcnt, p.voff, in.n, cl.c->status, cl.tile_counter(), epoch, cl.lb_err(), cl.s);
  hip_check(hipMemcpyAsync(cl.counters + CNT_NKEYS, p.voff + in.n, 8, hipMemcpyDeviceToDevice, cl.s),
            "copy");
  const uint32_t* h =
      static_cast<const uint32_t*>(readback(cl.c, cl.counters, (CNT_NKEYS + 2) * 4, cl.s));
  raise_packed(in, h[CNT_ERR]);
  std::memcpy(&p.nkeys, h + CNT_NKEYS, 8);
  if (p.nkeys >= 0xFFFFFFFFull) throw Error{SD_E_TOO_MANY, "more than 2^32 - 2 deletion variants"};
  return p;
}

void check_lookback(Call& cl) {
  const uint32_t* h = static_cast<const uint32_t*>(readback(cl.c, cl.counters + CNT_LBERR, 4, cl.s));
  if (h[0] & SD_ERRBIT_LOOKBACK) throw Error{SD_E_HIP, "internal error: a look-back wait timed out"};
  if (h[0] & SD_ERRBIT_PLACEMENT) throw Error{SD_E_HIP, "internal error: a counted pass misplaced"};
}

namespace {

constexpr uint32_t JOIN_LDS_MIN_Q = 8;  // segments with fewer query elements search global memory

int index_bits(uint64_t nkeys) {
  // segments of about 1/2 to 1/4 of the join kernel's LDS capacity
  int b = 0;
  while (b < 24 && (double)nkeys / (double)(1ull << b) > 0.4 * join_cap()) ++b;
  return b;
}

// Hash bits of a query tile's join segments: the index's own B, or fewer
// for a small tile (about `per` query elements a segment, at least 2^4
// segments; `per` is the cube root of the tile's element count, at least
// 64, unless SD_OPT_JOIN_ELEMS sets it; 1 keeps the index's own). The join runs one workgroup per segment, so with the
// index's 2^B segments a small query would launch mostly workgroups that
// find no query element, and each would stage its index segment in LDS for
// a few lookups; a coarser segment is the union of 2^(B - bits) index
// segments, searched in global memory.
int join_bits(const sd_ctx* c, const sd_index* idx, uint64_t nk) {
  if (c->join_elems == 1) return idx->bits;  // the index's own segments
  const uint64_t per =
      c->join_elems ? (uint64_t)c->join_elems : std::max<uint64_t>(64, (uint64_t)std::cbrt((double)nk));
  int b = 4;
  while (b < 24 && (nk >> (b + 1)) >= per) ++b;
  return std::min(b, idx->bits);
}

// Up to one query variant per 64 index elements the variants are looked up one
// by one, beyond that they are joined by reading the whole index: a lookup
// costs three to four scattered cache lines, an index element 8 bytes. k = 2,
// whole calls in ms, looked up / joined: 2M references, 10K queries 0.31 /
// 0.49, 30K 0.56 / 0.55, 200K 2.53 / 0.74; 5M references, 60K 1.01 / 1.18, 100K
// 1.49 / 1.29; 200K references, 3K 0.16 / 0.18, 10K 0.25 / 0.20.
constexpr uint64_t PROBE_RATIO = 64;

// A tile of queries against a hashed index through the pair bins: few queries
// look their variants up as they are generated, many are partitioned into bins
// and joined with the index's segments. Returns false where the general path
// has to run (positions beyond 32 bits, no shape of the pair bins that fits, more
// copies than the overflow area holds).
bool query_tile_binned(Call& cl0, const sd_index* idx, const DevSeqs& q, int k,
                       const WeightedSpec* w, TileOut* out) {
  sd_ctx* c = cl0.c;
  hipStream_t s = cl0.s;
  Scratch sc(c);
  Call cl{c, s, sc, cl0.tm, cl0.counters};
  u128* seq = sc.get<u128>(q.n);
  u128* planes = sc.get<u128>(q.n);
  uint32_t* vcnt = sc.get<uint32_t>(q.n);
  pack(cl, q, k, true, seq, planes, vcnt,
       reinterpret_cast<unsigned long long*>(cl.counters + CNT_SUMS));
  cl.tm.mark("q_pack_scan", (double)q.n * 48, 1);
  // small sets are not waited for here: their variants are looked up whatever
  // their number, and the flags are read with the result
  uint64_t nk = q.n * TYPICAL_VARIANTS[k];
  const bool known = nk > UNREAD_KEYS || nk * PROBE_RATIO > idx->n_keys;
  if (known) {
    const uint32_t* h = static_cast<const uint32_t*>(readback(c, cl.counters, CNT_TOTAL * 4, s));
    raise_packed(q, h[CNT_ERR]);
    nk = pack_total(h);
    if (nk >= 0xFFFFFFFFull) throw Error{SD_E_TOO_MANY, "more than 2^32 - 2 deletion variants"};
  }
  bool join = known && nk * PROBE_RATIO > idx->n_keys && idx->bits >= 1 && nk < 3000000000ull;
  // bins of the query elements (2,048 at most: longer runs of the generator's
  // tiles; 4,096 if those would hold more than 16K: 76M query elements against
  // 202M are generated in 0.36 or 0.45 ms and joined in 0.87 or 0.70), and as few
  // workgroups per bin as their LDS takes: each reads the bin's query elements,
  // and of its index elements about 3% have a query of the same hash and as many
  // others pass as the bitmap is filled
  PartOut p{};
  JoinParts parts{};
  uint64_t over_cap = 0;
  int sub = 0;
  if (join) {
    int lb = 1;
    const int most = (nk >> 11) > 16384 ? PART_MAX_LB : 11;
    while (lb < std::min(most, idx->bits) && (nk >> lb) > 2048) ++lb;
    auto too_many = [&] {
      const double mq = (double)(nk >> lb) / (1 << sub);
      const double mr = (double)(idx->n_keys >> lb) / (1 << sub);
      return mq > JOIN_QUERY_MAX || mr * (mq / JOIN_BITMAP + 0.03) > JOIN_SURVIVORS;
    };
    while (lb + sub < idx->bits && too_many()) ++sub;
    // (copies among the queries go to the overflow area: room for all elements where
    // memory is not bounded)
    const int nxl = nk >= (2u << 20) ? 3 : 0;
    over_cap = !memory_bounded(c) && nk <= (1ull << 28) ? nk : nk / 16 + 65536;
    p = part_out(cl, nk, lb, nxl, over_cap, cl.counters + CNT_OVER);
  }
  bool generated = !join;
  auto generate = [&] {
    generated = true;
    launch_gen_part(seq, vcnt, q.n, nk, k, idx->idbits, p, s);
    cl.tm.mark("q_vargen_part", (double)nk * 8 + (double)q.n * 20, 1);
  };
  // (the device waits for it: everything else is taken afterwards)
  if (join && !memory_bounded(c)) generate();
  if (join) parts = JoinParts{sc.get<JoinPart>(join_parts(p, sub)), cl.counters + CNT_PARTS};
  const char* const hint = join ? "pairs/join" : "pairs/probe";
  const std::string hint_runs = std::string(hint) + "/runs";
  // copies, if there are any: what the join left and long runs are followed up by
  // kernels of their own (known from the attempt before, or the last search)
  uint64_t runs = c->out_hint[hint_runs];
  bool follow = runs > 0, again = false;
  runs += runs / 4 + 4096;
  RunQueue queue{nullptr, 0, cl.counters + CNT_RUNS,
                 reinterpret_cast<unsigned long long*>(cl.counters + CNT_MISSED)};
  const bool hamming = c->metric == SD_METRIC_HAMMING;
  const PairSeqs ps{w ? planes : hamming ? seq : planes,
                    idx->ref_seq,
                    w ? seq : nullptr,
                    q.n,
                    idx->n_ref,
                    k,
                    w ? 3 : hamming ? 1 : 0,
                    0,
                    w ? w->subst : nullptr,
                    w ? w->indel : 0,
                    w ? w->max_score : 0};
  auto make_queue = [&] {
    if (queue.cap >= runs) return;
    queue.runs = sc.get<PairRun>(runs);
    queue.cap = (uint32_t)runs;
  };
  auto put_copies = [&](const PairBins& bins) {
    if (join)
      launch_join_runs(p, idx->E, idx->seg_start, idx->seg_end, idx->bits, sub, idx->idbits,
                       parts, queue, s);
    launch_put_runs(idx->E, idx->idbits, queue, queue.cap, bins, s);
  };
  const bool done = binned_pairs(
      // (queries that are in the index find each of their variants there: bins for that
      // cost nothing, and their counters have lines of their own: 3,000 queries of 5M
      // references 239 us, 233 with them)
      cl, hint, nk, join ? 0 : std::min<uint64_t>(nk + nk / 4, 640 << 10), ps,
      [&](const PairBins& bins) {
        if (again) launch_fill_u32(cl.counters + CNT_PARTS, 0, 4, s);
        if (!generated) generate();
        again = true;
        if (follow) make_queue();
        if (join)
          launch_join_bins(p, idx->E, idx->seg_start, idx->seg_end, idx->bits, sub, idx->idbits,
                           bins, parts, s);
        else
          launch_gen_probe(seq, q.n, k, idx->E, (uint32_t)idx->n_keys, idx->seg_start, idx->seg_end, idx->bits,
                           idx->idbits, bins, queue, s);
        if (follow) put_copies(bins);
      },
      [&](const PairBins& bins) {
        make_queue();
        put_copies(bins);
      },
      [&](const uint32_t* h, uint64_t* more) {
        if (!known) raise_packed(q, h[CNT_ERR]);
        nk = pack_total(h);
        if (join && h[CNT_OVER] > over_cap) return PairNext::give_up;
        const uint64_t over = join ? h[CNT_OVER] : 0, left = h[CNT_PARTS], queued = h[CNT_RUNS];
        const bool copies = over || left || queued;
        c->out_hint[hint_runs] = copies ? std::max<uint64_t>(queued, 1) : 0;
        if (!copies || (follow && queued <= queue.cap)) return PairNext::done;
        // what is queued, or about what the parts will queue
        runs = std::max(queued, over + left * 4096) + 4096;
        if (runs > (1ull << 30)) return PairNext::give_up;
        // (their candidates, from those that were summed; the next count is exact)
        if (queued > queue.cap) {
          unsigned long long sum = 0;
          std::memcpy(&sum, h + CNT_MISSED, 8);
          const double beyond = (double)(queued - queue.cap);
          *more = (uint64_t)std::min((double)sum * beyond / std::min(beyond, (double)RUN_SAMPLE),
                                     (double)(1u << 28));
        }
        // (a join's parts and its overflow area are still there; lookups queue anew)
        const PairNext next = join && !follow ? PairNext::add : PairNext::again;
        follow = true;
        return next;
      },
      [&](uint64_t* cand, uint64_t m) {
        return verify_candidates(cl, seq, planes, q.n, idx->ref_seq, idx->n_ref, cand, m, k, w);
      },
      "join", out);
  out->nkeys = nk;
  return done;
}

// One tile of queries: returns pool blocks (i = tile-local query id, j = ref
// id, d) sorted by (i, j) and their count.
TileOut query_tile(Call& cl, const sd_index* idx, const DevSeqs& q, int k, const WeightedSpec* w) {
  sd_ctx* c = cl.c;
  hipStream_t s = cl.s;
  TileOut out;
  if (q.n == 0) return out;
  if (idx->learned) return learned_tile(cl, idx, q, k, w);
  if (q.n >= (1ull << idx->idbits)) throw Error{SD_E_TOO_MANY, "query tile exceeds the index id width"};
  // (the knobs of the general path choose it)
  if (!c->join_elems && !c->pair_sort && !c->sort_items && if_memory_suffices(c, [&] {
        return query_tile_binned(cl, idx, q, k, w, &out);
      }))
    return out;
  out = TileOut();
  const Packed p = pack_and_count(cl, q, k, true);
  out.nkeys = p.nkeys;
  const uint32_t nk = (uint32_t)p.nkeys;
  cl.tm.mark("q_pack_scan", (double)q.n * 56, 2);

  // query elements, grouped by the top hash bits of the join segments
  const int bits = join_bits(c, idx, nk);
  const std::vector<Digit> digits = bits ? top_digits(64 - bits) : std::vector<Digit>();
  uint64_t* e1 = cl.sc.get<uint64_t>(nk);
  uint64_t* e2 = cl.sc.get<uint64_t>(nk);
  uint32_t* hist = cl.sc.get<uint32_t>(3 * 256);
  launch_fill_u32(hist, 0, 3 * 256, s);
  uint32_t shifts[3] = {0, 0, 0}, masks[3] = {0, 0, 0};
  for (size_t x = 0; x < digits.size(); ++x) {
    shifts[x] = (uint32_t)digits[x].shift;
    masks[x] = digits[x].mask;
  }
  const uint32_t spt = vargen_seqs_per_tile(q.n, nk);
  uint32_t* tcounts = nullptr;
  if (!digits.empty()) {
    tcounts = cl.sc.get<uint32_t>(((q.n + spt - 1) / spt) * 256);
  }
  launch_vargen_hash(p.seq, p.voff, q.n, k, true, e1, idx->idbits, digits.empty() ? 0 : 1, shifts,
                     masks, hist, tcounts, spt, s);
  std::vector<const uint32_t*> hists;
  for (size_t x = 0; x < digits.size(); ++x) hists.push_back(hist + 256 * x);
  // the first pass from the generator's counts, the later ones counted over
  // fixed tiles
  const CountedFirst first{tcounts, (q.n + spt - 1) / spt, p.voff, spt, q.n};
  bool flip = false;
  if (!digits.empty()) {
    flip = radix_sort(cl, e1, nullptr, nullptr, e2, nullptr, nullptr, 1, false, nk,
                      std::vector<Digit>(digits.begin(), digits.begin() + 1),
                      std::vector<const uint32_t*>(hists.begin(), hists.begin() + 1), &first);
    if (digits.size() > 1) {
      const bool f2 = counted_sort(cl, flip ? e2 : e1, flip ? e1 : e2, nk,
                                   std::vector<Digit>(digits.begin() + 1, digits.end()));
      if (f2) flip = !flip;
    }
  }
  const uint64_t* Eq = flip ? e2 : e1;
  const uint32_t nseg = 1u << bits;
  uint32_t* qs = cl.sc.get<uint32_t>(nseg);
  uint32_t* qe = cl.sc.get<uint32_t>(nseg);
  launch_seg_bounds(Eq, nk, 64u - (uint32_t)bits, qs, qe, s);
  // the index's segments at the same bits (its own directory, or coarser
  // bounds found in its sorted array)
  const uint32_t* rs = idx->seg_start;
  const uint32_t* re = idx->seg_end;
  if (bits < idx->bits) {
    uint32_t* crs = cl.sc.get<uint32_t>(nseg);
    uint32_t* cre = cl.sc.get<uint32_t>(nseg);
    launch_seg_bounds(idx->E, idx->n_keys, 64u - (uint32_t)bits, crs, cre, s);
    rs = crs;
    re = cre;
  }
  cl.tm.mark("q_vargen_passes", (double)nk * (8 + 16 * digits.size()),
             (bits < idx->bits ? 3 : 2) + (int)digits.size());

  // join against the index
  Cands cj = sharded_output(
      cl, nk / 4, "join",
      [&](const ShardArgs& out) {
        launch_join_seg(idx->E, rs, re, Eq, qs, qe, nseg, idx->idbits, JOIN_LDS_MIN_Q, out, s);
      },
      [&](uint64_t n) { return (double)nk * 8 + (double)n * 8; });
  cl.sc.blocks.push_back(cj.p);
  uint64_t* cand = cj.p;
  const uint64_t nc = cj.n;
  out.ncand = nc;
  TileOut v = verify_candidates(cl, p.seq, p.planes, q.n, idx->ref_seq, idx->n_ref, cand, nc, k, w);
  v.nkeys = out.nkeys;
  v.ncand = nc;
  return v;
}

}  // namespace

TileOut query_tile_eager(Call& cl, const sd_index* idx, const DevSeqs& q, int k) {
  return query_tile(cl, idx, q, k, nullptr);
}

namespace {

void check_index(const sd_ctx* c, const sd_index* idx, int k) {
  if (!idx) throw Error{SD_E_INVAL, "null index"};
  if (idx->device != c->device) throw Error{SD_E_INVAL, "index lives on another device"};
  if (k < 0 || k > idx->k) throw Error{SD_E_INVAL, "k must lie in [0, the index's k]"};
}

}  // namespace

// Sort (q, r) candidate pairs over the digits that can differ, then verify
// (or rescore) and compact them in order.
TileOut verify_candidates(Call& cl, const u128* qseq, const u128* qplanes, uint64_t nq,
                          const u128* rseq, uint64_t nr,
                          uint64_t* cand, uint64_t nc, int k, const WeightedSpec* w) {
  sd_ctx* c = cl.c;
  hipStream_t s = cl.s;
  TileOut out;
  if (nc >= 0xFFFFFFFFull) throw Error{SD_E_TOO_MANY, "more than 2^32 - 2 candidate pairs"};

  // unweighted: buckets by the top bits of q, each sorted and verified in LDS
  const int rbits = bits_for(nr ? nr - 1 : 0), qbits = bits_for(nq ? nq - 1 : 0);
  const BucketPlan bp = w ? BucketPlan() : bucket_plan(c, nc, qbits, rbits);
  if (bp.bits >= 0) {
    c->stats.n_pair_buckets += bp.nb;
    uint64_t* cand2 = cl.sc.get<uint64_t>(nc);
    out.i = dalloc_t<uint32_t>(c, nc);
    out.j = dalloc_t<uint32_t>(c, nc);
    out.d = dalloc_t<uint8_t>(c, nc);
    bool over = false;
    try {
      out.n = bucket_sort_verify(cl, bp, cand, nc, cand2, nq, nr,
                                 c->metric == SD_METRIC_HAMMING ? qseq : qplanes, rseq, k, 0,
                                 out.i, out.j, out.d, &over, "q_pair_sort", "q_verify");
    } catch (...) {
      dfree(c, out.i);
      dfree(c, out.j);
      dfree(c, out.d);
      throw;
    }
    if (!over) return out;
    dfree(c, out.i);
    dfree(c, out.j);
    dfree(c, out.d);
    out = TileOut();
    c->stats.n_pair_fallbacks += 1;
    cand = cand2;  // every candidate, bucketed (the first array was overwritten)
  }

  // sort (q, r) pairs over the digits that can differ
  const uint64_t* sorted = cand;
  if (nc > 1) {
    uint64_t* cand2 = cl.sc.get<uint64_t>(nc);
    std::vector<Digit> pd;
    const int rb = bits_for(nr ? nr - 1 : 0), qb = bits_for(nq ? nq - 1 : 0);
    for (int x = 0; x < (rb + 7) / 8; ++x) pd.push_back(Digit{0, 8 * x, 255u});
    for (int x = 0; x < (qb + 7) / 8; ++x) pd.push_back(Digit{0, 32 + 8 * x, 255u});
    bool pf;
    if (pair_sort_counted(c, nc)) {
      // large: counted passes over fixed tiles
      pf = counted_sort(cl, cand, cand2, (uint32_t)nc, pd);
    } else {
      // small: one histogram, then onesweep passes (fewer launches)
      uint32_t* phist = cl.sc.get<uint32_t>(8 * 256);
      launch_fill_u32(phist, 0, 8 * 256, s);
      launch_radix_hist(cand, nullptr, 1, nc, phist, s);
      std::vector<const uint32_t*> ph;
      for (const Digit& d : pd) ph.push_back(phist + (d.shift / 8) * 256);
      pf = radix_sort(cl, cand, nullptr, nullptr, cand2, nullptr, nullptr, 1, false, (uint32_t)nc,
                      pd, ph);
    }
    sorted = pf ? cand2 : cand;
  }
  cl.tm.mark("q_pair_sort", (double)nc * 16, 1);

  // verify (or rescore) and compact
  out.i = dalloc_t<uint32_t>(c, nc);
  out.j = dalloc_t<uint32_t>(c, nc);
  out.d = dalloc_t<uint8_t>(c, nc);
  try {
    unsigned long long* pcount = reinterpret_cast<unsigned long long*>(cl.counters + CNT_PAIRS);
    launch_fill_u64(reinterpret_cast<uint64_t*>(pcount), 0, 1, s);
    if (nc) {
      if (w) {
        const uint64_t tiles = (nc + weighted_tile() - 1) / weighted_tile();
        const uint32_t epoch = next_epoch(c, tiles, s);
        launch_verify_weighted(sorted, nc, qseq, rseq, k, w->subst, w->indel,
                               w->max_score, out.i, out.j, out.d, c->status, cl.tile_counter(),
                               epoch, pcount, cl.lb_err(), s);
      } else {
        const uint64_t tiles = (nc + compact_tile() - 1) / compact_tile();
        const uint32_t epoch = next_epoch(c, tiles, s);
        launch_verify_compact(sorted, nc, nq, nr, c->metric == SD_METRIC_HAMMING ? qseq : qplanes, rseq, k,
                              c->metric, 0, out.i, out.j, out.d, c->status,
                              cl.tile_counter(), epoch, pcount, cl.lb_err(), s);
      }
    }
    const uint32_t* h = static_cast<const uint32_t*>(readback(c, cl.counters + CNT_PAIRS, 12, s));
    uint64_t cnt;
    std::memcpy(&cnt, h, 8);
    if (h[2] & SD_ERRBIT_LOOKBACK) throw Error{SD_E_HIP, "internal error: a look-back wait timed out"};
    if (h[2] & SD_ERRBIT_PLACEMENT) throw Error{SD_E_HIP, "internal error: a counted pass misplaced"};
    if (h[2] & SD_ERRBIT_INDEX) throw Error{SD_E_HIP, "internal error: a candidate id out of range"};
    out.n = nc ? cnt : 0;
    cl.tm.mark("q_verify", (double)nc * 49, 1);
  } catch (...) {
    dfree(c, out.i);
    dfree(c, out.j);
    dfree(c, out.d);
    throw;
  }
  return out;
}

void index_free(sd_index* idx) {
  if (!idx) return;
  (void)hipSetDevice(idx->device);
  void* const blocks[] = {idx->ref_seq, idx->E,   idx->seg_start, idx->seg_end, idx->keys,
                          idx->kid,     idx->params, idx->coord,     idx->leaves};
  index_release(idx, blocks, 9);
  delete idx;
}

namespace {

// The nk variants of n packed sequences, in order, to E, by a partition into
// bins of their top hash bits and a sort of each bin in LDS. Bins too large for
// that (single variants shared by thousands of sequences) are sorted together
// by digit passes and put in their places. Returns the distinct elements, or 0
// if an overflow area was too small or those bins hold over a quarter of the
// elements: digit passes over everything do as well then.
//
// Against one histogram, five digit passes over everything and a copy: 2M
// sequences, k = 2 (202M elements), 14.5 and 2.4 ms of kernels.
uint64_t sorted_bins(Call& cl0, const u128* seq, const uint32_t* vcnt, uint64_t n, uint64_t nk,
                     int k, uint32_t idbits, uint64_t* E) {
  sd_ctx* c = cl0.c;
  hipStream_t s = cl0.s;
  Scratch sc(c);
  Call cl{c, s, sc, cl0.tm, cl0.counters};
  const PartPlan plan = sort_plan(nk);
  const int lb = plan.lb, lb1 = plan.lb1, nxl = plan.nxl;
  const uint64_t over_cap = nk / 16 + 65536;
  if (!plan_fits(plan, nk, over_cap)) return 0;
  uint32_t* over = cl.counters + CNT_OVER;
  const PartOut p1 = part_out(cl, nk, lb1, nxl, over_cap, lb1 < lb ? over + 1 : over);
  const PartOut p = lb1 < lb ? part_out(cl, nk, lb, nxl, over_cap, over) : p1;
  uint64_t* off = sc.get<uint64_t>(p.nbins + 1);
  uint32_t* cnt = sc.get<uint32_t>(p.nbins);
  const uint64_t big_cap = ((uint64_t)p.nbins << nxl) + 1;
  uint64_t* big = sc.get<uint64_t>(2 * big_cap);
  // (all memory is taken before the first launch)
  launch_gen_part(seq, vcnt, n, nk, k, idbits, p1, s);
  if (lb1 < lb) launch_part_split(p1, p, s);
  const uint64_t tiles = (p.nbins + scan_tile() - 1) / scan_tile();
  const uint32_t epoch = next_epoch(c, tiles, s);
  launch_bin_offsets(p, cnt, off, c->status, cl.tile_counter(), epoch, cl.lb_err(), s);
  auto* nbig = reinterpret_cast<unsigned long long*>(cl.counters + CNT_NBIG);
  auto* repeats = reinterpret_cast<unsigned long long*>(cl.counters + CNT_CAND);
  launch_sort_bins(p, off, E, big, nbig, repeats, s);
  auto counters = [&] {
    const uint32_t* h = static_cast<const uint32_t*>(readback(c, cl.counters, CNT_TOTAL * 4, s));
    if (h[CNT_LBERR] & SD_ERRBIT_LOOKBACK)
      throw Error{SD_E_HIP, "internal error: a look-back wait timed out"};
    if (h[CNT_LBERR] & SD_ERRBIT_PLACEMENT)
      throw Error{SD_E_HIP, "internal error: a counted pass misplaced"};
    return h;
  };
  const uint32_t* h = counters();
  if (h[CNT_OVER1] || h[CNT_OVER] > over_cap) return 0;
  uint64_t nb, rep;
  std::memcpy(&nb, h + CNT_NBIG, 8);
  std::memcpy(&rep, h + CNT_CAND, 8);
  if (nb) {
    std::vector<uint64_t> hb(2 * (nb + 1)), start(nb + 1);
    hip_check(hipMemcpyAsync(hb.data(), big, nb * 16, hipMemcpyDeviceToHost, s), "D2H big");
    const uint64_t n_over = h[CNT_OVER];
    hip_check(hipStreamSynchronize(s), "synchronise");
    hb[2 * nb] = p.slots;
    hb[2 * nb + 1] = p.slots + n_over;
    uint64_t tot = 0;
    for (uint64_t x = 0; x <= nb; ++x) {
      start[x] = tot;
      tot += hb[2 * x + 1] - hb[2 * x];
    }
    if (tot > nk / 4 + 65536) return 0;
    uint64_t* dstart = sc.get<uint64_t>(nb + 1);
    hip_check(hipMemcpyAsync(big, hb.data(), (nb + 1) * 16, hipMemcpyHostToDevice, s), "H2D big");
    hip_check(hipMemcpyAsync(dstart, start.data(), (nb + 1) * 8, hipMemcpyHostToDevice, s),
              "H2D starts");
    uint64_t* g1 = sc.get<uint64_t>(tot);
    uint64_t* g2 = sc.get<uint64_t>(tot);
    launch_gather_big(p.elem, big, dstart, (uint32_t)(nb + 1), g1, s);
    uint32_t* hist = sc.get<uint32_t>(8 * 256);
    launch_fill_u32(hist, 0, 8 * 256, s);
    launch_radix_hist(g1, nullptr, 1, tot, hist, s);
    const std::vector<Digit> digits = top_digits(0);
    std::vector<const uint32_t*> hists;
    for (const Digit& d : digits) hists.push_back(hist + (d.shift / 8) * 256);
    const bool flip = radix_sort(cl, g1, nullptr, nullptr, g2, nullptr, nullptr, 1, false,
                                 (uint32_t)tot, digits, hists);
    launch_place_bins(flip ? g2 : g1, tot, p.lb, off, E, repeats, s);
    h = counters();
    std::memcpy(&rep, h + CNT_CAND, 8);
  }
  if (!rep) return nk;
  // two variants of one sequence share a hash: rare, dropped by a pass over all
  uint64_t* uniq = sc.get<uint64_t>(nk);
  const uint64_t utiles = (nk + unique_tile() - 1) / unique_tile();
  const uint32_t uepoch = next_epoch(c, utiles, s);
  launch_fill_u64(reinterpret_cast<uint64_t*>(repeats), 0, 1, s);
  launch_unique_compact(E, nk, uniq, c->status, cl.tile_counter(), uepoch, repeats, cl.lb_err(), s);
  h = counters();
  uint64_t left;
  std::memcpy(&left, h + CNT_CAND, 8);
  hip_check(hipMemcpyAsync(E, uniq, left * 8, hipMemcpyDeviceToDevice, s), "copy index");
  return left;
}

// The same by digit passes over all elements; idx->E is taken here if it is not yet.
uint64_t sorted_passes(Call& cl, sd_index* idx, const u128* seq, const uint32_t* vcnt, uint64_t n,
                       uint64_t nk, int k) {
  sd_ctx* c = cl.c;
  hipStream_t s = cl.s;
  uint64_t* voff = cl.sc.get<uint64_t>(n + 1);
  const uint64_t stiles = (n + scan_tile() - 1) / scan_tile();
  const uint32_t sepoch = next_epoch(c, stiles, s);
  launch_scan_excl(vcnt, voff, n, c->status, cl.tile_counter(), sepoch, cl.lb_err(), s);
  uint64_t* e1 = cl.sc.get<uint64_t>(nk);
  uint64_t* e2 = cl.sc.get<uint64_t>(nk);
  uint32_t* unused = cl.sc.get<uint32_t>(3 * 256);
  const uint32_t z[3] = {0, 0, 0};
  launch_vargen_hash(seq, voff, n, k, true, e1, idx->idbits, 0, z, z, unused, nullptr,
                     VG_MAX_SEQS_PER_BLOCK, s);
  uint32_t* hist = cl.sc.get<uint32_t>(8 * 256);
  launch_fill_u32(hist, 0, 8 * 256, s);
  launch_radix_hist(e1, nullptr, 1, nk, hist, s);
  const std::vector<Digit> digits = top_digits((int)idx->idbits);
  std::vector<const uint32_t*> hists;
  for (const Digit& d : digits) hists.push_back(hist + (d.shift / 8) * 256);
  const bool flip = radix_sort(cl, e1, nullptr, nullptr, e2, nullptr, nullptr, 1, false,
                               (uint32_t)nk, digits, hists);
  uint64_t* sorted = flip ? e2 : e1;
  uint64_t* uniq = flip ? e1 : e2;
  unsigned long long* ucount = reinterpret_cast<unsigned long long*>(cl.counters + CNT_CAND);
  const uint64_t tiles = (nk + unique_tile() - 1) / unique_tile();
  const uint32_t epoch = next_epoch(c, tiles, s);
  launch_fill_u64(reinterpret_cast<uint64_t*>(ucount), 0, 1, s);
  launch_unique_compact(sorted, nk, uniq, c->status, cl.tile_counter(), epoch, ucount,
                        cl.lb_err(), s);
  const uint64_t left = *static_cast<const uint64_t*>(readback(c, ucount, 8, s));
  check_lookback(cl);
  if (!idx->E) idx->E = static_cast<uint64_t*>(index_alloc(c, idx, std::max<uint64_t>(left, 1) * 8));
  hip_check(hipMemcpyAsync(idx->E, uniq, left * 8, hipMemcpyDeviceToDevice, s), "copy index");
  return left;
}

}  // namespace

sd_index* index_build(sd_ctx* c, const sd_seqs* ref, int k, hipStream_t s) {
  check_seqs(ref);
  if (k < 0 || k > 3) throw Error{SD_E_INVAL, "k must be 0, 1, 2 or 3"};
  sd_index* idx = new sd_index();
  idx->device = c->device;
  idx->k = k;
  idx->n_ref = (uint64_t)ref->n;
  idx->idbits = ref->n <= (1ll << 24) ? 24u : 32u;
  try {
    Scratch sc(c);
    StageTimer tm(c, s);
    Call cl{c, s, sc, tm, fresh_counters(c, CNT_TOTAL, s)};
    const DevSeqs in = stage_seqs(c, sc, ref, s);
    idx->ref_seq = static_cast<u128*>(index_alloc(c, idx, std::max<uint64_t>(in.n, 1) * 16));
    uint64_t nk = 0;
    if (in.n) {
      uint32_t* vcnt = sc.get<uint32_t>(in.n);
      launch_pack(in.codes, in.offs, in.n, k, true, idx->ref_seq, sc.get<u128>(in.n), vcnt,
                  cl.counters + CNT_ERR, s,
                  reinterpret_cast<unsigned long long*>(cl.counters + CNT_SUMS));
      const uint32_t* h =
          static_cast<const uint32_t*>(readback(c, cl.counters, CNT_TOTAL * 4, s));
      raise_validation(h[CNT_ERR]);
      nk = pack_total(h);
      if (nk >= 0xFFFFFFFFull)
        throw Error{SD_E_TOO_MANY, "more than 2^32 - 2 deletion variants"};
      uint64_t kept = 0;
      // (positions of up to 2^31 elements and their regions' slack take 32 bits;
      // the digit passes' knob chooses them)
      if (nk < (1ull << 31) && !c->sort_items)
        if_memory_suffices(c, [&] {
          idx->E = static_cast<uint64_t*>(index_alloc(c, idx, nk * 8));
          return (kept = sorted_bins(cl, idx->ref_seq, vcnt, in.n, nk, k, idx->idbits, idx->E)) > 0;
        });
      if (!kept) kept = sorted_passes(cl, idx, idx->ref_seq, vcnt, in.n, nk, k);
      nk = kept;
    }
    idx->n_keys = nk;
    idx->bits = index_bits(nk);
    const uint32_t nseg = 1u << idx->bits;
    if (!idx->E) idx->E = static_cast<uint64_t*>(index_alloc(c, idx, 8));
    idx->seg_start = static_cast<uint32_t*>(index_alloc(c, idx, (size_t)nseg * 4));
    idx->seg_end = static_cast<uint32_t*>(index_alloc(c, idx, (size_t)nseg * 4));
    launch_seg_bounds(idx->E, nk, 64u - (uint32_t)idx->bits, idx->seg_start, idx->seg_end, s);
    hip_check(hipStreamSynchronize(s), "synchronise");
    idx->bytes = idx->n_ref * 16 + nk * 8 + (uint64_t)nseg * 8;
  } catch (...) {
    index_free(idx);
    throw;
  }
  return idx;
}

// Queries of one or more sets. Sets are packed into tiles of at most
// tile_seqs sequences (a set is never split); each tile runs the query
// pipeline and its sorted result is cut into per-set slices.
void query_sets(sd_ctx* c, const sd_index* idx, int nsets, const sd_seqs* sets, int k,
                const WeightedSpec* w, sd_pairs* outs, hipStream_t s) {
  check_index(c, idx, k);
  if (nsets < 0 || (nsets > 0 && (!sets || !outs))) throw Error{SD_E_INVAL, "bad set arrays"};
  for (int x = 0; x < nsets; ++x) check_seqs(&sets[x]);
  // the captured-graph batch takes unweighted queries on a hashed index
  if (c->batch_graph && !w && !idx->learned && nsets > 0) {
    query_sets_graph(c, idx, nsets, sets, k, outs, s);
    return;
  }
  c->stats = sd_stats{};
  // host-side phases, printed to stderr when SD_DEBUG_BATCH is set
  const bool dbg = std::getenv("SD_DEBUG_BATCH") != nullptr;
  auto t_last = std::chrono::steady_clock::now();
  auto lap = [&](const char* what) {
    if (!dbg) return;
    const auto now = std::chrono::steady_clock::now();
    std::fprintf(stderr, "batch: %-22s %8.3f ms\n", what,
                 std::chrono::duration<double, std::milli>(now - t_last).count());
    t_last = now;
  };
  const uint64_t id_limit = (1ull << idx->idbits) - 2;
  const uint64_t tile_limit =
      std::min<uint64_t>(id_limit, c->batch_tile_seqs ? (uint64_t)c->batch_tile_seqs : (4ull << 20));
  int first = 0;
  while (first < nsets) {
    // the tile: sets [first, last), whole sets while they fit
    uint64_t tot = 0;
    int last = first;
    while (last < nsets) {
      const sd_seqs& st = sets[last];
      if ((uint64_t)st.n > id_limit) throw Error{SD_E_TOO_MANY, "a query set exceeds the index id width"};
      if (last > first && tot + (uint64_t)st.n > tile_limit) break;
      tot += (uint64_t)st.n;
      ++last;
    }
    Scratch sc(c);
    StageTimer tm(c, s);
    Call cl{c, s, sc, tm, fresh_counters(c, CNT_TOTAL, s)};
    // concatenate the tile's sets into one device CSR
    DevSeqs q{nullptr, nullptr, tot};
    std::vector<uint32_t> base(last - first + 1, 0);
    {
      uint64_t qpos = 0;
      for (int x = first; x < last; ++x) {
        base[x - first] = (uint32_t)qpos;
        qpos += (uint64_t)sets[x].n;
      }
      base[last - first] = (uint32_t)qpos;
    }
    std::vector<SetRef> refs;  // the tile's sets, if all are on the device
    bool on_device = true;
    for (int x = first; x < last; ++x)
      if (sets[x].n) {
        on_device = on_device && sets[x].on_device;
        refs.push_back(
            SetRef{sets[x].codes, sets[x].offsets, base[x - first], (uint64_t)sets[x].n});
      }
    if (last - first == 1 && sets[first].on_device) {
      q = DevSeqs{sets[first].codes, sets[first].offsets, (uint64_t)sets[first].n};
    } else if (on_device && !refs.empty()) {
      SetRef* table = sc.get<SetRef>(refs.size());
      SetRef* host = reinterpret_cast<SetRef*>(stage_area(c, refs.size() * sizeof(SetRef)));
      std::copy(refs.begin(), refs.end(), host);
      hip_check(hipMemcpyAsync(table, host, refs.size() * sizeof(SetRef), hipMemcpyHostToDevice, s),
                "copy set table");
      stage_done(c, s);
      q.sets = table;
      q.nsets = (uint32_t)refs.size();
    } else {
      // sets on the host (or on both): their offsets on the host (device sets
      // read into pinned memory with one wait), checked and rebased on host threads into pinned
      // memory, one copy of the tile's offsets; codes one copy per device
      // set and one per run of host sets (through pinned memory)
      size_t dev_words = 0;
      std::vector<SetSpan> spans;
      for (int x = first; x < last; ++x)
        if (sets[x].n) {
          if (sets[x].on_device) dev_words += (size_t)sets[x].n + 1;
          spans.push_back(SetSpan{x, 0, sets[x].n});
        }
      const uint64_t pin_bytes = host_code_bytes(sets, spans);
      int64_t* area = stage_area(c, (dev_words + tot + 1) * 8 + pin_bytes);
      const std::vector<const int64_t*> so = set_offsets(sets, first, last, area, s);
      check_spans(so, spans, false, nullptr, nullptr);
      int64_t* hoffs = area + dev_words;
      const int64_t codes_tot = rebase_spans(so, spans, hoffs);
      uint8_t* codes = sc.get<uint8_t>((uint64_t)codes_tot + 1);
      int64_t* offs = sc.get<int64_t>(tot + 1);
      stage_codes(sets, so, spans, hoffs, codes, reinterpret_cast<uint8_t*>(hoffs + tot + 1), s);
      hip_check(hipMemcpyAsync(offs, hoffs, (tot + 1) * 8, hipMemcpyHostToDevice, s),
                "copy offsets");
      stage_done(c, s);
      q = DevSeqs{codes, offs, tot};
    }
    lap("tile inputs");
    TileOut r = query_tile(cl, idx, q, k, w);
    lap("tile pipeline");
    c->stats.n_seqs += (int64_t)tot;
    c->stats.n_keys += (int64_t)r.nkeys;
    c->stats.n_cand_raw += (int64_t)r.ncand;
    c->stats.n_pairs += (int64_t)r.n;
    const int ns = last - first;
    if (ns == 1) {
      finish_output(c, r.i, r.j, r.d, r.n, &outs[first], s);
    } else {
      // per-set slices of the (q, r)-sorted tile result
      uint32_t* dbase = sc.get<uint32_t>(ns + 1);
      uint64_t* bounds = sc.get<uint64_t>(ns + 1);
      hip_check(hipMemcpyAsync(dbase, base.data(), (ns + 1) * 4, hipMemcpyHostToDevice, s), "copy");
      launch_set_ranges(r.i, r.n, dbase, (uint32_t)(ns + 1), bounds, s);
      std::vector<uint64_t> hb(ns + 1);
      hip_check(hipMemcpyAsync(hb.data(), bounds, (ns + 1) * 8, hipMemcpyDeviceToHost, s), "bounds");
      hip_check(hipStreamSynchronize(s), "synchronise");
      bool host_out = true;
      for (int x = first; x < last; ++x) host_out = host_out && !outs[x].on_device;
      try {
        if (host_out) {
          // host results: the tile's result comes over once and is cut on the
          // host (ids made set-local on the way)
          std::vector<HostSlice> sl;
          for (int x = 0; x < ns; ++x) {
            host_result(c, hb[x + 1] - hb[x], &outs[first + x]);
            sl.push_back(HostSlice{first + x, hb[x], hb[x + 1] - hb[x], 0, -(int64_t)base[x]});
          }
          fill_host_slices(c, r.i, r.j, r.d, r.n, sl, outs, s);
        }
        std::vector<PairSlice> slices;
        for (int x = 0; x < ns && !host_out; ++x) {
          const uint64_t lo = hb[x], n = hb[x + 1] - hb[x];
          uint32_t* oi = dalloc_t<uint32_t>(c, n);
          uint32_t* oj = dalloc_t<uint32_t>(c, n);
          uint8_t* od = dalloc_t<uint8_t>(c, n);
          slices.push_back(
              PairSlice{r.i + lo, r.j + lo, r.d + lo, n, -(int64_t)base[x], oi, oj, od});
        }
        launch_copy_slices(slices.data(), (int)slices.size(), s);
        for (size_t x = 0; x < slices.size(); ++x)
          finish_output(c, slices[x].oi, slices[x].oj, slices[x].od, slices[x].n, &outs[first + x], s);
      } catch (...) {
        dfree(c, r.i);
        dfree(c, r.j);
        dfree(c, r.d);
        throw;
      }
      hip_check(hipStreamSynchronize(s), "synchronise");
      dfree(c, r.i);
      dfree(c, r.j);
      dfree(c, r.d);
    }
    tm.finish();
    lap("tile results");
    first = last;
  }
}

void query_weighted(sd_ctx* c, const sd_index* idx, int nsets, const sd_seqs* sets,
                    const uint8_t* subst, int indel, int max_score, sd_pairs* outs,
                    hipStream_t s) {
  if (!subst) throw Error{SD_E_INVAL, "null substitution table"};
  if (indel < 0 || indel > 255 || max_score < 0) throw Error{SD_E_INVAL, "bad costs"};
  Scratch sc(c);
  uint8_t* dsub = sc.get<uint8_t>(400);
  hip_check(hipMemcpyAsync(dsub, subst, 400, hipMemcpyHostToDevice, s), "copy costs");
  const WeightedSpec w{dsub, (uint32_t)indel, (uint32_t)max_score};
  query_sets(c, idx, nsets, sets, idx ? idx->k : 0, &w, outs, s);
}

}  // namespace sd
