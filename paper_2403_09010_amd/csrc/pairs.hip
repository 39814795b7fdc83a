// Candidate pairs to sorted results for gfx950 (Appendix A, XTNeighbor steps
// 6-7) without sorting the raw candidates:
//
//   producers         put each candidate (i << 32 | j) into a bin by a hash of
//                     the pair (pair_put), so a pair's repeats meet in one bin
//   k_pair_verify     one workgroup per bin: an LDS hash set drops the
//                     repeats, the distinct candidates are verified, and every
//                     kept pair takes a rank among its first id's pairs
//   k_pair_sums,      kept pairs per first id -> output offsets
//   k_pair_scan
//   k_pair_place      kept pairs to their first id's range of the output
//   k_pair_order      order inside each range by second id, final arrays
//
// About nine raw candidates per reported pair (1M sequences, k = 2) leave
// after one write and one read this way, instead of a sort of six passes:
// what is sorted is the reported pairs only, and by counting.
#include <algorithm>

#include "distance.h"
#include "pair_put.h"
#include "partition_tail.h"
#include "sd_device.h"
#include "sd_internal.h"

namespace sdk {

constexpr int PR_ROWS = 8;          // rows of candidates in flight per wave
constexpr uint32_t PR_LONG = 64;    // ranges with more pairs are ordered in LDS
constexpr uint32_t PR_MAX = 4096;   // the longest of them
enum : int { PM_LEV = 0, PM_HAMMING = 1, PM_PAIRED = 2, PM_WEIGHTED = 3, PM_SELF = 4 };

// Candidates from the regions of one level to those of the next, a tile at a
// time. Consecutive workgroups take consecutive regions (the region of XCD x is
// read and split by XCD x, so its next regions get even shares), or, with many
// tiles a region, consecutive tiles of one. What the
// regions of `in` lost is counted here, what those of `o` lose by the next
// kernel.
template <int NT, int TILE>
__global__ __launch_bounds__(NT) void k_pair_split(sd::PairBins in, sd::PairBins o,
                                                   sd::PairState* __restrict__ state,
                                                   uint32_t tiles) {
  constexpr int PER = TILE / NT;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lb = o.lb - in.lb;
  const uint32_t nb = 1u << lb;
  uint64_t* s_e = reinterpret_cast<uint64_t*>(lds);
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_e + TILE);
  uint32_t* s_tmp = s_cnt + nb;
  const uint32_t nsub = in.nbins << in.nxl;
  const uint32_t sub = tiles < 64 ? blockIdx.x % nsub : blockIdx.x / tiles;
  const uint32_t tile = tiles < 64 ? blockIdx.x / nsub : blockIdx.x - sub * tiles;
  const uint32_t bin = sub >> in.nxl, x = in.nxl ? sub & 7u : 0u;
  const unsigned long long put =
      in.lists ? in.lists[x * sd::PAIR_LIST_STRIDE] : in.cursor[(x * in.nbins + bin) << in.pad];
  if (tile == 0 && threadIdx.x == 0) {
    if (in.lists) state->lists[x] = put;
    if (put > in.region) {
      atomicOr(&state->flags, sd::PF_OVERFLOW | (in.lists ? sd::PF_LISTS : sd::PF_MID));
      atomicAdd(&state->raw[sub % sd::PACK_SUMS], put - in.region);
    }
  }
  // (with a full list the attempt is not answered: the candidates that it has are
  // counted, and nothing is split)
  if (in.lists) {
    bool full = false;
    for (uint32_t y = 0; y < nsub; ++y) full |= in.lists[y * sd::PAIR_LIST_STRIDE] > in.region;
    if (full) {
      if (tile == 0 && threadIdx.x == 0)
        atomicAdd(&state->raw[sub % sd::PACK_SUMS], min(put, (unsigned long long)in.region));
      return;
    }
  }
  // (a 64-bit minimum is a vector operation: the tile's bounds would follow it out of
  // the scalar registers)
  const uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane(
      (int)(uint32_t)min(put, (unsigned long long)in.region));
  const uint32_t t0 = tile * TILE;
  if (t0 >= c) return;
  const uint32_t m = min((uint32_t)TILE, c - t0);
  const uint64_t* __restrict__ src = in.base + (uint64_t)((bin << in.nxl) + x) * in.region + t0;
  const int shift = 64 - o.lb;
  const auto digit = [&](uint64_t v) { return (uint32_t)(pair_hash(v) >> shift) & (nb - 1); };
  for (uint32_t i = threadIdx.x; i < nb; i += NT) s_cnt[i] = 0;
  __syncthreads();
  uint64_t e[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = threadIdx.x + r * NT;
    e[r] = i < m ? src[i] : 0;
  }
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = threadIdx.x + r * NT;
    if (i < m) {
      s_e[i] = e[r];
      atomicAdd(&s_cnt[digit(e[r])], 1u);
    }
  }
  __syncthreads();
  const uint32_t slots = (o.nbins << o.nxl) * o.region;
  partition_tail<NT, TILE, 9, true, true>(s_e, m, s_cnt, s_tmp, lb, digit, bin << lb, o.base, o.cursor,
                                    o.region, o.nbins, o.nxl, slots, nullptr, 0, nullptr);
}

// One workgroup per bin, its hash set in LDS (TS slots for at most 7/8 as many
// distinct candidates; with more the bin is over, as with a full region). Kept
// pairs go to the front of the bin's own slots, with their rank and distance in
// arrays of as many.
//
// Bound: LDS latency of the set's inserts and the gathers of two packed
// sequences per distinct candidate.
template <int NT, int TSLOG, int MODE>
__global__ __launch_bounds__(NT) void k_pair_verify(
    sd::PairBins in, const u128* __restrict__ pa, const u128* __restrict__ sb,
    const u128* __restrict__ pa2, uint32_t na, uint32_t nb, int k,
    int self_pairs, const uint8_t* __restrict__ subst, uint32_t indel, uint32_t max_score,
    sd::PairBufs out) {
  constexpr uint32_t TS = 1u << TSLOG;
  extern __shared__ __align__(16) unsigned char lds[];
  unsigned long long* s_tab = reinterpret_cast<unsigned long long*>(lds);
  uint16_t* s_list = reinterpret_cast<uint16_t*>(lds + TS * 8);
  __shared__ uint32_t s_n, s_k;
  __shared__ uint8_t s_sub[MODE == PM_WEIGHTED ? 400 : 1];
  const uint32_t bin = blockIdx.x, nx = 1u << in.nxl, lane = threadIdx.x & 63u;
  constexpr uint32_t MOST = TS / 8 * 7;
  // (each thread inserts at most one candidate past MOST before it sees the count)
  static_assert(MOST - 1 + NT < TS, "the set always has a free slot");
  uint32_t total = 0;
  bool over = false;
  for (uint32_t x = 0; x < nx; ++x) {
    const uint32_t c = in.cursor[(x * in.nbins + bin) << in.pad];
    total += c;
    over |= c > in.region;
  }
  if (threadIdx.x == 0) {
    if (total) atomicAdd(&out.state->raw[bin % sd::PACK_SUMS], (unsigned long long)total);
    if (over) atomicOr(&out.state->flags, sd::PF_OVERFLOW);
    s_n = 0;
    s_k = 0;
    if (total == 0 || over) out.kept[bin] = 0;
  }
  if (total == 0 || over) return;  // (an overflow runs the producer again with more room)
  for (uint32_t i = threadIdx.x; i < TS; i += NT) s_tab[i] = 0;
  if (MODE == PM_WEIGHTED)
    for (uint32_t i = threadIdx.x; i < 400; i += NT) s_sub[i] = subst[i];
  __syncthreads();
  const uint64_t base = (uint64_t)(bin << in.nxl) * in.region;
  // waves share out the regions; each has PR_ROWS rows of 64 in flight
  constexpr uint32_t NW = NT / 64;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t parts = NW > nx ? NW / nx : 1u;
  for (uint32_t x = w & (nx - 1); x < nx; x += NW) {
    const uint32_t c = in.cursor[(x * in.nbins + bin) << in.pad];
    const uint64_t* p = in.base + base + (uint64_t)x * in.region;
    for (uint32_t t0 = (w >> in.nxl) * 64; t0 < c; t0 += parts * 64 * PR_ROWS) {
      uint64_t e[PR_ROWS];
#pragma unroll
      for (int u = 0; u < PR_ROWS; ++u) {
        const uint32_t t = t0 + u * parts * 64 + lane;
        e[u] = t < c ? p[t] : 0;
      }
#pragma unroll
      for (int u = 0; u < PR_ROWS; ++u) {
        const uint32_t t = t0 + u * parts * 64;
        if (t >= c) break;
        if (*(volatile uint32_t*)&s_n >= MOST) break;
        const uint64_t v = e[u];
        // a self search pairs i < j only (a candidate of one sequence with
        // itself can come from two of its variants that share a hash)
        bool fresh = t + lane < c && (!self_pairs || (uint32_t)(v >> 32) < (uint32_t)v);
        uint32_t slot = pair_hash_below(v, in.lb, TSLOG);
        if (fresh) {
          while (true) {  // ends: the set has a free slot
            const unsigned long long old = atomicCAS(&s_tab[slot], 0ull, (unsigned long long)v + 1);
            if (old == 0) break;
            if (old == v + 1) {
              fresh = false;
              break;
            }
            slot = (slot + 1) & (TS - 1);
          }
        }
        const uint64_t bal = __ballot(fresh);
        if (bal) {
          uint32_t at = 0;
          if (lane == 0) at = atomicAdd(&s_n, (uint32_t)__popcll(bal));
          at = __builtin_amdgcn_readfirstlane(at);
          if (fresh) s_list[at + mask_rank(bal)] = (uint16_t)slot;
        }
      }
    }
  }
  __syncthreads();
  const uint32_t n = s_n;
  if (n >= MOST) {
    if (threadIdx.x == 0) {
      atomicOr(&out.state->flags, sd::PF_OVERFLOW);
      out.kept[bin] = 0;
    }
    return;
  }
  for (uint32_t l0 = 0; l0 < n; l0 += NT) {
    const uint32_t l = l0 + threadIdx.x;
    bool keep = false;
    uint64_t v = 0;
    uint32_t d = 0;
    if (l < n) {
      v = s_tab[s_list[l]] - 1;
      const uint32_t i = (uint32_t)(v >> 32), j = (uint32_t)v;
      if (i < na && j < nb) {
        if (MODE == PM_WEIGHTED) {
          // pa: bit planes, pa2: packed keys of the first sequences
          if (pair_verdict<0>(pa, sb, nullptr, nullptr, i, j, k) != DROP) {
            d = weighted_keys(pa2[i], sb[j], s_sub, indel);
            keep = d <= max_score;
            d = d > 255u ? 255u : d;
          }
        } else if (MODE == PM_SELF || MODE == PM_PAIRED) {
          d = planes_verdict<MODE == PM_PAIRED>(pa, pa2, i, j, k);
          keep = d != DROP;
        } else {
          d = pair_verdict<MODE>(pa, sb, nullptr, nullptr, i, j, k);
          keep = d != DROP;
        }
      } else {  // an id out of range is an internal error: flagged, never read
        atomicOr(out.err, SD_ERRBIT_INDEX);
      }
    }
    const uint64_t bal = __ballot(keep);
    if (bal) {
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(&s_k, (uint32_t)__popcll(bal));
      at = __builtin_amdgcn_readfirstlane(at) + mask_rank(bal);
      if (keep) {
        const uint32_t i = (uint32_t)(v >> 32);
        const uint32_t r = atomicAdd(&out.icnt[i], 1u);
        if (r == PR_LONG) {
          const uint32_t q = atomicAdd(&out.state->nlong, 1u);
          if (q < out.long_cap) out.longs[q] = i;
        }
        if (r == PR_MAX) atomicOr(&out.state->flags, sd::PF_LONG);
        in.base[base + at] = v;
        out.rank[base + at] = r;
        out.kd[base + at] = (uint8_t)d;
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) out.kept[bin] = s_k;
}

// Exclusive scan of the pairs kept per first id (fewer than 2^32 in all), in two
// launches: the sums of tiles and groups of tiles, then each tile's own part, with
// the sums before it. One launch with a look-back from tile to tile took longer: 19 us for
// 1M ids and 100 for 10M, where these take 10 and 37.
constexpr int PS_NT = 256, PS_ROWS = 4, PS_TILE = PS_NT * 4 * PS_ROWS;

// lane's four counts of each row of its wave (the wave has PS_ROWS rows of 256 ids)
__device__ __forceinline__ void tile_counts(const uint32_t* __restrict__ icnt, uint64_t n,
                                            uint64_t first, uint4 (&c)[PS_ROWS]) {
#pragma unroll
  for (int r = 0; r < PS_ROWS; ++r) {
    const uint64_t i = first + r * 256;
    if (i + 4 <= n) {
      c[r] = *reinterpret_cast<const uint4*>(icnt + i);
    } else {
      c[r].x = i < n ? icnt[i] : 0u;
      c[r].y = i + 1 < n ? icnt[i + 1] : 0u;
      c[r].z = i + 2 < n ? icnt[i + 2] : 0u;
      c[r].w = 0u;
    }
  }
}

__device__ __forceinline__ uint64_t tile_first() {
  return (uint64_t)blockIdx.x * PS_TILE + (threadIdx.x >> 6) * (256 * PS_ROWS) +
         (threadIdx.x & 63u) * 4;
}

__global__ __launch_bounds__(PS_NT) void k_pair_sums(sd::PairBufs b, uint64_t n) {
  __shared__ uint32_t s_tmp[PS_NT / 64];
  uint4 c[PS_ROWS];
  tile_counts(b.icnt, n, tile_first(), c);
  uint32_t sum = 0, total;
#pragma unroll
  for (int r = 0; r < PS_ROWS; ++r) sum += c[r].x + c[r].y + c[r].z + c[r].w;
  block_excl_scan<PS_NT>(sum, s_tmp, &total);
  if (threadIdx.x == 0) {
    b.sums[blockIdx.x] = total;
    if (total) atomicAdd(&b.groups[blockIdx.x / sd::PAIR_GROUP], total);
  }
}

__global__ __launch_bounds__(PS_NT) void k_pair_scan(sd::PairBufs b, uint64_t n) {
  __shared__ uint32_t s_tmp[PS_NT / 64], s_wave[PS_NT / 64];
  const uint64_t first = tile_first();
  uint4 c[PS_ROWS];
  tile_counts(b.icnt, n, first, c);
  uint32_t sum = 0, before;
  const uint32_t g = blockIdx.x / sd::PAIR_GROUP;
  for (uint32_t x = threadIdx.x; x < g; x += PS_NT) sum += b.groups[x];
  for (uint32_t x = g * sd::PAIR_GROUP + threadIdx.x; x < blockIdx.x; x += PS_NT) sum += b.sums[x];
  block_excl_scan<PS_NT>(sum, s_tmp, &before);
  // the rows of a wave one after the other, the waves likewise
  uint32_t ex[PS_ROWS], run = 0;
#pragma unroll
  for (int r = 0; r < PS_ROWS; ++r) {
    const uint32_t v = c[r].x + c[r].y + c[r].z + c[r].w, incl = wave_incl_scan(v);
    ex[r] = run + incl - v;
    run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  }
  if ((threadIdx.x & 63u) == 0) s_wave[threadIdx.x >> 6] = run;
  __syncthreads();
  for (uint32_t w = 0; w < threadIdx.x >> 6; ++w) before += s_wave[w];
#pragma unroll
  for (int r = 0; r < PS_ROWS; ++r) {
    const uint64_t i = first + r * 256;
    uint4 o;
    o.x = before + ex[r];
    o.y = o.x + c[r].x;
    o.z = o.y + c[r].y;
    o.w = o.z + c[r].z;
    if (i + 4 <= n) {
      *reinterpret_cast<uint4*>(b.off + i) = o;
      if (i + 4 == n) b.off[n] = o.w + c[r].w;
    } else if (i < n) {
      const uint32_t v[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (i + x <= n) b.off[i + x] = v[x];
    }
  }
}

// Kept pairs to off[i] + rank. Bound: the random writes, a word and a byte per
// pair (8.6M pairs of 10M sequences: 0.47 ms; with the two ids in words of
// their own 0.66).
__global__ __launch_bounds__(64) void k_pair_place(sd::PairBins in, sd::PairBufs b) {
  const uint32_t n = b.kept[blockIdx.x];
  const uint64_t base = (uint64_t)(blockIdx.x << in.nxl) * in.region;
  for (uint32_t x = threadIdx.x; x < n; x += 64) {
    const uint64_t v = in.base[base + x];
    const uint32_t p = b.off[v >> 32] + b.rank[base + x];
    b.t[p] = v;
    b.td[p] = b.kd[base + x];
  }
}

// Ranges of PR_LONG + 1 to PR_MAX pairs: a bitonic sort in LDS, one workgroup
// per range in turn.
__device__ __forceinline__ void order_long(const sd::PairBufs& b, uint64_t* s_v,
                                           uint32_t* __restrict__ oi, uint32_t* __restrict__ oj,
                                           uint8_t* __restrict__ od, uint64_t cap) {
  const uint32_t nl = min(b.state->nlong, b.long_cap);
  for (uint32_t l = blockIdx.x; l < nl; l += gridDim.x) {
    const uint32_t i = b.longs[l], s = b.off[i], m = b.off[i + 1] - s;
    if (m > PR_MAX) continue;  // flagged by k_pair_verify
    uint32_t pw = 128;
    while (pw < m) pw <<= 1;
    for (uint32_t x = threadIdx.x; x < pw; x += 256)
      s_v[x] = x < m ? (b.t[s + x] << 8 & 0xFFFFFFFF00ull) | b.td[s + x] : ~0ull;
    __syncthreads();
    for (uint32_t a = 2; a <= pw; a <<= 1)
      for (uint32_t h = a >> 1; h > 0; h >>= 1) {
        for (uint32_t x = threadIdx.x; x < pw / 2; x += 256) {
          const uint32_t lo = 2 * x - (x & (h - 1)), hi = lo + h;
          const uint64_t u = s_v[lo], w = s_v[hi];
          if ((u > w) == ((lo & a) == 0)) {
            s_v[lo] = w;
            s_v[hi] = u;
          }
        }
        __syncthreads();
      }
    for (uint32_t x = threadIdx.x; x < m; x += 256)
      if (s + x < cap) {
        oi[s + x] = i;
        oj[s + x] = (uint32_t)(s_v[x] >> 8);
        od[s + x] = (uint8_t)s_v[x];
      }
    __syncthreads();
  }
}

// Position p's pair goes to the start of its first id's range plus the number
// of smaller second ids there: most ranges hold one to three pairs, neighbours
// in the same cache lines. The first workgroups order the few long ranges
// before, while the others are at work (10M sequences: 0.28 ms, where they took 0.23
// in a kernel of their own and the rest 0.14). The last kernel of a search also copies
// the call's counters beside its own, so that one read-back gets both.
__global__ __launch_bounds__(256) void k_pair_order(sd::PairBufs b, uint64_t n,
                                                    uint32_t* __restrict__ oi,
                                                    uint32_t* __restrict__ oj,
                                                    uint8_t* __restrict__ od, uint64_t cap,
                                                    const uint32_t* __restrict__ counters) {
  __shared__ uint64_t s_v[PR_MAX];
  const uint64_t total = b.off[n];
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      b.state->count = total;
      b.state->missed = *b.missed;
    }
    if (threadIdx.x < sd::PAIR_COUNTERS) b.state->counters[threadIdx.x] = counters[threadIdx.x];
  }
  // (nothing to order: the attempt is not answered, or the placed pairs are sorted)
  if (b.state->flags & (sd::PF_OVERFLOW | sd::PF_LONG)) return;
  order_long(b, s_v, oi, oj, od, cap);
  for (uint64_t p = (uint64_t)blockIdx.x * 256 + threadIdx.x; p < total;
       p += (uint64_t)gridDim.x * 256) {
    const uint64_t v = b.t[p];
    const uint32_t i = (uint32_t)(v >> 32), j = (uint32_t)v;
    const uint32_t s = b.off[i], e = b.off[i + 1];
    if (e - s > PR_LONG) continue;
    uint64_t at = s;
    for (uint32_t q = s; q < e; ++q) at += (uint32_t)b.t[q] < j;
    if (at < cap) {
      oi[at] = i;
      oj[at] = j;
      od[at] = b.td[p];
    }
  }
}

// A dense candidate array into the bins, or, PC_CHUNK at a time, to the lists in turn
// (612M candidates of 3,000 equal sequences: 108 ms with a reservation for each
// wave's 64, 1.9 with one for each chunk).
constexpr uint32_t PC_CHUNK = 8192;

__global__ __launch_bounds__(256) void k_pair_scatter(const uint64_t* __restrict__ cand,
                                                      uint64_t n, sd::PairBins o) {
  __shared__ unsigned long long s_at;
  if (o.lb > 0) {
    for (uint64_t p = (uint64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (uint64_t)gridDim.x * 256)
      pair_put(o, cand[p]);
    return;
  }
  for (uint64_t c = blockIdx.x; c * PC_CHUNK < n; c += gridDim.x) {
    const uint32_t x = (uint32_t)c & ((1u << o.nxl) - 1);
    const uint64_t* __restrict__ src = cand + c * PC_CHUNK;
    const uint32_t m = (uint32_t)min((uint64_t)PC_CHUNK, n - c * PC_CHUNK);
    if (threadIdx.x == 0) s_at = list_reserve(o, x, m);
    __syncthreads();
    const unsigned long long at = s_at;
    const uint32_t room = sd::list_room(at, m, o.region);
    uint64_t* __restrict__ dst = o.base + (uint64_t)x * o.region + at;
    for (uint32_t i = threadIdx.x; i < room; i += 256) dst[i] = src[i];
    __syncthreads();  // the next chunk's place
  }
}

}  // namespace sdk

namespace sd {

uint32_t pair_set_max(bool large) { return (large ? 8192u : 2048u) / 8 * 7; }

template <int NT, int TSLOG, int MODE>
static void verify_t(const PairBins& in, const PairSeqs& q, const PairBufs& b, hipStream_t s) {
  const size_t lds = ((size_t)8 << TSLOG) + ((7u << TSLOG) / 8 + NT) * 2;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&sdk::k_pair_verify<NT, TSLOG, MODE>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    (void)hipGetLastError();  // the launch reports any real problem
  hipLaunchKernelGGL((sdk::k_pair_verify<NT, TSLOG, MODE>), dim3(in.nbins), dim3(NT), lds, s, in,
                     q.a, q.b, q.a2, (uint32_t)q.na, (uint32_t)q.nb, q.k, q.self_pairs,
                     q.subst, q.indel, q.max_score, b);
}

template <int NT, int TSLOG>
static void verify_mode(const PairBins& in, const PairSeqs& q, const PairBufs& b, hipStream_t s) {
  switch (q.mode) {
    case sdk::PM_LEV: verify_t<NT, TSLOG, sdk::PM_LEV>(in, q, b, s); break;
    case sdk::PM_HAMMING: verify_t<NT, TSLOG, sdk::PM_HAMMING>(in, q, b, s); break;
    case sdk::PM_PAIRED: verify_t<NT, TSLOG, sdk::PM_PAIRED>(in, q, b, s); break;
    case sdk::PM_SELF: verify_t<NT, TSLOG, sdk::PM_SELF>(in, q, b, s); break;
    default: verify_t<NT, TSLOG, sdk::PM_WEIGHTED>(in, q, b, s); break;
  }
}

void launch_pair_verify(const PairBins& in, bool large, const PairSeqs& q, const PairBufs& b,
                        hipStream_t s) {
  if (large)
    verify_mode<512, 13>(in, q, b, s);
  else
    verify_mode<256, 11>(in, q, b, s);
}

void launch_pair_split(const PairBins& in, const PairBins& o, PairState* state, hipStream_t s) {
  constexpr int NT = 512, TILE = 8192;
  if (o.lb - in.lb > 9 || ((uint64_t)(o.nbins << o.nxl)) * o.region >= 0xFFFFFFFFull)
    throw Error{SD_E_HIP, "internal error: a pair split out of range"};
  const size_t lds = (size_t)TILE * 8 + ((size_t)4 << (o.lb - in.lb)) + NT / 64 * 4;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&sdk::k_pair_split<NT, TILE>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    (void)hipGetLastError();  // the launch reports any real problem
  const uint32_t tiles = (in.region + TILE - 1) / TILE;
  hipLaunchKernelGGL((sdk::k_pair_split<NT, TILE>), dim3(tiles * (in.nbins << in.nxl)), dim3(NT),
                     lds, s, in, o, state, tiles);
}

uint64_t pair_tiles(uint64_t na) { return (na + sdk::PS_TILE - 1) / sdk::PS_TILE; }

void launch_pair_scan(const PairBufs& b, uint64_t na, hipStream_t s) {
  const dim3 g((unsigned)pair_tiles(na));
  hipLaunchKernelGGL(sdk::k_pair_sums, g, dim3(sdk::PS_NT), 0, s, b, na);
  hipLaunchKernelGGL(sdk::k_pair_scan, g, dim3(sdk::PS_NT), 0, s, b, na);
}

void launch_pair_place(const PairBins& in, const PairBufs& b, hipStream_t s) {
  hipLaunchKernelGGL(sdk::k_pair_place, dim3(in.nbins), dim3(64), 0, s, in, b);
}

void launch_pair_order(const PairBufs& b, uint64_t n, uint32_t* oi, uint32_t* oj, uint8_t* od,
                       uint64_t cap, const uint32_t* counters, hipStream_t s) {
  const unsigned g = (unsigned)std::min<uint64_t>(std::max<uint64_t>((cap + 255) / 256, 1), 4096);
  hipLaunchKernelGGL(sdk::k_pair_order, dim3(g), dim3(256), 0, s, b, n, oi, oj, od, cap, counters);
}

void launch_pair_scatter(const uint64_t* cand, uint64_t n, const PairBins& o, hipStream_t s) {
  if (!n) return;
  const uint64_t per = o.lb > 0 ? 256 : sdk::PC_CHUNK;
  const unsigned g = (unsigned)std::min<uint64_t>((n + per - 1) / per, 16384);
  hipLaunchKernelGGL(sdk::k_pair_scatter, dim3(g), dim3(256), 0, s, cand, n, o);
}

}  // namespace sd
