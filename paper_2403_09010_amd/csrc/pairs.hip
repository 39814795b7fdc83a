// Candidate pairs to sorted results for gfx950 (Appendix A, XTNeighbor steps
// 6-7) without sorting the raw candidates:
//
//   producers         put each candidate (i << 32 | j) into a bin by a hash of
//                     the pair (pair_put), so a pair's repeats meet in one bin
//   k_pair_verify     one workgroup per bin: an LDS hash set drops the
//                     repeats, the distinct candidates are verified, and every
//                     kept pair takes a rank among its first id's pairs
//   (scan)            kept pairs per first id -> output offsets
//   k_pair_place      kept pairs to their first id's range of the output
//   k_pair_order      order inside each range by second id, final arrays
//   k_pair_long       the same for the few long ranges
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
constexpr uint32_t PR_LONG = 64;    // ranges with more pairs are ordered by k_pair_long
constexpr uint32_t PR_MAX = 4096;   // longest range it orders in LDS
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
  const uint32_t put = in.cursor[x * in.nbins + bin];
  if (put > in.region && tile == 0 && threadIdx.x == 0) {
    atomicOr(&state->flags, sd::PF_OVERFLOW);
    atomicAdd(&state->raw[sub % sd::PACK_SUMS], (unsigned long long)(put - in.region));
  }
  const uint32_t c = min(put, in.region), t0 = tile * TILE;
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
  partition_tail<NT, TILE, 9, true>(s_e, m, s_cnt, s_tmp, lb, digit, bin << lb, o.base, o.cursor,
                                    o.region, o.nbins, o.nxl, slots, nullptr, 0, nullptr);
}

// One workgroup per bin, its hash set in LDS (TS slots; the bin's regions hold
// at most 7/8 of that). Kept pairs go to the front of the bin's slots of the
// kept arrays, with their rank and distance.
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
  uint32_t total = 0;
  bool over = false;
  for (uint32_t x = 0; x < nx; ++x) {
    const uint32_t c = in.cursor[x * in.nbins + bin];
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
    const uint32_t c = in.cursor[x * in.nbins + bin];
    const uint64_t* __restrict__ p = in.base + base + (uint64_t)x * in.region;
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
        const uint64_t v = e[u];
        // a self search pairs i < j only (a candidate of one sequence with
        // itself can come from two of its variants that share a hash)
        bool fresh = t + lane < c && (!self_pairs || (uint32_t)(v >> 32) < (uint32_t)v);
        uint32_t slot = pair_hash_below(v, in.lb, TSLOG);
        if (fresh) {
          while (true) {  // ends: the set has more slots than the bin candidates
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
        out.kv[base + at] = v;
        out.rank[base + at] = r;
        out.kd[base + at] = (uint8_t)d;
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) out.kept[bin] = s_k;
}

// Kept pairs to off[i] + rank.
__global__ __launch_bounds__(64) void k_pair_place(sd::PairBins in, sd::PairBufs b) {
  const uint32_t n = b.kept[blockIdx.x];
  const uint64_t base = (uint64_t)(blockIdx.x << in.nxl) * in.region;
  for (uint32_t x = threadIdx.x; x < n; x += 64) {
    const uint64_t v = b.kv[base + x];
    const uint64_t p = b.off[v >> 32] + b.rank[base + x];
    b.ti[p] = (uint32_t)(v >> 32);
    b.tj[p] = (uint32_t)v;
    b.td[p] = b.kd[base + x];
  }
}

// Position p's pair goes to the start of its first id's range plus the number
// of smaller second ids there: most ranges hold one to three pairs, neighbours
// in the same cache lines. The last kernel of a search also copies the call's
// counters beside its own, so that one read-back gets both.
__global__ __launch_bounds__(256) void k_pair_order(sd::PairBufs b, uint64_t n,
                                                    uint32_t* __restrict__ oi,
                                                    uint32_t* __restrict__ oj,
                                                    uint8_t* __restrict__ od, uint64_t cap,
                                                    const uint32_t* __restrict__ counters) {
  const uint64_t total = b.off[n];
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) b.state->count = total;
    if (threadIdx.x < sd::PAIR_COUNTERS) b.state->counters[threadIdx.x] = counters[threadIdx.x];
  }
  for (uint64_t p = (uint64_t)blockIdx.x * 256 + threadIdx.x; p < total;
       p += (uint64_t)gridDim.x * 256) {
    const uint32_t i = b.ti[p], j = b.tj[p];
    const uint64_t s = b.off[i], e = b.off[i + 1];
    if (e - s > PR_LONG) continue;
    uint64_t at = s;
    for (uint64_t q = s; q < e; ++q) at += b.tj[q] < j;
    if (at < cap) {
      oi[at] = i;
      oj[at] = j;
      od[at] = b.td[p];
    }
  }
}

// Ranges of PR_LONG + 1 to PR_MAX pairs: a bitonic sort in LDS, one workgroup
// per range in turn.
__global__ __launch_bounds__(256) void k_pair_long(sd::PairBufs b, uint32_t* __restrict__ oi,
                                                   uint32_t* __restrict__ oj,
                                                   uint8_t* __restrict__ od, uint64_t cap) {
  __shared__ uint64_t s_v[PR_MAX];
  const uint32_t nl = min(b.state->nlong, b.long_cap);
  for (uint32_t l = blockIdx.x; l < nl; l += gridDim.x) {
    const uint32_t i = b.longs[l];
    const uint64_t s = b.off[i];
    const uint64_t m64 = b.off[i + 1] - s;
    if (m64 > PR_MAX) continue;  // flagged by k_pair_verify
    const uint32_t m = (uint32_t)m64;
    uint32_t pw = 128;
    while (pw < m) pw <<= 1;
    for (uint32_t x = threadIdx.x; x < pw; x += 256)
      s_v[x] = x < m ? ((uint64_t)b.tj[s + x] << 8) | b.td[s + x] : ~0ull;
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

// A dense candidate array into the bins.
__global__ __launch_bounds__(256) void k_pair_scatter(const uint64_t* __restrict__ cand,
                                                      uint64_t n, sd::PairBins o) {
  for (uint64_t p = (uint64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (uint64_t)gridDim.x * 256)
    pair_put(o, cand[p]);
}

}  // namespace sdk

namespace sd {

uint32_t pair_bin_max(bool large) { return (large ? 8192u : 2048u) / 8 * 7; }

template <int NT, int TSLOG, int MODE>
static void verify_t(const PairBins& in, const PairSeqs& q, const PairBufs& b, hipStream_t s) {
  const size_t lds = ((size_t)8 << TSLOG) + ((size_t)in.region << in.nxl) * 2;
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
  if ((in.region << in.nxl) > pair_bin_max(large))
    throw Error{SD_E_HIP, "internal error: a pair bin exceeds its hash set"};
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

void launch_pair_place(const PairBins& in, const PairBufs& b, hipStream_t s) {
  hipLaunchKernelGGL(sdk::k_pair_place, dim3(in.nbins), dim3(64), 0, s, in, b);
}

void launch_pair_order(const PairBufs& b, uint64_t n, uint32_t* oi, uint32_t* oj, uint8_t* od,
                       uint64_t cap, const uint32_t* counters, hipStream_t s) {
  const unsigned g = (unsigned)std::min<uint64_t>(std::max<uint64_t>((cap + 255) / 256, 1), 4096);
  hipLaunchKernelGGL(sdk::k_pair_long, dim3(std::min(512u, g)), dim3(256), 0, s, b, oi, oj, od,
                     cap);
  hipLaunchKernelGGL(sdk::k_pair_order, dim3(g), dim3(256), 0, s, b, n, oi, oj, od, cap, counters);
}

void launch_pair_scatter(const uint64_t* cand, uint64_t n, const PairBins& o, hipStream_t s) {
  if (!n) return;
  const unsigned g = (unsigned)std::min<uint64_t>((n + 255) / 256, 16384);
  hipLaunchKernelGGL(sdk::k_pair_scatter, dim3(g), dim3(256), 0, s, cand, n, o);
}

}  // namespace sd
