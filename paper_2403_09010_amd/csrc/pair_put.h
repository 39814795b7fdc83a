// Candidate pairs into bins by a hash of the pair (the input of pairs.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sd_device.h"
#include "sd_internal.h"

namespace sdk {

// (both halves mixed twice: the ids of a cluster are often consecutive, and one
// multiplication would leave their pairs on a lattice)
__device__ __forceinline__ uint64_t pair_hash(uint64_t v) {
  v = (v ^ (v >> 32)) * 0x9E3779B97F4A7C15ull;
  v = (v ^ (v >> 29)) * 0xBF58476D1CE4E5B9ull;
  return v ^ (v >> 32);
}

// `bits` hash bits below the lb bits that name the bin
__device__ __forceinline__ uint32_t pair_hash_below(uint64_t v, int lb, int bits) {
  return (uint32_t)(pair_hash(v) >> (64 - lb - bits)) & ((1u << bits) - 1);
}

// The place of n candidates in list x (taken by one lane).
__device__ __forceinline__ unsigned long long list_reserve(const sd::PairBins& o, uint32_t x,
                                                           uint32_t n) {
  return atomicAdd(&o.lists[x * sd::PAIR_LIST_STRIDE], (unsigned long long)n);
}

// The first active lane's value.
__device__ __forceinline__ unsigned long long first_lane(unsigned long long v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (unsigned long long)hi << 32 | lo;
}

// Adds a candidate to its bin (or, with lb = 0, to its XCD's list, one
// reservation for the active lanes); one that finds its region full is only
// counted.
// Each bin has a region per XCD (nxl = 3), so that an XCD's L2 completes the
// lines of its own regions. With ALIKE, lanes with the first active lane's pair
// reserve together: the variants of two equal sequences all give one pair, and an
// atomic takes its line 10 ns whichever lane it comes from.
template <bool ALIKE = false>
__device__ __forceinline__ void pair_put(const sd::PairBins& o, uint64_t v) {
  const uint32_t x = o.nxl ? blockIdx.x & 7u : 0u;
  if (o.lb == 0) {
    const uint64_t act = __ballot(true);
    const uint32_t n = (uint32_t)__popcll(act), rank = mask_rank(act);
    unsigned long long at = 0;
    if (rank == 0) at = list_reserve(o, x, n);
    at = first_lane(at);
    if (rank < sd::list_room(at, n, o.region)) o.base[(uint64_t)x * o.region + at + rank] = v;
    return;
  }
  const uint32_t b = (uint32_t)(pair_hash(v) >> (64 - o.lb));
  uint32_t* const cursor = &o.cursor[(x * o.nbins + b) << o.pad];
  uint32_t slot = 0;
  if (ALIKE) {
    const bool same = v == first_lane(v);
    const uint64_t peers = __ballot(same);
    const uint32_t rank = mask_rank(peers);
    if (!same || rank == 0) slot = atomicAdd(cursor, same ? (uint32_t)__popcll(peers) : 1u);
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot);
    if (same) slot = first + rank;
  } else {
    slot = atomicAdd(cursor, 1u);
  }
  if (slot < o.region) o.base[(uint64_t)((b << o.nxl) + x) * o.region + slot] = v;
}

// The lane's candidates v[u] with on[u], their reservations in flight together.
template <int N>
__device__ __forceinline__ void pair_put_rows(const sd::PairBins& o, const uint64_t (&v)[N],
                                              const bool (&on)[N]) {
  if (o.lb == 0) {
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (on[u]) pair_put(o, v[u]);
    return;
  }
  const uint32_t x = o.nxl ? blockIdx.x & 7u : 0u;
  uint32_t b[N], slot[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    b[u] = (uint32_t)(pair_hash(v[u]) >> (64 - o.lb));
    slot[u] = o.region;
    if (on[u]) slot[u] = atomicAdd(&o.cursor[(x * o.nbins + b[u]) << o.pad], 1u);
  }
#pragma unroll
  for (int u = 0; u < N; ++u)
    if (slot[u] < o.region) o.base[(uint64_t)((b[u] << o.nxl) + x) * o.region + slot[u]] = v[u];
}

}  // namespace sdk
