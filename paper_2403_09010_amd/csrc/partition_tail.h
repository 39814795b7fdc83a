// The common end of the partitioning kernels: an LDS tile to the regions of
// its bins.
#pragma once
#include "sd_device.h"

namespace sdk {

// m elements sit in s_e[0, m), the counts of their bins digit(e) in
// s_cnt[0, 2^lb). Reserves each bin's run in its region (one 64-bit atomic per
// two bins), puts the tile in bin order and writes it out. Bin b of the tile is
// bin bin0 + b of the output, whose region for this workgroup's XCD (nxl = 3:
// workgroups go to the XCDs in turn) starts at elem[((bin << nxl) + XCD) *
// region]. With DROP, a run's elements past its region are lost (the cursor
// counts them). Otherwise a run that does not fit goes to the overflow area
// from `slots` on as a whole (nothing is written from cap on); the bin's
// cursor then exceeds the region, and `fill` holds the elements the region
// received (written by the run that reached or crossed its end; no later run
// fits).
//
// Bound: the element writes. Each bin's runs land next to each other only if
// the same XCD wrote them, so with one region per XCD its L2 completes the
// cache lines at its own frontiers. Ordering the tile in LDS first beats
// scattering it from registers (100M random elements into 2^10 and 2^11 bins:
// 0.39 and 0.42 ms against 0.57 and 0.60). With TOGETHER all of a thread's
// elements are looked up before the first is written: 1G elements split in 3.34
// ms instead of 3.52; a generator, whose other workgroups use the waits, gets
// slower (4.66 instead of 4.36 ms).
template <int NT, int TILE, int MAXLB, bool DROP, bool TOGETHER = false, class Digit>
__device__ __forceinline__ void partition_tail(uint64_t* s_e, uint32_t m, uint32_t* s_cnt,
                                               uint32_t* s_tmp, int lb, const Digit& digit,
                                               uint32_t bin0, uint64_t* __restrict__ elem,
                                               uint32_t* __restrict__ cursor, uint32_t region,
                                               uint32_t nbins, int nxl, uint32_t slots,
                                               uint32_t* __restrict__ fill, uint32_t cap,
                                               uint32_t* __restrict__ over_count) {
  constexpr int PER = (TILE + NT - 1) / NT;
  // bins per thread: an even number, since two bins share a reservation
  constexpr int MAXQ = NT * 2 >= (1 << MAXLB) ? 2 : (1 << MAXLB) / NT;
  const uint32_t nb = 1u << lb;
  const uint32_t x = nxl ? blockIdx.x & 7u : 0u;
  const uint32_t per = max(2u, nb / NT), b0 = threadIdx.x * per;
  uint32_t c[MAXQ], g[MAXQ], sum = 0;
#pragma unroll
  for (int q = 0; q < MAXQ; ++q) {
    c[q] = (uint32_t)q < per && b0 + q < nb ? s_cnt[b0 + q] : 0u;
    sum += c[q];
  }
  // the reservations are in flight while the tile is put in order
  const uint32_t cu0 = x * nbins + bin0 + b0;
#pragma unroll
  for (int q = 0; q < MAXQ; q += 2)
    if (c[q] + c[q + 1]) {
      const unsigned long long old =
          atomicAdd(reinterpret_cast<unsigned long long*>(cursor + cu0 + q),
                    (unsigned long long)c[q + 1] << 32 | c[q]);
      g[q] = (uint32_t)old;
      g[q + 1] = (uint32_t)(old >> 32);
    }
  uint32_t total;
  const uint32_t ex0 = block_excl_scan<NT>(sum, s_tmp, &total);
  {
    uint32_t ex = ex0;
#pragma unroll
    for (int q = 0; q < MAXQ; ++q) {
      if (c[q]) s_cnt[b0 + q] = ex;
      ex += c[q];
    }
  }
  uint64_t e[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t t = threadIdx.x + r * NT;
    e[r] = t < m ? s_e[t] : 0;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < PER; ++r)
    if (threadIdx.x + r * NT < m) s_e[atomicAdd(&s_cnt[digit(e[r])], 1u)] = e[r];
  __syncthreads();
  // the counters become the output position of each bin's slot 0
  uint32_t ex = ex0;
#pragma unroll
  for (int q = 0; q < MAXQ; ++q) {
    if (c[q]) {
      const uint32_t base = (((bin0 + b0 + q) << nxl) + x) * region;
      uint32_t at = base + g[q];
      if (DROP) {
        // one slot before the region marks a run with no room
        if (g[q] >= region || c[q] > region - g[q]) at = 0xFFFFFFFFu;
        s_cnt[b0 + q] = at == 0xFFFFFFFFu ? at : at - ex;
      } else {
        if (g[q] < region && c[q] >= region - g[q])  // the one run that reaches the end
          fill[cu0 + q] = c[q] == region - g[q] ? region : g[q];
        if (g[q] >= region || c[q] > region - g[q]) at = slots + atomicAdd(over_count, c[q]);
        s_cnt[b0 + q] = at - ex;
      }
    }
    ex += c[q];
  }
  __syncthreads();
  const auto write = [&](uint64_t v, uint32_t to, uint32_t t) {
    const uint32_t p = to + t;
    if (DROP ? (to != 0xFFFFFFFFu && p < slots) : p < cap) elem[p] = v;
  };
  if (TOGETHER) {
    uint32_t to[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const uint32_t t = threadIdx.x + r * NT;
      e[r] = t < m ? s_e[t] : 0;
    }
#pragma unroll
    for (int r = 0; r < PER; ++r) to[r] = s_cnt[digit(e[r])];
#pragma unroll
    for (int r = 0; r < PER; ++r)
      if (threadIdx.x + r * NT < m) write(e[r], to[r], threadIdx.x + r * NT);
  } else {
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const uint32_t t = threadIdx.x + r * NT;
      if (t < m) {
        const uint64_t v = s_e[t];
        write(v, s_cnt[digit(v)], t);
      }
    }
  }
}

}  // namespace sdk
