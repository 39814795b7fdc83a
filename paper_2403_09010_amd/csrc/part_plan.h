// How a partition of variants into hash bins is laid out (partition.hip): the
// number of bins and levels for an input, the regions' sizes, and the hash bits
// below the bins'. Host arithmetic only.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace sd {

// Inputs of at least this many variants are generated and grouped by the
// large workgroups (1,024 threads, one or two on a CU).
constexpr uint64_t PART_BIG_KEYS = 16ull << 20;
// most bins (log2) one kernel partitions into
constexpr int PART_MAX_LB = 12;
// most bits of one split of a first partition's bins
constexpr int PART_MAX_SPLIT = 9;
// a safe mean for the bins of launch_sort_bins
constexpr uint32_t SORT_BIN_MEAN = 3200;

// most bins (log2) that a workgroup's threads reserve runs of
constexpr int tile_max_lb(int threads) { return threads >= 1024 ? PART_MAX_LB : 11; }

struct PartPlan {
  int lb;   // 2^lb bins at the end, ...
  int lb1;  // ... 2^lb1 of the first level (lb: one level)
  int nxl;  // 2^nxl regions per bin
};

// The bins of a search over nk variants (at least 1). Small inputs take 2^8 bins of
// 512 elements or more, so that every CU has one, and more bins only to keep
// them under 10K elements (what the small bitmap filters well). Large inputs
// take bins of 26K to 51K elements: with fewer a tile's runs get short (100M
// elements of 1M sequences: 0.52 ms into 2^11 bins, 0.60 into 2^12), with more
// the filter lets too many through. Beyond 2^12 bins of that size the partition
// takes a second level, into bins a quarter as large since more bins cost
// little there (and their second read comes from the L2): scattering 100M
// elements into 2^13 bins at once takes 0.92 ms, two levels of 2^8 and 2^5 0.43
// + 0.33; 1G elements group in 6.9 ms in bins of 31K elements and in 2.6 in
// bins of 15K. The first level has 2^8 bins, or as many as the split leaves it.
inline PartPlan search_plan(uint64_t nk) {
  int lb = 1;
  if (nk < PART_BIG_KEYS) {
    while (lb < 11 && ((nk >> lb) > 10240 || (lb < 8 && (nk >> lb) > 512))) ++lb;
  } else {
    lb = 11;
    while ((nk >> lb) > 51200) ++lb;
    if (lb > PART_MAX_LB) lb += 2;
  }
  return {lb, lb > PART_MAX_LB ? std::max(8, lb - PART_MAX_SPLIT) : lb, nk >= (2u << 20) ? 3 : 0};
}

// The bins that are sorted for an index of nk variants: at most SORT_BIN_MEAN
// elements each; small inputs take 2^8 bins of 512 or more, so that every CU has
// one. Beyond 2^11 bins the partition takes two levels.
inline PartPlan sort_plan(uint64_t nk) {
  int lb = 1;
  while ((nk >> lb) > SORT_BIN_MEAN || (lb < 8 && (nk >> lb) > 512)) ++lb;
  return {lb, lb > 11 ? std::max(8, lb - PART_MAX_SPLIT) : lb, nk >= (2u << 20) ? 3 : 0};
}

// Slots of a region: an eighth more than its mean share (small inputs: twice it)
// and six standard deviations of it.
inline uint64_t part_region(uint64_t nk, int lb, int nxl) {
  const double mean = (double)nk / (double)(1ull << (lb + nxl));
  return ((uint64_t)(mean * (nxl ? 1.125 : 2.0) + 6.0 * std::sqrt(mean)) + 64 + 15) / 16 * 16;
}

// Whether 2^lb bins for nk elements and over_cap slots behind them have positions
// of 32 bits.
inline bool part_fits(uint64_t nk, int lb, int nxl, uint64_t over_cap) {
  return (part_region(nk, lb, nxl) << (lb + nxl)) + over_cap < (1ull << 32);
}

// Whether the kernels take a plan for nk variants.
inline bool plan_fits(const PartPlan& p, uint64_t nk, uint64_t over_cap) {
  const int most = nk < PART_BIG_KEYS ? tile_max_lb(256) : tile_max_lb(1024);
  return p.lb >= p.lb1 && p.lb - p.lb1 <= PART_MAX_SPLIT && p.lb1 >= 1 && p.lb1 <= most &&
         part_fits(nk, p.lb1, p.nxl, over_cap) && part_fits(nk, p.lb, p.nxl, over_cap);
}

// The shift that brings an element's `bits` bits below the top `top` ones down,
// not into the id: equal hashes have equal bits there, whatever their ids.
constexpr int hash_shift(int top, int bits, int idbits) {
  return 64 - top - bits > idbits ? 64 - top - bits : idbits;
}

}  // namespace sd
