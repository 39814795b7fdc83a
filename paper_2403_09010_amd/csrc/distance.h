// Distances of packed sequences on the device: the final filters of the
// verification kernels.
#pragma once
#include "sd_device.h"

namespace sdk {

// ------------------------------------------------------------------ Levenshtein
//
// Bit-parallel edit distance (Myers 1999, in the global-distance form of
// Hyyro 2001): the pattern a (m <= 24 residues) lives in one 32-bit word, the
// text b is consumed one residue per step, and the score tracks the last row
// of the dynamic programme. Bits above m-1 carry junk that never reaches the
// low m bits (only shifts left and carries move bits, and they move upward).
__device__ __forceinline__ uint32_t lev_keys(u128 a, u128 b) {
  const uint32_t m = key_len(a), n = key_len(b);
  if (m == 0) return n;
  if (n == 0) return m;
  uint32_t ares[KEY_MAX_LEN];
#pragma unroll
  for (int t = 0; t < KEY_MAX_LEN; ++t) ares[t] = (uint32_t)t < m ? key_residue(a, t) : 31u;
  uint32_t pv = (1u << m) - 1u, mv = 0u, score = m;
  const uint32_t top = 1u << (m - 1);
  u128 text = b;
  for (uint32_t j = 0; j < n; ++j) {
    const uint32_t c = (uint32_t)(text >> 115) & 31u;
    text <<= 5;
    uint32_t eq = 0;
#pragma unroll
    for (int t = 0; t < KEY_MAX_LEN; ++t) eq |= (ares[t] == c ? 1u : 0u) << t;
    const uint32_t xv = eq | mv;
    const uint32_t xh = (((eq & pv) + pv) ^ pv) | eq;
    uint32_t ph = mv | ~(xh | pv);
    uint32_t mh = pv & xh;
    if (ph & top)
      ++score;
    else if (mh & top)
      --score;
    ph = (ph << 1) | 1u;
    mh = mh << 1;
    pv = mh | ~(xv | ph);
    mv = ph & xv;
  }
  return score;
}

// The same distance with the pattern as bit planes: plane b (bits [24 b,
// 24 b + 24) of pa) holds bit b of every residue of a, the length is in bits
// 127..120. The positions of a that match the text residue c are then
// ~OR_b (plane_b ^ (bit b of c ? all ones : 0)), a few bit operations per
// text residue instead of one comparison per pattern position.
__device__ __forceinline__ uint32_t lev_planes(u128 pa, u128 b) {
  const uint32_t m = (uint32_t)(pa >> 120), n = key_len(b);
  if (m == 0) return n;
  if (n == 0) return m;
  const uint64_t lo = (uint64_t)pa, hi = (uint64_t)(pa >> 64);
  const uint32_t P0 = (uint32_t)lo & 0xFFFFFFu, P1 = (uint32_t)(lo >> 24) & 0xFFFFFFu;
  const uint32_t P2 = (uint32_t)((lo >> 48) | (hi << 16)) & 0xFFFFFFu;
  const uint32_t P3 = (uint32_t)(hi >> 8) & 0xFFFFFFu, P4 = (uint32_t)(hi >> 32) & 0xFFFFFFu;
  const uint32_t mmask = (1u << m) - 1u;
  uint32_t pv = mmask, mv = 0u, score = m;
  const uint32_t top = 1u << (m - 1);
  uint64_t th = (uint64_t)(b >> 64), tl = (uint64_t)b;  // residue j at bits 115 - 5j .. 119 - 5j
  for (uint32_t j = 0; j < n; ++j) {
    const uint32_t c = (uint32_t)(th >> 51) & 31u;
    th = (th << 5) | (tl >> 59);
    tl <<= 5;
    const uint32_t x = (P0 ^ (0u - (c & 1u))) | (P1 ^ (0u - ((c >> 1) & 1u))) |
                       (P2 ^ (0u - ((c >> 2) & 1u))) | (P3 ^ (0u - ((c >> 3) & 1u))) |
                       (P4 ^ (0u - ((c >> 4) & 1u)));
    const uint32_t eq = ~x & mmask;
    const uint32_t xv = eq | mv;
    const uint32_t xh = (((eq & pv) + pv) ^ pv) | eq;
    uint32_t ph = mv | ~(xh | pv);
    uint32_t mh = pv & xh;
    if (ph & top)
      ++score;
    else if (mh & top)
      --score;
    ph = (ph << 1) | 1u;
    mh = mh << 1;
    pv = mh | ~(xv | ph);
    mv = ph & xv;
  }
  return score;
}

// The same distance where only a value of at most K matters, both strings as bit
// planes: K + 1 or more for pairs further apart. The furthest rows of the
// diagonals -K..K for 0..K edits (Ukkonen 1985; Myers 1986), where a run of
// equal residues is one count of trailing zeros in the diagonal's mismatch mask
// (bit t: residue t of a differs from residue t + d of b). About 65 operations for
// the masks and 60 for the rows at K = 2, the same for every length; lev_planes
// takes about 25 per residue.
template <int K>
__device__ __forceinline__ uint32_t lev_within(u128 pa, u128 pb) {
  const int m = (int)(pa >> 120), n = (int)(pb >> 120);
  uint32_t A[5], B[5];
  {
    const uint64_t lo = (uint64_t)pa, hi = (uint64_t)(pa >> 64);
    const uint64_t lo2 = (uint64_t)pb, hi2 = (uint64_t)(pb >> 64);
    A[0] = (uint32_t)lo & 0xFFFFFFu;
    A[1] = (uint32_t)(lo >> 24) & 0xFFFFFFu;
    A[2] = (uint32_t)((lo >> 48) | (hi << 16)) & 0xFFFFFFu;
    A[3] = (uint32_t)(hi >> 8) & 0xFFFFFFu;
    A[4] = (uint32_t)(hi >> 32) & 0xFFFFFFu;
    B[0] = (uint32_t)lo2 & 0xFFFFFFu;
    B[1] = (uint32_t)(lo2 >> 24) & 0xFFFFFFu;
    B[2] = (uint32_t)((lo2 >> 48) | (hi2 << 16)) & 0xFFFFFFu;
    B[3] = (uint32_t)(hi2 >> 8) & 0xFFFFFFu;
    B[4] = (uint32_t)(hi2 >> 32) & 0xFFFFFFu;
  }
  // per diagonal d: where it ends, its mismatches (all ones from there on), and
  // the furthest row with the edits so far
  int end[2 * K + 1], row[2 * K + 1] = {};
  uint32_t miss[2 * K + 1];
#pragma unroll
  for (int d = -K; d <= K; ++d) {
    uint32_t x = 0;
#pragma unroll
    for (int q = 0; q < 5; ++q) x |= A[q] ^ (d >= 0 ? B[q] >> (d >= 0 ? d : 0) : B[q] << (d < 0 ? -d : 0));
    end[d + K] = max(min(m, n - d), 0);
    miss[d + K] = x | (~0u << end[d + K]);
  }
  uint32_t dist = K + 1;
#pragma unroll
  for (int e = 0; e <= K; ++e) {
    int left = 0;  // the row of diagonal d - 1 before this edit
#pragma unroll
    for (int d = -e; d <= e; ++d) {
      const int old = row[d + K];
      int t = 0;
      if (e > 0) {
        t = d > -e && d < e ? old + 1 : 0;                       // substitution
        if (d - 1 >= -(e - 1) && d - 1 <= e - 1) t = max(t, left);              // b's residue added
        if (d + 1 <= e - 1 && d + 1 >= -(e - 1)) t = max(t, row[d + 1 + K] + 1);  // a's deleted
        t = min(t, end[d + K]);
      }
      t += __builtin_ctz(miss[d + K] >> t);
      left = old;
      row[d + K] = t;
      if (d == n - m && t >= m && dist > (uint32_t)e) dist = (uint32_t)e;
    }
  }
  return dist;
}

// Hamming distance of two packed keys of equal length (Section III C's
// filter): residues sit in 5-bit fields at bits [5 g, 5 g + 5), so a field of
// a XOR b is non-zero exactly where the residues differ; OR-ing each field's
// five bits into its lowest bit and counting those bits gives the distance.
// Fields past the length are zero in both keys.
__device__ __forceinline__ uint32_t hamming_keys(u128 a, u128 b) {
  constexpr uint64_t LOW = 0x0084210842108421ull;  // bits 0, 5, 10, ..., 55
  const u128 x = a ^ b;
  const uint64_t lo = (uint64_t)x & ((1ull << 60) - 1ull);         // fields 0..11
  const uint64_t hi = (uint64_t)(x >> 60) & ((1ull << 60) - 1ull);  // fields 12..23
  const uint64_t flo = (lo | (lo >> 1) | (lo >> 2) | (lo >> 3) | (lo >> 4)) & LOW;
  const uint64_t fhi = (hi | (hi >> 1) | (hi >> 2) | (hi >> 3) | (hi >> 4)) & LOW;
  return (uint32_t)(__popcll(flo) + __popcll(fhi));
}

// ------------------------------------------------------------------ verdicts

constexpr uint8_t DROP = 0xFFu;  // verdict of a pair over k

// The final filter of one candidate pair (i, j): its distance, or DROP.
// MODE 0: pa holds the bit-plane form of the first sequences (pack's planes)
// and the distance is Levenshtein; MODE 1: pa holds their packed keys and the
// distance is Hamming over equal lengths; MODE 2 (paired-chain records): pa
// and sb are the first chains (planes, keys), pa2 and sb2 the second, and the
// distance is the sum of the two chains' Levenshtein distances. The length
// difference bounds each distance from below and skips most far pairs.
template <int MODE>
__device__ __forceinline__ uint8_t pair_verdict(const u128* __restrict__ pa,
                                                const u128* __restrict__ sb,
                                                const u128* __restrict__ pa2,
                                                const u128* __restrict__ sb2, uint32_t i,
                                                uint32_t j, int k) {
  const u128 a = pa[i], b = sb[j];
  const int la = (int)(a >> 120), lb = (int)key_len(b);
  if (MODE == 1) {
    if (la == lb) {
      const uint32_t dd = hamming_keys(a, b);
      if (dd <= (uint32_t)k) return (uint8_t)dd;
    }
  } else if (MODE == 2) {
    const u128 a2 = pa2[i], b2 = sb2[j];
    const int la2 = (int)(a2 >> 120), lb2 = (int)key_len(b2);
    if (abs(la - lb) + abs(la2 - lb2) <= k) {
      const uint32_t d1 = lev_planes(a, b);
      if (d1 <= (uint32_t)k) {
        const uint32_t dd = d1 + lev_planes(a2, b2);
        if (dd <= (uint32_t)k) return (uint8_t)dd;
      }
    }
  } else if (abs(la - lb) <= k) {
    const uint32_t dd = lev_planes(a, b);
    if (dd <= (uint32_t)k) return (uint8_t)dd;
  }
  return DROP;
}

// The same for two sequences that both have bit planes (PAIRED: records, pa2 the
// second chains' planes): half the random reads of pair_verdict, from arrays that
// the Infinity Cache can hold.
template <bool PAIRED, int K>
__device__ __forceinline__ uint8_t planes_verdict_k(const u128* __restrict__ pa,
                                                    const u128* __restrict__ pa2, uint32_t i,
                                                    uint32_t j) {
  const u128 a = pa[i], b = pa[j];
  u128 a2 = 0, b2 = 0;
  if (PAIRED) {
    a2 = pa2[i];
    b2 = pa2[j];
  }
  uint32_t d = lev_within<K>(a, b);
  if (PAIRED && d <= (uint32_t)K) d += lev_within<K>(a2, b2);
  return d <= (uint32_t)K ? (uint8_t)d : DROP;
}

template <bool PAIRED>
__device__ __forceinline__ uint8_t planes_verdict(const u128* __restrict__ pa,
                                                  const u128* __restrict__ pa2, uint32_t i,
                                                  uint32_t j, int k) {
  switch (k) {
    case 0: return planes_verdict_k<PAIRED, 0>(pa, pa2, i, j);
    case 1: return planes_verdict_k<PAIRED, 1>(pa, pa2, i, j);
    case 2: return planes_verdict_k<PAIRED, 2>(pa, pa2, i, j);
    default: return planes_verdict_k<PAIRED, 3>(pa, pa2, i, j);
  }
}

// Minimum-cost global alignment of a and b with substitution costs sub[20][20]
// and a fixed indel cost, by the full dynamic programme (rows kept in
// registers: both strings have at most 24 residues).
__device__ __forceinline__ uint32_t weighted_keys(u128 a, u128 b, const uint8_t* sub,
                                                  uint32_t indel) {
  const uint32_t la = key_len(a), lb = key_len(b);
  uint32_t row[KEY_MAX_LEN + 1];
#pragma unroll
  for (int y = 0; y <= KEY_MAX_LEN; ++y) row[y] = (uint32_t)y * indel;
  for (uint32_t x = 1; x <= la; ++x) {
    const uint32_t ca = key_residue(a, (int)x - 1);
    uint32_t diag = row[0];
    row[0] = x * indel;
#pragma unroll
    for (int y = 1; y <= KEY_MAX_LEN; ++y) {
      if ((uint32_t)y <= lb) {
        const uint32_t cb = key_residue(b, y - 1);
        const uint32_t up = row[y];
        uint32_t best = diag + sub[ca * 20 + cb];
        const uint32_t del = up + indel, ins = row[y - 1] + indel;
        best = del < best ? del : best;
        best = ins < best ? ins : best;
        diag = up;
        row[y] = best;
      }
    }
  }
  uint32_t res = 0;
#pragma unroll
  for (int y = 0; y <= KEY_MAX_LEN; ++y)
    if ((uint32_t)y == lb) res = row[y];
  return res;
}

}  // namespace sdk
