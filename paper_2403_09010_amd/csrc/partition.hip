// Partitioned grouping path for gfx950: the automatic path of self searches and
// of queries against a hashed index, and the index build.
//
//   k_gen_part      generates every distinct <= k-deletion variant as a 64-bit
//                   element [hash | id] into an LDS tile, orders the tile by
//                   the top `lb` hash bits and writes each bin's run to the
//                   bin's region: one write of the elements, no sort pass
//   k_filter_group  one workgroup per bin: an LDS bitmap finds the elements
//                   whose hash may be shared, which are grouped by their full
//                   stored hash in LDS and emit their id pairs
//   k_part_split    a first level's bins, each split by further hash bits
//   k_sort_bins     bins in order of the whole element (index build)
//   k_join_bins     query bins joined with the index elements of the same bits
//   k_gen_probe     query variants looked up in the index as they are generated
//   k_join_runs,    queries and variants with more matches than a workgroup of
//   k_put_runs      those two follows
//
// Equal variants have equal hashes and so share a bin; a collision of hashes
// only adds a candidate that the verification rejects.
#include <algorithm>

#include "hashtab.h"
#include "pair_put.h"
#include "partition_tail.h"
#include "sd_device.h"
#include "sd_internal.h"

namespace sdk {

static __constant__ HashTab kHashTab = make_hash_tab();

// ------------------------------------------------------------------ generator

// Inclusive prefix XOR over each 32-lane half of the wave.
__device__ __forceinline__ uint32_t half_xor_scan(uint32_t v) {
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);  // row_shr:1
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);  // row_shr:2
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);  // row_shr:4
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);  // row_shr:8
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, true);  // row_bcast:15
  return v;
}

__device__ __forceinline__ uint32_t read_lane(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// Lane i's value of lane i + 1 (the last lane gets 0).
__device__ __forceinline__ uint32_t next_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, true);  // wave_shl:1
}

// 64-bit words as two 32-bit halves (rotations by less than 32 are one
// v_alignbit per half).
struct W2 {
  uint32_t lo, hi;
};
__device__ __forceinline__ W2 operator^(W2 a, W2 b) { return W2{a.lo ^ b.lo, a.hi ^ b.hi}; }
__device__ __forceinline__ W2 w2(uint64_t v) { return W2{(uint32_t)v, (uint32_t)(v >> 32)}; }
__device__ __forceinline__ W2 rotr_w2(W2 v, uint32_t n) {
  return W2{__builtin_amdgcn_alignbit(v.hi, v.lo, n), __builtin_amdgcn_alignbit(v.lo, v.hi, n)};
}
__device__ __forceinline__ W2 rotl_w2(W2 v, uint32_t n) {  // 0 < n < 32
  return W2{__builtin_amdgcn_alignbit(v.lo, v.hi, 32 - n),
            __builtin_amdgcn_alignbit(v.hi, v.lo, 32 - n)};
}

// Residue t (t <= 23) of a packed key.
__device__ __forceinline__ uint32_t residue_at(u128 key, uint32_t t) {
  const uint64_t lo = (uint64_t)key, top = (uint64_t)(key >> 56);
  const uint32_t s = 115 - 5 * t;
  return (uint32_t)((s >= 56 ? top : lo) >> (s >= 56 ? s - 56 : s)) & 31u;
}

// What lane t of a half wave needs of its sequence: the two bytes of the packed key
// that hold residue t, and the length.
struct SeqLane {
  uint32_t field, length;
};
__device__ __forceinline__ SeqLane load_lane(const u128* __restrict__ seq, uint32_t x, uint32_t t) {
  const unsigned char* p = reinterpret_cast<const unsigned char*>(seq + x);
  uint16_t f;
  __builtin_memcpy(&f, p + ((115 - 5 * min(t, 23u)) >> 3), 2);
  return SeqLane{f, p[15]};
}

// The end of the chunk of sequences from xa on whose variants fit the tile.
template <int TILE>
__device__ __forceinline__ uint32_t chunk_end(const uint32_t* s_pref, uint32_t xa, uint32_t ns) {
  uint32_t lo = xa + 1, hi = ns;
  const uint32_t p0 = s_pref[xa];
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (s_pref[mid] - p0 <= (uint32_t)TILE)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Deletion pairs in colexicographic order (pair u = p2 (p2 - 1) / 2 + p1, the
// same for every length: a string of length L has the first C(L, 2)): the LDS
// byte offsets of the pair's two words in its sequence's rows, and the bits of
// n1 and n2 that a canonical pair has (p2 in n1; p1 in n1, or in n2 if p2 =
// p1 + 1). Unused entries need bit 31, which no mask has.
constexpr int GP_ROW = KEY_MAX_LEN;
constexpr int GP_CHUNKS = (KEY_MAX_LEN * (KEY_MAX_LEN - 1) / 2 + 63) / 64;

struct PairLanes {
  uint4 e[GP_CHUNKS * 64];
};

constexpr PairLanes make_pair_lanes() {
  PairLanes t{};
  for (int u = 0; u < GP_CHUNKS * 64; ++u) t.e[u] = uint4{0, GP_ROW * 8, 1u << 31, 0};
  int u = 0;
  for (int p2 = 1; p2 < KEY_MAX_LEN; ++p2)
    for (int p1 = 0; p1 < p2; ++p1, ++u) {
      const bool adj = p2 == p1 + 1;
      t.e[u].x = (unsigned)p1 * 8;
      t.e[u].y = (unsigned)(GP_ROW + p2) * 8;
      t.e[u].z = (1u << p2) | (adj ? 0u : 1u << p1);
      t.e[u].w = adj ? 1u << p1 : 0u;
    }
  return t;
}

static __constant__ PairLanes kPairLanes = make_pair_lanes();

// A lane's deletion pairs, one per 64 of them.
struct LanePairs {
  uint32_t pa[GP_CHUNKS], pb[GP_CHUNKS], need1[GP_CHUNKS], need2[GP_CHUNKS];
  __device__ __forceinline__ void load(uint32_t lane) {
#pragma unroll
    for (int c = 0; c < GP_CHUNKS; ++c) {
      const uint4 v = kPairLanes.e[c * 64 + lane];
      pa[c] = v.x;
      pb[c] = v.y;
      need1[c] = v.z;
      need2[c] = v.w;
    }
  }
};

// Every distinct variant with at most k deletions of a wave's two sequences.
//
// With P[p] the prefix XORs of the position terms rotr(B[s_t], t) (the hash
// of hashtab.h) and Q[p] = P[p] ^ rotl(P[p + 1], 1), the variant without
// p1 < p2 < p3 hashes to
//   C[L - 3] ^ rotl(P[L], 3) ^ Q[p1] ^ rotl(Q[p2], 1) ^ rotl(Q[p3], 2)
// and with fewer deletions to the same form with fewer terms: one table word
// per deletion.
//
// Each 32-lane half has one sequence (`key`; the upper half's counts only with
// `two`): lane t holds residue t, the prefix XORs come from a scan over the
// lanes, the canonical-test masks (sd_device.h: n1, n2, n3) from ballots, and
// the variants with at most one deletion leave straight from the lanes' own
// values. The deletion pairs in colexicographic order (larger position major)
// are the same for every length, so lane l's pairs l, l + 64, ... are fixed for
// the whole kernel: their LDS offsets and the mask bits they need stay in
// registers. Triples run over the largest position p3 (uniform): their first
// two positions are the pairs below p3, whose hash words are already in
// registers and whose canonical lanes are a prefix of the pairs' ballots,
// except the range with p2 = p3 - 1, which has its own.
//
// put(hash, id, position): the lower half's sequence has id id0 and positions
// from its lanes' at0 on, the upper half's id0 + 1 and its own at0. rows: the
// wave's 4 GP_ROW words of LDS.
template <bool K3, class Put>
__device__ __forceinline__ void gen_step(SeqLane key, uint32_t id0, bool two, uint32_t at0, int k,
                                         uint64_t* rows, const uint64_t* s_b, const uint64_t* s_c,
                                         const LanePairs& lp, Put&& put) {
  constexpr int QS = GP_ROW;
  const uint32_t lane = threadIdx.x & 63u, half = lane >> 5, t = lane & 31u;
  const uint32_t L = key.length;
  const uint32_t r = t < L ? __builtin_amdgcn_ubfe(key.field, (115 - 5 * min(t, 23u)) & 7u, 5) : 31u;
  W2 term = rotr_w2(w2(s_b[r]), t);
  if (t >= L) term = W2{0, 0};
  const W2 incl{half_xor_scan(term.lo), half_xor_scan(term.hi)};
  const W2 q = incl ^ term ^ rotl_w2(incl, 1);
  const W2 plA{read_lane(incl.lo, 31), read_lane(incl.hi, 31)};
  const W2 plB{read_lane(incl.lo, 63), read_lane(incl.hi, 63)};
  const W2 pl{half ? plB.lo : plA.lo, half ? plB.hi : plA.hi};
  // n1 bit p: p = L - 1 or s[p] != s[p + 1] (residues past the end read
  // as 31, which no residue equals)
  const uint32_t r1 = next_lane(r);
  const bool c1 = t < L && (r != r1 || t + 1 == L);
  const uint64_t n1 = __builtin_amdgcn_ballot_w64(c1);
  if (k >= 2 && t < (uint32_t)QS) {
    const W2 base2 = w2(s_c[L >= 2 ? L - 2 : 0]) ^ rotl_w2(pl, 2);
    uint64_t* row = rows + half * 2 * QS;
    const W2 q2 = rotl_w2(q, 1) ^ base2;
    row[t] = ((uint64_t)q.hi << 32) | q.lo;
    row[QS + t] = ((uint64_t)q2.hi << 32) | q2.lo;
  }
  uint32_t atA, atB;
  {
    // none (lane L, where q = P[L] ^ rotl(P[L], 1)) and one deletion
    const bool keep = ((k >= 1 && c1) || t == L) && (!half || two);
    const W2 h = w2(s_c[t < L ? L - 1 : L & 31u]) ^ rotl_w2(pl, 1) ^ q;
    const uint64_t bal = __builtin_amdgcn_ballot_w64(keep);
    const uint32_t na = (uint32_t)__popc((uint32_t)bal);
    const uint32_t rank = mask_rank(bal) - (half ? na : 0u);
    if (keep) put(h, id0 + half, at0 + rank);
    atA = read_lane(at0, 0) + na;
    atB = read_lane(at0, 32) + (uint32_t)__popc((uint32_t)(bal >> 32));
  }
  if (k < 2) return;
  const uint32_t r2 = next_lane(r1);
  const uint64_t n2 = __builtin_amdgcn_ballot_w64(t < L && (r != r2 || t + 2 >= L));
  uint64_t n3 = 0;
  if (K3) n3 = __builtin_amdgcn_ballot_w64(t < L && (r != next_lane(r2) || t + 3 >= L));
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  // the words of two chunks of both sequences are read at once: most lengths have
  // two (the empty asm keeps the compiler from moving the reads to their uses,
  // each with its own wait)
  auto pair_word = [&](uint32_t sI, int c) {
    const unsigned char* Q = reinterpret_cast<const unsigned char*>(rows + sI * 2 * QS);
    return w2(*reinterpret_cast<const uint64_t*>(Q + lp.pa[c])) ^
           w2(*reinterpret_cast<const uint64_t*>(Q + lp.pb[c]));
  };
  W2 first[2][2];
#pragma unroll
  for (int x = 0; x < 4; ++x) first[x >> 1][x & 1] = pair_word(x >> 1, x & 1);
#pragma unroll
  for (int x = 0; x < 4; ++x)
    asm volatile("" : "+v"(first[x >> 1][x & 1].lo), "+v"(first[x >> 1][x & 1].hi));
#pragma unroll
  for (uint32_t sI = 0; sI < 2; ++sI) {
    if (sI && !two) break;
    const uint32_t SL = read_lane(L, sI ? 32 : 0);
    const uint32_t m1 = (uint32_t)(n1 >> (sI * 32)), m2 = (uint32_t)(n2 >> (sI * 32));
    const unsigned char* Q = reinterpret_cast<const unsigned char*>(rows + sI * 2 * QS);
    // (in a vector register: one AND-OR with the hash's mask in a scalar one)
    uint32_t id = id0 + sI;
    asm volatile("" : "+v"(id));
    uint32_t at = sI ? atB : atA;
    const uint32_t np = SL * (SL - 1) / 2;
    W2 pw[GP_CHUNKS];
    uint64_t kp[GP_CHUNKS], kq[GP_CHUNKS];
    const uint32_t m3 = (uint32_t)(n3 >> (sI * 32));
    pw[0] = first[sI][0];
    pw[1] = first[sI][1];
#pragma unroll
    for (int c = 0; c < GP_CHUNKS; ++c) {
      if ((uint32_t)c * 64 >= np) break;  // uniform
      if (c >= 2) pw[c] = pair_word(sI, c);
      const W2 h = pw[c];
      const bool keep = ((lp.need1[c] & ~m1) | (lp.need2[c] & ~m2)) == 0;
      const uint64_t bal = __builtin_amdgcn_ballot_w64(keep);
      if (keep) put(h, id, at + mask_rank(bal));
      at += (uint32_t)__popcll(bal);
      if (K3) {
        kp[c] = bal;
        // with p3 = p2 + 1: p2 needs n2, p1 needs n1, or n3 if p1, p2, p3 adjoin
        const uint32_t b2 = 1u << ((lp.pb[c] >> 3) - QS), b1 = lp.need1[c] & ~b2;
        kq[c] = __builtin_amdgcn_ballot_w64(((b2 & ~m2) | (b1 & ~m1) | (lp.need2[c] & ~m3)) == 0 &&
                         (lp.need1[c] >> 31) == 0);
      }
    }
    if (K3 && SL >= 3) {
      const W2 pls = sI ? plB : plA;
      // pw holds base2 ^ Q[p1] ^ rotl(Q[p2], 1)
      const W2 sw = w2(s_c[SL - 2]) ^ rotl_w2(pls, 2) ^ w2(s_c[SL - 3]) ^ rotl_w2(pls, 3);
      for (uint32_t p3 = 2; p3 < SL; ++p3) {
        if (!((m1 >> p3) & 1u)) continue;
        const W2 tw = sw ^ rotl_w2(w2(*reinterpret_cast<const uint64_t*>(Q + p3 * 8)), 2);
        const uint32_t u0 = (p3 - 1) * (p3 - 2) / 2, u1 = p3 * (p3 - 1) / 2;
#pragma unroll
        for (int c = 0; c < GP_CHUNKS; ++c) {
          const uint32_t c0 = (uint32_t)c * 64;
          if (c0 >= u1) break;  // uniform
          const uint64_t below0 = u0 >= c0 + 64 ? ~0ull : u0 > c0 ? (1ull << (u0 - c0)) - 1 : 0;
          const uint64_t below1 = u1 >= c0 + 64 ? ~0ull : (1ull << (u1 - c0)) - 1;
          const uint64_t bal = (kp[c] & below0) | (kq[c] & below1 & ~below0);
          if ((bal >> lane) & 1u) put(pw[c] ^ tw, id, at + mask_rank(bal));
          at += (uint32_t)__popcll(bal);
        }
      }
    }
  }
  // the next sequences' rows overwrite these
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// gen_step over a block's sequences, into an LDS tile that partition_tail
// orders and writes.
//
// Bound: vector instructions and LDS operations (about half of what either can
// issue, with four waves per SIMD; eight, in half the registers, take 30% longer),
// then the element writes. 101M variants of 1M sequences (k = 2): 0.46 ms, of
// which the generation alone is 0.26; 454M (k = 3) 2.57 ms; two workgroups of 512 threads on a CU, so that one generates
// while the other writes (one of 1,024: 0.55). Generating them in sequence
// order took 0.40 and the first radix pass another 0.39.
template <int NT, int TILE, bool K3>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_gen_part(const u128* __restrict__ seq,
                                                 const uint32_t* __restrict__ vcnt, uint32_t nseq,
                                                 int k, uint32_t idbits, uint32_t spb,
                                                 sd::PartOut o) {
  constexpr int NW = NT / 64;
  extern __shared__ __align__(16) unsigned char lds[];
  const uint32_t nb = 1u << o.lb;
  // (the tile last: what lies within 64 KiB needs no address arithmetic)
  // s_q: [NW][2][2][GP_ROW], per sequence Q, then rotl(Q, 1) ^ base
  uint64_t* s_q = reinterpret_cast<uint64_t*>(lds);
  uint64_t* s_b = s_q + NW * 4 * GP_ROW;               // [32]
  uint64_t* s_c = s_b + 32;                          // [32]
  uint32_t* s_pref = reinterpret_cast<uint32_t*>(s_c + 32);  // [NT + 2]
  uint32_t* s_tmp = s_pref + NT + 2;                 // [NW]
  uint32_t* s_cnt = s_tmp + NW;                      // [nb]
  uint64_t* s_e = reinterpret_cast<uint64_t*>(s_cnt + nb);
  const uint32_t s0 = blockIdx.x * spb;
  const uint32_t ns = min(spb, nseq - s0);
  const uint32_t lane = threadIdx.x & 63u, half = lane >> 5;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lomask = idbits >= 32 ? 0u : ~((1u << idbits) - 1u);
  const int binshift = 32 - o.lb;  // bin = high word of the element >> binshift
  {
    const uint32_t c = threadIdx.x < ns ? vcnt[s0 + threadIdx.x] : 0u;
    uint32_t total;
    const uint32_t ex = block_excl_scan<NT>(c, s_tmp, &total);
    if (threadIdx.x <= ns) s_pref[threadIdx.x] = ex;
    if (threadIdx.x == NT - 1 && ns == NT) s_pref[NT] = total;
  }
  if (threadIdx.x < 32) s_b[threadIdx.x] = kHashTab.b[threadIdx.x];
  if (threadIdx.x < 32) s_c[threadIdx.x] = kHashTab.c[threadIdx.x];
  __syncthreads();
  // the block's sequences in chunks that fit the tile (one chunk unless the
  // sequences have far more variants than the mean)
  uint32_t xa = 0;
  while (xa < ns) {
    const uint32_t p0 = s_pref[xa], xb = chunk_end<TILE>(s_pref, xa, ns);
    // (the pack kernel counted exactly the canonical sets, so the positions
    // handed out below end where the next sequence's begin)
    auto put = [&](W2 h, uint32_t id, uint32_t pos) {
      s_e[pos] = ((uint64_t)h.hi << 32) | ((h.lo & lomask) | id);
      atomicAdd(&s_cnt[h.hi >> binshift], 1u);
    };
    // this lane's deletion pairs (read for every chunk: their registers are
    // free while the tile is written; the empty asm keeps the compiler from
    // moving the loads out of the loop)
    uint32_t pl_lane = lane;
    asm volatile("" : "+v"(pl_lane));
    LanePairs lp;
    lp.load(pl_lane);
    uint32_t x = xa + 2 * w;
    // each half's sequence, loaded one step ahead
    SeqLane key{0, 0};
    if (x < xb) key = load_lane(seq, s0 + min(x + half, xb - 1), lane & 31u);
    for (uint32_t i = threadIdx.x; i < nb; i += NT) s_cnt[i] = 0;
    __syncthreads();
    for (; x < xb; x += 2 * NW) {
      const bool two = x + 1 < xb;
      const SeqLane cur = key;
      key = load_lane(seq, s0 + min(x + 2 * NW + half, xb - 1), lane & 31u);
      const uint32_t at0 = s_pref[min(x + half, xb)] - p0;
      gen_step<K3>(cur, s0 + x, two, at0, k, s_q + w * 4 * GP_ROW, s_b, s_c, lp, put);
    }
    __syncthreads();
    const int shift = 64 - o.lb;
    partition_tail<NT, TILE, sd::tile_max_lb(NT), false>(
        s_e, s_pref[xb] - p0, s_cnt, s_tmp, o.lb,
        [&](uint64_t v) { return (uint32_t)(v >> shift); }, 0, o.elem, o.cursor, o.region, o.nbins,
        o.nxl, o.slots, o.fill, o.cap, o.over_count);
    __syncthreads();
    xa = xb;
  }
}

// ------------------------------------------------------------------ paired chains

// Paired-chain records: a record (a, b) is the joined string a T b, whose
// variants delete up to two residues and never T (residue code 20). T equals no
// residue, so the canonical rule of single chains holds for the joined string
// with T's own bits cleared from the masks.
constexpr uint32_t PAIR_T = 20;

__device__ __forceinline__ uint64_t low_bits(uint32_t n) { return n >= 64 ? ~0ull : (1ull << n) - 1; }

// Distinct variants of each record with at most k <= 2 deletions (the sum over
// the canonical sets), their total as in k_pack.
__global__ __launch_bounds__(256) void k_paired_distinct(const u128* __restrict__ pa,
                                                         const u128* __restrict__ pb, uint64_t n,
                                                         int k, uint32_t* __restrict__ vcnt,
                                                         unsigned long long* __restrict__ sums) {
  __shared__ uint32_t s_tmp[4];
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  uint32_t c = 0;
  if (i < n) {
    const u128 a = pa[i], b = pb[i];
    const uint32_t la = (uint32_t)(a >> 120), L = la + 1 + (uint32_t)(b >> 120);
    uint64_t d1 = 0, d2 = 0;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      const uint64_t x = (uint64_t)(a >> (24 * q)) & 0xFFFFFFu, y = (uint64_t)(b >> (24 * q)) & 0xFFFFFFu;
      const uint64_t pl = x | (uint64_t)((PAIR_T >> q) & 1u) << la | y << (la + 1);
      d1 |= pl ^ (pl >> 1);
      d2 |= pl ^ (pl >> 2);
    }
    const uint64_t keep = ~(1ull << la);  // L >= 3
    const uint64_t n1 = ((d1 & low_bits(L - 1)) | 1ull << (L - 1)) & keep;
    const uint64_t n2 = ((d2 & low_bits(L - 2)) | 1ull << (L - 2)) & keep;
    c = 1;
    if (k >= 1) c += (uint32_t)__popcll(n1);
    if (k >= 2) {
      const uint32_t m = (uint32_t)__popcll(n1);
      c += m * (m - 1) / 2 - (uint32_t)__popcll(n1 & (n1 >> 1)) + (uint32_t)__popcll(n2 & (n1 >> 1));
    }
    vcnt[i] = c;
  }
  uint32_t total;
  block_excl_scan<256>(c, s_tmp, &total);
  if (threadIdx.x == 0 && total)
    atomicAdd(&sums[blockIdx.x % sd::PACK_SUMS], (unsigned long long)total);
}

// k_gen_part for paired-chain records: one record per wave, lane t holding
// position t of the joined string. The larger deleted position p2 is uniform
// and lane p1 has the other's hash word, so a pair costs one XOR with a word
// of p2 and the canonical lanes are mask bits; two values of p2 <= 32 share a
// step, one per half of the wave. Bound: vector instructions and LDS
// operations. 1M records, k = 2: 2.1 ms for 382M distinct variants; unranking
// each deletion set and hashing its whole joined string took 12.1 (470M).
template <int NT, int TILE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_gen_part_paired(
    const u128* __restrict__ sa, const u128* __restrict__ sb, const uint32_t* __restrict__ vcnt,
    uint32_t nrec, int k, uint32_t idbits, uint32_t spb, sd::PartOut o) {
  constexpr int NW = NT / 64;
  extern __shared__ __align__(16) unsigned char lds[];
  const uint32_t nb = 1u << o.lb;
  uint64_t* s_e = reinterpret_cast<uint64_t*>(lds);
  uint64_t* s_b = s_e + TILE;                        // [32]
  uint64_t* s_c = s_b + 32;                          // [64]
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_c + 64);
  uint32_t* s_pref = s_cnt + nb;                     // [NT + 1]
  uint32_t* s_tmp = s_pref + NT + 1;                 // [NW]
  const uint32_t s0 = blockIdx.x * spb;
  const uint32_t ns = min(spb, nrec - s0);
  const uint32_t t = threadIdx.x & 63u, half = t >> 5;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lomask = idbits >= 32 ? 0u : ~((1u << idbits) - 1u);
  const int binshift = 32 - o.lb;
  {
    const uint32_t c = threadIdx.x < ns ? vcnt[s0 + threadIdx.x] : 0u;
    uint32_t total;
    const uint32_t ex = block_excl_scan<NT>(c, s_tmp, &total);
    if (threadIdx.x <= ns) s_pref[threadIdx.x] = ex;
    if (threadIdx.x == NT - 1 && ns == NT) s_pref[NT] = total;
  }
  if (threadIdx.x < 32) s_b[threadIdx.x] = kHashTab.b[threadIdx.x];
  if (threadIdx.x < 64) s_c[threadIdx.x] = kHashTab.c[threadIdx.x];
  __syncthreads();
  uint32_t xa = 0;
  while (xa < ns) {
    const uint32_t p0 = s_pref[xa], xb = chunk_end<TILE>(s_pref, xa, ns);
    auto put = [&](W2 h, uint32_t id, uint32_t pos) {
      s_e[pos] = ((uint64_t)h.hi << 32) | ((h.lo & lomask) | id);
      atomicAdd(&s_cnt[h.hi >> binshift], 1u);
    };
    uint32_t x = xa + w;
    u128 ka = 0, kb = 0;  // the wave's record, loaded one step ahead
    if (x < xb) {
      ka = sa[s0 + x];
      kb = sb[s0 + x];
    }
    for (uint32_t i = threadIdx.x; i < nb; i += NT) s_cnt[i] = 0;
    __syncthreads();
    for (; x < xb; x += NW) {
      const u128 a = ka, b = kb;
      const uint32_t nx = min(x + NW, xb - 1);
      ka = sa[s0 + nx];
      kb = sb[s0 + nx];
      const uint32_t id = s0 + x;
      uint32_t at = __builtin_amdgcn_readfirstlane(s_pref[x] - p0);
      const uint32_t la = key_len(a), L = la + 1 + key_len(b);
      const uint32_t tb = t - la - 1;  // position in b
      const uint32_t r = t < la    ? residue_at(a, min(t, 23u))
                         : t == la ? PAIR_T
                         : t < L   ? residue_at(b, min(tb, 23u))
                                   : 31u;
      W2 word = w2(s_b[r]);
      if (half) word = W2{word.hi, word.lo};  // rotate by 32
      W2 term = rotr_w2(word, t & 31u);
      if (t >= L) term = W2{0, 0};
      W2 incl{half_xor_scan(term.lo), half_xor_scan(term.hi)};
      const W2 low{read_lane(incl.lo, 31), read_lane(incl.hi, 31)};
      if (half) incl = incl ^ low;
      const W2 q = incl ^ term ^ rotl_w2(incl, 1);
      const W2 pl{read_lane(incl.lo, 63), read_lane(incl.hi, 63)};
      // (residues past the end read as 31, which no position equals)
      const uint32_t r1 = next_lane(r);
      const bool c1 = t < L && t != la && (r != r1 || t + 1 == L);
      const uint64_t n1 = __ballot(c1);
      {
        // none (lane L, where q = P[L] ^ rotl(P[L], 1)) and one deletion
        const bool keep = (k >= 1 && c1) || t == L;
        const W2 h = w2(s_c[t < L ? L - 1 : L]) ^ rotl_w2(pl, 1) ^ q;
        const uint64_t bal = __ballot(keep);
        if (keep) put(h, id, at + mask_rank(bal));
        at += (uint32_t)__popcll(bal);
      }
      if (k < 2) continue;
      const uint32_t r2 = next_lane(r1);
      const uint64_t n2 = __ballot(t < L && t != la && (r != r2 || t + 2 >= L));
      const W2 base = w2(s_c[L - 2]) ^ rotl_w2(pl, 2);
      const W2 mine = base ^ q;  // lane p1's words
      W2 both{(uint32_t)__shfl((int)mine.lo, (int)(t & 31u), 64),
              (uint32_t)__shfl((int)mine.hi, (int)(t & 31u), 64)};
      // lanes p1 < p2 of the canonical pairs with p2 >= 1
      auto lanes_of = [&](uint32_t p2) {
        return (n1 & low_bits(p2 - 1)) | (n2 & (1ull << (p2 - 1)));
      };
      auto word_of = [&](uint32_t p2) {
        return rotl_w2(W2{read_lane(q.lo, (int)p2), read_lane(q.hi, (int)p2)}, 1);
      };
      uint64_t m = n1 & low_bits(33) & ~1ull;
      while (m) {
        const uint32_t a2 = (uint32_t)__builtin_ctzll(m);
        m &= m - 1;
        uint64_t bal = lanes_of(a2);
        W2 wa = word_of(a2), wb = wa;
        if (m) {
          const uint32_t b2 = (uint32_t)__builtin_ctzll(m);
          m &= m - 1;
          bal |= lanes_of(b2) << 32;
          wb = word_of(b2);
        }
        const W2 wd{half ? wb.lo : wa.lo, half ? wb.hi : wa.hi};
        if ((bal >> t) & 1u) put(both ^ wd, id, at + mask_rank(bal));
        at += (uint32_t)__popcll(bal);
      }
      for (m = n1 & ~low_bits(33); m; m &= m - 1) {
        const uint32_t p2 = (uint32_t)__builtin_ctzll(m);
        const uint64_t bal = lanes_of(p2);
        if ((bal >> t) & 1u) put(mine ^ word_of(p2), id, at + mask_rank(bal));
        at += (uint32_t)__popcll(bal);
      }
    }
    __syncthreads();
    const int shift = 64 - o.lb;
    partition_tail<NT, TILE, sd::tile_max_lb(NT), false>(
        s_e, s_pref[xb] - p0, s_cnt, s_tmp, o.lb,
        [&](uint64_t v) { return (uint32_t)(v >> shift); }, 0, o.elem, o.cursor, o.region, o.nbins,
        o.nxl, o.slots, o.fill, o.cap, o.over_count);
    __syncthreads();
    xa = xb;
  }
}

// ------------------------------------------------------------------ second level

// Splits the regions of a first partition by `lb` more hash bits, for inputs
// whose bins would be too large for k_filter_group. Consecutive workgroups take
// consecutive tiles of one sub-region of the first level, so the open lines of
// few bins are in each L2 at a time.
template <int NT, int TILE>
__global__ __launch_bounds__(NT) void k_part_split(sd::PartOut in, sd::PartOut o,
                                                   uint32_t tiles) {
  constexpr int PER = TILE / NT;
  extern __shared__ __align__(16) unsigned char lds[];
  const uint32_t lb = (uint32_t)(o.lb - in.lb), nb = 1u << lb;
  uint64_t* s_e = reinterpret_cast<uint64_t*>(lds);
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_e + TILE);
  uint32_t* s_tmp = s_cnt + nb;
  const uint32_t sub = blockIdx.x / tiles;
  const uint32_t bin = sub >> in.nxl, x = in.nxl ? sub & 7u : 0u;
  const uint32_t cu = x * in.nbins + bin;
  uint32_t c = in.cursor[cu];
  if (c > in.region) c = in.fill[cu];
  const uint32_t t0 = (blockIdx.x - sub * tiles) * TILE;
  if (t0 >= c) return;
  const uint32_t m = min((uint32_t)TILE, c - t0);
  const uint64_t* __restrict__ src = in.elem + (uint64_t)((bin << in.nxl) + x) * in.region + t0;
  const int shift = 64 - o.lb;
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
      atomicAdd(&s_cnt[(uint32_t)(e[r] >> shift) & (nb - 1)], 1u);
    }
  }
  __syncthreads();
  partition_tail<NT, TILE, sd::PART_MAX_SPLIT, false, true>(
      s_e, m, s_cnt, s_tmp, (int)lb, [&](uint64_t v) { return (uint32_t)(v >> shift) & (nb - 1); },
      bin << lb, o.elem, o.cursor, o.region, o.nbins, o.nxl, o.slots, o.fill, o.cap, o.over_count);
}

// ------------------------------------------------------------------ filter and group

// Sizes of a shape of k_filter_group with a bitmap of 2^SB bits in `LDS` bytes (as
// many as leave room for the shape's workgroups on a CU): a round groups FULL
// elements of at most CAP at once (pairs take the rest) and sorts them into NBK
// buckets. The elements and buckets lie where the first bitmap was.
template <int SB, int LDS>
struct FilterShape {
  static constexpr int SEEN = (1 << SB) / 8;   // bytes of the first bitmap
  static constexpr int TWICE = SEEN / 8;       // and of the second
  static constexpr int NBK = SEEN / 8 / 4;     // 4 bytes each
  static constexpr int CAP = (LDS - TWICE - NBK * 4) / 64 * 8;
  static constexpr int FULL = CAP - CAP / 8;
  static constexpr int BK_AT = CAP * 8;
  static constexpr int TWICE_AT = BK_AT + NBK * 4;
  static_assert(TWICE_AT >= SEEN && TWICE_AT + TWICE <= LDS, "layout");
};
constexpr int FG_ROWS = 8;      // elements in flight per thread
constexpr int FG_MAX_ROUNDS = 64;

// One workgroup per bin. First pass over the bin's elements: each sets the bit
// of its low hash bits in a bitmap of 2^SB bits; one that finds its bit set
// makes two marks in a second, independently indexed bitmap of an eighth of
// the size. Second pass: the elements whose marks are set (every element of a
// group of equal hashes, and 6% of the others at 0.1 elements per bit) are
// collected in LDS, put in order of a few more hash bits, and compared inside
// each of these small buckets; equal hashes give an id pair. If more
// candidates are found than LDS holds they are grouped in several rounds by
// further hash bits, each a pass over the elements. A bin that overflowed its
// regions, or whose round still does not fit (thousands of elements of one
// hash), is listed in big[] for the sort-and-runs path.
//
// Bound: the two reads of the elements, the second backwards, so that it begins
// with what the caches still hold; then LDS accesses, of which a wave has eight in
// flight where its rows are full. An element's two marks lie in one word: one
// access, for a few more false marks than two words would give. 1G elements in
// 2^17 bins: 2.59 ms (2.80 with a bounds check and a wait per access and marks in
// two words); 101M in 2^11 bins: 0.41 (0.43). Elements kept in registers between
// the two reads cost more than they save, since half as many waves fit: 2.96 and
// 0.58 ms.
template <int NT, int SB, int LDS, bool WIDE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8))) void k_filter_group(
    sd::PartOut in, sd::PairBins out, uint64_t* __restrict__ big,
    unsigned long long* __restrict__ nbig) {
  constexpr uint32_t idbits = WIDE ? 32 : 24;
  using F = FilterShape<SB, LDS>;
  constexpr int PER = (F::FULL + NT - 1) / NT;
  static_assert(F::NBK <= 4 * NT, "bucket scan");
  extern __shared__ __align__(16) unsigned char lds[];
  uint32_t* s_seen = reinterpret_cast<uint32_t*>(lds);
  uint32_t* s_tw = reinterpret_cast<uint32_t*>(lds + F::TWICE_AT);
  uint64_t* s_e = reinterpret_cast<uint64_t*>(lds);
  uint32_t* s_bk = reinterpret_cast<uint32_t*>(lds + F::BK_AT);
  __shared__ uint32_t s_n;
  __shared__ unsigned long long s_at;
  __shared__ uint32_t s_tmp[NT / 64];
  const uint32_t bin = blockIdx.x, nx = 1u << in.nxl;
  const uint32_t lane = threadIdx.x & 63u;
  if (bin == 0 && threadIdx.x == 0 && *in.over_count) {
    // the overflow area (elements of overflowed bins only)
    const unsigned long long y = atomicAdd(nbig, 1ull);
    big[2 * y] = in.slots;
    big[2 * y + 1] = min(in.slots + *in.over_count, in.cap);
  }
  uint32_t total = 0;
  bool over = false;
  for (uint32_t x = 0; x < nx; ++x) {
    const uint32_t c = in.cursor[x * in.nbins + bin];
    over |= c > in.region;
    total += c;
  }
  if (total < 2) return;
  const uint64_t base = (uint64_t)(bin << in.nxl) * in.region;
  if (over) {
    // its elements lie in the regions and in the overflow area
    if (threadIdx.x < nx) {
      const uint32_t cu = threadIdx.x * in.nbins + bin;
      uint32_t c = in.cursor[cu];
      if (c > in.region) c = in.fill[cu];
      const unsigned long long y = atomicAdd(nbig, 1ull);
      big[2 * y] = base + (uint64_t)threadIdx.x * in.region;
      big[2 * y + 1] = base + (uint64_t)threadIdx.x * in.region + c;
    }
    return;
  }
  for (uint32_t i = threadIdx.x; i < (uint32_t)F::SEEN / 4; i += NT) s_seen[i] = 0;
  for (uint32_t i = threadIdx.x; i < (uint32_t)F::TWICE / 4; i += NT) s_tw[i] = 0;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  // every element of the bin: waves share out the regions, and each takes
  // FG_ROWS rows of 64 elements at a time
  constexpr uint32_t NW = NT / 64, ROW = 64 * FG_ROWS;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t parts = NW > nx ? NW / nx : 1u;
  // (full: all of them are there, and no operation waits for a bounds check)
  auto stream = [&](bool back, auto&& f) {
    for (uint32_t x = w & (nx - 1); x < nx; x += NW) {
      const uint32_t c = in.cursor[x * in.nbins + bin];
      const uint64_t* __restrict__ p = in.elem + base + (uint64_t)x * in.region;
      const uint32_t first = (w >> in.nxl) * ROW, step = parts * ROW;
      if (first >= c) continue;
      const uint32_t steps = (c - first + step - 1) / step;
      for (uint32_t q = 0; q < steps; ++q) {
        const uint32_t t0 = first + (back ? steps - 1 - q : q) * step;
        uint64_t e[FG_ROWS];
        if (t0 + ROW <= c) {
#pragma unroll
          for (int u = 0; u < FG_ROWS; ++u) e[u] = p[t0 + u * 64 + lane];
          f(e, ROW, std::true_type{});
        } else {
#pragma unroll
          for (int u = 0; u < FG_ROWS; ++u) {
            const uint32_t i = t0 + u * 64 + lane;
            e[u] = i < c ? p[i] : 0;
          }
          f(e, c - t0, std::false_type{});
        }
      }
    }
  };
  auto hash = [](uint64_t e) { return (uint32_t)(e >> idbits); };
  // an element's two marks: bits of one word of the second bitmap, which its
  // topmost free hash bits choose (the first bitmap goes by the lowest ones)
  constexpr int TWBITS = SB - 8;  // log2 of its words
  const int twshift = max(64 - (int)idbits - in.lb - TWBITS, 0);
  auto mark_word = [&](uint32_t h) { return (h >> twshift) & ((1u << TWBITS) - 1); };
  auto marks = [](uint32_t h) { return 1u << (h & 31u) | 1u << ((h >> 5) & 31u); };
  stream(false, [&](const uint64_t(&e)[FG_ROWS], uint32_t left, auto full) {
    uint32_t old[FG_ROWS];
#pragma unroll
    for (int u = 0; u < FG_ROWS; ++u) {
      const uint32_t h = hash(e[u]);
      old[u] = 0;
      if (full || u * 64 + lane < left)
        old[u] = atomicOr(&s_seen[(h >> 5) & ((1u << (SB - 5)) - 1)], 1u << (h & 31u));
    }
#pragma unroll
    for (int u = 0; u < FG_ROWS; ++u) {
      const uint32_t h = hash(e[u]);
      if ((old[u] >> (h & 31u)) & 1u) atomicOr(&s_tw[mark_word(h)], marks(h));
    }
  });
  __syncthreads();
  const uint64_t idmask = (1ull << idbits) - 1;
  // bucket: the bits below the bin's; round: the next six
  constexpr int NBKLOG = __builtin_ctz(F::NBK);
  const int bkshift = sd::hash_shift(in.lb, NBKLOG, idbits);
  const int rdshift = sd::hash_shift(in.lb, NBKLOG + 6, idbits);
  uint32_t rounds = 1;
  for (uint32_t round = 0; round < rounds; ++round) {
    stream(true, [&](const uint64_t(&e)[FG_ROWS], uint32_t left, auto full) {
      uint64_t bal[FG_ROWS];
      uint32_t tw[FG_ROWS], tot = 0;
#pragma unroll
      for (int u = 0; u < FG_ROWS; ++u) tw[u] = s_tw[mark_word(hash(e[u]))];
#pragma unroll
      for (int u = 0; u < FG_ROWS; ++u) {
        const uint32_t need = marks(hash(e[u]));
        bool keep = (tw[u] & need) == need && (full || u * 64 + lane < left);
        if (rounds > 1) keep = keep && ((uint32_t)(e[u] >> rdshift) & (rounds - 1)) == round;
        bal[u] = __ballot(keep);
        tot += (uint32_t)__popcll(bal[u]);
      }
      if (tot) {
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s_n, tot);
        at = __builtin_amdgcn_readfirstlane(at);
        if (at + tot <= (uint32_t)F::FULL) {
#pragma unroll
          for (int u = 0; u < FG_ROWS; ++u) {
            if ((bal[u] >> lane) & 1u) s_e[at + mask_rank(bal[u])] = e[u];
            at += (uint32_t)__popcll(bal[u]);
          }
        }
      }
    });
    __syncthreads();
    const uint32_t m = s_n;
    __syncthreads();
    if (threadIdx.x == 0) s_n = 0;
    if (m > (uint32_t)F::FULL) {
      if (rounds == 1) {
        // again in rounds of about half a capacity
        while (rounds < (uint32_t)FG_MAX_ROUNDS && rounds * (uint32_t)F::FULL < 2 * m) rounds <<= 1;
        round = ~0u;
        __syncthreads();
        continue;
      }
      if (threadIdx.x < nx) {
        const uint32_t c = in.cursor[threadIdx.x * in.nbins + bin];
        const unsigned long long y = atomicAdd(nbig, 1ull);
        big[2 * y] = base + (uint64_t)threadIdx.x * in.region;
        big[2 * y + 1] = base + (uint64_t)threadIdx.x * in.region + c;
      }
      return;
    }
    // order the candidates by bucket
    uint64_t e[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const uint32_t i = threadIdx.x + r * NT;
      e[r] = i < m ? s_e[i] : 0;
    }
    for (uint32_t i = threadIdx.x; i < (uint32_t)F::NBK; i += NT) s_bk[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r)
      if (threadIdx.x + r * NT < m)
        atomicAdd(&s_bk[(uint32_t)(e[r] >> bkshift) & (F::NBK - 1)], 1u);
    __syncthreads();
    {
      constexpr int BPT = (F::NBK + NT - 1) / NT;
      uint32_t c[BPT], sum = 0;
#pragma unroll
      for (int q = 0; q < BPT; ++q) {
        const uint32_t b = threadIdx.x * BPT + q;
        c[q] = b < (uint32_t)F::NBK ? s_bk[b] : 0;
        sum += c[q];
      }
      uint32_t tot;
      uint32_t ex = block_excl_scan<NT>(sum, s_tmp, &tot);
#pragma unroll
      for (int q = 0; q < BPT; ++q) {
        const uint32_t b = threadIdx.x * BPT + q;
        if (b < (uint32_t)F::NBK) s_bk[b] = ex;
        ex += c[q];
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r)
      if (threadIdx.x + r * NT < m)
        s_e[atomicAdd(&s_bk[(uint32_t)(e[r] >> bkshift) & (F::NBK - 1)], 1u)] = e[r];
    __syncthreads();
    // (every bucket's entry is its end now)
    // each element pairs with the later ones of its bucket that share its hash
    // (not unrolled: three copies of seven times the loop took registers from the
    // passes over the elements)
    auto each_pair = [&](auto&& f) {
#pragma unroll 1
      for (uint32_t i = threadIdx.x; i < m; i += NT) {
        const uint64_t a = s_e[i];
        const uint32_t end = s_bk[(uint32_t)(a >> bkshift) & (F::NBK - 1)];
        for (uint32_t y = i + 1; y < end; ++y) {
          const uint64_t b = s_e[y];
          if (((b ^ a) >> idbits) == 0) {
            const uint64_t ia = a & idmask, ib = b & idmask;
            f(ia < ib ? ia << 32 | ib : ib << 32 | ia);
          }
        }
      }
    };
    // the pairs are counted first: a list per XCD takes them with one reservation
    // (a few bins hold groups of thousands: nothing here is per pair but its write),
    // and where they go to their bins they collect behind the candidates, so that
    // their reservations are in flight side by side
    uint32_t cnt = 0, tot;
    each_pair([&](uint64_t) { ++cnt; });
    const uint32_t at0 = block_excl_scan<NT>(cnt, s_tmp, &tot);
    if (tot > out.limit && threadIdx.x == 0)
      atomicAdd(out.missed, out.lb == 0 ? 1ull : (unsigned long long)tot);
    if (tot == 0 || (tot > out.limit && out.lb > 0)) {
      // (uniform: on to the barrier)
    } else if (out.lb == 0) {
      const uint32_t x = blockIdx.x & ((1u << out.nxl) - 1);
      if (threadIdx.x == 0) s_at = list_reserve(out, x, tot);
      __syncthreads();
      if (cnt) {
        const uint32_t room = sd::list_room(s_at, tot, out.region);
        uint64_t* dst = out.base + (uint64_t)x * out.region + s_at;
        uint32_t at = at0;
        each_pair([&](uint64_t v) {
          if (at < room) dst[at] = v;
          ++at;
        });
      }
    } else {
      uint64_t* s_pair = s_e + m;
      const uint32_t room = F::CAP - m;
      for (uint32_t w = 0; w < tot; w += room) {
        uint32_t at = at0 - w;  // (below 0: a large number)
        each_pair([&](uint64_t v) {
          if (at < room) s_pair[at] = v;
          ++at;
        });
        __syncthreads();
        const uint32_t np = min(tot - w, room);
        for (uint32_t i = threadIdx.x; i < np; i += NT) pair_put(out, s_pair[i]);
        __syncthreads();
      }
    }
    __syncthreads();  // the next round rewrites the LDS
  }
}

// ------------------------------------------------------------------ sorted bins

// An index keeps its elements in order of the whole word. Bins of the top hash
// bits are in order already; each fits LDS, where a counting pass by the next
// BITS hash bits leaves buckets of one or two elements on average, and an
// element's place in its bucket is the number of smaller ones there.

// elements of each bin
__global__ __launch_bounds__(256) void k_bin_totals(sd::PartOut in, uint32_t* __restrict__ cnt) {
  const uint32_t b = blockIdx.x * 256 + threadIdx.x;
  if (b >= in.nbins) return;
  uint32_t c = 0;
  for (uint32_t x = 0; x < (1u << in.nxl); ++x) c += in.cursor[x * in.nbins + b];
  cnt[b] = c;
}

// One workgroup per bin: its elements in order to out[off[bin], ...). A bin that
// does not fit (single variants shared by thousands of sequences) is left out:
// the element ranges of its regions go to big as [2x, 2x + 1), counted in *nbig.
// *repeats counts the elements that equal the one before them in the output.
//
// Bound: LDS accesses, and its element reads and writes, which take two thirds
// of its time at the rate of a copy (202M elements: 0.79 ms, 4.1 TB/s). Elements
// stay in registers until their bucket's start is known, one LDS write instead
// of two, and buckets are small because a wave waits for its largest one: with
// two writes and buckets of three elements 1.12 ms, and 1.17 by workgroups of
// 1,024 threads.
template <int NT, int CAP, int BITS, int R>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8))) void k_sort_bins(
    sd::PartOut in, const uint64_t* __restrict__ off, uint64_t* __restrict__ out,
    uint64_t* __restrict__ big, unsigned long long* __restrict__ nbig,
    unsigned long long* __restrict__ repeats) {
  constexpr int NBK = 1 << BITS, BPT = NBK / NT;
  static_assert(BPT * NT == NBK && NT >= 512, "buckets per thread, waves per region");
  extern __shared__ __align__(16) unsigned char lds[];
  uint64_t* s_e = reinterpret_cast<uint64_t*>(lds);
  uint32_t* s_bk = reinterpret_cast<uint32_t*>(s_e + CAP);  // NBK + 1
  uint32_t* s_tmp = s_bk + NBK + 1;
  const uint32_t bin = blockIdx.x, nx = 1u << in.nxl;
  // the waves share the bin's regions out: one lane's elements are its strip's
  // every `stride` in one region
  const uint32_t wave = threadIdx.x >> 6, mine = wave & (nx - 1);
  const uint32_t strip = (wave >> in.nxl) * 64 + (threadIdx.x & 63);
  const uint32_t stride = (NT / 64 >> in.nxl) * 64;
  uint32_t m = 0, c = 0;
  bool over = false;
  for (uint32_t x = 0; x < nx; ++x) {
    const uint32_t v = in.cursor[x * in.nbins + bin];
    m += v;
    over |= v > in.region || v > R * stride;
    if (x == mine) c = v;
  }
  if (over || m > (uint32_t)CAP) {
    if (threadIdx.x < nx) {
      const uint32_t x = threadIdx.x, cu = x * in.nbins + bin;
      const uint64_t a = (uint64_t)((bin << in.nxl) + x) * in.region;
      const uint64_t w = atomicAdd(nbig, 1ull);
      big[2 * w] = a;
      big[2 * w + 1] = a + (in.cursor[cu] > in.region ? in.fill[cu] : in.cursor[cu]);
    }
    return;
  }
  const uint64_t* __restrict__ src = in.elem + (uint64_t)((bin << in.nxl) + mine) * in.region;
  uint64_t e[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = strip + r * stride;
    e[r] = i < c ? src[i] : 0;
  }
  for (uint32_t i = threadIdx.x; i < (uint32_t)NBK; i += NT) s_bk[i] = 0;
  __syncthreads();
  const int shift = 64 - in.lb - BITS;
  uint32_t at[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (strip + r * stride < c) at[r] = atomicAdd(&s_bk[(uint32_t)(e[r] >> shift) & (NBK - 1)], 1u);
  __syncthreads();
  {
    uint32_t n[BPT], sum = 0, tot;
#pragma unroll
    for (int q = 0; q < BPT; ++q) sum += n[q] = s_bk[threadIdx.x * BPT + q];
    uint32_t ex = block_excl_scan<NT>(sum, s_tmp, &tot);
#pragma unroll
    for (int q = 0; q < BPT; ++q) {
      s_bk[threadIdx.x * BPT + q] = ex;
      ex += n[q];
    }
    if (threadIdx.x == 0) s_bk[NBK] = m;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (strip + r * stride < c) s_e[s_bk[(uint32_t)(e[r] >> shift) & (NBK - 1)] + at[r]] = e[r];
  __syncthreads();
  uint64_t* __restrict__ dst = out + off[bin];
  uint32_t same = 0;
  for (uint32_t i = threadIdx.x; i < m; i += NT) {
    const uint64_t a = s_e[i];
    const uint32_t bk = (uint32_t)(a >> shift) & (NBK - 1);
    const uint32_t s = s_bk[bk], end = s_bk[bk + 1];
    uint32_t p = s;
    for (uint32_t y = s; y < end; ++y) {
      const uint64_t b = s_e[y];
      const bool rep = b == a && y < i;
      same += rep;
      p += b < a || rep;
    }
    dst[p] = a;
  }
  if (same) atomicAdd(repeats, (unsigned long long)same);
}

// The m elements of the bins that were left out, in order, to their places.
__global__ __launch_bounds__(256) void k_place_bins(const uint64_t* __restrict__ X, uint64_t m,
                                                    int lb, const uint64_t* __restrict__ off,
                                                    uint64_t* __restrict__ out,
                                                    unsigned long long* __restrict__ repeats) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= m) return;
  const uint64_t e = X[i], first = e >> (64 - lb) << (64 - lb);
  uint64_t lo = 0, hi = i;  // the bin's first element
  while (lo < hi) {
    const uint64_t mid = (lo + hi) / 2;
    if (X[mid] < first)
      lo = mid + 1;
    else
      hi = mid;
  }
  out[off[e >> (64 - lb)] + (i - lo)] = e;
  if (i && X[i - 1] == e) atomicAdd(repeats, 1ull);
}

// ------------------------------------------------------------------ queries against an index

// First position in E[lo, hi) whose hash is at least h (E ascending), from a
// guess: the bracket of 16 on either side first (hashes are uniform, so that a
// segment of 1,200 elements misses by about 13), then wider ones, then a binary
// search inside.
__device__ __forceinline__ uint32_t lower_bound_near(const uint64_t* __restrict__ E, uint32_t lo,
                                                     uint32_t hi, uint32_t guess, uint64_t h,
                                                     uint32_t idbits) {
  uint32_t w = 16;
  while (true) {
    const uint32_t a = guess - lo > w ? guess - w : lo, b = hi - guess > w ? guess + w : hi;
    const bool below = a == lo || (E[a - 1] >> idbits) < h;
    const bool above = b == hi || (E[b] >> idbits) >= h;
    if (below && above) {
      lo = a;
      hi = b;
      break;
    }
    // (the half that missed is narrowed to, and the guess moves to its end)
    if (!below) hi = a;
    else lo = b;
    guess = below ? lo : hi;
    w = w < (1u << 28) ? w * 8 : ~0u;
  }
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if ((E[mid] >> idbits) < h)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

constexpr int PB_ROWS = 4;

// Few queries: each variant is looked up in the index as it is generated, from
// its place by interpolation in its directory segment; no query element is
// written, sorted or read.
//
// Bound: the latency of three to four dependent loads per variant. A variant
// shared by many references would hold its wave up: beyond the first PB_SHORT
// of a run, the rest is left to the waves of the workgroup, one run each; runs of more
// than RUN_MOST, and of more than RUN_LONG beyond the first PB_LONGS (copies: a query's
// every variant has one), are left to k_put_runs.
constexpr uint32_t PB_SHORT = 4, PB_QUEUE = 1024, PB_LONGS = 16;
constexpr uint32_t RUN_LONG = 256, RUN_MOST = 1024;

// The end of the run that holds position p, by steps that double (E[p] >> idbits is h).
__device__ __forceinline__ uint32_t run_end(const uint64_t* __restrict__ E, uint32_t p, uint32_t n,
                                            uint64_t h, uint32_t idbits) {
  uint64_t lo = (uint64_t)p + 1, step = 1;  // the end lies at lo or beyond
  while (lo - 1 + step < n && (E[lo - 1 + step] >> idbits) == h) {
    lo += step;
    step *= 2;
  }
  uint64_t hi = min(lo - 1 + step, (uint64_t)n);
  while (lo < hi) {
    const uint64_t mid = (lo + hi) / 2;
    if ((E[mid] >> idbits) == h)
      lo = mid + 1;
    else
      hi = mid;
  }
  return (uint32_t)lo;
}

// Adds the active lanes' runs to the queue (those past its room are only counted).
__device__ __forceinline__ void push_run(const sd::RunQueue& q, uint32_t p, uint32_t n,
                                         uint32_t id) {
  const uint64_t act = __ballot(true);
  uint32_t at = 0;
  if (mask_rank(act) == 0) at = atomicAdd(q.count, (uint32_t)__popcll(act));
  at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + mask_rank(act);
  if (at < q.cap)
    q.runs[at] = sd::PairRun{p, n, id};
  else if (at - q.cap < sd::RUN_SAMPLE)
    atomicAdd(q.missed, (unsigned long long)n);
}

template <bool K3>
__global__ __launch_bounds__(256) void k_gen_probe(const u128* __restrict__ seq, uint32_t nseq,
                                                   int k, const uint64_t* __restrict__ E,
                                                   uint32_t nkeys,
                                                   const uint32_t* __restrict__ seg_start,
                                                   const uint32_t* __restrict__ seg_end, int bits,
                                                   uint32_t idbits, sd::PairBins out,
                                                   sd::RunQueue longs) {
  __shared__ uint64_t s_q[4 * 4 * GP_ROW];
  __shared__ uint64_t s_b[32], s_c[32];
  __shared__ uint32_t s_run[PB_QUEUE], s_id[PB_QUEUE];  // runs left over: position, query
  __shared__ uint32_t s_runs, s_longs;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (threadIdx.x == 0) {
    s_runs = 0;
    s_longs = 0;
  }
  if (threadIdx.x < 32) {
    s_b[threadIdx.x] = kHashTab.b[threadIdx.x];
    s_c[threadIdx.x] = kHashTab.c[threadIdx.x];
  }
  LanePairs lp;
  lp.load(lane);
  __syncthreads();
  const uint64_t idmask = (1ull << idbits) - 1;
  auto put = [&](W2 v, uint32_t id, uint32_t) {
    const uint64_t full = (uint64_t)v.hi << 32 | v.lo, h = full >> idbits;
    const uint32_t seg = bits ? v.hi >> (32 - bits) : 0u;
    const uint32_t s = seg_start[seg], e = seg_end[seg];
    if (s >= e) return;
    const uint32_t frac = (uint32_t)((full << bits) >> 32);
    uint32_t p = lower_bound_near(E, s, e, s + (uint32_t)(((uint64_t)(e - s) * frac) >> 32), h,
                                  idbits);
    for (uint32_t c = 0; p < e; ++p, ++c) {
      const uint64_t r = E[p];
      if ((r >> idbits) != h) break;
      if (c == PB_SHORT) {
        const uint32_t x = atomicAdd(&s_runs, 1u);
        if (x < PB_QUEUE) {
          s_run[x] = p;
          s_id[x] = id;
          break;
        }
        if (e - p > RUN_MOST && (E[p + RUN_MOST] >> idbits) == h) {
          push_run(longs, p, run_end(E, p, e, h, idbits) - p, id);
          break;
        }
      }
      pair_put<true>(out, (uint64_t)id << 32 | (r & idmask));
    }
  };
  {
    const uint32_t x = (blockIdx.x * 4 + w) * 2;
    if (x < nseq) {
      const SeqLane key = load_lane(seq, min(x + (lane >> 5), nseq - 1), lane & 31u);
      gen_step<K3>(key, x, x + 1 < nseq, 0, k, s_q + w * 4 * GP_ROW, s_b, s_c, lp, put);
    }
  }
  __syncthreads();
  const uint32_t runs = min(s_runs, PB_QUEUE);
  for (uint32_t q = w; q < runs; q += 4) {  // a wave per run
    const uint32_t p0 = s_run[q], id = s_id[q];
    const uint64_t h = E[p0] >> idbits;
    auto at = [&](uint32_t i) {
      const uint64_t p = (uint64_t)p0 + i + lane;
      return p < nkeys ? E[p] : ~h << idbits;
    };
    const uint64_t r0 = at(0);
    const bool same = (r0 >> idbits) == h;
    if (__ballot(same) != ~0ull) {  // most runs end here
      if (same) pair_put(out, (uint64_t)id << 32 | (r0 & idmask));
      continue;
    }
    if (nkeys - p0 > RUN_LONG && (E[p0 + RUN_LONG] >> idbits) == h) {
      uint32_t before = 0;
      if (lane == 0) before = atomicAdd(&s_longs, 1u);
      before = (uint32_t)__builtin_amdgcn_readfirstlane((int)before);
      if (before >= PB_LONGS ||
          (nkeys - p0 > RUN_MOST && (E[p0 + RUN_MOST] >> idbits) == h)) {
        if (lane == 0) push_run(longs, p0, run_end(E, p0, nkeys, h, idbits) - p0, id);
        continue;
      }
    }
    pair_put(out, (uint64_t)id << 32 | (r0 & idmask));
    for (uint32_t i = 64;; i += 64 * PB_ROWS) {  // (PB_ROWS reads in flight together)
      uint64_t r[PB_ROWS];
      bool on[PB_ROWS];
#pragma unroll
      for (int u = 0; u < PB_ROWS; ++u) r[u] = at(i + u * 64);
#pragma unroll
      for (int u = 0; u < PB_ROWS; ++u) {
        on[u] = (r[u] >> idbits) == h;
        r[u] = (uint64_t)id << 32 | (r[u] & idmask);
      }
      pair_put_rows(out, r, on);
      if (__ballot(on[PB_ROWS - 1]) != ~0ull) break;
    }
  }
}

// Many queries: one workgroup per hash segment reads the segment's query
// elements (a bin of the generator, of which it takes 1 / 2^sub by further hash
// bits) and its index elements once, and pairs equal hashes.
//   1. the query elements set bits of a bitmap (SB: its bits, log2);
//   2. the index elements whose bit is set (those with a query of the same hash
//      and some of the others) collect in LDS and mark a smaller bitmap;
//   3. the query elements with their marks collect in the first bitmap's place;
//   4. the index survivors are put in order of a few more hash bits, and each
//      query survivor is compared with its bucket.
// If LDS does not hold the survivors, the steps run in rounds by further hash bits;
// where it does not hold those of a round either, or would take too many rounds
// (variants shared by thousands), the segment or the round is listed in `copies`.
//
// Bound: the one read of the index elements, at 8 bytes each. 200K queries
// (20M variants) against 202M index elements: 0.48 ms (3.4 TB/s); looking each
// element up by binary search in its sorted segment took 0.82, after two radix
// passes over the queries.
constexpr int JB_SB = 18;                      // query bitmap, bits (32 KiB)
constexpr int JB_TB = 15;                      // mark bitmap, bits
constexpr uint32_t JB_CAP = 5056;              // index survivors in LDS (two workgroups on a CU)
constexpr uint32_t JB_QCAP = (1u << JB_SB) / 64;  // query survivors
constexpr int JB_NBK = 1024;
constexpr uint32_t JB_SHARED = 48;  // index elements of one bucket: 4 on average
constexpr uint32_t JB_ROUNDS = 16;  // most rounds
constexpr size_t JB_LDS = (1 << JB_SB) / 8 + (1 << JB_TB) / 8 + JB_CAP * 8 + JB_NBK * 4;

template <int NT, bool WIDE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8))) void k_join_bins(
    sd::PartOut in, const uint64_t* __restrict__ E, const uint32_t* __restrict__ seg_start,
    const uint32_t* __restrict__ seg_end, int bits, int sub, sd::PairBins out,
    sd::JoinParts copies) {
  constexpr uint32_t idbits = WIDE ? 32 : 24;
  constexpr uint32_t NW = NT / 64, ROW = 64 * FG_ROWS;
  constexpr uint32_t PER = (JB_CAP + NT - 1) / NT;
  extern __shared__ __align__(16) unsigned char lds[];
  uint32_t* s_bq = reinterpret_cast<uint32_t*>(lds);
  uint64_t* s_qe = reinterpret_cast<uint64_t*>(lds);  // step 3 on
  uint32_t* s_br = s_bq + (1 << JB_SB) / 32;
  uint64_t* s_e = reinterpret_cast<uint64_t*>(s_br + (1 << JB_TB) / 32);
  uint32_t* s_bk = reinterpret_cast<uint32_t*>(s_e + JB_CAP);
  __shared__ uint32_t s_n, s_nq, s_shared;
  __shared__ unsigned long long s_at;
  __shared__ uint32_t s_tmp[NW];
  // the workgroups of a query bin follow each other on one XCD, whose L2 then
  // has the bin's elements
  const uint32_t nx = 1u << in.nxl, turn = blockIdx.x >> 3;
  const uint32_t seg = in.nbins >= 8
                           ? (((turn >> sub) * 8 + (blockIdx.x & 7u)) << sub) + (turn & ((1u << sub) - 1))
                           : blockIdx.x;
  const uint32_t bin = seg >> sub;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int segbits = in.lb + sub;
  const uint32_t r0 = seg_start[seg << (bits - segbits)];
  const uint32_t r1 = seg_end[((seg + 1) << (bits - segbits)) - 1];
  if (r0 >= r1) return;
  const uint64_t base = (uint64_t)(bin << in.nxl) * in.region;
  const uint32_t parts = NW > nx ? NW / nx : 1u;
  // the segment's query elements: f(rows, whether each lane has one)
  auto queries = [&](auto&& f) {
    for (uint32_t x = w & (nx - 1); x < nx; x += NW) {
      const uint32_t cu = x * in.nbins + bin;
      uint32_t c = in.cursor[cu];
      if (c > in.region) c = in.fill[cu];
      const uint64_t* __restrict__ p = in.elem + base + (uint64_t)x * in.region;
      for (uint32_t t0 = (w >> in.nxl) * ROW; t0 < c; t0 += parts * ROW) {
        uint64_t e[FG_ROWS];
#pragma unroll
        for (int u = 0; u < FG_ROWS; ++u) {
          const uint32_t i = t0 + u * 64 + lane;
          e[u] = i < c ? p[i] : 0;
        }
        bool valid[FG_ROWS];
#pragma unroll
        for (int u = 0; u < FG_ROWS; ++u)
          valid[u] = t0 + u * 64 + lane < c && (uint32_t)(e[u] >> 32) >> (32 - segbits) == seg;
        f(e, valid);
      }
    }
  };
  // marks as in k_filter_group: two bits of one word
  constexpr int TWBITS = JB_TB - 5;
  const int twshift = max(64 - (int)idbits - segbits - TWBITS, 0);
  auto hash = [](uint64_t e) { return (uint32_t)(e >> idbits); };
  auto mark_word = [&](uint32_t h) { return (h >> twshift) & ((1u << TWBITS) - 1); };
  auto marks = [](uint32_t h) { return 1u << (h & 31u) | 1u << ((h >> 5) & 31u); };
  auto bq_word = [](uint32_t h) { return (h >> 5) & ((1u << (JB_SB - 5)) - 1); };
  const uint64_t idmask = (1ull << idbits) - 1;
  constexpr int NBKLOG = __builtin_ctz(JB_NBK);
  const int bkshift = sd::hash_shift(segbits, NBKLOG, idbits);
  const int rdshift = sd::hash_shift(segbits, NBKLOG + 6, idbits);
  uint32_t rounds = 1;
  for (uint32_t round = 0; round < rounds; ++round) {
    auto mine = [&](uint64_t e) {
      return rounds == 1 || ((uint32_t)(e >> rdshift) & (rounds - 1)) == round;
    };
    for (uint32_t i = threadIdx.x; i < ((1 << JB_SB) + (1 << JB_TB)) / 32; i += NT) s_bq[i] = 0;
    if (threadIdx.x == 0) {
      s_n = 0;
      s_nq = 0;
      s_shared = 0;  // set where a bucket is large
    }
    __syncthreads();
    queries([&](const uint64_t(&e)[FG_ROWS], const bool(&valid)[FG_ROWS]) {
#pragma unroll
      for (int u = 0; u < FG_ROWS; ++u) {
        const uint32_t h = hash(e[u]);
        if (valid[u] && mine(e[u])) atomicOr(&s_bq[bq_word(h)], 1u << (h & 31u));
      }
    });
    __syncthreads();
    // the index elements whose bit is set (full: all rows of 64 are there)
    auto look = [&](const uint64_t(&e)[FG_ROWS], uint32_t left, auto full) {
      uint64_t bal[FG_ROWS];
      uint32_t bq[FG_ROWS], tot = 0;
#pragma unroll
      for (int u = 0; u < FG_ROWS; ++u) bq[u] = s_bq[bq_word(hash(e[u]))];
#pragma unroll
      for (int u = 0; u < FG_ROWS; ++u) {
        const uint32_t h = hash(e[u]);
        const bool keep = ((bq[u] >> (h & 31u)) & 1u) && (full || u * 64 + lane < left) && mine(e[u]);
        bal[u] = __ballot(keep);
        tot += (uint32_t)__popcll(bal[u]);
        if (keep) atomicOr(&s_br[mark_word(h)], marks(h));
      }
      if (tot) {
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s_n, tot);
        at = __builtin_amdgcn_readfirstlane(at);
        if (at + tot <= JB_CAP) {
#pragma unroll
          for (int u = 0; u < FG_ROWS; ++u) {
            if ((bal[u] >> lane) & 1u) s_e[at + mask_rank(bal[u])] = e[u];
            at += (uint32_t)__popcll(bal[u]);
          }
        }
      }
    };
    for (uint32_t t0 = r0 + w * ROW; t0 < r1; t0 += NW * ROW) {
      uint64_t e[FG_ROWS];
      if (t0 + ROW <= r1) {
#pragma unroll
        for (int u = 0; u < FG_ROWS; ++u) e[u] = E[t0 + u * 64 + lane];
        look(e, ROW, std::true_type{});
      } else {
#pragma unroll
        for (int u = 0; u < FG_ROWS; ++u) {
          const uint32_t i = t0 + u * 64 + lane;
          e[u] = i < r1 ? E[i] : 0;
        }
        look(e, r1 - t0, std::false_type{});
      }
    }
    __syncthreads();
    const uint32_t m = s_n;
    if (m == 0) {
      __syncthreads();
      continue;
    }
    // query survivors
    queries([&](const uint64_t(&e)[FG_ROWS], const bool(&valid)[FG_ROWS]) {
      uint64_t bal[FG_ROWS];
      uint32_t br[FG_ROWS], tot = 0;
#pragma unroll
      for (int u = 0; u < FG_ROWS; ++u) br[u] = s_br[mark_word(hash(e[u]))];
#pragma unroll
      for (int u = 0; u < FG_ROWS; ++u) {
        const uint32_t need = marks(hash(e[u]));
        bal[u] = __ballot((br[u] & need) == need && valid[u] && mine(e[u]));
        tot += (uint32_t)__popcll(bal[u]);
      }
      if (tot) {
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s_nq, tot);
        at = __builtin_amdgcn_readfirstlane(at);
        if (at + tot <= JB_QCAP) {
#pragma unroll
          for (int u = 0; u < FG_ROWS; ++u) {
            if ((bal[u] >> lane) & 1u) s_qe[at + mask_rank(bal[u])] = e[u];
            at += (uint32_t)__popcll(bal[u]);
          }
        }
      }
    });
    __syncthreads();
    const uint32_t nq = s_nq;
    if (m > JB_CAP || nq > JB_QCAP) {
      __syncthreads();  // (every thread has read the counts)
      const uint32_t need = max(m / (JB_CAP / 5 * 4), nq / (JB_QCAP / 5 * 4)) + 1;
      if (rounds == 1 && need <= JB_ROUNDS) {
        while (rounds < need) rounds <<= 1;
        round = ~0u;  // again, in rounds
      } else if (threadIdx.x == 0) {
        copies.at[atomicAdd(copies.count, 1u)] = sd::JoinPart{seg, round, rounds};
      }
      continue;
    }
    // the index survivors by bucket
    uint64_t e[PER];
#pragma unroll
    for (uint32_t r = 0; r < PER; ++r) {
      const uint32_t i = threadIdx.x + r * NT;
      e[r] = i < m ? s_e[i] : 0;
    }
    for (uint32_t i = threadIdx.x; i < (uint32_t)JB_NBK; i += NT) s_bk[i] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < PER; ++r)
      if (threadIdx.x + r * NT < m)
        atomicAdd(&s_bk[(uint32_t)(e[r] >> bkshift) & (JB_NBK - 1)], 1u);
    __syncthreads();
    {
      static_assert(JB_NBK <= NT, "one bucket per thread");
      const uint32_t c = threadIdx.x < (uint32_t)JB_NBK ? s_bk[threadIdx.x] : 0u;
      if (c > JB_SHARED) s_shared = 1;
      uint32_t tot;
      const uint32_t ex = block_excl_scan<NT>(c, s_tmp, &tot);
      if (threadIdx.x < (uint32_t)JB_NBK) s_bk[threadIdx.x] = ex;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < PER; ++r)
      if (threadIdx.x + r * NT < m)
        s_e[atomicAdd(&s_bk[(uint32_t)(e[r] >> bkshift) & (JB_NBK - 1)], 1u)] = e[r];
    __syncthreads();
    // (every bucket's entry is its end now)
    auto each_pair = [&](auto&& f) {
      for (uint32_t i = threadIdx.x; i < nq; i += NT) {
        const uint64_t a = s_qe[i];
        const uint32_t bk = (uint32_t)(a >> bkshift) & (JB_NBK - 1);
        const uint32_t end = s_bk[bk];
        for (uint32_t y = bk ? s_bk[bk - 1] : 0u; y < end; ++y) {
          const uint64_t b = s_e[y];
          if (((b ^ a) >> idbits) == 0) f((a & idmask) << 32 | (b & idmask));
        }
      }
    };
    // counted first, as in k_filter_group, for a list or where there may be very many
    uint32_t at = 0, cnt = 1, tot = 1;
    if (out.lb == 0 || s_shared) {
      cnt = 0;
      each_pair([&](uint64_t) { ++cnt; });
      at = block_excl_scan<NT>(cnt, s_tmp, &tot);
    }
    if (tot > out.limit && threadIdx.x == 0)
      atomicAdd(out.missed, out.lb == 0 ? 1ull : (unsigned long long)tot);
    if (tot == 0 || (tot > out.limit && out.lb > 0)) {
      // (uniform: on to the barrier)
    } else if (out.lb == 0) {
      const uint32_t x = blockIdx.x & ((1u << out.nxl) - 1);
      if (threadIdx.x == 0) s_at = list_reserve(out, x, tot);
      __syncthreads();
      if (cnt) {
        const uint32_t room = sd::list_room(s_at, tot, out.region);
        uint64_t* dst = out.base + (uint64_t)x * out.region + s_at;
        each_pair([&](uint64_t v) {
          if (at < room) dst[at] = v;
          ++at;
        });
      }
    } else {
      each_pair([&](uint64_t v) { pair_put(out, v); });
    }
    __syncthreads();  // the next round rewrites the LDS
  }
}

// Query elements that a join left: those of the listed segments or rounds (a
// workgroup takes one region of one of them) and, from the last gridDim.y - 1 on, those
// of the overflow area. Each is looked up, and its run of equal hashes queued.
__global__ __launch_bounds__(256) void k_join_runs(sd::PartOut in, const uint64_t* __restrict__ E,
                                                   const uint32_t* __restrict__ seg_start,
                                                   const uint32_t* __restrict__ seg_end, int bits,
                                                   int sub, uint32_t idbits, sd::JoinParts parts,
                                                   sd::RunQueue queue) {
  const uint32_t idmask = (uint32_t)((1ull << idbits) - 1);
  auto look_up = [&](uint64_t e, uint32_t r0, uint32_t r1) {
    const uint64_t h = e >> idbits;
    uint32_t lo = r0, hi = r1;
    while (lo < hi) {
      const uint32_t mid = lo + ((hi - lo) >> 1);
      if ((E[mid] >> idbits) < h)
        lo = mid + 1;
      else
        hi = mid;
    }
    if (lo < r1 && (E[lo] >> idbits) == h)
      push_run(queue, lo, run_end(E, lo, r1, h, idbits) - lo, (uint32_t)e & idmask);
  };
  const uint32_t nx = 1u << in.nxl;
  if (blockIdx.y == nx) {
    const uint32_t n = min(*in.over_count, in.cap - in.slots);
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
      const uint64_t e = in.elem[in.slots + i];
      const uint32_t seg = bits ? (uint32_t)(e >> 32) >> (32 - bits) : 0u;
      look_up(e, seg_start[seg], seg_end[seg]);
    }
    return;
  }
  const int segbits = in.lb + sub;
  const int rdshift = sd::hash_shift(segbits, __builtin_ctz(JB_NBK) + 6, (int)idbits);
  const uint32_t np = *parts.count;
  for (uint32_t y = blockIdx.x; y < np; y += gridDim.x) {
    const sd::JoinPart part = parts.at[y];
    const uint32_t cu = blockIdx.y * in.nbins + (part.seg >> sub);
    uint32_t c = in.cursor[cu];
    if (c > in.region) c = in.fill[cu];
    const uint32_t r0 = seg_start[part.seg << (bits - segbits)];
    const uint32_t r1 = seg_end[((part.seg + 1) << (bits - segbits)) - 1];
    const uint64_t* __restrict__ p =
        in.elem + (uint64_t)(((part.seg >> sub) << in.nxl) + blockIdx.y) * in.region;
    for (uint32_t i = threadIdx.x; i < c; i += 256) {
      const uint64_t e = p[i];
      if ((uint32_t)(e >> 32) >> (32 - segbits) == part.seg &&
          (part.rounds == 1 || ((uint32_t)(e >> rdshift) & (part.rounds - 1)) == part.round))
        look_up(e, r0, r1);
    }
  }
}

constexpr uint32_t PUT_LONG = 256;

// The candidates of the queued runs, `per` runs a workgroup: long ones one after the
// other by all threads, the others by the wave that read them, one reservation for all
// of a wave's and output positions shared out evenly (the owner of each by a search
// in the wave's scanned lengths).
//
// Bound: the candidate writes. 369M candidates, nearly all of 33,000 runs of 9,000:
// 1.4 ms together with the join before it; 350 when each query's lane walked its run.
__global__ __launch_bounds__(256) void k_put_runs(const uint64_t* __restrict__ E, uint32_t idbits,
                                                  sd::RunQueue q, uint32_t per, sd::PairBins out) {
  __shared__ uint32_t s_long[256], s_nl;
  __shared__ unsigned long long s_at;
  const uint64_t idmask = (1ull << idbits) - 1;
  const uint32_t n = min(*q.count, q.cap), lane = threadIdx.x & 63u;
  for (uint64_t b0 = (uint64_t)blockIdx.x * per; b0 < n; b0 += (uint64_t)gridDim.x * per) {
    const uint32_t m = (uint32_t)min((uint64_t)per, n - b0);
    if (threadIdx.x == 0) s_nl = 0;
    __syncthreads();
    sd::PairRun r{0, 0, 0};
    if (threadIdx.x < m) r = q.runs[b0 + threadIdx.x];
    if (r.n >= PUT_LONG) {
      s_long[atomicAdd(&s_nl, 1u)] = threadIdx.x;
      r.n = 0;
    }
    const uint32_t incl = wave_incl_scan(r.n), tot = __shfl(incl, 63, 64), excl = incl - r.n;
    if (tot) {
      const uint32_t x = (blockIdx.x + (threadIdx.x >> 6)) & ((1u << out.nxl) - 1);
      unsigned long long at = 0;
      uint32_t room = 0;
      if (out.lb == 0) {
        if (lane == 0) at = list_reserve(out, x, tot);
        at = first_lane(at);
        room = sd::list_room(at, tot, out.region);
      }
      uint64_t* dst = out.base + (uint64_t)x * out.region + at;
      for (uint32_t t0 = 0; t0 < tot; t0 += 64) {
        const uint32_t t = t0 + lane;
        uint32_t lo = 0, hi = 63;  // the first lane whose inclusive count exceeds t
        while (lo < hi) {
          const uint32_t mid = (lo + hi) >> 1;
          if (__shfl(incl, (int)mid, 64) <= t)
            lo = mid + 1;
          else
            hi = mid;
        }
        const uint32_t p = __shfl(r.p, (int)lo, 64) + t - __shfl(excl, (int)lo, 64);
        const uint64_t id = __shfl(r.id, (int)lo, 64);
        if (t < tot) {
          const uint64_t v = id << 32 | (E[p] & idmask);
          if (out.lb > 0)
            pair_put(out, v);
          else if (t < room)
            dst[t] = v;
        }
      }
    }
    __syncthreads();
    const uint32_t nl = s_nl;
    for (uint32_t y = 0; y < nl; ++y) {
      const sd::PairRun l = q.runs[b0 + s_long[y]];
      const uint64_t id = (uint64_t)l.id << 32;
      if (out.lb > 0) {
        for (uint32_t i = threadIdx.x; i < l.n; i += 256) pair_put(out, id | (E[l.p + i] & idmask));
        continue;
      }
      const uint32_t x = (blockIdx.x + y) & ((1u << out.nxl) - 1);
      __syncthreads();  // (the place of the run before is read)
      if (threadIdx.x == 0) s_at = list_reserve(out, x, l.n);
      __syncthreads();
      const uint32_t room = sd::list_room(s_at, l.n, out.region);
      uint64_t* dst = out.base + (uint64_t)x * out.region + s_at;
      for (uint32_t i = threadIdx.x; i < room; i += 256) dst[i] = id | (E[l.p + i] & idmask);
    }
    __syncthreads();
  }
}

}  // namespace sdk

namespace sd {

// Dynamic LDS beyond the default limit. It is asked for at each launch: the attribute
// is the device's own, and a context may be of any.
template <class F>
static void allow_lds(F* f, size_t bytes) {
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(f),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
    (void)hipGetLastError();  // the launch reports any real problem
}

template <int NT, int TILE>
static size_t gen_lds(int lb) {
  return (size_t)TILE * 8 + (NT / 64) * 4 * KEY_MAX_LEN * 8 + 64 * 8 + ((size_t)4 << lb) +
         (NT + 2) * 4 + (NT / 64) * 4;
}

template <int NT, int TILE>
static void gen_t(const u128* seq, const uint32_t* vcnt, uint32_t n, int k, uint32_t idbits,
                  uint32_t spb, const PartOut& o, hipStream_t s) {
  if (o.lb > tile_max_lb(NT)) throw Error{SD_E_HIP, "internal error: too many bins"};
  const unsigned g = (n + spb - 1) / spb;
  if (k == 3) {
    const size_t lds = gen_lds<NT, TILE>(o.lb);
    allow_lds(&sdk::k_gen_part<NT, TILE, true>, lds);
    hipLaunchKernelGGL((sdk::k_gen_part<NT, TILE, true>), dim3(g), dim3(NT), lds, s, seq, vcnt,
                       n, k, idbits, spb, o);
  } else {
    const size_t lds = gen_lds<NT, TILE>(o.lb);
    allow_lds(&sdk::k_gen_part<NT, TILE, false>, lds);
    hipLaunchKernelGGL((sdk::k_gen_part<NT, TILE, false>), dim3(g), dim3(NT), lds, s, seq, vcnt,
                       n, k, idbits, spb, o);
  }
}

// The bins as a producer's workgroups see them. One with a sixteenth of all expected
// candidates holds copies: far more pairs than bins were sized for, which would queue
// one by one for their counters (10,000 sequences with 300 copies of one, k = 2,
// 5.4M candidates: 10 ms). They are only counted then, and go to lists in the next
// attempt. (200,000 queries of 2M references without copies: 670,000 candidates, more
// than 4,096 of them from some workgroups.)
static PairBins with_limit(const PairBins& out) {
  PairBins o = out;
  o.limit = std::max(4096u, out.expect / 16);
  return o;
}

// Sequences per workgroup (at most `most`): their variants fill 15/16 of the
// tile on average.
static uint32_t seqs_per_tile(uint64_t n, uint64_t nkeys, uint32_t tile, uint32_t most) {
  const uint64_t per = (uint64_t)tile * 15 / 16 * n / std::max<uint64_t>(nkeys, 1);
  return (uint32_t)std::min<uint64_t>(most, std::max<uint64_t>(1, per));
}

void launch_gen_part(const u128* seq, const uint32_t* vcnt, uint64_t n, uint64_t nkeys,
                     int k, uint32_t idbits, const PartOut& o, hipStream_t s) {
  if (!n) return;
  if (nkeys < PART_BIG_KEYS) {
    // inputs of fewer tiles than CUs: a part of a tile for each CU (10K sequences,
    // k = 1, in 37 full tiles: 21 us; more and smaller parts than CUs queue for
    // the bins' cursors instead)
    const uint32_t most = (uint32_t)std::min<uint64_t>(256, std::max<uint64_t>(8, n / 256));
    gen_t<256, 4096>(seq, vcnt, (uint32_t)n, k, idbits, seqs_per_tile(n, nkeys, 4096, most), o, s);
  } else if (o.lb <= 11)  // two workgroups on a CU
    gen_t<512, 7680>(seq, vcnt, (uint32_t)n, k, idbits, seqs_per_tile(n, nkeys, 7680, 512), o, s);
  else
    gen_t<1024, 14336>(seq, vcnt, (uint32_t)n, k, idbits, seqs_per_tile(n, nkeys, 14336, 1024), o, s);
}

void launch_paired_distinct(const u128* pa, const u128* pb, uint64_t n, int k, uint32_t* vcnt,
                            unsigned long long* sums, hipStream_t s) {
  if (!n) return;
  hipLaunchKernelGGL(sdk::k_paired_distinct, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, pa,
                     pb, n, k, vcnt, sums);
}

template <int NT, int TILE>
static void gen_paired_t(const u128* sa, const u128* sb, const uint32_t* vcnt, uint32_t n, int k,
                         uint32_t idbits, uint32_t spb, const PartOut& o, hipStream_t s) {
  if (o.lb > tile_max_lb(NT)) throw Error{SD_E_HIP, "internal error: too many bins"};
  const size_t lds = (size_t)TILE * 8 + 96 * 8 + ((size_t)4 << o.lb) + (NT + 1) * 4 + NT / 64 * 4;
  allow_lds(&sdk::k_gen_part_paired<NT, TILE>, lds);
  hipLaunchKernelGGL((sdk::k_gen_part_paired<NT, TILE>), dim3((n + spb - 1) / spb), dim3(NT), lds,
                     s, sa, sb, vcnt, n, k, idbits, spb, o);
}

void launch_gen_part_paired(const u128* sa, const u128* sb, const uint32_t* vcnt, uint64_t n,
                            uint64_t nkeys, int k, uint32_t idbits, const PartOut& o,
                            hipStream_t s) {
  if (!n) return;
  if (k > 2) throw Error{SD_E_INVAL, "internal error: at most two deletions"};
  if (nkeys < PART_BIG_KEYS)
    gen_paired_t<256, 4096>(sa, sb, vcnt, (uint32_t)n, k, idbits, seqs_per_tile(n, nkeys, 4096, 256),
                            o, s);
  else if (o.lb <= 11)
    gen_paired_t<512, 7680>(sa, sb, vcnt, (uint32_t)n, k, idbits, seqs_per_tile(n, nkeys, 7680, 512),
                            o, s);
  else
    gen_paired_t<1024, 14336>(sa, sb, vcnt, (uint32_t)n, k, idbits,
                              seqs_per_tile(n, nkeys, 14336, 1024), o, s);
}

void launch_part_split(const PartOut& in, const PartOut& o, hipStream_t s) {
  constexpr int NT = 512, TILE = 8192;
  if (o.lb - in.lb > PART_MAX_SPLIT) throw Error{SD_E_HIP, "internal error: split too fine"};
  const size_t lds = (size_t)TILE * 8 + ((size_t)4 << (o.lb - in.lb)) + NT / 64 * 4;
  allow_lds(&sdk::k_part_split<NT, TILE>, lds);
  const uint32_t tiles = (in.region + TILE - 1) / TILE;
  hipLaunchKernelGGL((sdk::k_part_split<NT, TILE>), dim3(tiles * (in.nbins << in.nxl)), dim3(NT),
                     lds, s, in, o, tiles);
}

void launch_bin_offsets(const PartOut& in, uint32_t* cnt, uint64_t* off, uint64_t* status,
                        uint32_t* tile_counter, uint32_t epoch, uint32_t* err, hipStream_t s) {
  hipLaunchKernelGGL(sdk::k_bin_totals, dim3((in.nbins + 255) / 256), dim3(256), 0, s, in, cnt);
  launch_scan_excl(cnt, off, in.nbins, status, tile_counter, epoch, err, s);
}

void launch_sort_bins(const PartOut& in, const uint64_t* off, uint64_t* out, uint64_t* big,
                      unsigned long long* nbig, unsigned long long* repeats, hipStream_t s) {
  constexpr int NT = 512, CAP = 4032, BITS = 11, R = 9;
  const size_t lds = CAP * 8 + ((4 << BITS) + 4) + NT / 64 * 4;
  allow_lds(&sdk::k_sort_bins<NT, CAP, BITS, R>, lds);
  hipLaunchKernelGGL((sdk::k_sort_bins<NT, CAP, BITS, R>), dim3(in.nbins), dim3(NT), lds, s, in, off,
                     out, big, nbig, repeats);
}

void launch_place_bins(const uint64_t* X, uint64_t m, int lb, const uint64_t* off, uint64_t* out,
                       unsigned long long* repeats, hipStream_t s) {
  if (!m) return;
  hipLaunchKernelGGL(sdk::k_place_bins, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, X, m, lb,
                     off, out, repeats);
}

template <int NT, int SB, int LDS, bool WIDE>
static void filter_t(const PartOut& in, const PairBins& out, uint64_t* big,
                     unsigned long long* nbig, hipStream_t s) {
  allow_lds(&sdk::k_filter_group<NT, SB, LDS, WIDE>, LDS);
  hipLaunchKernelGGL((sdk::k_filter_group<NT, SB, LDS, WIDE>), dim3(in.nbins), dim3(NT), LDS, s, in,
                     with_limit(out), big, nbig);
}

template <bool WIDE>
static void filter_shape(bool small, const PartOut& in, const PairBins& out, uint64_t* big,
                         unsigned long long* nbig, hipStream_t s) {
  if (small)
    filter_t<256, 17, 20352, WIDE>(in, out, big, nbig, s);  // eight on a CU
  else
    filter_t<1024, 19, 81664, WIDE>(in, out, big, nbig, s);  // two
}

void launch_filter_group(const PartOut& in, uint64_t nkeys, uint32_t idbits, const PairBins& out,
                         uint64_t* big, unsigned long long* nbig, hipStream_t s) {
  // bins of up to 10K elements fill a small bitmap to a twelfth
  const bool small = nkeys >> in.lb <= 10240;
  if (idbits == 32)
    filter_shape<true>(small, in, out, big, nbig, s);
  else
    filter_shape<false>(small, in, out, big, nbig, s);
}

void launch_gen_probe(const u128* seq, uint64_t n, int k, const uint64_t* E, uint32_t nkeys,
                      const uint32_t* seg_start, const uint32_t* seg_end, int bits, uint32_t idbits,
                      const PairBins& out, const RunQueue& longs, hipStream_t s) {
  if (!n) return;
  const unsigned g = (unsigned)((n + 7) / 8);
  if (k == 3)
    hipLaunchKernelGGL((sdk::k_gen_probe<true>), dim3(g), dim3(256), 0, s, seq, (uint32_t)n, k, E, nkeys,
                       seg_start, seg_end, bits, idbits, out, longs);
  else
    hipLaunchKernelGGL((sdk::k_gen_probe<false>), dim3(g), dim3(256), 0, s, seq, (uint32_t)n, k, E, nkeys,
                       seg_start, seg_end, bits, idbits, out, longs);
}

void launch_join_bins(const PartOut& in, const uint64_t* E, const uint32_t* seg_start,
                      const uint32_t* seg_end, int bits, int sub, uint32_t idbits,
                      const PairBins& out, const JoinParts& copies, hipStream_t s) {
  if (in.lb + sub > bits) throw Error{SD_E_HIP, "internal error: join segments finer than the index"};
  auto launch = [&](auto kernel) {
    allow_lds(kernel, sdk::JB_LDS);
    hipLaunchKernelGGL(kernel, dim3(in.nbins << sub), dim3(1024), sdk::JB_LDS, s, in, E, seg_start,
                       seg_end, bits, sub, with_limit(out), copies);
  };
  if (idbits == 32)
    launch(&sdk::k_join_bins<1024, true>);
  else
    launch(&sdk::k_join_bins<1024, false>);
}

uint32_t join_parts(const PartOut& in, int sub) { return (in.nbins << sub) * sdk::JB_ROUNDS; }

void launch_join_runs(const PartOut& in, const uint64_t* E, const uint32_t* seg_start,
                      const uint32_t* seg_end, int bits, int sub, uint32_t idbits,
                      const JoinParts& copies, const RunQueue& queue, hipStream_t s) {
  hipLaunchKernelGGL(sdk::k_join_runs, dim3(256, (1u << in.nxl) + 1), dim3(256), 0, s, in, E,
                     seg_start, seg_end, bits, sub, idbits, copies, queue);
}

void launch_put_runs(const uint64_t* E, uint32_t idbits, const RunQueue& queue, uint64_t expect,
                     const PairBins& out, hipStream_t s) {
  // runs a workgroup: fewer of few runs, which may be long
  const uint32_t per = (uint32_t)std::min<uint64_t>(256, std::max<uint64_t>(8, expect / 2048));
  hipLaunchKernelGGL(sdk::k_put_runs, dim3(2048), dim3(256), 0, s, E, idbits, queue, per, out);
}

}  // namespace sd
