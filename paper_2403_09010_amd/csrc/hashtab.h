// The variant hash's constant words, shared by the generators (group.hip,
// partition.hip).
#pragma once
#include <stdint.h>

namespace sdk {

// 64-bit hash of a string y of length m: h(y) = C[m] xor the XOR over
// positions j of rotr(B[y_j], j), with B (per residue) and C (per length)
// fixed pseudo-random words. Rotation commutes with XOR, so a residue that
// moves one or two places left after a deletion changes its term by a left
// rotation of 1 or 2: with the prefix XORs P[i] of the undeleted string, the
// variant without positions p1 < p2 hashes to
//   C[m] ^ P[p1] ^ rotl(P[p2] ^ P[p1 + 1], 1) ^ rotl(P[L] ^ P[p2 + 1], 2),
// five LDS reads instead of rebuilding the 128-bit key. One deletion is the
// case p2 = L, none the case p1 = L, p2 = L + 1 (P is constant past L). Only
// the load balance and the rate of extra candidates depend on the hash.
struct HashTab {
  uint64_t b[32];  // per residue code (code 20 is the paired-chain join token)
  uint64_t c[64];  // per string length (paired-chain variants reach 49)
};

// splitmix64 (Steele, Lea and Flood, 2014) as a compile-time generator
constexpr uint64_t splitmix_next(uint64_t& state) {
  state += 0x9E3779B97F4A7C15ull;
  uint64_t z = state;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

constexpr HashTab make_hash_tab() {
  HashTab t{};
  uint64_t state = 0x5D3E1B7A2C4F9081ull;
  for (int x = 0; x < 32; ++x) t.b[x] = splitmix_next(state);
  for (int x = 0; x < 64; ++x) t.c[x] = splitmix_next(state);
  return t;
}

}  // namespace sdk
