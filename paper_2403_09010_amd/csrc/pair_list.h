// Candidate lists: places are counted in 64 bits. A list can be sent more than 2^32
// candidates (tens of thousands of copies of one sequence), of which it keeps what
// its room holds; a count that wrapped would look like a list with room.
#pragma once
#include <stdint.h>

namespace sd {

// A list's counter has a cache line of its own: eight counters on one line took an
// atomic each 10 ns together, whichever XCD they came from.
constexpr uint32_t PAIR_LIST_STRIDE = 16;  // 64-bit words

// How many of n candidates reserved from place `at` on there is room for.
constexpr uint32_t list_room(uint64_t at, uint32_t n, uint32_t region) {
  return at >= region ? 0u : region - (uint32_t)at < n ? region - (uint32_t)at : n;
}

}  // namespace sd
