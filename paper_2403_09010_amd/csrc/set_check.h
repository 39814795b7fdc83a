// Which sequences of a set on the device may be read.
#pragma once
#include <stdint.h>

namespace sd {

// Whether the `at`-th sequence of a set, its codes from a to b, lies in the set's
// codes, [0, end) with end the last offset. Where every sequence of a set does, its
// offsets start at 0 and never decrease; where they do not, at least one sequence
// does not, and the others can be read.
constexpr bool inside_set(uint64_t at, int64_t a, int64_t b, int64_t end) {
  return (at != 0 || a == 0) && a >= 0 && b >= a && b <= end;
}

}  // namespace sd
