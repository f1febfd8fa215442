// Which kernel, and in which form, a call goes to: rules on sizes and alignment alone (host-compilable: the CPU tests look at them).
#ifndef EJOIN_RULES_H
#define EJOIN_RULES_H

#include <stdint.h>

constexpr int64_t EJ_MEMORY_SIDE_CACHE = 256ll << 20;  // bytes of it

// Norms alone, from the last point on: where the rows have just been written, more of them than the memory-side cache holds, the last ones are
// still in it.  Rows of which all are there are read in the order in which they were written: the XCD that wrote a row still has it in its L2.
// Converted and normed, first to last and last to first, us: d = 16, rows of 100 MB 37.9 and 41.2, 128 46.8 and 50.0, 230 89.7 and 94.2, 250 102.0
// and 101.3, 275 128.1 and 116.2, 350 166.4 and 157.4, 500 230.3 and 229.5; d = 48, 128 MB 71.8 and 71.8, 250 132.7 and 132.2, 350 220.5 and
// 196.3, 500 310.3 and 295.5; d = 128, 650 MB 456 and 453, 950 MB 664 and 663; d = 16, 800 MB 357 and 360.  (A little of the cache is others'.)
inline bool norms_from_the_end(int64_t n, int64_t ld) {
  const int64_t bytes = n * ld * 2;
  return bytes > EJ_MEMORY_SIDE_CACHE / 16 * 15 && bytes <= EJ_MEMORY_SIDE_CACHE * 3;
}

#endif  // EJOIN_RULES_H
