// Which calls of a list of convolutions depend on one another.  Host code.
#pragma once

#include <stdint.h>

#include "emc2.h"

// What a call reads and writes, in bytes.
struct emc2_touched {
  uintptr_t lo[7], hi[7];   // [0]: the output; the input, weights, scale, shift, map and row count
};
// Row counts up to INT64_MAX are accepted ("no limit"): the input counts as far as the launch reads it, 2^31 - 1 rows, and a range ends
// at the last address at most, so that none wraps to nothing.
static inline emc2_touched emc2_touched_by(const emc2_conv_call& c) {
  const unsigned esz = c.dtype == EMC2_F32 ? 4 : 2;
  const uint64_t rows = c.n_in_rows > 0x7fffffff ? 0x7fffffff : (uint64_t)c.n_in_rows, cap = (uint64_t)c.capacity_out;
  const void* at[7] = {c.d_out, c.d_in, c.d_w, c.d_scale, c.d_shift, c.d_nbr, c.d_n_out};
  const uint64_t count[7] = {cap, rows, 27 * (uint64_t)c.cin, c.d_scale ? (uint64_t)c.cout : 0, c.d_shift ? (uint64_t)c.cout : 0, cap, 1};
  const unsigned size[7] = {c.cout * esz, c.cin * esz, c.cout * esz, 4, 4, 27 * 4, 4};
  emc2_touched t;
  for (int i = 0; i < 7; ++i) {
    t.lo[i] = (uintptr_t)at[i];
    const uint64_t room = UINTPTR_MAX - t.lo[i];
    t.hi[i] = count[i] > room / size[i] ? UINTPTR_MAX : t.lo[i] + count[i] * size[i];
  }
  return t;
}
// One writes what the other reads or writes: their order matters.
static inline bool emc2_ordered(const emc2_touched& a, const emc2_touched& b) {
  for (int i = 0; i < 7; ++i)
    if ((a.lo[0] < b.hi[i] && b.lo[i] < a.hi[0]) || (b.lo[0] < a.hi[i] && a.lo[i] < b.hi[0])) return true;
  return false;
}
