// Which tiles of consecutive rows an XCD takes, and in which order.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// Tiles of consecutive rows by XCD.  Workgroup b runs on XCD b % 8, and each XCD has its own L2, so neighbouring tiles, which gather
// largely the same rows, belong on one; but the neighbours a row has grow along the rows (z slowest: the ground's layers are dense,
// those far above and below it are not), and with an eighth of the rows each the XCD of the densest sets the time.  So the XCDs
// take runs of RUN consecutive tiles in turn, of 512 or 1024 rows: us, an eighth each / in runs: stride-2 64 -> 64 over 66 k rows
// 37 / 29.5, transposed over 223 k 44 / 38, 32 -> 32 over 304 k 66 / 59, stride-2 32 -> 64 over 223 k 40 / 35; runs of 256 to 2048 rows
// differ by 2 %.  (Not in k_spconv_span, whose tiles cost much the same and share planes: rounds of tiles dealt out, 60 / 65 over
// 248 k rows, 124 / 117 over 500 k; nor in k_spconv_i8, when it ran all 8-bit shapes: 111.1 / 111.7 a pass.)
// What is left of the tiles behind the last whole turn of eight runs goes to the XCDs by an eighth each, so that none has more than one
// tile above the least, and a level of less than a turn is on all of them: whole runs there left XCDs without a row and others with
// twice the rounds.  Capacity of the rows, us, an eighth each of all tiles / whole runs only / so: 32 -> 32 500 rows 5.3 / 12.3 / 5.3, 1 000
// 6.0 / 21.7 / 6.1, 12 000 9.0 / 13.7 / 9.1, 66 000 10.3 / 16.4 / 10.9; 16 -> 32 1 000 4.5 / 14.3 / 4.7; 64 -> 32 500 9.1 / 14.8 / 7.6.
template <int RUN> __host__ __device__ __forceinline__ int64_t emc2_xcd_tile(uint32_t xcd, int64_t slot, int64_t n_tiles) {   // the slot-th of the XCD's
  const uint32_t at = (uint32_t)slot, n = (uint32_t)n_tiles, left = n % (8 * RUN), whole = (n - left) / 8;   // row numbers are 32-bit
  return at < whole ? (at / RUN * 8 + xcd) * RUN + at % RUN : n - left + xcd * left / 8 + (at - whole);
}
template <int RUN> __host__ __device__ __forceinline__ int64_t emc2_xcd_tiles(uint32_t xcd, int64_t n_tiles) {   // how many it has
  const uint32_t n = (uint32_t)n_tiles, left = n % (8 * RUN);
  return (n - left) / 8 + (xcd + 1) * left / 8 - xcd * left / 8;
}
