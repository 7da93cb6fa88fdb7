// The 27 kernel-map entries of one output voxel, and the bit arithmetic of a stride-2 level's occupancy: shared by the
// kernel-map calls and the whole-stack builder.
#pragma once

#include "common.h"

// Keep the even-numbered bits of v (bit 2i -> bit i).
__device__ __forceinline__ uint32_t emc2_even_bits(uint64_t v) {
  v &= 0x5555555555555555ull;
  v = (v | (v >> 1)) & 0x3333333333333333ull;
  v = (v | (v >> 2)) & 0x0f0f0f0f0f0f0f0full;
  v = (v | (v >> 4)) & 0x00ff00ff00ff00ffull;
  v = (v | (v >> 8)) & 0x0000ffff0000ffffull;
  v = (v | (v >> 16)) & 0x00000000ffffffffull;
  return (uint32_t)v;
}

// Entries of one output voxel o.  The three x-taps of a (z, y) row are adjacent bits of the input cell index, so a row costs one 8-byte load
// (two when the bits straddle a word): 9..18 loads per voxel instead of 27.  S = stride (1 or 2).
// All loads are requested before the first entry is stored, without a branch around any.  The taps' ranks follow from one population
// count a row, and keys and addresses from one key a voxel and steps that are the same for the whole launch.  With a key, a word and
// a rank for each tap the vector units had as much to do as the memory: submanifold map of 7.5 M voxels 352 -> 288 us (932 MB that have
// to move, 3.2 TB/s), the eight maps of eight routed frames 174 -> 147, those of a 64-beam frame 36.7 -> 33.2.
// c: (b, z, y, x), sane: a cell that may be looked up; word(w): word w of the input's index.
template <int S, typename Word>
__device__ __forceinline__ void emc2_probe_at(int64_t o, const int4& c, bool sane, int64_t capacity_out, Word word, int32_t n_in, int gx,
                                              int gy, int gz, int32_t* __restrict__ nbr) {
  const int bx = c.w * S - 1, by = c.z * S - 1, bz = c.y * S - 1;
  const int lo = bx < 0 ? 0 : bx;                    // x range of this voxel's taps inside the grid
  const int hi = bx + 2 >= gx ? gx - 1 : bx + 2;
  const bool x_ok = sane && lo <= hi;
  const uint32_t skip = (uint32_t)(lo - bx), last = (uint32_t)(hi - lo);    // taps before the first inside, from it to the last inside
  const uint32_t inside = x_ok ? (2u << (hi - bx)) - (1u << skip) : 0u;     // taps inside, a bit each
  const int64_t plane = (int64_t)gy * gx;
  const int64_t key0 = (((int64_t)c.x * gz + bz) * gy + by) * gx + lo;      // of row 0's first tap inside
  cellword_t w0[9], w1[9];
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    const bool ok = x_ok && (unsigned)(bz + r / 3) < (unsigned)gz && (unsigned)(by + r % 3) < (unsigned)gy;
    const uint64_t key = (uint64_t)(key0 + (r / 3) * plane + (r % 3) * gx);
    const uint64_t w = ok ? key >> 5 : 0;
    w0[r] = word(w);
    w1[r] = word(w + (ok && ((uint32_t)key & 31u) + last > 31u ? 1 : 0));
    if (!ok) w0[r] = w1[r] = make_uint2(0u, 0u);
  }
  // (the compiler would otherwise request a row's words where they are used, behind the stores of the row before)
#pragma unroll
  for (int r = 0; r < 9; ++r) asm volatile("" : "+v"(w0[r].x), "+v"(w0[r].y), "+v"(w1[r].x), "+v"(w1[r].y));
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    const uint32_t sh = (uint32_t)(key0 + (r / 3) * plane + (r % 3) * gx) & 31u;
    const uint32_t bits = (__funnelshift_r(w0[r].x, w1[r].x, sh) << skip) & inside;
    const uint32_t b0 = bits & 1u, b1 = (bits >> 1) & 1u;
    const uint32_t at = w0[r].y + __popc(w0[r].x & ((1u << sh) - 1u));      // rank of the first tap inside
    const uint32_t pos = sh - skip;                                        // of tap 0 in the first word; taps at 32 and 33 are the second word's
    uint32_t rank[3];
    rank[0] = at;
    rank[1] = (int32_t)pos < 31 ? at + b0 : w1[r].y;
    rank[2] = (int32_t)pos < 30 ? at + b0 + b1 : w1[r].y + (pos == 31u ? b1 : 0u);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      // (a rank at or beyond n_in: only after a capacity overflow upstream)
      const int32_t j = ((bits >> t) & 1u) && (int32_t)rank[t] < n_in ? (int32_t)rank[t] : -1;
      // written once, read by a later kernel: a streaming store keeps the map from displacing the index in the caches
      __builtin_nontemporal_store(j, &nbr[(int64_t)(3 * r + t) * capacity_out + o]);
    }
  }
}

// The same by output row: its coordinates and the input's index in memory.
template <int S>
__device__ __forceinline__ void emc2_probe_voxel(int64_t o, const int4* __restrict__ out_coords, int64_t capacity_out,
                                                 const cellword_t* __restrict__ in_idx, int32_t n_in, int gx, int gy, int gz,
                                                 int n_batch, int32_t* __restrict__ nbr) {
  int4 c = out_coords[o];  // (b, z, y, x)
  // malformed coordinate: emit an empty column (the range checks keep every lookup in bounds)
  const bool sane = (unsigned)c.x < (unsigned)n_batch && (unsigned)c.y <= (1u << 20) && (unsigned)c.z <= (1u << 20) &&
                    (unsigned)c.w <= (1u << 20);
  if (!sane) c = make_int4(0, 0, 0, 0);
  emc2_probe_at<S>(o, c, sane, capacity_out, [in_idx](uint64_t w) { return in_idx[w]; }, n_in, gx, gy, gz, nbr);
}
