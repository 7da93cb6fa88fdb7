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

// One output voxel o.  The three x-taps of a (z, y) row are adjacent bits of the input cell index,
// so a row costs one 8-byte load (two when the bits straddle a word): 9..18 loads per voxel instead of 27.
// S = stride (1 or 2).
template <int S>
__device__ __forceinline__ void emc2_probe_voxel(int64_t o, const int4* __restrict__ out_coords, int64_t capacity_out,
                                                 const cellword_t* __restrict__ in_idx, int32_t n_in, int gx, int gy, int gz,
                                                 int n_batch, int32_t* __restrict__ nbr) {
  int4 c = out_coords[o];  // (b, z, y, x)
  // malformed coordinate: emit an empty column (the per-tap range checks below keep every lookup in bounds)
  const bool sane = (unsigned)c.x < (unsigned)n_batch && (unsigned)c.y <= (1u << 20) && (unsigned)c.z <= (1u << 20) &&
                    (unsigned)c.w <= (1u << 20);
  if (!sane) c = make_int4(0, 0, 0, 0);
  const int bx = c.w * S - 1, by = c.z * S - 1, bz = c.y * S - 1;
  const int lo = bx < 0 ? 0 : bx;                    // x range of this voxel's taps inside the grid
  const int hi = bx + 2 >= gx ? gx - 1 : bx + 2;
#pragma unroll
  for (int kz = 0; kz < 3; ++kz) {
    const int iz = bz + kz;
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) {
      const int iy = by + ky;
      const bool row_ok = sane && (iz >= 0) && (iz < gz) && (iy >= 0) && (iy < gy) && (lo <= hi);
      const uint64_t row = (((uint64_t)c.x * gz + (uint64_t)(row_ok ? iz : 0)) * gy + (uint64_t)(row_ok ? iy : 0)) * gx;
      const uint64_t w_lo = (row + (uint64_t)lo) >> 5, w_hi = (row + (uint64_t)hi) >> 5;
      cellword_t cw0 = make_uint2(0u, 0u), cw1 = make_uint2(0u, 0u);
      if (row_ok) {
        cw0 = in_idx[w_lo];
        cw1 = (w_hi != w_lo) ? in_idx[w_hi] : cw0;
      }
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) {
        const int ix = bx + kx;
        int32_t j = -1;
        if (row_ok && ix >= lo && ix <= hi) {
          const uint64_t key = row + (uint64_t)ix;
          const cellword_t cw = ((key >> 5) == w_lo) ? cw0 : cw1;
          const uint32_t bit = (uint32_t)key & 31u;
          if ((cw.x >> bit) & 1u) j = (int32_t)(cw.y + __popc(cw.x & ((1u << bit) - 1u)));
        }
        if (j >= n_in) j = -1;  // only after a capacity overflow upstream
        // written once, read by a later kernel: a streaming store keeps the map from displacing the index in the caches
        __builtin_nontemporal_store(j, &nbr[(int64_t)((kz * 3 + ky) * 3 + kx) * capacity_out + o]);
      }
    }
  }
}
