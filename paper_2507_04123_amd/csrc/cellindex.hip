// Cell index (occupancy bits + prefix-summed ranks): clear, mark, scan.
// The scan is the prefix-sum index search of the paper's Sec. 3.6: after it, the voxel index of
// any active cell is found with one 8-byte load.
#include "common.h"

namespace {

// One block per tile; thread t owns the half line (8 words, 64 bytes) t of the tile.  Flagged lines are zeroed and
// their flags lowered; a tile without a flagged line costs one 128-byte read.
__global__ void __launch_bounds__(256) k_index_clear(uint4* __restrict__ p, lineflag_t* __restrict__ flags) {
  lineflag_t* tf = flags + (int64_t)blockIdx.x * EMC2_LINES_PER_TILE;
  const lineflag_t f = tf[threadIdx.x >> 1];
  if (f) {
    uint4* t = p + ((int64_t)blockIdx.x * EMC2_SCAN_TILE + (int64_t)threadIdx.x * 8) / 2;
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  if (!__syncthreads_or(f != 0)) return;  // every thread has read its flag
  if (f && !(threadIdx.x & 1)) tf[threadIdx.x >> 1] = 0;
}

__global__ void __launch_bounds__(256) k_index_mark_coords(cellword_t* __restrict__ idx,
                                                           const int4* __restrict__ coords,
                                                           const int32_t* __restrict__ d_n, int64_t capacity,
                                                           int gx, int gy, int gz, int n_batch,
                                                           lineflag_t* __restrict__ flags) {
  int64_t n = *d_n;
  if (n > capacity) n = capacity;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int4 c = coords[i];  // (b, z, y, x)
  if ((unsigned)c.x >= (unsigned)n_batch || (unsigned)c.y >= (unsigned)gz || (unsigned)c.z >= (unsigned)gy ||
      (unsigned)c.w >= (unsigned)gx)
    return;  // malformed coordinate: ignore rather than write out of bounds
  const uint64_t key = (((uint64_t)c.x * gz + (uint64_t)c.y) * gy + (uint64_t)c.z) * gx + (uint64_t)c.w;
  atomicOr(&idx[key >> 5].x, 1u << ((uint32_t)key & 31u));
  flags[emc2_line_of_key(key)] = 1;
}

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = __shfl_up(v, d, 64);
    if ((int)(threadIdx.x & 63) >= d) v += t;
  }
  return v;
}

// Per-block popcount totals.  Thread t owns the 8 consecutive words [8t, 8t+8) of its tile.
__global__ void __launch_bounds__(256) k_scan_reduce(const cellword_t* __restrict__ idx, int64_t n_words,
                                                     uint32_t* __restrict__ partials,
                                                     const lineflag_t* __restrict__ flags) {
  const bool mine = flags[(int64_t)blockIdx.x * EMC2_LINES_PER_TILE + (threadIdx.x >> 1)] != 0;
  if (!__syncthreads_or(mine)) {  // no bit in this tile
    if (threadIdx.x == 0) partials[blockIdx.x] = 0u;
    return;
  }
  const int64_t base = (int64_t)blockIdx.x * EMC2_SCAN_TILE + (int64_t)threadIdx.x * 8;
  uint32_t s = 0;
  if (mine) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (base + j < n_words) s += __popc(idx[base + j].x);
  }
  __shared__ uint32_t wsum[4];
  const uint32_t inc = wave_inclusive_scan(s);
  if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// Exclusive scan of the block totals, 1024 of them per block, out of place: a block first sums everything before its
// piece (coalesced, from L2; 88 000 totals are 0.35 MB), so pieces need not wait for each other.  One block walking over
// all of them took 91 us at 88 000 totals.  The last block reports the total (clamped).
__global__ void __launch_bounds__(1024) k_scan_partials(const uint32_t* __restrict__ totals, int64_t n, int64_t capacity,
                                                        uint32_t* __restrict__ bases, int32_t* __restrict__ d_total,
                                                        int32_t* __restrict__ d_flags) {
  __shared__ uint32_t wsum[16], wbefore[16];
  const int64_t start = (int64_t)blockIdx.x * 1024;
  uint32_t before = 0;
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < start; i += 1024) before += totals[i];
  const int64_t i = start + threadIdx.x;
  const uint32_t v = i < n ? totals[i] : 0u;
  const uint32_t inc = wave_inclusive_scan(v), binc = wave_inclusive_scan(before);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) { wsum[w] = inc; wbefore[w] = binc; }
  __syncthreads();
  uint32_t run = inc - v;
  for (int j = 0; j < 16; ++j) run += wbefore[j] + (j < w ? wsum[j] : 0u);
  if (i < n) bases[i] = run;
  if (i == n - 1) {
    const uint32_t total = run + v;
    if ((int64_t)total > capacity) {
      atomicOr(d_flags, EMC2_DEVFLAG_CAPACITY);
      *d_total = (int32_t)capacity;
    } else {
      *d_total = (int32_t)total;
    }
  }
}

// Write each word's exclusive prefix (.y).
__global__ void __launch_bounds__(256) k_scan_apply(cellword_t* __restrict__ idx, int64_t n_words,
                                                    const uint32_t* __restrict__ partials,
                                                    const lineflag_t* __restrict__ flags) {
  const bool mine = flags[(int64_t)blockIdx.x * EMC2_LINES_PER_TILE + (threadIdx.x >> 1)] != 0;
  if (!__syncthreads_or(mine)) return;  // no bit, so no prefix field anybody reads
  const int64_t base = (int64_t)blockIdx.x * EMC2_SCAN_TILE + (int64_t)threadIdx.x * 8;
  uint32_t bits[8];
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    bits[j] = (mine && base + j < n_words) ? idx[base + j].x : 0u;
    s += __popc(bits[j]);
  }
  __shared__ uint32_t wsum[4];
  const uint32_t inc = wave_inclusive_scan(s);
  if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
  __syncthreads();
  uint32_t run = partials[blockIdx.x] + inc - s;
  const int w = threadIdx.x >> 6;
  for (int j = 0; j < w; ++j) run += wsum[j];
  if (mine) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (base + j < n_words) idx[base + j] = make_uint2(bits[j], run);
      run += __popc(bits[j]);
    }
  }
}

// Whole scan in one block (small grids: the coarse levels): thread t owns a contiguous run of words.
__global__ void __launch_bounds__(1024) k_scan_small(cellword_t* __restrict__ idx, int64_t n_words, int64_t capacity,
                                                     int32_t* __restrict__ d_total, int32_t* __restrict__ d_flags) {
  const int per = (int)((n_words + 1023) / 1024);
  const int64_t base = (int64_t)threadIdx.x * per;
  uint32_t s = 0;
  for (int j = 0; j < per; ++j)
    if (base + j < n_words) s += __popc(idx[base + j].x);
  __shared__ uint32_t wsum[16];
  const uint32_t inc = wave_inclusive_scan(s);
  if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
  __syncthreads();
  uint32_t run = inc - s;
  const int w = threadIdx.x >> 6;
  for (int j = 0; j < w; ++j) run += wsum[j];
  for (int j = 0; j < per; ++j)
    if (base + j < n_words) {
      const uint32_t bits = idx[base + j].x;
      idx[base + j] = make_uint2(bits, run);
      run += __popc(bits);
    }
  if (threadIdx.x == 1023) {
    if ((int64_t)run > capacity) {
      atomicOr(d_flags, EMC2_DEVFLAG_CAPACITY);
      *d_total = (int32_t)capacity;
    } else {
      *d_total = (int32_t)run;
    }
  }
}

// Apply step that derives its own base from the block totals (no separate scan of the totals): block b
// sums totals[0..b) cooperatively.  Quadratic in the number of blocks, so only used while that is moderate.
__global__ void __launch_bounds__(256) k_scan_apply_self(cellword_t* __restrict__ idx, int64_t n_words,
                                                         const uint32_t* __restrict__ totals, int64_t capacity,
                                                         int32_t* __restrict__ d_total, int32_t* __restrict__ d_flags,
                                                         const lineflag_t* __restrict__ flags) {
  // a line without bits has no prefix field anybody reads; the last block still reports the total
  const bool has_bits = flags[(int64_t)blockIdx.x * EMC2_LINES_PER_TILE + (threadIdx.x >> 1)] != 0;   // this thread's line
  if (!__syncthreads_or(has_bits) && blockIdx.x != gridDim.x - 1) return;
  __shared__ uint32_t wsum[4];
  __shared__ uint32_t base_s;
  uint32_t part = 0;
  for (int i = threadIdx.x; i < (int)blockIdx.x; i += 256) part += totals[i];
  {
    const uint32_t inc = wave_inclusive_scan(part);
    if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
    __syncthreads();
    if (threadIdx.x == 0) base_s = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
  }
  const int64_t base = (int64_t)blockIdx.x * EMC2_SCAN_TILE + (int64_t)threadIdx.x * 8;
  uint32_t bits[8];
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    bits[j] = (has_bits && base + j < n_words) ? idx[base + j].x : 0u;
    s += __popc(bits[j]);
  }
  const uint32_t inc = wave_inclusive_scan(s);
  __syncthreads();
  if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
  __syncthreads();
  uint32_t run = base_s + inc - s;
  const int w = threadIdx.x >> 6;
  for (int j = 0; j < w; ++j) run += wsum[j];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (has_bits && base + j < n_words) idx[base + j] = make_uint2(bits[j], run);
    run += __popc(bits[j]);
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 255) {
    if ((int64_t)run > capacity) {
      atomicOr(d_flags, EMC2_DEVFLAG_CAPACITY);
      *d_total = (int32_t)capacity;
    } else {
      *d_total = (int32_t)run;
    }
  }
}

// ---- the index from the marks -------------------------------------------------------------------------------------------------------

__global__ void __launch_bounds__(256) k_marks_zero(uint4* __restrict__ p, int64_t n16) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (int64_t)gridDim.x * 256) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// A thread's 8 words of marks (half a line).
struct Marks8 { uint32_t v[8]; };
__device__ __forceinline__ Marks8 load_marks(const uint32_t* __restrict__ marks, int64_t base, bool some) {
  Marks8 m;
  const uint4* p = reinterpret_cast<const uint4*>(marks + base);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint4 v = some ? p[h] : make_uint4(0u, 0u, 0u, 0u);
    m.v[4 * h] = v.x; m.v[4 * h + 1] = v.y; m.v[4 * h + 2] = v.z; m.v[4 * h + 3] = v.w;
  }
  return m;
}
__device__ __forceinline__ uint32_t count_marks(const Marks8& m) {
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) s += __popc(m.v[j]);
  return s;
}

// Eight words of the index: bits and ranks from `run` on, or zeros where the slot holds stale ones; the marks go back to zero.  The flags
// of the line are the even thread's; every thread has read them by now.
__device__ __forceinline__ void take_marks(cellword_t* __restrict__ idx, lineflag_t* __restrict__ flags, uint32_t* __restrict__ marks,
                                           lineflag_t* __restrict__ mark_flags, int64_t base, const Marks8& m, bool some, bool stale,
                                           uint32_t& run) {
  if (some || stale) {
    uint4* p = reinterpret_cast<uint4*>(idx + base);
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      const uint32_t r1 = run + __popc(m.v[j]);
      p[j / 2] = some ? make_uint4(m.v[j], run, m.v[j + 1], r1) : make_uint4(0u, 0u, 0u, 0u);
      run = r1 + __popc(m.v[j + 1]);
    }
  }
  if (some) {
    uint4* z = reinterpret_cast<uint4*>(marks + base);
    z[0] = make_uint4(0u, 0u, 0u, 0u);
    z[1] = make_uint4(0u, 0u, 0u, 0u);
  }
  if (!(threadIdx.x & 1)) {
    if (some != stale) flags[base >> EMC2_LINE_SHIFT] = some ? 1 : 0;
    if (some) mark_flags[base >> EMC2_LINE_SHIFT] = 0;
  }
}

// Popcounts by tile.  Thread t owns the 8 words [8t, 8t+8) of its tile, here and below.
__global__ void __launch_bounds__(256) k_marks_reduce(const uint32_t* __restrict__ marks, const lineflag_t* __restrict__ mark_flags,
                                                      uint32_t* __restrict__ partials) {
  const int64_t base = (int64_t)blockIdx.x * EMC2_SCAN_TILE + (int64_t)threadIdx.x * 8;
  const bool some = mark_flags[base >> EMC2_LINE_SHIFT] != 0;
  if (!__syncthreads_or(some)) {  // no bit in this tile
    if (threadIdx.x == 0) partials[blockIdx.x] = 0u;
    return;
  }
  __shared__ uint32_t wsum[4];
  const uint32_t inc = wave_inclusive_scan(count_marks(load_marks(marks, base, some)));
  if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// SELF: `sums` are the tiles' popcounts, and a block adds up those before its own; the last block reports the total.  Else they are their
// prefix sums.
template <bool SELF>
__global__ void __launch_bounds__(256) k_marks_apply(cellword_t* __restrict__ idx, lineflag_t* __restrict__ flags,
                                                     uint32_t* __restrict__ marks, lineflag_t* __restrict__ mark_flags,
                                                     const uint32_t* __restrict__ sums, int64_t capacity, int32_t* __restrict__ d_total,
                                                     int32_t* __restrict__ d_flags) {
  const int64_t base = (int64_t)blockIdx.x * EMC2_SCAN_TILE + (int64_t)threadIdx.x * 8;
  const bool some = mark_flags[base >> EMC2_LINE_SHIFT] != 0, stale = flags[base >> EMC2_LINE_SHIFT] != 0;
  const bool last = SELF && blockIdx.x == gridDim.x - 1;
  if (!__syncthreads_or(some || stale) && !last) return;
  const Marks8 m = load_marks(marks, base, some);
  const uint32_t s = count_marks(m);
  __shared__ uint32_t wsum[4], wbase[4];
  uint32_t part = 0;
  if constexpr (SELF)
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += 256) part += sums[i];
  const uint32_t inc = wave_inclusive_scan(s), binc = SELF ? wave_inclusive_scan(part) : 0u;
  if ((threadIdx.x & 63) == 63) {
    wsum[threadIdx.x >> 6] = inc;
    wbase[threadIdx.x >> 6] = binc;
  }
  __syncthreads();
  uint32_t run = SELF ? inc - s + wbase[0] + wbase[1] + wbase[2] + wbase[3] : sums[blockIdx.x] + inc - s;
  for (int j = 0; j < (int)(threadIdx.x >> 6); ++j) run += wsum[j];
  const uint32_t end = run + s;
  take_marks(idx, flags, marks, mark_flags, base, m, some, stale, run);
  if (last && threadIdx.x == 255) {
    if ((int64_t)end > capacity) atomicOr(d_flags, EMC2_DEVFLAG_CAPACITY);
    *d_total = (int64_t)end > capacity ? (int32_t)capacity : (int32_t)end;
  }
}

// The whole of a small grid (at most 8192 words) in one block, 8 words a thread.  A line is taken or left whole, beyond the grid's last word
// too: the flag that take_marks lowers speaks for both its halves, and what an index of a larger grid left in the second would be found
// by the next one.  (Slots are whole tiles.)
__global__ void __launch_bounds__(1024) k_marks_small(cellword_t* __restrict__ idx, lineflag_t* __restrict__ flags,
                                                      uint32_t* __restrict__ marks, lineflag_t* __restrict__ mark_flags, int64_t n_words,
                                                      int64_t capacity, int32_t* __restrict__ d_total, int32_t* __restrict__ d_flags) {
  const int64_t base = (int64_t)threadIdx.x * 8;
  const bool mine = (base >> EMC2_LINE_SHIFT << EMC2_LINE_SHIFT) < n_words;
  const bool some = mine && mark_flags[base >> EMC2_LINE_SHIFT] != 0, stale = mine && flags[base >> EMC2_LINE_SHIFT] != 0;
  const Marks8 m = load_marks(marks, base, some);
  const uint32_t s = count_marks(m);
  __shared__ uint32_t wsum[16];
  const uint32_t inc = wave_inclusive_scan(s);
  if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
  __syncthreads();
  uint32_t run = inc - s;
  for (int j = 0; j < (int)(threadIdx.x >> 6); ++j) run += wsum[j];
  const uint32_t end = run + s;
  take_marks(idx, flags, marks, mark_flags, base, m, some, stale, run);
  if (threadIdx.x == 1023) {
    if ((int64_t)end > capacity) atomicOr(d_flags, EMC2_DEVFLAG_CAPACITY);
    *d_total = (int64_t)end > capacity ? (int32_t)capacity : (int32_t)end;
  }
}

}  // namespace

static void zero_marks(emc2_ctx* ctx, hipStream_t stream) {
  const int64_t bytes = 4 * ctx->slot_words + (ctx->slot_words >> EMC2_LINE_SHIFT);      // slots are whole tiles: a multiple of 128
  hipLaunchKernelGGL(k_marks_zero, dim3(2048), dim3(256), 0, stream, (uint4*)ctx->marks, bytes / 16);
}

void emc2_marks_begin(emc2_ctx* ctx, hipStream_t stream) {
  ctx->marks_recorded = !ctx->marks_zeroed && emc2_capturing(stream);
  if (!ctx->marks_zeroed) zero_marks(ctx, stream);
  ctx->marks_zeroed = false;
}

// The launches that set the marks and took them over are issued.  If one failed, the next call clears them, and, for graphs that were
// recorded while they were zero, this one as well, if it still can.
static void marks_taken(emc2_ctx* ctx, hipStream_t stream) {
  const bool ok = hipPeekAtLastError() == hipSuccess;
  if (!ok) zero_marks(ctx, stream);
  ctx->marks_zeroed = ok && !ctx->marks_recorded;
}

void emc2_index_build(emc2_ctx* ctx, cellword_t* idx, int64_t n_cells, int64_t capacity, int32_t* d_total, hipStream_t stream) {
  const int64_t n_words = emc2_div_up(n_cells, 32), n_blocks = emc2_div_up(n_words, EMC2_SCAN_TILE);
  lineflag_t *flags = emc2_slot_flags(ctx, idx), *mark_flags = emc2_mark_flags(ctx);
  if (n_words <= 8 * 1024) {
    hipLaunchKernelGGL(k_marks_small, dim3(1), dim3(1024), 0, stream, idx, flags, ctx->marks, mark_flags, n_words, capacity, d_total,
                       ctx->dev_words);
  } else {
    hipLaunchKernelGGL(k_marks_reduce, dim3((unsigned)n_blocks), dim3(256), 0, stream, ctx->marks, mark_flags, ctx->partials);
    if (n_blocks <= EMC2_SCAN_SELF_TILES) {   // each apply block re-sums the earlier totals itself: at most 64 KB from L2
      hipLaunchKernelGGL(k_marks_apply<true>, dim3((unsigned)n_blocks), dim3(256), 0, stream, idx, flags, ctx->marks, mark_flags,
                         ctx->partials, capacity, d_total, ctx->dev_words);
    } else {
      uint32_t* bases = ctx->partials + ctx->n_partials;
      emc2_scan_totals(ctx, ctx->partials, n_blocks, capacity, bases, d_total, stream);
      hipLaunchKernelGGL(k_marks_apply<false>, dim3((unsigned)n_blocks), dim3(256), 0, stream, idx, flags, ctx->marks, mark_flags, bases,
                         capacity, d_total, ctx->dev_words);
    }
  }
  marks_taken(ctx, stream);
}

void emc2_index_clear(emc2_ctx* ctx, cellword_t* idx, hipStream_t stream) {
  hipLaunchKernelGGL(k_index_clear, dim3((unsigned)ctx->slot_tiles), dim3(256), 0, stream, (uint4*)idx,
                     emc2_slot_flags(ctx, idx));
}

void emc2_index_mark_coords(emc2_ctx* ctx, cellword_t* idx, const int32_t* d_coords, const int32_t* d_n,
                            int64_t capacity, const int32_t grid[3], int32_t n_batch, hipStream_t stream) {
  if (capacity < 1) return;
  hipLaunchKernelGGL(k_index_mark_coords, dim3((unsigned)emc2_div_up(capacity, 256)), dim3(256), 0, stream, idx,
                     (const int4*)d_coords, d_n, capacity, grid[0], grid[1], grid[2], n_batch, emc2_slot_flags(ctx, idx));
}

void emc2_scan_totals(emc2_ctx* ctx, const uint32_t* totals, int64_t n, int64_t capacity, uint32_t* bases, int32_t* d_total,
                      hipStream_t stream) {
  hipLaunchKernelGGL(k_scan_partials, dim3((unsigned)emc2_div_up(n, 1024)), dim3(1024), 0, stream, totals, n, capacity, bases, d_total,
                     ctx->dev_words);
}

void emc2_index_scan(emc2_ctx* ctx, cellword_t* idx, int64_t n_cells, int64_t capacity, int32_t* d_total,
                     hipStream_t stream) {
  const int64_t n_words = emc2_div_up(n_cells, 32);
  const int64_t n_blocks = emc2_div_up(n_words, EMC2_SCAN_TILE);
  if (n_words <= 8 * 1024) {
    // coarse levels: one block does it all (one launch instead of three)
    hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(1024), 0, stream, idx, n_words, capacity, d_total, ctx->dev_words);
    return;
  }
  hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)n_blocks), dim3(256), 0, stream, idx, n_words, ctx->partials,
                     emc2_slot_flags(ctx, idx));
  if (n_blocks <= EMC2_SCAN_SELF_TILES) {   // each apply block re-sums the earlier totals itself: at most 64 KB from L2
    hipLaunchKernelGGL(k_scan_apply_self, dim3((unsigned)n_blocks), dim3(256), 0, stream, idx, n_words, ctx->partials,
                       capacity, d_total, ctx->dev_words, emc2_slot_flags(ctx, idx));
    return;
  }
  uint32_t* bases = ctx->partials + ctx->n_partials;
  emc2_scan_totals(ctx, ctx->partials, n_blocks, capacity, bases, d_total, stream);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)n_blocks), dim3(256), 0, stream, idx, n_words, bases,
                     emc2_slot_flags(ctx, idx));
}
