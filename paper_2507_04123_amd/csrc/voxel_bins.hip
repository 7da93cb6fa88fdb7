// Voxelization of large clouds by bin of cells (paper Sec. 2 / Sec. 3.1 voxelization; Sec. 3.6 (3) prefix-sum index search).
//
// The pass over single points (voxelize.hip) is bound by the memory side of the fabric: one atomic a point (27 G/s on this part,
// whatever the address, the scope or the XCD that asks), then an 8-byte load (55 G/s at random places of an index of gigabytes, 200
// where a block stays inside 256 KB) and a 16-byte store (30 and 190).  Here the points are first moved next to the others of their
// bin of consecutive cells, and a block then owns a bin: its bits, ranks, counts and the order of its points live in LDS, every line
// of the index is written once, and the only atomics that leave a CU are one per bin and 8 192 points.
//
//   k_bin_points     points per bin
//   k_bin_starts     exclusive scan of them; the bins that have any
//   k_bin_points     the points again, each to its place: (x, y, z, intensity) and the cell inside the bin
//   k_bin_distinct   voxels per bin
//   k_scan_partials  exclusive scan of those (cellindex.hip): the rank of a bin's first voxel, the number of voxels
//   k_bin_voxels     a block a bin: index lines and flags, stale lines of the slot cleared, coordinates, counts, means
//
// Bound by memory and by the chain of a block's phases in LDS: 64 frames of 120 000 points (7.5 M voxels, of 5.8 G cells), us: count 36,
// move 121 (154 MB read, 264 written), voxels of the bins 34, scans 30, the bins 265 (690 MB); 1 081 -> 491 in all.  The point pass
// there: clear 81, mark 295, scan 261, second pass 367, means 77.
#include "voxel_point.h"

namespace {

constexpr int kMoveThreads = 1024, kMovePoints = 8;     // points a thread
constexpr int kWindow = 8192;                           // bins a block counts at a time
constexpr int kSmallPoints = 12;                        // points a thread of a small bin's block
constexpr uint32_t kSmallBin = 256 * kSmallPoints;      // points of a bin that one block takes
constexpr uint32_t kItemVoxels = 128;                   // voxels of a larger bin that one block takes
constexpr int kItemBlocks = 1024, kLargeBlocks = 512;

// words (of 32 cells) and lines (of 16 words) of a bin
template <int SHIFT> constexpr int kWords = 1 << (SHIFT - 5);
template <int SHIFT> constexpr int kLines = kWords<SHIFT> >> EMC2_LINE_SHIFT;

struct BinState { uint32_t small, large, items, unused; };   // bins of up to kSmallBin points, of more, blocks' shares of the latter

__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {   // inclusive
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = __shfl_up(v, d, 64);
    if ((int)(threadIdx.x & 63) >= d) v += t;
  }
  return v;
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d, 64);
  return v;
}

__global__ void __launch_bounds__(1024) k_bin_zero(uint32_t* __restrict__ counts, int64_t n, BinState* __restrict__ state) {
  const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  if (i < n) counts[i] = 0u;
  if (i == 0) *state = BinState{0u, 0u, 0u, 0u};
}

// The bins that a block's kept points lie in, lowest and highest (hi < 0: none kept).  Frames come one after the other, so these
// are a frame's or two; a window of them is counted in LDS at a time, and points of all frames mixed take more windows.
struct Range { int32_t lo, hi; };
__device__ __forceinline__ Range block_range(const int32_t (&bin)[kMovePoints]) {
  __shared__ int32_t lo_s, hi_s;
  if (threadIdx.x == 0) { lo_s = 0x7fffffff; hi_s = -1; }
  __syncthreads();
  int32_t lo = 0x7fffffff, hi = -1;
#pragma unroll
  for (int j = 0; j < kMovePoints; ++j)
    if (bin[j] >= 0) { lo = min(lo, bin[j]); hi = max(hi, bin[j]); }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    lo = min(lo, __shfl_xor(lo, d, 64));
    hi = max(hi, __shfl_xor(hi, d, 64));
  }
  if ((threadIdx.x & 63) == 0 && hi >= 0) { atomicMin(&lo_s, lo); atomicMax(&hi_s, hi); }
  __syncthreads();
  return Range{lo_s, hi_s};
}

// Counts (MOVE: and places) a block's points.  moved, cells: point and cell inside the bin, at the point's place.
template <int SHIFT, bool MOVE>
__global__ void __launch_bounds__(kMoveThreads) k_bin_points(const float* __restrict__ points, const int32_t* __restrict__ batch,
                                                             int64_t n_points, VoxParams prm, uint32_t* __restrict__ counts,
                                                             float4* __restrict__ moved, uint16_t* __restrict__ cells) {
  __shared__ uint32_t win[kWindow];
  const int64_t base = (int64_t)blockIdx.x * (kMoveThreads * kMovePoints) + threadIdx.x;
  int32_t bin[kMovePoints];
  uint32_t cell[kMovePoints], pos[kMovePoints];
  float4 p[kMovePoints];
#pragma unroll
  for (int j = 0; j < kMovePoints; ++j) {
    const PointCell pc = locate(points, batch, base + j * kMoveThreads, n_points, prm);
    bin[j] = pc.keep ? (int32_t)(pc.key >> SHIFT) : -1;
    cell[j] = (uint32_t)pc.key & ((1u << SHIFT) - 1u);
    p[j] = pc.p;
  }
  const Range r = block_range(bin);
  for (int32_t lo = r.lo; lo <= r.hi; lo += kWindow) {   // the same for the whole block
    const int32_t n = min(r.hi - lo + 1, kWindow);
    for (int32_t i = threadIdx.x; i < n; i += kMoveThreads) win[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kMovePoints; ++j)
      if (bin[j] >= lo && bin[j] - lo < n) pos[j] = atomicAdd(&win[bin[j] - lo], 1u);
    __syncthreads();
    for (int32_t i = threadIdx.x; i < n; i += kMoveThreads)
      if (win[i]) {
        const uint32_t at = atomicAdd(&counts[lo + i], win[i]);
        if (MOVE) win[i] = at;
      }
    __syncthreads();
    if (MOVE) {
#pragma unroll
      for (int j = 0; j < kMovePoints; ++j)
        if (bin[j] >= lo && bin[j] - lo < n) {
          const uint32_t to = win[bin[j] - lo] + pos[j];
          moved[to] = p[j];
          cells[to] = (uint16_t)cell[j];
        }
      __syncthreads();
    }
  }
}

// starts[i] = points before bin i (starts[n] = all), cursors the same; no voxels yet.  list: the bins of up to kSmallBin points from
// the front, those of more from the back, in any order: two bins of three of a frame have no point, and a block that finds that out
// takes 2 us.
__global__ void __launch_bounds__(1024) k_bin_starts(const uint32_t* __restrict__ counts, int64_t n, uint32_t* __restrict__ starts,
                                                     uint32_t* __restrict__ cursors, uint32_t* __restrict__ voxels,
                                                     uint32_t* __restrict__ list, BinState* __restrict__ state) {
  __shared__ uint32_t wsum[16], wbefore[16], wsmall[16], small_s;
  const int64_t first = (int64_t)blockIdx.x * 1024;
  uint32_t before = 0;
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < first; i += 1024) before += counts[i];
  const int64_t i = first + threadIdx.x;
  const uint32_t v = i < n ? counts[i] : 0u;
  const uint32_t inc = wave_scan(v);
  before = wave_sum(before);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool small = v > 0u && v <= kSmallBin;
  const unsigned long long smalls = __ballot(small);
  if (lane == 63) { wsum[w] = inc; wbefore[w] = before; wsmall[w] = (uint32_t)__popcll(smalls); }
  if (v > kSmallBin) list[n - 1 - atomicAdd(&state->large, 1u)] = (uint32_t)i;
  __syncthreads();
  uint32_t run = inc - v, at = (uint32_t)__popcll(smalls & ((1ull << lane) - 1ull)), all = 0;
  for (int j = 0; j < 16; ++j) {
    run += wbefore[j] + (j < w ? wsum[j] : 0u);
    at += j < w ? wsmall[j] : 0u;
    all += wsmall[j];
  }
  if (threadIdx.x == 0) small_s = all ? atomicAdd(&state->small, all) : 0u;
  __syncthreads();
  if (small) list[small_s + at] = (uint32_t)i;
  if (i < n) { starts[i] = run; cursors[i] = run; voxels[i] = 0u; }
  if (i == n - 1) starts[n] = run + v;
}

// Voxels of the bins with points: a wave a small bin; kLargeBlocks blocks share the larger ones and divide their voxels into items.
template <int SHIFT>
__global__ void __launch_bounds__(256) k_bin_distinct(BinState* __restrict__ state, const uint32_t* __restrict__ list,
                                                      const uint32_t* __restrict__ starts, int64_t n_bins,
                                                      const uint16_t* __restrict__ cells, uint32_t* __restrict__ voxels,
                                                      uint32_t* __restrict__ items) {
  __shared__ uint4 bits_s[4][kWords<SHIFT> / 4];
  __shared__ uint32_t fresh_s, at_s;                     // a larger bin's voxels; where its items begin (waves may still read the first)
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t fresh = 0;
  if (blockIdx.x < kLargeBlocks) {
    uint32_t* bits = reinterpret_cast<uint32_t*>(bits_s[0]);
    for (uint32_t k = blockIdx.x; k < state->large; k += kLargeBlocks) {
      const uint32_t bin = list[n_bins - 1 - k], begin = starts[bin], end = starts[bin + 1];
      for (int i = threadIdx.x; i < kWords<SHIFT>; i += 256) bits[i] = 0u;
      if (threadIdx.x == 0) fresh_s = 0u;
      __syncthreads();
      fresh = 0;
#pragma unroll 8
      for (uint32_t i = begin + threadIdx.x; i < end; i += 256) {
        const uint32_t c = cells[i], bit = 1u << (c & 31);
        fresh += (atomicOr(&bits[c >> 5], bit) & bit) == 0u;
      }
      fresh = wave_sum(fresh);
      if (lane == 0) atomicAdd(&fresh_s, fresh);
      __syncthreads();
      const uint32_t v = fresh_s, n = (v + kItemVoxels - 1) / kItemVoxels;       // at most 512
      if (threadIdx.x == 0) {
        voxels[bin] = v;
        at_s = atomicAdd(&state->items, n);
      }
      __syncthreads();
      const uint32_t at = at_s;
      for (uint32_t i = threadIdx.x; i < n; i += 256) items[at + i] = bin << 9 | i;
      __syncthreads();
    }
    return;
  }
  const uint32_t k = (blockIdx.x - kLargeBlocks) * 4 + wave;
  if (k >= state->small) return;
  const uint32_t bin = list[k], begin = starts[bin], end = starts[bin + 1];
#pragma unroll
  for (int i = 0; i < kWords<SHIFT> / 256; ++i) bits_s[wave][i * 64 + lane] = make_uint4(0u, 0u, 0u, 0u);
  __builtin_amdgcn_wave_barrier();                       // LDS accesses of a wave are in order
  uint32_t* bits = reinterpret_cast<uint32_t*>(bits_s[wave]);
#pragma unroll 4
  for (uint32_t i = begin + lane; i < end; i += 64) {
    const uint32_t c = cells[i], bit = 1u << (c & 31);
    fresh += (atomicOr(&bits[c >> 5], bit) & bit) == 0u;
  }
  fresh = wave_sum(fresh);
  if (lane == 0) voxels[bin] = fresh;
}

// What the blocks of k_bin_voxels are given.
struct BinArgs {
  VoxParams prm;
  const BinState* state;
  const uint32_t *list, *starts, *bases, *items;
  const float4* moved;
  const uint16_t* cells;
  cellword_t* idx;
  lineflag_t* flags;
  const int32_t* n_voxels;
  int64_t n_bins, slot_bins, capacity, bound;
  int4* coords;
  float4* feats;
  int32_t* counts;
  void* feats_lp;
};

// Coordinates of a cell of the bin whose first cell is c0 (b, z, y, x).
__device__ __forceinline__ int4 cell_at(const int4& c0, uint32_t cell, uint32_t gx, uint32_t gy, uint32_t gz) {
  const uint32_t x = (uint32_t)c0.w + cell, qy = x / gx;
  const uint32_t y = (uint32_t)c0.z + qy, qz = y / gy;
  const uint32_t z = (uint32_t)c0.y + qz, qb = z / gz;
  return make_int4(c0.x + (int)qb, (int)(z - qb * gz), (int)(y - qz * gy), (int)(x - qy * gx));
}

template <int SHIFT> struct BinLds {
  union {
    struct {
      uint32_t bits[kWords<SHIFT>];                      // occupancy of the bin
      uint16_t pre[kWords<SHIFT>];                       // its voxels before each word
    };
    uint16_t list[kSmallBin];                            // small bin: its points ordered by voxel, once bits and pre are done with
  };
  union {
    uint32_t count[kSmallBin / 2 + 1];                   // small bin: points of each voxel, then where they begin; 16 bits each
    struct {                                             // an item's voxels: points, the first of them, the sum of the others
      uint32_t n[kItemVoxels], first[EMC2_VOX_STASH][kItemVoxels];
      float sum[4][kItemVoxels];
    } item;
  };
  uint32_t wsum[4];
};

__device__ __forceinline__ uint32_t block_before(uint32_t v, uint32_t (&wsum)[4]) {   // exclusive
  const uint32_t inc = wave_scan(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
  __syncthreads();
  uint32_t run = inc - v;
  for (int j = 0; j < (int)(threadIdx.x >> 6); ++j) run += wsum[j];
  return run;
}

__device__ __forceinline__ uint32_t rank_in(const uint32_t* bits, const uint16_t* pre, uint32_t cell) {
  return pre[cell >> 5] + __popc(bits[cell >> 5] & ((1u << (cell & 31)) - 1u));
}

// Bits and ranks of the bin to LDS; WRITE: and its lines of the index, those that hold bits and those that held some before this
// call.  Returns the bin's voxels.
template <int SHIFT>
__device__ __forceinline__ uint32_t bin_ranks(BinLds<SHIFT>& s, const BinArgs& a, uint32_t bin, uint32_t begin, uint32_t n, uint32_t base,
                                              bool write) {
  constexpr int WPT = kWords<SHIFT> / 256;               // words a thread: 2, or 8 (half a line)
  constexpr int TPL = 16 / WPT;                          // threads a line
#pragma unroll
  for (int j = 0; j < WPT; ++j) s.bits[threadIdx.x * WPT + j] = 0u;
  __syncthreads();
#pragma unroll 4
  for (uint32_t i = threadIdx.x; i < n; i += 256) {
    const uint32_t c = a.cells[begin + i];
    atomicOr(&s.bits[c >> 5], 1u << (c & 31));
  }
  __syncthreads();
  uint32_t bits[WPT], sum = 0;
#pragma unroll
  for (int j = 0; j < WPT; ++j) {
    bits[j] = s.bits[threadIdx.x * WPT + j];
    sum += __popc(bits[j]);
  }
  uint32_t run = block_before(sum, s.wsum), in_line = sum;
#pragma unroll
  for (int d = 1; d < TPL; d <<= 1) in_line += __shfl_xor(in_line, d, 64);
  alignas(16) uint2 word[WPT];
#pragma unroll
  for (int j = 0; j < WPT; ++j) {
    s.pre[threadIdx.x * WPT + j] = (uint16_t)run;
    word[j] = in_line ? make_uint2(bits[j], base + run) : make_uint2(0u, 0u);
    run += __popc(bits[j]);
  }
  if (write) {
    lineflag_t* flag = a.flags + (int64_t)bin * kLines<SHIFT> + threadIdx.x / TPL;
    const bool stale = *flag != 0;                       // a line's threads are neighbours in one wave: all read before one writes
    if (in_line || stale) {
      uint4* dst = reinterpret_cast<uint4*>(a.idx + (int64_t)bin * kWords<SHIFT> + threadIdx.x * WPT);
#pragma unroll
      for (int j = 0; j < WPT / 2; ++j) dst[j] = reinterpret_cast<const uint4*>(word)[j];
    }
    if (threadIdx.x % TPL == 0 && (in_line != 0) != stale) *flag = in_line != 0;
  }
  __syncthreads();
  return s.wsum[0] + s.wsum[1] + s.wsum[2] + s.wsum[3];
}

// Voxel r of k points: the first of them in q, the sum of the others in rest.
template <int LP>
__device__ __forceinline__ void put_voxel(const BinArgs& a, int64_t r, const int4& c0, uint32_t cell, float4 (&q)[EMC2_VOX_STASH],
                                          const float4& rest, uint32_t k) {
  a.coords[r] = cell_at(c0, cell, (uint32_t)a.prm.grid[0], (uint32_t)a.prm.grid[1], (uint32_t)a.prm.grid[2]);
  a.counts[r] = (int32_t)k;
  emc2_store_mean(r, q, rest, (int32_t)k, a.feats, LP, a.feats_lp);
}

// A bin of at most kSmallBin points: they are ordered by voxel in LDS, then a thread takes a voxel.
template <int SHIFT, int LP>
__device__ __forceinline__ void small_bin(BinLds<SHIFT>& s, const BinArgs& a, uint32_t bin, uint32_t begin, uint32_t n, uint32_t base,
                                          const int4& c0) {
  const uint32_t voxels = bin_ranks<SHIFT>(s, a, bin, begin, n, base, true);
  for (uint32_t i = threadIdx.x; i < voxels / 2 + 1; i += 256) s.count[i] = 0u;
  __syncthreads();
  uint32_t vp[kSmallPoints];                             // voxel, and position among its points, of this thread's points
#pragma unroll
  for (int j = 0; j < kSmallPoints; ++j) {
    const uint32_t i = threadIdx.x + j * 256;
    vp[j] = 0;
    if (j * 256u < n && i < n) {                         // the first test is the block's
      const uint32_t v = rank_in(s.bits, s.pre, a.cells[begin + i]), sh = 16 * (v & 1);
      vp[j] = v | (atomicAdd(&s.count[v >> 1], 1u << sh) >> sh) << 16;
    }
  }
  __syncthreads();
  uint16_t* count = reinterpret_cast<uint16_t*>(s.count);
  const uint32_t per = (voxels + 255) / 256, v0 = threadIdx.x * per;    // consecutive voxels a thread
  uint32_t mine = 0;
  for (uint32_t j = 0; j < per; ++j)
    if (v0 + j < voxels) mine += count[v0 + j];
  uint32_t at = block_before(mine, s.wsum);
  for (uint32_t j = 0; j < per; ++j)
    if (v0 + j < voxels) {
      const uint32_t c = count[v0 + j];
      count[v0 + j] = (uint16_t)at;
      at += c;
    }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSmallPoints; ++j)
    if (j * 256u < n && threadIdx.x + j * 256 < n) s.list[count[vp[j] & 0xffffu] + (vp[j] >> 16)] = (uint16_t)(threadIdx.x + j * 256);
  __syncthreads();
  for (uint32_t v = threadIdx.x; v < voxels && (int64_t)base + v < a.capacity; v += 256) {   // beyond: reported by the scan
    const uint32_t from = count[v], k = (v + 1 < voxels ? count[v + 1] : n) - from;
    float4 q[EMC2_VOX_STASH], rest = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int j = 0; j < EMC2_VOX_STASH; ++j)
      q[j] = (uint32_t)j < k ? a.moved[begin + s.list[from + j]] : make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
    for (uint32_t j = EMC2_VOX_STASH; j < k; ++j) {
      const float4 p = a.moved[begin + s.list[from + j]];
      rest.x += p.x; rest.y += p.y; rest.z += p.z; rest.w += p.w;
    }
    put_voxel<LP>(a, (int64_t)base + v, c0, a.cells[begin + s.list[from]], q, rest, k);
  }
}

// Voxels [v0, v0 + kItemVoxels) of a larger bin, however many points they have: the block looks at all points of the bin.
template <int SHIFT, int LP>
__device__ __forceinline__ void item_of_bin(BinLds<SHIFT>& s, const BinArgs& a, uint32_t bin, uint32_t v0, uint32_t begin, uint32_t n,
                                            uint32_t base, const int4& c0) {
  const uint32_t voxels = bin_ranks<SHIFT>(s, a, bin, begin, n, base, v0 == 0);
  if (threadIdx.x < kItemVoxels) {
    s.item.n[threadIdx.x] = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) s.item.sum[j][threadIdx.x] = 0.f;
  }
  __syncthreads();
#pragma unroll 4
  for (uint32_t i = threadIdx.x; i < n; i += 256) {
    const uint32_t v = rank_in(s.bits, s.pre, a.cells[begin + i]) - v0;
    if (v >= kItemVoxels) continue;
    const uint32_t pos = atomicAdd(&s.item.n[v], 1u);
    if (pos < EMC2_VOX_STASH) {
      s.item.first[pos][v] = i;
    } else {
      const float4 p = a.moved[begin + i];
      unsafeAtomicAdd(&s.item.sum[0][v], p.x);
      unsafeAtomicAdd(&s.item.sum[1][v], p.y);
      unsafeAtomicAdd(&s.item.sum[2][v], p.z);
      unsafeAtomicAdd(&s.item.sum[3][v], p.w);
    }
  }
  __syncthreads();
  const uint32_t v = threadIdx.x;
  if (v >= kItemVoxels || v0 + v >= voxels || (int64_t)base + v0 + v >= a.capacity) return;
  const uint32_t k = s.item.n[v];
  float4 q[EMC2_VOX_STASH];
#pragma unroll
  for (int j = 0; j < EMC2_VOX_STASH; ++j)
    q[j] = (uint32_t)j < k ? a.moved[begin + s.item.first[j][v]] : make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
  put_voxel<LP>(a, (int64_t)base + v0 + v, c0, a.cells[begin + s.item.first[0][v]], q,
                make_float4(s.item.sum[0][v], s.item.sum[1][v], s.item.sum[2][v], s.item.sum[3][v]), k);
}

// Blocks [0, kItemBlocks) share the items of the larger bins.  Behind them a block for every bin of the slot and one more: the first
// state->small have a bin of the list (blocks that stay and take every 1 792nd were 20 % slower: bins have 1 to kSmallBin points).  They
// also share what the bins without points ask for, those past the grid among them -- stale lines cleared -- and the rows past the
// last voxel.
template <int SHIFT, int LP>
__global__ void __launch_bounds__(256) k_bin_voxels(const BinArgs a) {
  __shared__ BinLds<SHIFT> s;
  const BinState st = *a.state;
  if (blockIdx.x < kItemBlocks) {
    for (uint32_t k = blockIdx.x; k < st.items; k += kItemBlocks) {
      const uint32_t item = a.items[k], bin = item >> 9, begin = a.starts[bin];
      const int4 c0 = decode_key((uint64_t)bin << SHIFT, a.prm.grid[0], a.prm.grid[1], a.prm.grid[2]);
      item_of_bin<SHIFT, LP>(s, a, bin, (item & 511u) * kItemVoxels, begin, a.starts[bin + 1] - begin, a.bases[bin], c0);
      __syncthreads();                                   // the next item writes over this one's bits
    }
    return;
  }
  const uint32_t blk = blockIdx.x - kItemBlocks;
  constexpr int FT = kLines<SHIFT> / 8;                  // threads that look at a bin's flags
  if (threadIdx.x < FT && blk < a.slot_bins) {
    const int64_t i = (int64_t)blk * FT + threadIdx.x;
    uint2* f = reinterpret_cast<uint2*>(a.flags) + i;
    const uint2 v = *f;                                  // of a bin with points perhaps in the writing: looked at no further
    if ((v.x | v.y) != 0u && (blk >= a.n_bins || a.starts[blk] == a.starts[blk + 1])) {
      for (int j = 0; j < 8; ++j) {
        if (((j < 4 ? v.x >> (8 * j) : v.y >> (8 * (j - 4))) & 0xffu) == 0u) continue;
        uint4* line = reinterpret_cast<uint4*>(a.idx + ((i * 8 + j) << EMC2_LINE_SHIFT));
#pragma unroll
        for (int q = 0; q < 8; ++q) line[q] = make_uint4(0u, 0u, 0u, 0u);
      }
      *f = make_uint2(0u, 0u);
    }
  }
  if (blk < st.small) {
    const uint32_t bin = a.list[blk], begin = a.starts[bin];
    const int4 c0 = decode_key((uint64_t)bin << SHIFT, a.prm.grid[0], a.prm.grid[1], a.prm.grid[2]);
    small_bin<SHIFT, LP>(s, a, bin, begin, a.starts[bin + 1] - begin, a.bases[bin], c0);
    return;
  }
  const int64_t stride = (int64_t)(a.slot_bins + 1 - st.small) * 256;
  for (int64_t r = *a.n_voxels + (int64_t)(blk - st.small) * 256 + threadIdx.x; r < a.bound; r += stride) {
    a.feats[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    a.counts[r] = 0;
  }
}

template <int SHIFT>
void launch_bins(emc2_ctx* ctx, const float* d_points, const int32_t* d_batch, int64_t n_points, const VoxParams& prm, int64_t n_cells,
                 cellword_t* idx, int64_t capacity, int32_t* d_coords, float* d_feats, int32_t* d_counts, void* d_feats_lp, int lp,
                 int32_t* d_n_voxels, hipStream_t s) {
  const int64_t n = emc2_div_up(n_cells, (int64_t)1 << SHIFT), slot_bins = ctx->slot_tiles << (EMC2_BIN_SHIFT_TILE - SHIFT);
  uint32_t* counts = ctx->bins;                          // [n_bins] each
  uint32_t* starts = counts + ctx->n_bins;               // [n + 1]
  uint32_t* cursors = starts + ctx->n_bins;
  uint32_t* list = cursors + ctx->n_bins;
  uint32_t* voxels = list + ctx->n_bins;
  uint32_t* bases = voxels + ctx->n_bins;
  BinState* state = reinterpret_cast<BinState*>(bases + ctx->n_bins);
  float4* moved = reinterpret_cast<float4*>(ctx->pix_rank);         // scratch of the image pooling: 16 bytes a point,
  uint16_t* cells = reinterpret_cast<uint16_t*>(ctx->pool_acc);     // and 16 more, 2 for its cell,
  uint32_t* items = ctx->pool_acc + ctx->max_points;                // less than 1 for the items
  const dim3 pg((unsigned)emc2_div_up(n_points, kMoveThreads * kMovePoints)), pb(kMoveThreads);
  const dim3 sg((unsigned)emc2_div_up(n, 1024)), sb(1024);
  hipLaunchKernelGGL(k_bin_zero, sg, sb, 0, s, counts, n, state);
  hipLaunchKernelGGL((k_bin_points<SHIFT, false>), pg, pb, 0, s, d_points, d_batch, n_points, prm, counts, nullptr, nullptr);
  hipLaunchKernelGGL(k_bin_starts, sg, sb, 0, s, counts, n, starts, cursors, voxels, list, state);
  hipLaunchKernelGGL((k_bin_points<SHIFT, true>), pg, pb, 0, s, d_points, d_batch, n_points, prm, cursors, moved, cells);
  hipLaunchKernelGGL(k_bin_distinct<SHIFT>, dim3((unsigned)(kLargeBlocks + emc2_div_up(n, 4))), dim3(256), 0, s, state, list, starts, n,
                     cells, voxels, items);
  emc2_scan_totals(ctx, voxels, n, capacity, bases, d_n_voxels, s);
  const BinArgs a = {prm, state, list, starts, bases, items, moved, cells, idx, emc2_slot_flags(ctx, idx), d_n_voxels, n, slot_bins,
                     capacity, n_points < capacity ? n_points : capacity, (int4*)d_coords, (float4*)d_feats, d_counts, d_feats_lp};
  const dim3 vg((unsigned)(kItemBlocks + slot_bins + 1)), vb(256);
  if (lp == 0) hipLaunchKernelGGL((k_bin_voxels<SHIFT, 0>), vg, vb, 0, s, a);
  else if (lp == 1) hipLaunchKernelGGL((k_bin_voxels<SHIFT, 1>), vg, vb, 0, s, a);
  else hipLaunchKernelGGL((k_bin_voxels<SHIFT, 2>), vg, vb, 0, s, a);
}

}  // namespace

// Points of a call from which on the bins pay, if they are kDensePoints a scan tile or fewer on average, and if they are more; of its
// points a tile, from where on a bin is a quarter of a tile, and up to where bins pay at all.  The passes' launches and the bins of many
// points set the time of small clouds, the atomics on an index that fits no L2 that of the point pass.  On grids of 85 to 90 M cells a
// frame, points a tile in brackets, us, point pass / bins of a tile / of a quarter: 480 k of 4 (87) 85 / 86, 540 k of 9 (43) 117 / 84, 600 k of
// 5 (87) 101 / 91, 960 k of 8 (87) 149 / 100 / 122, 1.9 M of 16 (87) 273 / 138 / 213; 600 k of 4 (115) 94 / 109 / 79, of 3 (154) 87 / 108 / 81,
// 1.5 M of 6 (192) 176 / 128 / 116; and of a quarter 600 k of 2 (231) 83 / 85, of one (436) 78 / 92, 900 k of one (694) 98 / 116, 1.0 M of 2
// (385) 114 / 112, 1.2 M of 4 (231) 142 / 104, 1.4 M of 2 (539) 147 / 125, 1.0 M of one (770) 107 / 118, 3.0 M (2 300) 267 / 332.  Frames mixed
// point by point, 1.9 M of 16: 288 / 166.
constexpr int64_t kBinPoints = 524288, kDenseBinPoints = 1000000, kDensePoints = 200, kBinTiles = 1024, kFinePoints = 100, kMostPoints = 720;

static int64_t tiles_of(int64_t n_cells) { return emc2_div_up(n_cells, (int64_t)1 << EMC2_BIN_SHIFT_TILE); }

bool emc2_bins_pay(int64_t n_points, int64_t n_cells) {
  const int64_t tiles = tiles_of(n_cells);               // (an item names its bin in 23 bits)
  return n_points >= (n_points <= kDensePoints * tiles ? kBinPoints : kDenseBinPoints) && tiles >= kBinTiles && tiles < ((int64_t)1 << 21) &&
         n_points <= kMostPoints * tiles;
}

void emc2_voxelize_bins(emc2_ctx* ctx, const float* d_points, const int32_t* d_batch, int64_t n_points, const VoxParams& prm,
                        int64_t n_cells, cellword_t* idx, int64_t capacity, int32_t* d_coords, float* d_feats, int32_t* d_counts,
                        void* d_feats_lp, int lp, int32_t* d_n_voxels, hipStream_t s) {
  const bool fine = n_points >= kFinePoints * tiles_of(n_cells) && emc2_div_up(n_cells, (int64_t)1 << EMC2_BIN_SHIFT_FINE) <= EMC2_BINS_MAX;
  const auto launch = fine ? launch_bins<EMC2_BIN_SHIFT_FINE> : launch_bins<EMC2_BIN_SHIFT_TILE>;
  launch(ctx, d_points, d_batch, n_points, prm, n_cells, idx, capacity, d_coords, d_feats, d_counts, d_feats_lp, lp, d_n_voxels, s);
}
