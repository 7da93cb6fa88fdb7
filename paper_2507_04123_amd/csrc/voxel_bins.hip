// Voxelization of large clouds by bin of cells (paper Sec. 2 / Sec. 3.1 voxelization; Sec. 3.6 (3) prefix-sum index search).
//
// The pass over single points (voxelize.hip) is bound by the memory side of the fabric: one atomic a point (27 G/s on this part,
// whatever the address, the scope or the XCD that asks), then an 8-byte load (55 G/s at random places of an index of gigabytes, 200
// where a block stays inside 256 KB) and a 16-byte store (30 and 190).  Here the points are first moved next to the others of their
// bin of consecutive cells, and a block then owns a bin: its bits, ranks, counts and the order of its points live in LDS, every line
// of the index is written once, and the atomics that leave a CU are two per bin and 8 192 points (of points in no order at all up to two
// a point), one per word of a larger bin and 16 384 points, and the counters of the lists.
//
//   k_bin_points     points per bin
//   k_bin_starts     exclusive scan of them; the bins that have any, and what the larger ones are divided into
//   k_bin_points     the points again, each to its place: (x, y, z, intensity) and the cell inside the bin
//   k_bin_distinct   voxels per bin; the bits of the larger ones
//   k_scan_partials  exclusive scan of those (cellindex.hip): the rank of a bin's first voxel, the number of voxels
//   k_bin_voxels     a block a bin of up to kSmallBin points: index lines and flags, coordinates, counts, means; stale lines cleared
//   k_bin_parts      the same of the larger bins, in parts of their voxels
//
// Bound by memory and by the chain of a block's phases in LDS: a 64-beam frame 64 times (7.5 M voxels, of 5.8 G cells), us: count 55, move
// 123 (154 MB read, 303 written), voxels of the bins 35, scans 35, the bins 254 (177 MB read, 469 written; a wave issues in 18 % of its
// cycles, LDS busy 24 %), no larger ones 4; 1 081 -> 507 in all.  The point pass there: clear 81, mark 295, scan 261, second pass 367,
// means 77.
#include "voxel_point.h"

namespace {

constexpr int kMoveThreads = 1024, kMovePoints = 8;     // points a thread
constexpr int kWindow = 8192;                           // bins a block counts at a time
constexpr int kSmallPoints = 12;                        // points a thread of a small bin's block
constexpr uint32_t kSmallBin = 256 * kSmallPoints;      // points of a bin that one block takes
constexpr uint32_t kChunk = 16384;                      // points of a larger bin that one block marks
constexpr int kChunkBlocks = 512;
constexpr int kPartThreads = 1024, kPartBlocks = 256;   // one a CU
constexpr uint32_t kPartVoxels = 4096, kPartPoints = 16384;   // voxels, and points of them, of a larger bin that one block takes
constexpr uint32_t kLongVoxel = 32;                     // points of a voxel that a wave adds up from

// words (of 32 cells) and lines (of 16 words) of a bin
template <int SHIFT> constexpr int kWords = 1 << (SHIFT - 5);
template <int SHIFT> constexpr int kLines = kWords<SHIFT> >> EMC2_LINE_SHIFT;

// Bins of up to kSmallBin points, of more; the latter's chunks of points, and parts of voxels.
struct BinState { uint32_t small, large, chunks, parts; };

// Parts of a larger bin of so many points and at most so many voxels: so many voxels fit a block's LDS, and where they have many points a
// part has fewer of them, since each point is five atomics in LDS (up to as many parts as there are blocks: each looks at all points).
__device__ __forceinline__ uint32_t bin_parts(uint32_t points, uint32_t voxels) {
  return max((voxels + kPartVoxels - 1) / kPartVoxels, min((points + kPartPoints - 1) / kPartPoints, (uint32_t)kPartBlocks));
}

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

__global__ void __launch_bounds__(1024) k_bin_zero(uint32_t* __restrict__ counts, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  if (i < n) counts[i] = 0u;
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

// Counts (MOVE: and places) a block's points.  moved, cells: point and cell inside the bin, at the point's place.  On the way the first
// of the two launches resets the state, and the second one clears the bits of the larger bins.
template <int SHIFT, bool MOVE>
__global__ void __launch_bounds__(kMoveThreads) k_bin_points(const float* __restrict__ points, const int32_t* __restrict__ batch,
                                                             int64_t n_points, VoxParams prm, uint32_t* __restrict__ counts,
                                                             float4* __restrict__ moved, uint16_t* __restrict__ cells,
                                                             BinState* __restrict__ state, uint4* __restrict__ bits) {
  __shared__ uint32_t win[kWindow];
  if (!MOVE) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *state = BinState{0u, 0u, 0u, 0u};
  } else {
    const int64_t n = (int64_t)state->large * (kWords<SHIFT> / 4);
    for (int64_t i = (int64_t)blockIdx.x * kMoveThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kMoveThreads)
      bits[i] = make_uint4(0u, 0u, 0u, 0u);
  }
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

// starts[i] = points before bin i (starts[n] = all), cursors the same; no voxels yet.  list: the bins of up to kSmallBin points, in any
// order: two bins of three of a frame have no point, and a block that finds that out takes 2 us.  The larger bins have a number each,
// and are divided into chunks (number, bin, first point, end) and parts (number, bin, part); a bin has no more voxels than points or
// cells.
__global__ void __launch_bounds__(1024) k_bin_starts(const uint32_t* __restrict__ counts, int64_t n, uint32_t bin_cells,
                                                     uint32_t* __restrict__ starts, uint32_t* __restrict__ cursors,
                                                     uint32_t* __restrict__ voxels, uint32_t* __restrict__ list,
                                                     uint4* __restrict__ chunks, uint4* __restrict__ parts, BinState* __restrict__ state) {
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
  if (v > kSmallBin) {
    const uint32_t place = atomicAdd(&state->large, 1u);
    const uint32_t c = (v + kChunk - 1) / kChunk, q = bin_parts(v, min(v, bin_cells));
    const uint32_t c0 = atomicAdd(&state->chunks, c), q0 = atomicAdd(&state->parts, q);
    for (uint32_t j = 0; j < c; ++j) chunks[c0 + j] = make_uint4(place, (uint32_t)i, run + j * kChunk, run + min(v, (j + 1) * kChunk));
    for (uint32_t j = 0; j < q; ++j) parts[q0 + j] = make_uint4(place, (uint32_t)i, j, 0u);
  }
  if (i < n) { starts[i] = run; cursors[i] = run; voxels[i] = 0u; }
  if (i == n - 1) starts[n] = run + v;
}

// Voxels of the bins with points: a wave a small bin; kChunkBlocks blocks share the larger ones' points, and their bits.  The counts of
// the points go back to zero, as the next call finds them.
template <int SHIFT>
__global__ void __launch_bounds__(256) k_bin_distinct(const BinState* __restrict__ state, const uint32_t* __restrict__ list,
                                                      const uint32_t* __restrict__ starts, int64_t n_bins,
                                                      const uint16_t* __restrict__ cells, const uint4* __restrict__ chunks,
                                                      uint32_t* __restrict__ voxels, uint32_t* __restrict__ all_bits,
                                                      uint32_t* __restrict__ counts) {
  __shared__ uint4 bits_s[4][kWords<SHIFT> / 4];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t zero = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (zero < n_bins) counts[zero] = 0u;
  uint32_t fresh = 0;
  if (blockIdx.x < kChunkBlocks) {
    uint32_t* bits = reinterpret_cast<uint32_t*>(bits_s[0]);
    for (uint32_t k = blockIdx.x; k < state->chunks; k += kChunkBlocks) {
      const uint4 chunk = chunks[k];
      const uint32_t bin = chunk.y, begin = chunk.z, end = chunk.w;
      for (int i = threadIdx.x; i < kWords<SHIFT>; i += 256) bits[i] = 0u;
      __syncthreads();
      for (uint32_t i = begin + threadIdx.x; i < end; i += 8 * 256) {
        uint32_t c[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) c[q] = cells[min(i + q * 256, end - 1)];      // (the last point again: no other bit)
#pragma unroll
        for (int q = 0; q < 8; ++q) atomicOr(&bits[c[q] >> 5], 1u << (c[q] & 31));
      }
      __syncthreads();
      uint32_t* to = all_bits + (int64_t)chunk.x * kWords<SHIFT>;
      fresh = 0;
      for (int i = threadIdx.x; i < kWords<SHIFT>; i += 256)
        if (bits[i]) fresh += __popc(bits[i] & ~atomicOr(&to[i], bits[i]));
      fresh = wave_sum(fresh);
      if (lane == 0) atomicAdd(&voxels[bin], fresh);
      __syncthreads();                                   // the next chunk writes over this one's bits
    }
    return;
  }
  const uint32_t k = (blockIdx.x - kChunkBlocks) * 4 + wave;
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
  const uint32_t *list, *starts, *bases, *voxels;
  const uint4* bits;
  const uint4* parts;
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
    uint16_t list[kSmallBin];                            // its points ordered by voxel, once bits and pre are done with
  };
  uint32_t count[kSmallBin / 2 + 1];                     // points of each voxel, then where they begin; 16 bits each
  uint32_t wsum[4];
};
template <int SHIFT> struct PartLds {
  uint32_t bits[kWords<SHIFT>];
  uint16_t pre[kWords<SHIFT>];
  uint32_t n[kPartVoxels], first[EMC2_VOX_STASH][kPartVoxels];          // a voxel's points, the first of them, the sum of the others
  float sum[4][kPartVoxels];
  uint32_t wsum[kPartThreads / 64];
};

template <int WAVES> __device__ __forceinline__ uint32_t block_before(uint32_t v, uint32_t (&wsum)[WAVES]) {   // exclusive
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

// Ranks of the bin's words from its bits in LDS; write: and its lines of the index, those that hold bits and those that held some
// before this call.  Every thread of the block calls it, behind a barrier; the ranks are there when it returns.
template <int SHIFT, int WAVES, typename Lds>
__device__ __forceinline__ uint32_t bin_ranks(Lds& s, const BinArgs& a, uint32_t bin, uint32_t base, bool write) {
  constexpr int USED = WAVES * 64 < kWords<SHIFT> / 2 ? WAVES * 64 : kWords<SHIFT> / 2;
  constexpr int WPT = kWords<SHIFT> / USED;              // words a thread: 2, or 8 (half a line)
  constexpr int TPL = 16 / WPT;                          // threads a line
  const bool used = (int)threadIdx.x < USED;
  uint32_t bits[WPT], sum = 0;
#pragma unroll
  for (int j = 0; j < WPT; ++j) {
    bits[j] = used ? s.bits[threadIdx.x * WPT + j] : 0u;
    sum += __popc(bits[j]);
  }
  uint32_t run = block_before<WAVES>(sum, s.wsum), in_line = sum;
#pragma unroll
  for (int d = 1; d < TPL; d <<= 1) in_line += __shfl_xor(in_line, d, 64);
  if (used) {
    alignas(16) uint2 word[WPT];
#pragma unroll
    for (int j = 0; j < WPT; ++j) {
      s.pre[threadIdx.x * WPT + j] = (uint16_t)run;
      word[j] = in_line ? make_uint2(bits[j], base + run) : make_uint2(0u, 0u);
      run += __popc(bits[j]);
    }
    if (write) {
      lineflag_t* flag = a.flags + (int64_t)bin * kLines<SHIFT> + threadIdx.x / TPL;
      const bool stale = *flag != 0;                     // a line's threads are neighbours in one wave: all read before one writes
      if (in_line || stale) {
        uint4* dst = reinterpret_cast<uint4*>(a.idx + (int64_t)bin * kWords<SHIFT> + threadIdx.x * WPT);
#pragma unroll
        for (int j = 0; j < WPT / 2; ++j) dst[j] = reinterpret_cast<const uint4*>(word)[j];
      }
      if (threadIdx.x % TPL == 0 && (in_line != 0) != stale) *flag = in_line != 0;
    }
  }
  __syncthreads();
  uint32_t all = 0;
#pragma unroll
  for (int j = 0; j < WAVES; ++j) all += s.wsum[j];
  return all;
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
  for (int i = threadIdx.x; i < kWords<SHIFT>; i += 256) s.bits[i] = 0u;
  __syncthreads();
#pragma unroll 4
  for (uint32_t i = threadIdx.x; i < n; i += 256) {
    const uint32_t c = a.cells[begin + i];
    atomicOr(&s.bits[c >> 5], 1u << (c & 31));
  }
  __syncthreads();
  const uint32_t voxels = bin_ranks<SHIFT, 4>(s, a, bin, base, true);
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
  uint32_t at = block_before<4>(mine, s.wsum);
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
  const uint32_t lane = threadIdx.x & 63;
  for (uint32_t v = threadIdx.x; v - threadIdx.x < voxels; v += 256) {       // the same for the whole block
    const bool live = v < voxels && (int64_t)base + v < a.capacity;          // beyond: reported by the scan
    const uint32_t from = live ? count[v] : 0u, k = live ? (v + 1 < voxels ? count[v + 1] : n) - from : 0u;
    float4 rest = make_float4(0.f, 0.f, 0.f, 0.f);
    const auto add = [&](float4& to, uint32_t j) {
      const float4 p = a.moved[begin + s.list[j]];
      to.x += p.x; to.y += p.y; to.z += p.z; to.w += p.w;
    };
    if (k <= kLongVoxel)
      for (uint32_t j = EMC2_VOX_STASH; j < k; ++j) add(rest, from + j);
    // (Many points of a voxel one after the other, by the thread that has it, set the time of a bin -- frames padded with points at the
    // origin: 600 000 points of 8 frames, in each a voxel of 2 500 419 / 127 us, 8 of 300 172 / 129, 20 of 40 108 / 102.)
    for (unsigned long long left = __ballot(k > kLongVoxel); left != 0ull; left &= left - 1ull) {
      const int owner = __ffsll(left) - 1;
      const uint32_t f = __shfl(from, owner, 64), m = __shfl(k, owner, 64);
      float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
      for (uint32_t j = EMC2_VOX_STASH + lane; j < m; j += 64) add(sum, f + j);
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        sum.x += __shfl_xor(sum.x, d, 64); sum.y += __shfl_xor(sum.y, d, 64);
        sum.z += __shfl_xor(sum.z, d, 64); sum.w += __shfl_xor(sum.w, d, 64);
      }
      if ((int)lane == owner) rest = sum;
    }
    if (!live) continue;
    float4 q[EMC2_VOX_STASH];
#pragma unroll
    for (int j = 0; j < EMC2_VOX_STASH; ++j)
      q[j] = (uint32_t)j < k ? a.moved[begin + s.list[from + j]] : make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
    put_voxel<LP>(a, (int64_t)base + v, c0, a.cells[begin + s.list[from]], q, rest, k);
  }
}

// A block for every bin of the slot and one more: the first state->small have a bin of the list (blocks that stay and take every
// 1 792nd were 20 % slower: bins have 1 to kSmallBin points).  They also share what the bins without points ask for, those past the
// grid among them -- stale lines cleared -- and the rows past the last voxel.
template <int SHIFT, int LP>
__global__ void __launch_bounds__(256) k_bin_voxels(const BinArgs a) {
  __shared__ BinLds<SHIFT> s;
  const uint32_t small = a.state->small, blk = blockIdx.x;
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
  if (blk < small) {
    const uint32_t bin = a.list[blk], begin = a.starts[bin];
    const int4 c0 = decode_key((uint64_t)bin << SHIFT, a.prm.grid[0], a.prm.grid[1], a.prm.grid[2]);
    small_bin<SHIFT, LP>(s, a, bin, begin, a.starts[bin + 1] - begin, a.bases[bin], c0);
    return;
  }
  const int64_t stride = (int64_t)(a.slot_bins + 1 - small) * 256;
  for (int64_t r = *a.n_voxels + (int64_t)(blk - small) * 256 + threadIdx.x; r < a.bound; r += stride) {
    a.feats[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    a.counts[r] = 0;
  }
}

// The bins of more points than that, in parts of kPartVoxels voxels, however many points these have: a block takes the bin's bits as
// k_bin_distinct left them and looks at all points of the bin once, so a part's voxels are as many as the LDS of a CU has room for.
// us, 128 voxels a block of 256 threads that marks the bin anew (the point pass in brackets) / so: 960 000 points in a layer each of 8 frames
// 148 (120) / 97, in 100 tiles 234 (116) / 104, in 10 860 (115) / 118, half of them in one 1 490 (254) / 295, all 3 115 (282) / 361, all in
// 3 000 cells 4 188 (1 067) / 362; 7.7 M of 64 frames, a layer each 978 (863) / 423, in 100 tiles 5 141 (921) / 627.  A cloud that
// lies in one bin is the slower one still: every part looks at all of its points.
template <int SHIFT, int LP>
__global__ void __launch_bounds__(kPartThreads) k_bin_parts(const BinArgs a) {
  __shared__ PartLds<SHIFT> s;
  constexpr int B = 8;                                   // points a thread looks at together
  const uint32_t t = threadIdx.x, parts = a.state->parts;
  for (uint32_t at = blockIdx.x; at < parts; at += kPartBlocks) {
    const uint4 part = a.parts[at];
    const uint32_t bin = part.y, begin = a.starts[bin], n = a.starts[bin + 1] - begin, base = a.bases[bin];
    const uint32_t voxels = a.voxels[bin], each = (voxels + bin_parts(n, voxels) - 1) / bin_parts(n, voxels), v0 = part.z * each;
    if (v0 >= voxels) continue;                          // the same for the whole block; the parts were counted before the voxels
    for (int i = t; i < kWords<SHIFT> / 4; i += kPartThreads)
      reinterpret_cast<uint4*>(s.bits)[i] = a.bits[(int64_t)part.x * (kWords<SHIFT> / 4) + i];
    for (uint32_t i = t; i < each; i += kPartThreads) {
      s.n[i] = 0u;
#pragma unroll
      for (int j = 0; j < 4; ++j) s.sum[j][i] = 0.f;
    }
    __syncthreads();
    bin_ranks<SHIFT, kPartThreads / 64>(s, a, bin, base, v0 == 0);
    for (uint32_t i0 = t; i0 < n; i0 += B * kPartThreads) {
      uint32_t v[B], pos[B];
#pragma unroll
      for (int q = 0; q < B; ++q) v[q] = a.cells[begin + min(i0 + q * kPartThreads, n - 1)];
#pragma unroll
      for (int q = 0; q < B; ++q) v[q] = i0 + q * kPartThreads < n ? rank_in(s.bits, s.pre, v[q]) - v0 : each;
#pragma unroll
      for (int q = 0; q < B; ++q) {
        pos[q] = v[q] < each ? atomicAdd(&s.n[v[q]], 1u) : 0u;
        if (v[q] < each && pos[q] < EMC2_VOX_STASH) s.first[pos[q]][v[q]] = i0 + q * kPartThreads;
      }
      float4 p[B];
#pragma unroll
      for (int q = 0; q < B; ++q)
        if (pos[q] >= EMC2_VOX_STASH) p[q] = a.moved[begin + i0 + q * kPartThreads];
#pragma unroll
      for (int q = 0; q < B; ++q)
        if (pos[q] >= EMC2_VOX_STASH) {
          unsafeAtomicAdd(&s.sum[0][v[q]], p[q].x);
          unsafeAtomicAdd(&s.sum[1][v[q]], p[q].y);
          unsafeAtomicAdd(&s.sum[2][v[q]], p[q].z);
          unsafeAtomicAdd(&s.sum[3][v[q]], p[q].w);
        }
    }
    __syncthreads();
    const int4 c0 = decode_key((uint64_t)bin << SHIFT, a.prm.grid[0], a.prm.grid[1], a.prm.grid[2]);
    for (uint32_t v = t; v < each; v += kPartThreads) {
      if (v0 + v >= voxels || (int64_t)base + v0 + v >= a.capacity) break;
      const uint32_t k = s.n[v];
      float4 q[EMC2_VOX_STASH];
#pragma unroll
      for (int j = 0; j < EMC2_VOX_STASH; ++j)
        q[j] = (uint32_t)j < k ? a.moved[begin + s.first[j][v]] : make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
      put_voxel<LP>(a, (int64_t)base + v0 + v, c0, a.cells[begin + s.first[0][v]], q,
                    make_float4(s.sum[0][v], s.sum[1][v], s.sum[2][v], s.sum[3][v]), k);
    }
    __syncthreads();                                     // the next part writes over this one's
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
  // scratch of the image pooling, of 16 bytes a point each: the points moved; and, a quarter each, their cells (2 bytes a point), the
  // bits of the larger bins (at most a third of a bit mask a point of theirs: 2.7), their chunks, and their parts (far less than 1)
  float4* moved = reinterpret_cast<float4*>(ctx->pix_rank);
  const int64_t quarter = (ctx->max_points + 3) / 4 * 4;             // (the scratch ends 256 words and more behind max_points * 4)
  uint16_t* cells = reinterpret_cast<uint16_t*>(ctx->pool_acc);
  uint32_t* bits = ctx->pool_acc + quarter;
  uint4* chunks = reinterpret_cast<uint4*>(ctx->pool_acc + 2 * quarter);
  uint4* parts = reinterpret_cast<uint4*>(ctx->pool_acc + 3 * quarter);
  const dim3 pg((unsigned)emc2_div_up(n_points, kMoveThreads * kMovePoints)), pb(kMoveThreads);
  const dim3 sg((unsigned)emc2_div_up(n, 1024)), sb(1024);
  // The counts are zero between calls, unless a launch of the last one failed; a clearing that is only recorded may never run.  (A call that
  // fails clears them too, if it still can, for graphs that were recorded while they were zero.)
  const auto zero_counts = [&] { hipLaunchKernelGGL(k_bin_zero, dim3((unsigned)emc2_div_up(ctx->n_bins, 1024)), sb, 0, s, counts, ctx->n_bins); };
  const bool recorded = !ctx->bins_zeroed && emc2_capturing(s);
  if (!ctx->bins_zeroed) zero_counts();
  ctx->bins_zeroed = false;
  hipLaunchKernelGGL((k_bin_points<SHIFT, false>), pg, pb, 0, s, d_points, d_batch, n_points, prm, counts, nullptr, nullptr, state, nullptr);
  hipLaunchKernelGGL(k_bin_starts, sg, sb, 0, s, counts, n, 1u << SHIFT, starts, cursors, voxels, list, chunks, parts, state);
  hipLaunchKernelGGL((k_bin_points<SHIFT, true>), pg, pb, 0, s, d_points, d_batch, n_points, prm, cursors, moved, cells, state, (uint4*)bits);
  hipLaunchKernelGGL(k_bin_distinct<SHIFT>, dim3((unsigned)(kChunkBlocks + emc2_div_up(n, 4))), dim3(256), 0, s, state, list, starts, n,
                     cells, chunks, voxels, bits, counts);
  emc2_scan_totals(ctx, voxels, n, capacity, bases, d_n_voxels, s);
  const BinArgs a = {prm, state, list, starts, bases, voxels, (const uint4*)bits, parts, moved, cells, idx, emc2_slot_flags(ctx, idx), d_n_voxels,
                     n, slot_bins, capacity, n_points < capacity ? n_points : capacity, (int4*)d_coords, (float4*)d_feats, d_counts,
                     d_feats_lp};
#define VOXELS(LP)                                                                                                          \
  {                                                                                                                         \
    hipLaunchKernelGGL((k_bin_voxels<SHIFT, LP>), dim3((unsigned)(slot_bins + 1)), dim3(256), 0, s, a);                      \
    hipLaunchKernelGGL((k_bin_parts<SHIFT, LP>), dim3(kPartBlocks), dim3(kPartThreads), 0, s, a);                            \
  }
  if (lp == 0) VOXELS(0) else if (lp == 1) VOXELS(1) else VOXELS(2)
#undef VOXELS
  const bool ok = hipPeekAtLastError() == hipSuccess;
  if (!ok) zero_counts();
  ctx->bins_zeroed = ok && !recorded;
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
  const int64_t tiles = tiles_of(n_cells);
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
