// The walk of the kernels whose blocks keep all weights in LDS (spconv_resident.hip, spconv_i8.hip): waves that take tiles of 32 rows by
// themselves.  Why, and against what, is said in the two files.
//
// What a wave waits for is arranged so: the first tile's rows are requested before the block's one barrier, so that they come while
// the weights do; a tile's entries behind all rows of the tile before (loads return in order, so whatever is requested after
// entries, which come from memory, waits for them); and a tile's first rows before the results of the tile before are stored.  Against
// entries requested behind a tile's first group and rows behind the barrier and the stores, us: 32 -> 64 3 k rows 7.9 / 7.5, 304 k 41 / 38,
// stride-2 69 k 14.5 / 13.9, 223 k 28.8 / 27.6; 64 -> 32 transposed 223 k 24.8 / 24.5, 22 k 10.8 / 10.3; all sizes and maps of five frames
// 3.4 and 2.1 % on average.  Two groups of rows in flight instead of one: int8 64 -> 32 69 k 9.7 / 10.4, and 64 columns spill.
// kRowsFirst: how a block copies its weights.  15 waves don't divide their pieces, and the loop that copies them waits for each turn's
// loads, nine where 12 waves had one; with one, and the first rows requested behind it, a few tiles a wave take up to a fifth less.  us, 12 waves and
// the loop / 15 / so: 16-bit 64 -> 32 submanifold 8 600 rows 7.9 / 8.6 / 7.3, 16 k 8.8 / 9.4 / 8.2, 69 k - / 25.0 / 24.6, stride-2 31 k 9.4 / 9.1 /
// 8.5, any row from anywhere 15 k 8.3 / 9.5 / 7.6; int8 64 -> 64 stride-2 69 k (12 waves) 14.6 / - / 13.3, 64 -> 32 20 k - / 6.3 / 5.9, E4M3 6.8 / 6.5.
// Shapes that lose by it keep the loop: 16-bit 32 -> 64 level up to 30 k rows, +1.2 % beyond; E4M3 64 -> 64 and 8-bit 128 -> 32 -2 to +1 % up to
// 30 k rows, +1.4 % beyond.
#pragma once

#include "common.h"
#include "xcd_tiles.h"

namespace emc2_resident {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native vector: real loads and stores
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Waves of a block, one block a CU, for registers up to 128 (what the LDS beside the weights holds the entries of) or 168 a lane; a form's
// kernel takes the former unless it would spill: rows by address (inputs of 4 GiB and more) and int8 64 -> 64.  us, 12 / 15: 32 -> 64 submanifold
// 304 k rows 37.5 / 34.6, stride-2 223 k 27.9 / 23.5, 69 k 14.4 / 12.7; 64 -> 32 transposed 166 k 20.2 / 20.0, submanifold 66 k 24.5 / 23.2; E4M3 64 -> 64
// 304 k 44.0 / 40.6; int8 128 -> 32 165 k 44.5 / 41.8.  (int8 64 -> 64 with fp16 results would fit with kRowsFirst: the same on average.)
constexpr int kRWaves = 15, kRWavesWide = 12;
constexpr int kRRows = 32;                // output rows of a wave
constexpr int kRRun = 16;                 // tiles of a run: 512 rows
constexpr int64_t kRCUs = 256;            // compute units of the part; one block fits each

// OP: KS 64-byte parts of a row, NT column tiles of 16, the accumulator, run(weights, rows, accumulator) for 16 rows, 16 columns and a
// part, and store(row, columns' accumulators), which a lane calls with channels 16j + 4q .. + 3 of its row: 16 * mt + m of the tile; kRowsFirst.
template <typename OP, bool BUF>
__device__ __forceinline__ void walk(const OP& op, uint32_t block, uint32_t n_blocks, const void* __restrict__ in, const u32x4* __restrict__ wp,
                                     const int32_t* __restrict__ nbr, const int32_t* __restrict__ d_n_out, int64_t capacity_out,
                                     int32_t n_in, int32_t* __restrict__ dev_flags, const void* __restrict__ zrow) {
  constexpr int KS = OP::KS, NT = OP::NT, MT = 2;
  constexpr uint32_t ROW = 64 * KS;         // bytes of a row
  typedef typename OP::acc_t acc_t;
  constexpr int WT = KS * NT * 64;          // 16-byte weight pieces of a tap
  constexpr int NA = MT * KS;               // operand loads of a tap
  __shared__ u32x4 wl[27 * WT];
  constexpr int WAVES = OP::template waves<BUF>;
  __shared__ int32_t ent_s[WAVES][27 * kRRows];
  __shared__ uint32_t taken_s;              // tiles of the block that its waves have taken
  int64_t n_out = *d_n_out;
  if (n_out > capacity_out) n_out = capacity_out;
  // The blocks of an XCD take its tiles one by one, so that few tiles are spread over all of them.
  const uint32_t blocks = n_blocks / 8, blk = block / 8;
  const int64_t n_tiles = (n_out + kRRows - 1) / kRRows, tiles = emc2_xcd_tiles<kRRun>(block % 8, n_tiles);
  if ((int64_t)blk >= tiles) return;        // uniform for the block
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = lane & 15, q = lane >> 4, half = lane >> 5, row = lane & 31;
  const __amdgpu_buffer_rsrc_t rows =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(in), 0, BUF ? (int)((uint32_t)n_in * ROW) : 0, 0x00020000);
  unsigned long long oob = 0ull;            // lanes that saw an entry outside [0, n_in)
  // A wave takes the block's next tile while it works on the last: tiles have from one to nine groups.
  if (threadIdx.x == 0) taken_s = WAVES;
  const auto take = [&] {
    uint32_t k = 0;
    if (lane == 0) k = atomicAdd(&taken_s, 1u);
    return (int64_t)blk + (int64_t)__builtin_amdgcn_readfirstlane(k) * blocks;
  };
  int64_t slot = blk + (int64_t)wave * blocks, row0 = 0;

  // half h of the wave holds the entries of taps 2i + h of the 32 rows (past the last tile: the last one's again)
  int32_t e[14];
  const auto entries = [&](int64_t at) {
    const int64_t r0 = emc2_xcd_tile<kRRun>(block % 8, at < tiles ? at : tiles - 1, n_tiles) * kRRows;
    const int32_t* p = nbr + r0 + (r0 + row < n_out ? row : 0);
#pragma unroll
    for (int i = 0; i < 14; ++i) e[i] = (p + (int64_t)(2 * i) * capacity_out)[i < 13 && half ? capacity_out : 0];
  };
  entries(slot);
  int32_t* ent = ent_s[wave];
  acc_t acc[MT][NT];
  u32x4 a[3][NA];                           // operands in flight, of a group's three taps
  uint32_t groups = 0, g = 0;               // groups still to request; the one in flight
#define EMC2_LOAD(G, KX)                                                                                                     \
  _Pragma("unroll") for (int mt_ = 0; mt_ < MT; ++mt_) {                                                                     \
    const int32_t j_ = ent[(3 * (G) + (KX)) * kRRows + 16 * mt_ + m];                                                        \
    _Pragma("unroll") for (int ks_ = 0; ks_ < KS; ++ks_) {                                                                   \
      if constexpr (BUF)   /* absent: 2^32 less a row, and a piece of the row: out of range, zero */                         \
        a[KX][mt_ * KS + ks_] =                                                                                              \
            __builtin_amdgcn_raw_buffer_load_b128(rows, (int)((uint32_t)j_ * ROW + 16u * (uint32_t)q + 64u * ks_), 0, 0);    \
      else                                                                                                                   \
        a[KX][mt_ * KS + ks_] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(j_ >= 0 ? in : zrow) +         \
                                                                (j_ >= 0 ? (int64_t)j_ * ROW : 0) + 16 * q + 64 * ks_);      \
    }                                                                                                                        \
  }
  // the weights are the first operand, so that a lane ends up with four consecutive channels of one row
#define EMC2_TAP(G, KX)                                                                                                      \
  _Pragma("unroll") for (int ks = 0; ks < KS; ++ks) {                                                                        \
    const u32x4* w_ = wl + ((3 * (G) + (KX)) * KS + ks) * (NT * 64) + lane;                                                  \
    u32x4 b[NT];                                                                                                             \
    _Pragma("unroll") for (int j = 0; j < NT; ++j) b[j] = w_[j * 64];                                                        \
    _Pragma("unroll") for (int mt = 0; mt < MT; ++mt)                                                                        \
      _Pragma("unroll") for (int j = 0; j < NT; ++j) acc[mt][j] = OP::run(b[j], a[KX][mt * KS + ks], acc[mt][j]);            \
  }
  // The entries of the tile at `slot` as rows the kernel may read (absent and beyond the input: -1), [tap][row]; the groups to run, and the
  // first of them requested (a tile without a neighbour runs group 0 on zeros).
  const auto begin = [&] {
    row0 = emc2_xcd_tile<kRRun>(block % 8, slot, n_tiles) * kRRows;
    const int32_t dead = row0 + row < n_out ? 0 : -1;
    groups = 0;
#pragma unroll
    for (int i = 0; i < 14; ++i) {
      const int32_t j = max(emc2_entry(e[i], dead, n_in, oob), -1);
      const unsigned long long some = __ballot(j >= 0);
#pragma unroll
      for (int t = 0; t < 2; ++t)
        if (2 * i + t < 27 && (t == 0 ? some & 0xffffffffull : some >> 32) != 0ull) groups |= 1u << ((2 * i + t) / 3);
      if (2 * i + half < 27) ent[(2 * i + half) * kRRows + row] = j;
    }
    __builtin_amdgcn_wave_barrier();        // LDS accesses of a wave are in order
    g = 0;
    if (groups != 0) {
      g = __builtin_ctz(groups);
      groups &= groups - 1;
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) EMC2_LOAD(g, kx)
    } else {
#pragma unroll
      for (int kx = 0; kx < 3; ++kx)
#pragma unroll
        for (int i = 0; i < NA; ++i) a[kx][i] = u32x4{0u, 0u, 0u, 0u};
    }
  };
  if constexpr (OP::kRowsFirst) {
    constexpr int WN = (27 * WT + WAVES * 64 - 1) / (WAVES * 64);
    u32x4 w[WN];                            // a thread's share, all of it requested before the first rows and stored behind their requests
#pragma unroll
    for (int i = 0; i < WN; ++i) w[i] = wp[min((int)threadIdx.x + i * WAVES * 64, 27 * WT - 1)];
    if (slot < tiles) begin();
#pragma unroll
    for (int i = 0; i < WN; ++i)
      if ((int)threadIdx.x + i * WAVES * 64 < 27 * WT) wl[threadIdx.x + i * WAVES * 64] = w[i];
  } else {
    for (int p = threadIdx.x; p < 27 * WT; p += WAVES * 64) wl[p] = wp[p];
    if (slot < tiles) begin();
  }
  // the weights and the counter of the tiles are in LDS; the loads of the first rows stay in flight
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

  while (slot < tiles) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[mt][j] = acc_t{0, 0, 0, 0};
    const int64_t next = take();
    while (groups != 0) {
      const uint32_t then = __builtin_ctz(groups);
      groups &= groups - 1;
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) {
        EMC2_TAP(g, kx)
        if constexpr (!BUF) __builtin_amdgcn_sched_barrier(0);   // (or the next addresses, of 64 bits, are kept beside the operands)
        EMC2_LOAD(then, kx)
      }
      g = then;
    }
    entries(next);                          // behind all of this tile's rows, which so do not wait for them
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) EMC2_TAP(g, kx)
    const int64_t done0 = row0;
    slot = next;
    if (slot < tiles) begin();              // its first rows come while this tile's are stored
    op.store(done0, m, q, n_out, acc);
  }
#undef EMC2_LOAD
#undef EMC2_TAP
  emc2_report_oob(oob, dev_flags);
}

}  // namespace emc2_resident
