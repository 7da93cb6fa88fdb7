// Voxelization and every kernel map of one or more stacks in one call (paper Sec. 3.1 data bridge, Sec. 3.5 kernel maps,
// Sec. 3.6 (3) prefix-sum index search): the same results as emc2_voxelize followed by emc2_build_kmap per level.
//
// What bounds the call-by-call form is launches: a 120 000-point frame through four levels is 28 dependent launches,
// most of them with 1-3 us of work, and a dependent launch costs 4.7 us on this part whatever it does.  Here a stack is a
// chain of phases, one launch each, and a launch carries everything that is ready by then, of every level and of every
// stack of the call (blocks are dealt to jobs by ranges):
//
//   phase   finest level (0)                  level l >= 1, built from level l - 1
//   1       clear flagged lines; zero the scan's sums of all levels
//   2       mark the points' cells
//   3       popcount sums (over 4 tiles)      gather 1
//   4       prefix fields                     gather 2, expand 1
//   5       points -> stashes                 gather 3, expand 2
//   6       means                             gather 4, expand 3
//   7                                         expand 4
//   last    kernel maps of all levels: once the last level is expanded, with the means for up to three levels
// A phase in which no stack has anything to do is not launched; a small cloud on a small grid is one launch (k_stack_small).
//
// gather l: a coarse word is read off the fine level's bits (27 cells behind every coarse cell: nine bit rows OR-ed, then
// one shift-or and an even-bit compress), so no atomics are needed, nothing has to be cleared first, and the word's
// popcount joins the scan's sums in the same pass.  expand l: prefix fields and coordinates in one pass.
// A frame of 120 000 points through four levels: 28 launches before, 7 now; 109 us, the last launch at the rate of a copy.
#include <string.h>

#include "kmap_probe.h"
#include "voxel_point.h"

namespace {

constexpr int kStacks = 4;                       // stacks per launch chain (kernel arguments hold their descriptions)
constexpr int kLevels = EMC2_STACK_MAX_LEVELS;
// Words per block of gather / expand: 8 lines where a level is at most 1 024 such granules (half a round of the chip), else
// 32 lines.  A coarse level is a chain of dependent loads on little data, which more blocks shorten: levels 2 and 3 of a
// 64-beam frame, gathers and expansions, 22 + 12 us of launches before, 11 + 8 now.  A fine one is mostly empty granules, which
// cost their blocks: levels 1 of eight routed frames in small granules 66 -> 119 us.
constexpr int kGranuleWords = 128;
constexpr int kGranuleMax = 512;
constexpr int64_t kSmallGranules = 1024;
constexpr int kSuper = 64;                       // sums per super-sum: a block's base is at most units/64 + 63 reads
constexpr int kPrefixTiles = 4;                  // tiles per block of the prefix pass
constexpr int kMaxJobs = 24;

struct DevLevel {
  cellword_t* idx;
  lineflag_t* flags;
  uint32_t* sums;         // popcount sums per unit (level 0: a tile of 2048 words; above: a granule)
  uint32_t* supers;       // sums of 64 of them
  int4* coords;
  int32_t* n;
  int32_t* subm;
  int32_t* down;
  int64_t cap;
  int64_t cells;
  int32_t g[3];
  int32_t units;
  int32_t words;          // of a unit
};

struct DevStack {
  VoxParams prm;
  int32_t expert;               // < 0: d_batch holds frame ids; else: it holds scene ids, routed by `route` / `slot`
  int32_t n_levels;
  int32_t lp;
  const int32_t* batch;
  const int32_t* route;         // expert of every scene
  const int32_t* slot;          // position of every scene in its expert's group
  int32_t* group_batch;         // the frame id each point got, or NULL
  float4* feats;
  int32_t* counts;
  void* feats_lp;
  float4* stash;
  int64_t stash_pitch;
  unsigned long long* first;    // per point: the first of its voxel
  int32_t* dev_words;
  int64_t zero_rows;
  DevLevel lv[kLevels];
};

enum Role { R_CLEAR = 0, R_ZERO, R_MARK, R_SUM, R_PREFIX, R_SCATTER, R_MEAN, R_GATHER, R_EXPAND, R_PROBE };

struct Job {
  int32_t role, stack, level;
  uint32_t first;               // first block of the job
};

struct Args {
  const float* points;
  int64_t n_points;
  int32_t n_jobs, n_stacks;
  uint32_t blocks;
  Job job[kMaxJobs];
  DevStack st[kStacks];
};
static_assert(sizeof(Args) <= 4096, "kernel arguments");

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = __shfl_up(v, d, 64);
    if ((int)(threadIdx.x & 63) >= d) v += t;
  }
  return v;
}

// Quotients of cell keys: 32-bit wherever the grid's keys fit (several times cheaper).
__device__ __forceinline__ uint64_t div_key(uint64_t a, uint32_t b) {
  return (a >> 32) == 0 ? (uint64_t)((uint32_t)a / b) : a / b;
}

// The frame id of point i in a routed stack: its scene's slot in its expert's group, -1 if another expert's.
__device__ __forceinline__ int32_t routed_frame(const DevStack& st, int64_t i) {
  const int32_t s = st.batch ? st.batch[i] : 0;
  return s >= 0 && s < st.prm.n_batch && st.route[s] == st.expert ? st.slot[s] : -1;
}

// A point's cell in a stack.
__device__ __forceinline__ PointCell locate_in(const Args& a, const DevStack& st, int64_t i) {
  PointCell pc = locate(a.points, st.expert < 0 ? st.batch : nullptr, i, a.n_points, st.prm);
  if (st.expert >= 0 && pc.keep) {
    const int32_t b = routed_frame(st, i);
    pc.keep = b >= 0 && b < st.prm.n_batch;
    pc.c.x = b;
    pc.key += (uint64_t)(pc.keep ? b : 0) * st.prm.grid[2] * (uint64_t)st.prm.grid[1] * st.prm.grid[0];
  }
  return pc;
}

__device__ __forceinline__ void report_total(const DevStack& st, const DevLevel& lv, uint32_t total) {
  if ((int64_t)total > lv.cap) {
    atomicOr(st.dev_words, EMC2_DEVFLAG_CAPACITY);
    *lv.n = (int32_t)lv.cap;
  } else {
    *lv.n = (int32_t)total;
  }
}

// Two tiles per block, one thread per line: zero the flagged lines and lower their flags.
__device__ __forceinline__ void role_clear(const DevLevel& lv, uint32_t blk) {
  const int64_t tile = (int64_t)blk * 2 + (threadIdx.x >> 7);
  if (tile >= lv.units) return;
  const int64_t line = tile * EMC2_LINES_PER_TILE + (threadIdx.x & 127);
  if (!lv.flags[line]) return;
  uint4* p = reinterpret_cast<uint4*>(lv.idx + (line << EMC2_LINE_SHIFT));
#pragma unroll
  for (int i = 0; i < 8; ++i) p[i] = make_uint4(0u, 0u, 0u, 0u);
  lv.flags[line] = 0;
}

__device__ __forceinline__ void role_zero(const DevStack& st) {
  for (int l = 0; l < st.n_levels; ++l)
    for (int i = threadIdx.x; i < (st.lv[l].units + kSuper - 1) / kSuper; i += 256) st.lv[l].supers[i] = 0u;
}

__device__ __forceinline__ void role_mark(const Args& a, const DevStack& st, uint32_t blk) {
  const int64_t i = (int64_t)blk * 256 + threadIdx.x;
  if (i < st.zero_rows) {   // what the points are accumulated into; at most min(n_points, capacity) voxels exist
    st.feats[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    st.counts[i] = 0;
  }
  if (st.expert >= 0 && st.group_batch && i < a.n_points) st.group_batch[i] = routed_frame(st, i);
  emc2_mark_point<2>(locate_in(a, st, i), i, a.n_points, reinterpret_cast<uint32_t*>(st.lv[0].idx), st.lv[0].flags, st.first);
}

// Four tiles per block, a wave each (no block barrier); a lane owns two adjacent lines = 32 words.
__device__ __forceinline__ void role_sum(const DevLevel& lv, uint32_t blk) {
  const int64_t tile = (int64_t)blk * 4 + (threadIdx.x >> 6);
  if (tile >= lv.units) return;
  const int lane = threadIdx.x & 63;
  const uint32_t f = reinterpret_cast<const uint16_t*>(lv.flags + tile * EMC2_LINES_PER_TILE)[lane];
  uint32_t s = 0;
  if (f) {
    const uint4* p = reinterpret_cast<const uint4*>(lv.idx + tile * EMC2_SCAN_TILE + lane * 32);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if ((f >> (8 * h)) & 0xffu)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint4 v = p[8 * h + i];
          s += __popc(v.x) + __popc(v.z);
        }
  }
  s = wave_sum(s);
  if (lane == 0) {
    lv.sums[tile] = s;
    if (s) atomicAdd(&lv.supers[tile / kSuper], s);
  }
}

// Sum of the units before `unit`, the same in every lane of the wave.
__device__ __forceinline__ uint32_t base_of(const DevLevel& lv, int64_t unit) {
  const int lane = threadIdx.x & 63;
  uint32_t s = 0;
#pragma unroll 4
  for (int i = lane; i < (int)(unit / kSuper); i += 64) s += lv.supers[i];
  const int64_t i = unit / kSuper * kSuper + lane;
  if (i < unit) s += lv.sums[i];
  return wave_sum(s);
}

// Four tiles per block, a wave each; a lane owns two adjacent lines.  An index of at most four tiles (8 192 words, what the
// single calls scan in one block too) is one block, which finds its tiles' bases itself, through LDS, and needs no popcount
// sums from a launch before this one.  One level on 200 000 cells, as a graph: 2 000 points 42.2 us call by call, 44.8 with
// the sums of a launch of their own, 40.6 so; 20 000 points 49.2 / 52.3 / 47.6.
__device__ __forceinline__ void role_prefix(const DevStack& st, const DevLevel& lv, uint32_t blk) {
  __shared__ uint32_t tsum[kPrefixTiles];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t tile = (int64_t)blk * kPrefixTiles + wave;
  const bool whole = lv.units <= kPrefixTiles;   // uniform for the block
  const bool mine = tile < lv.units;
  const uint32_t f = mine ? reinterpret_cast<const uint16_t*>(lv.flags + tile * EMC2_LINES_PER_TILE)[lane] : 0u;
  const bool last = tile == lv.units - 1;
  if (!whole && __ballot(f != 0) == 0ull && !last) return;   // no bit, so no prefix field anybody reads
  uint4* p = reinterpret_cast<uint4*>(lv.idx + tile * EMC2_SCAN_TILE + lane * 32);
  uint4 v[16];
  uint32_t s = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bool have = ((f >> (8 * h)) & 0xffu) != 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      v[8 * h + i] = have ? p[8 * h + i] : make_uint4(0u, 0u, 0u, 0u);
      s += __popc(v[8 * h + i].x) + __popc(v[8 * h + i].z);
    }
  }
  const uint32_t inc = wave_scan(s);
  uint32_t base = 0;
  if (whole) {
    if (lane == 63) tsum[wave] = inc;
    __syncthreads();
    for (int j = 0; j < wave; ++j) base += tsum[j];
  } else {
    base = base_of(lv, tile);
  }
  uint32_t run = base + inc - s;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bool have = ((f >> (8 * h)) & 0xffu) != 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      uint4 w = v[8 * h + i];
      w.y = run;
      run += __popc(w.x);
      w.w = run;
      run += __popc(w.z);
      if (have) p[8 * h + i] = w;
    }
  }
  if (last && lane == 63) report_total(st, lv, run);
}

__device__ __forceinline__ void role_scatter(const Args& a, const DevStack& st, uint32_t blk) {
  const int64_t i = (int64_t)blk * 256 + threadIdx.x;
  const PointCell pc = locate_in(a, st, i);
  if (!pc.keep) return;
  const DevLevel& lv = st.lv[0];
  const int32_t r = cell_lookup(lv.idx, pc.key);
  if (r < 0 || r >= lv.cap) return;      // beyond capacity: reported by the scan, dropped here
  emc2_stash_point(i, r, pc, st.first, lv.coords, st.feats, st.counts, st.stash, st.stash_pitch);
}

__device__ __forceinline__ void role_mean(const DevStack& st, uint32_t blk) {
  const int64_t r = (int64_t)blk * 256 + threadIdx.x;
  if (r < *st.lv[0].n) emc2_voxel_mean(r, st.stash, st.stash_pitch, st.feats, st.counts, st.lp, st.feats_lp);
}

// The 32 bits of word w of level `lv` from the bits of the finer level `in`.  An output at ox reads 2ox-1 .. 2ox+1 on every
// axis: the (up to) nine input rows of an output row segment are OR-ed as bit strings that start at 2*ox-1, then output
// bit i is S[2i] | S[2i+1] | S[2i+2].
__device__ __forceinline__ uint32_t gather_word(const DevLevel& in, const DevLevel& lv, int64_t w) {
  const uint32_t gox = (uint32_t)lv.g[0], goy = (uint32_t)lv.g[1], goz = (uint32_t)lv.g[2];
  const int gx = in.g[0], gy = in.g[1], gz = in.g[2];
  uint64_t key = (uint64_t)w * 32;
  const uint64_t end = key + 32 < (uint64_t)lv.cells ? key + 32 : (uint64_t)lv.cells;
  uint32_t bits = 0;
  int pos = 0;
  while (key < end) {
    const uint64_t row = div_key(key, gox);
    const uint32_t ox = (uint32_t)(key - row * gox);
    const uint64_t t = div_key(row, goy);
    const int oy = (int)(row - t * goy);
    const uint64_t b = div_key(t, goz);
    const int oz = (int)(t - b * goz);
    const int len = (int)((end - key) < (uint64_t)(gox - ox) ? (end - key) : (uint64_t)(gox - ox));
    const int xs = 2 * (int)ox - 1 < 0 ? 0 : 2 * (int)ox - 1;
    const int xe0 = 2 * ((int)ox + len - 1) + 1;
    const int xe = xe0 < gx ? xe0 : gx - 1;
    const int nb = xe - xs + 1;                       // 1 .. 65 input bits per row
    const int shl = xs - (2 * (int)ox - 1);           // 1 where the row's first bit would be x = -1, else 0
    uint64_t lo = 0;                                  // bits 0..63 of the OR of the rows, bit 0 <-> x = 2*ox - 1
    uint32_t hi = 0;                                  // bit 64
    // All 27 loads of the nine rows are in flight together: a row outside the grid re-reads the centre row's word and is
    // masked, a second or third word that the row does not reach re-reads the first.  With a branch per row the nine
    // round trips followed each other (the phase that gathers a 64-beam frame's level 1: 24.0 -> 18.4 us).
    uint32_t w0[9], w1[9], w2[9];
    int sh[9];
    bool in_row[9];
#pragma unroll
    for (int d = 0; d < 9; ++d) {
      const int iz = 2 * oz + d / 3 - 1, iy = 2 * oy + d % 3 - 1;
      in_row[d] = iz >= 0 && iz < gz && iy >= 0 && iy < gy;
      const uint64_t k = ((b * gz + (uint64_t)(in_row[d] ? iz : 2 * oz)) * gy + (uint64_t)(in_row[d] ? iy : 2 * oy)) * gx + (uint64_t)xs;
      const cellword_t* p = in.idx + (k >> 5);
      sh[d] = (int)(k & 31u);
      w0[d] = p[0].x;
      w1[d] = p[sh[d] + nb > 32 ? 1 : 0].x;
      w2[d] = p[sh[d] + nb > 64 ? 2 : 0].x;
    }
#pragma unroll
    for (int d = 0; d < 9; ++d) {
      const uint32_t v1 = sh[d] + nb > 32 ? w1[d] : 0u, v2 = sh[d] + nb > 64 ? w2[d] : 0u;
      const uint64_t w01 = ((uint64_t)v1 << 32) | w0[d];
      uint64_t r = (w01 >> sh[d]) | (sh[d] ? (uint64_t)v2 << (64 - sh[d]) : 0ull);
      uint32_t e = (v2 >> sh[d]) & 1u;                // bit 64 of the row's string
      if (nb < 64) r &= (1ull << nb) - 1ull;
      if (nb < 65) e = 0u;
      if (!in_row[d]) { r = 0ull; e = 0u; }
      hi |= shl ? (uint32_t)(r >> 63) : e;            // with shl there are at most 64 bits before the shift
      lo |= r << shl;
    }
    const uint64_t u = lo | (lo >> 1) | ((uint64_t)hi << 63) | (lo >> 2) | ((uint64_t)hi << 62);
    uint32_t m = emc2_even_bits(u);
    if (len < 32) m &= (1u << len) - 1u;
    bits |= m << pos;
    pos += len;
    key += (uint64_t)len;
  }
  return bits;
}

// One granule of level l: which of its lines can hold a bit (line flags of the fine level), then the words of those.  All
// threads look at flags, 8 or 32 to a line; then a word each.
__device__ __forceinline__ void role_gather(const DevStack& st, int l, uint32_t blk) {
  __shared__ uint32_t act_s[4], old_s[4], sum_s[4];
  const DevLevel& in = st.lv[l - 1];
  const DevLevel& lv = st.lv[l];
  const int lines = lv.words >> EMC2_LINE_SHIFT, subs = 256 / lines;     // 8 and 32, or 32 and 8
  const int wave = threadIdx.x >> 6;
  const int64_t line0 = (int64_t)blk * lines;
  {
    const int line = (int)threadIdx.x / subs, sub = (int)threadIdx.x % subs;
    const uint32_t gox = (uint32_t)lv.g[0], goy = (uint32_t)lv.g[1], goz = (uint32_t)lv.g[2];
    const uint64_t k0 = (uint64_t)(line0 + line) << (5 + EMC2_LINE_SHIFT);
    uint64_t k1 = k0 + (32u << EMC2_LINE_SHIFT);
    if (k1 > (uint64_t)lv.cells) k1 = (uint64_t)lv.cells;
    bool any = false;
    if (k0 < k1) {
      const uint64_t r0 = div_key(k0, gox), r1 = div_key(k1 - 1, gox);
      const uint32_t nc = (uint32_t)(r1 - r0 + 1) * 9u;
      for (uint32_t c = (uint32_t)sub; c < nc; c += (uint32_t)subs) {
        const uint64_t row = r0 + c / 9u;
        const int d = (int)(c % 9u);
        const uint64_t t = div_key(row, goy);
        const int oy = (int)(row - t * goy);
        const uint64_t b = div_key(t, goz);
        const int oz = (int)(t - b * goz);
        const int iz = 2 * oz + d / 3 - 1, iy = 2 * oy + d % 3 - 1;
        if (iz < 0 || iz >= in.g[2] || iy < 0 || iy >= in.g[1]) continue;
        const int ox0 = row == r0 ? (int)(k0 - r0 * gox) : 0;
        const int ox1 = row == r1 ? (int)(k1 - 1 - r1 * gox) : (int)gox - 1;
        const int xs = 2 * ox0 - 1 < 0 ? 0 : 2 * ox0 - 1;
        const int xe = 2 * ox1 + 1 < in.g[0] ? 2 * ox1 + 1 : in.g[0] - 1;
        const uint64_t rb = ((b * in.g[2] + (uint64_t)iz) * in.g[1] + (uint64_t)iy) * in.g[0];
        // at most 512 output cells of a row, so at most 1 025 input cells: they touch up to three lines of 512
        const uint64_t f0 = emc2_line_of_key(rb + (uint64_t)xs), f1 = emc2_line_of_key(rb + (uint64_t)xe);
        uint32_t f = 0;
#pragma unroll
        for (int q = 0; q < 3; ++q) f |= in.flags[f0 + q < f1 ? f0 + q : f1];
        any |= f != 0u;
      }
    }
    // lines of this wave (64 / subs of them), a bit each
    const unsigned long long some = __ballot(any), was = __ballot(sub == 0 && lv.flags[line0 + line] != 0);
    uint32_t act = 0, old = 0;
    for (int q = 0; q < 64 / subs; ++q) {
      const unsigned long long m = ((1ull << subs) - 1ull) << (q * subs);     // subs is 8 or 32
      act |= (some & m) != 0ull ? 1u << q : 0u;
      old |= (was & m) != 0ull ? 1u << q : 0u;
    }
    if ((threadIdx.x & 63) == 0) {
      act_s[wave] = act;
      old_s[wave] = old;
    }
  }
  __syncthreads();
  uint32_t act = 0, old = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    act |= act_s[q] << (q * lines / 4);
    old |= old_s[q] << (q * lines / 4);
  }
  const uint32_t write = act | old;
  if ((int)threadIdx.x < lines && ((write >> threadIdx.x) & 1u)) lv.flags[line0 + threadIdx.x] = (lineflag_t)((act >> threadIdx.x) & 1u);
  uint32_t s = 0;
#pragma unroll
  for (int i = 0; i < kGranuleMax / 256; ++i) {
    const int wi = (int)threadIdx.x + 256 * i;
    const int line = wi >> EMC2_LINE_SHIFT;
    if (wi >= lv.words || !((write >> line) & 1u)) continue;
    const int64_t w = (int64_t)blk * lv.words + wi;
    const uint32_t bits = ((act >> line) & 1u) ? gather_word(in, lv, w) : 0u;
    lv.idx[w] = make_uint2(bits, 0u);
    s += __popc(bits);
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sum_s[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    s = sum_s[0] + sum_s[1] + sum_s[2] + sum_s[3];
    lv.sums[blk] = s;
    if (s) atomicAdd(&lv.supers[blk / kSuper], s);
  }
}

// x past the row's end goes on in the next row, plane, frame.
__device__ __forceinline__ void carry(int4& c, const DevLevel& lv) {
  while (c.w >= lv.g[0]) {
    c.w -= lv.g[0];
    if (++c.z >= lv.g[1]) {
      c.z = 0;
      if (++c.y >= lv.g[2]) {
        c.y = 0;
        ++c.x;
      }
    }
  }
}

// One granule of level l: prefix fields of its flagged words and the coordinates of their set bits.  In a small granule (a
// coarse level: few, dense words) a half wave takes a word, a lane its bit, so that a store writes consecutive rows; in a
// large one (many words, mostly empty) a thread walks the bits of its two words.  The other way round either costs more:
// level 3 of a 64-beam frame 13 us by walking and 9 so, the levels 1 of eight routed frames 43 us by walking and 48 so.
__device__ __forceinline__ void role_expand(const DevStack& st, int l, uint32_t blk) {
  __shared__ uint32_t wsum[4], word_s[kGranuleWords], pre_s[kGranuleWords];
  __shared__ int4 at_s[kGranuleWords];                                // (b, z, y, x) of a word's bit 0
  const DevLevel& lv = st.lv[l];
  const bool last = (int)blk == lv.units - 1;
  const int words = lv.words, wi = 2 * (int)threadIdx.x;              // two adjacent words, one line
  const int64_t w0 = (int64_t)blk * words + wi;
  const bool have = wi < words && lv.flags[w0 >> EMC2_LINE_SHIFT] != 0;
  if (!__syncthreads_or(have) && !last) return;
  uint4* p = reinterpret_cast<uint4*>(lv.idx + w0);
  uint4 v = have ? *p : make_uint4(0u, 0u, 0u, 0u);
  const uint32_t base = base_of(lv, blk);
  const uint32_t s = __popc(v.x) + __popc(v.z);
  const uint32_t inc = wave_scan(s);
  if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = inc;
  __syncthreads();
  uint32_t run = inc - s;                                             // rows of the granule before these words
  for (int j = 0; j < (int)(threadIdx.x >> 6); ++j) run += wsum[j];
  const uint32_t total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  if (last && threadIdx.x == 0) report_total(st, lv, base + total);
  if (have) {
    v.y = base + run;
    v.w = base + run + __popc(v.x);
    *p = v;
  }
  if (words == kGranuleMax) {
    if (s == 0u) return;
    int4 c = decode_key((uint64_t)w0 * 32, lv.g[0], lv.g[1], lv.g[2]);   // (b, z, y, x) of the first word's bit 0
    uint64_t bits = ((uint64_t)v.z << 32) | v.x;
    int at = 0;                                                          // bit position c refers to
    int64_t r = base + run;
    while (bits) {
      const int j = __ffsll((unsigned long long)bits) - 1;
      bits &= bits - 1;
      c.w += j - at;
      at = j;
      carry(c, lv);
      if (r < lv.cap) lv.coords[r] = c;
      ++r;
    }
    return;
  }
  if (wi < words) {
    word_s[wi] = v.x;
    word_s[wi + 1] = v.z;
    pre_s[wi] = base + run;
    pre_s[wi + 1] = base + run + __popc(v.x);
  }
  if ((int)threadIdx.x < words) at_s[threadIdx.x] = decode_key(((uint64_t)blk * words + threadIdx.x) * 32, lv.g[0], lv.g[1], lv.g[2]);
  __syncthreads();
  const int bit = threadIdx.x & 31;
#pragma unroll 4
  for (int i = (int)threadIdx.x >> 5; i < kGranuleWords; i += 8) {
    const uint32_t w = word_s[i];
    if (!((w >> bit) & 1u)) continue;
    const uint32_t r = pre_s[i] + __popc(w & ((1u << bit) - 1u));
    int4 c = at_s[i];
    c.w += bit;
    carry(c, lv);
    if ((int64_t)r < lv.cap) lv.coords[r] = c;
  }
}

// Every kernel map of every stack.  The blocks share the device's own row counts: map by map in 256-row pieces, an
// XCD's blocks (blockIdx % 8) taking a contiguous range of each map, so that neighbouring rows probe one L2.
__device__ __forceinline__ void role_probe(const Args& a, uint32_t blk, uint32_t blocks) {
  const int64_t x = blk & 7, at0 = blk >> 3, step = blocks >> 3;    // blocks is a multiple of 8
  int64_t at = at0;
  for (int s = 0; s < a.n_stacks; ++s) {
    const DevStack& st = a.st[s];
    for (int l = 0; l < st.n_levels; ++l) {
      const DevLevel& lv = st.lv[l];
      const int32_t n = *lv.n;
      const int64_t pieces = (n + 255) / 256, chunk = (pieces + 7) / 8;
#pragma unroll
      for (int kind = 0; kind < 2; ++kind) {
        int32_t* nbr = kind == 0 ? lv.down : lv.subm;
        if (!nbr) continue;
        const DevLevel& in = kind == 0 ? st.lv[l > 0 ? l - 1 : 0] : lv;
        const int32_t n_in = *in.n;
        for (; at < chunk; at += step) {
          const int64_t o = (x * chunk + at) * 256 + threadIdx.x;
          if (o >= n || x * chunk + at >= pieces) continue;
          if (kind == 0)
            emc2_probe_voxel<2>(o, lv.coords, lv.cap, in.idx, n_in, in.g[0], in.g[1], in.g[2], st.prm.n_batch, nbr);
          else
            emc2_probe_voxel<1>(o, lv.coords, lv.cap, in.idx, n_in, in.g[0], in.g[1], in.g[2], st.prm.n_batch, nbr);
        }
        at -= chunk;      // the remainder carries into the next map, so short maps do not idle blocks
      }
    }
  }
}

template <uint32_t ROLES>
__global__ void __launch_bounds__(256) k_stack_phase(const Args a) {
  int j = 0;
  while (j + 1 < a.n_jobs && blockIdx.x >= a.job[j + 1].first) ++j;
  const int role = a.job[j].role, l = a.job[j].level;
  const uint32_t blk = blockIdx.x - a.job[j].first;
  const DevStack& st = a.st[a.job[j].stack];
#define EMC2_ROLE(R, CALL) if ((ROLES >> R) & 1u) { if (role == R) { CALL; return; } }
  EMC2_ROLE(R_CLEAR, role_clear(st.lv[0], blk))
  EMC2_ROLE(R_ZERO, role_zero(st))
  EMC2_ROLE(R_MARK, role_mark(a, st, blk))
  EMC2_ROLE(R_SUM, role_sum(st.lv[0], blk))
  EMC2_ROLE(R_PREFIX, role_prefix(st, st.lv[0], blk))
  EMC2_ROLE(R_SCATTER, role_scatter(a, st, blk))
  EMC2_ROLE(R_MEAN, role_mean(st, blk))
  EMC2_ROLE(R_GATHER, role_gather(st, l, blk))
  EMC2_ROLE(R_EXPAND, role_expand(st, l, blk))
  EMC2_ROLE(R_PROBE, role_probe(a, blk, gridDim.x - a.job[j].first))
#undef EMC2_ROLE
}

// A small cloud on a small grid in ONE launch: a level of at most kPrefixTiles tiles and kSmallCloud points.  The whole index fits the
// LDS of a CU, so every block of the launch builds all of it (bits, and ranks of their words) from all the points, and then
// takes a share of the voxels, from their points to their kernel-map entries, which it looks up in its own copy: nothing
// waits for another block.  On 200 000 cells, with the convolution behind it, as a graph, us, phases / so: 1 100 points 31 / 18,
// 2 000 32 / 19, 8 000 36 / 25, 15 000 36 / 31 (all blocks read all points).  A cloud of fewer points than the block has threads, or of
// more than 15 a thread, keeps the phases; neither line is where this stops paying: 3 points 25 / 16, 500 30 / 18, 900 31 / 18, 16 384 35 / 32.
constexpr int kSmallThreads = 1024, kSmallPer = 15;
constexpr int64_t kSmallCloud = kSmallThreads * kSmallPer;
constexpr int kSmallBlocks = 32;
constexpr int kSmallShare = (int)kSmallCloud / kSmallBlocks + 1;    // voxels of a block
constexpr int kSmallWords = kPrefixTiles * EMC2_SCAN_TILE;

__global__ void __launch_bounds__(kSmallThreads) k_stack_small(const Args a) {
  __shared__ uint32_t bits_s[kSmallWords];
  __shared__ uint16_t pre_s[kSmallWords];                             // voxels before each word: at most kSmallCloud
  __shared__ uint32_t wsum[kSmallThreads / 64];
  __shared__ uint32_t cnt_s[kSmallShare];                             // points of each voxel of the share, the first of them, the sum
  __shared__ uint16_t first_s[EMC2_VOX_STASH][kSmallShare];           // of the others
  __shared__ float rest_s[4][kSmallShare];
  const DevStack& st = a.st[blockIdx.y];
  const DevLevel& lv = st.lv[0];
  const int t = threadIdx.x, n_points = (int)a.n_points;
  constexpr int WPT = kSmallWords / kSmallThreads;                    // words a thread: half a line
  uint32_t key[kSmallPer];                                            // cell of each of the thread's points (-1: dropped)
  float4 pt[kSmallPer];
#pragma unroll
  for (int j = 0; j < kSmallPer; ++j) {
    key[j] = 0xffffffffu;
    if (j * kSmallThreads < n_points) {                               // uniform
      const PointCell pc = locate(a.points, st.batch, j * kSmallThreads + t, n_points, st.prm);
      if (pc.keep) key[j] = (uint32_t)pc.key;
      pt[j] = pc.p;
    }
  }
#pragma unroll
  for (int j = 0; j < WPT; ++j) bits_s[j * kSmallThreads + t] = 0u;
  if (t < kSmallShare) {
    cnt_s[t] = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) rest_s[j][t] = 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSmallPer; ++j)
    if (key[j] != 0xffffffffu) atomicOr(&bits_s[key[j] >> 5], 1u << (key[j] & 31u));
  __syncthreads();
  uint32_t b[WPT], s = 0;
#pragma unroll
  for (int j = 0; j < WPT; ++j) {
    b[j] = bits_s[t * WPT + j];
    s += __popc(b[j]);
  }
  const uint32_t inc = wave_scan(s);
  if ((t & 63) == 63) wsum[t >> 6] = inc;
  __syncthreads();
  uint32_t run = inc - s, total = 0;
#pragma unroll
  for (int j = 0; j < kSmallThreads / 64; ++j) {
    run += j < (t >> 6) ? wsum[j] : 0u;
    total += wsum[j];
  }
  const uint32_t in_line = s + __shfl_xor(s, 1, 64);
  // the index: the lines that hold bits and those that held some before, dealt to the blocks
  if ((t >> 1) % kSmallBlocks == (int)blockIdx.x && (t >> 8) < lv.units) {
    const bool stale = lv.flags[t >> 1] != 0;                         // a line's two threads are neighbours
    if (in_line || stale) {
      uint4* p = reinterpret_cast<uint4*>(lv.idx + t * WPT);
      uint32_t r = run;
#pragma unroll
      for (int j = 0; j < WPT; j += 2) {
        const uint32_t r1 = r + __popc(b[j]);
        p[j / 2] = make_uint4(b[j], r, b[j + 1], r1);
        r = r1 + __popc(b[j + 1]);
      }
    }
    if (!(t & 1) && (in_line != 0) != stale) lv.flags[t >> 1] = in_line != 0;
  }
#pragma unroll
  for (int j = 0; j < WPT; ++j) {
    pre_s[t * WPT + j] = (uint16_t)run;
    run += __popc(b[j]);
  }
  if (blockIdx.x == 0 && t == 0) report_total(st, lv, total);
  const int32_t n = (int64_t)total > lv.cap ? (int32_t)lv.cap : (int32_t)total;
  for (int64_t r = n + (int64_t)blockIdx.x * kSmallThreads + t; r < st.zero_rows; r += kSmallBlocks * kSmallThreads) {
    st.feats[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    st.counts[r] = 0;
  }
  __syncthreads();
  const int32_t v0 = (int32_t)((int64_t)n * blockIdx.x / kSmallBlocks), share = (int32_t)((int64_t)n * (blockIdx.x + 1) / kSmallBlocks) - v0;
#pragma unroll
  for (int j = 0; j < kSmallPer; ++j) {
    if (key[j] == 0xffffffffu) continue;
    const uint32_t v = pre_s[key[j] >> 5] + __popc(bits_s[key[j] >> 5] & ((1u << (key[j] & 31u)) - 1u)) - (uint32_t)v0;
    if (v >= (uint32_t)share) continue;
    const uint32_t pos = atomicAdd(&cnt_s[v], 1u);
    if (pos < EMC2_VOX_STASH) {
      first_s[pos][v] = (uint16_t)(j * kSmallThreads + t);
    } else {
      unsafeAtomicAdd(&rest_s[0][v], pt[j].x);
      unsafeAtomicAdd(&rest_s[1][v], pt[j].y);
      unsafeAtomicAdd(&rest_s[2][v], pt[j].z);
      unsafeAtomicAdd(&rest_s[3][v], pt[j].w);
    }
  }
  __syncthreads();
  // a thread a voxel
  if (t < share) {
    const int64_t r = v0 + t;
    const int32_t k = (int32_t)cnt_s[t];
    float4 q[EMC2_VOX_STASH];
    PointCell pc;
#pragma unroll
    for (int j = 0; j < EMC2_VOX_STASH; ++j) {
      q[j] = make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
      if (j < k) {
        const PointCell at = locate(a.points, st.batch, first_s[j][t], n_points, st.prm);
        q[j] = at.p;
        if (j == 0) pc = at;
      }
    }
    lv.coords[r] = pc.c;
    st.counts[r] = k;
    emc2_store_mean(r, q, make_float4(rest_s[0][t], rest_s[1][t], rest_s[2][t], rest_s[3][t]), k, st.feats, st.lp, st.feats_lp);
    if (lv.subm) {
      auto word = [&](uint64_t w) { return make_uint2(bits_s[w], (uint32_t)pre_s[w]); };
      emc2_probe_at<1>(r, pc.c, true, lv.cap, word, n, lv.g[0], lv.g[1], lv.g[2], lv.subm);
    }
  }
}

struct Phase {
  Args* a;
  void begin() { a->n_jobs = 0; a->blocks = 0; }
  void add(int role, int stack, int level, int64_t blocks) {
    if (blocks <= 0) return;
    Job& j = a->job[a->n_jobs++];
    j.role = role; j.stack = stack; j.level = level; j.first = a->blocks;
    a->blocks += (uint32_t)blocks;
  }
  template <uint32_t ROLES> void launch(hipStream_t s) {
    if (a->n_jobs) hipLaunchKernelGGL(k_stack_phase<ROLES>, dim3(a->blocks), dim3(256), 0, s, *a);
  }
};

// Host-side checks of one stack and its device description.
emc2_status describe(const emc2_stack& s, int64_t n_points, DevStack* d) {
  emc2_ctx* ctx = s.ctx;
  if (!s.d_feats || !s.d_counts || s.n_levels < 1 || s.n_levels > kLevels)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_build_stacks: null argument or n_levels outside [1, %d]", kLevels);
  emc2_status ok = emc2_voxel_args_ok(ctx, &s.spec, n_points, s.level[0].capacity, s.level[0].slot, "emc2_build_stacks");
  if (ok != EMC2_OK) return ok;
  if (s.d_feats_lp && s.lp_dtype != EMC2_F16 && s.lp_dtype != EMC2_BF16)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_build_stacks: lp_dtype must be F16 or BF16");
  if (s.expert > 2) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_build_stacks: expert %d beyond 2", s.expert);
  if (s.expert >= 0 && (!s.d_route || !s.d_slot))
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_build_stacks: a routed stack needs d_route and d_slot");
  memset(d, 0, sizeof(*d));
  d->prm = emc2_vox_params(&s.spec);
  d->expert = s.expert;
  d->n_levels = s.n_levels;
  d->lp = s.d_feats_lp ? (s.lp_dtype == EMC2_F16 ? 1 : 2) : 0;
  d->batch = s.d_batch;
  d->route = s.d_route;
  d->slot = s.d_slot;
  d->group_batch = s.d_group_batch;
  d->feats = (float4*)s.d_feats;
  d->counts = s.d_counts;
  d->feats_lp = s.d_feats_lp;
  d->stash = ctx->stash;
  d->stash_pitch = ctx->max_voxels;
  d->first = ctx->first;
  d->dev_words = ctx->dev_words;
  d->zero_rows = n_points < s.level[0].capacity ? n_points : s.level[0].capacity;
  int32_t g[3] = {s.spec.grid[0], s.spec.grid[1], s.spec.grid[2]};
  uint32_t* sums = ctx->stack_sums;
  uint32_t* sums_end = ctx->stack_sums + ctx->n_stack_sums;
  for (int l = 0; l < s.n_levels; ++l) {
    const emc2_stack_level& L = s.level[l];
    if (l > 0)
      for (int a = 0; a < 3; ++a) g[a] = (g[a] - 1) / 2 + 1;
    if (L.capacity < 1 || L.capacity > ctx->max_voxels || L.slot < 0 || L.slot >= ctx->n_slots || !L.d_coords || !L.d_n ||
        (l > 0 && !L.d_down_nbr) || (l == 0 && L.d_down_nbr))
      return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_build_stacks: level %d: bad capacity, slot or pointers", l);
    for (int q = 0; q < l; ++q)
      if (s.level[q].slot == L.slot) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_build_stacks: levels share slot %d", L.slot);
    DevLevel& v = d->lv[l];
    v.idx = ctx->slots[L.slot];
    v.flags = emc2_slot_flags(ctx, v.idx);
    v.coords = (int4*)L.d_coords;
    v.n = L.d_n;
    v.subm = L.d_subm_nbr;
    v.down = L.d_down_nbr;
    v.cap = L.capacity;
    for (int a = 0; a < 3; ++a) v.g[a] = g[a];
    v.cells = (int64_t)g[0] * g[1] * g[2] * s.spec.n_batch;
    const int64_t words = emc2_div_up(v.cells, 32);
    v.words = l == 0 ? EMC2_SCAN_TILE : emc2_div_up(words, kGranuleWords) <= kSmallGranules ? kGranuleWords : kGranuleMax;
    const int64_t units = emc2_div_up(words, v.words);
    v.units = (int32_t)units;
    v.sums = sums;
    v.supers = sums + units;
    sums += units + emc2_div_up(units, kSuper);
    if (sums > sums_end) return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_build_stacks: scan scratch too small for this stack");
  }
  return EMC2_OK;
}

// The slots now describe this stack's levels: only once every stack of the call has passed its checks, since none is
// built when one is refused.
void publish(const emc2_stack& s, const DevStack& d) {
  for (int l = 0; l < s.n_levels; ++l) {
    SlotMeta& m = s.ctx->meta[s.level[l].slot];
    for (int a = 0; a < 3; ++a) m.grid[a] = d.lv[l].g[a];
    m.n_batch = s.spec.n_batch;
    m.valid = true;
  }
}

}  // namespace

extern "C" emc2_status emc2_build_stacks(const emc2_stack* stacks, int32_t n_stacks, const float* d_points, int64_t n_points,
                                         void* stream) {
  if (!stacks || n_stacks < 1) return EMC2_ERR_INVALID_ARG;
  for (int i = 0; i < n_stacks; ++i)
    if (!stacks[i].ctx) return emc2_fail(stacks[0].ctx, EMC2_ERR_INVALID_ARG, "emc2_build_stacks: stack %d has no context", i);
  emc2_ctx* ctx0 = stacks[0].ctx;
  if (n_stacks > kStacks) return emc2_fail(ctx0, EMC2_ERR_UNSUPPORTED, "emc2_build_stacks: more than %d stacks", kStacks);
  if (n_points < 0 || (n_points > 0 && !d_points)) return emc2_fail(ctx0, EMC2_ERR_INVALID_ARG, "emc2_build_stacks: bad points");
  for (int i = 0; i < n_stacks; ++i) {
    if (stacks[i].spec.stride_f != stacks[0].spec.stride_f)
      return emc2_fail(ctx0, EMC2_ERR_INVALID_ARG, "emc2_build_stacks: stacks read the same points: one stride_f");
    for (int q = 0; q < i; ++q)
      if (stacks[q].ctx == stacks[i].ctx)
        return emc2_fail(ctx0, EMC2_ERR_INVALID_ARG, "emc2_build_stacks: two stacks on one context (they share its scratch)");
  }
  Args a;
  a.points = d_points;
  a.n_points = n_points;
  a.n_stacks = n_stacks;
  int deepest = 1;
  for (int i = 0; i < n_stacks; ++i) {
    const emc2_status st = describe(stacks[i], n_points, &a.st[i]);
    if (st != EMC2_OK) {
      if (stacks[i].ctx != ctx0) emc2_fail(ctx0, st, "%s", stacks[i].ctx->err);
      return st;
    }
    if (a.st[i].n_levels > deepest) deepest = a.st[i].n_levels;
  }
  for (int i = 0; i < n_stacks; ++i) publish(stacks[i], a.st[i]);
  hipStream_t s = (hipStream_t)stream;
  bool small = n_points >= kSmallThreads && n_points <= kSmallCloud;
  for (int i = 0; i < n_stacks; ++i) small = small && a.st[i].n_levels == 1 && a.st[i].expert < 0 && a.st[i].lv[0].units <= kPrefixTiles;
  if (small) {
    hipLaunchKernelGGL(k_stack_small, dim3(kSmallBlocks, (unsigned)n_stacks), dim3(kSmallThreads), 0, s, a);
    return emc2_check_hip(ctx0, hipGetLastError(), "emc2_build_stacks launch");
  }
  Phase p{&a};
  const int64_t point_blocks = emc2_div_up(n_points, 256);
  // maps of all levels: 2 048 blocks of 4 waves fill the chip; fewer where the capacities say so
  int64_t rows = 0;
  for (int i = 0; i < n_stacks; ++i)
    for (int l = 0; l < a.st[i].n_levels; ++l)
      rows += ((a.st[i].lv[l].subm ? 1 : 0) + (a.st[i].lv[l].down ? 1 : 0)) * emc2_div_up(a.st[i].lv[l].cap, 256);
  const int64_t probe_blocks = (rows < 2048 ? emc2_div_up(rows, 8) * 8 : 2048);
  const int last = deepest <= 3 ? 6 : deepest + 3;
  for (int ph = 1; ph <= last; ++ph) {
    p.begin();
    for (int i = 0; i < n_stacks; ++i) {
      const DevStack& d = a.st[i];
      const int64_t tiles = d.lv[0].units;
      if (ph == 1) { p.add(R_CLEAR, i, 0, emc2_div_up(tiles, 2)); p.add(R_ZERO, i, 0, 1); }
      if (ph == 2) p.add(R_MARK, i, 0, point_blocks);
      if (ph == 3 && tiles > kPrefixTiles) p.add(R_SUM, i, 0, emc2_div_up(tiles, 4));   // the prefix pass of fewer sums them itself
      if (ph == 4) p.add(R_PREFIX, i, 0, emc2_div_up(tiles, kPrefixTiles));
      if (ph == 5) p.add(R_SCATTER, i, 0, point_blocks);
      if (ph == 6) p.add(R_MEAN, i, 0, emc2_div_up(d.zero_rows, 256));
      if (ph - 2 >= 1 && ph - 2 < d.n_levels) p.add(R_GATHER, i, ph - 2, d.lv[ph - 2].units);
      if (ph - 3 >= 1 && ph - 3 < d.n_levels) p.add(R_EXPAND, i, ph - 3, d.lv[ph - 3].units);
    }
    if (ph == last && rows > 0) p.add(R_PROBE, 0, 0, probe_blocks);
#define BITS(R) (1u << R)
    switch (ph) {
      case 1: p.launch<BITS(R_CLEAR) | BITS(R_ZERO)>(s); break;
      case 2: p.launch<BITS(R_MARK)>(s); break;
      case 3: p.launch<BITS(R_SUM) | BITS(R_GATHER)>(s); break;
      case 4: p.launch<BITS(R_PREFIX) | BITS(R_GATHER) | BITS(R_EXPAND)>(s); break;
      case 5: p.launch<BITS(R_SCATTER) | BITS(R_GATHER) | BITS(R_EXPAND)>(s); break;
      // the last phase, at 6 or later, gathers and expands nothing any more: its kernel carries no other role's registers
      case 6:
        if (ph == last) p.launch<BITS(R_MEAN) | BITS(R_PROBE)>(s);
        else p.launch<BITS(R_MEAN) | BITS(R_GATHER) | BITS(R_EXPAND)>(s);
        break;
      default:
        if (ph == last) p.launch<BITS(R_PROBE)>(s);
        else p.launch<BITS(R_GATHER) | BITS(R_EXPAND)>(s);
        break;
    }
#undef BITS
  }
  return emc2_check_hip(ctx0, hipGetLastError(), "emc2_build_stacks launch");
}
