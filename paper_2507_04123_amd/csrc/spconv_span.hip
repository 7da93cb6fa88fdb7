// Submanifold convolution on the matrix cores, rows staged by producer waves (paper Sec. 3.5 sparse convolution over the
// non-empty voxels; Sec. 3.6 keeping data on chip between dependent steps).
//
// Voxels are indexed in ascending order of their linear cell key (x fastest).  The three taps of one (dz, dy) pair -- a
// group, kx = 0, 1, 2 -- therefore read input rows that differ by one position along x: for a run of consecutive output
// rows they touch nearly the same short interval [lo, hi] of input rows.  A block owns a tile of 64 * MT consecutive output
// rows and fetches that interval ONCE per group, as one contiguous run of feature rows, into LDS; each tap then reads its
// operand from there through a per-row offset.  Absent neighbours read a zeroed row.
//
// What bounds it and why the work is split this way.  The same kernel with every wave doing everything (rows through
// registers into a tile of its own) spent 42 % of a wave's time in the matrix phase: issuing the loads of the next group
// stalled a wave for 1 100-1 500 cycles (a CU takes a 1 KB load every ~20 cycles, and an in-order wave cannot issue matrix
// instructions behind a load that has not been accepted), moving the rows into LDS cost 650-840 more, analysis and weight
// copies 350, the barrier 550.  Here four waves (one per SIMD) only compute and four only feed them: the producers find the
// intervals, turn kernel-map entries into LDS offsets, and move rows and weights to LDS with direct global -> LDS loads, one
// pass ahead.  The computing waves hold 16 * MT rows by COUT columns of accumulators each and read nothing but LDS.  A block
// stays and walks over its tiles, so that a tile's first pass is fetched while the last tile's results are stored.
// What a pass of 384 rows costs now: 3 000 cycles of computing (144 matrix instructions, 2 304 if back to back), against
// ~3 500 of feeding it.  Neither is a unit's rate: the loads into LDS (74 KB) take 16.4 cycles a KB, 1 200, when issued without
// a stop, the operand reads (240 KB) 4.2, 1 000, and a third more for bank conflicts; side by side the two do not slow each
// other (measured on kernels of only reads, only loads, both).  What is left of the 3 500 is the wait for a pass's loads, which
// are one pass ahead, with the analysis of map entries and the offsets in front of them.  (LdsUtil, 28 %, counts 4 cycles a
// read and no load into LDS.)  Tried against it: the 32x32x16 instructions (computing 2 750, feeding the same: no gain),
// weights straight from global memory into registers (longer: the vector-memory path takes them at the rate of the rows),
// separate waves for loads and for the map (2 + 2: longer), the map read by the computing waves (spills), an order of tiles that
// keeps neighbouring planes in one L2 (no gain).
// 64 -> 64, us before / now: 70 k rows 33 / 25-28, 223 k 65 / 58, 248 k bf16 71 / 60, 573 k 142 / 107, 852 k 210 / 161.
// 128 -> 128 (bf16) on the register-direct kernel (whole taps at a time then), / here:
// 4 k rows 36 / 19, 32 k 39 / 26, 48 k 70 / 39, 67 k 104 / 71; 29 k rows of a sparse frame 33 / 39: a tile across two planes needs
// three passes for some groups, up to 30 in all where the others have 12-18, and with a tile a block it sets the time.
// 128 -> 128 spills 302 scalar registers into vector lanes (64 -> 64 none).
//
// One pass is what is computed between two barriers.  Normally a group is one pass.  A group whose interval does not fit
// the row buffer is split into two passes of half of the tile's rows if each half's interval fits (next to a denser plane
// the interval is up to twice the rows), else into three passes, one per tap, that gather exactly the rows the tap names.
// Rows and taps that are not a pass's own read the zeroed row, so that there is one form of the matrix code (branches
// around it make the compiler keep two copies of the accumulators).  With finite weights results never depend on which: an
// output row adds its taps in ascending order in all three forms, and what reads the zeroed row adds nothing.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "common.h"
#include "spconv_mfma.h"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native vector: real loads and stores
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int DT> struct MmaS;
template <> struct MmaS<EMC2_F16> {
  static __device__ __forceinline__ floatx4 run(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t cvt2(float x, float y) {   // round to nearest even
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{x, y}), half2v));
  }
};
template <> struct MmaS<EMC2_BF16> {
  static __device__ __forceinline__ floatx4 run(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t cvt2(float x, float y) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{x, y}), bf16x2));
  }
};

constexpr int kSpanThreads = 512;    // waves 0-3 compute, waves 4-7 feed them
constexpr int64_t kSpanCUs = 256;    // compute units of the part; one block fits each
// A pass takes 64 input channels: 128 are two passes a group, the lower channels of its three taps and then the upper.
constexpr int kPassChannels = 64;

// TR: rows of one of the two row buffers, what the LDS holds beside the rest.  A tile is 64 * mt rows, mt in
// [MT0, MT0 + 4); kFirst, kNext: what a block's first tile (with the launch's start and end) and each further one cost,
// measured in 0.1 us.
template <int CIN, int COUT> struct SpanCfg;
template <> struct SpanCfg<64, 64> {    // (heights 1 and 2 cost 6.3 and 7.4 us a tile and were never the best by more than 1 us)
  static constexpr int TR = 400, MT0 = 3, MTS = 4;
  static constexpr uint32_t kFirst[MTS] = {165, 170, 185, 215}, kNext[MTS] = {87, 110, 136, 165};
};
template <> struct SpanCfg<128, 128> {
  static constexpr int TR = 224, MT0 = 1, MTS = 3;
  static constexpr uint32_t kFirst[MTS] = {185, 215, 250}, kNext[MTS] = {180, 260, 330};
};

template <int CIN, int COUT> struct SpanLds {
  static constexpr int CH = kPassChannels / 8;                // 16-byte pieces of a row in a pass
  static constexpr int KS = kPassChannels / 32;               // steps of a tap in a pass
  static constexpr int KH = CIN / kPassChannels;              // passes that make up the channels
  static constexpr int W16 = KS * (COUT / 16) * 64;           // 16-byte weight pieces per tap
  static constexpr int TR = SpanCfg<CIN, COUT>::TR, MTM = SpanCfg<CIN, COUT>::MT0 + SpanCfg<CIN, COUT>::MTS - 1;
  u32x4 w[2][3 * W16];               // weights of a group
  u32x4 rows[2][(TR + 1) * CH];      // rows of a pass; row TR is zero
  uint16_t off[2][4][16][MTM][4];    // [pass][computing wave][m][mt][tap]: where output row 64*mt + 16*wave + m reads
  u32x2 part[2][9][4][MTM];          // [tile][group][producer][mt]: lowest and highest row named (0xffffffff, -1: none)
  float scale[COUT], shift[COUT];
};

// Pieces of a row are swapped about so that 16 consecutive rows, read at the same piece, fall on the 16 different 16-byte
// columns of the 64 banks.
template <int CH> __device__ __forceinline__ uint32_t swizzle_of(uint32_t row) { return (row / (16 / CH)) % CH; }

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63; }

// The barrier between passes.  A wave has its LDS accesses behind it when it arrives, and a producer, which calls
// loads_done() first, its loads into LDS; stores of results and loads of kernel-map entries stay in flight.
__device__ __forceinline__ void sync_all() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ void loads_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ void load_to_lds16(const void* src_lane, u32x4* dst_wave) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src_lane,
                                   (__attribute__((address_space(3))) void*)dst_wave, 16, 0, 0);
}

// minimum / maximum over each row of 16 lanes
__device__ __forceinline__ uint32_t row_min(uint32_t v) {
  v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, true));
  v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x124, 0xf, 0xf, true));
  v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x122, 0xf, 0xf, true));
  return min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x121, 0xf, 0xf, true));
}
__device__ __forceinline__ int32_t row_max(int32_t v) {
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true));
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, true));
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x122, 0xf, 0xf, true));
  return max(v, __builtin_amdgcn_mov_dpp(v, 0x121, 0xf, 0xf, true));
}

// How a tile's nine groups are run; the same in every wave.  Lanes 4g .. 4g+3 hold group g; the masks have its bit at 4g.
struct Plan {
  uint32_t lo_a, lo_b;            // intervals of the tile's first and second half (lane 4g: group g)
  int32_t hi_a, hi_b;
  unsigned long long any, one, two;   // some entry; one pass; two passes (neither: three)
};

template <int CIN, int COUT, int MT>
__device__ __forceinline__ Plan make_plan(const SpanLds<CIN, COUT>& s, uint32_t tb) {
  constexpr int TR = SpanLds<CIN, COUT>::TR;
  constexpr int H = (MT + 1) / 2;
  const uint32_t l = lane_id() < 36 ? lane_id() : 35;
  Plan p;
  p.lo_a = p.lo_b = 0xffffffffu;
  p.hi_a = p.hi_b = -1;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const u32x2 v = s.part[tb][l / 4][l % 4][mt];
    if (mt < H) {
      p.lo_a = min(p.lo_a, v[0]);
      p.hi_a = max(p.hi_a, (int32_t)v[1]);
    } else {
      p.lo_b = min(p.lo_b, v[0]);
      p.hi_b = max(p.hi_b, (int32_t)v[1]);
    }
  }
#define EMC2_QUAD(V, OP, T)                                                                \
  V = OP(V, (T)__builtin_amdgcn_update_dpp(0, (int)V, 0xB1, 0xf, 0xf, false));             \
  V = OP(V, (T)__builtin_amdgcn_update_dpp(0, (int)V, 0x4E, 0xf, 0xf, false));
  EMC2_QUAD(p.lo_a, min, uint32_t) EMC2_QUAD(p.lo_b, min, uint32_t)
  EMC2_QUAD(p.hi_a, max, int32_t) EMC2_QUAD(p.hi_b, max, int32_t)
#undef EMC2_QUAD
  const bool in = lane_id() < 36 && (lane_id() & 3) == 0;
  const bool a = p.hi_a >= 0, b = p.hi_b >= 0;
  const uint32_t lo = min(p.lo_a, p.lo_b);
  const int32_t hi = max(p.hi_a, p.hi_b);
  p.any = __ballot(in && (a || b));
  p.one = __ballot(in && (a || b) && (uint32_t)hi - lo < (uint32_t)TR);
  p.two = __ballot(in && (!a || (uint32_t)p.hi_a - p.lo_a < (uint32_t)TR) && (!b || (uint32_t)p.hi_b - p.lo_b < (uint32_t)TR));
  return p;
}

// One pass of a computing wave: three taps of its MT 16-row tiles.  Operands of a step (one tap, 32 channels) are read
// while the step before is multiplied.  The weights are the first operand, so that a lane ends up with four consecutive
// channels of one row.
template <int DT, int CIN, int COUT, int MT>
__device__ __forceinline__ void compute(const SpanLds<CIN, COUT>& s, uint32_t rb, uint32_t wb, uint32_t wave,
                                        floatx4 (&acc)[MT][COUT / 16]) {
  constexpr int KS = SpanLds<CIN, COUT>::KS, NT = COUT / 16, STEPS = 3 * KS, READS = MT + NT;
  const uint32_t lane = lane_id(), q16 = (lane >> 4) * 16;
  const char* rows = reinterpret_cast<const char*>(s.rows[rb]);
  const u32x4* w = s.w[wb] + lane;
  u32x2 of[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) of[i] = *reinterpret_cast<const u32x2*>(s.off[rb][wave][lane & 15][i]);
  u32x4 a[2][MT], b[2][NT];
#define EMC2_READ(STEP)                                                                                                  \
  {                                                                                                                      \
    _Pragma("unroll") for (int j = 0; j < NT; ++j) b[(STEP) & 1][j] = w[((STEP) * NT + j) * 64];                         \
    _Pragma("unroll") for (int i = 0; i < MT; ++i) {                                                                     \
      const uint32_t o_ = (STEP) / KS == 0 ? of[i][0] & 0xffffu : (STEP) / KS == 1 ? of[i][0] >> 16 : of[i][1];          \
      a[(STEP) & 1][i] = *reinterpret_cast<const u32x4*>(rows + (o_ ^ (q16 + 64u * ((STEP) % KS))));                     \
    }                                                                                                                    \
  }
  EMC2_READ(0)
  __builtin_amdgcn_sched_group_barrier(0x100, MT + READS, 0);
#pragma unroll
  for (int st = 0; st < STEPS; ++st) {
    if (st + 1 < STEPS) EMC2_READ(st + 1)
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = MmaS<DT>::run(b[st & 1][j], a[st & 1][i], acc[i][j]);
    constexpr int PER = MT * NT / READS > 0 ? MT * NT / READS : 1;   // matrix instructions per read
    if (st + 1 < STEPS) {
#pragma unroll
      for (int r = 0; r < READS; ++r) {
        __builtin_amdgcn_sched_group_barrier(0x008, PER, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      if (MT * NT > PER * READS) __builtin_amdgcn_sched_group_barrier(0x008, MT * NT - PER * READS, 0);
    } else {
      __builtin_amdgcn_sched_group_barrier(0x008, MT * NT, 0);
    }
  }
#undef EMC2_READ
}

// Folded affine, ReLU and rounding in registers, then 16-byte pieces of rows: lane (m, q) holds channels 16j + 4q .. + 3 of
// row m; one lane swap per pair of column tiles leaves it eight consecutive channels.  (ReLU by a compile-time switch: as a
// branch per value it cost 4 000 cycles a tile.)
template <int DT, int CIN, int COUT, int MT, bool RELU>
__device__ __forceinline__ void finish_tile(const SpanLds<CIN, COUT>& s, floatx4 (&acc)[MT][COUT / 16], uint32_t row0, uint32_t n_out,
                                            uint16_t* __restrict__ out) {
  const uint32_t m = lane_id() & 15, q = lane_id() >> 4;
  char* base = reinterpret_cast<char*>(out) + (int64_t)row0 * (COUT * 2);      // the same for the whole wave
  const uint32_t at = m * (COUT * 2) + 16 * (2 * (q & 1) + (q >> 1));
  const bool whole = row0 + 64 * (MT - 1) + 16 <= n_out;
#pragma unroll
  for (int jp = 0; jp < COUT / 32; ++jp) {
    floatx4 sc[2], sh[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      sc[e] = *reinterpret_cast<const floatx4*>(s.scale + 16 * (2 * jp + e) + 4 * q);
      sh[e] = *reinterpret_cast<const floatx4*>(s.shift + 16 * (2 * jp + e) + 4 * q);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      u32x2 h[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        floatx4 v = acc[mt][2 * jp + e];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[i] = fmaf(v[i], sc[e][i], sh[e][i]);
          if constexpr (RELU) v[i] = fmaxf(v[i], 0.f);   // NaN -> 0
        }
        h[e] = u32x2{MmaS<DT>::cvt2(v[0], v[1]), MmaS<DT>::cvt2(v[2], v[3])};
      }
      const u32x2 x = __builtin_amdgcn_permlane16_swap(h[0][0], h[1][0], false, false);
      const u32x2 y = __builtin_amdgcn_permlane16_swap(h[0][1], h[1][1], false, false);
      if (whole || row0 + 64 * mt + m < n_out)
        *reinterpret_cast<u32x4*>(base + 64 * mt * (COUT * 2) + 64 * jp + at) = u32x4{x[0], y[0], x[1], y[1]};
    }
  }
}
template <int DT, int CIN, int COUT, int MT>
__device__ __forceinline__ void store_tile(const SpanLds<CIN, COUT>& s, int epilogue, floatx4 (&acc)[MT][COUT / 16], uint32_t row0,
                                           uint32_t n_out, uint16_t* __restrict__ out) {
  if (epilogue == EMC2_EPI_AFFINE_RELU) finish_tile<DT, CIN, COUT, MT, true>(s, acc, row0, n_out, out);
  else finish_tile<DT, CIN, COUT, MT, false>(s, acc, row0, n_out, out);
}

// Tiles tile0, tile0 + step, .. below tile_end, each of 64 * MT rows.
template <int DT, int CIN, int COUT, int MT>
__device__ __forceinline__ void computing_wave(const SpanLds<CIN, COUT>& s, uint32_t wave, int epilogue, uint32_t tile0, uint32_t step,
                                               uint32_t tile_end, uint32_t n_out, uint16_t* __restrict__ out) {
  constexpr int NT = COUT / 16;
  floatx4 acc[MT][NT];
  uint32_t rb = 0, wb = 0, tb = 0;
  for (uint32_t tile = tile0; tile < tile_end; tile += step, tb ^= 1) {
    sync_all();                                    // the tile's intervals are in LDS
    const Plan p = make_plan<CIN, COUT, MT>(s, tb);
    if (tile != tile0) store_tile<DT, CIN, COUT, MT>(s, epilogue, acc, (tile - step) * (64 * MT) + 16 * wave, n_out, out);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    unsigned long long todo = p.any;
    uint32_t left = 0;                             // passes of the group, the same number for each share of the channels
    while (todo != 0ull) {
      const unsigned long long bit = todo & (0ull - todo);
      const uint32_t kinds = (p.one & bit) ? 1 : (p.two & bit) ? 2 : 3;
      if (left == 0) left = kinds * SpanLds<CIN, COUT>::KH;
      sync_all();
      compute<DT, CIN, COUT, MT>(s, rb, wb, wave, acc);
      rb ^= 1;
      --left;
      if (left == 0 || left == kinds) wb ^= 1;     // the next pass has other weights
      if (left == 0) todo ^= bit;
    }
    if (tile + step >= tile_end) store_tile<DT, CIN, COUT, MT>(s, epilogue, acc, tile * (64 * MT) + 16 * wave, n_out, out);
  }
}

// The waves that feed: producer w looks after the rows of computing wave w, 64*mt + 16*w + m of a tile (lane = 16*mt + m,
// mt 4 and 5 in a second register).  The next tile's entries of a group are requested as soon as this tile's are done with and
// looked through two groups later; nothing waits for them but what uses them.
template <int DT, int CIN, int COUT, int MT>
__device__ __forceinline__ void feeding_wave(SpanLds<CIN, COUT>& s, uint32_t w, const uint16_t* __restrict__ in,
                                             const u32x4* __restrict__ wp, const int32_t* __restrict__ nbr, int64_t capacity,
                                             int32_t n_in, int32_t* __restrict__ dev_flags, uint32_t tile0, uint32_t step,
                                             uint32_t tile_end, uint32_t n_out) {
  using L = SpanLds<CIN, COUT>;
  constexpr int TR = L::TR, CH = L::CH, RPI = 64 / CH, W16 = L::W16, G16 = 3 * W16;
  constexpr int H = (MT + 1) / 2, NE = (MT + 3) / 4;
  static_assert(TR % RPI == 0 && 64 * MT <= TR && TR * CH * 16 < 65536, "whole loads, a tap's rows and 16-bit offsets");
  static_assert(G16 % 256 == 0 && W16 % 64 == 0, "whole loads of weights for each producer, of one tap each");
  const uint32_t lane = lane_id(), m = lane & 15;
  // role in a load of RPI rows: row within it and piece of the row; a producer's loads are every fourth, which leaves the
  // swapping of pieces the same in all of them
  static_assert((4 * RPI / (16 / CH)) % CH == 0, "swizzle of every fourth load is the same");
  const uint32_t lrow = lane / CH, lpiece = (lane % CH) ^ swizzle_of<CH>(w * RPI + lrow);
  const uint32_t lat = lrow * (CIN * 2) + lpiece * 16;

  int32_t e[27][NE];              // kernel-map entries: of the current tile until its group is done, then of the next
  uint32_t row[NE], rows_in[NE];  // output row; rows that its entries may name (none for a row past n_out)
  int32_t seen = -1;              // largest entry seen
  uint32_t rb = 0, wb = 0;
#define EMC2_ROWS(TILE)                                                              \
  _Pragma("unroll") for (int i = 0; i < NE; ++i) {                                   \
    const uint32_t mt_ = 4 * i + (lane >> 4), r_ = (TILE) * (64 * MT) + 64 * mt_ + 16 * w + m; \
    const bool live_ = mt_ < MT && r_ < n_out;                                       \
    row[i] = live_ ? r_ : 0;                                                         \
    rows_in[i] = live_ ? (uint32_t)n_in : 0u;                                        \
  }
#define EMC2_ENTRIES(G)                                                              \
  _Pragma("unroll") for (int kx = 0; kx < 3; ++kx) {                                 \
    const int32_t* src_ = nbr + (int64_t)(3 * (G) + kx) * capacity;                  \
    _Pragma("unroll") for (int i = 0; i < NE; ++i) e[3 * (G) + kx][i] = src_[row[i]]; \
  }
  // rows [LO, HI] to the row buffer, from its start (rows past HI re-read row HI and are never referenced)
#define EMC2_FETCH(LO, HI)                                                                                        \
  {                                                                                                               \
    const uint32_t lo_ = (LO), last_ = (uint32_t)(HI) - lo_;                                                      \
    const char* base_ = in_h + (int64_t)lo_ * (CIN * 2);                                                          \
    uint32_t i_ = w;                                                                                              \
    for (; i_ * RPI + RPI <= last_ + 1; i_ += 4) load_to_lds16(base_ + i_ * (RPI * CIN * 2) + lat, s.rows[rb] + i_ * 64); \
    if (i_ * RPI <= last_)                                                                                        \
      load_to_lds16(base_ + min(i_ * RPI + lrow, last_) * (uint32_t)(CIN * 2) + lpiece * 16, s.rows[rb] + i_ * 64); \
  }
  // where each of this producer's rows reads at the taps of group G: tiles [M0, M1) in the interval that starts at LO, the
  // others and absent neighbours (-1, beyond any interval) the zeroed row
#define EMC2_OFFSET(R) ((R) * (CH * 16) | swizzle_of<CH>(R) * 16)
#define EMC2_OFFSETS(G, WHOLE, M0, M1, LO)                                                                             \
  _Pragma("unroll") for (int i = 0; i < NE; ++i) {                                                                \
    uint32_t o_[3];                                                                                               \
    const uint32_t mt_ = 4 * i + (lane >> 4);                                                                     \
    _Pragma("unroll") for (int kx = 0; kx < 3; ++kx) {                                                            \
      uint32_t at_ = min((uint32_t)e[3 * (G) + kx][i] - (LO), (uint32_t)TR);                                      \
      if (!(WHOLE)) at_ = mt_ >= (M0) && mt_ < (M1) ? at_ : (uint32_t)TR;                                         \
      o_[kx] = EMC2_OFFSET(at_);                                                                                  \
    }                                                                                                             \
    if (mt_ < MT) *reinterpret_cast<u32x2*>(s.off[rb][w][m][mt_]) = u32x2{o_[0] | o_[1] << 16, o_[2]};            \
  }
#define EMC2_WEIGHTS(G)                                                                                           \
  _Pragma("unroll") for (int i = 0; i < G16 / 256; ++i)                                                           \
    load_to_lds16(wp + (int64_t)((3 * (G) + (i * 4 + w) * 64 / W16) * L::KH + h) * W16 + (i * 4 + w) * 64 % W16 + lane, \
                  s.w[wb] + (i * 4 + w) * 64);

  // the rows that the entries of group G name, per 16 output rows; the entries are in registers
#define EMC2_ANALYSE(G, TB)                                                                                       \
  _Pragma("unroll") for (int i = 0; i < NE; ++i) {                                                                \
    uint32_t lo_ = 0xffffffffu;                                                                                   \
    int32_t hi_ = -1;                                                                                             \
    _Pragma("unroll") for (int kx = 0; kx < 3; ++kx) {                                                            \
      int32_t& j_ = e[3 * (G) + kx][i];                                                                           \
      seen = max(seen, j_);                                                                                       \
      j_ = (uint32_t)j_ < rows_in[i] ? j_ : -1;                                                                   \
      lo_ = min(lo_, (uint32_t)j_);                                                                               \
      hi_ = max(hi_, j_);                                                                                         \
    }                                                                                                             \
    lo_ = row_min(lo_);                                                                                           \
    hi_ = row_max(hi_);                                                                                           \
    if (m == 0 && 4 * i + (lane >> 4) < MT) s.part[TB][G][w][4 * i + (lane >> 4)] = u32x2{lo_, (uint32_t)hi_};     \
  }
  // waits for the entries of group G here, so that nothing that uses them waits for loads issued since
#define EMC2_ARRIVED(G)                                                                                           \
  _Pragma("unroll") for (int kx = 0; kx < 3; ++kx)                                                                \
    _Pragma("unroll") for (int i = 0; i < NE; ++i) asm volatile("" : "+v"(e[3 * (G) + kx][i]));

  EMC2_ROWS(tile0)
#pragma unroll
  for (int g = 0; g < 9; ++g) EMC2_ENTRIES(g)
#pragma unroll
  for (int g = 0; g < 9; ++g) EMC2_ANALYSE(g, 0)
  uint32_t tb = 0;
  for (uint32_t tile = tile0; tile < tile_end; tile += step, tb ^= 1) {
    sync_all();
    const Plan p = make_plan<CIN, COUT, MT>(s, tb);
    // the next tile's entries; past the last tile, its own again
    EMC2_ROWS(tile + step < tile_end ? tile + step : tile)
    // opaque: the addresses of 27 taps would otherwise stay alive from tile to tile, and spill
    asm volatile("" : "+s"(capacity));
#pragma unroll
    for (int g = 0; g < 9; ++g) {
      const unsigned long long bit = 1ull << (4 * g);
      // the next tile's entries of the last group but one have had a pass to arrive in
      if (g > 1) EMC2_ARRIVED(g - 2)
      if (p.any & bit) {
        const uint32_t lo_a = __builtin_amdgcn_readlane(p.lo_a, 4 * g), lo_b = __builtin_amdgcn_readlane(p.lo_b, 4 * g);
        const int32_t hi_a = __builtin_amdgcn_readlane(p.hi_a, 4 * g), hi_b = __builtin_amdgcn_readlane(p.hi_b, 4 * g);
#pragma unroll 1
        for (uint32_t h = 0; h < (uint32_t)L::KH; ++h) {       // the channels of the pass
          const char* in_h = reinterpret_cast<const char*>(in) + h * (kPassChannels * 2);
          if (h > 0) {
            loads_done();
            sync_all();
            rb ^= 1;
            wb ^= 1;
          }
          if (p.one & bit) {
            const uint32_t lo = min(lo_a, lo_b);
            EMC2_FETCH(lo, max(hi_a, hi_b))
            EMC2_WEIGHTS(g)
            __builtin_amdgcn_sched_barrier(0);
            EMC2_OFFSETS(g, true, 0, MT, lo)
          } else if (p.two & bit) {
            EMC2_FETCH(lo_a, hi_a)
            EMC2_WEIGHTS(g)
            __builtin_amdgcn_sched_barrier(0);
            EMC2_OFFSETS(g, false, 0, H, lo_a)
            loads_done();
            sync_all();
            rb ^= 1;
            EMC2_FETCH(lo_b, hi_b)
            __builtin_amdgcn_sched_barrier(0);
            EMC2_OFFSETS(g, false, H, MT, lo_b)
          } else {
            EMC2_WEIGHTS(g)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
              if (kx > 0) {
                loads_done();
                sync_all();
                rb ^= 1;
              }
              // row p of the buffer <- what output row p of the tile reads at this tap (absent: row 0, not referenced)
#pragma unroll
              for (int i = 0; i < NE; ++i) {
                const uint32_t mt = 4 * i + (lane >> 4);
                const uint32_t at = e[3 * g + kx][i] >= 0 ? 64 * mt + 16 * w + m : (uint32_t)TR;
                uint32_t o[3];
#pragma unroll
                for (int t = 0; t < 3; ++t) o[t] = t == kx ? EMC2_OFFSET(at) : EMC2_OFFSET((uint32_t)TR);
                if (mt < MT) *reinterpret_cast<u32x2*>(s.off[rb][w][m][mt]) = u32x2{o[0] | o[1] << 16, o[2]};
              }
#pragma unroll
              for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int q = 0; q < 16 / RPI; ++q) {
                  const int32_t j = __shfl(e[3 * g + kx][mt / 4], (mt % 4) * 16 + q * RPI + lrow, 64);
                  const uint32_t r0 = 64 * mt + 16 * w + q * RPI;
                  const uint32_t piece = (lane % CH) ^ swizzle_of<CH>(r0 + lrow);
                  load_to_lds16(in_h + (int64_t)max(j, 0) * (CIN * 2) + piece * 16, s.rows[rb] + r0 * CH);
                }
            }
          }
        }
        if (g > 1) EMC2_ANALYSE(g - 2, tb ^ 1)
        loads_done();
        EMC2_ENTRIES(g)
        sync_all();
        rb ^= 1;
        wb ^= 1;
      } else {
        if (g > 1) EMC2_ANALYSE(g - 2, tb ^ 1)
        EMC2_ENTRIES(g)
      }
    }
    EMC2_ANALYSE(7, tb ^ 1)
    EMC2_ANALYSE(8, tb ^ 1)
  }
#undef EMC2_ROWS
#undef EMC2_ENTRIES
#undef EMC2_FETCH
#undef EMC2_OFFSETS
#undef EMC2_OFFSET
#undef EMC2_WEIGHTS
#undef EMC2_ANALYSE
#undef EMC2_ARRIVED
  emc2_report_oob(__ballot(seen >= n_in), dev_flags);
}

template <int DT, int CIN, int COUT>
__global__ void __launch_bounds__(kSpanThreads, 2)
k_spconv_span(const uint16_t* __restrict__ in, const u32x4* __restrict__ wp, const float* __restrict__ scale,
              const float* __restrict__ shift, int epilogue, const int32_t* __restrict__ nbr,
              const int32_t* __restrict__ d_n_out, int64_t capacity_out, int32_t n_in, int32_t* __restrict__ dev_flags,
              uint16_t* __restrict__ out) {
  __shared__ SpanLds<CIN, COUT> s;
  static_assert(sizeof(s) <= 160 * 1024, "LDS of a CU");
  int64_t n64 = *d_n_out;
  if (n64 > capacity_out) n64 = capacity_out;
  if (n64 <= 0) return;
  const uint32_t n = (uint32_t)n64;
  // Tile height: the one with which the tiles of the slowest block cost least.
  using Cfg = SpanCfg<CIN, COUT>;
  const uint32_t step = gridDim.x / 8;
  uint32_t mt = 0, cost = 0xffffffffu;
#pragma unroll
  for (uint32_t i = 0; i < (uint32_t)Cfg::MTS; ++i) {
    const uint32_t rows = 64 * (Cfg::MT0 + i), tiles = (n + rows - 1) / rows, rounds = ((tiles + 7) / 8 + step - 1) / step;
    const uint32_t c = Cfg::kFirst[i] + (rounds - 1) * Cfg::kNext[i];
    if (c < cost) {
      cost = c;
      mt = Cfg::MT0 + i;
    }
  }
  // XCD-aware: workgroup b runs on XCD b % 8; XCD x walks over a contiguous range of tiles, its blocks side by side
  const uint32_t tiles = (n + 64 * mt - 1) / (64 * mt), chunk = (tiles + 7) / 8;
  const uint32_t first = (blockIdx.x % 8) * chunk, tile0 = first + blockIdx.x / 8;
  const uint32_t end = first + chunk < tiles ? first + chunk : tiles;
  if (tile0 >= end) return;          // uniform for the block
  for (uint32_t i = threadIdx.x; i < COUT; i += kSpanThreads) {
    s.scale[i] = epilogue != EMC2_EPI_NONE ? scale[i] : 1.f;
    s.shift[i] = epilogue != EMC2_EPI_NONE ? shift[i] : -0.f;   // x * 1 + -0 is x
  }
  constexpr int CH = SpanLds<CIN, COUT>::CH;
  if (threadIdx.x < 2 * CH) s.rows[threadIdx.x / CH][Cfg::TR * CH + threadIdx.x % CH] = u32x4{0u, 0u, 0u, 0u};
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#define EMC2_RUN(I)                                                                                                            \
  if constexpr (I < Cfg::MTS) {                                                                                                \
    if (mt == Cfg::MT0 + I) {                                                                                                  \
      constexpr int MT = Cfg::MT0 + I;                                                                                         \
      if (wave < 4) computing_wave<DT, CIN, COUT, MT>(s, wave, epilogue, tile0, step, end, n, out);                            \
      else feeding_wave<DT, CIN, COUT, MT>(s, wave - 4, in, wp, nbr, capacity_out, n_in, dev_flags, tile0, step, end, n);      \
      return;                                                                                                                  \
    }                                                                                                                          \
  }
  EMC2_RUN(0) EMC2_RUN(1) EMC2_RUN(2) EMC2_RUN(3)
#undef EMC2_RUN
}

template <int DT, int CIN, int COUT>
void launch_span(const void* d_in, const void* d_wp, const float* d_scale, const float* d_shift, int epilogue,
                 const int32_t* d_nbr, const int32_t* d_n_out, int64_t capacity_out, int32_t n_in, int32_t* dev_flags,
                 void* d_out, hipStream_t s) {
  // one block a CU; fewer where the capacity has fewer of the smallest tiles
  const int64_t tiles = emc2_div_up(emc2_div_up(capacity_out, 64 * SpanCfg<CIN, COUT>::MT0), 8) * 8;
  hipLaunchKernelGGL((k_spconv_span<DT, CIN, COUT>), dim3((unsigned)(tiles < kSpanCUs ? tiles : kSpanCUs)), dim3(kSpanThreads), 0, s,
                     (const uint16_t*)d_in, (const u32x4*)d_wp, d_scale, d_shift, epilogue, d_nbr, d_n_out, capacity_out, n_in,
                     dev_flags, (uint16_t*)d_out);
}

}  // namespace

// 64 -> 64 and 128 -> 128: at 32 channels a pass has a quarter of the matrix work for half of the bytes, and what a
// tile costs besides its passes shows (two blocks a CU, 1.0 M rows 97 us against 97-105 on the register-direct kernel, 304 k
// rows 43 against 39).
// Weights: the packed layout of the register-direct kernel (emc2_spconv_direct_pack).
bool emc2_spconv_span_supported(int cin, int cout) { return (cin == 64 && cout == 64) || (cin == 128 && cout == 128); }

void emc2_spconv_span_launch(emc2_dtype dtype, const void* d_in, const void* d_wp, const float* d_scale,
                             const float* d_shift, int epilogue, const int32_t* d_nbr, const int32_t* d_n_out,
                             int64_t capacity_out, int32_t n_in, int32_t* dev_flags, int cin, int cout, void* d_out,
                             hipStream_t stream) {
#define CASE(DTV, CI, CO)                                                                                           \
  if (dtype == DTV && cin == CI && cout == CO) {                                                                    \
    launch_span<DTV, CI, CO>(d_in, d_wp, d_scale, d_shift, epilogue, d_nbr, d_n_out, capacity_out, n_in, dev_flags, \
                             d_out, stream);                                                                        \
    return;                                                                                                         \
  }
  CASE(EMC2_F16, 64, 64) CASE(EMC2_BF16, 64, 64) CASE(EMC2_F16, 128, 128) CASE(EMC2_BF16, 128, 128)
#undef CASE
}
