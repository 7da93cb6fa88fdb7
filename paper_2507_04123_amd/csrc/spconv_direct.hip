// Register-direct MFMA sparse convolution (paper Sec. 3.5 sparse convolution over the non-empty voxels;
// Sec. 3.6 operator fusion).
//
// Measured on this part, the local data share serves a wave's 16-byte read in 4.2 cycles without bank conflicts and a
// 16-byte write in 13.8, per CU.  A gather-GEMM that stages the gathered rows in LDS
// (write the tile, read it back as the A operand, read the weights as the B operand) then spends more
// LDS cycles per tap than matrix-core cycles, and that -- not memory latency, not the matrix cores --
// bounds it.  This kernel keeps the gathered rows out of LDS altogether:
//
//   v_mfma_f32_16x16x32_{f16,bf16}: the A operand of lane (m = lane % 16, q = lane / 16) is the 8
//   consecutive input channels 8q .. 8q+7 of row m of the tile, i.e. 16 contiguous bytes of the feature
//   row nbr[k][o_m].  Four lanes cover 64 contiguous bytes of one row, so a single global_load_dwordx4
//   per (16-row tile, 32 channels) IS the A operand: global -> VGPR -> matrix core, nothing in between.
//   Absent neighbours read past the end of the input's buffer descriptor, which yields zeros (inputs of 4 GiB and more:
//   a zeroed row instead, an address select).
//
// LDS holds only the weights of the current and the next tap (packed in B-fragment order, copied once
// per block and tap, requested three taps ahead) and a small tile for the epilogue's transposition.
//
// A block is 4 waves; a wave owns 32 consecutive output rows (2 tiles of 16) and all Cout columns, so the fp32
// accumulators never leave registers.  Gathers run 3
// taps ahead of their use; kernel-map entries two (dz,dy) groups ahead.  Every load is unconditional so the
// compiler can count the loads in flight.  Shapes: 64 -> 64, and 64 -> 128 / 128 -> 128, where a tap's matrix work per gathered byte
// doubles and the kernel leaves the staged per-tap kernel behind by a third.  (32 -> 64 and 64 -> 32: spconv_resident.hip.)
//
// 128 input channels are taken in two shares, the lower 64 of a group's three taps and then the upper: the order in which
// the kernel of the submanifold maps adds, so that the map hint never changes a bit.  A row's two 128-byte lines are still
// read once each.  Against whole taps (83 KB of LDS, 360 registers, one block a CU; now 50 KB, 250, two): transposed 128 -> 128
// over 304 k rows 310 / 255 us, stride-2 over 69 k 104 / 93, over 27 k 35.4 / 38.0 (a block a CU: twice the barriers show; a
// barrier for every two steps, with 64 KB of weights, 36.9 there and 258 over 304 k).
//
// Leaving out: a block first reads all 27 map entries of its rows, keeps them in LDS, and runs only the (dz, dy) groups in which
// some row has one.  A stride-2 map leaves 31-41 % of the (group, 128 rows) pairs empty, a transposed one 52-62 % (a line of
// fine sites has one or two of three dy and dz).  Alone, us before / with it: transposed 64 -> 64 over 223 k rows 59 / 45
// (38 since the XCDs take the rows in runs).
// Submanifold maps (a fifth of the groups empty) and 128 output channels gain less than the longer way to the first operands costs
// (64 -> 128 over 67 k 50 / 52, 128 -> 128 in whole taps 103 / 113), so they keep the straight walk over the 27 taps.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "common.h"
#include "spconv_mfma.h"
#include "xcd_tiles.h"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native vector: real loads and stores
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int DT> struct MmaD;
template <> struct MmaD<EMC2_F16> {
  static __device__ __forceinline__ floatx4 run(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint16_t cvt(float v) { return __half_as_ushort(__float2half_rn(v)); }
};
template <> struct MmaD<EMC2_BF16> {
  static __device__ __forceinline__ floatx4 run(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint16_t cvt(float v) { return __builtin_bit_cast(uint16_t, __float2bfloat16(v)); }
};

constexpr int kDWaves = 4;
constexpr int kDThreads = kDWaves * 64;
constexpr int64_t kDGrid = 8192;   // blocks of a launch whose blocks loop over tiles: ten rounds of the chip at 3 blocks a CU

// Packed weight layout of this kernel: piece index ((k*KS + t)*NT + j)*64 + lane, lane = 16*q + n, holds the
// 8 values W[k][32t + 8q + e][16j + n], e = 0..7 -- the B operand of k-step t, column tile j.
__global__ void __launch_bounds__(256) k_pack_weights_direct(const uint16_t* __restrict__ w, int cin, int cout,
                                                             uint4* __restrict__ packed) {
  const int ks = cin / 32, nt = cout / 16;
  const int total = 27 * ks * nt * 64;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= total) return;
  const int lane = p & 63;
  int f = p >> 6;
  const int j = f % nt; f /= nt;
  const int t = f % ks; f /= ks;
  const int k = f;
  const int n = 16 * j + (lane & 15);
  const int c0 = 32 * t + 8 * (lane >> 4);
  const uint16_t* src = w + ((int64_t)k * cin + c0) * cout + n;
  uint32_t v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
    v[e] = (uint32_t)src[(2 * e) * cout] | ((uint32_t)src[(2 * e + 1) * cout] << 16);
  packed[p] = make_uint4(v[0], v[1], v[2], v[3]);
}

template <int CIN, int COUT, bool BUF> struct DirectCfg {
  // 16-row tiles per wave: fewer rows per wave mean fewer accumulators and operands in flight, so more
  // waves fit a SIMD and cover each other's stalls; more rows per wave reuse a weight fragment read more often
  static constexpr int MT = 2;
  // waves per SIMD the register allocator must leave room for, as many as no form spills at (the 128-channel shapes keep
  // 64 accumulators and as many operands in flight)
  static constexpr int MINW = CIN >= 128 || COUT >= 128 ? 2 : 3;
};

// Levels of at most so many tiles, a block a CU, walk straight over the 27 taps: there the entries' way to the first operands shows,
// with few neighbours to hide it: 64 -> 64 over 21 k rows 12.6 / 14; at 40 k, beyond the line, straight / leaving out 18.8 / 14.9.
constexpr int64_t kStraightTiles = 256;
constexpr int kRun = 4;                  // tiles of a run: 512 rows

// Rows of the input through a buffer descriptor: 32-bit offsets, and the hardware returns zero for an offset at or beyond
// the end without fetching anything, so an absent neighbour costs neither an address select nor a cache access.  64-beam
// frame 524 -> 512 us; transposed 64 -> 64 over 223 k rows, where seven entries of eight are absent, 65 -> 48 us.
__device__ __forceinline__ u32x4 buffer_row16(__amdgpu_buffer_rsrc_t rows, uint32_t byte) {
  return __builtin_amdgcn_raw_buffer_load_b128(rows, (int)byte, 0, 0);
}

template <int DT, int CIN, int COUT, bool LOOP, bool BUF>
__global__ void __launch_bounds__(kDThreads, (DirectCfg<CIN, COUT, BUF>::MINW))
k_spconv_direct(const uint16_t* __restrict__ in, const u32x4* __restrict__ wp, const float* __restrict__ scale,
                const float* __restrict__ shift, int epilogue, const int32_t* __restrict__ nbr,
                const int32_t* __restrict__ d_n_out, int64_t capacity_out, int32_t n_in, int32_t* __restrict__ dev_flags,
                const uint16_t* __restrict__ zrow, int64_t straight_tiles, uint16_t* __restrict__ out) {
  constexpr int KH = CIN > 64 ? CIN / 64 : 1; // shares of the channels, one after the other over the three taps of a group
  constexpr int KS = CIN / 32 / KH;           // k-steps per tap and share
  constexpr int NT = COUT / 16;               // 16-column tiles
  constexpr int MT = DirectCfg<CIN, COUT, BUF>::MT;   // 16-row tiles per wave
  constexpr int R = 16 * MT;                  // rows per wave
  static_assert(MT == 2, "the lane-swap broadcast below handles two tiles");
  constexpr int W16 = KS * NT * 64;           // 16-byte weight pieces per tap and share
  constexpr int WPT = (W16 + kDThreads - 1) / kDThreads;
  static_assert((W16 & (W16 - 1)) == 0, "piece count is a power of two");
  // a tap with fewer pieces than threads is copied redundantly by the surplus threads (same values to the
  // same place) rather than under a branch
  constexpr int WMASK = W16 - 1;
  constexpr int NA = MT * KS;                 // A-operand loads per tap and share
  constexpr int OCH = COUT / 8;               // 16-byte pieces per output row
  constexpr int OPITCH = (OCH + 1) * 8;       // epilogue tile row pitch in 16-bit units
  constexpr bool SKIP = COUT <= 64;           // can leave groups out
  // per wave: a 16-row tile of the epilogue and, before it, its rows' map entries
  constexpr int OWN16 = SKIP && 27 * R / 4 > 16 * (OCH + 1) ? 27 * R / 4 : 16 * (OCH + 1);
  __shared__ u32x4 wl[2][W16];
  __shared__ u32x4 otile_s[kDWaves][OWN16];
  __shared__ uint32_t groups_s[SKIP ? kDWaves : 1];

  // raw buffer of the input rows (word 3: 32-bit data format, no swizzle)
  const __amdgpu_buffer_rsrc_t rows =
      __builtin_amdgcn_make_buffer_rsrc((void*)const_cast<uint16_t*>(in), 0, BUF ? (int)((uint32_t)n_in * (CIN * 2)) : 0, 0x00020000);
  int64_t n_out = *d_n_out;
  if (n_out > capacity_out) n_out = capacity_out;
  const int64_t n_tiles = (n_out + kDWaves * R - 1) / (kDWaves * R);
  const int64_t xcd_tiles = emc2_xcd_tiles<kRun>(blockIdx.x % 8, n_tiles);
  int64_t slot = blockIdx.x / 8;
  if (slot >= xcd_tiles) return;   // uniform for the block
  do {
  const int64_t tile_id = emc2_xcd_tile<kRun>(blockIdx.x % 8, slot, n_tiles);
  // Opaque copies: the compiler would otherwise keep the addresses of all 27 taps alive from tile to tile and spill up to
  // 90 registers for it.
  int tid = threadIdx.x;
  int64_t nbr_pitch = capacity_out;
  if constexpr (LOOP) asm volatile("" : "+v"(tid), "+s"(nbr_pitch), "+s"(wp), "+s"(nbr), "+s"(zrow));

  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int m = lane & 15, q = lane >> 4;
  const int64_t wave_row0 = tile_id * (kDWaves * R) + (int64_t)wave * R;

  // lane l holds the kernel-map entries of row l % R of this wave's R rows
  const bool live = wave_row0 + (lane % R) < n_out;
  const int32_t* nrow = nbr + (live ? wave_row0 + (lane % R) : 0);
  const int32_t dead = live ? 0 : -1;   // OR-ed into kernel-map entries: rows past n_out have no neighbours
  unsigned long long oob = 0ull;        // lanes that saw an entry outside [0, n_in)

  floatx4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[mt][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  int32_t jq[3][3];         // kernel-map entries of groups g, g+1, g+2 (as loaded; masked where used)
  u32x4 areg[3][NA];        // A operands in flight; tap x lives in set x % 3
  u32x4 wq[3][WPT];         // weights in flight; tap x lives in set x % 3

#define EMC2_IDX_LOAD(GROUP, DST)                                                                        \
  _Pragma("unroll") for (int kx_ = 0; kx_ < 3; ++kx_)                                                    \
      jq[DST][kx_] = nrow[(int64_t)(3 * ((GROUP) < 9 ? (GROUP) : 8) + kx_) * nbr_pitch];
  // A operands of one tap and share: tile mt, k-step ks <- 16 bytes at channel 64*SHARE + 32*ks + 8*q of row JROW[16*mt + m]
  // The entries of rows 16*mt .. 16*mt+15 sit in lanes 16*mt .. 16*mt+15 of both halves; every lane needs the one of
  // its column m for each mt.  A lane-swap instruction broadcasts each 16-lane row to all four rows (no LDS
  // round trip: a ds_bpermute per tile costs a serialized ~120-cycle wait each).
#define EMC2_A_LOAD(JROW, SHARE, SET)                                                                    \
  {                                                                                                      \
    const uint32_t jr_ = (uint32_t)max((JROW), -1);   /* any negative entry is an absent neighbour */    \
    const u32x2 jm_ = __builtin_amdgcn_permlane16_swap(jr_, jr_, false, false);      /* 0101 -> 0000 | 1111 */ \
  _Pragma("unroll") for (int mt_ = 0; mt_ < MT; ++mt_) {                                                 \
    const int32_t j_ = (int32_t)jm_[mt_];                                                                \
    if constexpr (BUF) {                                                                                 \
      /* absent: 2^32 less a row, and a piece of the row: out of range, zero */                          \
      const uint32_t at_ = (uint32_t)j_ * (uint32_t)(CIN * 2) + 16u * (uint32_t)q + 128u * (SHARE);      \
      _Pragma("unroll") for (int ks_ = 0; ks_ < KS; ++ks_)                                               \
          areg[SET][mt_ * KS + ks_] = buffer_row16(rows, at_ + 64u * (uint32_t)ks_);                     \
    } else {                                                                                             \
      const uint16_t* src_ = (j_ >= 0 ? in + (int64_t)j_ * CIN : zrow) + 8 * q + 64 * (SHARE);           \
      _Pragma("unroll") for (int ks_ = 0; ks_ < KS; ++ks_)                                               \
          areg[SET][mt_ * KS + ks_] = *reinterpret_cast<const u32x4*>(src_ + 32 * ks_);                  \
    }                                                                                                    \
  }                                                                                                      \
  }
#define EMC2_W_LOAD(TAP, SHARE, SET)                                                                     \
  {                                                                                                      \
    const u32x4* wsrc_ = wp + (int64_t)((TAP) * KH + (SHARE)) * W16;                                     \
    _Pragma("unroll") for (int i_ = 0; i_ < WPT; ++i_)                                                   \
        wq[SET][i_] = wsrc_[(tid + i_ * kDThreads) & WMASK];                                     \
  }
#define EMC2_W_STORE(BUF, SET)                                                                           \
  _Pragma("unroll") for (int i_ = 0; i_ < WPT; ++i_)                                                     \
      wl[BUF][(tid + i_ * kDThreads) & WMASK] = wq[SET][i_];

  // the matrix work of one tap: operands of set SET, weights in WB
#define EMC2_TAP(WB, SET)                                                                                \
  _Pragma("unroll") for (int ks = 0; ks < KS; ++ks) {                                                    \
    u32x4 b[NT];                                                                                         \
    _Pragma("unroll") for (int j = 0; j < NT; ++j) b[j] = (WB)[(ks * NT + j) * 64 + lane];               \
    _Pragma("unroll") for (int mt = 0; mt < MT; ++mt)                                                    \
      _Pragma("unroll") for (int j = 0; j < NT; ++j)                                                     \
          acc[mt][j] = MmaD<DT>::run(areg[SET][mt * KS + ks], b[j], acc[mt][j]);                         \
  }
  const bool skip = SKIP && n_tiles > straight_tiles;     // the same for all blocks
  if (skip) {
    // The entries as rows the kernel may read (absent and beyond the input: -1), [tap][row], and the groups to run.
    int32_t* ent = reinterpret_cast<int32_t*>(otile_s[wave]);
    constexpr int NL = 14;                                     // loads, of two taps each (a half of the wave)
    const int sub = lane / R, row = lane % R;
    int32_t e[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) e[i] = nrow[(int64_t)(2 * i + sub < 27 ? 2 * i + sub : 26) * nbr_pitch];
    uint32_t groups = 0;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int32_t j = max(emc2_entry(e[i], dead, n_in, oob), -1);
      const unsigned long long some = __ballot(j >= 0);
#pragma unroll
      for (int t = 0; t < 2; ++t)
        if (2 * i + t < 27 && (t == 0 ? some & 0xffffffffull : some >> 32) != 0ull) groups |= 1u << ((2 * i + t) / 3);
      if (2 * i + sub < 27) ent[(2 * i + sub) * R + row] = j;
    }
    if (lane == 0) groups_s[wave] = groups;
    __syncthreads();
    groups = 0;
#pragma unroll
    for (int w = 0; w < kDWaves; ++w) groups |= groups_s[w];
    groups = __builtin_amdgcn_readfirstlane(groups);
#define EMC2_ENTRIES(GROUP) \
  _Pragma("unroll") for (int kx_ = 0; kx_ < 3; ++kx_) jq[0][kx_] = ent[(3 * (GROUP) + kx_) * R + row];
    if (groups != 0) {
      // prologue: entries, operands and weights of the first group; the weights of its first tap to LDS
      int g = __builtin_ctz(groups);
      groups &= groups - 1;
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) EMC2_W_LOAD(3 * g + kx, 0, kx)
      EMC2_ENTRIES(g)
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) EMC2_A_LOAD(jq[0][kx], 0, kx)
      EMC2_W_STORE(0, 0)
      __syncthreads();
      uint32_t buf = 0;
      while (true) {
        const int32_t past = groups != 0 ? 0 : -1;        // after the last group: no operands, the same weights again
        g = groups != 0 ? __builtin_ctz(groups) : g;
        EMC2_ENTRIES(g)
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
          // weights of the next group's tap: global -> registers (the set was emptied at the end of the previous tap)
          EMC2_W_LOAD(3 * g + kx, 0, kx)
          EMC2_TAP(wl[buf], kx)
          EMC2_A_LOAD(jq[0][kx] | past, 0, kx)            // the freed register set takes the next group's operands
          __builtin_amdgcn_wave_barrier();
          // weights of the next tap: registers -> the other LDS buffer; the barrier publishes them and retires the buffer
          // just read
          buf ^= 1;
          EMC2_W_STORE(buf, (kx + 1) % 3)
          __syncthreads();
        }
        if (past != 0) break;
        groups &= groups - 1;
      }
    }
#undef EMC2_ENTRIES
  }
  if (!skip) {
  // prologue: map entries of groups 0..2; weights of tap 0 to LDS; A operands of taps 0..2
  EMC2_IDX_LOAD(0, 0)
  EMC2_IDX_LOAD(1, 1)
  EMC2_IDX_LOAD(2, 2)
  EMC2_W_LOAD(0, 0, 0)
  EMC2_W_STORE(0, 0)
  EMC2_W_LOAD(1, 0, 1)
  EMC2_W_LOAD(2, 0, 2)
  EMC2_A_LOAD(emc2_entry(jq[0][0], dead, n_in, oob), 0, 0)
  EMC2_A_LOAD(emc2_entry(jq[0][1], dead, n_in, oob), 0, 1)
  EMC2_A_LOAD(emc2_entry(jq[0][2], dead, n_in, oob), 0, 2)
  __syncthreads();

  for (int g = 0; g < 9; ++g) {
    // kernel-map entries of group g + 3, requested a whole group before anything touches them
    int32_t jn[3];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) jn[kx] = nrow[(int64_t)(3 * (g + 3 < 9 ? g + 3 : 8) + kx) * nbr_pitch];
    const int32_t past = g < 8 ? 0 : -1;      // entries of "group 9" do not exist
#pragma unroll
    for (int h = 0; h < KH; ++h) {
#pragma unroll
      for (int kx = 0; kx < 3; ++kx) {
        const int at = 3 * (KH * g + h) + kx; // steps are numbered in the order in which they are taken
        // weights three steps on: global -> registers (the set was emptied at the end of the previous step)
        if (h + 1 < KH) EMC2_W_LOAD(3 * g + kx, h + 1, kx)
        else EMC2_W_LOAD(g < 8 ? 3 * (g + 1) + kx : 26, 0, kx)
        EMC2_TAP(wl[at & 1], kx)
        // the freed register set takes the A operands three steps on
        if (h + 1 < KH) EMC2_A_LOAD(emc2_entry(jq[0][kx], dead, n_in, oob), h + 1, kx)
        else EMC2_A_LOAD(emc2_entry(jq[1][kx], dead | past, n_in, oob), 0, kx)
        __builtin_amdgcn_wave_barrier();
        // weights of the next step: registers -> the other LDS buffer; the barrier publishes them and retires the
        // buffer just read
        EMC2_W_STORE((at + 1) & 1, (kx + 1) % 3)
        __syncthreads();
      }
    }
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
      jq[0][kx] = jq[1][kx];
      jq[1][kx] = jq[2][kx];
      jq[2][kx] = jn[kx];
    }
  }
  }
#undef EMC2_IDX_LOAD
#undef EMC2_A_LOAD
#undef EMC2_W_LOAD
#undef EMC2_W_STORE
#undef EMC2_TAP
  emc2_report_oob(oob, dev_flags);

  // epilogue: lane (m, q) holds column 16*j + m of rows 16*mt + 4*q + e.  Scale/shift/ReLU/convert in
  // registers, then each 16-row tile goes through LDS so that the global stores are whole 16-byte pieces.
  float sc[NT], sh[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    sc[j] = (epilogue != EMC2_EPI_NONE) ? scale[16 * j + m] : 1.f;
    sh[j] = (epilogue != EMC2_EPI_NONE) ? shift[16 * j + m] : 0.f;
  }
  uint16_t* otile = reinterpret_cast<uint16_t*>(otile_s[wave]);
  constexpr int OPI = 64 / OCH;               // rows one store instruction covers
  constexpr int ONI = (16 + OPI - 1) / OPI;   // store instructions per 16-row tile
  const int orow = lane / OCH, ochunk = lane % OCH;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = acc[mt][j][e];
        if (epilogue != EMC2_EPI_NONE) v = fmaf(v, sc[j], sh[j]);
        if (epilogue == EMC2_EPI_AFFINE_RELU) v = v > 0.f ? v : 0.f;
        otile[(4 * q + e) * OPITCH + 16 * j + m] = MmaD<DT>::cvt(v);
      }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < ONI; ++i) {
      const int r = i * OPI + orow;
      if (r < 16) {
        const u32x4 piece = *reinterpret_cast<const u32x4*>(otile + r * OPITCH + ochunk * 8);
        const int64_t o = wave_row0 + mt * 16 + r;
        if (o < n_out) *reinterpret_cast<u32x4*>(out + o * COUT + ochunk * 8) = piece;
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  slot += gridDim.x / 8;
  if constexpr (LOOP) __syncthreads();   // the next tile refills the weight buffers
  } while (LOOP && slot < xcd_tiles);
}

template <int DT, int CIN, int COUT>
void launch_direct(const void* d_in, const void* d_wp, const float* d_scale, const float* d_shift, int epilogue,
                   const int32_t* d_nbr, const int32_t* d_n_out, int64_t capacity_out, int32_t n_in, int32_t* dev_flags,
                   const void* d_zero_row, bool skip, void* d_out, hipStream_t s) {
  const int64_t rows_per_block = kDWaves * 16 * DirectCfg<CIN, COUT, true>::MT;
  // The host knows a level's capacity, up to 8 times the level below, not how many voxels it got.  Blocks without a tile
  // cost about 0.25 us per thousand: 32 -> 64 over 573 k rows took 97 us in a grid for 11.3 M rows (88 k blocks) and 75 us
  // in one for 573 k.  A loop over tiles costs the kernel up to a tenth in registers and instruction order (128 -> 128: 110
  // against 127 us), so it is used only where the grid would be several times kDGrid; the grid is then kDGrid blocks
  // (32 -> 64 over 573 k rows 97 -> 80 us, over 852 k 119 -> 109).
  const int64_t blocks = emc2_div_up(emc2_div_up(capacity_out, rows_per_block), 8) * 8;
#define LAUNCH(LOOP, BUF, BLOCKS)                                                                                           \
  hipLaunchKernelGGL((k_spconv_direct<DT, CIN, COUT, LOOP, BUF>), dim3((unsigned)(BLOCKS)), dim3(kDThreads), 0, s,           \
                     (const uint16_t*)d_in, (const u32x4*)d_wp, d_scale, d_shift, epilogue, d_nbr, d_n_out, capacity_out,     \
                     n_in, dev_flags, (const uint16_t*)d_zero_row, skip ? kStraightTiles : INT64_MAX, (uint16_t*)d_out)
  // Offsets into the input are 32-bit, and the absent neighbour's, 2^32 less a row, must lie at or beyond its end.
  const bool buf = ((int64_t)n_in + 1) * CIN * 2 <= ((int64_t)1 << 32);
  if (blocks <= 4 * kDGrid) {
    if (buf) LAUNCH(false, true, blocks);
    else LAUNCH(false, false, blocks);
  } else {
    if (buf) LAUNCH(true, true, kDGrid);
    else LAUNCH(true, false, kDGrid);
  }
#undef LAUNCH
}

}  // namespace

bool emc2_spconv_direct_supported(int cin, int cout) {
  return (cin == 64 && (cout == 64 || cout == 128)) || (cin == 128 && cout == 128);
}

bool emc2_spconv_direct_order(int cin, int cout) {
  return emc2_spconv_direct_supported(cin, cout) || emc2_spconv_resident_supported(cin, cout) || (cin == 32 && cout == 32);
}

void emc2_spconv_direct_pack(const void* d_w, int cin, int cout, void* d_packed, hipStream_t stream) {
  const int total = 27 * (cin / 32) * (cout / 16) * 64;
  hipLaunchKernelGGL(k_pack_weights_direct, dim3((unsigned)emc2_div_up(total, 256)), dim3(256), 0, stream,
                     (const uint16_t*)d_w, cin, cout, (uint4*)d_packed);
}

void emc2_spconv_direct_launch(emc2_dtype dtype, const void* d_in, const void* d_wp, const float* d_scale,
                               const float* d_shift, int epilogue, const int32_t* d_nbr, const int32_t* d_n_out,
                               int64_t capacity_out, int32_t n_in, int32_t* dev_flags, int cin, int cout,
                               const void* d_zero_row, bool skip, void* d_out, hipStream_t stream) {
#define CASE(DTV, CI, CO)                                                                                              \
  if (dtype == DTV && cin == CI && cout == CO) {                                                                       \
    launch_direct<DTV, CI, CO>(d_in, d_wp, d_scale, d_shift, epilogue, d_nbr, d_n_out, capacity_out, n_in, dev_flags,  \
                               d_zero_row, skip, d_out, stream);                                                       \
    return;                                                                                                            \
  }
  CASE(EMC2_F16, 64, 64) CASE(EMC2_BF16, 64, 64)
  CASE(EMC2_F16, 128, 128) CASE(EMC2_F16, 64, 128) CASE(EMC2_BF16, 128, 128) CASE(EMC2_BF16, 64, 128)
#undef CASE
}
