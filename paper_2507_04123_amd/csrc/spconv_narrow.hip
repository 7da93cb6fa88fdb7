// Sparse convolution 16 -> 32 and 32 -> 32 on the CDNA4 matrix cores (paper Sec. 3.5: 3D sparse convolution over non-empty
// voxels; Sec. 3.6: data movement overlapped with compute, operator fusion): the first stage of every stack.
//
// Few channels: a row is 32 or 64 bytes, its 27 map entries 108, its output 64, so the work is moving maps and rows, and what
// a kernel loses is waiting.  All taps' weights (27 or 54 KB) stay in LDS from the block's one barrier on; after it the waves go
// their own ways, tile after tile, and wait for nothing but their own loads: no barrier and no weights per tap.  As in the
// register-direct kernel a load IS the matrix operand.  16 channels, v_mfma_f32_32x32x16: lane (m = lane % 32, h = lane / 32)
// holds channels 8h .. 8h+7 of row m, one 16-byte load for 32 rows and a tap.  32 channels, v_mfma_f32_16x16x32: lane
// (m = lane % 16, q = lane / 16) holds channels 8q .. 8q+7, one load for 16 rows (whole 64-byte rows: half the lines a 32x32x16
// operand would touch).  Absent neighbours read past the end of the input's buffer descriptor, which yields zeros.
//
// 32 rows a wave: two taps' entries share a load (a half of the wave each) and two lane swaps hand them out; 128 registers,
// so 16 waves a CU, as many as the weights leave room for.  The taps are unrolled (the compiler counts the loads in flight), 12
// or 6 of them requested ahead; the next tile's entries are requested before the last taps' products.
// Alone, us, before (16 -> 32: rows staged in LDS, a barrier a tap; 32 -> 32: register-direct, weights of a tap at a time) / now:
// 16 -> 32 stride-2 to 985 k rows 76 / 58, to 529 k in bf16 45 / 33.5, submanifold over 60 k 14.6 / 10.8, 11.5 / 7.7 in a 16-beam
// frame; 32 -> 32 submanifold over 985 k 107 / 97, bf16 over 529 k 70 / 66, 64-beam frame 40.4 / 37.4.
// Requests 6, 9, 12, 18, 27 taps ahead: 63, 61, 58, 59, 58 (16 -> 32); 4, 6, 9, 12: 98, 97, 96, 97 (32 -> 32).  The next tile's
// entries requested a whole tile ahead: the same.  2048 blocks instead of what is resident: 62.  What is left is traffic: 395 MB
// a launch for 32 -> 32 over 985 k rows, 4.1 TB/s where a copy reaches 4.3, 232 of them necessary (rows fetched by more than one
// L2, or again after they were displaced; with an eighth of the rows an XCD 352, in the same time); 191 MB and 3.3 TB/s for 16 -> 32.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "common.h"
#include "spconv_mfma.h"
#include "xcd_tiles.h"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int DT> struct MmaN;
template <> struct MmaN<EMC2_F16> {
  static __device__ __forceinline__ floatx16 run(u32x4 a, u32x4 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ floatx4 run(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint16_t cvt(float v) { return __half_as_ushort(__float2half_rn(v)); }
};
template <> struct MmaN<EMC2_BF16> {
  static __device__ __forceinline__ floatx16 run(u32x4 a, u32x4 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ floatx4 run(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint16_t cvt(float v) { return __builtin_bit_cast(uint16_t, __float2bfloat16(v)); }
};

constexpr int kNRows = 32;                // output rows per wave
constexpr int kNRun = 32;                 // tiles of a run: 1024 rows
constexpr int kNCout = 32;
constexpr int kNPitch = kNCout / 8 + 1;   // epilogue tile row pitch in 16-byte pieces

template <int CIN> struct NarrowCfg {
  static constexpr int WAVES = CIN == 16 ? 4 : 8;      // that share the weights: 16 waves a CU either way
  static constexpr int GRID = 256 * 16 / WAVES;        // blocks resident at once; they loop over the tiles
  static constexpr int LPT = CIN / 16;                 // operand loads per tap
  static constexpr int DEPTH = CIN == 16 ? 12 : 6;     // operands in flight, in taps
  static constexpr int PIECES = 27 * CIN * kNCout / 8; // of 16 bytes, all weights
};

template <int DT, int CIN, bool BUF>
__device__ __forceinline__ void run_narrow(uint32_t block, uint32_t n_blocks, const uint16_t* __restrict__ in, const u32x4* __restrict__ wp,
                                           const float* __restrict__ scale, const float* __restrict__ shift, int epilogue,
                                           const int32_t* __restrict__ nbr, const int32_t* __restrict__ d_n_out, int64_t capacity_out,
                                           int32_t n_in, int32_t* __restrict__ dev_flags, const uint16_t* __restrict__ zrow,
                                           uint16_t* __restrict__ out) {
  using C = NarrowCfg<CIN>;
  constexpr int D = C::DEPTH, LPT = C::LPT;
  __shared__ u32x4 wl[C::PIECES];
  __shared__ u32x4 otile_s[C::WAVES][kNRows * kNPitch];
  const __amdgpu_buffer_rsrc_t rows =
      __builtin_amdgcn_make_buffer_rsrc((void*)const_cast<uint16_t*>(in), 0, BUF ? (int)((uint32_t)n_in * (CIN * 2)) : 0, 0x00020000);
  int64_t n_out = *d_n_out;
  if (n_out > capacity_out) n_out = capacity_out;
  const int64_t n_tiles = (n_out + kNRows - 1) / kNRows;
  const int64_t tiles = emc2_xcd_tiles<kNRun>(block % 8, n_tiles);
  if ((int64_t)(block / 8) * C::WAVES >= tiles) return;   // uniform for the block
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = lane & 31, h = lane >> 5;                      // entries: row and half
  const int piece0 = CIN == 16 ? h : lane >> 4;                // operands: 16-byte piece of the row
  const int64_t step = (int64_t)(n_blocks / 8) * C::WAVES;
  int64_t slot = (int64_t)(block / 8) * C::WAVES + wave;

  unsigned long long oob = 0ull;   // lanes that saw an entry outside [0, n_in)
  // half h of the wave holds the entries of taps 2i + h of the 32 rows
  int32_t e[14];
  // (past the last tile: the last one's again)
  const auto entries = [&](int64_t at) {
    const int64_t row0 = emc2_xcd_tile<kNRun>(block % 8, at < tiles ? at : tiles - 1, n_tiles) * kNRows;
    const int32_t own = row0 + m < n_out ? m : 0;
    if constexpr (BUF) {   // one address in scalar registers and a 32-bit offset per half
      const uint32_t even = 4u * (uint32_t)own, off = even + (h ? 4u * (uint32_t)capacity_out : 0u);
#pragma unroll
      for (int i = 0; i < 14; ++i)
        e[i] = *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(nbr + ((int64_t)(2 * i) * capacity_out + row0)) +
                                                 (i < 13 ? off : even));
    } else {
      const int32_t* at_row = nbr + row0 + own;
#pragma unroll
      for (int i = 0; i < 14; ++i) e[i] = (at_row + (int64_t)(2 * i) * capacity_out)[i < 13 && h ? capacity_out : 0];
    }
  };
  entries(slot);
  for (int p = threadIdx.x; p < C::PIECES; p += C::WAVES * 64) wl[p] = wp[p];
  float sc[LPT], sh[LPT];
#pragma unroll
  for (int k = 0; k < LPT; ++k) {
    const int col = CIN == 16 ? m : 16 * k + (lane & 15);
    sc[k] = epilogue != EMC2_EPI_NONE ? scale[col] : 1.f;
    sh[k] = epilogue != EMC2_EPI_NONE ? shift[col] : 0.f;
  }
  __syncthreads();

  for (; slot < tiles; slot += step) {
    const int64_t row0 = emc2_xcd_tile<kNRun>(block % 8, slot, n_tiles) * kNRows;
    const int32_t dead = row0 + m < n_out ? 0 : -1;
    int32_t j[28][LPT];
    u32x4 a[D][LPT];
    const auto load = [&](int t) {
      if (t % 2 == 0) {   // entries of an even tap and the next one: the halves of the wave swapped
        const uint32_t v = (uint32_t)max(emc2_entry(e[t / 2], dead, n_in, oob), -1);
        const u32x2 s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          if constexpr (LPT == 1) {
            j[t + k][0] = (int32_t)s[k];
          } else {        // rows 0-15 and 16-31 to all four quarters
            const u32x2 r = __builtin_amdgcn_permlane16_swap(s[k], s[k], false, false);
            j[t + k][0] = (int32_t)r[0];
            j[t + k][1] = (int32_t)r[1];
          }
        }
      }
#pragma unroll
      for (int l = 0; l < LPT; ++l) {
        const int32_t r = j[t][l];
        if constexpr (BUF)   // absent: 2^32 less a row, and a piece of the row: out of range, zero
          a[t % D][l] = __builtin_amdgcn_raw_buffer_load_b128(rows, (int)((uint32_t)r * (CIN * 2u) + 16u * (uint32_t)piece0), 0, 0);
        else
          a[t % D][l] = *reinterpret_cast<const u32x4*>((r >= 0 ? in + (int64_t)r * CIN : zrow) + 8 * piece0);
      }
    };
#pragma unroll
    for (int t = 0; t < D; ++t) load(t);
    floatx16 acc;
    floatx4 acc4[2][2];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = acc4[i / 8][i / 4 % 2][i % 4] = 0.f;
#pragma unroll
    for (int t = 0; t < 27; ++t) {
      if constexpr (CIN == 16) {
        acc = MmaN<DT>::run(a[t % D][0], wl[t * 64 + lane], acc);
      } else {
        const u32x4 b0 = wl[t * 128 + lane], b1 = wl[t * 128 + 64 + lane];
#pragma unroll
        for (int l = 0; l < 2; ++l) {
          acc4[l][0] = MmaN<DT>::run(a[t % D][l], b0, acc4[l][0]);
          acc4[l][1] = MmaN<DT>::run(a[t % D][l], b1, acc4[l][1]);
        }
      }
      if (t + D < 27) load(t + D);
      if (t + D == 27) entries(slot + step);
    }
    // 32x32: the lane holds column m, element i is row 8 * (i / 4) + 4 * h + i % 4; 16x16: column 16 * j + lane % 16 of rows
    // 16 * l + 4 * (lane / 16) + e
    uint16_t* otile = reinterpret_cast<uint16_t*>(otile_s[wave]);
    const auto put = [&](float v, int row, int col, int k) {
      if (epilogue != EMC2_EPI_NONE) v = fmaf(v, sc[k], sh[k]);
      if (epilogue == EMC2_EPI_AFFINE_RELU) v = v > 0.f ? v : 0.f;
      otile[row * (kNPitch * 8) + col] = MmaN<DT>::cvt(v);
    };
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if constexpr (CIN == 16) put(acc[i], 8 * (i / 4) + 4 * h + i % 4, m, 0);
      else put(acc4[i / 8][i / 4 % 2][i % 4], 16 * (i / 8) + 4 * (lane >> 4) + i % 4, 16 * (i / 4 % 2) + (lane & 15), i / 4 % 2);
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 16 * i + lane / 4, c = lane % 4;
      const u32x4 piece = otile_s[wave][r * kNPitch + c];
      if (row0 + r < n_out) reinterpret_cast<u32x4*>(out)[(row0 + r) * 4 + c] = piece;
    }
    __builtin_amdgcn_wave_barrier();
  }
  emc2_report_oob(oob, dev_flags);
}

template <int DT, int CIN, bool BUF, int CALLS>
__global__ void __launch_bounds__(NarrowCfg<CIN>::WAVES * 64, 4) k_spconv_narrow(const emc2_conv_batch<CALLS> b) {
  const emc2_conv_place at = emc2_conv_of_block(b);
  const emc2_conv_args& c = b.call[at.call];
  run_narrow<DT, CIN, BUF>(at.block, at.blocks, (const uint16_t*)c.d_in, (const u32x4*)c.d_w, c.d_scale, c.d_shift, c.epilogue, c.d_nbr,
                           c.d_n_out, c.capacity_out, c.n_in, c.dev_flags, (const uint16_t*)c.d_zero_row, (uint16_t*)c.d_out);
}

template <int DT, int CIN> void launch_narrow(const emc2_conv_args* calls, int n, hipStream_t s) {
  using C = NarrowCfg<CIN>;
  emc2_conv_batch<kConvBatch> b;
  b.n = n;
  uint32_t blocks = 0;
  // Offsets into the input are 32-bit, and the absent neighbour's, 2^32 less a row, must lie at or beyond its end; so are the
  // offsets into two taps of the map.
  bool buf = true;
  for (int i = 0; i < n; ++i) {
    b.call[i] = calls[i];
    b.first[i] = blocks;
    const int64_t own = emc2_div_up(emc2_div_up(calls[i].capacity_out, kNRows * C::WAVES), 8) * 8;
    blocks += (uint32_t)(own < C::GRID ? own : C::GRID);
    buf = buf && ((int64_t)calls[i].n_in + 1) * CIN * 2 <= ((int64_t)1 << 32) && calls[i].capacity_out < ((int64_t)1 << 29);
  }
#define LAUNCH(BUF, CALLS, ARGS) \
  hipLaunchKernelGGL((k_spconv_narrow<DT, CIN, BUF, CALLS>), dim3(blocks), dim3(C::WAVES * 64), 0, s, ARGS)
  if (n == 1) {
    if (buf) LAUNCH(true, 1, emc2_conv_one(b));
    else LAUNCH(false, 1, emc2_conv_one(b));
  } else {
    if (buf) LAUNCH(true, kConvBatch, b);
    else LAUNCH(false, kConvBatch, b);
  }
#undef LAUNCH
}

}  // namespace

bool emc2_spconv_narrow_supported(int cin, int cout) { return (cin == 16 || cin == 32) && cout == kNCout; }

void emc2_spconv_narrow_launch(emc2_dtype dtype, int cin, const emc2_conv_args* calls, int n, hipStream_t stream) {
#define CASE(D, CI) \
  if (dtype == D && cin == CI) launch_narrow<D, CI>(calls, n, stream);
  CASE(EMC2_F16, 16) CASE(EMC2_BF16, 16) CASE(EMC2_F16, 32) CASE(EMC2_BF16, 32)
#undef CASE
}
