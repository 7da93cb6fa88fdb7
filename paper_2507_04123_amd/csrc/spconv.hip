// Sparse convolution over a kernel map (paper Sec. 3.5: customised 3D sparse convolution over the
// non-empty voxels; Sec. 3.6: graph fusion -> affine + ReLU fused into the epilogue).
// This file: argument checks, dispatch, and the vector-ALU kernel (fp32 path and channel counts
// the MFMA kernels do not cover).  The MFMA gather-GEMM lives in spconv_mfma.hip.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "common.h"
#include "conv_order.h"
#include "spconv_mfma.h"

namespace {

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(__half v) { return __half2float(v); }
__device__ __forceinline__ float to_f32(__hip_bfloat16 v) { return __bfloat162float(v); }
__device__ __forceinline__ void from_f32(float* p, float v) { *p = v; }
__device__ __forceinline__ void from_f32(__half* p, float v) { *p = __float2half_rn(v); }
__device__ __forceinline__ void from_f32(__hip_bfloat16* p, float v) { *p = __float2bfloat16(v); }

// Output-stationary: `cout` consecutive threads own one output row; taps outer, input channels inner.
template <typename T>
__global__ void __launch_bounds__(256) k_spconv_alu(const T* __restrict__ in, const T* __restrict__ w,
                                                    const float* __restrict__ scale, const float* __restrict__ shift,
                                                    int epilogue, const int32_t* __restrict__ nbr,
                                                    const int32_t* __restrict__ d_n_out, int64_t capacity_out,
                                                    int32_t n_in, int32_t* __restrict__ dev_flags, int cin, int cout,
                                                    int rows_per_block, T* __restrict__ out) {
  int64_t n = *d_n_out;
  if (n > capacity_out) n = capacity_out;
  const int row = threadIdx.x / cout;
  const int d = threadIdx.x - row * cout;
  const int64_t o = (int64_t)blockIdx.x * rows_per_block + row;
  if (row >= rows_per_block || o >= n) return;
  float acc = 0.f;
  for (int k = 0; k < 27; ++k) {
    const int32_t j = nbr[(int64_t)k * capacity_out + o];
    if (j < 0) continue;
    if (j >= n_in) {   // names a row the input does not hold: absent, and reported
      if (d == 0) atomicOr(dev_flags, EMC2_DEVFLAG_MAP);
      continue;
    }
    const T* xr = in + (int64_t)j * cin;
    const T* wk = w + (int64_t)k * cin * cout + d;
    for (int c = 0; c < cin; ++c) acc = fmaf(to_f32(xr[c]), to_f32(wk[(int64_t)c * cout]), acc);
  }
  if (epilogue != EMC2_EPI_NONE) acc = fmaf(acc, scale[d], shift[d]);
  if (epilogue == EMC2_EPI_AFFINE_RELU) acc = acc > 0.f ? acc : 0.f;
  from_f32(out + o * cout + d, acc);
}

// Small-channel kernel (Cin in {4, 16}, Cout in {16, 32}: the input layers that sit below the matrix-core
// tile sizes).  One thread owns one output row and all of its Cout accumulators; a tap's weights are LDS
// broadcasts and a tap nobody in the wave has is skipped.  These layers have few rows (one wave per 64 of
// them, a handful of waves per CU), so latency, not bandwidth, is what they can lose time to: all 27
// kernel-map entries of a row are requested at once, and the feature rows of a whole batch of taps (27 at
// Cin = 4, 9 at Cin = 16) are requested together, unconditionally (absent entries re-read row 0), before
// the first of them is used -- two memory round trips per batch instead of two per tap.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// SPLIT: neighbouring threads that share a row, COUT / SPLIT channels each.
template <typename T, int CIN, int COUT, int SPLIT>
__global__ void __launch_bounds__(256) k_spconv_small(const T* __restrict__ in, const T* __restrict__ w,
                                                      const float* __restrict__ scale, const float* __restrict__ shift,
                                                      int epilogue, const int32_t* __restrict__ nbr,
                                                      const int32_t* __restrict__ d_n_out, int64_t capacity_out,
                                                      int32_t n_in, int32_t* __restrict__ dev_flags, T* __restrict__ out) {
  __shared__ float wl[27 * CIN * COUT];
  for (int i = threadIdx.x; i < 27 * CIN * COUT; i += 256) wl[i] = to_f32(w[i]);
  int64_t n = *d_n_out;
  if (n > capacity_out) n = capacity_out;
  constexpr int CO = COUT / SPLIT;
  const int64_t o = ((int64_t)blockIdx.x * 256 + threadIdx.x) / SPLIT;
  const int d0 = (int)threadIdx.x % SPLIT * CO;
  const bool live = o < n;
  const int32_t* nrow = nbr + (live ? o : 0);
  const int32_t dead = live ? 0 : -1;
  constexpr int ROW_BYTES = CIN * (int)sizeof(T);
  static_assert(ROW_BYTES == 8 || ROW_BYTES % 16 == 0, "feature rows are read with 8- or 16-byte loads");
  constexpr int RW = ROW_BYTES / 4;               // 32-bit words per feature row
  constexpr int TB = ROW_BYTES <= 8 ? 27 : 9;     // taps whose rows are in flight together
  int32_t j[27];
  unsigned long long oob = 0ull;   // lanes that saw an entry outside [0, n_in)
#pragma unroll
  for (int k = 0; k < 27; ++k) j[k] = nrow[(int64_t)k * capacity_out];
  float acc[CO];
#pragma unroll
  for (int d = 0; d < CO; ++d) acc[d] = 0.f;
  __syncthreads();   // weights in LDS
#pragma unroll
  for (int k0 = 0; k0 < 27; k0 += TB) {
    uint32_t xr[TB][RW];
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      const int32_t jj = j[k0 + t] = emc2_entry(j[k0 + t], dead, n_in, oob);   // masked once, used twice
      const char* src = reinterpret_cast<const char*>(in + (int64_t)(jj >= 0 ? jj : 0) * CIN);
      if constexpr (ROW_BYTES == 8) {
        const u32x2_t v = *reinterpret_cast<const u32x2_t*>(src);
        xr[t][0] = v.x; xr[t][1] = v.y;
      } else {
#pragma unroll
        for (int q = 0; q < ROW_BYTES / 16; ++q) {
          const u32x4_t v = reinterpret_cast<const u32x4_t*>(src)[q];
          xr[t][4 * q] = v.x; xr[t][4 * q + 1] = v.y; xr[t][4 * q + 2] = v.z; xr[t][4 * q + 3] = v.w;
        }
      }
    }
#pragma unroll
    for (int t = 0; t < TB; ++t) {
      const int k = k0 + t;
      const bool have = j[k] >= 0;
      if (__ballot(have) == 0ull) continue;  // wave-uniform
      if (have) {
        const float* wk = wl + k * CIN * COUT + d0;
#pragma unroll
        for (int c = 0; c < CIN; ++c) {
          T xe;
          if constexpr (sizeof(T) == 2) {
            const uint16_t bits = (uint16_t)(xr[t][c / 2] >> (16 * (c % 2)));
            xe = __builtin_bit_cast(T, bits);
          } else {
            xe = __builtin_bit_cast(T, xr[t][c]);
          }
          const float xv = to_f32(xe);
#pragma unroll
          for (int d = 0; d < CO; ++d) acc[d] = fmaf(xv, wk[c * COUT + d], acc[d]);
        }
      }
    }
  }
  emc2_report_oob(oob, dev_flags);
  if (!live) return;
  alignas(16) T yr[CO];
#pragma unroll
  for (int d = 0; d < CO; ++d) {
    float v = acc[d];
    if (epilogue != EMC2_EPI_NONE) v = fmaf(v, scale[d0 + d], shift[d0 + d]);
    if (epilogue == EMC2_EPI_AFFINE_RELU) v = v > 0.f ? v : 0.f;
    from_f32(&yr[d], v);
  }
  constexpr int OUT_BYTES = CO * (int)sizeof(T);
  static_assert(OUT_BYTES % 16 == 0, "output rows are written with 16-byte stores");
  char* dst = reinterpret_cast<char*>(out + o * COUT + d0);
#pragma unroll
  for (int q = 0; q < OUT_BYTES / 16; ++q) reinterpret_cast<u32x4_t*>(dst)[q] = reinterpret_cast<const u32x4_t*>(yr)[q];
}

// Small-channel 16-bit kernel on the matrix cores (Cin in {4, 16}, Cout in {16, 32}).  Memory access as in
// k_spconv_small -- lane = output row, every kernel-map entry and feature row requested with whole-wave loads that
// touch a few cache lines each -- but the contraction runs on v_mfma_f32_4x4x4 (16 blocks of 4x4x4 per instruction):
// as the B operand, lane l supplies 4 input channels of ITS row (8 bytes, exactly what it loaded); as the A
// operand it supplies W[tap][4 channels][4g + l % 4], the same 4x4 weight block for every block of rows; the result
// leaves 4 consecutive output channels of row l in lane l's four accumulator registers, so the epilogue is
// per-lane and the stores are whole 16-byte pieces of the lane's own row.  The vector-ALU kernel spends its time
// re-reading weights from LDS for every multiply-add (one LDS read per 4 of them); here a weight block is read
// once per tap and 4 channels for 64 rows, and a tap none of them has costs nothing.
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

template <int DT> struct Mma4;
template <> struct Mma4<EMC2_F16> {
  static __device__ __forceinline__ float4_t run(u32x2_t a, u32x2_t b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(half4_t, a), __builtin_bit_cast(half4_t, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t cvt2(float lo, float hi) {
    return (uint32_t)__half_as_ushort(__float2half_rn(lo)) | ((uint32_t)__half_as_ushort(__float2half_rn(hi)) << 16);
  }
};
template <> struct Mma4<EMC2_BF16> {
  static __device__ __forceinline__ float4_t run(u32x2_t a, u32x2_t b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(short4_t, a), __builtin_bit_cast(short4_t, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t cvt2(float lo, float hi) {
    return (uint32_t)__builtin_bit_cast(uint16_t, __float2bfloat16(lo)) |
           ((uint32_t)__builtin_bit_cast(uint16_t, __float2bfloat16(hi)) << 16);
  }
};

// A wave takes 64 rows.  With 128, a weight block's read serving both halves, a frame's launch was less than a round of the chip and each of
// its waves had twice the loads to wait for.  Entries and rows requested together: all 27 and 9 of 4 channels, 9 and 3 of 16.  us, 128
// rows a wave, 9 entries and rows (3 of 16 channels) at a time / 64 rows, the same / so: 4 -> 16 1 000 rows 6.9 / 4.5 / 4.3, 17 k 7.9 / 5.5 /
// 5.2, 118 k 9.8 / 7.9 / 7.7, 471 k 20.7 / 18.4 / 19.0, 942 k 34.0 / 29.5 / 30.6; 4 -> 32 17 k 10.4 / 7.6 / 7.2, 118 k 13.5 / 11.7 / 11.5, 471 k
// 29.4 / 30.0 / 27.9, 942 k 48.8 / 46.3 / 45.2; 16 -> 16 17 k 12.6 / 8.7 / 7.9, 118 k 17.4 / 14.6 / 13.2, 471 k 31.9 / 30.7 / 30.2, 942 k 56.1 /
// 51.5 / 50.5.  All 27 rows of 4 channels at once: 5.7, 8.4, 22.0, 35.4 (fewer waves); 27 entries and 9 rows of 16: 7.6, 13.6, 32.1, 54.4.
// A block beyond the rows has nothing to do, and a capacity of all points has many of them: it leaves when it has seen the row count, which
// comes while a thread's share of the weights does.  us, all blocks to the end / so: 16 -> 16 1 000 rows of 450 k 13.3 / 10.2, of 960 k
// 22.3 / 10.2; 4 -> 16 8.7 / 6.5, 16.0 / 6.5; 4 -> 32 10.0 / 9.3, 17.0 / 9.4; full capacities, which have all weights of a thread in flight now:
// 16 -> 16 222 k rows 21.4 / 19.9, 562 k 39.2 / 36.5; 4 -> 32 20.2 / 19.8, 33.0 / 32.6; 4 -> 16 12.6 / 12.5, 22.9 / 22.3.  The count first, then the
// weights: 1 % longer than before.  The first entries before the weights: 4 -> 32 357 k 25 / 27.5, 16 -> 16 1 500 rows 5.8 / 6.0.  (128 rows a wave are still the better ones of 4 -> 32 between
// 205 k and 360 k rows under some maps: 222 k 18.6 / 19.8, 357 k 21.1 to 24.8 / 22.6 to 24.8, 303 k 24.4 / 22.2.)
template <int DT, int CIN, int COUT>
__device__ __forceinline__ void run_rows(uint32_t block, const uint16_t* __restrict__ in, const uint16_t* __restrict__ w,
                                         const float* __restrict__ scale, const float* __restrict__ shift, int epilogue,
                                         const int32_t* __restrict__ nbr, const int32_t* __restrict__ d_n_out, int64_t capacity_out,
                                         int32_t n_in, int32_t* __restrict__ dev_flags, uint16_t* __restrict__ out) {
  constexpr int KB = CIN / 4;                 // 4-channel blocks of an input row
  constexpr int G = COUT / 4;                 // 4-channel groups of an output row
  constexpr int EB = CIN == 4 ? 27 : 9;       // taps whose entries are in flight together
  constexpr int TB = CIN == 4 ? 9 : 3;        // and whose rows are
  constexpr int RW = CIN / 2;                 // 32-bit words per input row
  static_assert(27 % EB == 0 && EB % TB == 0 && CIN % 4 == 0 && COUT % 8 == 0, "shapes this kernel covers");
  // weights as A operands: wl[((tap * KB + kb) * G + g) * 4 + j] = W[tap][4kb + 0..3][4g + j], 8 bytes
  constexpr int WN = 27 * KB * G * 4, WT = (WN + 255) / 256;
  __shared__ u32x2_t wl[WN];
  u32x2_t wv[WT];                             // a thread's share, requested before the row count is looked at
#pragma unroll
  for (int i = 0; i < WT; ++i) {
    const int e = min((int)threadIdx.x + 256 * i, WN - 1), j = e & 3;
    int f = e >> 2;
    const int g = f % G; f /= G;
    const int kb = f % KB;
    const int tap = f / KB;
    const uint16_t* src = w + ((int64_t)tap * CIN + 4 * kb) * COUT + 4 * g + j;
    wv[i] = u32x2_t{(uint32_t)src[0] | ((uint32_t)src[COUT] << 16), (uint32_t)src[2 * COUT] | ((uint32_t)src[3 * COUT] << 16)};
  }
  int64_t n = *d_n_out;
  if (n > capacity_out) n = capacity_out;
  asm volatile("" ::: "memory");              // (else the loads sink below the branch)
  if ((int64_t)block * 256 >= n) return;      // uniform for the block
#pragma unroll
  for (int i = 0; i < WT; ++i)
    if ((int)threadIdx.x + 256 * i < WN) wl[threadIdx.x + 256 * i] = wv[i];
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)block * 256 + threadIdx.x;
  const bool live = row < n;
  const int32_t* nrow = nbr + (live ? row : 0);
  const int32_t dead = live ? 0 : -1;
  unsigned long long oob = 0ull;
  float4_t acc[G];
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = float4_t{0.f, 0.f, 0.f, 0.f};
  __syncthreads();   // weights in LDS
  const int jq = lane & 3;
#pragma unroll 1
  for (int e0 = 0; e0 < 27; e0 += EB) {
    int32_t e[EB];
#pragma unroll
    for (int t = 0; t < EB; ++t) e[t] = nrow[(int64_t)(e0 + t) * capacity_out];
#pragma unroll
    for (int k = 0; k < EB; k += TB) {
      int32_t j[TB];
      uint32_t x[TB][RW];
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        j[t] = emc2_entry(e[k + t], dead, n_in, oob);
        const char* src = reinterpret_cast<const char*>(in + (int64_t)(j[t] >= 0 ? j[t] : 0) * CIN);
        if constexpr (RW == 2) {
          const u32x2_t v = *reinterpret_cast<const u32x2_t*>(src);
          x[t][0] = v.x; x[t][1] = v.y;
        } else {
#pragma unroll
          for (int q = 0; q < RW / 4; ++q) {
            const u32x4_t v = reinterpret_cast<const u32x4_t*>(src)[q];
            x[t][4 * q] = v.x; x[t][4 * q + 1] = v.y; x[t][4 * q + 2] = v.z; x[t][4 * q + 3] = v.w;
          }
        }
      }
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        const bool have = j[t] >= 0;
        if (__ballot(have) == 0ull) continue;   // wave-uniform: nobody has this tap
        const u32x2_t* wt = wl + (e0 + k + t) * KB * G * 4 + jq;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const u32x2_t b = have ? u32x2_t{x[t][2 * kb], x[t][2 * kb + 1]} : u32x2_t{0u, 0u};   // an absent neighbour adds zero
#pragma unroll
          for (int g = 0; g < G; ++g) acc[g] = Mma4<DT>::run(wt[(kb * G + g) * 4], b, acc[g]);
        }
      }
    }
  }
  emc2_report_oob(oob, dev_flags);
  // lane l holds output channels 4g .. 4g+3 of its row in acc[g]
  if (!live) return;
  uint32_t y[COUT / 2];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = acc[g][i];
      if (epilogue != EMC2_EPI_NONE) v[i] = fmaf(v[i], scale[4 * g + i], shift[4 * g + i]);
      if (epilogue == EMC2_EPI_AFFINE_RELU) v[i] = v[i] > 0.f ? v[i] : 0.f;
    }
    y[2 * g] = Mma4<DT>::cvt2(v[0], v[1]);
    y[2 * g + 1] = Mma4<DT>::cvt2(v[2], v[3]);
  }
  u32x4_t* dst = reinterpret_cast<u32x4_t*>(out + row * COUT);
#pragma unroll
  for (int q = 0; q < COUT / 8; ++q) dst[q] = u32x4_t{y[4 * q], y[4 * q + 1], y[4 * q + 2], y[4 * q + 3]};
}

template <int DT, int CIN, int COUT, int CALLS>
__global__ void __launch_bounds__(256, 4) k_spconv_rows(const emc2_conv_batch<CALLS> b) {
  const emc2_conv_place at = emc2_conv_of_block(b);
  const emc2_conv_args& c = b.call[at.call];
  run_rows<DT, CIN, COUT>(at.block, (const uint16_t*)c.d_in, (const uint16_t*)c.d_w, c.d_scale, c.d_shift, c.epilogue,
                          c.d_nbr, c.d_n_out, c.capacity_out, c.n_in, c.dev_flags, (uint16_t*)c.d_out);
}

void launch_rows(emc2_dtype dtype, int cin, int cout, const emc2_conv_args* calls, int n, hipStream_t s) {
  emc2_conv_batch<kConvBatch> b;
  b.n = n;
  uint32_t blocks = 0;
  for (int i = 0; i < n; ++i) {
    b.call[i] = calls[i];
    b.first[i] = blocks;
    blocks += (uint32_t)emc2_div_up(calls[i].capacity_out, 256);
  }
#define EMC2_ROWS(D, CI, CO)                                                                                                     \
  if (dtype == D && cin == CI && cout == CO) {                                                                                   \
    if (n == 1) hipLaunchKernelGGL((k_spconv_rows<D, CI, CO, 1>), dim3(blocks), dim3(256), 0, s, emc2_conv_one(b));              \
    else hipLaunchKernelGGL((k_spconv_rows<D, CI, CO, kConvBatch>), dim3(blocks), dim3(256), 0, s, b);                           \
  }
  EMC2_ROWS(EMC2_F16, 4, 16) EMC2_ROWS(EMC2_F16, 4, 32) EMC2_ROWS(EMC2_F16, 16, 16)
  EMC2_ROWS(EMC2_BF16, 4, 16) EMC2_ROWS(EMC2_BF16, 4, 32) EMC2_ROWS(EMC2_BF16, 16, 16)
#undef EMC2_ROWS
}

// Rows of a launch up to which four threads share a row (fp32): a launch of so many is bound by the chain of a thread's multiply-adds
// and LDS reads of weights, a quarter as long so.  A thread a row / four, us: 4 -> 16 2 000 rows 13.2 / 7.0, 20 000 13.4 / 7.4, 65 536
// 14.6 / 10.0; 4 -> 32 24.0 / 9.9, 24.1 / 10.4, 26.4 / 14.3; 16 -> 16 42.0 / 16.3, 42.2 / 18.3, 43.8 / 36.9.
constexpr int64_t kSplitRows = 65536;

template <typename T>
bool launch_small(const void* d_in, const void* d_w, const float* d_scale, const float* d_shift, int epilogue,
                  const int32_t* d_nbr, const int32_t* d_n_out, int64_t capacity_out, int32_t n_in, int32_t* dev_flags,
                  int cin, int cout, void* d_out, hipStream_t s) {
#define EMC2_SMALL_AS(CI, CO, SPLIT)                                                                                             \
  hipLaunchKernelGGL((k_spconv_small<T, CI, CO, SPLIT>), dim3((unsigned)emc2_div_up(capacity_out * SPLIT, 256)), dim3(256), 0, s, \
                     (const T*)d_in, (const T*)d_w, d_scale, d_shift, epilogue, d_nbr, d_n_out, capacity_out, n_in, dev_flags,    \
                     (T*)d_out)
#define EMC2_SMALL(CI, CO)                                                                                            \
  if (cin == CI && cout == CO) {                                                                                      \
    if (sizeof(T) == 4 && capacity_out <= kSplitRows) EMC2_SMALL_AS(CI, CO, (sizeof(T) == 4 ? 4 : 1));                \
    else EMC2_SMALL_AS(CI, CO, 1);                                                                                    \
    return true;                                                                                                      \
  }
  EMC2_SMALL(4, 16) EMC2_SMALL(4, 32) EMC2_SMALL(16, 16)
#undef EMC2_SMALL
#undef EMC2_SMALL_AS
  return false;
}

template <typename T>
void launch_alu(const void* d_in, const void* d_w, const float* d_scale, const float* d_shift, int epilogue,
                const int32_t* d_nbr, const int32_t* d_n_out, int64_t capacity_out, int32_t n_in, int32_t* dev_flags,
                int cin, int cout, void* d_out, hipStream_t s) {
  if (launch_small<T>(d_in, d_w, d_scale, d_shift, epilogue, d_nbr, d_n_out, capacity_out, n_in, dev_flags, cin, cout, d_out, s))
    return;
  const int rows = 256 / cout;
  hipLaunchKernelGGL(k_spconv_alu<T>, dim3((unsigned)emc2_div_up(capacity_out, rows)), dim3(256), 0, s, (const T*)d_in,
                     (const T*)d_w, d_scale, d_shift, epilogue, d_nbr, d_n_out, capacity_out, n_in, dev_flags, cin, cout, rows,
                     (T*)d_out);
}

}  // namespace

extern "C" int32_t emc2_spconv_uses_mfma(emc2_dtype dtype, int32_t cin, int32_t cout) {
  return (dtype == EMC2_F16 || dtype == EMC2_BF16) && emc2_spconv_mfma_supported(cin, cout) ? 1 : 0;
}

// shapes of the thread-per-row vector-ALU kernel (fp32) and of the small-channel matrix-core kernel (16-bit)
static bool small_covers(int cin, int cout) { return (cin == 4 && (cout == 16 || cout == 32)) || (cin == 16 && cout == 16); }
static bool rows_covers(int cin, int cout) { return small_covers(cin, cout); }

extern "C" const char* emc2_spconv_kernel(emc2_dtype dtype, int32_t cin, int32_t cout, int32_t map_hint) {
  if (dtype != EMC2_F32 && dtype != EMC2_F16 && dtype != EMC2_BF16) return nullptr;
  if (emc2_spconv_uses_mfma(dtype, cin, cout)) {
    if (emc2_spconv_narrow_supported(cin, cout)) return "k_spconv_narrow";
    if (emc2_spconv_resident_supported(cin, cout)) return "k_spconv_direct_resident";
    if (!emc2_spconv_direct_supported(cin, cout)) return "k_spconv_mfma";
    return (map_hint == EMC2_CONV_SUBM && emc2_spconv_span_supported(cin, cout)) ? "k_spconv_span" : "k_spconv_direct";
  }
  if (dtype == EMC2_F32) return small_covers(cin, cout) ? "k_spconv_small" : "k_spconv_alu";
  return rows_covers(cin, cout) ? "k_spconv_rows" : "k_spconv_alu";
}

extern "C" emc2_status emc2_pack_weights(emc2_ctx* ctx, emc2_dtype dtype, const void* d_w, int32_t cin, int32_t cout,
                                         void* d_packed, void* stream) {
  if (!ctx) return EMC2_ERR_INVALID_ARG;
  if (!d_w || !d_packed || d_w == d_packed) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_pack_weights: bad pointers");
  if (!emc2_spconv_uses_mfma(dtype, cin, cout))
    return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_pack_weights: (dtype, Cin=%d, Cout=%d) does not use the MFMA path", cin,
                     cout);
  // the fragment order is a function of (Cin, Cout) alone: whichever kernel a call later selects for this
  // shape reads the same packed weights
  if (emc2_spconv_direct_order(cin, cout))
    emc2_spconv_direct_pack(d_w, cin, cout, d_packed, (hipStream_t)stream);
  else
    emc2_spconv_mfma_pack(d_w, cin, cout, d_packed, (hipStream_t)stream);
  return emc2_check_hip(ctx, hipGetLastError(), "emc2_pack_weights launch");
}

// The kernels that a launch can hold several calls of.
enum ConvKind { CONV_SINGLE, CONV_ROWS, CONV_NARROW, CONV_RESIDENT };

static ConvKind kind_of(emc2_dtype dtype, int cin, int cout) {
  if (dtype == EMC2_F32) return CONV_SINGLE;
  if (emc2_spconv_narrow_supported(cin, cout)) return CONV_NARROW;
  if (emc2_spconv_resident_supported(cin, cout)) return CONV_RESIDENT;
  return !emc2_spconv_uses_mfma(dtype, cin, cout) && rows_covers(cin, cout) ? CONV_ROWS : CONV_SINGLE;
}

static emc2_status check_conv(const emc2_conv_call& c) {
  emc2_ctx* ctx = c.ctx;
  if (!ctx) return EMC2_ERR_INVALID_ARG;
  const emc2_dtype dtype = c.dtype;
  const emc2_wlayout w_layout = c.w_layout;
  const emc2_epilogue epilogue = c.epilogue;
  const int32_t map_hint = c.map_hint, cin = c.cin, cout = c.cout;
  const int64_t capacity_out = c.capacity_out, n_in_rows = c.n_in_rows;
  const void *d_in = c.d_in, *d_w = c.d_w, *d_out = c.d_out;
  const float *d_scale = c.d_scale, *d_shift = c.d_shift;
  if (!d_in || !d_w || !c.d_nbr || !c.d_n_out || !d_out)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv: null argument");
  if (epilogue != EMC2_EPI_NONE && epilogue != EMC2_EPI_AFFINE && epilogue != EMC2_EPI_AFFINE_RELU)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv: bad epilogue");
  if ((epilogue == EMC2_EPI_NONE) != (d_scale == nullptr) || (d_scale == nullptr) != (d_shift == nullptr))
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv: scale/shift must be given iff the epilogue is affine");
  if (capacity_out < 1) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv: capacity_out < 1");
  if (n_in_rows < 0) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv: n_in_rows < 0");
  if (cin < 1 || cout < 1 || cin > 1024 || cout > 256)
    return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_spconv: channels outside Cin<=1024, Cout<=256");
  if (dtype != EMC2_F32 && dtype != EMC2_F16 && dtype != EMC2_BF16)
    return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_spconv: bad dtype");
  if (w_layout != EMC2_W_PLAIN && w_layout != EMC2_W_PACKED)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv: bad weight layout");
  if (map_hint != EMC2_MAP_ANY && map_hint != EMC2_CONV_SUBM && map_hint != EMC2_CONV_STRIDED)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv: bad map_hint");
  const bool mfma = emc2_spconv_uses_mfma(dtype, cin, cout) != 0;
  if (w_layout == EMC2_W_PACKED && !mfma)
    return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_spconv: packed weights need an MFMA-covered (dtype, Cin, Cout)");
  // the matrix-core and small-channel kernels move rows as 8- or 16-byte pieces
  if (dtype != EMC2_F32 && (((uintptr_t)d_in | (uintptr_t)d_out | (uintptr_t)d_w) & 15u))
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv: 16-bit d_in, d_w and d_out must be 16-byte aligned");
  return EMC2_OK;
}

// n calls of one kind, checked; of CONV_SINGLE one.
static emc2_status issue_convs(const emc2_conv_call* const* calls, int n, hipStream_t s) {
  const emc2_conv_call& c = *calls[0];
  emc2_ctx* ctx = c.ctx;
  const emc2_dtype dtype = c.dtype;
  const int cin = c.cin, cout = c.cout;
  emc2_conv_args a[kConvBatch];
  for (int i = 0; i < n; ++i) {
    const emc2_conv_call& t = *calls[i];
    const void* w = t.d_w;
    if (t.w_layout == EMC2_W_PLAIN && emc2_spconv_uses_mfma(dtype, cin, cout)) {
      // stream order protects the shared scratch
      if (emc2_spconv_direct_order(cin, cout)) emc2_spconv_direct_pack(w, cin, cout, t.ctx->wpack, s);
      else emc2_spconv_mfma_pack(w, cin, cout, t.ctx->wpack, s);
      w = t.ctx->wpack;
    }
    a[i] = emc2_conv_args{t.d_in, w, t.d_scale, t.d_shift, t.d_nbr, t.d_n_out, t.ctx->zero_row, t.d_out, t.capacity_out,
                          t.n_in_rows > 0x7fffffff ? 0x7fffffff : (int32_t)t.n_in_rows, (int32_t)t.epilogue, t.ctx->dev_words};
  }
  const emc2_conv_args& x = a[0];
  switch (kind_of(dtype, cin, cout)) {
    case CONV_ROWS: launch_rows(dtype, cin, cout, a, n, s); break;
    case CONV_NARROW: emc2_spconv_narrow_launch(dtype, cin, a, n, s); break;
    case CONV_RESIDENT: emc2_spconv_resident_launch(dtype, cin, a, n, s); break;
    default:
#define ALU(T)                                                                                                                    \
  launch_alu<T>(x.d_in, x.d_w, x.d_scale, x.d_shift, x.epilogue, x.d_nbr, x.d_n_out, x.capacity_out, x.n_in, x.dev_flags, cin, cout, \
                x.d_out, s)
      if (dtype == EMC2_F32) ALU(float);
      else if (!emc2_spconv_uses_mfma(dtype, cin, cout)) {
        if (dtype == EMC2_F16) ALU(__half);
        else ALU(__hip_bfloat16);
      }
#undef ALU
      else if (!emc2_spconv_direct_supported(cin, cout))
        emc2_spconv_mfma_launch(dtype, x.d_in, x.d_w, x.d_scale, x.d_shift, x.epilogue, x.d_nbr, x.d_n_out, x.capacity_out, x.n_in,
                                x.dev_flags, cin, cout, x.d_out, s);
      else if (c.map_hint == EMC2_CONV_SUBM && emc2_spconv_span_supported(cin, cout))
        // pays where the three kx taps of a group name nearly the same rows
        emc2_spconv_span_launch(dtype, x.d_in, x.d_w, x.d_scale, x.d_shift, x.epilogue, x.d_nbr, x.d_n_out, x.capacity_out, x.n_in,
                                x.dev_flags, cin, cout, x.d_out, s);
      else
        emc2_spconv_direct_launch(dtype, x.d_in, x.d_w, x.d_scale, x.d_shift, x.epilogue, x.d_nbr, x.d_n_out, x.capacity_out, x.n_in,
                                  x.dev_flags, cin, cout, x.d_zero_row, c.map_hint != EMC2_CONV_SUBM, x.d_out, s);
  }
  return emc2_check_hip(ctx, hipGetLastError(), "emc2_spconv launch");
}

extern "C" emc2_status emc2_spconv(emc2_ctx* ctx, emc2_dtype dtype, const void* d_in, const void* d_w,
                                   emc2_wlayout w_layout, const float* d_scale, const float* d_shift,
                                   emc2_epilogue epilogue, const int32_t* d_nbr, int32_t map_hint,
                                   const int32_t* d_n_out, int64_t capacity_out, int64_t n_in_rows, int32_t cin,
                                   int32_t cout, void* d_out, void* stream) {
  const emc2_conv_call c = {ctx, d_in, d_w, d_scale, d_shift, d_nbr, d_n_out, d_out, capacity_out, n_in_rows, dtype, w_layout, epilogue,
                            map_hint, cin, cout};
  const emc2_status st = check_conv(c);
  if (st != EMC2_OK) return st;
  const emc2_conv_call* one = &c;
  return issue_convs(&one, 1, (hipStream_t)stream);
}

static bool in_launch(const emc2_conv_call* const* batch, int m, const emc2_conv_call* c) {
  for (int i = 0; i < m; ++i)
    if (batch[i] == c) return true;
  return false;
}

constexpr int kListPlanned = 64;     // calls of a list that are looked at together

extern "C" emc2_status emc2_spconv_list(const emc2_conv_call* calls, int32_t n, void* stream) {
  if (n < 0 || (n > 0 && !calls)) return EMC2_ERR_INVALID_ARG;
  for (int32_t i = 0; i < n; ++i)
    if (!calls[i].ctx) return emc2_fail(calls[0].ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv_list: call %d has no context", i);
  // Calls of one kernel that do not wait for anything still to be issued share a launch: small levels of several branches -- three
  // scales of a frame, experts without a scene -- fill a fraction of the chip each and take a launch's 4.5 us at least, and one
  // after the other each ends in a tail of its own.  4 -> 16 -> 32 of three scales (64-beam frame): 6 launches 68 us, 2 launches 41;
  // five small scenes' layers 1373 -> 1330 us a pass.  Otherwise the order stays that of the list.  (Plain weights of the matrix
  // kernels go through scratch, one call at a time.)
  emc2_status refused = EMC2_OK;
  int32_t end = 0;                     // the first refused call: nothing behind it is issued
  while (end < n && (refused = check_conv(calls[end])) == EMC2_OK) ++end;
  bool done[kListPlanned] = {};
  emc2_touched t[kListPlanned];
  const bool planned = end <= kListPlanned;
  for (int32_t i = 0; planned && i < end; ++i) t[i] = emc2_touched_by(calls[i]);
  const emc2_conv_call* at = nullptr;
  emc2_status st = EMC2_OK;
  for (int32_t i = 0; st == EMC2_OK && i < end; ++i) {
    if (planned && done[i]) continue;
    const emc2_conv_call& c = calls[i];
    const emc2_conv_call* batch[kConvBatch] = {&c};
    int m = 1;
    if (planned && kind_of(c.dtype, c.cin, c.cout) != CONV_SINGLE &&
        (c.w_layout == EMC2_W_PACKED || !emc2_spconv_uses_mfma(c.dtype, c.cin, c.cout))) {
      for (int32_t j = i + 1; j < end && m < kConvBatch; ++j) {
        const emc2_conv_call& d = calls[j];
        if (done[j] || d.dtype != c.dtype || d.cin != c.cin || d.cout != c.cout || d.w_layout != c.w_layout) continue;
        bool waits = false;             // for an earlier call still to be issued, or for one of this launch
        for (int32_t k = i; !waits && k < j; ++k) waits = (!done[k] || k == i || in_launch(batch, m, calls + k)) && emc2_ordered(t[k], t[j]);
        if (waits) continue;
        batch[m++] = &d;
        done[j] = true;
      }
    }
    st = issue_convs(batch, m, (hipStream_t)stream);
    at = &c;
  }
  if (st == EMC2_OK && end < n) st = refused, at = calls + end;
  // the caller asks the first call's context what went wrong, whichever call it was
  if (st != EMC2_OK && at->ctx != calls[0].ctx) emc2_fail(calls[0].ctx, st, "%s", at->ctx->err);
  return st;
}
