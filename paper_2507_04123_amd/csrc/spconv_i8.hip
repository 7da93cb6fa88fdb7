// Quantised sparse convolution on the int8 matrix cores (paper Sec. 3.6 (2): model quantisation is one of the
// deployment optimisations; the paper gives no scheme, the one here is stated in emc2.h).
//
// As in the register-direct 16-bit kernels: v_mfma_i32_16x16x64_i8 takes, in lane (m = lane % 16,
// q = lane / 16), the 16 consecutive input channels 16q .. 16q+15 of row m of the tile, i.e. 16 contiguous bytes
// of the feature row nbr[k][o_m]; a 64-channel int8 row is exactly the four lanes' 64 bytes, so ONE
// global_load_dwordx4 per 16-row tile and tap is the operand (half the bytes and half the cache lines of the
// fp16 kernel, twice the multiply-accumulates per matrix instruction).  Absent neighbours read past the end of the input's buffer
// descriptor, which yields zeros (4 GiB and more: a zeroed row).
// Up to 64 x 64 and 128 x 32 channels (110 KB of weights at most) a block keeps all weights in LDS and its waves take tiles by
// themselves (resident_walk.h); 128 -> 64 takes the weights of a tap at a time.  The former for all shapes / so, us, submanifold, int8
// and E4M3: 64 -> 64 69 k rows 16.7 / 13.1 and 18.0 / 15.0, 165 k 28.8 / 24.6 and 30.8 / 25.3, 304 k 43 / 37 and 48 / 41, stride-2 69 k
// 19.6 / 15.0, transposed 223 k 28 / 22; 64 -> 32 69 k 14.2 / 10.1; 128 -> 32 304 k 87 / 57.  What that form lost: a barrier and a copy of
// weights a tap, taps that none of a wave's rows have, and the last round of blocks.  Maps that name any row from anywhere, for which it has fewer
// waves to a CU, are 6 to 18 % faster so up to 30 k rows and within -9 and +7 % beyond (64 -> 64 223 k rows 35.0 / 37.0, E4M3 38.8 / 41.1).
// Accumulation is exact (int32); the epilogue is
// a fixed sequence of individually rounded fp32 operations, so results are bit-reproducible.
#include <hip/hip_fp16.h>

#include "common.h"
#include "resident_walk.h"

#pragma clang fp contract(off)

namespace {

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kQWaves = 4;
constexpr int kQThreads = kQWaves * 64;

__device__ __forceinline__ int quant_i8(float v, float inv_scale) {
  float r = rintf(v * inv_scale);  // to nearest, ties to even
  if (!(r == r)) r = 0.f;
  r = r > 127.f ? 127.f : r;
  r = r < -127.f ? -127.f : r;
  return (int)r;
}

// E4M3 (bias 7, no infinities, largest value 448): nearest finite value of t, ties to the even code, saturating,
// NaN -> 0, a result of zero always +0.  Integer arithmetic on the fp32 bits, so that no conversion mode of the
// hardware enters: above the subnormal range the 20 low mantissa bits are rounded away (the carry runs into the
// exponent by itself); below 2^-6 the value is a multiple of 2^-9.
__device__ __forceinline__ uint32_t quant_e4m3(float t) {
  if (!(t == t)) return 0u;
  const float a = fabsf(t);
  uint32_t code;
  if (a >= 448.0f) {
    code = 0x7Eu;
  } else if (a < 0.015625f) {
    code = (uint32_t)rintf(a * 512.0f);          // exact product; ties to even; 8 is the first normal code
  } else {
    const uint32_t bits = __float_as_uint(a);
    const uint32_t r = (bits + 0x7FFFFu + ((bits >> 20) & 1u)) >> 20;   // (exponent << 3 | mantissa), rounded to nearest even
    code = r - (120u << 3);
    code = code > 0x7Eu ? 0x7Eu : code;          // 464 .. 448 rounds up to a code that is not a number: saturate
  }
  return (code != 0u && t < 0.0f) ? (code | 0x80u) : code;
}

template <bool E4M3>
__device__ __forceinline__ uint32_t quant_code(float v, float inv_scale) {
  if constexpr (E4M3) return quant_e4m3(v * inv_scale);
  else return (uint32_t)quant_i8(v, inv_scale) & 0xffu;
}

// The codes of four values, the first in the low byte.
template <bool E4M3>
__device__ __forceinline__ uint32_t quant_codes(const float (&v)[4], float inv_scale) {
  uint32_t o = 0u;
  if constexpr (E4M3) {
    // The conversion rounds as quant_e4m3 does, subnormals included (compared for all 2^32 values); what it does not say itself: numbers
    // beyond 448 saturate, what is not a number is 0, and so is what rounds to -0.
    float t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float x = v[k] * inv_scale;
      t[k] = x == x ? __builtin_amdgcn_fmed3f(x, -448.0f, 448.0f) : 0.0f;
    }
    o = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(t[0], t[1], 0, false);
    o = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(t[2], t[3], (int)o, true);
    const uint32_t some = (o & 0x7f7f7f7fu) + 0x7f7f7f7fu;      // a byte's top bit: its other seven are not all zero
    o &= some | 0x7f7f7f7fu;
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) o |= ((uint32_t)quant_i8(v[k], inv_scale) & 0xffu) << (8 * k);
  }
  return o;
}

// Elementwise, bound by memory: at one value a thread (2 bytes in, 1 out) a launch was bound by its wave count, 21.2 us
// for 223 k x 64 values (2.0 TB/s) in int8; now 9.5 (4.5 TB/s).  E4M3, 165 k x 64, with the codes put together from the values' bits /
// by the conversion, 8.6 / 6.2 us.  VEC: a thread turns 8 values into one 8-byte store, its loads 16 bytes wide (two of
// them for fp32), which needs x 16-byte and q 8-byte aligned; any other address takes the one-value form.  16 values a thread: the
// same; two and four such pieces a thread, all requested first: int8 10.0 and 11.0, E4M3 7.2 and 7.3.
template <typename T, bool E4M3, bool VEC>
__global__ void __launch_bounds__(256) k_quantize(const T* __restrict__ x, int64_t n, float inv_scale, uint8_t* __restrict__ q) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if constexpr (VEC) {
    const int64_t i = t * 8;
    if (i + 8 <= n) {
      alignas(16) T v[8];
#pragma unroll
      for (int k = 0; k < (int)sizeof(v) / 16; ++k)
        reinterpret_cast<u32x4*>(v)[k] = reinterpret_cast<const u32x4*>(x + i)[k];
      u32x2 o;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float f[4] = {(float)v[4 * h], (float)v[4 * h + 1], (float)v[4 * h + 2], (float)v[4 * h + 3]};
        o[h] = quant_codes<E4M3>(f, inv_scale);
      }
      *reinterpret_cast<u32x2*>(q + i) = o;
    } else {
      for (int64_t k = i; k < n; ++k) q[k] = (uint8_t)quant_code<E4M3>((float)x[k], inv_scale);
    }
  } else {
    if (t < n) q[t] = (uint8_t)quant_code<E4M3>((float)x[t], inv_scale);
  }
}

template <typename T, bool E4M3>
void launch_quantize(const void* d_x, int64_t n, float inv_scale, void* d_q, hipStream_t s) {
  if ((((uintptr_t)d_x & 15u) | ((uintptr_t)d_q & 7u)) == 0)
    hipLaunchKernelGGL((k_quantize<T, E4M3, true>), dim3((unsigned)emc2_div_up(n, 8 * 256)), dim3(256), 0, s, (const T*)d_x, n,
                       inv_scale, (uint8_t*)d_q);
  else
    hipLaunchKernelGGL((k_quantize<T, E4M3, false>), dim3((unsigned)emc2_div_up(n, 256)), dim3(256), 0, s, (const T*)d_x, n,
                       inv_scale, (uint8_t*)d_q);
}

// Packed layout: 16-byte piece ((k*KS + t)*NT + j)*64 + lane, lane = 16*q + n, holds W[k][64t + 16q + e][16j + n],
// e = 0..15 -- the B operand of k-step t, column tile j.
__global__ void __launch_bounds__(256) k_pack_weights_i8(const int8_t* __restrict__ w, int cin, int cout, uint4* __restrict__ packed) {
  const int ks = cin / 64, nt = cout / 16;
  const int total = 27 * ks * nt * 64;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= total) return;
  const int lane = p & 63;
  int f = p >> 6;
  const int j = f % nt; f /= nt;
  const int t = f % ks; f /= ks;
  const int k = f;
  const int n = 16 * j + (lane & 15);
  const int c0 = 64 * t + 16 * (lane >> 4);
  const int8_t* src = w + ((int64_t)k * cin + c0) * cout + n;
  uint32_t v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t word = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) word |= (uint32_t)(uint8_t)src[(int64_t)(4 * e + b) * cout] << (8 * b);
    v[e] = word;
  }
  packed[p] = make_uint4(v[0], v[1], v[2], v[3]);
}

// F8: 0 = int8 operands, exact int32 accumulation (v_mfma_i32_16x16x64_i8); 1 = E4M3 operands, fp32 accumulation
//     (two v_mfma_f32_16x16x32_fp8_fp8 per 16-byte operand: its low and its high 8 bytes; features and packed weights
//     split the same way, so the contraction pairs the same channels).
// OUTQ: int8 operands: 1 = int8 output (re-quantised), 0 = fp16 output; E4M3 operands: 1 = fp32 output, 0 = fp16 output.
// 128 -> 64.  Rows a wave: a launch is bound by the chain of 27 taps (operand latency, weights through LDS, a barrier each) until enough
// waves cover each other, then by LDS reads of weights, which feed half the products with 32 rows a wave that they feed with
// 64.  A level of up to kQSmall rows, three blocks of 32-row waves a CU, runs those.  Beyond, int8 runs 64 rows,
// but a step of them, a block a CU, takes nearly as long if few of its blocks are there, so that a rest of less than half a
// step runs 32 rows, behind the whole steps of the same launch: all 64 rows / all 32 / both, fp16 out, 223 k rows 86 / 81 / 73 us.
// The row count is the device's, so the kernel holds both forms.  E4M3 runs two matrix instructions for every operand read, so that
// 32 rows are the better ones nearly everywhere (60 / 52, 76 / 69, 112 / 115).
constexpr int64_t kQSmall = 3 * 256 * 128;
constexpr int64_t kQStep = 256 * 256;    // rows of a block of 64-row waves a CU

// TALL: holds the form with 64 rows a wave too.  MINW: waves per SIMD the register allocator must leave room for, as many as
// neither form spills at.
template <int F8> struct QCfg {
  static constexpr bool TALL = !F8;
  static constexpr int MINW = TALL ? 2 : 3;
};

template <int F8> struct QAcc { typedef intx4 type; };
template <> struct QAcc<1> { typedef floatx4 type; };

// Input rows through a buffer descriptor, as in the register-direct 16-bit kernel: zeros at or beyond its end.
// Against a zeroed row, with the kernel below for all shapes: layers of a 64-beam frame with their quantiser int8 138 -> 130 us.
__device__ __forceinline__ u32x4 buffer_row16(__amdgpu_buffer_rsrc_t rows, uint32_t byte) {
  return __builtin_amdgcn_raw_buffer_load_b128(rows, (int)byte, 0, 0);
}

template <int CIN, int COUT, int OUTQ, int F8> struct QLds {
  static constexpr int W16 = CIN / 64 * (COUT / 16) * 64;    // 16-byte weight pieces per tap
  static constexpr int ES = F8 ? (OUTQ ? 4 : 2) : (OUTQ ? 1 : 2);   // bytes per output element
  static constexpr int OCH = COUT * ES / 16;                 // 16-byte pieces per output row
  u32x4 w[2][W16];
  u32x4 otile[kQWaves][16 * (OCH + 1)];
};

// One block's rows, 16 * MT a wave: tile `slot` of this block's XCD among those of rows [row_begin, n_out).
template <int CIN, int COUT, int OUTQ, int F8, bool BUF, int MT>
__device__ __forceinline__ void
run_i8(int64_t slot, int64_t row_begin, QLds<CIN, COUT, OUTQ, F8>& lds, const int8_t* __restrict__ in, const u32x4* __restrict__ wp,
       const float* __restrict__ mul, const float* __restrict__ add, int relu, float inv_out_scale, const int32_t* __restrict__ nbr,
       int64_t n_out, int64_t capacity_out, int32_t n_in, int32_t* __restrict__ dev_flags, const int8_t* __restrict__ zrow,
       void* __restrict__ out) {
  const __amdgpu_buffer_rsrc_t rows =
      __builtin_amdgcn_make_buffer_rsrc((void*)const_cast<int8_t*>(in), 0, BUF ? (int)((uint32_t)n_in * CIN) : 0, 0x00020000);
  constexpr int KS = CIN / 64;                // k-steps per tap
  constexpr int NT = COUT / 16;               // 16-column tiles
  constexpr int R = 16 * MT;                  // rows per wave
  constexpr int W16 = QLds<CIN, COUT, OUTQ, F8>::W16;
  constexpr int WPT = (W16 + kQThreads - 1) / kQThreads;
  static_assert(MT == 2 || MT == 4, "the lane-swap broadcast below handles two or four tiles");
  static_assert((W16 & (W16 - 1)) == 0, "piece count is a power of two");
  constexpr int WMASK = W16 - 1;              // surplus threads copy redundantly rather than under a branch
  constexpr int NA = MT * KS;                 // A-operand loads per tap
  constexpr int ES = QLds<CIN, COUT, OUTQ, F8>::ES, OCH = QLds<CIN, COUT, OUTQ, F8>::OCH;
  constexpr int OPITCH = (OCH + 1) * 16;      // epilogue tile row pitch in bytes
  u32x4 (*wl)[W16] = lds.w;

  // XCD-aware tile assignment: workgroup b runs on XCD b % 8; XCD x takes a contiguous range of tiles
  const int64_t n_tiles = (n_out - row_begin + kQWaves * R - 1) / (kQWaves * R);
  const int64_t chunk = (n_tiles + 7) / 8;
  const int64_t tile_id = (int64_t)(blockIdx.x % 8) * chunk + slot;
  if (slot >= chunk || tile_id >= n_tiles) return;         // uniform for the block

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int m = lane & 15, q = lane >> 4;
  const int64_t wave_row0 = row_begin + tile_id * (kQWaves * R) + (int64_t)wave * R;

  // lane l holds the kernel-map entries of row l % R of this wave's R rows
  const bool live = wave_row0 + lane % R < n_out;
  const int32_t* nrow = nbr + (live ? wave_row0 + lane % R : 0);
  const int32_t dead = live ? 0 : -1;   // OR-ed into kernel-map entries: rows past n_out have no neighbours
  unsigned long long oob = 0ull;        // lanes that saw an entry outside [0, n_in)

  typedef typename QAcc<F8>::type acc_t;
  acc_t acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[mt][j] = acc_t{0, 0, 0, 0};

  int32_t jq[3][3];         // kernel-map entries of groups g, g+1, g+2 (as loaded; masked where used)
  u32x4 areg[3][NA];        // A operands in flight; tap x lives in set x % 3
  u32x4 wq[3][WPT];         // weights in flight; tap x lives in set x % 3

#define EMC2_IDX_LOAD(GROUP, DST)                                                                        \
  _Pragma("unroll") for (int kx_ = 0; kx_ < 3; ++kx_)                                                    \
      jq[DST][kx_] = nrow[(int64_t)(3 * ((GROUP) < 9 ? (GROUP) : 8) + kx_) * capacity_out];
  // A operands of one tap: tile mt, k-step ks <- 16 bytes at channel 64*ks + 16*q of row JROW[16*mt + m].
  // Lane-swap instructions broadcast each 16-lane row of the entries (0123, of 32 rows 0101) to all four rows.
#define EMC2_A_LOAD(JROW, SET)                                                                           \
  {                                                                                                      \
    const uint32_t jr_ = (uint32_t)max((JROW), -1);   /* any negative entry is an absent neighbour */    \
    u32x2 h_ = {jr_, jr_};                                                                               \
    if constexpr (MT == 4) h_ = __builtin_amdgcn_permlane32_swap(jr_, jr_, false, false);  /* 0101 | 2323 */ \
    const u32x2 lo_ = __builtin_amdgcn_permlane16_swap(h_[0], h_[0], false, false);  /* 0000 | 1111 */   \
    const u32x2 hi_ = __builtin_amdgcn_permlane16_swap(h_[1], h_[1], false, false);  /* 2222 | 3333 */   \
    const int32_t jm_[4] = {(int32_t)lo_[0], (int32_t)lo_[1], (int32_t)hi_[0], (int32_t)hi_[1]};         \
  _Pragma("unroll") for (int mt_ = 0; mt_ < MT; ++mt_) {                                                 \
    const int32_t j_ = jm_[mt_];                                                                         \
    if constexpr (BUF) {                                                                                 \
      /* absent: 2^32 less a row, and a piece of the row: out of range, zero */                          \
      const uint32_t at_ = (uint32_t)j_ * (uint32_t)CIN + 16u * (uint32_t)q;                             \
      _Pragma("unroll") for (int ks_ = 0; ks_ < KS; ++ks_)                                               \
          areg[SET][mt_ * KS + ks_] = buffer_row16(rows, at_ + 64u * (uint32_t)ks_);                     \
    } else {                                                                                             \
      const int8_t* src_ = (j_ >= 0 ? in + (int64_t)j_ * CIN : zrow) + 16 * q;                           \
      _Pragma("unroll") for (int ks_ = 0; ks_ < KS; ++ks_)                                               \
          areg[SET][mt_ * KS + ks_] = *reinterpret_cast<const u32x4*>(src_ + 64 * ks_);                  \
    }                                                                                                    \
  }                                                                                                      \
  }
#define EMC2_W_LOAD(TAP, SET)                                                                            \
  {                                                                                                      \
    const u32x4* wsrc_ = wp + (int64_t)(TAP) * W16;                                                      \
    _Pragma("unroll") for (int i_ = 0; i_ < WPT; ++i_)                                                   \
        wq[SET][i_] = wsrc_[(threadIdx.x + i_ * kQThreads) & WMASK];                                     \
  }
#define EMC2_W_STORE(BUF, SET)                                                                           \
  _Pragma("unroll") for (int i_ = 0; i_ < WPT; ++i_)                                                     \
      wl[BUF][(threadIdx.x + i_ * kQThreads) & WMASK] = wq[SET][i_];

  // prologue: map entries of groups 0..2; weights of tap 0 to LDS; A operands of taps 0..2
  EMC2_IDX_LOAD(0, 0)
  EMC2_IDX_LOAD(1, 1)
  EMC2_IDX_LOAD(2, 2)
  EMC2_W_LOAD(0, 0)
  EMC2_W_STORE(0, 0)
  EMC2_W_LOAD(1, 1)
  EMC2_W_LOAD(2, 2)
  EMC2_A_LOAD(emc2_entry(jq[0][0], dead, n_in, oob), 0)
  EMC2_A_LOAD(emc2_entry(jq[0][1], dead, n_in, oob), 1)
  EMC2_A_LOAD(emc2_entry(jq[0][2], dead, n_in, oob), 2)
  __syncthreads();

  for (int g = 0; g < 9; ++g) {
    // kernel-map entries of group g + 3, requested a whole group before anything touches them
    int32_t jn[3];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) jn[kx] = nrow[(int64_t)(3 * (g + 3 < 9 ? g + 3 : 8) + kx) * capacity_out];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
      const int tap = 3 * g + kx;
      EMC2_W_LOAD(tap + 3 < 27 ? tap + 3 : 26, kx)   // weights of tap + 3: global -> registers
      const u32x4* wb = wl[tap & 1];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        u32x4 b[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) b[j] = wb[(ks * NT + j) * 64 + lane];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            if constexpr (F8) {
              const u32x4 av = areg[kx][mt * KS + ks], bv = b[j];
              const long a_lo = (long)(((unsigned long)av.y << 32) | av.x), a_hi = (long)(((unsigned long)av.w << 32) | av.z);
              const long b_lo = (long)(((unsigned long)bv.y << 32) | bv.x), b_hi = (long)(((unsigned long)bv.w << 32) | bv.z);
              acc[mt][j] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a_lo, b_lo, acc[mt][j], 0, 0, 0);
              acc[mt][j] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a_hi, b_hi, acc[mt][j], 0, 0, 0);
            } else {
              acc[mt][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(intx4, areg[kx][mt * KS + ks]),
                                                                 __builtin_bit_cast(intx4, b[j]), acc[mt][j], 0, 0, 0);
            }
          }
      }
      // the freed register set takes the A operands of tap + 3 (entries of "group 9" do not exist)
      const int32_t past = g < 8 ? 0 : -1;
      EMC2_A_LOAD(emc2_entry(jq[1][kx], dead | past, n_in, oob), kx)
      __builtin_amdgcn_wave_barrier();
      // weights of tap + 1: registers -> the other LDS buffer; the barrier publishes them and retires the one just read
      EMC2_W_STORE((tap + 1) & 1, (kx + 1) % 3)
      __syncthreads();
    }
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
      jq[0][kx] = jq[1][kx];
      jq[1][kx] = jq[2][kx];
      jq[2][kx] = jn[kx];
    }
  }
#undef EMC2_IDX_LOAD
#undef EMC2_A_LOAD
#undef EMC2_W_LOAD
#undef EMC2_W_STORE
  emc2_report_oob(oob, dev_flags);

  // epilogue: lane (m, q) holds column 16*j + m of rows 16*mt + 4*q + e.  int -> fp32, multiply, add (each rounded
  // on its own), ReLU, convert; each 16-row tile goes through LDS so that global stores are whole 16-byte pieces.
  float ml[NT], ad[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    ml[j] = mul[16 * j + m];
    ad[j] = add[16 * j + m];
  }
  uint8_t* otile = reinterpret_cast<uint8_t*>(lds.otile[wave]);
  constexpr int OPI = 64 / OCH;               // rows one store instruction covers
  constexpr int ONI = (16 + OPI - 1) / OPI;   // store instructions per 16-row tile
  const int orow = lane / OCH, ochunk = lane % OCH;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = (float)acc[mt][j][e];
        v = v * ml[j];
        v = v + ad[j];
        if (relu) v = v > 0.f ? v : 0.f;
        uint8_t* dst = otile + (4 * q + e) * OPITCH + (16 * j + m) * ES;
        if (F8 && OUTQ) *reinterpret_cast<float*>(dst) = v;
        else if (OUTQ) *reinterpret_cast<int8_t*>(dst) = (int8_t)quant_i8(v, inv_out_scale);
        else *reinterpret_cast<uint16_t*>(dst) = __half_as_ushort(__float2half_rn(v));
      }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < ONI; ++i) {
      const int r = i * OPI + orow;
      if (r < 16) {
        const u32x4 piece = *reinterpret_cast<const u32x4*>(otile + r * OPITCH + ochunk * 16);
        const int64_t o = wave_row0 + mt * 16 + r;
        if (o < n_out) *reinterpret_cast<u32x4*>(reinterpret_cast<uint8_t*>(out) + o * (COUT * ES) + ochunk * 16) = piece;
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

template <int CIN, int COUT, int OUTQ, int F8, bool BUF>
__global__ void __launch_bounds__(kQThreads, (QCfg<F8>::MINW))
k_spconv_i8(const int8_t* __restrict__ in, const u32x4* __restrict__ wp, const float* __restrict__ mul,
            const float* __restrict__ add, int relu, float inv_out_scale, const int32_t* __restrict__ nbr,
            const int32_t* __restrict__ d_n_out, int64_t capacity_out, int32_t n_in, int32_t* __restrict__ dev_flags,
            const int8_t* __restrict__ zrow, void* __restrict__ out) {
  __shared__ QLds<CIN, COUT, OUTQ, F8> lds;
  int64_t n_out = *d_n_out;
  if (n_out > capacity_out) n_out = capacity_out;
  // rows [0, tall) in tiles of 64-row waves, the others in tiles of 32-row waves
  using Cfg = QCfg<F8>;
  int64_t slot = blockIdx.x / 8, tall = 0;
  if constexpr (Cfg::TALL) {
    if (n_out > kQSmall) {
      tall = n_out - n_out % kQStep;
      if (n_out - tall >= kQStep / 2) tall = n_out;
    }
  }
  const int64_t tall_slots = (tall + 8 * kQWaves * 64 - 1) / (8 * kQWaves * 64);
  // Blocks without a tile, of which a large capacity has many, end before anything else is computed: 40 k rows in a capacity of
  // 6 M, int8 64 -> 64 13.6 -> 11.0, 64 -> 32 12.7 -> 10.1, 128 -> 64 20.9 -> 18.0.
  if ((slot - tall_slots) * (8 * kQWaves * 32) >= n_out - tall + 7 * kQWaves * 32) return;
  if constexpr (Cfg::TALL) {
    if (slot < tall_slots) {
      run_i8<CIN, COUT, OUTQ, F8, BUF, 4>(slot, 0, lds, in, wp, mul, add, relu, inv_out_scale,
                                          nbr, tall, capacity_out, n_in, dev_flags, zrow, out);
      return;
    }
    slot -= tall_slots;
  }
  run_i8<CIN, COUT, OUTQ, F8, BUF, 2>(slot, tall, lds, in, wp, mul, add, relu, inv_out_scale,
                                      nbr, n_out, capacity_out, n_in, dev_flags, zrow, out);
}

// Shapes whose weights a CU's LDS holds whole: the walk of resident_walk.h.
template <int CIN, int COUT, int OUTQ, int F8> struct Op8 {
  static constexpr int KS = CIN / 64, NT = COUT / 16;
  template <bool BUF> static constexpr int waves =
      BUF && (F8 || CIN == 128 || COUT == 32) ? emc2_resident::kRWaves : emc2_resident::kRWavesWide;
  static constexpr bool kRowsFirst = CIN == 64 && (COUT == 32 || !F8);
  typedef typename QAcc<F8>::type acc_t;
  const float *mul, *add;
  int relu;
  float inv_out_scale;
  void* out;
  static __device__ __forceinline__ acc_t run(u32x4 w, u32x4 a, acc_t c) {
    if constexpr (F8) {
      const long w_lo = (long)(((unsigned long)w.y << 32) | w.x), w_hi = (long)(((unsigned long)w.w << 32) | w.z);
      const long a_lo = (long)(((unsigned long)a.y << 32) | a.x), a_hi = (long)(((unsigned long)a.w << 32) | a.z);
      c = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(w_lo, a_lo, c, 0, 0, 0);
      return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(w_hi, a_hi, c, 0, 0, 0);
    } else {
      return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(intx4, w), __builtin_bit_cast(intx4, a), c, 0, 0, 0);
    }
  }
  // int -> fp32, multiply, add (each rounded on its own), ReLU, convert; lane swaps gather a lane's 16 (or, of 32 int8 columns, 8) bytes
  // of a row.
  __device__ __forceinline__ void store(int64_t row0, int m, int q, int64_t n_out, acc_t (&acc)[2][NT]) const {
    uint32_t w[2][NT];                        // int8: four channels each
#pragma unroll
    for (int jp = 0; jp < NT / 2; ++jp) {
      floatx4 ml[2], ad[2];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ml[t][e] = mul[16 * (2 * jp + t) + 4 * q + e];
          ad[t][e] = add[16 * (2 * jp + t) + 4 * q + e];
        }
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const int64_t o = row0 + 16 * mt + m;
        u32x2 h[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          floatx4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float x = (float)acc[mt][2 * jp + t][e];
            x = x * ml[t][e];
            x = x + ad[t][e];
            if (relu) x = x > 0.f ? x : 0.f;
            v[e] = x;
          }
          if constexpr (F8 && OUTQ) {
            if (o < n_out) *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(out) + o * COUT + 16 * (2 * jp + t) + 4 * q) = v;
          } else if constexpr (OUTQ) {
            uint32_t p = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) p |= ((uint32_t)quant_i8(v[e], inv_out_scale) & 0xffu) << (8 * e);
            w[mt][2 * jp + t] = p;
          } else {
#pragma unroll
            for (int e = 0; e < 2; ++e)
              h[t][e] = (uint32_t)__half_as_ushort(__float2half_rn(v[2 * e])) | (uint32_t)__half_as_ushort(__float2half_rn(v[2 * e + 1])) << 16;
          }
        }
        if constexpr (!OUTQ) {
          const u32x2 x = __builtin_amdgcn_permlane16_swap(h[0][0], h[1][0], false, false);
          const u32x2 y = __builtin_amdgcn_permlane16_swap(h[0][1], h[1][1], false, false);
          if (o < n_out)
            *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(out) + o * COUT + 32 * jp + 8 * (2 * (q & 1) + (q >> 1))) =
                u32x4{x[0], y[0], x[1], y[1]};
        }
      }
    }
    if constexpr (!F8 && OUTQ) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const int64_t o = row0 + 16 * mt + m;
        uint8_t* dst = reinterpret_cast<uint8_t*>(out) + o * COUT;
        if constexpr (NT == 4) {   // rows of lanes and column tiles change places
          const u32x2 a = __builtin_amdgcn_permlane32_swap(w[mt][0], w[mt][2], false, false);
          const u32x2 b = __builtin_amdgcn_permlane32_swap(w[mt][1], w[mt][3], false, false);
          const u32x2 c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
          const u32x2 d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
          if (o < n_out) *reinterpret_cast<u32x4*>(dst + 16 * q) = u32x4{c[0], c[1], d[0], d[1]};
        } else {
          const u32x2 x = __builtin_amdgcn_permlane16_swap(w[mt][0], w[mt][1], false, false);
          if (o < n_out) *reinterpret_cast<u32x2*>(dst + 16 * (q & 1) + 8 * (q >> 1)) = x;
        }
      }
    }
  }
};

template <int CIN, int COUT, int OUTQ, int F8, bool BUF>
__global__ void __launch_bounds__((Op8<CIN, COUT, OUTQ, F8>::template waves<BUF> * 64))
k_spconv_i8_resident(const int8_t* __restrict__ in, const u32x4* __restrict__ wp, const float* __restrict__ mul,
                     const float* __restrict__ add, int relu, float inv_out_scale, const int32_t* __restrict__ nbr,
                     const int32_t* __restrict__ d_n_out, int64_t capacity_out, int32_t n_in, int32_t* __restrict__ dev_flags,
                     const int8_t* __restrict__ zrow, void* __restrict__ out) {
  const Op8<CIN, COUT, OUTQ, F8> op = {mul, add, relu, inv_out_scale, out};
  emc2_resident::walk<Op8<CIN, COUT, OUTQ, F8>, BUF>(op, blockIdx.x, gridDim.x, in, wp, nbr, d_n_out, capacity_out, n_in, dev_flags, zrow);
}

template <int CIN, int COUT, int OUTQ, int F8 = 0>
void launch_i8(const void* d_in, const void* d_wp, const float* d_mul, const float* d_add, int relu, float inv_out_scale,
               const int32_t* d_nbr, const int32_t* d_n_out, int64_t capacity_out, int32_t n_in, int32_t* dev_flags,
               const void* d_zero_row, void* d_out, hipStream_t s) {
  // Offsets into the input are 32-bit, and the absent neighbour's, 2^32 less a row, must lie at or beyond its end.
  const bool buf = ((int64_t)n_in + 1) * CIN <= ((int64_t)1 << 32);
  if constexpr (CIN * COUT <= 4096) {       // the LDS of a CU holds the weights of all taps
    const int64_t own = emc2_div_up(emc2_div_up(capacity_out, emc2_resident::kRRows), 8) * 8;
    const unsigned blocks = (unsigned)(own < emc2_resident::kRCUs ? own : emc2_resident::kRCUs);
#define LAUNCH(BUF)                                                                                                           \
  hipLaunchKernelGGL((k_spconv_i8_resident<CIN, COUT, OUTQ, F8, BUF>), dim3(blocks),                                          \
                     dim3(Op8<CIN, COUT, OUTQ, F8>::template waves<BUF> * 64), 0, s, (const int8_t*)d_in, (const u32x4*)d_wp, d_mul, d_add,    \
                     relu, inv_out_scale, d_nbr, d_n_out, capacity_out, n_in, dev_flags, (const int8_t*)d_zero_row, d_out)
    if (buf) LAUNCH(true);
    else LAUNCH(false);
#undef LAUNCH
  } else {
    int64_t blocks = emc2_div_up(capacity_out, kQWaves * 32);
    if (QCfg<F8>::TALL && capacity_out > kQSmall) {
      // kQSmall rows in small tiles, or whole steps in large ones and half a step in small ones
      const int64_t mixed = capacity_out / (kQWaves * 64) + kQStep / 2 / (kQWaves * 32) + 1;
      blocks = mixed > kQSmall / (kQWaves * 32) ? mixed : kQSmall / (kQWaves * 32);
    }
#define LAUNCH(BUF)                                                                                                           \
  hipLaunchKernelGGL((k_spconv_i8<CIN, COUT, OUTQ, F8, BUF>), dim3((unsigned)(blocks + 8)),            \
                     dim3(kQThreads), 0, s, (const int8_t*)d_in, (const u32x4*)d_wp, d_mul, d_add, relu, inv_out_scale, d_nbr, \
                     d_n_out, capacity_out, n_in, dev_flags, (const int8_t*)d_zero_row, d_out)
    if (buf) LAUNCH(true);
    else LAUNCH(false);
#undef LAUNCH
  }
}

bool i8_shape_ok(int cin, int cout) { return (cin == 64 || cin == 128) && (cout == 32 || cout == 64); }

}  // namespace

extern "C" int32_t emc2_spconv_i8_supported(int32_t cin, int32_t cout) { return i8_shape_ok(cin, cout) ? 1 : 0; }

extern "C" emc2_status emc2_quantize_i8(emc2_ctx* ctx, emc2_dtype dtype, const void* d_x, int64_t n, float inv_scale,
                                        int8_t* d_q, void* stream) {
  if (!ctx) return EMC2_ERR_INVALID_ARG;
  if (n < 0 || (n > 0 && (!d_x || !d_q))) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_quantize_i8: bad argument");
  if (!(inv_scale == inv_scale)) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_quantize_i8: inv_scale is not a number");
  if (n == 0) return EMC2_OK;
  hipStream_t s = (hipStream_t)stream;
  if (dtype == EMC2_F32) launch_quantize<float, false>(d_x, n, inv_scale, d_q, s);
  else if (dtype == EMC2_F16) launch_quantize<__half, false>(d_x, n, inv_scale, d_q, s);
  else return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_quantize_i8: input must be F32 or F16");
  return emc2_check_hip(ctx, hipGetLastError(), "emc2_quantize_i8 launch");
}

extern "C" emc2_status emc2_pack_weights_i8(emc2_ctx* ctx, const int8_t* d_w, int32_t cin, int32_t cout, void* d_packed,
                                            void* stream) {
  if (!ctx) return EMC2_ERR_INVALID_ARG;
  if (!d_w || !d_packed) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_pack_weights_i8: null argument");
  if (!i8_shape_ok(cin, cout))
    return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_pack_weights_i8: Cin must be 64 or 128 and Cout 32 or 64");
  const int total = 27 * (cin / 64) * (cout / 16) * 64;
  hipLaunchKernelGGL(k_pack_weights_i8, dim3((unsigned)emc2_div_up(total, 256)), dim3(256), 0, (hipStream_t)stream, d_w, cin,
                     cout, (uint4*)d_packed);
  return emc2_check_hip(ctx, hipGetLastError(), "emc2_pack_weights_i8 launch");
}

extern "C" emc2_status emc2_spconv_i8(emc2_ctx* ctx, const int8_t* d_in, const void* d_w_packed, const float* d_mul,
                                      const float* d_add, int32_t relu, emc2_dtype out_dtype, float inv_out_scale,
                                      const int32_t* d_nbr, const int32_t* d_n_out, int64_t capacity_out, int64_t n_in_rows,
                                      int32_t cin, int32_t cout, void* d_out, void* stream) {
  if (!ctx) return EMC2_ERR_INVALID_ARG;
  if (!d_in || !d_w_packed || !d_mul || !d_add || !d_nbr || !d_n_out || !d_out)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv_i8: null argument");
  if (capacity_out < 1) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv_i8: capacity_out < 1");
  if (n_in_rows < 0) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv_i8: n_in_rows < 0");
  if (((uintptr_t)d_in | (uintptr_t)d_w_packed | (uintptr_t)d_out) & 15u)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv_i8: d_in, d_w_packed and d_out must be 16-byte aligned");
  const int32_t n_in = n_in_rows > 0x7fffffff ? 0x7fffffff : (int32_t)n_in_rows;
  if (!i8_shape_ok(cin, cout))
    return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_spconv_i8: Cin must be 64 or 128 and Cout 32 or 64");
  if (out_dtype != EMC2_I8 && out_dtype != EMC2_F16)
    return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_spconv_i8: output must be I8 or F16");
  if (out_dtype == EMC2_I8 && !(inv_out_scale == inv_out_scale))
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv_i8: inv_out_scale is not a number");
  hipStream_t s = (hipStream_t)stream;
  const int rl = relu ? 1 : 0;
#define CASE(CI, CO)                                                                                                        \
  if (cin == CI && cout == CO) {                                                                                            \
    if (out_dtype == EMC2_I8)                                                                                               \
      launch_i8<CI, CO, 1>(d_in, d_w_packed, d_mul, d_add, rl, inv_out_scale, d_nbr, d_n_out, capacity_out, n_in,           \
                           ctx->dev_words, ctx->zero_row, d_out, s);                                                        \
    else                                                                                                                    \
      launch_i8<CI, CO, 0>(d_in, d_w_packed, d_mul, d_add, rl, inv_out_scale, d_nbr, d_n_out, capacity_out, n_in,           \
                           ctx->dev_words, ctx->zero_row, d_out, s);                                                        \
  }
  CASE(64, 32) CASE(64, 64) CASE(128, 32) CASE(128, 64)
#undef CASE
  return emc2_check_hip(ctx, hipGetLastError(), "emc2_spconv_i8 launch");
}

// ---------------------------------------------------------------------------------------------------------
// E4M3 variant: same kernel, same packed-weight byte order (emc2_pack_weights_i8 permutes bytes, whatever they encode)
// ---------------------------------------------------------------------------------------------------------
extern "C" emc2_status emc2_quantize_e4m3(emc2_ctx* ctx, emc2_dtype dtype, const void* d_x, int64_t n, float inv_scale,
                                          uint8_t* d_q, void* stream) {
  if (!ctx) return EMC2_ERR_INVALID_ARG;
  if (n < 0 || (n > 0 && (!d_x || !d_q))) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_quantize_e4m3: bad argument");
  if (!(inv_scale == inv_scale)) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_quantize_e4m3: inv_scale is not a number");
  if (n == 0) return EMC2_OK;
  hipStream_t s = (hipStream_t)stream;
  if (dtype == EMC2_F32) launch_quantize<float, true>(d_x, n, inv_scale, d_q, s);
  else if (dtype == EMC2_F16) launch_quantize<__half, true>(d_x, n, inv_scale, d_q, s);
  else return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_quantize_e4m3: input must be F32 or F16");
  return emc2_check_hip(ctx, hipGetLastError(), "emc2_quantize_e4m3 launch");
}

extern "C" emc2_status emc2_spconv_e4m3(emc2_ctx* ctx, const uint8_t* d_in, const void* d_w_packed, const float* d_mul,
                                        const float* d_add, int32_t relu, emc2_dtype out_dtype, const int32_t* d_nbr,
                                        const int32_t* d_n_out, int64_t capacity_out, int64_t n_in_rows, int32_t cin,
                                        int32_t cout, void* d_out, void* stream) {
  if (!ctx) return EMC2_ERR_INVALID_ARG;
  if (!d_in || !d_w_packed || !d_mul || !d_add || !d_nbr || !d_n_out || !d_out)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv_e4m3: null argument");
  if (capacity_out < 1) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv_e4m3: capacity_out < 1");
  if (n_in_rows < 0) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv_e4m3: n_in_rows < 0");
  if (((uintptr_t)d_in | (uintptr_t)d_w_packed | (uintptr_t)d_out) & 15u)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_spconv_e4m3: d_in, d_w_packed and d_out must be 16-byte aligned");
  if (!i8_shape_ok(cin, cout))
    return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_spconv_e4m3: Cin must be 64 or 128 and Cout 32 or 64");
  if (out_dtype != EMC2_F32 && out_dtype != EMC2_F16)
    return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "emc2_spconv_e4m3: output must be F32 or F16");
  const int32_t n_in = n_in_rows > 0x7fffffff ? 0x7fffffff : (int32_t)n_in_rows;
  hipStream_t s = (hipStream_t)stream;
  const int rl = relu ? 1 : 0;
#define CASE(CI, CO)                                                                                                         \
  if (cin == CI && cout == CO) {                                                                                             \
    if (out_dtype == EMC2_F32)                                                                                               \
      launch_i8<CI, CO, 1, 1>(d_in, d_w_packed, d_mul, d_add, rl, 0.f, d_nbr, d_n_out, capacity_out, n_in, ctx->dev_words,   \
                              ctx->zero_row, d_out, s);                                                                      \
    else                                                                                                                     \
      launch_i8<CI, CO, 0, 1>(d_in, d_w_packed, d_mul, d_add, rl, 0.f, d_nbr, d_n_out, capacity_out, n_in, ctx->dev_words,   \
                              ctx->zero_row, d_out, s);                                                                      \
  }
  CASE(64, 32) CASE(64, 64) CASE(128, 32) CASE(128, 64)
#undef CASE
  return emc2_check_hip(ctx, hipGetLastError(), "emc2_spconv_e4m3 launch");
}
