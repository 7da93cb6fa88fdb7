// Register-direct convolution with resident weights (paper Sec. 3.5 sparse convolution over the non-empty voxels; Sec. 3.6 keeping
// data on chip between dependent steps): 32 -> 64 and 64 -> 32, every map.  The walk itself: resident_walk.h.
//
// The operands as in spconv_direct.hip: lane (m, q) of v_mfma_f32_16x16x32 supplies 16 contiguous bytes of the feature row that its
// output row names, so a load from global memory is the operand; absent neighbours read past the end of the input's buffer
// descriptor (inputs of 4 GiB and more: a zeroed row).  There a block of four waves copied each tap's weights through registers to
// LDS, with a barrier a tap, and ran every (dz, dy) group that some row of its 128 had: a group of three taps took 3.3 us of a
// CU's time, of which the gathers were a third.  These shapes' weights are 110 KB, which the LDS of a CU holds whole.  A block of 15
// waves, one a CU, copies them once, behind the only barrier; then each wave takes tiles of 32 rows by itself, runs only the
// groups that its own rows have (5.1 of nine under a stride-2 map where blocks of 128 rows have 5.8, 2.7 where they have 3.5 under a
// transposed one), reads weights from LDS wherever it is, and takes the next tile when it is done (tiles of one group next to
// tiles of nine).  It is bound by the gathers' loads (eight routed frames: 265 MB a launch at 3.7 TB/s, where a copy reaches 4.3, and 1 483
// cycles a load; matrix cores busy 25 %, LDS 18 %, a wave issues in 17 % of its cycles): two groups requested ahead gain nothing, loads
// that take whole 128-byte rows, lanes swapped afterwards, neither.  64 -> 64 in two halves of the columns, gathering twice, is 8 and
// 25 % slower than spconv_direct.hip (223 k rows transposed 38 / 41, stride-2 51 / 64).
// Alone, us, spconv_direct.hip's way / so with 12 waves: stride-2 32 -> 64 69 k rows 20.0 / 17.1, 223 k 32.7 / 27.5, 893 k 115 / 90, 1.3 M
// 170 / 136; submanifold 304 k 46 / 40, 1.2 M 180 / 140; transposed 64 -> 32 54 k 12.8 / 10.6, 223 k 32 / 26, 304 k 43 / 33, 893 k
// 101 / 70; submanifold 87 / 85; any row from anywhere 223 k 85 / 88 and 103 / 103.  What the later order of the walk and 15 waves gave:
// resident_walk.h.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "common.h"
#include "resident_walk.h"
#include "spconv_mfma.h"

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef emc2_resident::u32x4 u32x4;
typedef emc2_resident::u32x2 u32x2;

template <int DT> struct MmaR;
template <> struct MmaR<EMC2_F16> {
  static __device__ __forceinline__ floatx4 run(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t cvt2(float x, float y) {   // round to nearest even
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{x, y}), half2v));
  }
};
template <> struct MmaR<EMC2_BF16> {
  static __device__ __forceinline__ floatx4 run(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ uint32_t cvt2(float x, float y) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{x, y}), bf16x2));
  }
};

using emc2_resident::kRCUs;
using emc2_resident::kRRows;

template <int DT, int CIN, int COUT> struct Op16 {
  static constexpr int KS = CIN / 32, NT = COUT / 16;
  template <bool BUF> static constexpr int waves = BUF ? emc2_resident::kRWaves : emc2_resident::kRWavesWide;
  static constexpr bool kRowsFirst = CIN == 64;
  typedef floatx4 acc_t;
  const float *scale, *shift;
  int epilogue;
  uint16_t* out;
  static __device__ __forceinline__ floatx4 run(u32x4 w, u32x4 a, floatx4 c) { return MmaR<DT>::run(w, a, c); }
  __device__ __forceinline__ void store(int64_t row0, int m, int q, int64_t n_out, floatx4 (&acc)[2][NT]) const {
    // Folded affine, ReLU and rounding in registers: lane (m, q) holds channels 16j + 4q .. + 3 of row m; one lane swap per pair of
    // column tiles leaves it eight consecutive channels.
#pragma unroll
    for (int jp = 0; jp < NT / 2; ++jp) {
      floatx4 sc[2], sh[2];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int c = 16 * (2 * jp + t) + 4 * q + i;
          sc[t][i] = epilogue != EMC2_EPI_NONE ? scale[c] : 1.f;
          sh[t][i] = epilogue != EMC2_EPI_NONE ? shift[c] : -0.f;     // x * 1 + -0 is x
        }
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        u32x2 h[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          floatx4 v = acc[mt][2 * jp + t];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v[i] = fmaf(v[i], sc[t][i], sh[t][i]);
            if (epilogue == EMC2_EPI_AFFINE_RELU) v[i] = fmaxf(v[i], 0.f);   // NaN -> 0
          }
          h[t] = u32x2{MmaR<DT>::cvt2(v[0], v[1]), MmaR<DT>::cvt2(v[2], v[3])};
        }
        const u32x2 x = __builtin_amdgcn_permlane16_swap(h[0][0], h[1][0], false, false);
        const u32x2 y = __builtin_amdgcn_permlane16_swap(h[0][1], h[1][1], false, false);
        const int64_t o = row0 + 16 * mt + m;
        if (o < n_out)
          *reinterpret_cast<u32x4*>(out + o * COUT + 32 * jp + 8 * (2 * (q & 1) + (q >> 1))) = u32x4{x[0], y[0], x[1], y[1]};
      }
    }
  }
};

template <int DT, int CIN, int COUT, bool BUF, int CALLS>
__global__ void __launch_bounds__((Op16<DT, CIN, COUT>::template waves<BUF> * 64)) k_spconv_direct_resident(const emc2_conv_batch<CALLS> b) {
  const emc2_conv_place at = emc2_conv_of_block(b);
  const emc2_conv_args& c = b.call[at.call];
  const Op16<DT, CIN, COUT> op = {c.d_scale, c.d_shift, c.epilogue, (uint16_t*)c.d_out};
  emc2_resident::walk<Op16<DT, CIN, COUT>, BUF>(op, at.block, at.blocks, c.d_in, (const u32x4*)c.d_w, c.d_nbr, c.d_n_out, c.capacity_out, c.n_in,
                                                c.dev_flags, c.d_zero_row);
}

template <int DT, int CIN, int COUT> void launch_resident(const emc2_conv_args* calls, int n, hipStream_t s) {
  emc2_conv_batch<kConvBatch> b;
  b.n = n;
  uint32_t blocks = 0;
  // Offsets into the input are 32-bit, and the absent neighbour's, 2^32 less a row, must lie at or beyond its end.
  bool buf = true;
  for (int i = 0; i < n; ++i) {
    b.call[i] = calls[i];
    b.first[i] = blocks;
    const int64_t own = emc2_div_up(emc2_div_up(calls[i].capacity_out, kRRows), 8) * 8;
    blocks += (uint32_t)(own < kRCUs ? own : kRCUs);
    buf = buf && ((int64_t)calls[i].n_in + 1) * CIN * 2 <= ((int64_t)1 << 32);
  }
#define LAUNCH(BUF, CALLS, ARGS) \
  hipLaunchKernelGGL((k_spconv_direct_resident<DT, CIN, COUT, BUF, CALLS>), dim3(blocks),           \
                     dim3(Op16<DT, CIN, COUT>::template waves<BUF> * 64), 0, s, ARGS)
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

bool emc2_spconv_resident_supported(int cin, int cout) { return (cin == 32 && cout == 64) || (cin == 64 && cout == 32); }

void emc2_spconv_resident_launch(emc2_dtype dtype, int cin, const emc2_conv_args* calls, int n, hipStream_t stream) {
#define CASE(D, CI, CO) \
  if (dtype == D && cin == CI) launch_resident<D, CI, CO>(calls, n, stream);
  CASE(EMC2_F16, 32, 64) CASE(EMC2_BF16, 32, 64) CASE(EMC2_F16, 64, 32) CASE(EMC2_BF16, 64, 32)
#undef CASE
}
