// Internal interface of the MFMA sparse-conv kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "emc2.h"

// What a convolution's launch is given, checked; one of several in a launch (their blocks come one after the other).
struct emc2_conv_args {
  const void *d_in, *d_w;               // d_w as the kernel reads it
  const float *d_scale, *d_shift;
  const int32_t *d_nbr, *d_n_out;
  const void* d_zero_row;
  void* d_out;
  int64_t capacity_out;
  int32_t n_in, epilogue;
  int32_t* dev_flags;
};
constexpr int kConvBatch = 4;           // calls a launch can hold
// A launch of one call has a form of its own: where the block looks for its call, the arguments are read a dependent scalar load later.
// us, looked for / so: 16 -> 32 over 4 000 rows 4.9 / 4.8, 32 -> 64 8.0 / 7.75, over 12 000 8.55 / 8.25, 64 -> 32 over 4 000 8.0 / 7.8.
template <int CALLS> struct emc2_conv_batch {
  int32_t n;
  uint32_t first[CALLS];                // first block of each (of kernels that deal tiles to XCDs a multiple of 8)
  emc2_conv_args call[CALLS];
};
static inline emc2_conv_batch<1> emc2_conv_one(const emc2_conv_batch<kConvBatch>& b) { return {1, {0}, {b.call[0]}}; }
// The call that this block belongs to, the block's number in it and how many blocks it has.
struct emc2_conv_place { int call; uint32_t block, blocks; };
template <int CALLS> __device__ __forceinline__ emc2_conv_place emc2_conv_of_block(const emc2_conv_batch<CALLS>& b) {
  if constexpr (CALLS == 1) return {0, blockIdx.x, gridDim.x};
  int i = 0;
  while (i + 1 < b.n && blockIdx.x >= b.first[i + 1]) ++i;
  return {i, blockIdx.x - b.first[i], (i + 1 < b.n ? b.first[i + 1] : gridDim.x) - b.first[i]};
}

// true iff (cin, cout) is covered by an MFMA instantiation (16-bit dtypes only)
bool emc2_spconv_mfma_supported(int cin, int cout);

// Re-order W[27][Cin][Cout] (16-bit) into MFMA B-fragment order (same byte size).
void emc2_spconv_mfma_pack(const void* d_w, int cin, int cout, void* d_packed, hipStream_t stream);

// d_wp: weights already in fragment order.
// n_in: rows of d_in; a kernel-map entry outside [0, n_in) is treated as absent and raises EMC2_DEVFLAG_MAP in
// *dev_flags (the same two arguments on every launcher below).
void emc2_spconv_mfma_launch(emc2_dtype dtype, const void* d_in, const void* d_wp, const float* d_scale,
                             const float* d_shift, int epilogue, const int32_t* d_nbr, const int32_t* d_n_out,
                             int64_t capacity_out, int32_t n_in, int32_t* dev_flags, int cin, int cout, void* d_out,
                             hipStream_t stream);

// Span-gather variant (one contiguous fetch of input rows per group of three kx taps): profitable for
// kernel maps whose three kx taps name nearly the same rows (submanifold maps over voxels sorted by key).
// Same arguments and results as emc2_spconv_mfma_launch.
bool emc2_spconv_span_supported(int cin, int cout);
void emc2_spconv_span_launch(emc2_dtype dtype, const void* d_in, const void* d_wp, const float* d_scale,
                             const float* d_shift, int epilogue, const int32_t* d_nbr, const int32_t* d_n_out,
                             int64_t capacity_out, int32_t n_in, int32_t* dev_flags, int cin, int cout, void* d_out,
                             hipStream_t stream);

// 16 -> 32 and 32 -> 32, every map.  Weights as emc2_spconv_mfma_pack (16) and emc2_spconv_direct_pack (32) order them.
// d_zero_row: >= 256 zero bytes in device memory.
bool emc2_spconv_narrow_supported(int cin, int cout);
void emc2_spconv_narrow_launch(emc2_dtype dtype, int cin, const emc2_conv_args* calls, int n, hipStream_t stream);

// Register-direct variant (A operands straight from global memory, 16x16x32 MFMA; LDS holds weights only).
// Its packed weight layout, emc2_spconv_direct_pack's, differs from the staged kernel's; emc2_spconv_direct_order: the shapes
// packed so, those of this kernel and of the span kernel and 32 -> 32.  d_zero_row: >= 256 zero bytes in device memory.  skip:
// larger levels leave out the groups of taps that no row of a block has (pays where the map is not a submanifold one; the
// results are the same for finite weights).
bool emc2_spconv_direct_supported(int cin, int cout);
bool emc2_spconv_direct_order(int cin, int cout);
void emc2_spconv_direct_pack(const void* d_w, int cin, int cout, void* d_packed, hipStream_t stream);
void emc2_spconv_direct_launch(emc2_dtype dtype, const void* d_in, const void* d_wp, const float* d_scale,
                               const float* d_shift, int epilogue, const int32_t* d_nbr, const int32_t* d_n_out,
                               int64_t capacity_out, int32_t n_in, int32_t* dev_flags, int cin, int cout,
                               const void* d_zero_row, bool skip, void* d_out, hipStream_t stream);

// Register-direct with all weights of a block's columns in LDS: the shapes and the packed layout of the register-direct kernel.
bool emc2_spconv_resident_supported(int cin, int cout);
void emc2_spconv_resident_launch(emc2_dtype dtype, int cin, const emc2_conv_args* calls, int n, hipStream_t stream);
