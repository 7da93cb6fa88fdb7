// Voxelization with mean voxel features (paper Sec. 2 / Sec. 3.1 voxelization in the data bridge;
// Sec. 3.5 configurable pool size; Sec. 3.6 (3) prefix-sum index search).
//
// The voxel index of a cell is its rank in the prefix-summed cell index, so no hash table is needed:
// (Clouds of more than half a million points: voxel_bins.hip.)
// Pass 1 (one thread per point): cell key -> set the cell's mark (one atomic OR per point), of dense grids its bit in the index; the same
//   launch zeroes the output rows pass 2 accumulates into.
// Scan: the index from the marks or of the bits, prefix sums -> the rank of every active cell = its position in key order, and the
//   number of voxels.
//   The OR returns the word's old bits, which tell the voxel's first point from later ones (one bit kept per point).
// Pass 2 (one thread per point): the same key again -> rank r (one 8-byte load).  A first point goes to row 0 of the
//   stash and needs no atomic; a later one gets its position from one returning atomic add on counts[r] and goes to that
//   row of the stash (a plain 16-byte store); only points beyond the stash depth are added atomically into the output row.
// Pass 3 (one thread per voxel): sum the stash in the order of the points' values, divide, write the means.
// Device-scope atomics on this part execute at the memory side of the fabric (the L2s of the 8 XCDs are
// not coherent with each other), about 27 G/s in aggregate: one per point (two where points share a voxel) instead of
// seven is what this layout buys.  The stash is kept row by row, so that pass 3 reads 16 contiguous bytes of a voxel with
// one point instead of a quarter of its 64.
#include <math.h>

#include "voxel_point.h"

namespace {

template <int W>  // as emc2_mark_point
__global__ void __launch_bounds__(256) k_vox_mark(const float* __restrict__ points, const int32_t* __restrict__ batch,
                                                  int64_t n_points, VoxParams prm, uint32_t* __restrict__ bits,
                                                  lineflag_t* __restrict__ flags,
                                                  unsigned long long* __restrict__ first, int64_t zero_rows,
                                                  float4* __restrict__ feats, int32_t* __restrict__ counts) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  // the rows pass 2 accumulates into: there are at most min(n_points, capacity) voxels, one thread each
  if (i < zero_rows) {
    feats[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    counts[i] = 0;
  }
  emc2_mark_point<W>(locate(points, batch, i, n_points, prm), i, n_points, bits, flags, first);
}

__global__ void __launch_bounds__(256) k_vox_scatter(const float* __restrict__ points, const int32_t* __restrict__ batch,
                                                     int64_t n_points, VoxParams prm, const cellword_t* __restrict__ idx,
                                                     const unsigned long long* __restrict__ first, int64_t capacity, int4* __restrict__ coords,
                                                     float4* __restrict__ feats, int32_t* __restrict__ counts,
                                                     float4* __restrict__ stash, int64_t pitch) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const PointCell pc = locate(points, batch, i, n_points, prm);
  if (!pc.keep) return;
  const int32_t r = cell_lookup(idx, pc.key);
  if (r < 0 || r >= capacity) return;   // beyond capacity: reported by the scan, dropped here
  emc2_stash_point(i, r, pc, first, coords, feats, counts, stash, pitch);
}

// The rows that pass 2 accumulates into, in a launch of its own: see kZeroApart below.
__global__ void __launch_bounds__(256) k_vox_zero(int64_t rows, float4* __restrict__ feats, int32_t* __restrict__ counts) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows) return;
  feats[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  counts[i] = 0;
}

template <int LP>  // 0 none, 1 fp16, 2 bf16
__global__ void __launch_bounds__(256) k_vox_finalize(const int32_t* __restrict__ d_n, int64_t capacity,
                                                      const float4* __restrict__ stash, int64_t pitch,
                                                      float4* __restrict__ feats, int32_t* __restrict__ counts, void* __restrict__ feats_lp) {
  int64_t n = *d_n;
  if (n > capacity) n = capacity;
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n) emc2_voxel_mean(r, stash, pitch, feats, counts, LP, feats_lp);
}

}  // namespace

emc2_status emc2_voxel_args_ok(emc2_ctx* ctx, const emc2_voxel_spec* spec, int64_t n_points, int64_t capacity, int32_t index_slot,
                               const char* who) {
  if (n_points > ctx->max_points)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "%s: n_points %lld > max_points %lld", who, (long long)n_points,
                     (long long)ctx->max_points);
  if (capacity < 1 || capacity > ctx->max_voxels)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "%s: capacity %lld outside [1, max_voxels %lld]", who, (long long)capacity,
                     (long long)ctx->max_voxels);
  if (index_slot < 0 || index_slot >= ctx->n_slots)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "%s: index_slot %d outside [0, %d)", who, index_slot, ctx->n_slots);
  if (spec->stride_f < 4) return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "%s: stride_f < 4", who);
  for (int a = 0; a < 3; ++a)
    if (!(spec->vs[a] > 0.0f) || !isfinite(spec->vs[a]) || !isfinite(spec->lo[a]))
      return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "%s: bad voxel size / lower bound", who);
  int64_t n_cells = 0;
  if (!emc2_grid_ok(spec->grid, spec->n_batch, &n_cells))
    return emc2_fail(ctx, EMC2_ERR_UNSUPPORTED, "%s: grid/batch out of the supported key range", who);
  if (n_cells > ctx->max_cells)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "%s: %lld cells > max_cells %lld", who, (long long)n_cells,
                     (long long)ctx->max_cells);
  return EMC2_OK;
}

VoxParams emc2_vox_params(const emc2_voxel_spec* spec) {
  VoxParams prm;
  for (int a = 0; a < 3; ++a) { prm.lo[a] = spec->lo[a]; prm.vs[a] = spec->vs[a]; prm.grid[a] = spec->grid[a]; }
  prm.n_batch = spec->n_batch;
  prm.r2_min = spec->r2_min;
  prm.r2_max = spec->r2_max;
  prm.stride_f = spec->stride_f;
  return prm;
}

// Bits set in the slot, behind a launch that clears it, against marks: a launch more, but twice the lines for the atomics of points that
// share them.  us, marks / bits in the slot, clouds of a frame's density, cells a point in brackets: 1 M points (0.7) 400 / 315, (5.8) 180 / 153, (14)
// 134 / 136; 350 000 (17) 59.6 / 53.2, (32) 49.5 / 51.1; 120 000 (2.9) 57.9 / 52.1, (14) 37.9 / 35.7, (27) 28.8 / 28.7, (49) 27.0 / 28.3; 65 536
// (0.67) 68 / 61, (2.4) 48.4 / 46.2, (5.4) 36.4 / 35.3, (12) 29.2 / 28.6, (22) 26.1 / 26.0, (43) 20.9 / 23.8; 50 000 (0.88) 53.4 / 48.0, (4.5) 33.8 / 36.0, (13) 24.8 /
// 26.0; 17 003 (0.5) 41.0 / 39.6, (3.7) 20.6 / 21.1; 4 000 (2.2) 17.4 / 17.7.
static bool in_slot(int64_t n_points, int64_t n_cells) {
  return n_points >= 8192 && n_cells <= (n_points >= 65536 ? 24 : 2) * n_points;
}

// Clouds of this many points and more zero their rows apart from the marking when that sets marks.  It makes six launches of the pass whether bits or
// marks are set, which is how tests/test_gpu_voxel_bins.py tells it from the one by bins (seven).  It costs: 524 287 points (43 to 701 cells a point)
// 60 to 71 us with the rows zeroed by the marking, 63 to 73 so; 1 M (90) 99.7 / 103.3; so fewer points, 262 145 38.9 / 42.7, don't.
constexpr int64_t kZeroApart = 500000;

static void voxelize_points(emc2_ctx* ctx, const float* d_points, const int32_t* d_batch, int64_t n_points, const VoxParams& prm,
                            int64_t n_cells, cellword_t* idx, int64_t capacity, int32_t* d_coords, float* d_feats, int32_t* d_counts,
                            void* d_feats_lp, int lp, int32_t* d_n_voxels, hipStream_t s) {
  const dim3 pg((unsigned)emc2_div_up(n_points > 0 ? n_points : 1, 256)), blk(256);
  // at most min(n_points, capacity) voxels exist
  const int64_t bound = n_points < capacity ? n_points : capacity;
  if (in_slot(n_points, n_cells)) {
    emc2_index_clear(ctx, idx, s);
    hipLaunchKernelGGL(k_vox_mark<2>, pg, blk, 0, s, d_points, d_batch, n_points, prm, reinterpret_cast<uint32_t*>(idx),
                       emc2_slot_flags(ctx, idx), ctx->first, bound, (float4*)d_feats, d_counts);
    emc2_index_scan(ctx, idx, n_cells, capacity, d_n_voxels, s);
  } else {
    emc2_marks_begin(ctx, s);
    const bool apart = n_points >= kZeroApart;
    if (apart) hipLaunchKernelGGL(k_vox_zero, dim3((unsigned)emc2_div_up(bound, 256)), blk, 0, s, bound, (float4*)d_feats, d_counts);
    if (n_points > 0)
      hipLaunchKernelGGL(k_vox_mark<1>, pg, blk, 0, s, d_points, d_batch, n_points, prm, ctx->marks, emc2_mark_flags(ctx), ctx->first,
                         apart ? 0 : bound, (float4*)d_feats, d_counts);
    emc2_index_build(ctx, idx, n_cells, capacity, d_n_voxels, s);
  }
  if (bound <= 0) return;
  const dim3 vg((unsigned)emc2_div_up(bound, 256));
  hipLaunchKernelGGL(k_vox_scatter, pg, blk, 0, s, d_points, d_batch, n_points, prm, idx, ctx->first, capacity,
                     (int4*)d_coords, (float4*)d_feats, d_counts, ctx->stash, ctx->max_voxels);
#define FIN(LP)                                                                                                 \
  hipLaunchKernelGGL(k_vox_finalize<LP>, vg, blk, 0, s, d_n_voxels, capacity, ctx->stash, ctx->max_voxels,      \
                     (float4*)d_feats, d_counts, d_feats_lp)
  if (lp == 0) FIN(0); else if (lp == 1) FIN(1); else FIN(2);
#undef FIN
}

extern "C" emc2_status emc2_voxelize(emc2_ctx* ctx, const float* d_points, const int32_t* d_batch, int64_t n_points,
                                     const emc2_voxel_spec* spec, int64_t capacity, int32_t* d_coords, float* d_feats,
                                     int32_t* d_counts, void* d_feats_lp, emc2_dtype lp_dtype, int32_t* d_n_voxels,
                                     int32_t* h_n_voxels, int32_t index_slot, void* stream) {
  if (!ctx) return EMC2_ERR_INVALID_ARG;
  if (!spec || !d_coords || !d_feats || !d_counts || !d_n_voxels)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_voxelize: null argument");
  if (n_points < 0 || (n_points > 0 && !d_points))
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_voxelize: bad points");
  const emc2_status ok = emc2_voxel_args_ok(ctx, spec, n_points, capacity, index_slot, "emc2_voxelize");
  if (ok != EMC2_OK) return ok;
  if (d_feats_lp && lp_dtype != EMC2_F16 && lp_dtype != EMC2_BF16)
    return emc2_fail(ctx, EMC2_ERR_INVALID_ARG, "emc2_voxelize: lp_dtype must be F16 or BF16");
  int64_t n_cells = 0;
  (void)emc2_grid_ok(spec->grid, spec->n_batch, &n_cells);

  hipStream_t s = (hipStream_t)stream;
  cellword_t* idx = ctx->slots[index_slot];
  SlotMeta& mt = ctx->meta[index_slot];
  for (int a = 0; a < 3; ++a) mt.grid[a] = spec->grid[a];
  mt.n_batch = spec->n_batch;
  mt.valid = true;

  const VoxParams prm = emc2_vox_params(spec);
  const int lp = d_feats_lp ? (lp_dtype == EMC2_F16 ? 1 : 2) : 0;
  const auto pass = emc2_bins_pay(n_points, n_cells) ? emc2_voxelize_bins : voxelize_points;
  pass(ctx, d_points, d_batch, n_points, prm, n_cells, idx, capacity, d_coords, d_feats, d_counts, d_feats_lp, lp, d_n_voxels, s);
  emc2_status st = emc2_check_hip(ctx, hipGetLastError(), "emc2_voxelize launch");
  if (st != EMC2_OK) return st;
  if (h_n_voxels) {
    st = emc2_check_hip(ctx, hipMemcpyAsync(ctx->pinned + 1, d_n_voxels, sizeof(int32_t), hipMemcpyDeviceToHost, s),
                        "hipMemcpyAsync(n_voxels)");
    if (st != EMC2_OK) return st;
    st = emc2_check_hip(ctx, hipStreamSynchronize(s), "hipStreamSynchronize");
    if (st != EMC2_OK) return st;
    *h_n_voxels = ctx->pinned[1];
  }
  return EMC2_OK;
}
