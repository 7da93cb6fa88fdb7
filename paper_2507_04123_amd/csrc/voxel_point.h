// One point -> its cell, and one voxel's stash -> its mean: the two definitions every voxelizing kernel shares.
#pragma once

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <math.h>

#include "common.h"

// The cell index and the range filter are defined by individually rounded IEEE fp32 operations;
// plain operators under this pragma stay unfused (intrinsics from headers would not).
#pragma clang fp contract(off)

struct VoxParams {
  float lo[3];
  float vs[3];
  int32_t grid[3];
  int32_t n_batch;
  float r2_min, r2_max;
  int32_t stride_f;
};

// Cell along one axis per the definition: fp32 subtract, fp32 IEEE division, floor; -1 if outside.
__device__ __forceinline__ int cell_of(float p, float lo, float vs, int g) {
  const float t = (p - lo) / vs;  // separately rounded ops: contraction is off in this file
  if (!(t >= 0.0f) || !(t < (float)g)) return -1;
  return (int)floorf(t);
}

struct PointCell {
  float4 p;       // x, y, z, intensity
  int4 c;         // (b, z, y, x)
  uint64_t key;
  bool keep;
};

// Both point passes call this, so they agree on every point's fate and cell bit for bit.
__device__ __forceinline__ PointCell locate(const float* __restrict__ points, const int32_t* __restrict__ batch, int64_t i,
                                            int64_t n_points, const VoxParams& prm) {
  PointCell r;
  r.keep = i < n_points;
  r.p = make_float4(0.f, 0.f, 0.f, 0.f);
  r.c = make_int4(0, 0, 0, 0);
  r.key = 0;
  if (r.keep) {
    const float* p = points + i * prm.stride_f;
    if ((prm.stride_f & 3) == 0) {
      r.p = *reinterpret_cast<const float4*>(p);
    } else {
      r.p = make_float4(p[0], p[1], p[2], p[3]);
    }
    const int b = batch ? batch[i] : 0;
    const int cx = cell_of(r.p.x, prm.lo[0], prm.vs[0], prm.grid[0]);
    const int cy = cell_of(r.p.y, prm.lo[1], prm.vs[1], prm.grid[1]);
    const int cz = cell_of(r.p.z, prm.lo[2], prm.vs[2], prm.grid[2]);
    const float xx = r.p.x * r.p.x, yy = r.p.y * r.p.y;
    const float r2 = xx + yy;  // each product rounded on its own (no fused multiply-add)
    r.keep = (b >= 0) && (b < prm.n_batch) && (cx >= 0) && (cy >= 0) && (cz >= 0) && (r2 >= prm.r2_min) &&
             (r2 < prm.r2_max) && (fabsf(r.p.w) <= 3.402823466e38f);  // last test rejects NaN/inf intensity
    r.c = make_int4(b, cz, cy, cx);
    r.key = (((uint64_t)b * prm.grid[2] + (uint64_t)cz) * prm.grid[1] + (uint64_t)cy) * prm.grid[0] + (uint64_t)cx;
  }
  return r;
}

// Sets the bit of a kept point's cell in `bits`, W 32-bit words from one word of bits to the next: marks (1) or an index (2).  Whoever finds
// it clear is the first of its voxel; the 64 answers of a wave
// (points 64w .. 64w+63) go to first[w], written for every wave that holds a point.  Every lane of the wave calls this.
template <int W>
__device__ __forceinline__ void emc2_mark_point(const PointCell& pc, int64_t i, int64_t n_points, uint32_t* __restrict__ bits,
                                                lineflag_t* __restrict__ flags, unsigned long long* __restrict__ first) {
  bool mine = false;
  if (pc.keep) {
    const uint32_t bit = 1u << ((uint32_t)pc.key & 31u);
    mine = (atomicOr(&bits[W * (pc.key >> 5)], bit) & bit) == 0u;
    flags[emc2_line_of_key(pc.key)] = 1;   // this line now holds a bit
  }
  const unsigned long long m = __ballot(mine);
  if ((threadIdx.x & 63) == 0 && i < n_points) first[i >> 6] = m;
}

// Point i joins voxel r.  The voxel's first point (nearly every point of a LiDAR frame is one) takes row 0 of the stash
// and writes the coordinates, with no atomic: the second pass over 7.7 M points 483 -> 368 us, the means 185 -> 80 us.  A further point gets its
// position from one returning atomic add; those beyond the stash are added atomically into the output row.
__device__ __forceinline__ void emc2_stash_point(int64_t i, int32_t r, const PointCell& pc,
                                                 const unsigned long long* __restrict__ first, int4* __restrict__ coords,
                                                 float4* __restrict__ feats, int32_t* __restrict__ counts,
                                                 float4* __restrict__ stash, int64_t pitch) {
  if ((first[i >> 6] >> (i & 63)) & 1ull) {
    coords[r] = pc.c;
    stash[r] = pc.p;
    return;
  }
  const int32_t pos = 1 + atomicAdd(&counts[r], 1);
  if (pos < EMC2_VOX_STASH) {
    stash[pos * pitch + r] = pc.p;
  } else {
    float* f = reinterpret_cast<float*>(feats + r);
    unsafeAtomicAdd(f + 0, pc.p.x);
    unsafeAtomicAdd(f + 1, pc.p.y);
    unsafeAtomicAdd(f + 2, pc.p.z);
    unsafeAtomicAdd(f + 3, pc.p.w);
  }
}

// Mean of voxel r: the points v (at most EMC2_VOX_STASH, the rest at infinity), the sum s of its further ones, cnt in all; lp: 0
// none, 1 fp16, 2 bf16 copy.  The points come in arrival order, which differs from run to run.  They are summed in the order of
// their values (x, then y, z, intensity) instead, so that a voxel of up to EMC2_VOX_STASH points -- nearly every voxel of a LiDAR
// frame -- gets the same mean, bit for bit, in every run and for every order of the input.
__device__ __forceinline__ void emc2_store_mean(int64_t r, float4 (&v)[EMC2_VOX_STASH], float4 s, int32_t cnt, float4* __restrict__ feats,
                                                int lp, void* __restrict__ feats_lp) {
  auto before = [](const float4& a, const float4& b) {
    if (a.x != b.x) return a.x < b.x;
    if (a.y != b.y) return a.y < b.y;
    if (a.z != b.z) return a.z < b.z;
    return a.w < b.w;
  };
  auto order = [&](int a, int b) {   // compare-exchange: v[a] <= v[b] afterwards
    if (before(v[b], v[a])) { const float4 t = v[a]; v[a] = v[b]; v[b] = t; }
  };
  static_assert(EMC2_VOX_STASH == 4, "the sorting network below orders four entries");
  order(0, 1); order(2, 3); order(0, 2); order(1, 3); order(1, 2);
#pragma unroll
  for (int j = 0; j < EMC2_VOX_STASH; ++j)
    if (j < cnt) { s.x += v[j].x; s.y += v[j].y; s.z += v[j].z; s.w += v[j].w; }
  const float c = (float)cnt;
  const float4 m = make_float4(s.x / c, s.y / c, s.z / c, s.w / c);
  feats[r] = m;
  if (lp == 1) {
    __half2* o = reinterpret_cast<__half2*>(feats_lp) + 2 * r;
    o[0] = __floats2half2_rn(m.x, m.y);
    o[1] = __floats2half2_rn(m.z, m.w);
  } else if (lp == 2) {
    __hip_bfloat16* o = reinterpret_cast<__hip_bfloat16*>(feats_lp) + 4 * r;
    o[0] = __float2bfloat16(m.x); o[1] = __float2bfloat16(m.y);
    o[2] = __float2bfloat16(m.z); o[3] = __float2bfloat16(m.w);
  }
}

// Mean of voxel r from its stash, the number of points after its first (which becomes the count) and what overflowed the
// stash.
__device__ __forceinline__ void emc2_voxel_mean(int64_t r, const float4* __restrict__ stash, int64_t pitch,
                                                float4* __restrict__ feats, int32_t* __restrict__ counts, int lp,
                                                void* __restrict__ feats_lp) {
  const int32_t cnt = counts[r] + 1;
  counts[r] = cnt;
  const float4 s = feats[r];   // what overflowed the stash (zero for almost every voxel)
  const int k = cnt < EMC2_VOX_STASH ? cnt : EMC2_VOX_STASH;
  float4 v[EMC2_VOX_STASH];
#pragma unroll
  for (int j = 0; j < EMC2_VOX_STASH; ++j)
    v[j] = j < k ? stash[j * pitch + r] : make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
  emc2_store_mean(r, v, s, cnt, feats, lp, feats_lp);
}

// Host side (voxelize.hip): the checks of a voxelization's arguments, and the kernels' view of a grid.
emc2_status emc2_voxel_args_ok(emc2_ctx* ctx, const emc2_voxel_spec* spec, int64_t n_points, int64_t capacity, int32_t index_slot,
                               const char* who);
VoxParams emc2_vox_params(const emc2_voxel_spec* spec);

// Voxelization of large clouds by bin of cells (voxel_bins.hip): whether a call takes it, and its launches.
bool emc2_bins_pay(int64_t n_points, int64_t n_cells);
void emc2_voxelize_bins(emc2_ctx* ctx, const float* d_points, const int32_t* d_batch, int64_t n_points, const VoxParams& prm,
                        int64_t n_cells, cellword_t* idx, int64_t capacity, int32_t* d_coords, float* d_feats, int32_t* d_counts,
                        void* d_feats_lp, int lp, int32_t* d_n_voxels, hipStream_t s);
