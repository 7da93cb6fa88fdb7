// Internal declarations shared by the translation units of libemc2.so (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "emc2.h"

// ---------------------------------------------------------------------------------------------
// Cell index: one 8-byte word per 32 consecutive cells of the linear key space
//   .x = occupancy bits (bit j <=> cell 32*w + j is an active voxel)
//   .y = number of active cells in all earlier words (exclusive prefix sum of popcounts)
// Because voxels are listed in ascending key order, the voxel index of an active cell is simply
// its rank: word.y + popcount(word.x & lower-bit mask).  This is the prefix-sum index search of
// the paper's Sec. 3.6, giving an O(1) lookup.
// ---------------------------------------------------------------------------------------------
typedef uint2 cellword_t;

__device__ __forceinline__ int32_t cell_lookup(const cellword_t* __restrict__ idx, uint64_t key) {
  const cellword_t w = idx[key >> 5];
  const uint32_t bit = (uint32_t)key & 31u;
  if (!((w.x >> bit) & 1u)) return -1;
  return (int32_t)(w.y + __popc(w.x & ((1u << bit) - 1u)));
}

// Linear key -> (b, z, y, x).  Keys below 2^32 (every single-frame grid here) take 32-bit divisions, which are
// several times cheaper than the 64-bit ones.
__device__ __forceinline__ int4 decode_key(uint64_t key, int gx, int gy, int gz) {
  if ((key >> 32) == 0) {
    uint32_t k = (uint32_t)key;
    const uint32_t x = k % (uint32_t)gx; k /= (uint32_t)gx;
    const uint32_t y = k % (uint32_t)gy; k /= (uint32_t)gy;
    const uint32_t z = k % (uint32_t)gz; k /= (uint32_t)gz;
    return make_int4((int)k, (int)z, (int)y, (int)x);
  }
  uint64_t k = key;
  const int x = (int)(k % (uint64_t)gx); k /= (uint64_t)gx;
  const int y = (int)(k % (uint64_t)gy); k /= (uint64_t)gy;
  const int z = (int)(k % (uint64_t)gz); k /= (uint64_t)gz;
  return make_int4((int)k, z, y, x);
}

// points a voxel's stash holds before further ones are added atomically (LiDAR voxels hold 1-2 points)
#define EMC2_VOX_STASH 4


// Device status bits (OR-ed by kernels, read by emc2_status_sync).
#define EMC2_DEVFLAG_CAPACITY 1
#define EMC2_DEVFLAG_MAP 2        // a kernel-map entry named a row outside [0, n_in_rows)

// A kernel-map entry as a conv kernel uses it.  Rows past n_out (`dead` = -1, else 0) have no neighbours; an
// entry at or beyond the `n_in` rows the caller says the input holds is treated as absent (never read) and
// remembered in the wave-uniform mask `oob`, which emc2_report_oob turns into a status bit at the kernel's end.
__device__ __forceinline__ int32_t emc2_entry(int32_t j, int32_t dead, int32_t n_in, unsigned long long& oob) {
  j |= dead;
  oob |= __ballot(j >= n_in);
  return j < n_in ? j : -1;
}
__device__ __forceinline__ void emc2_report_oob(unsigned long long oob, int32_t* __restrict__ flags) {
  if (oob != 0ull && (threadIdx.x & 63) == 0) atomicOr(flags, EMC2_DEVFLAG_MAP);
}

struct SlotMeta {
  int32_t grid[3];
  int32_t n_batch;
  bool valid;
};

struct emc2_ctx {
  int device;
  int64_t max_points, max_voxels, max_cells;
  int32_t n_slots;          // user-visible slots; two more internal ones follow
  int64_t slot_words;       // cellwords per slot (a whole number of tiles); the line flags follow them
  int64_t slot_tiles;
  cellword_t** slots;       // host array [n_slots + 2] of device pointers
  SlotMeta* meta;           // host array [n_slots + 2]
  float4* stash;            // [EMC2_VOX_STASH][max_voxels] points of each voxel: row 0 its first, then in arrival order
  unsigned long long* first;  // [max_points / 64 + 1] one bit per point: the first of its voxel
  uint32_t* partials;       // scan partial sums [n_partials], then the bases made of them [n_partials]
  int64_t n_partials;
  uint32_t* marks;          // [slot_words] occupancy bits of the index that is being built, [slot_words / 16] line flags behind them
  bool marks_zeroed;        // they are zero
  bool marks_recorded;      // the present call's clearing of them was recorded into a graph, which may never run
  uint32_t* bins;           // [6 * n_bins + 4] large clouds by bin of cells (voxel_bins.hip)
  int64_t n_bins;
  bool bins_zeroed;         // the first n_bins of them are zero
  uint32_t* stack_sums;     // popcount sums of every level of a stack (stack.hip)
  int64_t n_stack_sums;
  int32_t* dev_words;       // [0] status flags, [2] voxel count of an index rebuilt from coordinates (others unused)
  void* wpack;              // scratch for weights re-ordered per call (27*128*128 16-bit values)
  void* zero_row;           // 256 zero bytes: the feature row an absent neighbour reads
  // image pooling: per-pixel cell rank / position within the cell / sorted order, per-cell list starts
  int32_t *pix_rank, *pix_pos, *pix_perm, *pix_srank;   // [max_points] each
  int32_t* cell_start;      // [max_voxels]
  uint32_t* pool_acc;       // [(max_points/64 + 2) * 256] partial results of cells that cross a block boundary
  int32_t* fuse_src;        // [2 * max_voxels] source rows of a fused set when the caller does not keep them
  int32_t* pinned;          // pinned host staging for counts / status (4 ints)
  char err[256];
};

#define EMC2_SCAN_TILE 2048  // cellwords per scan block (256 threads x 8)
#define EMC2_TILE_SHIFT 11   // log2(EMC2_SCAN_TILE)
#define EMC2_SCAN_SELF_TILES 16384  // scans of up to so many tiles take two launches and no second half of `partials`
#define EMC2_LINE_SHIFT 4    // log2 of the cellwords per flagged line: 16 words = 128 bytes = 512 cells
#define EMC2_LINES_PER_TILE (EMC2_SCAN_TILE >> EMC2_LINE_SHIFT)

// Bins of the voxelization of large clouds: 2^14 cells, or a whole scan tile of 2^16 where that makes more than EMC2_BINS_MAX.
#define EMC2_BIN_SHIFT_FINE 14
#define EMC2_BIN_SHIFT_TILE (5 + EMC2_TILE_SHIFT)
#define EMC2_BINS_MAX 131072

// Line flags of an index slot.  The active cells of a LiDAR frame fill a fraction of a percent of the finest
// grid, and scattered objects touch single cache lines of it, so every index slot carries one flag byte per
// 128-byte line (16 words, 512 cells), stored behind its words:
// INVARIANT: a line whose flag is 0 holds no occupancy bit (its prefix fields are unspecified and never
// read: a lookup tests the bit first).  Every kernel that sets bits raises the flag of the line it writes
// (a plain byte store: all writers store the same value); clear, scan, the stride-2 marking and the
// expansion to coordinates read a tile's 128 flag bytes first and touch only the flagged lines.
typedef uint8_t lineflag_t;
static inline lineflag_t* emc2_slot_flags(const emc2_ctx* ctx, cellword_t* idx) {
  return reinterpret_cast<lineflag_t*>(idx + ctx->slot_words);
}
// flag index of the line that holds cell `key`
__host__ __device__ __forceinline__ uint64_t emc2_line_of_key(uint64_t key) { return key >> (5 + EMC2_LINE_SHIFT); }

// host helpers (context.hip)
emc2_status emc2_fail(emc2_ctx* ctx, emc2_status st, const char* fmt, ...);
emc2_status emc2_check_hip(emc2_ctx* ctx, hipError_t e, const char* what);
bool emc2_grid_ok(const int32_t grid[3], int32_t n_batch, int64_t* n_cells);
bool emc2_capturing(hipStream_t stream);   // launches on it are recorded (or it cannot be told)

// Marks: occupancy bits of the index that a voxelization, pooling or fusion builds, 4 bytes per 32 cells, and a flag byte per 512 cells (64
// bytes of bits), kept with the index's own.  Both are zero between calls: emc2_index_build, which takes the bits over into the slot, zeroes
// them behind itself, and zeroes the lines that the slot still holds of an earlier index in the same pass.  Bits set in the slot itself have
// to wait for a launch that clears it: with one less for each of the three calls, and each scan a little shorter, the bridge of a 64-beam
// frame takes 150 -> 135 us.  (A
// stack keeps that launch, of 5 us: its first gather reads what lies about the marks, and the maps, which read the same places of
// the index later, then find less of it in the caches: 120 000 points 33 -> 41 us, 300 000 47 -> 56.)
// Dense grids keep it too (voxelize.hip and pool.hip say which): marks lie twice as close as the index's bits, and atomics on a line
// are served one after the other.  Marks at the index's pitch would be as fast there, but slower on sparse grids: fusion 22.2 -> 25.7 us, the
// bridge 132 -> 139.
static inline lineflag_t* emc2_mark_flags(const emc2_ctx* ctx) { return reinterpret_cast<lineflag_t*>(ctx->marks + ctx->slot_words); }

// cell-index construction (cellindex.hip); all asynchronous on `stream`
// The marks are about to be set: zeroes them if a launch of an earlier call failed.
void emc2_marks_begin(emc2_ctx* ctx, hipStream_t stream);
// the slot's index over ceil(n_cells/32) words from the marks, with prefix sums; min(total, capacity) to d_total and
// EMC2_DEVFLAG_CAPACITY when total > capacity
void emc2_index_build(emc2_ctx* ctx, cellword_t* idx, int64_t n_cells, int64_t capacity, int32_t* d_total, hipStream_t stream);
// zero every flagged tile of the slot (whatever grid it last held) and lower its flag
void emc2_index_clear(emc2_ctx* ctx, cellword_t* idx, hipStream_t stream);
// exclusive scan of popcounts over ceil(n_cells/32) words; writes min(total, capacity) to d_total
// and raises EMC2_DEVFLAG_CAPACITY when total > capacity
void emc2_index_scan(emc2_ctx* ctx, cellword_t* idx, int64_t n_cells, int64_t capacity, int32_t* d_total,
                     hipStream_t stream);
// bases[i] = sum of the n totals before i; the sum of all, clamped and reported like that of the index, to d_total
void emc2_scan_totals(emc2_ctx* ctx, const uint32_t* totals, int64_t n, int64_t capacity, uint32_t* bases, int32_t* d_total,
                      hipStream_t stream);
// set the bits of coords[0..*d_n) (b,z,y,x) in a cleared index
void emc2_index_mark_coords(emc2_ctx* ctx, cellword_t* idx, const int32_t* d_coords, const int32_t* d_n,
                            int64_t capacity, const int32_t grid[3], int32_t n_batch, hipStream_t stream);

// text of the last host-side error of emc2_build_kmap_static (kmap.hip); what emc2_last_error(NULL) returns
const char* emc2_static_last_error();

// Blocks of a launch whose threads step through the pieces of a device-side row count: two rounds of the chip.  The host
// knows only the rows' capacity, several times the count, and blocks without work cost about 0.25 us per thousand.  With the
// pooling's last pass per block boundary: bridge of a 375 x 1242 image and 120 000 points 160 -> 154 us.
static inline unsigned emc2_piece_blocks(int64_t pieces, int64_t threads) {
  const int64_t b = (pieces + threads - 1) / threads;
  return (unsigned)(b < 4096 ? b : 4096);
}
static inline int64_t emc2_div_up(int64_t a, int64_t b) { return (a + b - 1) / b; }
