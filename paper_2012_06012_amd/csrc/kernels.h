// Host-side launchers of the transpose stages (implemented in kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/mgt.h"
#include "mgt_internal.h"

namespace mgt {

// Geometry shared by host and device.
constexpr int kBlock = 256;         // threads per workgroup (4 wave64)
constexpr int kSub = 2048;          // cells sorted in LDS at once
// Geometry of the records-only partition pass when its tiles hold at least
// kWideSub cells: twice the cells per LDS sort, so each digit's run of
// records is twice as long (kernels_wide.hip).
constexpr int kWideBlock = 512;
constexpr int kWideSub = 4096;
constexpr int kMaxPassBits = 8;     // digit bits of a bits-mode pass (fan-out 256)
constexpr int kMaxLastPassBits = 9; // the records-only pass in its 512-thread form (fan-out 512)
constexpr int kScanBlock = 4096;    // elements per scan workgroup

// Arguments of a partition pass (hist and scatter share them).
struct PassArgs {
  const ItemDev* items;
  const Seg* segs;
  uint32_t nseg;
  uint32_t pass;
  const uint64_t* tstart;     // nseg + 1
  const uint64_t* hstart;     // nseg + 1
  const uint2* ks_in;         // (key, size) records, pass >= 2
  const uint2* rk_in;         // (row, cell index) records, pass >= 2
  const uint8_t* pay_in;      // payload bytes, pass >= 2
  uint2* ks_out;
  uint2* rk_out;
  uint8_t* pay_out;           // unused when rso_out is set
  uint32_t* rso_out;          // last pass of two or more: per cell (row, cell index, byte
                              // offset of the payload in pay_in as two words) in place of
                              // rk_out; no payload is moved
  uint32_t* hcnt;             // [entry] cells of (segment, digit, tile)
  uint32_t* hbyt;             // [entry] payload bytes of (segment, digit, tile)
  uint32_t* ttot;             // [tile] payload bytes of the tile
  const uint64_t* ocnt;       // exclusive scan of hcnt (n + 1)
  const uint64_t* obyt;       // exclusive scan of hbyt (n + 1)
  const uint64_t* tsrc;       // exclusive scan of ttot (tiles + 1)
  int32_t* item_status;
  int32_t* abort_flag;
  uint64_t g8;                // grid size (multiple of 8)
  uint32_t tile_cells;        // multiple of kSub
  int32_t offset_width;
  int32_t has_val;            // first pass: the items carry vval (view operations)
  // Packed records: a call with exactly one records-only pass, made without
  // perm and not as a view operation, keeps (column | size << s, row) after
  // the first pass and (column | size << s, row, payload offset) after the
  // second, s being the item's column bits (ItemDev::pk_shift, <= 28),
  // provided every payload size is below 2^(32 - s) bytes; the first
  // histogram checks that and sets *no_pack otherwise.
  int32_t pk_on;
  int32_t* no_pack;           // zero at the start of the call (uploaded with the status words)
  int32_t pk_keys;            // with pk_on and no fixed-width item: the first histogram writes
                              // (column | size << s) per cell into rk_out, which the first pass
                              // reads instead of the columns and offsets
  int32_t pk_split;           // set by the launcher: a slim packed-only kernel runs beside this
                              // one and takes packed records (this one returns on them)
  int32_t slim0;              // first pass: packed records go to the slim first pass, in its
                              // bits-only form (1: every item split by column bits) or its
                              // partition form (2: some item split by partition, fan-out
                              // at most 512); 0: the plain kernel only
  int32_t rec12;              // the slim kernel writes 12-byte packed records (column | size,
                              // row, payload offset minus the finish bucket's first byte as a
                              // signed 32-bit word) unless *big_seg is set
  const int32_t* big_seg;
};

struct ChildArgs {
  const ItemDev* items;
  const Seg* segs;            // parents
  uint32_t nseg;
  uint32_t pass;              // pass whose output the children describe (0-based)
  const uint64_t* tstart;
  const uint64_t* hstart;
  const uint64_t* ocnt;
  const uint64_t* obyt;
  Seg* children;
  uint32_t* child_tiles;
  uint32_t* child_hsize;
  uint32_t tile_cells;
  const int32_t* abort_flag;
  int32_t* big_seg;           // non-null where the children are the last pass's input
                              // segments: set to 1 if one holds 2^31 payload bytes or more
};

struct FinishArgs {
  const ItemDev* items;
  uint32_t n_items;           // <= nbuckets: every item has at least one bucket
  const Seg* buckets;
  uint32_t nbuckets;
  const uint2* ks_in;
  const uint2* rk_in;
  const uint8_t* pay_in;      // payload level buffer (the one before the last pass if rso_in)
  const uint32_t* rso_in;     // (row, cell index, payload offset in pay_in) records of the
                              // last pass, read in place of rk_in, or null
  const int32_t* abort_flag;
  const int32_t* item_status;
  int32_t* d_status;          // the caller's status words (may be null), written with the tails
  int32_t offset_width;
  uint64_t g8;                // grid size (multiple of 8)
  int32_t pk_on;              // as in PassArgs
  const int32_t* no_pack;
  uint8_t* bucket_done;       // [nbuckets] gathering finish with packed records: 1 where
                              // k_finish_bucket wrote the bucket (k_finish skips it), else 0;
                              // null: k_finish takes every bucket
  uint32_t grid;              // k_finish_bucket: workgroups (one or two per CU)
  uint32_t bk_threads;        // k_finish_bucket: 1024 (buckets up to 9,216 cells, one
                              // workgroup per CU) or 512 (up to 4,608 cells, two per CU)
  uint32_t skip_done;         // k_finish_bucket: leave buckets already marked 1 alone (a
                              // 1,024-thread launch after a 512-thread one)
  int32_t rec12;              // packed records are 12 bytes (see PassArgs) unless *big_seg
  const int32_t* big_seg;
};

// Copies n bytes (a multiple of 4) from host memory to dst through kernel
// arguments, in chunks of kUploadChunk bytes: no staging buffer, no memcpy.
constexpr uint32_t kUploadChunk = 3072;
hipError_t launch_upload(void* dst, const void* src, size_t n, hipStream_t s);
hipError_t launch_validate(const ItemDev* items, uint32_t n_items, uint64_t max_len,
                           int32_t* item_status, int32_t* abort_flag, int32_t offset_width,
                           hipStream_t s);
// Exclusive scans of `narr` (1 or 2) u32 arrays of length *n (<= n_max) into
// u64 outputs of length n + 1 (out[n] = total).
hipError_t launch_scan(const uint32_t* in0, uint64_t* out0, const uint32_t* in1, uint64_t* out1,
                       const uint64_t* n_dev, uint64_t n_max, uint64_t* block_sums,
                       hipStream_t s);
// out[k] = w * (in[0] + ... + in[k-1]) for k = 0..n, as offsets of width ow
// (4 or 8); block_sums as for launch_scan.
hipError_t launch_scan_offsets(const uint32_t* in, uint64_t n, uint32_t w, int ow, void* out,
                               uint64_t* block_sums, hipStream_t s);
// Per-cell sort key and carried value of a view operation (LocalTranspose or
// ViewSwap, Section 3) on one item whose bounds are already on the device.
struct ViewArgs {
  const ItemDev* items;       // item 0: row_ptr over the virtual rows, status slot
  const int64_t* bounds;      // device, n_parts + 1 partition bounds of X
  int32_t n_parts;
  const int32_t* col;         // the matrix's own column ids
  uint32_t* keys;             // out: sort key per cell (becomes the item's col)
  uint32_t* vals;             // out: value per cell (becomes the output column id)
  uint64_t nnz, n_virtual;    // cells; rows of the input CSR (n_rows, or R * n_rows)
  int64_t n_rows, n_cols;     // of the matrix X the views represent
  int32_t op;                 // 0 LocalTranspose, 1 ViewSwap
  int32_t column_view;        // input is in column view
  int32_t validate;
  int32_t offset_width;
  int32_t* item_status;
  int32_t* abort_flag;
};
hipError_t launch_view_keys(const ViewArgs& a, hipStream_t s);
hipError_t launch_pass_hist(const PassArgs& a, hipStream_t s);
hipError_t launch_pass_scatter(const PassArgs& a, hipStream_t s);
hipError_t launch_pass_scatter_wide(const PassArgs& a, hipStream_t s);  // records-only pass
hipError_t launch_pass0_slim(const PassArgs& a, hipStream_t s);         // packed first pass (slim)
hipError_t launch_children(const ChildArgs& a, hipStream_t s);
hipError_t launch_finish(const FinishArgs& a, hipStream_t s);
// Whole-bucket finish of a gathering call with packed records (runs before
// launch_finish, which then skips the buckets it wrote).
hipError_t launch_finish_bucket(const FinishArgs& a, hipStream_t s);
// A small matrix in one launch (two for a partitioned call; see k_direct). Its
// arguments travel with the launch: no upload, no workspace.
constexpr uint32_t kDirectCols = 256;   // columns a workgroup may own
constexpr uint32_t kDirectWgs = 256;    // workgroups that share the columns
constexpr int32_t kDirectParts = 256;   // partitions whose bounds fit the arguments
struct DirectArgs {
  const void* row_ptr;
  const int32_t* col;
  const void* poff;
  const uint8_t* payload;
  void* t_row_ptr;
  int32_t* t_col;
  void* t_poff;               // may be null (fixed-width cells)
  uint8_t* t_payload;
  uint32_t* perm;             // may be null
  int64_t* xfer_cells;        // partitioned calls (n_parts > 0)
  int64_t* xfer_bytes;
  int64_t* part_cell_off;
  int64_t* part_byte_off;
  int64_t* sdispls;           // may be null
  int64_t* rdispls;           // may be null
  int32_t* d_status;          // may be null
  int64_t n_rows, n_cols;     // < 2^31
  uint64_t payload_bytes;     // < 2^32
  uint32_t nnz;               // > 0
  uint32_t cols_per_wg;       // <= kDirectCols
  uint32_t n_wg;              // cols_per_wg * n_wg >= n_cols
  int32_t lg;                 // offsets of 2^lg bytes (2 or 3)
  int32_t fixed_w;            // bytes of every cell, or -1
  int32_t n_parts;            // 0: plain call
  int32_t bounds[kDirectParts + 1];
};
static_assert(sizeof(DirectArgs) <= 2048, "kernel argument size");
hipError_t launch_direct(const DirectArgs& a, hipStream_t s);
// A mid-size matrix in two launches (see tiles.hip): tiles sorted by column bucket, then one workgroup per bucket.
constexpr uint32_t kTileMax = 16384;     // cells of a tile
constexpr uint32_t kTileSub = 4096;      // cells of a tile ranked at once
constexpr uint32_t kTileTiles = 512;     // tiles of a call
constexpr uint32_t kTileBuckets = 2048;  // buckets of a call
constexpr uint32_t kTileCols = 512;      // columns of a bucket
constexpr uint32_t kTileCap = 4608;      // cells of a bucket held at once
constexpr uint32_t kTileBins = 4096;     // column runs of a table of uneven buckets
struct TileArgs {
  const void* row_ptr;
  const int32_t* col;
  const void* poff;
  const uint8_t* payload;
  void* t_row_ptr;
  int32_t* t_col;
  void* t_poff;               // may be null (fixed-width cells)
  uint8_t* t_payload;
  uint32_t* perm;             // may be null
  int64_t* xfer_cells;        // partitioned calls (n_parts > 0)
  int64_t* xfer_bytes;
  int64_t* part_cell_off;
  int64_t* part_byte_off;
  int64_t* sdispls;           // may be null
  int64_t* rdispls;           // may be null
  int32_t* d_status;          // may be null
  uint2* table;               // workspace: [tile][bucket] (start | cells << 16, bytes before)
  uint32_t* recs;             // workspace: the records, tile by tile
  uint32_t* bad;              // workspace: a flag per tile (validate)
  uint16_t* lut;              // workspace, or null for buckets of cpb columns each: the bucket
                              // of every run of 2^lut_shift columns (k_tile_bounds)
  uint32_t* bcol;             // with lut: every bucket's first column, n_buckets + 1 entries
  uint32_t lut_shift, tile_target;  // with lut: and the cells a bucket aims for
  const uint32_t* vval;       // view operations: the value of every cell, in place of its row
  uint64_t nnz, payload_bytes;  // payload_bytes < 2^32
  int64_t n_rows, n_cols;     // < 2^31
  uint32_t cpb;               // columns per bucket
  uint32_t magic;             // 2^32 / cpb rounded up (cpb > 1)
  uint32_t n_buckets, n_tiles, tile_cells;
  uint32_t g8;                // n_buckets rounded up to a multiple of 8
  int32_t lg;                 // offsets of 2^lg bytes (2 or 3)
  int32_t fixed_w;            // bytes of every cell, or -1
  int32_t n_parts;            // 0: plain call; <= kDirectParts
  int32_t validate;
  uint64_t* xpart;            // partitioned calls of their own: workspace for X and B by pieces
};
// The counting of a partitioned call's transfer matrices (tiles.hip) goes by
// shares of 2^kXferLg cells, cut into pieces at the partitions.
constexpr int kXferLg = 12;
inline uint32_t xfer_pieces(uint64_t nnz, int32_t n_parts) {
  return (uint32_t)((nnz + (1ull << kXferLg) - 1) >> kXferLg) + (uint32_t)n_parts - 1u;
}
struct TileBounds {
  int32_t bounds[kDirectParts + 1];
};
// Single call: the item's arguments travel with the launches. perm decides the
// record form.
hipError_t launch_tiles(const TileArgs& a, const TileBounds& b, hipStream_t s);
// A view operation's sort keys and carried values (as launch_view_keys, with
// the arguments beside the launch); its tiles then take keys as columns and
// the values as vval.
struct TileView {
  const void* row_ptr;        // over the virtual rows
  const int32_t* col;
  uint32_t* keys;
  uint32_t* vals;
  uint64_t nnz, n_virtual;    // cells; rows of the input CSR
  int64_t n_rows, n_cols;     // of the matrix the views represent
  int32_t op, column_view, n_parts, lg;
};
hipError_t launch_tile_keys(const TileView& v, const TileBounds& b, hipStream_t s);
// Batch: the items' arguments lie in memory, with running totals of their
// tiles, buckets, and pieces of the counting of partitioned items (n_items + 1
// entries each).
struct TileBatch {
  const TileArgs* items;
  const uint32_t* tile_base;
  const uint32_t* bucket_base;
  const uint32_t* piece_base;
  const int32_t* bounds;      // kDirectParts + 1 per partitioned item, in order
  const uint32_t* part_item;  // per item: its index among the partitioned ones
  uint32_t n_items;
  uint32_t n_tiles, n_buckets, n_pieces;  // the totals
  uint32_t max_buckets;       // of one item
  int32_t idx;                // every item has perm
  const int32_t* abort_flag;  // of the batch's items that make the passes, launched before: set if
                              // one of them failed, which cancels these too (null: there are none)
};
hipError_t launch_tile_batch(const TileBatch& b, hipStream_t s);
// mgt_symmetrize's stages after the transpose of the stored triangle
// (symmetric.hip). Every offset array has width ow.
struct SymArgs {
  uint64_t n, nnz;             // rows (= columns) and stored cells
  uint64_t pbytes;             // payload bytes of the triangle (and of its transpose)
  uint64_t cap_cells;          // capacity of s_col (2 nnz) and of s_payload (2 pbytes)
  uint64_t cap_bytes;
  int32_t ow, lower, validate;
  const void* row_ptr;         // the stored triangle
  const int32_t* col;
  const void* poff;
  const uint8_t* payload;
  const void* t_row_ptr;       // its transpose
  const int32_t* t_col;
  const void* t_poff;
  const uint8_t* t_payload;
  void* s_row_ptr;             // the full symmetric matrix
  int32_t* s_col;
  void* s_poff;
  uint8_t* s_payload;
  int64_t* d_sizes;            // cells and payload bytes of S (may be null)
  int32_t* d_status;           // the caller's status word (may be null)
  int32_t* st;                 // the call's status: the transpose's, then these stages'
  uint32_t* cnt;               // per row of S: cells, payload bytes
  uint32_t* byt;
  uint64_t* ocnt;              // their exclusive scans (n + 1 entries)
  uint64_t* obyt;
  uint64_t* scan;              // scratch of launch_scan for n entries
};
hipError_t launch_symmetrize(const SymArgs& a, hipStream_t s);

// The allocation-free transpose (runtime.cpp), called by mgt_transpose_noalloc.
int noalloc_call(mgt_plan_t p, int32_t partitioned, const void* row_ptr, const int32_t* col,
                 const void* payload_off, const uint8_t* payload, void* t_row_ptr, int32_t* t_col,
                 void* t_payload_off, uint8_t* t_payload, uint32_t* perm, int64_t* xfer_cells,
                 int64_t* xfer_bytes, int64_t* part_cell_off, int64_t* part_byte_off,
                 int64_t* sdispls, int64_t* rdispls, void* ws, size_t ws_bytes, int32_t* d_status,
                 hipStream_t stream);
// Scratch needed by launch_scan for n_max elements (bytes).
inline uint64_t scan_scratch_bytes(uint64_t n_max) {
  return 2 * 8 * ((n_max + kScanBlock - 1) / kScanBlock + 1) + 64;
}

}  // namespace mgt
