// The two-launch transpose of mid-size matrices: tiles sorted by column bucket,
// then one workgroup per bucket that collects its cells from every tile.
//
//   k_tile_sort   a workgroup sorts a tile of up to 16,384 consecutive cells
//                 by bucket (a run of `cpb` columns) and writes their records
//                 in that order, with the tile's row of a table: for every
//                 bucket, where its cells start in the tile, how many there
//                 are, and the payload bytes of the tile's earlier buckets.
//   k_tile_merge  a workgroup adds up its bucket's column of that table (the
//                 cells and bytes of all earlier buckets: its place in the
//                 output), collects the bucket's records tile by tile (input
//                 order), ranks them by column in LDS and writes the outputs
//                 in final order, each payload read from the input.
//
// A partitioned call's transfer matrices are counted by workgroups of their own
// beside the tiles, and added up by one beside the buckets.
//
// us per call, this form and the passes (8-byte offsets; 1-8 floats per cell):
// 100 K cells 28 and 54, 300 K 36 and 65, 1 M 49 and 120, 4 M 151 and 414; 4.3 M
// cells of 23 bytes over 37 partitions 189 and 869; 6 M cells of 0 to 7 bytes
// with perm and device checks 218 and 571. Columns that crowd leave some buckets
// to one workgroup for long, as they do in the passes: half of the cells in one
// column 300 K 950 and 1,019, 4 M 13,115 and 16,354.
//
// Against the passes of kernels.hip: no histogram launches, no scans of
// (digit, tile) counts and no segment tables between launches; records move
// once, payloads go from the input to their place. It takes one level of up to
// kTileBuckets buckets, so it ends where buckets outgrow the LDS of a
// workgroup. A single call with equal buckets needs nothing prepared in memory: its
// arguments travel with the launches (uneven buckets take a launch before them,
// batches an uploaded table of items).
//
// Record of a cell (3 words, a 4th for perm): payload offset (or the payload
// itself, up to 4 bytes), row, column within the bucket << 22 | size,
// input index. A size the field cannot hold is looked up again in the offsets.
// (Payloads of up to 8 bytes in a word more were no faster: 4.3 M cells of 8
// bytes 143 us, against 146 us for 9 bytes read from the input.)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/mgt.h"
#include "kernels.h"
#include "payload.h"
#include "prims.h"

namespace mgt {
namespace tl {

constexpr int kTh = 512;                 // threads of both kernels, two or more workgroups per CU
constexpr int kNW = kTh / kWave;
constexpr int kSortItems = kTileSub / kTh;  // cells per lane and piece of k_tile_sort
constexpr int kSortWave = kSortItems * kWave;
constexpr uint32_t kInline = 4;             // payload bytes a record holds itself
constexpr uint32_t kSizeBits = 22;          // of a record's size field; all ones: look it up
constexpr uint32_t kSizeMask = (1u << kSizeBits) - 1u;
static_assert(kTileCols <= 1 << 10, "column field of a record");

__device__ __forceinline__ int64_t ld_off(const void* p, uint64_t i, int lg) {
  return lg == 2 ? (int64_t)gm((const int32_t*)p)[i] : gm((const int64_t*)p)[i];
}
__device__ __forceinline__ uint32_t ld_lo(const void* p, uint64_t i, int lg) {
  return *gm((const uint32_t*)((const uint8_t*)p + (i << lg)));
}
__device__ __forceinline__ void st_off(void* p, uint64_t i, int64_t v, int lg) {
  if (lg == 2) gm((int32_t*)p)[i] = (int32_t)v;
  else gm((int64_t*)p)[i] = v;
}
__device__ __forceinline__ int ceil_log2(uint32_t x) { return x <= 1 ? 0 : 32 - __clz(x - 1); }

// The thread index, opaque to the compiler where it is read: indexes derived
// from it are recomputed there instead of being kept in registers throughout.
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Batches: the item whose range of `base` (running totals) holds v, found by the
// whole workgroup, and its arguments (uniform, so they load as scalars).
__device__ __forceinline__ uint32_t coop_item(const uint32_t* base, uint32_t n, uint32_t v) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const uint32_t step = (hi - lo + kTh - 1) / kTh;
    const uint32_t p = lo + threadIdx.x * step;
    int c = __syncthreads_count(p < hi && gm(base)[p] <= v);
    c = c < 1 ? 1 : c;
    lo += (uint32_t)(c - 1) * step;
    hi = min(lo + step, hi);
  }
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
}
typedef const __attribute__((address_space(4))) TileArgs* ItemPtr;
__device__ __forceinline__ TileArgs load_item(const TileArgs* items, uint32_t i) {
  TileArgs a;
  __builtin_memcpy(&a, (ItemPtr)(items + i), sizeof(TileArgs));
  return a;
}

// Whether the call's inputs were found invalid (MGT_VALIDATE): k_tile_sort left
// a flag per tile. Every thread of the workgroup must call it.
__device__ __forceinline__ bool any_bad(const TileArgs& a) {
  if (!a.validate) return false;
  bool bad = false;
  for (uint32_t t = threadIdx.x; t < a.n_tiles; t += kTh) bad |= gm(a.bad)[t] != 0u;
  return __syncthreads_or(bad) != 0;
}

// ----------------------------------------------------------------------------- uneven buckets

// Bucket bounds for inputs known to crowd some columns (the transpose of a
// stored triangle: the low columns of a lower one). Equal runs of columns would
// leave a few buckets many times over what a workgroup holds, and the call
// waiting for them (4 M cells of a lower triangle: k_tile_merge 219 us with
// equal runs, 108 with these and 18 for this kernel). One workgroup samples the columns, weighs every run of
// 2^lut_shift columns by its sampled cells over the target and its columns over
// the column limit, and cuts where the running weight passes a whole number.
// Its time is the samples' latency, so calls that do not know their columns to
// be crowded keep equal runs.
constexpr int kBoundTh = 1024;
constexpr uint32_t kSamples = 8192;

__global__ __launch_bounds__(kBoundTh) void k_tile_bounds(TileArgs a) {
  __shared__ uint32_t hist[kTileBins];
  __shared__ uint64_t red[kBoundTh / kWave];
  constexpr int kPer = kTileBins / kBoundTh;
  for (uint32_t i = threadIdx.x; i < kTileBins; i += kBoundTh) hist[i] = 0;
  __syncthreads();
  const uint32_t n_cols = (uint32_t)a.n_cols;
  // kSamples evenly spaced groups of four cells (the call has more than 4 kSamples)
  typedef uint32_t col4 __attribute__((ext_vector_type(4), aligned(4)));
  const uint64_t step = a.nnz / kSamples, ns = 4ull * kSamples;
  constexpr int kQ = kSamples / kBoundTh;
  col4 c[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q)
    c[q] = *(const GMEM col4*)gm(a.col + ((uint64_t)q * kBoundTh + threadIdx.x) * step);
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
#pragma unroll
    for (int j = 0; j < 4; ++j) atomicAdd(&hist[min(c[q][j], n_cols - 1u) >> a.lut_shift], 1u);
  }
  __syncthreads();
  // weights in 2^-32 of a bucket
  const uint64_t per_cell = (a.nnz << 32) / (ns * a.tile_target);
  const uint64_t per_col = (1ull << 32) / (kTileCols - (1u << a.lut_shift));
  const uint32_t b0 = threadIdx.x * kPer;
  uint64_t v[kPer], s = 0, tot;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const uint64_t c0 = min((uint64_t)(b0 + q) << a.lut_shift, (uint64_t)n_cols);
    const uint64_t c1 = min((uint64_t)(b0 + q + 1) << a.lut_shift, (uint64_t)n_cols);
    v[q] = hist[b0 + q] * per_cell + (c1 - c0) * per_col;
    s += v[q];
  }
  uint64_t ex = block_excl_scan<kBoundTh / kWave>(s, red, tot);
  const uint32_t last = a.n_buckets - 1;
  __shared__ uint32_t ends[kBoundTh];  // the bucket of each thread's last run
  ends[threadIdx.x] = min((uint32_t)((ex + s - v[kPer - 1]) >> 32), last);
  __syncthreads();
  uint32_t prev = threadIdx.x ? ends[threadIdx.x - 1] : 0u;
  if (threadIdx.x == 0) gm(a.bcol)[0] = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const uint32_t d = min((uint32_t)(ex >> 32), last);
    const uint64_t c0 = min((uint64_t)(b0 + q) << a.lut_shift, (uint64_t)n_cols);
    gm(a.lut)[b0 + q] = (uint16_t)d;
    for (uint32_t x = prev + 1; x <= d; ++x) gm(a.bcol)[x] = (uint32_t)c0;  // (skipped buckets are empty)
    prev = d;
    ex += v[q];
  }
  if (threadIdx.x == kBoundTh - 1)
    for (uint32_t x = prev + 1; x <= a.n_buckets; ++x) gm(a.bcol)[x] = n_cols;
}

// ----------------------------------------------------------------------------- tile sort

struct SortLds {
  uint32_t incl[kTileSub];  // row starts per position, then their inclusive scan
  uint64_t red[2 * kNW];
};
// Beside it, sized by the call's buckets: 16-bit (bucket, wave) counts, then
// positions; the next position of every bucket; payload bytes per bucket.
extern __shared__ uint16_t s_dyn[];
inline uint32_t sort_dyn_bytes(uint32_t n_buckets) { return n_buckets * (2u * kNW + 8u); }

// Row owning cell k: the last row starting at or before it, found by the whole
// workgroup (each round probes kTh evenly spaced rows).
__device__ __forceinline__ uint32_t coop_row(const void* rp, int lg, uint64_t n_rows, uint64_t k) {
  uint64_t lo = 0, hi = n_rows;
  while (hi - lo > 1) {
    const uint64_t step = (hi - lo + kTh - 1) / kTh;
    const uint64_t p = lo + (uint64_t)threadIdx.x * step;
    const bool ok = p < hi && (uint64_t)ld_off(rp, min(p, n_rows), lg) <= k;
    int c = __syncthreads_count(ok);
    c = c < 1 ? 1 : c;
    lo = lo + (uint64_t)(c - 1) * step;
    hi = min(lo + step, hi);
  }
  return (uint32_t)lo;
}

// Rows of the cells [kb, kb + m), the first of which lies in row r0: the row
// starts after it counted per position (incl zero before, and a barrier after
// that), then scanned: cell kb + i lies in row r0 + incl[i]. Returns the rows
// that start among them. Every thread must call both.
__device__ __forceinline__ void mark_rows(const void* rp, int lg, uint64_t n_rows, uint64_t kb, uint32_t m,
                                          uint32_t r0, uint32_t* incl) {
  bool more = true;
  for (uint64_t base = (uint64_t)r0 + 1; more; base += kTh) {
    const uint64_t r = base + threadIdx.x;
    bool stop = r >= n_rows;
    if (!stop) {
      const uint64_t v = (uint64_t)ld_off(rp, r, lg);
      if (v >= kb && v < kb + m) atomicAdd(&incl[v - kb], 1u);
      stop = v >= kb + m;
    }
    more = !__syncthreads_or(stop);
  }
}
__device__ __forceinline__ uint32_t scan_rows(uint32_t* incl, uint32_t* red) {
  constexpr int kPer = kTileSub / kTh;
  const uint32_t p0 = threadIdx.x * kPer;
  uint32_t v[kPer], s = 0, rows;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    v[q] = incl[p0 + q];
    s += v[q];
  }
  uint32_t ex = block_excl_scan<kNW>(s, red, rows);
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    ex += v[q];
    incl[p0 + q] = ex;
  }
  return rows;
}

// Device-side data checks of this tile's share of the inputs (as k_validate). The
// rows' share can be far larger than the tile (few cells over many rows), so
// kRows of its offsets are in flight per thread while that many are left: 2^24
// rows of 100 cells 47 ms with one, 33 so (by the passes 43).
__device__ bool tile_bad(const TileArgs& a, uint32_t t) {
  bool bad = false;
  const uint64_t n_rows = (uint64_t)a.n_rows, nnz = a.nnz;
  const uint64_t pr = (n_rows + a.n_tiles) / a.n_tiles;  // n_rows + 1 offsets, rounded up
  const uint64_t r1 = min(n_rows + 1, (t + 1) * pr);
  constexpr int kRows = 8;
  uint64_t i = t * pr + threadIdx.x;
  for (; i + (kRows - 1) * kTh < min(r1, n_rows); i += kRows * kTh) {
    int64_t v[kRows], w[kRows];
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      v[q] = ld_off(a.row_ptr, i + (uint64_t)q * kTh, a.lg);
      w[q] = ld_off(a.row_ptr, i + (uint64_t)q * kTh + 1, a.lg);
    }
#pragma unroll
    for (int q = 0; q < kRows; ++q) bad |= w[q] < v[q] || (q == 0 && i == 0 && v[q] != 0);
  }
  for (; i < r1; i += kTh) {
    const int64_t v = ld_off(a.row_ptr, i, a.lg);
    if (i == 0 && v != 0) bad = true;
    if (i == n_rows ? v != (int64_t)nnz : ld_off(a.row_ptr, i + 1, a.lg) < v) bad = true;
  }
  const uint64_t k0 = (uint64_t)t * a.tile_cells;
  const uint64_t k1 = t + 1 == a.n_tiles ? nnz + 1 : min(nnz + 1, k0 + a.tile_cells);
  for (uint64_t k = k0 + threadIdx.x; k < k1; k += kTh) {
    if (a.fixed_w < 0) {
      const int64_t v = ld_off(a.poff, k, a.lg);
      if (k == 0 && v != 0) bad = true;
      if (k == nnz) {
        if (v != (int64_t)a.payload_bytes) bad = true;
      } else {
        const int64_t d = ld_off(a.poff, k + 1, a.lg) - v;
        if (d < 0 || d >= ((int64_t)1 << 32)) bad = true;
      }
    }
    if (k < nnz) {
      const int32_t c = gm(a.col)[k];
      if (c < 0 || (int64_t)c >= a.n_cols) bad = true;
    }
  }
  return bad;
}

// ----------------------------------------------------------------------------- transfer matrices

struct NoBounds {};
struct XferLds {
  uint32_t cnt[kDirectParts], byt[kDirectParts];
  int32_t lb[kDirectParts + 1];      // the partition bounds
  uint32_t start[kDirectParts + 1];  // the first cell of every source partition
};

// The cells are counted in shares of 2^kXferLg, each cut where a source partition
// starts: share w's cells of source s are piece w + s (pieces follow the cells, a
// step in w or in s each, so a piece is one pair). A workgroup takes a piece, two
// rounds of loads, so its time does not hang on how the partitions share the cells
// (1 M cells, 64 partitions, all cells in one: 410 us with as many workgroups for
// each partition, now 78; 8 such items of 300 K in a batch 490 and 126).
// The first piece of source s:
__device__ __forceinline__ uint32_t xfer_first(const XferLds& L, uint32_t s) {
  return (L.start[s] >> kXferLg) + s;
}

// Counts piece p by the owners of its cells' columns into L.cnt and L.byt;
// bounds: the item's partition bounds. Returns its source partition. Ends with a
// barrier.
__device__ __forceinline__ uint32_t xfer_count(const TileArgs& a, uint32_t p, const int32_t* bounds,
                                               XferLds& L) {
  const uint32_t R = (uint32_t)a.n_parts, tid = threadIdx.x;
  static_assert(kDirectParts < kTh, "a partition bound per thread");
  if (tid <= R) {
    const int32_t b = bounds[tid];
    L.lb[tid] = b;
    L.start[tid] = (uint32_t)min((uint64_t)ld_off(a.row_ptr, (uint32_t)b, a.lg), a.nnz);
  }
  if (tid < R) {
    L.cnt[tid] = 0;
    L.byt[tid] = 0;
  }
  __syncthreads();
  // the last source whose first piece is p or before (at least the first one, as its is 0)
  const uint32_t s = (uint32_t)max(__syncthreads_count(tid < R && xfer_first(L, tid) <= p), 1) - 1u;
  const uint64_t w = p > s ? p - s : 0u;
  const uint64_t kb = max((uint64_t)L.start[s], w << kXferLg), ke = min((uint64_t)L.start[s + 1], (w + 1) << kXferLg);
  constexpr uint64_t kQ = 4, kChunk = kTh * kQ;
  for (uint64_t c0 = kb; c0 < ke; c0 += kChunk) {
    uint32_t c[kQ], p0[kQ], p1[kQ];
#pragma unroll
    for (uint32_t q = 0; q < kQ; ++q) {
      const uint64_t k = min(c0 + q * kTh + tid, ke - 1);
      c[q] = (uint32_t)gm(a.col)[k];
      p0[q] = a.fixed_w < 0 ? ld_lo(a.poff, k, a.lg) : 0u;
      p1[q] = a.fixed_w < 0 ? ld_lo(a.poff, k + 1, a.lg) : (uint32_t)a.fixed_w;
    }
    uint32_t owner[kQ] = {};  // the last partition starting at or before the column
    for (uint32_t len = R; len > 1; len -= len / 2) {
#pragma unroll
      for (uint32_t q = 0; q < kQ; ++q)
        owner[q] += L.lb[owner[q] + len / 2] <= (int32_t)c[q] ? len / 2 : 0u;
    }
#pragma unroll
    for (uint32_t q = 0; q < kQ; ++q) {
      if (c0 + q * kTh >= ke) break;  // (block-uniform)
      const bool act = c0 + q * kTh + tid < ke;
      // runs of equal owners in consecutive lanes add up first (sorted rows
      // give a wave few owners), one atomic pair per run
      const uint32_t d = act ? owner[q] : 0xffffffffu, z = act ? p1[q] - p0[q] : 0u;
      const uint32_t lane = lane_id();
      const uint32_t prev = __shfl_up(d, 1, kWave), next = __shfl_down(d, 1, kWave);
      const uint64_t heads = ballot(lane == 0 || prev != d);
      const bool tail = lane == kWave - 1 || next != d;
      const uint32_t incl = wave_incl_scan_u32(z);
      const int h = 63 - (int)__clzll(heads & ((2ull << lane) - 1ull));
      const uint32_t base = __shfl(incl - z, h, kWave);
      if (act && tail) {
        atomicAdd(&L.cnt[d], lane - (uint32_t)h + 1u);
        atomicAdd(&L.byt[d], incl - base);
      }
    }
  }
  __syncthreads();
  return s;
}

// A batch's partitioned items: the counts are added to X and B, which the sort
// has cleared.
__global__ __launch_bounds__(kTh) void k_tile_xfer(TileBatch bt) {
  __shared__ XferLds L;
  const uint32_t i = coop_item(bt.piece_base, bt.n_items, blockIdx.x);
  const TileArgs a = load_item(bt.items, i);
  const uint32_t s = xfer_count(a, blockIdx.x - bt.piece_base[i],
                                bt.bounds + (uint64_t)bt.part_item[i] * (kDirectParts + 1), L);
  const uint32_t R = (uint32_t)a.n_parts;
  for (uint32_t d = threadIdx.x; d < R; d += kTh) {
    if (!L.cnt[d]) continue;
    const uint64_t e = (uint64_t)s * R + d;
    __hip_atomic_fetch_add(gm((unsigned long long*)a.xfer_cells + e), (unsigned long long)L.cnt[d],
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(gm((unsigned long long*)a.xfer_bytes + e), (unsigned long long)L.byt[d],
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// A call of its own: piece p's counts to its row of xpart (cells | bytes << 32
// by destination), which start after every source's pieces (first | number << 32).
__device__ __forceinline__ void xfer_piece(const TileArgs& a, uint32_t p, const int32_t* bounds, XferLds& L) {
  xfer_count(a, p, bounds, L);
  const uint32_t R = (uint32_t)a.n_parts, d = threadIdx.x;
  if (d >= R) return;
  gm(a.xpart)[((uint64_t)p + 1) * R + d] = L.cnt[d] | (uint64_t)L.byt[d] << 32;
  if (p == 0) {
      const uint32_t c0 = L.start[d], c1 = L.start[d + 1];
    const uint32_t n = c1 > c0 ? ((c1 - 1u) >> kXferLg) - (c0 >> kXferLg) + 1u : 0u;
    gm(a.xpart)[d] = xfer_first(L, d) | (uint64_t)n << 32;
  }
}

// X and B from the pieces, by one workgroup (all zero for an input that failed
// its checks), kEntries entries of a thread and two pieces of each in flight. src:
// LDS for kDirectParts words. Ends with a barrier.
__device__ void xfer_sum(const TileArgs& a, bool bad, uint64_t* src) {
  const uint32_t R = (uint32_t)a.n_parts, rr = R * R;
  constexpr int kEntries = 4;
  const GMEM uint64_t* const part = gm(a.xpart);
  for (uint32_t s = threadIdx.x; s < R; s += kTh) src[s] = bad ? 0ull : part[s];
  __syncthreads();
  for (uint32_t e0 = threadIdx.x; e0 < rr; e0 += kEntries * kTh) {
    uint32_t n[kEntries], row[kEntries];
    uint64_t v[kEntries][2];
#pragma unroll
    for (int q = 0; q < kEntries; ++q) {
      const uint32_t e = min(e0 + q * kTh, rr - 1u), s = e / R;
      n[q] = e0 + q * kTh < rr ? (uint32_t)(src[s] >> 32) : 0u;
      row[q] = n[q] ? ((uint32_t)src[s] + 1u) * R + (e - s * R) : 0u;
      v[q][0] = part[row[q]];
      v[q][1] = part[row[q] + (n[q] > 1u ? R : 0u)];
    }
#pragma unroll
    for (int q = 0; q < kEntries; ++q) {
      uint64_t cells = 0, bytes = 0;
      auto add = [&](bool in, uint64_t x) {
        cells += in ? x & 0xffffffffu : 0u;
        bytes += in ? x >> 32 : 0u;
      };
      add(n[q] > 0u, v[q][0]);
      add(n[q] > 1u, v[q][1]);
      auto more = [&](auto k, uint32_t j) {  // k of them from j on
        uint64_t x[k()];
#pragma unroll
        for (uint32_t i = 0; i < k(); ++i) x[i] = part[row[q] + min(j + i, n[q] - 1u) * R];
#pragma unroll
        for (uint32_t i = 0; i < k(); ++i) add(j + i < n[q], x[i]);
      };
      uint32_t j = 2;
      for (; j + 4u < n[q]; j += 16) more(std::integral_constant<uint32_t, 16>{}, j);
      if (j < n[q]) more(std::integral_constant<uint32_t, 4>{}, j);
      const uint32_t e = e0 + q * kTh;
      if (e >= rr) break;
      gm(a.xfer_cells)[e] = (int64_t)cells;
      gm(a.xfer_bytes)[e] = (int64_t)bytes;
    }
  }
  __syncthreads();
}

// Partition offsets and displacements from X and B, by one workgroup.
__device__ void tile_tails(const TileArgs& a, uint64_t* red) {
  const uint32_t R = (uint32_t)a.n_parts, d = threadIdx.x;
  uint64_t cells = 0, bytes = 0, sent = 0;
  if (d < R) {
#pragma unroll 8
    for (uint32_t r = 0; r < R; ++r) {
      if (a.rdispls) a.rdispls[(uint64_t)d * R + r] = (int64_t)cells;
      if (a.sdispls) a.sdispls[(uint64_t)d * R + r] = (int64_t)sent;
      cells += (uint64_t)a.xfer_cells[(uint64_t)r * R + d];
      bytes += (uint64_t)a.xfer_bytes[(uint64_t)r * R + d];
      sent += (uint64_t)a.xfer_cells[(uint64_t)d * R + r];
    }
  }
  uint64_t tc, tb;
  const uint64_t ec = block_excl_scan<kNW>(cells, red, tc);
  const uint64_t eb = block_excl_scan<kNW>(bytes, red, tb);
  if (d < R) {
    a.part_cell_off[d] = (int64_t)ec;
    a.part_byte_off[d] = (int64_t)eb;
  }
  if (d == 0) {
    a.part_cell_off[R] = (int64_t)tc;
    a.part_byte_off[R] = (int64_t)tb;
  }
}

// kIdx: the record carries the cell's input index (perm).
// The tile's columns and sizes are read twice: counted first, which gives every
// bucket its place in the tile, then ranked and stored in pieces of kTileSub
// cells. Tiles of four pieces instead of one leave runs four times as long and
// a quarter of the table for k_tile_merge, whose time goes with the number of
// lines it reads. Bound by the latency of its steps with two workgroups per CU
// in flight; the records are stored straight to their place in the tile's own
// region (whole lines by the time they leave the L2).
// kVal: every cell carries a value of its own (vval) in place of its row id.
// kParts: a partitioned call of its own; the workgroups past the tiles count its
// transfer matrices, a piece each, into xpart for the merge's first workgroup to
// add up. In a launch between the two kernels, with atomic adds, the calls took
// (137 K cells, 13 partitions) 30.3 us, beside the tiles 24.0; (1 M, 64) 71.5 and 67;
// (4.3 M, 37) 185 and 181.
template <bool kIdx, bool kBatch, bool kVal = false, bool kParts = false>
__global__ __launch_bounds__(kTh, 4) void k_tile_sort(TileArgs one, TileBatch bt,
                                                      std::conditional_t<kParts, TileBounds, NoBounds> pb) {
  constexpr int kWords = kIdx ? 4 : 3;
  __shared__ union {
    SortLds sort;
    XferLds xfer;
  } U;
  SortLds& L = U.sort;
  uint32_t t = blockIdx.x;
  if constexpr (kParts) {
    if (t >= one.n_tiles) {
      xfer_piece(one, t - one.n_tiles, pb.bounds, U.xfer);
      return;
    }
  }
  TileArgs a = one;
  if constexpr (kBatch) {
    const uint32_t i = coop_item(bt.tile_base, bt.n_items, t);
    a = load_item(bt.items, i);
    t -= bt.tile_base[i];
  }
  const uint32_t G = a.n_buckets;
  uint16_t* const wc = (uint16_t*)__builtin_assume_aligned(s_dyn, 16);
  uint32_t* const next = (uint32_t*)(wc + G * kNW);
  uint32_t* const byt = next + G;
  const uint32_t w = threadIdx.x / kWave, lane = lane_id();
  const uint64_t k0 = (uint64_t)t * a.tile_cells;
  const uint32_t n = (uint32_t)min((uint64_t)a.tile_cells, a.nnz - k0);
  for (uint32_t i = threadIdx.x; i < G; i += kTh) {
    next[i] = 0;
    byt[i] = 0;
  }
  if (a.validate) {
    const bool bad = __syncthreads_or(tile_bad(a, t)) != 0;
    if (threadIdx.x == 0) gm(a.bad)[t] = bad ? 1u : 0u;
  }
  // the transfer matrices of a batch's item start at zero (k_tile_xfer adds to them)
  if (kBatch && a.n_parts > 0)
    for (uint64_t e = (uint64_t)t * kTh + threadIdx.x; e < (uint64_t)a.n_parts * a.n_parts;
         e += (uint64_t)a.n_tiles * kTh) {
      gm(a.xfer_cells)[e] = 0;
      gm(a.xfer_bytes)[e] = 0;
    }
  // bucket of a column, and the bucket's first column
  auto bucket = [&](uint32_t col, uint32_t& first) {
    // (clamped: columns out of range are undefined input, but stay in bounds)
    const uint32_t c = min(col, (uint32_t)a.n_cols - 1u);
    uint32_t d;
    if (a.lut) {  // uniform
      d = gm(a.lut)[c >> a.lut_shift];
      first = gm(a.bcol)[d];
    } else {
      d = a.cpb > 1u ? __umulhi(c, a.magic) : c;
      if (d * a.cpb > c) --d;  // the reciprocal is rounded up
      first = d * a.cpb;
    }
    return d;
  };
  uint32_t r0 = 0;
  if constexpr (!kVal) r0 = coop_row(a.row_ptr, a.lg, (uint64_t)a.n_rows, k0);
  __syncthreads();
  for (uint32_t c0 = 0; c0 < n; c0 += kTileSub) {  // cells per bucket
    uint32_t col[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r)
      col[r] = (uint32_t)gm(a.col)[k0 + min(c0 + (uint32_t)r * kTh + threadIdx.x, n - 1)];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      uint32_t first;
      if (c0 + (uint32_t)r * kTh + threadIdx.x < n) atomicAdd(&next[bucket(col[r], first)], 1u);
    }
  }
  __syncthreads();
  // every bucket's place in the tile (kPer consecutive buckets per thread)
  constexpr int kPerG = kTileBuckets / kTh;
  const uint32_t g0 = threadIdx.x * kPerG;
  {
    uint32_t s = 0, c[kPerG], tot;
#pragma unroll
    for (int q = 0; q < kPerG; ++q) {
      c[q] = g0 + q < G ? next[g0 + q] : 0u;
      s += c[q];
    }
    uint32_t ex = block_excl_scan<kNW>(s, (uint32_t*)L.red, tot);
#pragma unroll
    for (int q = 0; q < kPerG; ++q) {
      if (g0 + q < G) next[g0 + q] = ex;
      ex += c[q];
    }
  }
  const int dbits = ceil_log2(G);
  uint32_t* const rec = a.recs + k0 * kWords;
  for (uint32_t c0 = 0; c0 < n; c0 += kTileSub) {
    const uint32_t m = min(kTileSub, n - c0);
    const uint64_t kb = k0 + c0;
    // key: column within the bucket and size; at: the (bucket, wave) counter
    uint32_t off[kSortItems], key[kSortItems], at[kSortItems], dig[kSortItems], end;
    uint32_t val[kVal ? kSortItems : 1];
    {
      uint32_t col[kSortItems];
#pragma unroll
      for (int r = 0; r < kSortItems; ++r) {
        const uint32_t i = w * kSortWave + r * kWave + lane;
        col[r] = (uint32_t)gm(a.col)[kb + min(i, m - 1)];
        off[r] = a.fixed_w < 0 ? ld_lo(a.poff, kb + min(i, m), a.lg)
                               : (uint32_t)(kb + min(i, m)) * (uint32_t)a.fixed_w;
      }
      if constexpr (kVal) {
#pragma unroll
        for (int r = 0; r < kSortItems; ++r)
          val[r] = gm(a.vval)[kb + min(w * kSortWave + r * kWave + lane, m - 1)];
      }
      const uint32_t e = min(w * kSortWave + kSortWave, m);
      end = a.fixed_w < 0 ? ld_lo(a.poff, kb + e, a.lg) : (uint32_t)(kb + e) * (uint32_t)a.fixed_w;
      for (uint32_t i = threadIdx.x; i < kTileSub; i += kTh) L.incl[i] = 0;
      for (uint32_t i = threadIdx.x; i < G * kNW / 2; i += kTh) ((uint32_t*)wc)[i] = 0;
      __syncthreads();
      if constexpr (!kVal) mark_rows(a.row_ptr, a.lg, (uint64_t)a.n_rows, kb, m, r0, L.incl);
#pragma unroll
      for (int r = 0; r < kSortItems; ++r) {  // a cell's size: the next cell's offset minus its own
        uint32_t nx = (uint32_t)__shfl_down((int)off[r], 1);
        const uint32_t wrap = r + 1 < kSortItems
            ? (uint32_t)__builtin_amdgcn_readlane((int)off[r + 1 < kSortItems ? r + 1 : r], 0) : end;
        if (lane == kWave - 1) nx = wrap;
        uint32_t first;
        const uint32_t z = nx - off[r];
        dig[r] = bucket(col[r], first);
        at[r] = dig[r] * kNW + w;
        key[r] = ((min(col[r], (uint32_t)a.n_cols - 1u) - first) << kSizeBits) | min(z, kSizeMask);
        if (w * kSortWave + r * kWave + lane < m && z) atomicAdd(&byt[dig[r]], z);
      }
    }
    uint32_t rank[kSortItems];
    wave_ranks(wc, at, dig, m > w * kSortWave ? m - w * kSortWave : 0u, dbits, rank);
    uint32_t rows = 0;
    if constexpr (kVal) __syncthreads();  // all counters are in
    else rows = scan_rows(L.incl, (uint32_t*)L.red);  // (likewise)
    // counts to positions: the bucket's next one, then wave by wave
    for (uint32_t g = threadIdx.x; g < G; g += kTh) {
      v4 c = *(const v4*)&wc[g * kNW];
      uint32_t p = next[g];
      v4 o;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t lo = p;
        p += c[j] & 0xffffu;
        o[j] = lo | (p << 16);
        p += c[j] >> 16;
      }
      *(v4*)&wc[g * kNW] = o;
      next[g] = p;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      const uint32_t i = w * kSortWave + r * kWave + lane;
      if (i >= m) continue;
      const uint32_t z = key[r] & kSizeMask;
      uint32_t x = off[r];
      // a small payload goes in place of its offset, from the aligned words that hold
      // it (each holds one of its bytes; the array's first and last word may hold up
      // to three bytes of its neighbours, no further word is read)
      if (z && z <= kInline && (uint64_t)x + z <= a.payload_bytes) {
        const uint8_t* const p = a.payload + x;
        const uint32_t sh = 8u * ((uint32_t)(uintptr_t)p & 3u);
        const GMEM uint32_t* const q = gm((const uint32_t*)((uintptr_t)p & ~(uintptr_t)3));
        const uint32_t nb = ((uint32_t)(uintptr_t)p & 3u) + z;
        const uint32_t w0 = q[0], w1 = nb > 4u ? q[1] : 0u;
        x = (uint32_t)((((uint64_t)w1 << 32) | w0) >> sh);
      }
      const uint32_t row = kVal ? val[kVal ? r : 0] : r0 + L.incl[i];
      const uint32_t p = (uint32_t)wc[at[r]] + rank[r];
      GMEM uint32_t* const o = gm(rec + (uint64_t)p * kWords);
      if constexpr (kWords == 3) {
        o[0] = x;
        o[1] = row;
        o[2] = key[r];
      } else {
        typedef uint32_t r4 __attribute__((ext_vector_type(4), aligned(4)));
        *(GMEM r4*)o = r4{x, row, key[r], (uint32_t)kb + i};
      }
    }
    r0 += rows;    // the row of the piece's last cell; later rows start at the next piece or after
    __syncthreads();  // rows and positions have been read
  }
  {  // the tile's row of the table: (start, cells) and the bytes of the earlier buckets
    uint32_t s = 0, b[kPerG], tot;
#pragma unroll
    for (int q = 0; q < kPerG; ++q) {
      b[q] = g0 + q < G ? byt[g0 + q] : 0u;
      s += b[q];
    }
    uint32_t eb = block_excl_scan<kNW>(s, (uint32_t*)L.red, tot);
    uint32_t start = g0 && g0 <= G ? next[g0 - 1] : 0u;  // (every bucket's end is in `next` by now)
    uint2* const row = a.table + (uint64_t)t * G;
#pragma unroll
    for (int q = 0; q < kPerG; ++q) {
      if (g0 + q < G) {
        const uint32_t end = next[g0 + q];
        gm(row)[g0 + q].x = start | ((end - start) << 16);
        gm(row)[g0 + q].y = eb;
        start = end;
      }
      eb += b[q];
    }
  }
}

// ----------------------------------------------------------------------------- view keys

// Sort key and carried value of every cell of a view operation (see k_view_keys
// in kernels.hip for the four cases), kTileSub cells per workgroup.
__global__ __launch_bounds__(kTh) void k_tile_keys(TileView v, TileBounds b) {
  __shared__ uint32_t incl[kTileSub];
  __shared__ int32_t lb[kDirectParts + 1];
  __shared__ uint32_t red[kNW];
  const uint32_t R = (uint32_t)v.n_parts;
  for (uint32_t i = threadIdx.x; i <= R; i += kTh) lb[i] = b.bounds[i];
  for (uint32_t i = threadIdx.x; i < kTileSub; i += kTh) incl[i] = 0;
  const uint64_t k0 = (uint64_t)blockIdx.x * kTileSub;
  const uint32_t m = (uint32_t)min((uint64_t)kTileSub, v.nnz - k0);
  const uint32_t r0 = coop_row(v.row_ptr, v.lg, v.n_virtual, k0);
  __syncthreads();
  mark_rows(v.row_ptr, v.lg, v.n_virtual, k0, m, r0, incl);
  scan_rows(incl, red);
  __syncthreads();
  // the last partition starting at or before x
  auto owner = [&](int64_t x) {
    uint32_t lo = 0, hi = R;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (lb[mid] <= x) lo = mid;
      else hi = mid;
    }
    return lo;
  };
  constexpr int kPer = kTileSub / kTh;
  int32_t col[kPer];
#pragma unroll
  for (int r = 0; r < kPer; ++r) col[r] = gm(v.col)[k0 + min((uint32_t)(r * kTh) + threadIdx.x, m - 1)];
#pragma unroll
  for (int r = 0; r < kPer; ++r) {
    const uint32_t i = (uint32_t)(r * kTh) + threadIdx.x;
    if (i >= m) break;
    const uint32_t row = r0 + incl[i];
    uint64_t key;
    uint32_t val;
    if (!v.column_view) {
      key = v.op == 0 ? (uint64_t)owner(row) * (uint64_t)v.n_cols + (uint64_t)(int64_t)col[r]
                      : (uint64_t)owner(col[r]) * (uint64_t)v.n_rows + row;
      val = v.op == 0 ? row : (uint32_t)col[r];
    } else {
      const uint32_t i_row = row % (uint32_t)v.n_rows;
      key = v.op == 0 ? (uint64_t)(int64_t)col[r] : i_row;
      val = v.op == 0 ? i_row : (uint32_t)col[r];
    }
    gm(v.keys)[k0 + i] = (uint32_t)key;
    gm(v.vals)[k0 + i] = val;
  }
}

// ----------------------------------------------------------------------------- bucket merge

constexpr int kMergeItems = kTileCap / kTh;  // cells per lane of a bucket held at once
constexpr uint32_t kMergeWave = kMergeItems * kWave;
constexpr uint32_t kMergeLead = 8;  // one workgroup per XCD, so the buckets' own mapping stays

struct MergeLds {
  // output order: row, payload offset (or payload), size then byte prefix.
  // Before that, in `row`: the record of every cell, or its tile.
  uint32_t row[kTileCap], src[kTileCap], bp[kTileCap + 1];
  union {
    struct {
      uint32_t ex[kTileTiles];  // first cell (bucket order) of every tile's run
      uint16_t st[kTileTiles];  // where the run starts in the tile
    };
    alignas(16) uint8_t stage[kNW][kStage];  // after the records are read, single-chunk buckets only
  };
  alignas(16) uint16_t wc[kTileCols * kNW];  // (column, wave) counts, then first positions
  uint32_t red[kNW];
  uint64_t red64[2 * kNW];
};

// Size of a record's cell: from the offsets where the field cannot hold it
// (its payload is not inline, so x is its offset: the last cell starting there).
__device__ __forceinline__ uint32_t rec_size(const TileArgs& a, uint32_t key, uint32_t x) {
  uint32_t z = key & kSizeMask;
  if (z == kSizeMask) {
    if (a.fixed_w >= 0) return (uint32_t)a.fixed_w;
    uint64_t lo = 0, hi = a.nnz;
    while (hi - lo > 1) {
      const uint64_t mid = (lo + hi) >> 1;
      if (ld_lo(a.poff, mid, a.lg) <= x) lo = mid;
      else hi = mid;
    }
    z = ld_lo(a.poff, lo + 1, a.lg) - x;
  }
  return z;
}

// The words of record i (byte offsets stay below 2^32: 2^23 records of 16 bytes).
template <uint32_t kWords>
__device__ __forceinline__ const GMEM uint32_t* record(const TileArgs& a, uint32_t i) {
  return (const GMEM uint32_t*)(gm((const uint8_t*)a.recs) + i * (4u * kWords));
}

// Cells of a run (or of a thread's share of one) up to which the threads list
// them one by one.
constexpr uint32_t kShortRun = 32;

// The tile of every cell of bucket cells [q0, q0 + m), in tl[0..m): the tile
// runs' starts marked and spread upwards (ex: every tile's first cell, n cells
// in all). Ends with a barrier.
template <int kItems>
__device__ __forceinline__ void cell_tiles(const uint32_t* ex, uint32_t T, uint32_t n, uint32_t q0,
                                           uint32_t m, uint32_t* tl, uint32_t* red) {
  for (uint32_t i = threadIdx.x; i < m; i += kTh) tl[i] = 0;
  __syncthreads();
  for (uint32_t t = threadIdx.x; t < T; t += kTh) {
    const uint32_t e = ex[t], end = t + 1 < T ? ex[t + 1] : n;
    if (end > e && end > q0 && e < q0 + m) tl[max(e, q0) - q0] = t + 1;
  }
  __syncthreads();
  // inclusive maximum: each thread's run, then over the threads
  uint32_t v[kItems], s = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t i = threadIdx.x * kItems + j;
    v[j] = i < m ? tl[i] : 0u;
    s = max(s, v[j]);
  }
  uint32_t inc = s;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t u = (uint32_t)__shfl_up((int)inc, o, kWave);
    if (lane_id() >= (uint32_t)o) inc = max(inc, u);
  }
  const uint32_t w = threadIdx.x / kWave;
  if (lane_id() == kWave - 1) red[w] = inc;
  __syncthreads();
  uint32_t run = (uint32_t)__shfl_up((int)inc, 1, kWave);
  if (lane_id() == 0) run = 0;
#pragma unroll
  for (int i = 0; i < kNW; ++i)
    if ((uint32_t)i < w) run = max(run, red[i]);
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t i = threadIdx.x * kItems + j;
    run = max(run, v[j]);
    if (i < m) tl[i] = run;
  }
  __syncthreads();
}

// Two workgroups per CU (80 KB of LDS each), so one's collection and ranking
// run beside the other's payload reads. Bound by those: each payload that is
// not inline costs a 128-byte line from the memory-side cache or HBM, and a CU
// holds about 65 such reads in flight. Buckets run in plain column order within
// each XCD, so neighbouring buckets share the lines of the table and of the
// tiles' records in its L2.
// A bucket of more than kCap cells (skewed columns) is taken in chunks: column
// totals first, then every chunk's cells to their column's running place.
template <bool kIdx, bool kBatch>
__global__ __launch_bounds__(kTh, 4) void k_tile_merge(TileArgs one, TileBatch bt) {
  constexpr int kItems = kMergeItems;
  constexpr uint32_t kCap = kTileCap, kWaveCells = kMergeWave;
  constexpr uint32_t kWords = kIdx ? 4 : 3;
  __shared__ MergeLds L;
  // one workgroup per item besides the buckets': status, end offsets, and a
  // partitioned item's matrices, offsets and displacements. A batch's are the
  // last ones; a single call's is the first of the first eight (the others leave),
  // so that a long sum over the partitions runs beside the buckets.
  const uint32_t g8 = kBatch ? (bt.n_buckets + 7u) & ~7u : one.g8;
  const bool tail = kBatch ? blockIdx.x >= g8 : blockIdx.x < kMergeLead;
  if (!kBatch && tail && blockIdx.x) return;
  uint32_t g = (uint32_t)xcd_tile(kBatch ? blockIdx.x : blockIdx.x - kMergeLead, g8);
  TileArgs a = one;
  if constexpr (kBatch) {
    if (!tail && g >= bt.n_buckets) return;
    const uint32_t i = tail ? blockIdx.x - g8 : coop_item(bt.bucket_base, bt.n_items, g);
    a = load_item(bt.items, (uint32_t)__builtin_amdgcn_readfirstlane((int)i));
    g -= bt.bucket_base[i];
  }
  // (set by an earlier launch or not at all: the same for every workgroup)
  const bool cancelled = kBatch && bt.abort_flag && gm(bt.abort_flag)[0] != 0;
  const bool bad = any_bad(a) || cancelled;
  if (tail) {
    if (threadIdx.x == 0) {
      if (a.d_status) *a.d_status = cancelled ? MGT_ECANCELED : bad ? MGT_ERANGE : MGT_OK;
      if (!bad) {
        st_off(a.t_row_ptr, (uint64_t)a.n_cols, (int64_t)a.nnz, a.lg);
        if (a.t_poff) st_off(a.t_poff, a.nnz, (int64_t)a.payload_bytes, a.lg);
      }
    }
    if (!kBatch && a.n_parts > 0) xfer_sum(a, bad, (uint64_t*)L.row);
    if (!bad && a.n_parts > 0) tile_tails(a, L.red64);
    return;
  }
  if (bad) return;
  const uint32_t G = a.n_buckets, T = a.n_tiles;
  if (g >= G) return;
  const uint32_t col0 = a.lut ? gm(a.bcol)[g] : g * a.cpb;
  const uint32_t nc = a.lut ? gm(a.bcol)[g + 1] - col0 : min(a.cpb, (uint32_t)a.n_cols - col0);
  // the bucket's column of the table: its place in the output, and its runs.
  // `per` tiles per thread; with fewer tiles than threads, `lanes` threads per
  // tile share its run.
  constexpr int kPerT = kTileTiles / kTh;
  const uint32_t per = (T + kTh - 1) / kTh;
  const uint32_t lanes_lg = T * 2 > (uint32_t)kTh ? 0u : 31u - (uint32_t)__clz((uint32_t)kTh / T);
  const uint32_t t0 = lanes_lg ? threadIdx.x >> lanes_lg : threadIdx.x * per;
  const uint32_t sub = threadIdx.x & ((1u << lanes_lg) - 1u);
  uint32_t len[kPerT], ex[kPerT], first[kPerT];  // a run: cells, first cell, first record
  uint32_t n, cell0;
  uint64_t byte0;
  {
    uint64_t s = 0, sb = 0;  // s: cells of the runs, and before them in their tiles << 32
    uint32_t st[kPerT];
#pragma unroll
    for (int j = 0; j < kPerT; ++j) {
      uint2 e = make_uint2(0u, 0u);
      if ((uint32_t)j < per && t0 + j < T) {
        const GMEM uint2* const q = gm(a.table) + (uint64_t)(t0 + j) * G + g;
        e.x = q->x;
        e.y = q->y;
      }
      st[j] = e.x & 0xffffu;
      len[j] = e.x >> 16;
      first[j] = (t0 + j) * a.tile_cells + st[j];
      if (sub == 0) {
        s += (uint64_t)len[j] | ((uint64_t)st[j] << 32);
        sb += e.y;
      }
    }
    uint64_t tot;
    block_excl_scan2<kNW>(s, sb, L.red64, tot, byte0);
    n = (uint32_t)__builtin_amdgcn_readfirstlane((int)tot);
    cell0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tot >> 32));
    uint32_t e = (uint32_t)s;
    if (sub) e -= len[0];  // (the threads of one tile: the first one's run is in their prefix)
#pragma unroll
    for (int j = 0; j < kPerT; ++j) {
      ex[j] = e;
      e += len[j];
    }
  }
  if (n == 0) {
    for (uint32_t c = threadIdx.x; c < nc; c += kTh)
      st_off(a.t_row_ptr, (uint64_t)col0 + c, (int64_t)cell0, a.lg);
    return;
  }
  const bool multi = n > kCap;  // block-uniform
  // Short runs: each thread lists its runs' records. Long ones (columns that
  // crowd into few tiles) would leave one thread to it, so their starts are
  // marked and spread instead (cell_tiles).
  bool lng = multi;
#pragma unroll
  for (int j = 0; j < kPerT; ++j) lng |= (len[j] >> lanes_lg) > kShortRun;
  lng = __syncthreads_or(lng) != 0;  // block-uniform
  if (lng) {
#pragma unroll
    for (int j = 0; j < kPerT; ++j)
      if ((uint32_t)j < per && t0 + j < T && sub == 0) {
        L.ex[t0 + j] = ex[j];
        L.st[t0 + j] = (uint16_t)(first[j] - (t0 + j) * a.tile_cells);
      }
  } else {
#pragma unroll
    for (int j = 0; j < kPerT; ++j)
      for (uint32_t i = sub; i < len[j]; i += 1u << lanes_lg) L.row[ex[j] + i] = first[j] + i;
  }
  __syncthreads();
  // chunked buckets: running first cell and byte of every column (bucket
  // relative), in the last words of `src` and `bp`, which chunks leave free
  const uint32_t chunk = multi ? kCap - kTileCols : kCap;
  uint32_t* const run_c = L.src + chunk;
  uint32_t* const run_b = L.bp + chunk + 1;
  auto column = [&](uint32_t key) { return min(key >> kSizeBits, nc - 1u); };
  if (multi) {
    for (uint32_t c = threadIdx.x; c < nc; c += kTh) {
      run_c[c] = 0;
      run_b[c] = 0;
    }
    for (uint32_t q0 = 0; q0 < n; q0 += chunk) {
      const uint32_t m = min(chunk, n - q0);
      cell_tiles<kItems>(L.ex, T, n, q0, m, L.row, L.red);
      for (uint32_t i = threadIdx.x; i < m; i += kTh) {
        const uint32_t t = L.row[i] - 1u;
        const GMEM uint32_t* const r = record<kWords>(a, t * a.tile_cells + L.st[t] + (q0 + i - L.ex[t]));
        const uint32_t key = r[2], d = column(key);
        atomicAdd(&run_c[d], 1u);
        atomicAdd(&run_b[d], rec_size(a, key, r[0]));
      }
      __syncthreads();
    }
    uint32_t v = 0, u = 0, vt, ut;  // nc <= kTileCols == kTh
    if (threadIdx.x < nc) {
      v = run_c[threadIdx.x];
      u = run_b[threadIdx.x];
    }
    block_excl_scan2<kNW>(v, u, L.red64, vt, ut);
    if (threadIdx.x < nc) {
      run_c[threadIdx.x] = v;
      run_b[threadIdx.x] = u;
      st_off(a.t_row_ptr, (uint64_t)col0 + threadIdx.x, (int64_t)cell0 + v, a.lg);
    }
  }
  for (uint32_t q0 = 0; q0 < n; q0 += chunk) {
    const uint32_t tid = opaque(threadIdx.x);
    const uint32_t w = tid / kWave, lane = tid % kWave;
    const uint32_t m = min(chunk, n - q0);
    __syncthreads();  // the previous chunk's positions have been read
    if (lng) cell_tiles<kItems>(L.ex, T, n, q0, m, L.row, L.red);
    uint32_t x[kItems], row[kItems], key[kItems], idx[kIdx ? kItems : 1];
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      const uint32_t i = min(w * kWaveCells + q * kWave + lane, m - 1u);
      uint32_t ri = L.row[i];
      if (lng) {
        const uint32_t t = ri - 1u;
        ri = t * a.tile_cells + L.st[t] + (q0 + i - L.ex[t]);
      }
      const GMEM uint32_t* const r = record<kWords>(a, ri);
      x[q] = r[0];
      row[q] = r[1];
      key[q] = r[2];
      if constexpr (kIdx) idx[q] = r[3];
    }
    uint32_t pos[kItems];  // every cell's place in output order (bucket relative)
    const uint32_t mine = m > w * kWaveCells ? m - w * kWaveCells : 0u;  // the wave's cells
    for (uint32_t e = tid; e < nc * (kNW / 2); e += kTh) ((uint32_t*)L.wc)[e] = 0;
    __syncthreads();
    uint32_t at[kItems], d[kItems];
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      d[q] = column(key[q]);
      at[q] = d[q] * kNW + w;
    }
    wave_ranks(L.wc, at, d, mine, ceil_log2(nc), pos);
    __syncthreads();
    // column-major scan of the counters (eight per column, one column per thread)
    static_assert(kTileCols == kTh, "one column per thread");
    v4 c = v4{0u, 0u, 0u, 0u};
    if (tid < nc) c = *(const v4*)&L.wc[tid * kNW];
    uint32_t s = 0, tot;
#pragma unroll
    for (int j = 0; j < 4; ++j) s += (c[j] & 0xffffu) + (c[j] >> 16);
    uint32_t ex = block_excl_scan<kNW>(s, L.red, tot);
    if (tid < nc) {
      if (!multi) st_off(a.t_row_ptr, (uint64_t)col0 + tid, (int64_t)cell0 + ex, a.lg);
      v4 o;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t lo = ex;
        ex += c[j] & 0xffffu;
        o[j] = lo | (ex << 16);
        ex += c[j] >> 16;
      }
      *(v4*)&L.wc[tid * kNW] = o;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kItems; ++q) pos[q] += L.wc[at[q]];
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      if ((uint32_t)q * kWave + lane >= mine) continue;
      const uint32_t p = pos[q];
      L.row[p] = row[q];
      L.src[p] = x[q];
      L.bp[p] = rec_size(a, key[q], x[q]);
      if constexpr (kIdx) {
        uint64_t at = (uint64_t)cell0 + p;
        if (multi) {
          const uint32_t d = column(key[q]);
          at = (uint64_t)cell0 + run_c[d] + (p - L.wc[d * kNW]);
        }
        gm(a.perm)[at] = idx[q];
      }
    }
    __syncthreads();
    {  // sizes -> exclusive byte prefix in output order
      uint32_t v[kItems], s = 0, tot;
#pragma unroll
      for (int q = 0; q < kItems; ++q) {
        const uint32_t p = tid * kItems + q;
        v[q] = p < m ? L.bp[p] : 0u;
        s += v[q];
      }
      uint32_t ex = block_excl_scan<kNW>(s, L.red, tot);
#pragma unroll
      for (int q = 0; q < kItems; ++q) {
        const uint32_t p = tid * kItems + q;
        if (p < m) L.bp[p] = ex;
        ex += v[q];
      }
      if (tid == 0) L.bp[m] = tot;
      __syncthreads();
    }
    // outputs in output order, kPay cells per lane with their payloads in flight
    constexpr int kPay = 3;
#pragma unroll 1
    for (int g0 = 0; g0 < kItems; g0 += kPay) {
      uint32_t z[kPay], b[kPay], o[kPay], r[kPay];
      v4 va[kPay], vb[kPay];
      bool shorts = true;
#pragma unroll
      for (int q = 0; q < kPay; ++q) {
        const uint32_t p = (uint32_t)(g0 + q) * kTh + tid;
        const bool act = g0 + q < kItems && p < m;
        const uint32_t pc = act ? p : 0u;
        b[q] = L.bp[pc];
        z[q] = act ? L.bp[pc + 1] - b[q] : 0u;
        o[q] = L.src[pc];
        r[q] = L.row[pc];
        va[q] = v4{o[q], 0u, 0u, 0u};
        vb[q] = v4{0u, 0u, 0u, 0u};
        shorts &= z[q] <= 32u;
        if (z[q] > kInline && z[q] <= 32u)
          get_bytes(a.payload + o[q], a.payload, a.payload + a.payload_bytes, z[q], va[q], vb[q]);
      }
#pragma unroll
      for (int q = 0; q < kPay; ++q) {
        const uint32_t p = (uint32_t)(g0 + q) * kTh + tid;
        if (g0 + q >= kItems || p >= m) continue;
        uint64_t at = (uint64_t)cell0 + p, bt = byte0 + b[q];
        if (multi) {
          uint32_t lo = 0, hi = nc;  // the cell's column: the last one starting at or before p
          while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if ((uint32_t)L.wc[mid * kNW] <= p) lo = mid;
            else hi = mid;
          }
          const uint32_t ds = L.wc[lo * kNW];
          at = (uint64_t)cell0 + run_c[lo] + (p - ds);
          bt = byte0 + run_b[lo] + (b[q] - L.bp[ds]);
          if (z[q] > 32u) copy_long(a.t_payload + bt, a.payload + o[q], z[q]);
          else if (z[q]) put_global(a.t_payload + bt, va[q], vb[q], z[q]);
        }
        gm(a.t_col)[at] = (int32_t)r[q];
        if (a.t_poff) st_off(a.t_poff, at, (int64_t)bt, a.lg);
      }
      if (multi) continue;
      // a wave's 64 payloads are one run of output bytes: packed in LDS, then
      // written 16 bytes per lane
      const bool staged = __all(shorts);
#pragma unroll
      for (int q = 0; q < kPay; ++q) {
        const uint32_t p = (uint32_t)(g0 + q) * kTh + tid;
        const uint64_t act = ballot(g0 + q < kItems && p < m);  // a prefix of the lanes
        if (act == 0) continue;                                  // wave-uniform
        if (!staged) {
          if (z[q] > 32u) copy_long(a.t_payload + byte0 + b[q], a.payload + o[q], z[q]);
          else if (z[q]) put_global(a.t_payload + byte0 + b[q], va[q], vb[q], z[q]);
          continue;
        }
        const uint32_t lastl = 63u - (uint32_t)__clzll(act);
        const uint32_t b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b[q]);
        const uint32_t rel = b[q] - b0;
        const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)(rel + z[q]), (int)lastl);
        write_run(L.stage[w], a.t_payload + byte0 + b0, rel, tot, va[q], vb[q], z[q]);
      }
    }
    if (multi) {
      __syncthreads();
      if (tid < nc) {
        const uint32_t i0 = L.wc[tid * kNW], i1 = tid + 1 < nc ? (uint32_t)L.wc[(tid + 1) * kNW] : m;
        run_c[tid] += i1 - i0;
        run_b[tid] += L.bp[i1] - L.bp[i0];
      }
    }
  }
}

}  // namespace tl

static_assert(sizeof(tl::MergeLds) <= 80 * 1024, "two workgroups per CU");

template <bool kIdx>
static void launch_tile_kernels(const TileArgs& a, const TileBounds& b, hipStream_t s) {
  const TileBatch none{};
  if (a.lut) hipLaunchKernelGGL(tl::k_tile_bounds, dim3(1), dim3(tl::kBoundTh), 0, s, a);
  const dim3 th(tl::kTh);
  const uint32_t dyn = tl::sort_dyn_bytes(a.n_buckets);
  const tl::NoBounds nob{};
  if (a.vval)
    hipLaunchKernelGGL((tl::k_tile_sort<kIdx, false, true>), dim3(a.n_tiles), th, dyn, s, a, none, nob);
  else if (a.n_parts > 0)
    hipLaunchKernelGGL((tl::k_tile_sort<kIdx, false, false, true>), dim3(a.n_tiles + xfer_pieces(a.nnz, a.n_parts)), th,
                       dyn, s, a, none, b);
  else
    hipLaunchKernelGGL((tl::k_tile_sort<kIdx, false>), dim3(a.n_tiles), th, dyn, s, a, none, nob);
  hipLaunchKernelGGL((tl::k_tile_merge<kIdx, false>), dim3(tl::kMergeLead + a.g8), th, 0, s, a, none);
}

hipError_t launch_tile_keys(const TileView& v, const TileBounds& b, hipStream_t s) {
  const uint64_t nb = (v.nnz + kTileSub - 1) / kTileSub;
  hipLaunchKernelGGL(tl::k_tile_keys, dim3((unsigned)nb), dim3(tl::kTh), 0, s, v, b);
  return hipGetLastError();
}

hipError_t launch_tiles(const TileArgs& a, const TileBounds& b, hipStream_t s) {
  if (a.perm) launch_tile_kernels<true>(a, b, s);
  else launch_tile_kernels<false>(a, b, s);
  return hipGetLastError();
}

template <bool kIdx>
static void launch_batch_kernels(const TileBatch& b, hipStream_t s) {
  const TileArgs none{};
  hipLaunchKernelGGL((tl::k_tile_sort<kIdx, true>), dim3(b.n_tiles), dim3(tl::kTh),
                     tl::sort_dyn_bytes(b.max_buckets), s, none, b, tl::NoBounds{});
  if (b.n_pieces) hipLaunchKernelGGL(tl::k_tile_xfer, dim3(b.n_pieces), dim3(tl::kTh), 0, s, b);
  hipLaunchKernelGGL((tl::k_tile_merge<kIdx, true>), dim3(((b.n_buckets + 7u) & ~7u) + b.n_items),
                     dim3(tl::kTh), 0, s, none, b);
}

hipError_t launch_tile_batch(const TileBatch& b, hipStream_t s) {
  if (b.idx) launch_batch_kernels<true>(b, s);
  else launch_batch_kernels<false>(b, s);
  return hipGetLastError();
}

}  // namespace mgt
