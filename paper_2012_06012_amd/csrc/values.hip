// Conversions between repeated cells and XCSR value lists (Section 2: one cell
// per (row, column) pair whose value is a list of values, plus a count of
// values per cell). Both forms are CSRs over the same payload array: the
// payload bytes keep their order, so these kernels move only row offsets,
// column ids, payload offsets and counts.
//
// Inputs that break the CSR invariants cannot make these kernels access
// memory out of bounds: every offset read is clamped into [0, nnz] (or the
// payload size) before it indexes anything.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/mgt.h"
#include "kernels.h"
#include "prims.h"

namespace mgt {
namespace vl {

constexpr int kB = 256;

__device__ __forceinline__ uint64_t ld_o(const void* p, uint64_t i, int ow) {
  const int64_t v = ow == 4 ? (int64_t)gm((const int32_t*)p)[i] : gm((const int64_t*)p)[i];
  return v < 0 ? 0u : (uint64_t)v;
}
__device__ __forceinline__ void st_o(void* p, uint64_t i, uint64_t v, int ow) {
  if (ow == 4) gm((int32_t*)p)[i] = (int32_t)v;
  else gm((int64_t*)p)[i] = (int64_t)v;
}
__device__ __forceinline__ uint64_t gtid() { return (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; }
__device__ __forceinline__ uint64_t gstride() { return (uint64_t)gridDim.x * blockDim.x; }

// Coalescing. Heads (cells that start a run of equal columns inside their
// row) are kept as a bitmap of one 64-bit word per 64 cells, so the flags and
// their scan move 1/8 byte and 1/16 byte per cell in place of 4 and 8:
//   k_heads      column changes, one ballot word per wave round (reads col)
//   k_row_heads  row starts, ORed in
//   k_head_sums  heads per chunk of kChunkWords words
//   k_head_pref  heads before every word (the chunk's base is the sum of the
//                earlier chunks), the number of output cells m and the last
//                payload offset
//   k_emit       heads to their slots, run lengths, output row offsets
// The bound is memory: col twice, the payload offsets once (every line holds
// a head unless runs are long), the outputs once. 24 M cells in runs of two
// on average (8-byte offsets): 346 -> 122 us against the form before (4-byte
// flags, 8-byte slots and a 4-byte array of run starts, all in memory); k_emit
// takes 81 of them, at 5.7 TB/s.
constexpr int kChunkWords = 4 * kB;  // words per workgroup of k_head_sums / k_head_pref

__device__ __forceinline__ uint32_t low_bits(uint64_t m, uint32_t l) {  // set bits of m below l
  return (uint32_t)__popcll(m & ((1ull << l) - 1ull));
}

__global__ __launch_bounds__(kB) void k_heads(const int32_t* col, uint64_t nnz, uint64_t* words) {
  const uint32_t lane = lane_id();
  const uint64_t nw = (nnz + 63) >> 6;
  const uint64_t waves = gstride() / kWave;
  constexpr int kRounds = 4;  // words per wave and step, their loads in flight together
  for (uint64_t w0 = gtid() / kWave * kRounds; w0 < nw; w0 += waves * kRounds) {
    int32_t c[kRounds], p[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const uint64_t k = min(((w0 + r) << 6) + lane, nnz - 1);
      c[r] = gm(col)[k];
      p[r] = gm(col)[k ? k - 1 : 0];
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const uint64_t k = ((w0 + r) << 6) + lane;
      const uint64_t m = ballot(k < nnz && (k == 0 || c[r] != p[r]));
      if (lane == 0 && w0 + r < nw) gm(words)[w0 + r] = m;
    }
  }
}

// The starts of neighbouring rows fall into the same words: a wave ORs them
// together first, one atomic per word and wave, as the number of atomics
// bounds the kernel (1 M rows of 23 cells: 27.1 us with one atomic per row, now 6.9).
__global__ __launch_bounds__(kB) void k_row_heads(const void* rp, int ow, uint64_t n_rows,
                                                  uint64_t nnz, uint64_t* words) {
  const uint32_t lane = lane_id();
  for (uint64_t i0 = gtid() - lane; i0 < n_rows; i0 += gstride()) {  // whole waves
    const uint64_t i = min(i0 + lane, n_rows - 1);  // (the last row's bit again, past the end)
    const uint64_t a = min(ld_o(rp, i, ow), nnz), b = min(ld_o(rp, i + 1, ow), nnz);
    const uint32_t w = (uint32_t)(a >> 6);
    uint64_t m = a < b ? 1ull << (a & 63) : 0ull;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint64_t v = __shfl_down((unsigned long long)m, o, kWave);
      const uint32_t u = (uint32_t)__shfl_down((int)w, o, kWave);
      if (lane + o < kWave && u == w) m |= v;
    }
    const uint32_t prev = (uint32_t)__shfl_up((int)w, 1, kWave);
    if (m && (lane == 0 || prev != w))
      __hip_atomic_fetch_or(gm((unsigned long long*)words + w), m, __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The thread's four words of its chunk, and how many heads they hold.
__device__ __forceinline__ uint32_t chunk_words(const uint64_t* words, uint64_t nw, uint64_t (&x)[4]) {
  const uint64_t w0 = (uint64_t)blockIdx.x * kChunkWords + 4 * threadIdx.x;
  uint32_t c = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    x[j] = w0 + j < nw ? gm(words)[w0 + j] : 0ull;
    c += (uint32_t)__popcll(x[j]);
  }
  return c;
}

__global__ __launch_bounds__(kB) void k_head_sums(const uint64_t* words, uint64_t nw, uint32_t* sums) {
  __shared__ uint32_t red[kB / kWave];
  uint64_t x[4];
  uint32_t tot;
  block_excl_scan<kB / kWave>(chunk_words(words, nw, x), red, tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kB) void k_head_pref(const uint64_t* words, uint64_t nw,
                                                  const uint32_t* sums, uint32_t* pref,
                                                  const void* poff, int ow, uint64_t nnz,
                                                  void* o_poff, int64_t* d_m) {
  __shared__ uint32_t red[2][kB / kWave];
  uint64_t x[4];
  const uint32_t c = chunk_words(words, nw, x);
  uint32_t part = 0, base, tot;
  for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kB) part += sums[i];
  block_excl_scan<kB / kWave>(part, red[0], base);
  uint32_t ex = block_excl_scan<kB / kWave>(c, red[1], tot) + base;
  const uint64_t w0 = (uint64_t)blockIdx.x * kChunkWords + 4 * threadIdx.x;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (w0 + j <= nw) pref[w0 + j] = ex;  // pref[nw] = m
    ex += (uint32_t)__popcll(x[j]);
  }
  if (w0 <= nw && nw < w0 + 4) {  // the thread that wrote pref[nw] (words past nw are empty)
    st_o(o_poff, ex, ld_o(poff, nnz, ow), ow);
    if (d_m) *d_m = (int64_t)ex;
  }
}

// Heads before cell k (k <= nnz).
__device__ __forceinline__ uint32_t heads_before(const uint64_t* words, const uint32_t* pref, uint64_t k) {
  const uint32_t l = (uint32_t)k & 63u;
  return gm(pref)[k >> 6] + (l ? low_bits(gm(words)[k >> 6], l) : 0u);
}

// The cell of head number q < m, searched among the words from w on.
__device__ uint64_t head_cell(const uint64_t* words, const uint32_t* pref, uint64_t nw, uint64_t w,
                              uint32_t q) {
  uint64_t lo = w, hi = nw;  // pref[lo] <= q, the answer's word is in [lo, hi)
  while (hi - lo > 1) {
    const uint64_t mid = (lo + hi) >> 1;
    if (gm(pref)[mid] <= q) lo = mid;
    else hi = mid;
  }
  uint64_t m = gm(words)[lo];
  for (uint32_t j = q - gm(pref)[lo]; j; --j) m &= m - 1ull;
  return (lo << 6) + (uint32_t)__ffsll((unsigned long long)m) - 1u;
}

// The first `cell_blocks` workgroups take the cells, one word per wave round
// and kRounds words in flight; the others take the row offsets.
__global__ __launch_bounds__(kB) void k_emit(const int32_t* col, const void* poff, int ow,
                                             uint64_t nnz, const uint64_t* words,
                                             const uint32_t* pref, uint32_t cell_blocks,
                                             const void* rp, uint64_t n_rows, int32_t* o_col,
                                             void* o_poff, uint32_t* o_counts, void* o_rp) {
  if (blockIdx.x >= cell_blocks) {
    const uint64_t stride = (uint64_t)(gridDim.x - cell_blocks) * kB;
    for (uint64_t i = (uint64_t)(blockIdx.x - cell_blocks) * kB + threadIdx.x; i <= n_rows; i += stride)
      st_o(o_rp, i, heads_before(words, pref, min(ld_o(rp, i, ow), nnz)), ow);
    return;
  }
  const uint32_t lane = lane_id();
  const uint64_t nw = (nnz + 63) >> 6;
  constexpr int kRounds = 4;
  const uint64_t waves = (uint64_t)cell_blocks * (kB / kWave);
  for (uint64_t w0 = ((uint64_t)blockIdx.x * (kB / kWave) + threadIdx.x / kWave) * kRounds; w0 < nw;
       w0 += waves * kRounds) {
    uint64_t m[kRounds + 1];
    uint32_t p[kRounds];
#pragma unroll
    for (int r = 0; r <= kRounds; ++r) {  // (wave-uniform addresses)
      m[r] = w0 + r < nw ? gm(words)[w0 + r] : 0ull;
      if (r < kRounds) p[r] = gm(pref)[min(w0 + r, nw)];
    }
    int32_t c[kRounds];
    uint64_t o[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const uint64_t k = min(((w0 + r) << 6) + lane, nnz - 1);
      c[r] = 0;
      o[r] = 0;
      if ((m[r] >> lane) & 1ull) {
        c[r] = gm(col)[k];
        o[r] = ld_o(poff, k, ow);
      }
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      if (!((m[r] >> lane) & 1ull)) continue;
      const uint64_t k = ((w0 + r) << 6) + lane;
      const uint32_t q = p[r] + low_bits(m[r], lane);
      gm(o_col)[q] = c[r];
      st_o(o_poff, q, o[r], ow);
      if (o_counts) {
        // up to the next head: in this word, in the next one, or searched for
        const uint64_t above = (m[r] >> lane) >> 1;
        uint64_t next;
        if (above) next = k + (uint32_t)__ffsll((unsigned long long)above);
        else if (m[r + 1]) next = ((w0 + r + 1) << 6) + (uint32_t)__ffsll((unsigned long long)m[r + 1]) - 1u;
        else if (q + 1 < gm(pref)[nw]) next = head_cell(words, pref, nw, w0 + r, q + 1);
        else next = nnz;
        gm(o_counts)[q] = (uint32_t)(next - k);
      }
    }
  }
}

// Expansion: row offsets in values, and the status word (MGT_OK; a later
// kernel overwrites it on a cell that is not a whole number of values).
__global__ __launch_bounds__(kB) void k_expand_rows(const void* rp, const void* poff, int ow,
                                                    uint64_t n_rows, uint64_t nnz, uint32_t w,
                                                    void* o_rp, int32_t* d_status) {
  if (gtid() == 0 && d_status) *d_status = MGT_OK;
  for (uint64_t i = gtid(); i <= n_rows; i += gstride())
    st_o(o_rp, i, ld_o(poff, min(ld_o(rp, i, ow), nnz), ow) / w, ow);
}

// Whether an offset of the workgroup's share (nnz + 1 over the grid, rounded up)
// is not a whole number of values.
__device__ __forceinline__ bool share_bad(const void* poff, int ow, uint64_t nnz, uint32_t w) {
  bool bad = false;
  const uint64_t per = (nnz + gridDim.x) / gridDim.x;
  const uint64_t k1 = min(nnz + 1, (blockIdx.x + 1) * per);
  for (uint64_t k = blockIdx.x * per + threadIdx.x; k < k1; k += kB) {
    const uint64_t v = ld_o(poff, k, ow);
    bad |= (v >> 32) ? (v % w) != 0 : ((uint32_t)v % w) != 0;
  }
  return bad;
}

// The last cells of [0, hi) whose payload offsets are at most b0 and at most
// b1 >= b0 (cell 0 if none), found by the whole workgroup: each round probes kB
// evenly spaced cells for both, their loads in flight together.
__device__ __forceinline__ void coop_last_le(const void* poff, int ow, uint64_t hi, uint64_t b0,
                                             uint64_t b1, uint64_t& c0, uint64_t& c1) {
  uint64_t lo0 = 0, hi0 = hi, lo1 = 0, hi1 = hi;
  while (hi0 - lo0 > 1 || hi1 - lo1 > 1) {
    const uint64_t st0 = (hi0 - lo0 + kB - 1) / kB, st1 = (hi1 - lo1 + kB - 1) / kB;
    const uint64_t p0 = lo0 + (uint64_t)threadIdx.x * st0, p1 = lo1 + (uint64_t)threadIdx.x * st1;
    const uint64_t v0 = ld_o(poff, min(p0, hi - 1), ow), v1 = ld_o(poff, min(p1, hi - 1), ow);
    const int n0 = max(1, __syncthreads_count(p0 < hi0 && v0 <= b0));
    const int n1 = max(1, __syncthreads_count(p1 < hi1 && v1 <= b1));
    lo0 += (uint64_t)(n0 - 1) * st0;
    hi0 = min(lo0 + st0, hi0);
    lo1 += (uint64_t)(n1 - 1) * st1;
    hi1 = min(lo1 + st1, hi1);
  }
  c0 = lo0;
  c1 = max(lo0, lo1);
}

// One output cell per value, kExVals values per workgroup: the cell holding
// byte q * w is the last cell whose payload offset is at most q * w. The
// workgroup finds its first and last cell once, counts in LDS where the cells
// between them start, and scans the counts: the payload offsets are read once,
// in order, where a binary search per value read about 23 of them one after
// another. A range of more than kExCells cells (long runs of empty cells)
// is searched per value instead, so no input makes one workgroup walk it (600 K
// values in the first and the last of 300 K cells: 28.9 us by plain binary searches,
// 20.6 by way of samples in LDS).
// Bound by the latency of its steps (search, walk, scan, store), with 4 + ow
// bytes stored per value. 24 M values of 6 M cells, 8-byte offsets: 536 -> 122
// us against the binary search per value.
// Each workgroup also checks its share of the offsets (status only).
constexpr int kExVals = 2048;
constexpr uint64_t kExCells = 8 * kExVals;
constexpr int kExSamples = 1024;

__global__ __launch_bounds__(kB) void k_expand_cells(const int32_t* col, const void* poff, int ow,
                                                     uint64_t nnz, uint64_t nvals, uint32_t w,
                                                     int32_t* o_col, void* o_poff,
                                                     int32_t* d_status) {
  __shared__ uint32_t incl[kExVals], samples[kExSamples];
  __shared__ uint32_t red[kB / kWave];
  const bool bad = share_bad(poff, ow, nnz, w);
  for (uint64_t q0 = (uint64_t)blockIdx.x * kExVals; q0 < nvals; q0 += (uint64_t)gridDim.x * kExVals) {
    const uint32_t n = (uint32_t)min((uint64_t)kExVals, nvals - q0);
    const uint64_t b0 = q0 * w, b1 = (q0 + n) * w;
    uint64_t c0, c1;
    coop_last_le(poff, ow, nnz, b0, b1 - 1, c0, c1);
    const bool walk = c1 - c0 <= kExCells;  // block-uniform
    if (walk) {
      for (uint32_t i = threadIdx.x; i < (uint32_t)kExVals; i += kB) incl[i] = 0;
      __syncthreads();
      for (uint64_t k = c0 + 1 + threadIdx.x; k <= c1; k += kB) {
        const uint64_t o = ld_o(poff, k, ow);
        const uint64_t d = o > b0 ? o - b0 : 0;
        // (whole values: d is a multiple of w; clamped for offsets that are not in order)
        const uint64_t at = (d >> 32) ? d / w : (uint64_t)((uint32_t)d / w);
        atomicAdd(&incl[min(at, (uint64_t)kExVals - 1)], 1u);
      }
      __syncthreads();
      constexpr int kPer = kExVals / kB;
      const uint32_t p0 = threadIdx.x * kPer;
      uint32_t v[kPer], s = 0;
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        v[j] = incl[p0 + j];
        s += v[j];
      }
      uint32_t tot;
      uint32_t ex = block_excl_scan<kB / kWave>(s, red, tot);
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        ex += v[j];
        incl[p0 + j] = ex;
      }
      __syncthreads();
    }
    if (!walk) {
      // the starts of kExSamples evenly spaced cells of the range in LDS, in bytes
      // past b0: each value's place among them, then among the cells between two,
      // kSide values of a thread at a time (more take registers that the walk
      // misses). Values of 2^32 bytes and more per workgroup do without samples.
      const uint32_t last = (uint32_t)(c1 - c0), step = last / kExSamples + 1u;
      const bool fits = (uint64_t)n * w < ~0u;
      for (uint32_t i = threadIdx.x; i < (uint32_t)kExSamples; i += kB) {
        const uint64_t o = ld_o(poff, c0 + min((uint64_t)i * step, (uint64_t)last), ow);
        samples[i] = (uint32_t)min(o > b0 ? o - b0 : 0, (uint64_t)~0u);
      }
      __syncthreads();
      constexpr int kSide = 2;
      static_assert(kExVals % (kSide * kB) == 0, "whole rounds");
#pragma unroll 1
      for (uint32_t i0 = threadIdx.x; i0 < n; i0 += kSide * kB) {
        uint32_t f[kSide] = {};  // the last cell starting at or before the value (the first one does)
#pragma unroll 1
        for (uint32_t d = fits ? kExSamples / 2 : 0; d; d >>= 1) {
#pragma unroll
          for (int j = 0; j < kSide; ++j) f[j] += samples[f[j] + d] <= (i0 + j * kB) * w ? d : 0u;
        }
#pragma unroll
        for (int j = 0; j < kSide; ++j) f[j] = (uint32_t)min((uint64_t)f[j] * step, (uint64_t)last);
#pragma unroll 1
        for (uint32_t d = 1u << (31 - __clz((int)(fits ? step : last))); d; d >>= 1) {
#pragma unroll
          for (int j = 0; j < kSide; ++j) {
            const uint32_t k = (uint32_t)min((uint64_t)f[j] + d, (uint64_t)last);
            f[j] = ld_o(poff, c0 + k, ow) <= (q0 + i0 + j * kB) * w ? k : f[j];
          }
        }
#pragma unroll
        for (int j = 0; j < kSide; ++j) incl[i0 + j * kB] = f[j];
      }
      __syncthreads();
    }
    constexpr int kOut = kExVals / kB;  // values per thread, their columns in flight together
    int32_t c[kOut];
#pragma unroll
    for (int j = 0; j < kOut; ++j) {
      const uint32_t i = min((uint32_t)(j * kB) + threadIdx.x, n - 1);
      const uint64_t cell = min(c0 + incl[i], nnz - 1);
      c[j] = gm(col)[cell];
    }
#pragma unroll
    for (int j = 0; j < kOut; ++j) {
      const uint32_t i = (uint32_t)(j * kB) + threadIdx.x;
      if (i >= n) break;
      gm(o_col)[q0 + i] = c[j];
      if (o_poff) st_o(o_poff, q0 + i, (q0 + i) * w, ow);
    }
    __syncthreads();  // incl is reused
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && o_poff) st_o(o_poff, nvals, nvals * w, ow);
  if (bad && d_status) *d_status = MGT_ERANGE;
}

// The same with one value per thread, searched among all the cells, for calls of
// few values, alone (kExFew) or beside the cells: there the workgroups of k_expand_cells are
// too few to hide their steps. us per call, this and k_expand_cells: 300 K cells,
// a value in each 11.0 and 12.3, in every 8th 11.0 and 25.9; 1 M, each 18.2 and 16.6,
// every 2nd 14.8 and 16.4; 5 M, every 4th 42 and 33, every 6th 35 and 38, every 100th
// 16 and 32; 20 M, every 8th 97 and 85, every 12th 74 and 94.
constexpr uint64_t kExFew = 1 << 19;
inline bool expand_far(uint64_t nnz, uint64_t nvals) { return nvals <= kExFew + nnz / 12; }

__global__ __launch_bounds__(kB) void k_expand_far(const int32_t* col, const void* poff, int ow,
                                                   uint64_t nnz, uint64_t nvals, uint32_t w,
                                                   int32_t* o_col, void* o_poff, int32_t* d_status) {
  const bool bad = share_bad(poff, ow, nnz, w);
  for (uint64_t q = gtid(); q < nvals; q += gstride()) {
    const uint64_t b = q * w;
    uint64_t lo = 0, hi = nnz;
    while (hi - lo > 1) {
      const uint64_t mid = (lo + hi) >> 1;
      if (ld_o(poff, mid, ow) <= b) lo = mid;
      else hi = mid;
    }
    gm(o_col)[q] = gm(col)[lo];
    if (o_poff) st_o(o_poff, q, b, ow);
  }
  if (gtid() == 0 && o_poff) st_o(o_poff, nvals, nvals * w, ow);
  if (bad && d_status) *d_status = MGT_ERANGE;
}

inline dim3 grid_for(uint64_t n) {
  uint64_t g = (n + kB - 1) / kB;
  g = g < 1 ? 1 : (g > 16384 ? 16384 : g);
  return dim3((unsigned)g);
}

// Workspace layout: head bitmap (8 bytes per 64 cells), heads before each of
// its words (4 bytes per 64 cells), heads per chunk, scan scratch.
struct VlLayout {
  uint64_t o_words, o_pref, o_sums, o_scan, bytes;
};
inline uint64_t up256(uint64_t x) { return (x + 255) & ~(uint64_t)255; }
inline uint64_t head_chunks(uint64_t nnz) { return ((nnz + 63) / 64) / kChunkWords + 1; }
inline VlLayout vl_layout(uint64_t nnz) {
  const uint64_t nw = (nnz + 63) / 64;
  VlLayout y;
  y.o_words = 0;
  y.o_pref = up256(8 * nw);
  y.o_sums = y.o_pref + up256(4 * (nw + 1));
  y.o_scan = y.o_sums + up256(4 * head_chunks(nnz));
  y.bytes = y.o_scan + up256(scan_scratch_bytes(nnz + 1));
  return y;
}

}  // namespace vl
}  // namespace mgt

using namespace mgt;

#define MGT_VL_HIP(x)                              \
  do {                                             \
    if ((x) != hipSuccess) return MGT_EHIP;        \
  } while (0)

extern "C" {

int mgt_value_lists_workspace(int64_t nnz, size_t* workspace_bytes) {
  if (nnz < 0 || !workspace_bytes) return MGT_EINVAL;
  if ((uint64_t)nnz >= (1ull << 32)) return MGT_EUNSUPPORTED;
  *workspace_bytes = (size_t)vl::vl_layout((uint64_t)nnz).bytes;
  return MGT_OK;
}

int mgt_coalesce(int64_t n_rows, int64_t nnz, int32_t offset_width, const void* row_ptr,
                 const int32_t* col, const void* payload_off, void* o_row_ptr, int32_t* o_col,
                 void* o_payload_off, uint32_t* o_counts, int64_t* d_m, void* workspace,
                 size_t workspace_bytes, hipStream_t stream) {
  if (n_rows < 0 || nnz < 0 || (offset_width != 4 && offset_width != 8)) return MGT_EINVAL;
  if ((uint64_t)nnz >= (1ull << 32) || n_rows >= (1ll << 31)) return MGT_EUNSUPPORTED;
  if (!row_ptr || !payload_off || !o_row_ptr || !o_payload_off) return MGT_EINVAL;
  if (nnz > 0 && (!col || !o_col)) return MGT_EINVAL;
  if (!workspace || ((uintptr_t)workspace & 255u)) return MGT_EINVAL;
  const uint64_t n = (uint64_t)nnz, r = (uint64_t)n_rows;
  const vl::VlLayout y = vl::vl_layout(n);
  if (workspace_bytes < y.bytes) return MGT_ENOMEM;
  uint8_t* W = (uint8_t*)workspace;
  uint64_t* words = (uint64_t*)(W + y.o_words);
  uint32_t* pref = (uint32_t*)(W + y.o_pref);
  uint32_t* sums = (uint32_t*)(W + y.o_sums);
  const int ow = offset_width;
  const uint64_t nw = (n + 63) / 64;
  const dim3 block(vl::kB);
  if (n) {
    hipLaunchKernelGGL(vl::k_heads, vl::grid_for((nw + 3) / 4 * kWave), block, 0, stream, col, n, words);
    if (r)
      hipLaunchKernelGGL(vl::k_row_heads, vl::grid_for(r), block, 0, stream, row_ptr, ow, r, n, words);
  }
  // (the last chunk also holds the slot past the last word)
  const dim3 chunks((unsigned)vl::head_chunks(n));
  if (chunks.x > 1)
    hipLaunchKernelGGL(vl::k_head_sums, chunks, block, 0, stream, words, nw, sums);
  hipLaunchKernelGGL(vl::k_head_pref, chunks, block, 0, stream, words, nw, sums, pref, payload_off, ow,
                     n, o_payload_off, d_m);
  const uint32_t cells = n ? vl::grid_for((nw + 3) / 4 * kWave).x : 0;
  const uint32_t rows = vl::grid_for(r + 1).x;
  hipLaunchKernelGGL(vl::k_emit, dim3(cells + rows), block, 0, stream, col, payload_off, ow, n, words,
                     pref, cells, row_ptr, r, o_col, o_payload_off, o_counts, o_row_ptr);
  MGT_VL_HIP(hipGetLastError());
  return MGT_OK;
}

int mgt_expand(int64_t n_rows, int64_t nnz, int64_t payload_bytes, int32_t offset_width,
               int32_t value_bytes, const void* row_ptr, const int32_t* col,
               const void* payload_off, void* o_row_ptr, int32_t* o_col, void* o_payload_off,
               int32_t* d_status, hipStream_t stream) {
  if (n_rows < 0 || nnz < 0 || payload_bytes < 0 || value_bytes <= 0) return MGT_EINVAL;
  if (offset_width != 4 && offset_width != 8) return MGT_EINVAL;
  if (payload_bytes % value_bytes) return MGT_EINVAL;
  const uint64_t nvals = (uint64_t)(payload_bytes / value_bytes);
  if (nvals >= (1ull << 32) || (uint64_t)nnz >= (1ull << 32) || n_rows >= (1ll << 31))
    return MGT_EUNSUPPORTED;
  if (offset_width == 4 && payload_bytes >= (1ll << 31)) return MGT_EUNSUPPORTED;
  if (!row_ptr || !payload_off || !o_row_ptr) return MGT_EINVAL;
  if (nnz > 0 && !col) return MGT_EINVAL;
  if (nvals > 0 && (!o_col || nnz == 0)) return MGT_EINVAL;
  const uint64_t n = (uint64_t)nnz, r = (uint64_t)n_rows;
  const uint32_t w = (uint32_t)value_bytes;
  const int ow = offset_width;
  hipLaunchKernelGGL(vl::k_expand_rows, vl::grid_for(r + 1), dim3(vl::kB), 0, stream, row_ptr,
                     payload_off, ow, r, n, w, o_row_ptr, d_status);
  // at least one workgroup (for the status), and enough to check the offsets side by side
  const bool far = vl::expand_far(n, nvals);
  const uint64_t vals = far ? vl::kB : vl::kExVals;
  const uint64_t blocks = std::max<uint64_t>((nvals + vals - 1) / vals,
                                             (n + 1 + 8 * vl::kB - 1) / (8 * vl::kB));
  const dim3 grid((unsigned)std::min<uint64_t>(blocks, 1u << 20));
  if (far)
    hipLaunchKernelGGL(vl::k_expand_far, grid, dim3(vl::kB), 0, stream, col, payload_off, ow, n, nvals, w,
                       o_col, o_payload_off, d_status);
  else
    hipLaunchKernelGGL(vl::k_expand_cells, grid, dim3(vl::kB), 0, stream, col, payload_off, ow, n, nvals, w,
                       o_col, o_payload_off, d_status);
  MGT_VL_HIP(hipGetLastError());
  return MGT_OK;
}

int mgt_counts_to_offsets(int64_t nnz, const uint32_t* counts, int32_t value_bytes,
                          int32_t offset_width, void* payload_off, void* workspace,
                          size_t workspace_bytes, hipStream_t stream) {
  if (nnz < 0 || value_bytes <= 0 || (offset_width != 4 && offset_width != 8)) return MGT_EINVAL;
  if ((uint64_t)nnz >= (1ull << 32)) return MGT_EUNSUPPORTED;
  if (!payload_off || (nnz > 0 && !counts)) return MGT_EINVAL;
  if (!workspace || ((uintptr_t)workspace & 255u)) return MGT_EINVAL;
  const uint64_t n = (uint64_t)nnz;
  const vl::VlLayout y = vl::vl_layout(n);
  if (workspace_bytes < y.bytes) return MGT_ENOMEM;
  uint8_t* W = (uint8_t*)workspace;
  MGT_VL_HIP(launch_scan_offsets(counts, n, (uint32_t)value_bytes, offset_width, payload_off,
                                 (uint64_t*)(W + y.o_scan), stream));
  return MGT_OK;
}

}  // extern "C"
