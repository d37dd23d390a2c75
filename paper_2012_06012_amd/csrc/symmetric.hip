// Unordered multigraphs stored as one triangle (Section 2: an unordered edge
// gives M_ij = M_ji = e, so the symmetric matrix is kept as its lower or upper
// triangle). mgt_symmetrize builds the full symmetric matrix S: every stored
// off-diagonal cell (i, j, e) appears as (i, j, e) and as (j, i, e), a stored
// diagonal cell once. The mirrored cells of row i are row i of the stored
// triangle's transpose T (which the caller's plan computes first) without its
// diagonal cells; row i of S is the stored row then the mirrored cells (lower
// storage), or the mirrored cells then the stored row (upper storage).
//
// Stages: k_sym_count (cells and payload bytes of every row of S) -> exclusive
// scans -> k_sym_fill (a workgroup per 2,048 cells of S: column ids, payload
// offsets, payload bytes; others write the row offsets and the tail: end
// offsets, sizes, status).
// Offsets are clamped into their arrays before they index anything, so
// invalid inputs cannot make these kernels access memory out of bounds.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/mgt.h"
#include "kernels.h"
#include "payload.h"
#include "prims.h"

namespace mgt {
namespace sym {

constexpr int kB = 256;

__device__ __forceinline__ uint64_t ld_o(const void* p, uint64_t i, int ow) {
  const int64_t v = ow == 4 ? (int64_t)gm((const int32_t*)p)[i] : gm((const int64_t*)p)[i];
  return v < 0 ? 0u : (uint64_t)v;
}
__device__ __forceinline__ void st_o(void* p, uint64_t i, uint64_t v, int ow) {
  if (ow == 4) gm((int32_t*)p)[i] = (int32_t)v;
  else gm((int64_t*)p)[i] = (int64_t)v;
}

// The mirrored range [m0, m1) of row i of T: its cells minus the diagonal ones,
// which lead the row for lower storage (T's row i holds source rows >= i in
// ascending order) and close it for upper storage (source rows <= i).
struct Range {
  uint64_t m0, m1;
};
__device__ __forceinline__ Range mirrored(const SymArgs& a, uint64_t i) {
  uint64_t q0 = min(ld_o(a.t_row_ptr, i, a.ow), a.nnz);
  uint64_t q1 = min(ld_o(a.t_row_ptr, i + 1, a.ow), a.nnz);
  q1 = max(q0, q1);
  if (a.lower)
    while (q0 < q1 && (uint64_t)gm(a.t_col)[q0] == i) ++q0;
  else
    while (q1 > q0 && (uint64_t)gm(a.t_col)[q1 - 1] == i) --q1;
  return Range{q0, q1};
}

__device__ __forceinline__ void flag(int32_t* st, int32_t code) {
  atomicCAS(st, (int32_t)MGT_OK, code);
}

// Cells and payload bytes of every row of S (one thread per row).
__global__ __launch_bounds__(kB) void k_sym_count(SymArgs a) {
  if (*(volatile int32_t*)a.st != MGT_OK) return;
  for (uint64_t i = (uint64_t)blockIdx.x * kB + threadIdx.x; i < a.n; i += (uint64_t)gridDim.x * kB) {
    const uint64_t rs = min(ld_o(a.row_ptr, i, a.ow), a.nnz);
    const uint64_t re = max(rs, min(ld_o(a.row_ptr, i + 1, a.ow), a.nnz));
    const Range m = mirrored(a, i);
    const uint64_t s1 = min(ld_o(a.poff, re, a.ow), a.pbytes);
    const uint64_t bs = s1 - min(min(ld_o(a.poff, rs, a.ow), a.pbytes), s1);
    const uint64_t t1 = min(ld_o(a.t_poff, m.m1, a.ow), a.pbytes);
    const uint64_t bm = t1 - min(min(ld_o(a.t_poff, m.m0, a.ow), a.pbytes), t1);
    const uint64_t cells = (re - rs) + (m.m1 - m.m0), bytes = bs + bm;
    if (bytes >> 32) flag(a.st, MGT_EUNSUPPORTED);
    gm(a.cnt)[i] = (uint32_t)cells;
    gm(a.byt)[i] = (uint32_t)bytes;
    if (a.validate)
      for (uint64_t k = rs; k < re; ++k) {
        const int64_t c = gm(a.col)[k];
        if (a.lower ? c > (int64_t)i : c < (int64_t)i) flag(a.st, MGT_ERANGE);
      }
  }
}

// S by output cells, kFillCells per workgroup, whatever the rows' lengths: the
// workgroup finds the row of its first cell, counts in LDS where the rows after
// it start and scans the counts. A workgroup walks about kFillRows rows at most:
// where more lie between two of its cells (a long stretch of empty ones), it
// searches the cells' rows instead (2^24 vertices, edges among 8,000 of them: 97
// ms for the call with one workgroup walking the rest, now 55, of which the
// transpose takes 49). Cell j of row i comes from the stored row or
// from T's row, both read in order, so every access runs along its array; a
// wave's 64 payloads are one run of output bytes and go out through LDS.
// Bound by the loads of the rows' fields (about ten per cell, nearly all from
// the L1). One wave per row, each lane copying its cell, took 272 us on 4 M
// cells of 8 bytes on average in rows of 32 (8 M cells of S); this takes 134.
constexpr int kFillCells = 2048;
constexpr int kFillPer = kFillCells / kB;
constexpr uint64_t kFillRows = 8 * kFillCells;

__global__ __launch_bounds__(kB) void k_sym_fill(SymArgs a, uint32_t cell_blocks) {
  __shared__ uint32_t incl[kFillCells];
  __shared__ alignas(16) uint8_t stage[kB / kWave][kStage];
  __shared__ uint32_t red[kB / kWave];
  const int32_t st = *(volatile int32_t*)a.st;
  const uint32_t w = threadIdx.x / kWave;
  if (blockIdx.x >= cell_blocks) {  // the row offsets, and the tail
    const uint64_t stride = (uint64_t)(gridDim.x - cell_blocks) * kB;
    const uint64_t i0 = (uint64_t)(blockIdx.x - cell_blocks) * kB + threadIdx.x;
    if (i0 == 0 && a.d_status) *a.d_status = st;
    if (st != MGT_OK) return;
    const uint64_t cells = a.n ? min(a.ocnt[a.n], a.cap_cells) : 0;
    for (uint64_t i = i0; i < a.n; i += stride) st_o(a.s_row_ptr, i, a.ocnt[i], a.ow);
    if (i0 == 0) {
      const uint64_t bytes = a.n ? min(a.obyt[a.n], a.cap_bytes) : 0;
      st_o(a.s_row_ptr, a.n, cells, a.ow);
      st_o(a.s_poff, cells, bytes, a.ow);
      if (a.d_sizes) {
        a.d_sizes[0] = (int64_t)cells;
        a.d_sizes[1] = (int64_t)bytes;
      }
    }
    return;
  }
  if (st != MGT_OK) return;
  const uint64_t total = min(a.ocnt[a.n], a.cap_cells);
  const uint64_t q0 = (uint64_t)blockIdx.x * kFillCells;
  if (q0 >= total) return;
  const uint32_t m = (uint32_t)min((uint64_t)kFillCells, total - q0);
  for (uint32_t i = threadIdx.x; i < (uint32_t)kFillCells; i += kB) incl[i] = 0;
  uint64_t lo = 0, hi = a.n;  // the last row starting at or before q0
  while (hi - lo > 1) {
    const uint64_t step = (hi - lo + kB - 1) / kB;
    const uint64_t p = lo + (uint64_t)threadIdx.x * step;
    const int c = max(1, __syncthreads_count(p < hi && a.ocnt[min(p, a.n)] <= q0));
    lo += (uint64_t)(c - 1) * step;
    hi = min(lo + step, hi);
  }
  const uint64_t r0 = lo;
  __syncthreads();
  bool more = true;
  for (uint64_t base = r0 + 1; more; base += kB) {
    const uint64_t r = base + threadIdx.x;
    bool stop = r >= a.n;
    if (!stop) {
      const uint64_t v = a.ocnt[r];
      if (v >= q0 && v < q0 + m) atomicAdd(&incl[v - q0], 1u);
      stop = v >= q0 + m;
    }
    more = !__syncthreads_or(stop);
    if (more && base > r0 + kFillRows) {  // (block-uniform)
      // the last row starting at or before each cell, and what it is past the
      // one of the cell before
#pragma unroll 1
      for (uint32_t i = threadIdx.x; i < m; i += kB) {
        uint64_t row[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const uint64_t q = q0 + (i > (uint32_t)e ? i - e : 0u);
          uint64_t first = r0, end = a.n;
          while (end - first > 1) {
            const uint64_t mid = (first + end) >> 1;
            if (a.ocnt[mid] <= q) first = mid;
            else end = mid;
          }
          row[e] = first;
        }
        incl[i] = (uint32_t)(i ? row[0] - row[1] : row[0] - r0);
      }
      __syncthreads();
      more = false;
    }
  }
  {
    const uint32_t p0 = threadIdx.x * kFillPer;
    uint32_t v[kFillPer], s = 0, tot;
#pragma unroll
    for (int j = 0; j < kFillPer; ++j) {
      v[j] = incl[p0 + j];
      s += v[j];
    }
    uint32_t ex = block_excl_scan<kB / kWave>(s, red, tot);
#pragma unroll
    for (int j = 0; j < kFillPer; ++j) {
      ex += v[j];
      incl[p0 + j] = ex;
    }
  }
  __syncthreads();
  constexpr int kPay = 2;  // cells per lane whose fields and payloads are in flight together (4: no faster)
  const uint64_t top = a.nnz;  // (> 0: S has a cell)
#pragma unroll 1
  for (int g = 0; g < kFillPer; g += kPay) {
    uint64_t ob[kPay];
    uint32_t z[kPay];
    int32_t col[kPay];
    const uint8_t *src[kPay], *from[kPay];
    v4 va[kPay], vb[kPay];
    bool ok = true;
#pragma unroll
    for (int e = 0; e < kPay; ++e) {
      const uint32_t p = (uint32_t)(g + e) * kB + threadIdx.x;
      const bool act = p < m;
      const uint64_t i = r0 + incl[act ? p : 0u], q = q0 + (act ? p : 0u);
      const uint64_t c0 = a.ocnt[i], c1 = a.ocnt[i + 1], b0 = a.obyt[i];
      const uint64_t rs = min(ld_o(a.row_ptr, i, a.ow), top);
      const uint64_t re = max(rs, min(ld_o(a.row_ptr, i + 1, a.ow), top));
      const uint64_t ns = re - rs, nm = c1 - c0 - ns, j = q - c0;
      // T's row without its diagonal cells: they lead it for lower storage
      const uint64_t t0 = a.lower ? ld_o(a.t_row_ptr, i + 1, a.ow) - nm : ld_o(a.t_row_ptr, i, a.ow);
      const uint64_t m0 = min(t0, top);
      const bool mir = a.lower ? j >= ns : j < nm;
      const uint64_t first = mir ? m0 : rs;
      const uint64_t k = min(first + (a.lower ? (mir ? j - ns : j) : (mir ? j : j - nm)), top - 1);
      const void* const po = mir ? a.t_poff : a.poff;
      const uint64_t o = min(ld_o(po, k, a.ow), a.pbytes);
      const uint64_t o1 = max(o, min(ld_o(po, k + 1, a.ow), a.pbytes));
      const uint64_t of = min(ld_o(po, first, a.ow), o);
      // bytes of the part that comes first in the row, for cells of the second
      uint64_t before = 0;
      if (a.lower ? mir : !mir) {
        const void* const pf = a.lower ? a.poff : a.t_poff;
        const uint64_t f0 = a.lower ? rs : m0, f1 = a.lower ? re : min(m0 + nm, top);
        const uint64_t x = ld_o(pf, f0, a.ow), y = ld_o(pf, f1, a.ow);
        before = y > x ? y - x : 0;
      }
      ob[e] = b0 + before + (o - of);
      z[e] = act ? (uint32_t)(o1 - o) : 0u;
      // (only offsets that decrease, in unvalidated inputs, can pass the end)
      if (ob[e] > a.cap_bytes || z[e] > a.cap_bytes - ob[e]) z[e] = 0;
      col[e] = gm(mir ? a.t_col : a.col)[k];
      from[e] = mir ? a.t_payload : a.payload;
      src[e] = from[e] + o;
      ok &= z[e] <= 32u;
    }
#pragma unroll
    for (int e = 0; e < kPay; ++e) {
      va[e] = v4{0u, 0u, 0u, 0u};
      vb[e] = v4{0u, 0u, 0u, 0u};
      if (z[e] && z[e] <= 32u) get_bytes(src[e], from[e], from[e] + a.pbytes, z[e], va[e], vb[e]);
    }
#pragma unroll
    for (int e = 0; e < kPay; ++e) {
      const uint32_t p = (uint32_t)(g + e) * kB + threadIdx.x;
      if (p < m) {
        gm(a.s_col)[q0 + p] = col[e];
        st_o(a.s_poff, q0 + p, ob[e], a.ow);
      }
      const uint64_t act = ballot(p < m);  // a prefix of the lanes
      if (act == 0) continue;              // wave-uniform
      // the wave's run of output bytes, if its cells lie in it as they should
      const uint64_t base = wave_bcast(ob[e], 0);
      const uint64_t end = wave_bcast(ob[e] + z[e], 63 - (int)__clzll(act));
      const uint64_t rel = ob[e] - base;
      if (__all(ok && (p >= m || (ob[e] >= base && rel + z[e] <= end - base))) && end - base <= 2048u) {
        write_run(stage[w], a.s_payload + base, (uint32_t)rel, (uint32_t)(end - base), va[e], vb[e], z[e]);
      } else if (z[e]) {
        if (z[e] <= 32u) put_global(a.s_payload + ob[e], va[e], vb[e], z[e]);
        else copy_long(a.s_payload + ob[e], src[e], z[e]);
      }
    }
  }
}

}  // namespace sym

hipError_t launch_symmetrize(const SymArgs& a, hipStream_t s) {
  const uint64_t n = a.n;
  if (n) {
    const uint64_t g = std::min<uint64_t>((n + sym::kB - 1) / sym::kB, 65536);
    hipLaunchKernelGGL(sym::k_sym_count, dim3((unsigned)g), dim3(sym::kB), 0, s, a);
    hipError_t e = launch_scan(a.cnt, a.ocnt, a.byt, a.obyt, nullptr, n, a.scan, s);
    if (e != hipSuccess) return e;
  }
  // (S holds at most 2 nnz cells; workgroups past its end leave at once)
  const uint64_t cells = n ? (2 * a.nnz + sym::kFillCells - 1) / sym::kFillCells : 0;
  const uint64_t rows = std::min<uint64_t>(n / sym::kB + 1, 4096);
  hipLaunchKernelGGL(sym::k_sym_fill, dim3((unsigned)(cells + rows)), dim3(sym::kB), 0, s, a,
                     (uint32_t)cells);
  return hipGetLastError();
}

}  // namespace mgt
