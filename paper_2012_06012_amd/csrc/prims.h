// Wave64 / workgroup primitives for gfx950 (CDNA4): lane masks, DPP and
// shuffle scans, workgroup scans, and the ballot multisplit used to rank
// equal digits stably without atomics.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mgt {

constexpr int kWave = 64;

__device__ __forceinline__ uint32_t lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Number of set bits of m in lanes below the calling lane (v_mbcnt).
__device__ __forceinline__ uint32_t popc_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

// Inclusive wave scan of a 32-bit value with DPP: Hillis-Steele inside each
// 16-lane row (row_shr 1, 2, 4, 8, zero-filled at the row edge), then
// row_bcast15 / row_bcast31 carry the row totals into the rows above.
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// Inclusive wave scan of a 64-bit value: the same DPP steps on both words.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, kCtrl, kRows, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), kCtrl, kRows, 0xf, false);
  return (uint64_t)lo | ((uint64_t)hi << 32);
}
__device__ __forceinline__ uint64_t wave_incl_scan_u64(uint64_t v) {
  v += dpp_u64<0x111, 0xf>(v);  // row_shr:1
  v += dpp_u64<0x112, 0xf>(v);  // row_shr:2
  v += dpp_u64<0x114, 0xf>(v);  // row_shr:4
  v += dpp_u64<0x118, 0xf>(v);  // row_shr:8
  v += dpp_u64<0x142, 0xa>(v);  // row_bcast:15
  v += dpp_u64<0x143, 0xc>(v);  // row_bcast:31
  return v;
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) { return wave_incl_scan_u32(v); }
__device__ __forceinline__ uint64_t wave_incl_scan(uint64_t v) { return wave_incl_scan_u64(v); }

template <class T>
__device__ __forceinline__ T wave_bcast(T v, int lane) { return __shfl(v, lane, kWave); }

// Exclusive scan over a workgroup of NW waves. `scratch` holds at least NW
// values. Every thread of the workgroup must call it. Returns the exclusive
// prefix; `total` receives the workgroup total. Every thread adds up the wave
// totals itself (broadcast LDS reads in flight together): no serial pass by
// one thread and a barrier less.
template <int NW, class T>
__device__ __forceinline__ T block_excl_scan(T v, T* scratch, T& total) {
  const T inc = wave_incl_scan(v);
  const int w = threadIdx.x / kWave;
  if (lane_id() == kWave - 1) scratch[w] = inc;
  __syncthreads();
  T before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const T t = scratch[i];
    if (i < w) before += t;
    all += t;
  }
  total = all;
  __syncthreads();
  return inc - v + before;
}

// Two such scans sharing their barriers. `scratch` holds at least 2 NW values.
template <int NW, class T, class U>
__device__ __forceinline__ void block_excl_scan2(T& v, U& u, uint64_t* scratch, T& vtotal, U& utotal) {
  const T vi = wave_incl_scan(v);
  const U ui = wave_incl_scan(u);
  const int w = threadIdx.x / kWave;
  if (lane_id() == kWave - 1) {
    scratch[2 * w] = vi;
    scratch[2 * w + 1] = ui;
  }
  __syncthreads();
  T vb = 0, va = 0;
  U ub = 0, ua = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const T t = (T)scratch[2 * i];
    const U x = (U)scratch[2 * i + 1];
    if (i < w) {
      vb += t;
      ub += x;
    }
    va += t;
    ua += x;
  }
  vtotal = va;
  utotal = ua;
  v = vi - v + vb;
  u = ui - u + ub;
  __syncthreads();
}

// Lanes of the wave whose `digit` equals the calling lane's digit, among the
// lanes where `active` holds. `dbits` (wave-uniform) bounds the digit width.
// A bit costs five vector instructions: the bit as a full mask, its ballot, and
// one three-input logic operation per half.
__device__ __forceinline__ uint64_t match_peers(uint32_t digit, bool active, int dbits) {
  const uint64_t act = ballot(active);
  uint32_t lo = (uint32_t)act, hi = (uint32_t)(act >> 32);
  for (int b = 0; b < dbits; ++b) {
    const uint32_t s = (uint32_t)((int32_t)(digit << (31 - b)) >> 31);
    const uint64_t v = ballot(s != 0u);
    lo &= ~((uint32_t)v ^ s);
    hi &= ~((uint32_t)(v >> 32) ^ s);
  }
  return (uint64_t)lo | ((uint64_t)hi << 32);
}

// Stable ranks of a wave's N rounds of 64 cells among the cells of their digit
// in the same wave, in cell order (cell r * 64 + lane of the wave; the first
// `n` of them are there, the others get rank 0). wc: one 16-bit counter per
// (digit, wave), zero before and the wave's counts after; at[r] is the index of
// cell r's counter, and the counters of waves 2v and 2v + 1 share an aligned
// word. The matches of all rounds advance bit by bit together. The counters
// are read by every lane and added to by each digit's first lane, round by
// round: a wave's LDS operations execute in order, so the rounds need no wait
// between them.
template <int N>
__device__ __forceinline__ void wave_ranks(uint16_t* wc, const uint32_t (&at)[N], const uint32_t (&digit)[N],
                                           uint32_t n, int dbits, uint32_t (&rank)[N]) {
  const uint32_t lane = lane_id();
  uint32_t lo[N], hi[N];
#pragma unroll
  for (int r = 0; r < N; ++r) {
    const uint64_t act = ballot((uint32_t)r * kWave + lane < n);
    lo[r] = (uint32_t)act;
    hi[r] = (uint32_t)(act >> 32);
  }
  for (int b = 0; b < dbits; ++b) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const uint32_t s = (uint32_t)((int32_t)(digit[r] << (31 - b)) >> 31);
      const uint64_t v = ballot(s != 0u);
      lo[r] &= ~((uint32_t)v ^ s);
      hi[r] &= ~((uint32_t)(v >> 32) ^ s);
    }
  }
#pragma unroll
  for (int r = 0; r < N; ++r) {
    rank[r] = 0;
    if ((uint32_t)r * kWave + lane < n) {
      const uint32_t below = __builtin_amdgcn_mbcnt_hi(hi[r], __builtin_amdgcn_mbcnt_lo(lo[r], 0u));
      const uint32_t old = wc[at[r]];
      if (below == 0)
        __hip_atomic_fetch_add((uint32_t*)wc + (at[r] >> 1),
                               (uint32_t)(__popc(lo[r]) + __popc(hi[r])) << (16u * (at[r] & 1u)),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      rank[r] = old + below;
    }
  }
}

// XCD-aware tile order: the hardware deals workgroups round robin over the 8
// XCDs, so this gives each XCD a contiguous run of tiles (neighbouring tiles
// then share that XCD's L2). `g8` is the grid size, a multiple of 8.
__device__ __forceinline__ uint64_t xcd_tile(uint64_t b, uint64_t g8) {
  return (b & 7u) * (g8 >> 3) + (b >> 3);
}

// Global-memory (address space 1) views of generic pointers. Accesses through
// them compile to global_* instructions, which only the vector-memory counter
// tracks; flat_* accesses are tracked by the LDS counter as well, so every
// wait for an LDS result would also wait for all outstanding HBM traffic.
#define GMEM __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ GMEM T* gm(T* p) { return (GMEM T*)p; }
template <typename T>
__device__ __forceinline__ const GMEM T* gm(const T* p) { return (const GMEM T*)p; }

}  // namespace mgt
