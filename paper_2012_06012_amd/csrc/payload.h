// Payload bytes of any size and alignment: cells of up to 32 bytes through
// registers, runs of a wave's cells through LDS. gfx950 takes unaligned global
// and LDS accesses of up to 16 bytes, so no byte is shifted into place: a cell
// is two 16-byte loads, and is stored in at most six exact pieces.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "prims.h"

namespace mgt {

typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32u __attribute__((aligned(1)));
typedef uint16_t u16u __attribute__((aligned(1)));
typedef uint32_t v4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kStage = 2048 + 16;  // LDS bytes of a wave's run: 64 cells of up to 32 bytes

// Writes the z <= 32 low bytes of (a, b), in at most six pieces (kDwords: z is a
// multiple of 4, at most four).
template <bool kDwords, class P4, class P2, class P1, class PH, class PB>
__device__ __forceinline__ void put_pieces(P4 p4, P2 p2, P1 p1, PH ph, PB pb, const v4& a, const v4& b,
                                           uint32_t z) {
  if (z >= 16u) p4(0u, a);
  if (z >= 32u) p4(16u, b);
  const uint32_t o1 = z & 16u;
  const v4 u = o1 ? b : a;
  if (z & 8u) p2(o1, u.x, u.y);
  const uint32_t o2 = z & 24u;
  const uint32_t s0 = (z & 8u) ? u.z : u.x, s1 = (z & 8u) ? u.w : u.y;
  if (z & 4u) p1(o2, s0);
  if constexpr (kDwords) return;
  const uint32_t o3 = z & 28u;
  const uint32_t s = (z & 4u) ? s1 : s0;
  if (z & 2u) ph(o3, (uint16_t)s);
  if (z & 1u) pb(z & 30u, (uint8_t)((z & 2u) ? s >> 16 : s));
}
__device__ __forceinline__ void put_lds(uint8_t* d, const v4& a, const v4& b, uint32_t z) {
  put_pieces<false>([&](uint32_t o, const v4& x) { *(u32x4u*)(d + o) = u32x4u{x.x, x.y, x.z, x.w}; },
             [&](uint32_t o, uint32_t x, uint32_t y) { *(u32x2u*)(d + o) = u32x2u{x, y}; },
             [&](uint32_t o, uint32_t x) { *(u32u*)(d + o) = x; },
             [&](uint32_t o, uint16_t x) { *(u16u*)(d + o) = x; },
             [&](uint32_t o, uint8_t x) { d[o] = x; }, a, b, z);
}
template <bool kDwords = false>
__device__ __forceinline__ void put_global(uint8_t* dst, const v4& a, const v4& b, uint32_t z) {
  GMEM uint8_t* const d = gm(dst);
  put_pieces<kDwords>([&](uint32_t o, const v4& x) { *(GMEM u32x4u*)(d + o) = u32x4u{x.x, x.y, x.z, x.w}; },
             [&](uint32_t o, uint32_t x, uint32_t y) { *(GMEM u32x2u*)(d + o) = u32x2u{x, y}; },
             [&](uint32_t o, uint32_t x) { *(GMEM u32u*)(d + o) = x; },
             [&](uint32_t o, uint16_t x) { *(GMEM u16u*)(d + o) = x; },
             [&](uint32_t o, uint8_t x) { d[o] = x; }, a, b, z);
}
// The z <= 32 bytes at src (any alignment) as two 16-byte values (what follows
// them is not cleared), from an array at [begin, end), no byte outside it: whole
// 16-byte loads where 32 bytes follow; at the array's end its last 32 bytes,
// shifted down; in an array shorter than that, byte by byte.
__device__ __forceinline__ void get_bytes(const uint8_t* src, const uint8_t* begin, const uint8_t* end,
                                          uint32_t z, v4& a, v4& b) {
  const GMEM uint8_t* const s = gm(src);
  if (src + 32 <= end) {
    const u32x4u x = *(const GMEM u32x4u*)s;
    a = v4{x.x, x.y, x.z, x.w};
    if (z > 16u) {
      const u32x4u y = *(const GMEM u32x4u*)(s + 16);
      b = v4{y.x, y.y, y.z, y.w};
    }
  } else if (end - begin >= 32) {
    const GMEM uint8_t* const e = gm(end - 32);
    const u32x4u x = *(const GMEM u32x4u*)e, y = *(const GMEM u32x4u*)(e + 16);
    const uint32_t by = (uint32_t)(src - (end - 32));  // 1..31
    uint32_t w[9] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w, 0u};
#pragma unroll
    for (int step = 4; step >= 1; step >>= 1)
#pragma unroll
      for (int j = 0; j < 8; ++j) w[j] = (by & (4u * step)) ? (j + step < 8 ? w[j + step] : 0u) : w[j];
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = __builtin_amdgcn_alignbyte(w[j + 1], w[j], by & 3u);
    a = v4{w[0], w[1], w[2], w[3]};
    b = v4{w[4], w[5], w[6], w[7]};
  } else {
    a = v4{0u, 0u, 0u, 0u};
    b = a;
#pragma unroll 1
    for (uint32_t j = 0; j < 8; ++j) {
      uint32_t v = 0;
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i)
        if (4 * j + i < z) v |= (uint32_t)s[4 * j + i] << (8 * i);
      a.x = j == 0 ? v : a.x;
      a.y = j == 1 ? v : a.y;
      a.z = j == 2 ? v : a.z;
      a.w = j == 3 ? v : a.w;
      b.x = j == 4 ? v : b.x;
      b.y = j == 5 ? v : b.y;
      b.z = j == 6 ? v : b.z;
      b.w = j == 7 ? v : b.w;
    }
  }
}
// A payload of over 32 bytes, by one lane.
__device__ __forceinline__ void copy_long(uint8_t* dst, const uint8_t* src, uint32_t z) {
  const GMEM uint8_t* s = gm(src);
  GMEM uint8_t* d = gm(dst);
  for (; z >= 64u; z -= 64u, s += 64, d += 64) {
    u32x4u v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = ((const GMEM u32x4u*)s)[j];
#pragma unroll
    for (int j = 0; j < 4; ++j) ((GMEM u32x4u*)d)[j] = v[j];
  }
  for (; z >= 16u; z -= 16u, s += 16, d += 16) *(GMEM u32x4u*)d = *(const GMEM u32x4u*)s;
  for (uint32_t j = 0; j < z; ++j) d[j] = s[j];
}

// A wave's payloads are one run of tot <= 2,048 output bytes at dst, each lane's
// z <= 32 bytes at rel: packed in LDS (16-byte aligned), then written 16 bytes
// per lane. Called by whole waves.
__device__ __forceinline__ void write_run(uint8_t* stage, uint8_t* dst, uint32_t rel, uint32_t tot,
                                          const v4& a, const v4& b, uint32_t z) {
  if (__all(((rel | z) & 3u) == 0u)) {
    // whole dwords, one by one: unaligned wide LDS writes cost more (28-byte
    // cells: the 1,024-thread finish 2.18 ms this way, 2.35 in pieces)
    const uint32_t v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t* const d = (uint32_t*)(stage + rel);
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j)
      if (4u * j < z) d[j] = v[j];
  } else {
    put_lds(stage + rel, a, b, z);
  }
  __builtin_amdgcn_wave_barrier();
  for (uint32_t e = lane_id() * 16u; e < tot; e += kWave * 16u) {
    const v4 s = *(const v4*)(stage + e);
    if (e + 16u <= tot) *(GMEM u32x4u*)gm(dst + e) = u32x4u{s.x, s.y, s.z, s.w};
    else put_global(dst + e, s, s, tot - e);
  }
  __builtin_amdgcn_wave_barrier();
}

}  // namespace mgt
