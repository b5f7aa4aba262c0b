// Binary members as 32-point words: adders over the bits of several members
// (bit-sliced counts), and stored values turned into words.
#pragma once
#include "device_common.h"
#include "pid_internal.h"

namespace pidk {

// Sum and carry of three bits, per bit position.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}

// c[0..3] = bit planes of the number of set bits among b[0..7].
__device__ __forceinline__ void count8(const uint32_t (&b)[8], uint32_t (&c)[4]) {
  const uint32_t s0 = xor3(b[0], b[1], b[2]), t0 = maj3(b[0], b[1], b[2]);
  const uint32_t s1 = xor3(b[3], b[4], b[5]), t1 = maj3(b[3], b[4], b[5]);
  const uint32_t s2 = xor3(s0, s1, b[6]), t2 = maj3(s0, s1, b[6]);
  c[0] = s2 ^ b[7];
  const uint32_t t3 = s2 & b[7];
  const uint32_t u0 = xor3(t0, t1, t2), v0 = maj3(t0, t1, t2);
  c[1] = u0 ^ t3;
  const uint32_t v1 = u0 & t3;
  c[2] = v0 ^ v1;
  c[3] = v0 & v1;
}

// The lowest bits of the 16 bytes of v as 16 bits (bytes weighted by 1, 2, 4,
// ... in two dot products per 8 bytes).
__device__ __forceinline__ uint32_t low_bits16(uint4 v) {
  uint32_t lo = __builtin_amdgcn_udot4(v.x & 0x01010101u, 0x08040201u, 0u, false);
  lo = __builtin_amdgcn_udot4(v.y & 0x01010101u, 0x80402010u, lo, false);
  uint32_t hi = __builtin_amdgcn_udot4(v.z & 0x01010101u, 0x08040201u, 0u, false);
  hi = __builtin_amdgcn_udot4(v.w & 0x01010101u, 0x80402010u, hi, false);
  return lo | (hi << 8);
}

// Bit k of the result: whether byte k of v is nonzero.  (v_lerp_u8 averages
// bytes: (b + 255) / 2 has its highest bit set exactly for b >= 1.)
__device__ __forceinline__ uint32_t nz16(uint4 v) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  uint32_t t[2] = {0u, 0u};
#pragma unroll
  for (int k = 0; k < 4; ++k)
    t[k >> 1] = __builtin_amdgcn_udot4(__builtin_amdgcn_lerp(w[k], ~0u, 0u) & 0x80808080u,
                                       (k & 1) ? 0x80402010u : 0x08040201u, t[k >> 1], false);
  return (t[0] | (t[1] << 8)) >> 7;
}

// P (8 bit planes of counts) += c (4 planes).
__device__ __forceinline__ void add4(uint32_t (&P)[8], const uint32_t (&c)[4]) {
  uint32_t cy = 0u;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const uint32_t a = P[k];
    if (k < 4) {
      P[k] = xor3(a, c[k], cy);
      cy = maj3(a, c[k], cy);
    } else {
      P[k] = a ^ cy;
      cy = a & cy;
    }
  }
}

// S (KT planes) += x (KX planes); the caller's counts fit in KT planes.
template <int KT, int KX>
__device__ __forceinline__ void add_planes(uint32_t (&S)[KT], const uint32_t (&x)[KX]) {
  uint32_t cy = 0u;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const uint32_t a = S[k];
    if (k < KX) {
      S[k] = xor3(a, x[k], cy);
      cy = maj3(a, x[k], cy);
    } else {
      S[k] = a ^ cy;
      cy = a & cy;
    }
  }
}

// Stored values of T, rows of any alignment: a tile is 2048 points, a lane
// takes L = 2 sizeof(T) blocks of 16 bytes, 64 blocks apart (each load of the
// wave is 1 KB of the row), P = 16 / sizeof(T) points and bits each.
template <typename T, bool STEP>
struct SrcValues {
  static constexpr int V = 1, TILE = 2048;
  static constexpr int P = 16 / (int)sizeof(T), L = 32 / P;
  static constexpr int BATCH = L <= 2 ? 4 : (L <= 4 ? 2 : 1);   // members loaded together
  typedef T Elem;
  struct Raw { Vec16<T> v[L]; };
  static __device__ __forceinline__ Vec16<T> load16u(const T* p) {   // p aligned as a T
    return load16_nt_any(p);
  }
  static __device__ __forceinline__ uint32_t bits(const Vec16<T>& v, const Extract& ex) {
    if constexpr (!STEP) {
      return nz16(__builtin_bit_cast(uint4, v));
    } else {
      uint32_t w = 0u;
#pragma unroll
      for (int p = 0; p < P; ++p) w |= (uint32_t)(extract_bit<MODE_STEP>(v.v[p], ex) != 0) << p;
      return w;
    }
  }
  __device__ __forceinline__ Raw load(const T* row, int64_t tile, int lane) const {
    Raw r;
#pragma unroll
    for (int k = 0; k < L; ++k) r.v[k] = load16u(row + tile * TILE + (64 * k + lane) * P);
    return r;
  }
  __device__ __forceinline__ void words(const Raw& r, const Extract& ex, uint32_t (&b)[1]) const {
    b[0] = 0u;
#pragma unroll
    for (int k = 0; k < L; ++k) b[0] |= bits(r.v[k], ex) << (P * k);
  }
  // The ragged last tile: the blocks of load(), those that reach past m read P
  // points before m and shifted.  Needs m >= P, so that no load sits under a
  // branch: with one the single-pass kernel waited for each member's loads in turn
  // (n = 33 FP32 on 90^3, thresholded: 53 us, 38 so; 42 in two passes).
  typedef Raw EdgeRaw;
  __device__ __forceinline__ EdgeRaw load_edge(const T* row, int64_t tile, int64_t m, int lane) const {
    EdgeRaw r;
#pragma unroll
    for (int k = 0; k < L; ++k) r.v[k] = load16u(row + min(tile * TILE + (64 * k + lane) * P, m - P));
    return r;
  }
  // Its words: where the order of a tile's points does not matter (they meet only
  // the same points of the other members) ...
  __device__ __forceinline__ void words_edge(const EdgeRaw& r, int64_t tile, int64_t m, int lane, const Extract& ex,
                                             uint32_t (&b)[1]) const {
    b[0] = 0u;
#pragma unroll
    for (int k = 0; k < L; ++k) b[0] |= edge_bits(r, k, tile, m, lane, ex) << (P * k);
  }
  // ... and in the order of the points, lane l's word holding the 32 points from
  // tile * TILE + 32 l (called by the whole wave).  Word w is the blocks of L
  // neighbouring lanes of one load: they meet by lane moves, the j-th of such lanes
  // keeps the word of the j-th load, and the words change places.  (Loaded in this
  // order, L blocks of 16 bytes from 32 points per lane, every load of the wave touches
  // 64 lines: FP64, n = 1,000 on 65,488 points, whole call 160 us, 138 so.)
  __device__ __forceinline__ void words_tail(const EdgeRaw& r, int64_t tile, int64_t m, int lane, const Extract& ex,
                                             uint32_t (&b)[1]) const {
    const int j = lane % L;
    uint32_t own = 0u;
#pragma unroll
    for (int k = 0; k < L; ++k) {
      int e = (int)(edge_bits(r, k, tile, m, lane, ex) << (P * j));
      e |= __builtin_amdgcn_update_dpp(0, e, 0xB1, 0xF, 0xF, false);                          // quad_perm [1,0,3,2]
      if constexpr (L > 2) e |= __builtin_amdgcn_update_dpp(0, e, 0x4E, 0xF, 0xF, false);     // quad_perm [2,3,0,1]
      if constexpr (L > 4) e |= __builtin_amdgcn_update_dpp(0, e, 0x141, 0xF, 0xF, false);    // row_half_mirror
      if constexpr (L > 8) e |= __builtin_amdgcn_update_dpp(0, e, 0x140, 0xF, 0xF, false);    // row_mirror
      own = j == k ? (uint32_t)e : own;
    }
    b[0] = (uint32_t)__shfl((int)own, (lane % (2 * P)) * L + lane / (2 * P), 64);
  }
  // Rows of fewer than P points, read point by point: the first block of lane 0.
  // (A form of its own: where one function chose between this and vector loads,
  // the compiler merged them into byte loads, and the ragged tile of n = 3,314 U8
  // masks of 65,293 points took 190 of 250 us.)
  __device__ __forceinline__ EdgeRaw load_short(const T* row, int64_t m) const {
    EdgeRaw r{};
#pragma unroll
    for (int p = 0; p < P; ++p) r.v[0].v[p] = row[min((int64_t)p, m - 1)];
    return r;
  }
  __device__ __forceinline__ void words_short(const EdgeRaw& r, int64_t m, int lane, const Extract& ex,
                                              uint32_t (&b)[1]) const {
    b[0] = lane == 0 ? bits(r.v[0], ex) & ((1u << (int)m) - 1u) : 0u;
  }

 private:
  // The bits of the k-th block of load_edge(), zeros past m.
  static __device__ __forceinline__ uint32_t edge_bits(const EdgeRaw& r, int k, int64_t tile, int64_t m, int lane,
                                                       const Extract& ex) {
    const int left = (int)max((int64_t)0, min((int64_t)P, m - (tile * TILE + (64 * k + lane) * P)));
    return left > 0 ? (bits(r.v[k], ex) >> (P - left)) & ((1u << left) - 1u) : 0u;
  }
};

// U8 masks (a nonzero byte counts as 1) whose rows are not 4-byte aligned (16-byte loads there cost 5-8 %
// more): the chunk is read as 16-byte blocks aligned down from its first byte,
// a bytes (0..15) before it; a block holds points 16k - a .. 16k - a + 15, so a
// lane's 16 points are the top 16 - a bits of its block's and the low a bits of
// the next lane's.  Block 128, one address for the wave, completes lane 63; it
// is read only if a != 0, when it holds a byte of the chunk.
struct SrcBytes : SrcValues<uint8_t, false> {
  struct Raw { uint4 a, b, c; int sh; };
  __device__ __forceinline__ Raw load(const uint8_t* row, int64_t tile, int lane) const {
    const uint8_t* cp = row + tile * TILE;
    const int a = (int)(reinterpret_cast<uintptr_t>(cp) & 15);
    const uint4* bp = reinterpret_cast<const uint4*>(cp - a);
    return Raw{bp[lane], bp[64 + lane], bp[a != 0 ? 128 : 127], a};
  }
  __device__ __forceinline__ void words(const Raw& r, const Extract&, uint32_t (&b)[1]) const {
    const int hA = (int)nz16(r.a), hB = (int)nz16(r.b), hC = (int)nz16(r.c);
    const int b0 = __builtin_amdgcn_readfirstlane(hB);
    const uint32_t nA = (uint32_t)__builtin_amdgcn_update_dpp(b0, hA, 0x130, 0xF, 0xF, false);   // wave_shl:1
    const uint32_t nB = (uint32_t)__builtin_amdgcn_update_dpp(hC, hB, 0x130, 0xF, 0xF, false);
    const uint32_t lo = (((uint32_t)hA >> r.sh) | (nA << (16 - r.sh))) & 0xffffu;
    const uint32_t hi = ((uint32_t)hB >> r.sh) | (nB << (16 - r.sh));
    b[0] = lo | (hi << 16);
  }
};
inline bool bytes_misaligned(const pid_ensemble& e) {
  return ((reinterpret_cast<uintptr_t>(e.data) | (uintptr_t)e.ld) & 3) != 0;
}

}  // namespace pidk
