// Bit-packed binary masks: one bit per grid point, 32 points per 32-bit word
// (point x of a row is bit x mod 32 of word x / 32, little-endian bytes, so
// bit x mod 8 of byte x / 8).  PID-mean of binary masks (Sec. 4.1 with the
// binary reduction of Sec. 3.2) in exact integers, from popcounts:
//   m_i = sum_x b_i(x),   s(x) = sum_j b_j(x),   S_i = sum_x b_i(x) s(x),
//   IN_in = S_i / (N m_i),  IN_out = S_i / sum_k m_k,
// so the results are bitwise those of the oracle's exact integer form.  Two
// streaming passes over the bits:
//   1. column counts: for every word, the members are added bit-sliced (a
//      vertical counter: plane k holds bit k of the 32 points' counts), up to
//      255 members per group into 8 planes; the groups' planes are then added
//      with a bit-sliced ripple-carry adder into KT planes of the count s;
//   2. row sums: S_i = sum_w sum_k 2^k popcount(b_i(w) & P_k(w)) and
//      m_i = sum_w popcount(b_i(w)), per lane in registers, per wave by a fixed
//      tree, per tile into int64 partials reduced in a fixed order.
// (Up to 127 members: one pass, k_bits_single.hip.)
// U8 0/1 masks and thresholded fields (the sharp isovalue, Sec. 3.1 Eq. 2)
// take the same path: their first pass reads the stored values once, turns
// them into bits, packs them into a workspace copy and counts them, and the
// row pass reads the packed copy.  The packing kernel writes the packed
// layout from U8 masks for callers that keep them packed.
#include "bits_source.h"
#include "device_common.h"
#include "mean_finish.h"
#include "pid_internal.h"
#include "pid_timing.h"

#include <algorithm>
#include <type_traits>

namespace pidk {

// ---------------------------------------------------------------- U8 -> bits
// A chunk of 2048 points of a row is 64 words; lane l holds word l / 2
// (even l) or 32 + l / 2 (odd l) of it.
__device__ __forceinline__ int chunk_word(int lane) { return (lane & 1) ? 32 + (lane >> 1) : (lane >> 1); }

// The lane's word of chunk c of a U8 row, for any row alignment.  The wave
// reads the chunk as 16-byte blocks aligned down from its first byte (a
// misalignment of a bytes): lane l loads blocks l and 64 + l, and lane 63
// also block 128 when a > 0; block k holds points 16k - a .. 16k - a + 15 of
// the chunk.  A block is loaded only if it holds a point of the row below m,
// so no load leaves the 16-byte block (and page) of a valid byte; points
// outside the chunk or at or past m are shifted or masked out.  Lane l's 16
// points from 16l are the top 16 - a bits of its block's bits and the low a
// bits of its right neighbour's; likewise from 1024 + 16l.  Neighbouring
// lanes then swap one half-word.  Wave-uniform call.
// Lane l's word from its two pieces hA, hB (blocks l and 64 + l of the
// aligned-down run) and, when the chunk is not 16-byte aligned (a != 0, the
// same for the whole wave), the neighbours' low bits shifted in; lane 63
// takes them from hC (block 128).
__device__ __forceinline__ uint32_t u8_assemble(uint32_t hA, uint32_t hB, uint32_t hC, int a, int64_t rem, int lane) {
  uint32_t lo = hA, hi = hB;
  if (a != 0) {   // wave-uniform: shift in the neighbours' low bits
    uint32_t nA = (uint32_t)__shfl_down((int)hA, 1, 64);
    uint32_t nB = (uint32_t)__shfl_down((int)hB, 1, 64);
    const uint32_t b0 = (uint32_t)__shfl((int)hB, 0, 64);
    if (lane == 63) {
      nA = b0;
      nB = hC;
    }
    lo = ((hA >> a) | (nA << (16 - a))) & 0xffffu;
    hi = ((hB >> a) | (nB << (16 - a))) & 0xffffu;
  }
  const uint32_t r = (uint32_t)__shfl_xor((int)((lane & 1) ? lo : hi), 1, 64);
  uint32_t wd = (lane & 1) ? (r | (hi << 16)) : (lo | (r << 16));
  const int64_t left = rem - 32 * (int64_t)chunk_word(lane);   // points of the word below m
  if (left < 32) wd = left <= 0 ? 0u : (wd & ((1u << left) - 1u));
  return wd;
}

__device__ __forceinline__ uint32_t chunk_word_u8(const uint8_t* row, int64_t c, int64_t m, int lane) {
  const uint8_t* cp = row + c * 2048;
  const int a = (int)(reinterpret_cast<uintptr_t>(cp) & 15);
  const uint4* bp = reinterpret_cast<const uint4*>(cp - a);
  const int64_t rem = m - c * 2048;   // points of the row from the chunk's first one
  uint32_t hA, hB;
  if (rem >= 2048) {   // a full chunk (wave-uniform): no guards on the loads
    hA = nz16(bp[lane]);
    hB = nz16(bp[64 + lane]);
  } else {
    hA = (16 * lane - a < rem) ? nz16(bp[lane]) : 0u;
    hB = (16 * (64 + lane) - a < rem) ? nz16(bp[64 + lane]) : 0u;
  }
  const uint32_t hC = (a != 0 && lane == 63 && 16 * 128 - a < rem) ? nz16(bp[128]) : 0u;
  return u8_assemble(hA, hB, hC, a, rem, lane);
}

// A chunk inside the row (m - 2048 c >= 2048): the three blocks a lane needs,
// loaded without a branch, so that several rows' loads can be in flight
// together.  Block 128 is one address for the whole wave (only lane 63 uses
// it, and only when a != 0, where it holds a byte of the chunk); when the
// chunk is aligned and ends the row it would lie past the row, and block 127
// is read instead (unused).
struct U8Blocks {
  uint4 a, b, c;
};
__device__ __forceinline__ U8Blocks chunk_blocks_u8_full(const uint8_t* row, int64_t c, int64_t m, int lane) {
  const uint8_t* cp = row + c * 2048;
  const int a = (int)(reinterpret_cast<uintptr_t>(cp) & 15);
  const uint4* bp = reinterpret_cast<const uint4*>(cp - a);
  U8Blocks r;
  r.a = bp[lane];
  r.b = bp[64 + lane];
  r.c = bp[(a != 0 || m - c * 2048 > 2048) ? 128 : 127];
  return r;
}
__device__ __forceinline__ uint32_t chunk_word_u8_full(const U8Blocks& k, const uint8_t* row, int64_t c, int64_t m,
                                                       int lane) {
  const int a = (int)(reinterpret_cast<uintptr_t>(row + c * 2048) & 15);
  return u8_assemble(nz16(k.a), nz16(k.b), nz16(k.c), a, m - c * 2048, lane);
}

// ---------------------------------------------------------------- packing
// Wave per (chunk of 2048 points, 16 rows): grid.x covers four chunks per
// block, grid.y 16 rows per block.
__global__ __launch_bounds__(256) void pack_bits_kernel(const uint8_t* __restrict__ U, int64_t ld, int n, int64_t m,
                                                        uint32_t* __restrict__ out, int64_t ldw) {
  const int lane = threadIdx.x & 63;
  const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t W = (m + 31) / 32;
  if (c * 64 >= W) return;   // whole wave
  const int64_t wi = c * 64 + chunk_word(lane);
  const int i1 = min(n, (int)blockIdx.y * 16 + 16);
  int i = blockIdx.y * 16;
  if (m - c * 2048 >= 2048) {   // the chunk lies inside every row: four rows' blocks loaded first
    for (; i + 3 < i1; i += 4) {
      U8Blocks k[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) k[q] = chunk_blocks_u8_full(U + (int64_t)(i + q) * ld, c, m, lane);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        out[(int64_t)(i + q) * ldw + wi] = chunk_word_u8_full(k[q], U + (int64_t)(i + q) * ld, c, m, lane);
    }
  }
  for (; i + 3 < i1; i += 4) {   // four rows in flight
    uint32_t wd[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) wd[q] = chunk_word_u8(U + (int64_t)(i + q) * ld, c, m, lane);
    if (wi < W) {
#pragma unroll
      for (int q = 0; q < 4; ++q) out[(int64_t)(i + q) * ldw + wi] = wd[q];
    }
  }
  for (; i < i1; ++i) {
    const uint32_t wd = chunk_word_u8(U + (int64_t)i * ld, c, m, lane);
    if (wi < W) out[(int64_t)i * ldw + wi] = wd;
  }
}

// ---------------------------------------------------------------- pass 1
// Stored values (U8 0/1 masks, or fields under the sharp isovalue).  Block =
// four waves on one chunk of 2048 points (blockIdx.x) and one member group
// (blockIdx.y): wave q packs the group's rows q, q + 4, ... of the chunk into
// pk, one word per lane, and counts them (at most 64), eight rows at a time by
// carry-save adders; waves 1-3 pass their planes through LDS and wave 0 adds
// them into gpart[g][k][w] (row stride Wp).  Which points of the chunk a word
// holds is the loader's choice (SrcValues; the row pass reads words and planes
// alike); a chunk that reaches past m holds its points in order, in the words
// below W.
// HBM-bound: N = 10,000 U8 masks on 50^3, 1.25 GB read and 156 MB written,
// 311 us with bits moved by shifts, lane permutes and a plane-by-plane counter
// (about 2.8 operations a point) and one row at a
// time in the ragged chunk; 290-304 us so, 4.7-4.9 TB/s of reads and writes (a
// large copy moves 4.6 here).  Thresholded FP32 rows that are not 16-byte
// aligned (N = 200 on 81^3): whole call 463 -> 104 us.
template <typename Src>
__global__ __launch_bounds__(256) void count_pack_kernel(const typename Src::Elem* __restrict__ U, int64_t ld, int n,
                                                         int64_t m, int chunk, Extract ex, Src src,
                                                         uint32_t* __restrict__ pk, int64_t Wp,
                                                         uint32_t* __restrict__ gpart) {
  __shared__ uint32_t red[3][8][64];
  constexpr int FB = Src::L <= 4 ? 4 : 2;   // rows in flight
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int64_t c = blockIdx.x;
  const int g = blockIdx.y;
  const int64_t W = (m + 31) / 32;
  const int64_t wi = c * 64 + lane;
  const int i0 = g * chunk, i1 = min(n, i0 + chunk);
  uint32_t P[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) P[k] = 0u;
  // how: 0 the chunk lies inside the rows, 1 it is their ragged end, 2 rows of
  // fewer points than a vector
  auto rows = [&](auto how) {
    constexpr int HOW = decltype(how)::value;
    for (int i = i0 + wave; i < i1; i += 32) {   // rows i, i + 4, ..., i + 28
      // (rows past the group re-read its last one: every load of the batch is
      // issued before the first is waited for)
      uint32_t b[8];
#pragma unroll
      for (int q0 = 0; q0 < 8; q0 += FB) {
        if (i + 4 * q0 >= i1) {   // (whole wave)
#pragma unroll
          for (int q = 0; q < FB; ++q) b[q0 + q] = 0u;
          continue;
        }
        typename std::conditional<HOW == 0, typename Src::Raw, typename Src::EdgeRaw>::type raw[FB];
#pragma unroll
        for (int q = 0; q < FB; ++q) {
          const typename Src::Elem* row = U + (int64_t)min(i + 4 * (q0 + q), i1 - 1) * ld;
          if constexpr (HOW == 0) raw[q] = src.load(row, c, lane);
          else if constexpr (HOW == 1) raw[q] = src.load_edge(row, c, m, lane);
          else raw[q] = src.load_short(row, m);
        }
#pragma unroll
        for (int q = 0; q < FB; ++q) {
          uint32_t w[1];
          if constexpr (HOW == 0) src.words(raw[q], ex, w);
          else if constexpr (HOW == 1) src.words_tail(raw[q], c, m, lane, ex, w);
          else src.words_short(raw[q], m, lane, ex, w);
          const bool in = i + 4 * (q0 + q) < i1;   // (whole wave)
          b[q0 + q] = in ? w[0] : 0u;
          if (in && wi < W) pk[(int64_t)(i + 4 * (q0 + q)) * Wp + wi] = w[0];
        }
      }
      uint32_t cnt[4];
      count8(b, cnt);
      add4(P, cnt);
    }
  };
  if (m - c * 2048 >= 2048) rows(std::integral_constant<int, 0>());
  else if (m >= Src::P) rows(std::integral_constant<int, 1>());
  else rows(std::integral_constant<int, 2>());
  if (wave > 0) {
#pragma unroll
    for (int k = 0; k < 8; ++k) red[wave - 1][k][lane] = P[k];
  }
  __syncthreads();
  if (wave != 0 || wi >= W) return;
#pragma unroll
  for (int w = 0; w < 3; ++w) {   // counts of at most 255 in all: 8 planes
    uint32_t x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = red[w][k][lane];
    add_planes(P, x);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) gpart[((int64_t)g * 8 + k) * Wp + wi] = P[k];
}

// V consecutive words of a row from word w0, inside the row and 4V-byte
// aligned for V > 1.
template <int V>
struct Words {
  uint32_t v[V];
};

template <int V>
__device__ __forceinline__ Words<V> load_words(const uint32_t* row, int64_t w0) {
  Words<V> r;
  if constexpr (V == 4) {
    const uint4 t = *reinterpret_cast<const uint4*>(row + w0);
    r.v[0] = t.x; r.v[1] = t.y; r.v[2] = t.z; r.v[3] = t.w;
  } else if constexpr (V == 2) {
    const uint2 t = *reinterpret_cast<const uint2*>(row + w0);
    r.v[0] = t.x; r.v[1] = t.y;
  } else {
    r.v[0] = row[w0];
  }
  return r;
}

// The same without a branch, for a row's ragged end: words at or past W repeat
// word W - 1 (the caller masks them).
template <int V>
__device__ __forceinline__ Words<V> load_words_tail(const uint32_t* row, int64_t w0, int64_t W) {
  Words<V> r;
#pragma unroll
  for (int q = 0; q < V; ++q) r.v[q] = row[min(w0 + q, W - 1)];
  return r;
}

// Packed input.  Block = four waves on V consecutive words per lane from
// (blockIdx.x * 64 + lane) * V and member group blockIdx.y: wave q counts
// the group's rows q, q + 4, ... (at most 64, so 7 bits of its 8 planes),
// waves 1-3 pass their planes through LDS and wave 0 adds them (bit-sliced
// ripple-carry, in wave order).  Bits past m in the last word are masked off.
template <int V>
__global__ __launch_bounds__(256) void b1_count_kernel(const uint32_t* __restrict__ U, int64_t ldw, int n, int64_t W,
                                                       uint32_t lastmask, int chunk, int64_t Wp,
                                                       uint32_t* __restrict__ gpart) {
  __shared__ uint32_t red[3][8][64 * V];
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int64_t w0 = ((int64_t)blockIdx.x * 64 + lane) * V;
  const bool live = w0 < W;   // (no early return: a barrier follows)
  const int g = blockIdx.y;
  const int i0 = g * chunk, i1 = min(n, i0 + chunk);
  uint32_t mask[V];
#pragma unroll
  for (int q = 0; q < V; ++q) mask[q] = (w0 + q < W) ? ((w0 + q == W - 1) ? lastmask : 0xffffffffu) : 0u;
  const bool full = ((int64_t)blockIdx.x + 1) * (64 * V) <= W;
  uint32_t P[V][8];
#pragma unroll
  for (int q = 0; q < V; ++q)
#pragma unroll
    for (int k = 0; k < 8; ++k) P[q][k] = 0u;
  auto rows = [&](auto fc) {
    constexpr bool FULL = decltype(fc)::value;
    for (int i = i0 + wave; i < i1; i += 32) {   // rows i, i + 4, ..., i + 28
      // (rows past the group re-read its last one and count as empty)
      Words<V> a[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const uint32_t* row = U + (int64_t)min(i + 4 * r, i1 - 1) * ldw;
        if constexpr (FULL) a[r] = load_words<V>(row, w0);
        else a[r] = load_words_tail<V>(row, w0, W);
      }
#pragma unroll
      for (int q = 0; q < V; ++q) {
        uint32_t b[8], cnt[4];
#pragma unroll
        for (int r = 0; r < 8; ++r) b[r] = (i + 4 * r < i1) ? a[r].v[q] & mask[q] : 0u;
        count8(b, cnt);
        add4(P[q], cnt);
      }
    }
  };
  if (full) rows(std::true_type());
  else if (live) rows(std::false_type());
  if (wave > 0) {
#pragma unroll
    for (int q = 0; q < V; ++q)
#pragma unroll
      for (int k = 0; k < 8; ++k) red[wave - 1][k][lane * V + q] = P[q][k];
  }
  __syncthreads();
  if (wave != 0 || !live) return;
#pragma unroll
  for (int w = 0; w < 3; ++w)
#pragma unroll
    for (int q = 0; q < V; ++q) {
      uint32_t x[8];   // counts of at most 255 in all: 8 planes
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = red[w][k][lane * V + q];
      add_planes(P[q], x);
    }
#pragma unroll
  for (int q = 0; q < V; ++q)
    if (w0 + q < W) {
#pragma unroll
      for (int k = 0; k < 8; ++k) gpart[((int64_t)g * 8 + k) * Wp + w0 + q] = P[q][k];
    }
}

// Block of 256 / SL words x SL group slices: thread (word w, slice q) adds
// the 8-plane counts of groups q, q + SL, ... with a bit-sliced ripple-carry
// adder; the slices' counts are then added pairwise through LDS (integers, so
// the order of the additions does not change them) and the KT planes of the
// count s written.  Words W..Wp-1 are padding, set to 0.  SL = 16 when there
// are many groups, else 1.
template <int SL, int KT>
__global__ __launch_bounds__(256) void b1_combine_kernel(const uint32_t* __restrict__ gpart, int groups, int64_t W,
                                                         int64_t Wp, uint32_t* __restrict__ planes) {
  constexpr int WB = 256 / SL;   // words per block
  __shared__ uint32_t lds[SL > 1 ? SL / 2 : 1][KT][SL > 1 ? WB : 1];
  const int wl = threadIdx.x % WB, q = threadIdx.x / WB;
  const int64_t w = (int64_t)blockIdx.x * WB + wl;
  uint32_t S[KT];
#pragma unroll
  for (int k = 0; k < KT; ++k) S[k] = 0u;
  if (w < W) {
    for (int g = q; g < groups; g += SL) {
      uint32_t a[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) a[k] = gpart[((int64_t)g * 8 + k) * Wp + w];
      add_planes(S, a);
    }
  }
  if constexpr (SL > 1) {
#pragma unroll
    for (int h = SL / 2; h >= 1; h >>= 1) {
      if (q >= h && q < 2 * h) {
#pragma unroll
        for (int k = 0; k < KT; ++k) lds[q - h][k][wl] = S[k];
      }
      __syncthreads();
      if (q < h) {
        uint32_t a[KT];
#pragma unroll
        for (int k = 0; k < KT; ++k) a[k] = lds[q][k][wl];
        add_planes(S, a);
      }
      __syncthreads();
    }
  }
  if (q == 0 && w < Wp) {
#pragma unroll
    for (int k = 0; k < KT; ++k) planes[(int64_t)k * Wp + w] = S[k];
  }
}

// ---------------------------------------------------------------- pass 2
// Sums over the wave of a[0..7]: lanes 0, 16, 32 and 48 end with those of
// a[0], a[2], a[1], a[3] in r[0] and of a[4], a[6], a[5], a[7] in r[1].  Two
// values share a register after each lane swap, so eight sums take little more
// than one.
__device__ __forceinline__ int swap_add32(int x, int y) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
  return (int)(r[0] + r[1]);
}
__device__ __forceinline__ int swap_add16(int x, int y) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
  return (int)(r[0] + r[1]);
}
__device__ __forceinline__ void wave_sum8(const int (&a)[8], int (&r)[2]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    int v = swap_add16(swap_add32(a[4 * j], a[4 * j + 1]), swap_add32(a[4 * j + 2], a[4 * j + 3]));
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);    // quad_perm [1,0,3,2]
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);    // quad_perm [2,3,0,1]
    v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);   // row_half_mirror
    v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);   // row_mirror
    r[j] = v;
  }
}

// Up to 16 planes.  Wave (tile blockIdx.x, `mw` members from (4 blockIdx.y +
// wave) mw, mw a multiple of 8): the count planes of the tile's V words per lane stay in registers while
// the wave runs over its members, the next four rows in flight; after every
// eight members their sums over the wave are written as the tile's partials
// part[0][i][tile] = m, part[1][i][tile] = S (int64, row length ntiles; the
// sums of a tile stay below 64 V 32 2^16 < 2^31).
// Bound by the vector ALU, 2 KT + 1 operations per word: N = 10,000 on 50^3
// 100 us with 16 planes, the planes loaded again for every 16 members and
// loads under a branch each; 62 us so (14 planes).
template <int KT, int V>
__global__ __launch_bounds__(256) void b1_rows_kernel(const uint32_t* __restrict__ U, int64_t ldw, int n, int64_t W,
                                                      uint32_t lastmask, const uint32_t* __restrict__ planes,
                                                      int64_t Wp, int ntiles, int mw, long long* __restrict__ part) {
  static_assert(KT <= 16, "sums of a tile in 32 bits");
  const int lane = threadIdx.x & 63;
  const int i0 = ((int)blockIdx.y * 4 + wave_id()) * mw;
  if (i0 >= n) return;                       // whole wave (no barrier follows)
  const int i1 = min(n, i0 + mw);
  const int tile = blockIdx.x;
  const int64_t w0 = ((int64_t)tile * 64 + lane) * V;
  // every word of the tile in the row, and whole: no clamps, no masks
  const bool full = ((int64_t)tile + 1) * (64 * V) <= (lastmask == 0xffffffffu ? W : W - 1);
  uint32_t P[KT][V], mask[V];
#pragma unroll
  for (int q = 0; q < V; ++q) mask[q] = (w0 + q < W) ? ((w0 + q == W - 1) ? lastmask : 0xffffffffu) : 0u;
#pragma unroll
  for (int k = 0; k < KT; ++k) {   // (words past the planes' end: any, they are masked)
    const Words<V> pw = load_words<V>(planes + (int64_t)k * Wp, min(w0, Wp - V));
#pragma unroll
    for (int q = 0; q < V; ++q) P[k][q] = pw.v[q];
  }
  auto load = [&](Words<V> (&b)[4], int i, auto fc) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t* row = U + (int64_t)min(i + r, i1 - 1) * ldw;
      if constexpr (decltype(fc)::value) b[r] = load_words<V>(row, w0);
      else b[r] = load_words_tail<V>(row, w0, W);
    }
  };
  auto count = [&](const Words<V>& b, int& am, int& as, auto fc) {
    uint32_t cm = 0u, ck[KT];
#pragma unroll
    for (int k = 0; k < KT; ++k) ck[k] = 0u;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const uint32_t x = decltype(fc)::value ? b.v[q] : b.v[q] & mask[q];
      cm += __popc(x);
#pragma unroll
      for (int k = 0; k < KT; ++k) ck[k] += __popc(x & P[k][q]);
    }
    uint32_t sv = 0u;
#pragma unroll
    for (int k = 0; k < KT; ++k) sv += ck[k] << k;
    am = (int)cm;
    as = (int)sv;
  };
  auto run = [&](auto fc) {
    Words<V> ba[4], bb[4];
    load(ba, i0, fc);
    for (int i = i0; i < i1; i += 8) {
      int am[8], as[8];
      load(bb, i + 4, fc);
#pragma unroll
      for (int r = 0; r < 4; ++r) count(ba[r], am[r], as[r], fc);
      load(ba, i + 8, fc);
#pragma unroll
      for (int r = 0; r < 4; ++r) count(bb[r], am[4 + r], as[4 + r], fc);
      int rm[2], rs[2];
      wave_sum8(am, rm);
      wave_sum8(as, rs);
      if ((lane & 15) == 0) {
        const int row = lane >> 4;             // rows 0..3 hold members 0, 2, 1, 3 of each four
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int64_t e = i + 4 * j + 2 * (row & 1) + (row >> 1);
          if (e < i1) {
            part[e * ntiles + tile] = rm[j];
            part[((int64_t)n + e) * ntiles + tile] = rs[j];
          }
        }
      }
    }
  };
  if (full) run(std::true_type());
  else run(std::false_type());
}

// 32 planes (more than 65,535 members): 64-bit sums.  Wave (tile blockIdx.x,
// members as above).
template <int V>
__global__ __launch_bounds__(256) void b1_rows_wide_kernel(const uint32_t* __restrict__ U, int64_t ldw, int n,
                                                           int64_t W, uint32_t lastmask,
                                                           const uint32_t* __restrict__ planes, int64_t Wp, int ntiles,
                                                           int mw, long long* __restrict__ part) {
  const int lane = threadIdx.x & 63;
  const int i0 = ((int)blockIdx.y * 4 + wave_id()) * mw;
  const int i1 = min(n, i0 + mw);
  const int64_t w0 = ((int64_t)blockIdx.x * 64 + lane) * V;
  uint32_t P[32][V], mask[V];
#pragma unroll
  for (int q = 0; q < V; ++q) mask[q] = (w0 + q < W) ? ((w0 + q == W - 1) ? lastmask : 0xffffffffu) : 0u;
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    const Words<V> pw = load_words<V>(planes + (int64_t)k * Wp, min(w0, Wp - V));
#pragma unroll
    for (int q = 0; q < V; ++q) P[k][q] = pw.v[q];
  }
  for (int i = i0; i < i1; ++i) {
    const Words<V> b = load_words_tail<V>(U + (int64_t)i * ldw, w0, W);
    long long ms = 0, ss = 0;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const uint32_t x = b.v[q] & mask[q];
      ms += __popc(x);
#pragma unroll
      for (int k = 0; k < 32; ++k) ss += (long long)__popc(x & P[k][q]) << k;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      ms += __shfl_xor(ms, o, 64);
      ss += __shfl_xor(ss, o, 64);
    }
    if (lane == 0) {
      part[(int64_t)i * ntiles + blockIdx.x] = ms;
      part[((int64_t)n + i) * ntiles + blockIdx.x] = ss;
    }
  }
}

// ---------------------------------------------------------------- finalize
// Wave per (quantity q, member i): the tile partials part[q][i][*] summed
// (int64, so exactly), into red[q][i].
__global__ __launch_bounds__(256) void b1_reduce_kernel(const long long* __restrict__ part, int nparts, int n,
                                                        long long* __restrict__ red) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= 2 * (int64_t)n) return;   // whole wave
  const long long* p = part + row * nparts;
  long long s = 0;
  for (int b = lane; b < nparts; b += 64) s += p[b];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) red[row] = s;
}

// One block: tot = sum_k m_k (int64, exact), into red[2n].
__global__ __launch_bounds__(1024) void b1_total_kernel(long long* __restrict__ red, int n) {
  __shared__ long long acc[16];
  long long s = 0;
  for (int i = threadIdx.x; i < n; i += 1024) s += red[i];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) acc[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long t = 0;
    for (int k = 0; k < 16; ++k) t += acc[k];
    red[2 * (int64_t)n] = t;
  }
}

// Thread per member: m_i, IN_in = S_i / (N m_i), IN_out = S_i / tot and the
// depth, each ratio one FP64 division of exact integers (0 when the divisor
// is 0).
__global__ __launch_bounds__(256) void b1_ratios_kernel(const long long* __restrict__ red, int n,
                                                        double* __restrict__ m_out, double* __restrict__ in_in,
                                                        double* __restrict__ in_out, double* __restrict__ depth) {
#pragma clang fp contract(off)
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const double mm = (double)red[i], a = (double)red[n + i], tot = (double)red[2 * (int64_t)n];
  const double ii = (mm > 0.0) ? a / ((double)n * mm) : 0.0;
  const double oo = (tot > 0.0) ? a / tot : 0.0;
  if (m_out) m_out[i] = mm;
  if (in_in) in_in[i] = ii;
  if (in_out) in_out[i] = oo;
  if (depth) depth[i] = ii < oo ? ii : oo;
}

// ---------------------------------------------------------------- host side
namespace {

// The tile partials reduced per member, then the ratios (and ranks, see
// mean_finish.h).  Up to 2048 members every block of the ratios forms the
// total mass by itself; beyond, one block of 1024 threads forms it once (n =
// 10,000: 9.4 us for the two launches against 12.7 us).
hipError_t b1_finalize(const long long* part, int nblk, int64_t n, long long* red, const pid_out& out, hipStream_t st) {
  KernelTimer tm("pidmean_finalize", st);
  hipLaunchKernelGGL(b1_reduce_kernel, dim3((unsigned)((2 * n + 3) / 4)), 256, 0, st, part, nblk, (int)n, red);
  if (n <= 2048) {
    launch_mean_finish(red, n, out, st);
  } else {
    hipLaunchKernelGGL(b1_total_kernel, 1, 1024, 0, st, red, (int)n);
    hipLaunchKernelGGL(b1_ratios_kernel, dim3((unsigned)((n + 255) / 256)), 256, 0, st, red, (int)n, out.mass,
                       out.in_in, out.in_out, out.depth);
  }
  return hipGetLastError();
}

// At most kBitsSingleN members: one pass over the stored values.
hipError_t single_pass_mean(const B1Plan& p, const pid_ensemble& e, int iso_kind, const ExtractHost& exh,
                            const pid_out& out, void* ws, hipStream_t st) {
  Carve c(ws);
  long long* part = c.take<long long>((size_t)2 * e.n * p.blocks);
  long long* red = c.take<long long>((size_t)2 * e.n);
  int nblk = 0;
  const hipError_t err = launch_bits_single(e, iso_kind, exh, part, p.blocks, &nblk, st);
  return err != hipSuccess ? err : b1_finalize(part, nblk, e.n, red, out, st);
}

// Pass 2 and the finalize, on packed rows U (row stride ldw words, vector
// loads when `aligned`).
hipError_t b1_rows_finalize(const B1Plan& p, const uint32_t* U, int64_t ldw, bool aligned, int64_t n, int64_t m,
                            const uint32_t* planes, long long* part, long long* red, const pid_out& out,
                            hipStream_t st) {
  const int rem = (int)(m % 32);
  const uint32_t lastmask = rem ? ((1u << rem) - 1u) : 0xffffffffu;
  const int v = aligned ? (p.kt <= 16 ? 4 : 2) : 1;
  const int ntiles = (int)((p.W + 64 * v - 1) / (64 * v));
  {
    KernelTimer tm("pidmean", st);
    // members per wave: the planes are loaded once for up to 32, fewer while
    // that leaves less than 2 waves per SIMD
    int mw = 32;
    while (mw > 8 && (int64_t)ntiles * ((n + mw - 1) / mw) < 2048) mw /= 2;
    const dim3 grid((unsigned)ntiles, (unsigned)((n + 4 * mw - 1) / (4 * mw)));
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, grid, 256, 0, st, U, ldw, (int)n, p.W, lastmask, planes, p.Wp, ntiles, mw, part);
    };
    switch (p.kt) {
      case 8: v == 4 ? go(b1_rows_kernel<8, 4>) : go(b1_rows_kernel<8, 1>); break;
      case 10: v == 4 ? go(b1_rows_kernel<10, 4>) : go(b1_rows_kernel<10, 1>); break;
      case 12: v == 4 ? go(b1_rows_kernel<12, 4>) : go(b1_rows_kernel<12, 1>); break;
      case 14: v == 4 ? go(b1_rows_kernel<14, 4>) : go(b1_rows_kernel<14, 1>); break;
      case 16: v == 4 ? go(b1_rows_kernel<16, 4>) : go(b1_rows_kernel<16, 1>); break;
      default: v == 2 ? go(b1_rows_wide_kernel<2>) : go(b1_rows_wide_kernel<1>); break;
    }
  }
  return b1_finalize(part, ntiles, n, red, out, st);
}

template <int KT>
void launch_combine(const B1Plan& p, const uint32_t* gpart, uint32_t* planes, hipStream_t st) {
  if (p.groups >= 32)
    hipLaunchKernelGGL((b1_combine_kernel<16, KT>), dim3((unsigned)((p.Wp + 15) / 16)), 256, 0, st, gpart, p.groups,
                       p.W, p.Wp, planes);
  else
    hipLaunchKernelGGL((b1_combine_kernel<1, KT>), dim3((unsigned)((p.Wp + 255) / 256)), 256, 0, st, gpart, p.groups,
                       p.W, p.Wp, planes);
}

hipError_t b1_combine(const B1Plan& p, const uint32_t* gpart, uint32_t* planes, hipStream_t st) {
  switch (p.kt) {
    case 8: launch_combine<8>(p, gpart, planes, st); break;
    case 10: launch_combine<10>(p, gpart, planes, st); break;
    case 12: launch_combine<12>(p, gpart, planes, st); break;
    case 14: launch_combine<14>(p, gpart, planes, st); break;
    case 16: launch_combine<16>(p, gpart, planes, st); break;
    default: launch_combine<32>(p, gpart, planes, st); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_b1_mean(const pid_ensemble& e, const pid_out& out, void* ws, hipStream_t st) {
  const B1Plan p = b1_plan(e.n, e.m);
  if (p.single) return single_pass_mean(p, e, PID_ISO_NONE, ExtractHost{}, out, ws, st);
  Carve c(ws);
  uint32_t* gpart = c.take<uint32_t>((size_t)p.groups * 8 * p.Wp);
  uint32_t* planes = c.take<uint32_t>((size_t)p.kt * p.Wp);
  long long* part = c.take<long long>((size_t)2 * e.n * p.ntiles);
  long long* red = c.take<long long>((size_t)2 * e.n + 1);
  const uint32_t* U = reinterpret_cast<const uint32_t*>(e.data);
  const int64_t ldw = e.ld / 32;
  const int rem = (int)(e.m % 32);
  const uint32_t lastmask = rem ? ((1u << rem) - 1u) : 0xffffffffu;
  const bool aligned = (reinterpret_cast<uintptr_t>(e.data) & 15) == 0 && ldw % 4 == 0;
  {
    KernelTimer tm("pidmean_colsum", st);
    if (aligned)
      hipLaunchKernelGGL((b1_count_kernel<4>), dim3((unsigned)((p.W + 255) / 256), (unsigned)p.groups), 256, 0, st,
                         U, ldw, (int)e.n, p.W, lastmask, p.chunk, p.Wp, gpart);
    else
      hipLaunchKernelGGL((b1_count_kernel<1>), dim3((unsigned)((p.W + 63) / 64), (unsigned)p.groups), 256, 0, st,
                         U, ldw, (int)e.n, p.W, lastmask, p.chunk, p.Wp, gpart);
    hipError_t err = b1_combine(p, gpart, planes, st);
    if (err != hipSuccess) return err;
  }
  return b1_rows_finalize(p, U, ldw, aligned, e.n, e.m, planes, part, red, out, st);
}

template <typename Src>
static void launch_count_pack(const pid_ensemble& e, const Extract& ex, const B1Plan& p, uint32_t* pk,
                              uint32_t* gpart, hipStream_t st) {
  hipLaunchKernelGGL((count_pack_kernel<Src>), dim3((unsigned)((e.m + 2047) / 2048), (unsigned)p.groups), 256, 0, st,
                     reinterpret_cast<const typename Src::Elem*>(e.data), e.ld, (int)e.n, e.m, p.chunk, ex, Src{}, pk, p.Wp,
                     gpart);
}

hipError_t launch_mask_bits_mean(const pid_ensemble& e, int iso_kind, const ExtractHost& exh, const pid_out& out,
                                 void* ws, hipStream_t st) {
  const B1Plan p = b1_plan(e.n, e.m);
  if (p.single) return single_pass_mean(p, e, iso_kind, exh, out, ws, st);
  Carve c(ws);
  uint32_t* gpart = c.take<uint32_t>((size_t)p.groups * 8 * p.Wp);
  uint32_t* planes = c.take<uint32_t>((size_t)p.kt * p.Wp);
  long long* part = c.take<long long>((size_t)2 * e.n * p.ntiles);
  long long* red = c.take<long long>((size_t)2 * e.n + 1);
  uint32_t* pk = c.take<uint32_t>((size_t)e.n * p.Wp);
  {
    KernelTimer tm("pidmean_colsum", st);
    const Extract ex = __builtin_bit_cast(Extract, exh);
    if (iso_kind == PID_ISO_NONE) {   // U8 0/1 masks
      if (bytes_misaligned(e)) launch_count_pack<SrcBytes>(e, ex, p, pk, gpart, st);
      else launch_count_pack<SrcValues<uint8_t, false>>(e, ex, p, pk, gpart, st);
    } else {                          // the sharp isovalue on stored values
      switch (e.dtype) {
        case PID_F64: launch_count_pack<SrcValues<double, true>>(e, ex, p, pk, gpart, st); break;
        case PID_F32: launch_count_pack<SrcValues<float, true>>(e, ex, p, pk, gpart, st); break;
        case PID_F16: launch_count_pack<SrcValues<f16, true>>(e, ex, p, pk, gpart, st); break;
        case PID_BF16: launch_count_pack<SrcValues<bf16_t, true>>(e, ex, p, pk, gpart, st); break;
        default: launch_count_pack<SrcValues<uint8_t, true>>(e, ex, p, pk, gpart, st); break;
      }
    }
    hipError_t err = b1_combine(p, gpart, planes, st);
    if (err != hipSuccess) return err;
  }
  return b1_rows_finalize(p, pk, p.Wp, true, e.n, e.m, planes, part, red, out, st);
}

hipError_t launch_pack_bits(const pid_ensemble& e, uint32_t* out, int64_t out_ldw, hipStream_t st) {
  const int64_t chunks = (e.m + 2047) / 2048;
  const dim3 grid((unsigned)((chunks + 3) / 4), (unsigned)((e.n + 15) / 16));
  hipLaunchKernelGGL(pack_bits_kernel, grid, 256, 0, st, reinterpret_cast<const uint8_t*>(e.data), e.ld, (int)e.n,
                     e.m, out, out_ldw);
  return hipGetLastError();
}

}  // namespace pidk
