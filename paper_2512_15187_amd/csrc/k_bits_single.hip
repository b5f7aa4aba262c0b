// PID-mean of at most 127 binary members in one pass over the stored values
// (bit-packed masks, U8 0/1 masks, or fields under the sharp isovalue), in
// exact integers:
//   m_i = sum_x b_i(x),  s(x) = sum_j b_j(x),  S_i = sum_x b_i(x) s(x).
// A workgroup owns all members on a tile of points, one 32-point word (or V of
// them) per lane and member, so the counts s of its points are complete after
// one exchange through LDS and the bits, still in registers, are multiplied
// with them at once: nothing is read twice and neither count planes nor a
// packed copy go through memory (the passes of k_bits.hip, for more members,
// read the bits twice and write and read the planes of s).
//
// Per tile a wave forms the words of its members (at most 8), adds them
// bit-sliced (carry-save adders of two three-input operations each) into 4
// planes, the waves' planes meet in LDS, and per member and word
// S += sum_k 2^k popcount(b & P_k) over the KT planes of s.  That last step is
// 2 KT + 1 operations per 32 points and bounds packed input together with the
// HBM read; U8 and field input is bound by its read.  Whole calls against the
// two passes, N = 50: packed 352^3 192 -> 81 us, 512^3 509 -> 210 us (839 MB,
// 4.0 TB/s); U8 512^3 1864 -> 1120 us (6.7 GB, 6.0 TB/s); FP32 fields, N = 48
// on 128^3, 97 -> 87 us; unaligned rows (N = 30 on 81^3) 72 -> 28 us.
#include "bits_source.h"
#include "pid_internal.h"
#include "pid_timing.h"

#include <algorithm>
#include <type_traits>

namespace pidk {

namespace {

constexpr int kRows = 8;        // members per wave
constexpr int kWavePlanes = 4;  // planes of a count of up to kRows

// Where a lane's words come from.  load() issues the loads of one member's
// words of a tile that lies inside the row; words() turns them into bits;
// load_edge() and words_edge() do it for the ragged last tile, load_short() and
// words_short() for rows of fewer than P points.  Which point sits in which
// bit is the same for every member, and nothing else depends on it.  (Stored
// values: SrcValues in bits_source.h.)

// Bit-packed rows: V consecutive words per lane (V = 4, 2: rows aligned to
// 4V bytes; V = 1: any).
template <int VW>
struct SrcBits {
  static constexpr int V = VW, TILE = 64 * VW * 32;   // points per tile
  static constexpr int BATCH = 4;                     // members loaded together
  typedef uint32_t Elem;                              // stored unit of the row stride
  struct Raw { uint32_t w[V]; };
  uint32_t lastmask;
  __device__ __forceinline__ Raw load(const uint32_t* row, int64_t tile, int lane) const {
    Raw r;
    const uint32_t* p = row + (tile * 64 + lane) * V;
    if constexpr (V == 4) __builtin_memcpy(&r, reinterpret_cast<const uint4*>(p), 16);
    else if constexpr (V == 2) __builtin_memcpy(&r, reinterpret_cast<const uint2*>(p), 8);
    else r.w[0] = p[0];
    return r;
  }
  __device__ __forceinline__ void words(const Raw& r, const Extract&, uint32_t (&b)[V]) const {
#pragma unroll
    for (int q = 0; q < V; ++q) b[q] = r.w[q];
  }
  // (the ragged last tile)
  static constexpr int P = 1;
  __device__ __forceinline__ Raw load_edge(const uint32_t* row, int64_t tile, int64_t m, int lane) const {
    Raw r;
#pragma unroll
    for (int q = 0; q < V; ++q) r.w[q] = row[min((tile * 64 + lane) * V + q, (m + 31) / 32 - 1)];
    return r;
  }
  __device__ __forceinline__ void words_edge(const Raw& r, int64_t tile, int64_t m, int lane, const Extract&,
                                             uint32_t (&b)[V]) const {
    const int64_t W = (m + 31) / 32;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const int64_t w = (tile * 64 + lane) * V + q;
      b[q] = w < W ? r.w[q] & (w == W - 1 ? lastmask : 0xffffffffu) : 0u;
    }
  }
};

// Sum of v over the wave as a 64-bit scalar, exact while every row of 16
// lanes sums below 2^31.
__device__ __forceinline__ long long wave_sum16(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);    // quad_perm [1,0,3,2]
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);    // quad_perm [2,3,0,1]
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);   // row_half_mirror
  v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);   // row_mirror
  return (long long)__builtin_amdgcn_readlane(v, 0) + (long long)__builtin_amdgcn_readlane(v, 16) +
         (long long)__builtin_amdgcn_readlane(v, 32) + (long long)__builtin_amdgcn_readlane(v, 48);
}

// part[0][i][block] = m_i, part[1][i][block] = S_i of the block's tiles
// blockIdx.x, blockIdx.x + gridDim.x, ...
template <typename Src, int KT, int NWMAX>
__global__ __launch_bounds__(64 * NWMAX) void bits_single_kernel(const typename Src::Elem* __restrict__ U, int64_t ld,
                                                                 int n, int64_t m, int64_t nfull, int64_t ntiles,
                                                                 Extract ex, Src src, long long* __restrict__ part) {
  constexpr int V = Src::V;
  __shared__ __align__(16) uint32_t cw[NWMAX][kWavePlanes][64 * V];   // the waves' planes
  __shared__ __align__(16) uint32_t tot[KT][64 * V];                  // the planes of s
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int nw = blockDim.x >> 6;
  const int i0 = wave * kRows;
  const int nr = min(kRows, n - i0);                     // members of this wave, >= 1
  const typename Src::Elem* rows = U + (int64_t)i0 * ld;
  uint32_t am[kRows], as[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) am[r] = as[r] = 0u;

  auto process = [&](uint32_t (&b)[kRows][V]) {
    uint32_t c[kWavePlanes][V];
#pragma unroll
    for (int q = 0; q < V; ++q) {
      uint32_t col[kRows], cq[kWavePlanes];
#pragma unroll
      for (int r = 0; r < kRows; ++r) col[r] = b[r][q];
      count8(col, cq);
#pragma unroll
      for (int k = 0; k < kWavePlanes; ++k) c[k][q] = cq[k];
    }
#pragma unroll
    for (int k = 0; k < kWavePlanes; ++k)
#pragma unroll
      for (int q = 0; q < V; ++q) cw[wave][k][lane * V + q] = c[k][q];
    lds_barrier();
    // the waves' counts of word t, added by thread t
    for (int t = threadIdx.x; t < 64 * V; t += 64 * nw) {
      uint32_t S[KT];
#pragma unroll
      for (int k = 0; k < KT; ++k) S[k] = k < kWavePlanes ? cw[0][k][t] : 0u;
      for (int w = 1; w < nw; ++w) {
        uint32_t cy = 0u;
#pragma unroll
        for (int k = 0; k < KT; ++k) {
          const uint32_t x = k < kWavePlanes ? cw[w][k][t] : 0u;
          const uint32_t s = xor3(S[k], x, cy);
          cy = maj3(S[k], x, cy);
          S[k] = s;
        }
      }
#pragma unroll
      for (int k = 0; k < KT; ++k) tot[k][t] = S[k];
    }
    lds_barrier();
    uint32_t P[KT][V];
#pragma unroll
    for (int k = 0; k < KT; ++k)
#pragma unroll
      for (int q = 0; q < V; ++q) P[k][q] = tot[k][lane * V + q];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      if (r < nr) {
        uint32_t ck[KT];
#pragma unroll
        for (int k = 0; k < KT; ++k) ck[k] = 0u;
#pragma unroll
        for (int q = 0; q < V; ++q) {
          am[r] += __popc(b[r][q]);
#pragma unroll
          for (int k = 0; k < KT; ++k) ck[k] += __popc(b[r][q] & P[k][q]);
        }
#pragma unroll
        for (int k = 0; k < KT; ++k) as[r] += ck[k] << k;
      }
    }
  };

  // BATCH members' loads are issued together; rows past n re-read row n - 1
  // and count as empty
  // how: 0 a whole tile, 1 the ragged last one, 2 that of rows of fewer than P points
  auto tile_step = [&](int64_t tile, auto how) {
    constexpr int HOW = decltype(how)::value;
    uint32_t b[kRows][V];
#pragma unroll
    for (int r0 = 0; r0 < kRows; r0 += Src::BATCH) {
      if (r0 < nr) {
        auto batch = [&](auto load, auto words) {
          decltype(load(src, rows)) raw[Src::BATCH];
#pragma unroll
          for (int q = 0; q < Src::BATCH; ++q) raw[q] = load(src, rows + (int64_t)min(r0 + q, nr - 1) * ld);
#pragma unroll
          for (int q = 0; q < Src::BATCH; ++q) {
            words(src, raw[q], b[r0 + q]);
            const uint32_t keep = r0 + q < nr ? 0xffffffffu : 0u;
#pragma unroll
            for (int v = 0; v < V; ++v) b[r0 + q][v] &= keep;
          }
        };
        typedef const typename Src::Elem* Row;
        if constexpr (HOW == 0)
          batch([&](const auto& s, Row p) { return s.load(p, tile, lane); },
                [&](const auto& s, const auto& x, auto& w) { s.words(x, ex, w); });
        else if constexpr (HOW == 1)
          batch([&](const auto& s, Row p) { return s.load_edge(p, tile, m, lane); },
                [&](const auto& s, const auto& x, auto& w) { s.words_edge(x, tile, m, lane, ex, w); });
        else
          batch([&](const auto& s, Row p) { return s.load_short(p, m); },
                [&](const auto& s, const auto& x, auto& w) { s.words_short(x, m, lane, ex, w); });
      } else {
#pragma unroll
        for (int q = 0; q < Src::BATCH; ++q)
#pragma unroll
          for (int v = 0; v < V; ++v) b[r0 + q][v] = 0u;
      }
    }
    process(b);
  };
  for (int64_t tile = blockIdx.x; tile < nfull; tile += gridDim.x) tile_step(tile, std::integral_constant<int, 0>());
  if (nfull < ntiles && blockIdx.x == (unsigned)(nfull % gridDim.x)) {
    if constexpr (Src::P == 1) tile_step(nfull, std::integral_constant<int, 1>());
    else if (m >= Src::P) tile_step(nfull, std::integral_constant<int, 1>());
    else tile_step(nfull, std::integral_constant<int, 2>());
  }
  const int nblk = gridDim.x;
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    if (r < nr) {
      const long long ms = wave_sum16((int)am[r]), ss = wave_sum16((int)as[r]);
      if (lane == 0) {
        part[(size_t)(i0 + r) * nblk + blockIdx.x] = ms;
        part[((size_t)n + i0 + r) * nblk + blockIdx.x] = ss;
      }
    }
  }
}

template <typename Src>
hipError_t launch_src(const pid_ensemble& e, int64_t ld, const Extract& ex, const Src& src, long long* part,
                      int64_t max_blocks, int* nblk, hipStream_t st) {
  const int64_t ntiles = (e.m + Src::TILE - 1) / Src::TILE;
  const int64_t nfull = e.m / Src::TILE;
  const int nw = (int)((e.n + kRows - 1) / kRows);
  // Workgroups: about 8 waves per CU (14 with 4 words per lane), each streaming
  // its share of the tiles; more streams are slower (U8, N = 50 on 256^3: 175,
  // 180, 191 and 236 us with 7, 14, 28 and 112 waves per CU; packed on 352^3:
  // 108, 76, 82 and 106 us).  Thresholded 16-bit fields 16: they compare twice
  // the points a byte as FP32 (N = 33 on 3,673,760 points 87, 65 and 55 us with 5,
  // 10 and 15 waves per CU, 74 in two passes; N = 44 106, 81 with 6 and 12, 98 in
  // two passes).
  const int waves = Src::V == 4 ? 14 : (sizeof(typename Src::Elem) == 2 ? 16 : 8);
  const int64_t fit = (int64_t)device_cu_count() * std::max(1, waves / nw);
  *nblk = (int)std::min(ntiles, std::min(max_blocks, std::max(fit, (ntiles + 8000) / 8001)));
  const typename Src::Elem* U = reinterpret_cast<const typename Src::Elem*>(e.data);
  const dim3 block(64 * nw);
  auto go = [&](auto k) {
    hipLaunchKernelGGL(k, dim3(*nblk), block, 0, st, U, ld, (int)e.n, e.m, nfull, ntiles, ex, src, part);
    return hipGetLastError();
  };
  // counts of at most 56 members: 6 planes (the caller takes 4 words per lane
  // only there, and 2 only beyond)
  if constexpr (Src::V == 4) return go(bits_single_kernel<Src, 6, 8>);
  else if constexpr (Src::V == 2) return go(bits_single_kernel<Src, 7, 16>);
  else return nw <= 7 ? go(bits_single_kernel<Src, 6, 8>) : go(bits_single_kernel<Src, 7, 16>);
}

}  // namespace

hipError_t launch_bits_single(const pid_ensemble& e, int iso_kind, const ExtractHost& exh, long long* part,
                              int64_t max_blocks, int* nblk, hipStream_t st) {
  KernelTimer tm("pidmean", st);
  const Extract ex = __builtin_bit_cast(Extract, exh);
  if (e.dtype == PID_B1) {
    const int64_t ldw = e.ld / 32;
    const int rem = (int)(e.m % 32);
    const uint32_t mask = rem ? ((1u << rem) - 1u) : 0xffffffffu;
    const bool aligned = (reinterpret_cast<uintptr_t>(e.data) & 15) == 0 && ldw % 4 == 0;
    if (aligned && e.n <= 56) return launch_src(e, ldw, ex, SrcBits<4>{mask}, part, max_blocks, nblk, st);
    if (aligned) return launch_src(e, ldw, ex, SrcBits<2>{mask}, part, max_blocks, nblk, st);
    return launch_src(e, ldw, ex, SrcBits<1>{mask}, part, max_blocks, nblk, st);
  }
  if (iso_kind == PID_ISO_NONE && bytes_misaligned(e))
    return launch_src(e, e.ld, ex, SrcBytes{}, part, max_blocks, nblk, st);
  if (iso_kind == PID_ISO_NONE) return launch_src(e, e.ld, ex, SrcValues<uint8_t, false>{}, part, max_blocks, nblk, st);
  switch (e.dtype) {
    case PID_F64: return launch_src(e, e.ld, ex, SrcValues<double, true>{}, part, max_blocks, nblk, st);
    case PID_F32: return launch_src(e, e.ld, ex, SrcValues<float, true>{}, part, max_blocks, nblk, st);
    case PID_F16: return launch_src(e, e.ld, ex, SrcValues<f16, true>{}, part, max_blocks, nblk, st);
    case PID_BF16: return launch_src(e, e.ld, ex, SrcValues<bf16_t, true>{}, part, max_blocks, nblk, st);
    default: return launch_src(e, e.ld, ex, SrcValues<uint8_t, true>{}, part, max_blocks, nblk, st);
  }
}

}  // namespace pidk
