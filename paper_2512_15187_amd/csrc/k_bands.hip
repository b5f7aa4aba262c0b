// Contour-boxplot bands of a ranked ensemble (the pipeline of Sec. 1 and the
// boxplot views of Sec. 6 / 6.1): members binarised at a threshold; the
// median is the deepest member; the band of the k deepest members is bounded
// by the per-point union and intersection of their binarised masks.
//
// One streaming pass over the rows of the k_outer deepest members (gathered
// through `order`), HBM-bound: each lane owns one 16-byte chunk of points
// and keeps, per point, one bit in each of five 32-bit masks.  The decision
// u >= threshold is that of FP64 on the extracted value: stored values are
// compared in their own type with the smallest value of it at or above the
// threshold, which decides the same; isovalue models are evaluated in FP64.
// U8, 100 members on 128^3: 74 us with a branch around every load and FP64
// compares, 38 so (5.5 TB/s); whole calls, FP16
// 120 -> 79 us, FP32 rows that are not aligned, 60 members on 81^3, 46 -> 25 us.
#include "bits_source.h"
#include "device_common.h"
#include "pid_internal.h"
#include "pid_timing.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace pidk {

struct BandArgs {
  const void* U;
  int64_t ld;
  int n;
  int64_t m;
  const int32_t* order;
  int k_inner, k_outer;
  double thr;
  float thr_f;            // smallest float >= thr
  uint32_t thr_u8;        // (256 - t) in both halves, t = the smallest 0..256 >= thr
  uint8_t* out;
};

// Bit p: byte p of v >= the threshold (256 - t added to each byte carries into
// bit 8 exactly then).
__device__ __forceinline__ uint32_t ge_bytes(uint32_t v, uint32_t add) {
  const uint32_t e = (v & 0x00ff00ffu) + add, o = ((v >> 8) & 0x00ff00ffu) + add;
  return ((e >> 8) & 0x00010001u) | (o & 0x01000100u);
}

// The decision on one stored value.
template <int MODE, typename T>
__device__ __forceinline__ bool decide_point(T raw, const BandArgs& a, const Extract& ex) {
  if constexpr (MODE == MODE_NONE && sizeof(T) < 8) return to_float(raw) >= a.thr_f;
  else return extract_d<MODE>(raw, ex) >= a.thr;
}

// The decisions on a chunk, bit p for point p.
template <typename T, int MODE>
__device__ __forceinline__ uint32_t decide(const Vec16<T>& v, const BandArgs& a, const Extract& ex) {
  constexpr int P = 16 / (int)sizeof(T);
  if constexpr (MODE == MODE_NONE && sizeof(T) == 1) {
    const uint4 q = __builtin_bit_cast(uint4, v);
    return low_bits16(make_uint4(ge_bytes(q.x, a.thr_u8), ge_bytes(q.y, a.thr_u8), ge_bytes(q.z, a.thr_u8),
                                 ge_bytes(q.w, a.thr_u8)));
  } else {
    uint32_t b = 0u;
#pragma unroll
    for (int p = 0; p < P; ++p) b |= (decide_point<MODE>(v.v[p], a, ex) ? 1u : 0u) << p;
    return b;
  }
}

// members whose chunks are loaded together (fewer for 1- and 2-byte input,
// whose chunks carry more points to decide)
template <typename T>
constexpr int band_rows() { return sizeof(T) >= 4 ? 16 : 8; }

// A block covers the points of 64 lanes; its four waves take interleaved
// rounds of members (wave w: members 4r*UNR + w*UNR ... of round r) and meet
// in LDS, where the masks combine by OR / AND (exact, order-free).  A round's
// indices are one load, a round ahead (lane q holds the round's q-th; scalar
// loads are waited for one by one), and its rows' loads are issued together: entries past k_outer or outside 0..n-1 read row 0 and
// leave the masks as they are, and a chunk that reaches past m is read P points
// before m, its decisions shifted.  Rows of fewer than P points are read point by point,
// in a loop of their own.
template <typename T, int MODE>
__global__ __launch_bounds__(256) void bands_kernel(BandArgs a, Extract ex) {
  constexpr int P = 16 / (int)sizeof(T);   // points per lane
  constexpr int UNR = band_rows<T>();
  constexpr uint32_t ALL = (1u << P) - 1u;
  __shared__ uint32_t sh[4][6][64];
  const int lane = threadIdx.x & 63, wv = wave_id();
  const int64_t x0 = ((int64_t)blockIdx.x * 64 + lane) * P;
  const bool active = x0 < a.m;            // no early return: every wave reaches the barrier
  const int cnt = active ? (int)min((int64_t)P, a.m - x0) : 0;
  const int64_t xs = max((int64_t)0, min(x0, a.m - P));
  const int shift = active ? (int)(x0 - xs) : 0;
  const T* __restrict__ U = reinterpret_cast<const T*>(a.U);
  uint32_t med = 0, ui = 0, ii = ALL, uo = 0, io = ALL, bad = 0;
  auto see = [&](int j, uint32_t b) {
    if (j == 0) med = b;
    if (j < a.k_inner) { ui |= b; ii &= b; }
    uo |= b;
    io &= b;
  };
  if (a.m >= P) {
    auto entry = [&](int j0) { return a.order[min(j0 + (lane & (UNR - 1)), a.k_outer - 1)]; };
    int next = entry(wv * UNR);
    for (int j0 = wv * UNR; j0 < a.k_outer; j0 += 4 * UNR) {
      const int mine = next;
      Vec16<T> v[UNR];
      int idx[UNR];
#pragma unroll
      for (int q = 0; q < UNR; ++q) {
        const int k = __builtin_amdgcn_readlane(mine, q);
        const bool ok = (unsigned)k < (unsigned)a.n;
        if (!ok) bad = 1;                  // an index outside 0..n-1 is never read
        idx[q] = (ok && j0 + q < a.k_outer) ? k : -1;
        v[q] = load16_any(U + (int64_t)max(idx[q], 0) * a.ld + xs);
      }
      next = entry(j0 + 4 * UNR);
      asm volatile("" ::: "memory");       // (issued here, not sunk to where they are used)
#pragma unroll
      for (int q = 0; q < UNR; ++q) {
        if (idx[q] >= 0) see(j0 + q, decide<T, MODE>(v[q], a, ex) >> shift);   // (whole wave)
        // U8 through a model: 16 FP64 evaluations a chunk, one chunk at a time
        // (eight interleaved fill all registers: STEP, 53 members of 2.4M points,
        // a call 230 us, 71 with the loads under a branch each; the kernel takes
        // 47 so)
        if constexpr (MODE != MODE_NONE && sizeof(T) == 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    for (int j = wv; j < a.k_outer; j += 4) {
      const int k = __builtin_amdgcn_readfirstlane(a.order[j]);
      if ((unsigned)k >= (unsigned)a.n) {
        bad = 1;
        continue;
      }
      uint32_t b = 0u;
      for (int p = 0; p < (int)a.m; ++p) b |= (decide_point<MODE>(U[(int64_t)k * a.ld + p], a, ex) ? 1u : 0u) << p;
      see(j, b);
    }
  }
  sh[wv][0][lane] = med;
  sh[wv][1][lane] = ui;
  sh[wv][2][lane] = ii;
  sh[wv][3][lane] = uo;
  sh[wv][4][lane] = io;
  sh[wv][5][lane] = bad;
  __syncthreads();
  if (wv != 0 || !active) return;
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    med |= sh[w][0][lane];
    ui |= sh[w][1][lane];
    ii &= sh[w][2][lane];
    uo |= sh[w][3][lane];
    io &= sh[w][4][lane];
    bad |= sh[w][5][lane];
  }
  // the codes of four points as the bytes of a word: x * (1 + 2^7 + 2^14 + 2^21)
  // brings bit k of a nibble to bit 8 k
  auto spread = [](uint32_t nib) { return (nib * 0x00204081u) & 0x01010101u; };
  uint32_t word[(P + 3) / 4];
#pragma unroll
  for (int w = 0; w < (P + 3) / 4; ++w) {
    auto nib = [&](uint32_t mask) { return spread((mask >> (4 * w)) & 0xfu); };
    word[w] = nib(med) | (nib(ui) << 1) | (nib(ii) << 2) | (nib(uo) << 3) | (nib(io) << 4) |
              (bad ? 0x80808080u : 0u);
  }
  if (cnt == P) {
    __builtin_memcpy(a.out + x0, word, P);
  } else {
    // (constant indices: an indexed word[] is kept in LDS, whose address the compiler
    // takes from the dispatch packet in host memory: U8, 3 members of 899,491
    // points 15.3 us, 9.5 with byte stores)
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (p < cnt) a.out[x0 + p] = (uint8_t)(word[p / 4] >> (8 * (p % 4)));
  }
}

template <typename T>
static void launch_bands_t(const BandArgs& a, int kind, const Extract& ex, hipStream_t st) {
  constexpr int P = 16 / (int)sizeof(T);
  const int64_t lanes = (a.m + P - 1) / P;
  const unsigned grid = (unsigned)((lanes + 63) / 64);
  switch (kind) {
    case PID_ISO_GAUSSIAN: hipLaunchKernelGGL((bands_kernel<T, MODE_GAUSS>), grid, 256, 0, st, a, ex); break;
    case PID_ISO_STEP: hipLaunchKernelGGL((bands_kernel<T, MODE_STEP>), grid, 256, 0, st, a, ex); break;
    case PID_ISO_RAMP: case PID_ISO_TENT: case PID_ISO_DENSITY:
      if constexpr (sizeof(T) >= 2 && !std::is_same<T, bf16_t>::value)
        hipLaunchKernelGGL((bands_kernel<T, MODE_MODEL>), grid, 256, 0, st, a, ex);
      break;
    default: hipLaunchKernelGGL((bands_kernel<T, MODE_NONE>), grid, 256, 0, st, a, ex); break;
  }
}

hipError_t launch_bands(const pid_ensemble& e, int iso_kind, const ExtractHost& exh, const int32_t* order,
                        int64_t k_inner, int64_t k_outer, double threshold, uint8_t* out, hipStream_t st) {
  const Extract ex = __builtin_bit_cast(Extract, exh);
  BandArgs a{};
  a.U = e.data;
  a.ld = e.ld;
  a.n = (int)e.n;
  a.m = e.m;
  a.order = order;
  a.k_inner = (int)k_inner;
  a.k_outer = (int)k_outer;
  a.thr = threshold;
  a.thr_f = (float)threshold;
  if ((double)a.thr_f < threshold) a.thr_f = std::nextafter(a.thr_f, INFINITY);
  a.thr_u8 = (256u - (uint32_t)std::ceil(std::min(256.0, std::max(0.0, threshold)))) * 0x00010001u;
  a.out = out;
  KernelTimer tm("bands", st);
  switch (e.dtype) {
    case PID_F64: launch_bands_t<double>(a, iso_kind, ex, st); break;
    case PID_F32: launch_bands_t<float>(a, iso_kind, ex, st); break;
    case PID_F16: launch_bands_t<f16>(a, iso_kind, ex, st); break;
    case PID_BF16: launch_bands_t<bf16_t>(a, iso_kind, ex, st); break;
    default: launch_bands_t<uint8_t>(a, iso_kind, ex, st); break;
  }
  return hipGetLastError();
}

}  // namespace pidk
