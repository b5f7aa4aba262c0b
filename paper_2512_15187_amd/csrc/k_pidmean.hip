// PID-mean (Sec. 4.1) as one streaming pass over the ensemble.
//
// Both inclusions of PID-mean share the numerator
//     A_i = sum_x w_x u_i(x) s(x),   s(x) = sum_j u_j(x)   (= N * sum_x w u_i ubar),
// and the denominators are the masses m_i = sum_x w u_i and
// m(ubar) = (1/N) sum_k m_k.  Hence IN_in = A_i / (N m_i) and
// IN_out = A_i / sum_k m_k, and the ensemble has to be read once only: a
// workgroup owns a tile of points and all N members.  Each wave loads a slice
// of the members with 16-byte loads, applies the isovalue model in registers,
// and writes its partial column sums to LDS; after one barrier every lane holds
// s(x) for its points and accumulates m_i and A_i for the members it loaded.
// Per tile the sums are FP32 (FP64 for FP64 input), across tiles FP64.
// Per-workgroup partials are reduced in a fixed order by pidmean_reduce, and
// mean_finish_kernel forms the depths and ranks.  Binary input (U8 masks, thresholded
// values) takes the exact popcount passes of k_bits.hip instead.
#include "device_common.h"
#include <hip/hip_ext.h>
#include "mean_finish.h"
#include "pid_internal.h"
#include "pid_timing.h"

#include <algorithm>
#include <cstdlib>
#include <type_traits>

namespace pidk {

template <typename T>
using ComputeT = typename std::conditional<sizeof(T) == 8, double, float>::type;

// The piecewise-linear models (ramp, tent, density) are built for FP64, FP32
// and FP16 fields.
template <typename T>
constexpr bool has_models() {
  return std::is_same<T, double>::value || std::is_same<T, float>::value || std::is_same<T, f16>::value;
}

template <typename CT, typename T>
__device__ __forceinline__ CT to_ct(T raw) {
  if constexpr (std::is_same<CT, double>::value) return to_double(raw);
  else return to_float(raw);
}

template <int MODE, typename T, typename CT>
__device__ __forceinline__ CT extract_ct(T raw, const Extract& e) {
  if constexpr (std::is_same<CT, double>::value) return extract_d<MODE>(raw, e);
  else return extract_f<MODE, T, true>(raw, e);
}

// ---------------------------------------------------------------------------
// Soft path.  SFROM: column sums are read from `sglob` (two-pass mode) and the
// member range of this workgroup is blockIdx.y * nwaves * MPW + ...
// A workgroup handles at most a few tens of tiles, so per-lane FP32 sums stay
// short; lanes are combined in FP64.  Soft masks (MODE_NONE) keep only the
// raw 16-byte vectors in registers and widen them again in the second phase;
// fields keep the extracted probabilities.
// part layout: [2][n][grid.x] doubles (m, then A).
// Waves per SIMD that the registers have to allow: the row pass of thresholded
// fields would take 134 to 143 (three waves instead of four: FP32, n = 200 on
// 100,096 weighted points 59 -> 67 us).
template <typename T, int MODE, int MPW, bool SFROM>
constexpr int soft_waves() {
  return SFROM && MODE == MODE_STEP && (sizeof(T) == 4 || (sizeof(T) == 2 && MPW <= 8)) ? 4 : 1;
}

template <typename T, int MODE, int MPW, bool WEIGHTED, bool SFROM, int NWMAX>
__global__ __launch_bounds__(64 * NWMAX, (soft_waves<T, MODE, MPW, SFROM>())) void pidmean_soft_kernel(
    const T* __restrict__ U, int64_t ld, int n, int64_t m, const float* __restrict__ w,
    Extract ex, int64_t ntiles, const void* __restrict__ sglob, double* __restrict__ part) {
  using CT = ComputeT<T>;
  constexpr int PPL = Vec16<T>::N;
  constexpr int TP = 64 * PPL;
  constexpr bool KEEP_RAW = (MODE == MODE_NONE);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  CT* sbuf = reinterpret_cast<CT*>(smem_raw);
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int nw = blockDim.x >> 6;
  const int mbase = (SFROM ? blockIdx.y * nw * MPW : 0) + wave * MPW;

  CT accm[MPW], acca[MPW];
#pragma unroll
  for (int r = 0; r < MPW; ++r) { accm[r] = CT(0); acca[r] = CT(0); }

  int it = 0;
  // WHOLE: the tile lies inside the rows
  auto step = [&](int64_t tile, auto whole) {
    constexpr bool WHOLE = decltype(whole)::value;
    const int64_t x0 = tile * TP + (int64_t)lane * PPL;
    const bool full = WHOLE || (x0 + PPL <= m);
    // Every member's load is unconditional, so that they are all in flight
    // together (a load under a branch of its own is waited for before the
    // next one is issued); rows past n re-read row n - 1 and stay out of
    // the sums.  Vector loads at any row address, the ragged last tile's
    // shifted (rows shorter than a vector take guarded loads).  With element
    // loads where rows are not 16-byte aligned, PID-mean of FP16 n = 64 on
    // 201^3 took 502 us; now 211 (4.9 TB/s).
    const bool fast = WHOLE || (tile + 1) * TP <= m;
    // (Up to 32 FP64 members not non-temporal: tiles of unaligned rows share lines.
    // mean_weighted of n = 13 on rows of 3,644,944 points, 8-byte aligned, 168 -> 155
    // us; of n = 40 on 1,000,000 aligned points 112 -> 120.)
    auto load = [](const T* row) { return sizeof(T) == 8 && MPW == 4 ? load16_any(row) : load16_nt_any(row); };
    Vec16<T> vv[MPW];
    if (fast) {
#pragma unroll
      for (int r = 0; r < MPW; ++r) vv[r] = load(U + (int64_t)min(mbase + r, n - 1) * ld + x0);
    } else if (m >= PPL) {
      const TailLoad<T> tail(x0, m);
#pragma unroll
      for (int r = 0; r < MPW; ++r) vv[r] = tail(U + (int64_t)min(mbase + r, n - 1) * ld);
    } else {
#pragma unroll
      for (int r = 0; r < MPW; ++r) {
        Vec16<T> v{};
        if (mbase + r < n) v = load16_guarded(U + (int64_t)(mbase + r) * ld, x0, m);
        vv[r] = v;
      }
    }
    Vec16<T> raw[KEEP_RAW ? MPW : 1];
    CT u[KEEP_RAW ? 1 : MPW][PPL];
    CT sp[PPL];
#pragma unroll
    for (int p = 0; p < PPL; ++p) sp[p] = CT(0);
#pragma unroll
    for (int r = 0; r < MPW; ++r) {
      const bool rv = mbase + r < n;   // (rows past n: their sums are never written)
      if constexpr (KEEP_RAW) {
        raw[r] = vv[r];
        if (rv) {
#pragma unroll
          for (int p = 0; p < PPL; ++p) sp[p] += extract_ct<MODE, T, CT>(vv[r].v[p], ex);
        }
      } else {
#pragma unroll
        for (int p = 0; p < PPL; ++p) {
          CT val = rv ? extract_ct<MODE, T, CT>(vv[r].v[p], ex) : CT(0);
          if (!full) val = (x0 + p < m) ? val : CT(0);
          u[r][p] = val;
          sp[p] += val;
        }
      }
    }

    if constexpr (KEEP_RAW) {
#pragma unroll
      for (int r = 0; r < MPW; ++r) opaque(raw[r]);   // widen again in phase 2
    }
    CT s[PPL];
    if constexpr (SFROM) {
      const CT* sg = reinterpret_cast<const CT*>(sglob);
      if (fast) {   // PPL values, a multiple of 16 bytes at a 16-byte boundary
        static_assert((PPL * sizeof(CT)) % 16 == 0, "whole 16-byte loads");
#pragma unroll
        for (int q = 0; q < (int)(PPL * sizeof(CT) / 16); ++q) {
          const uint4 t = *reinterpret_cast<const uint4*>(sg + x0 + q * (16 / sizeof(CT)));
          __builtin_memcpy(&s[q * (16 / sizeof(CT))], &t, 16);
        }
      } else {
#pragma unroll
        for (int p = 0; p < PPL; ++p) {
          const CT t = sg[min(x0 + p, m - 1)];
          s[p] = (x0 + p < m) ? t : CT(0);
        }
      }
    } else {
      CT* sb = sbuf + (size_t)(it & 1) * nw * TP;
#pragma unroll
      for (int p = 0; p < PPL; ++p) sb[wave * TP + lane * PPL + p] = sp[p];
      lds_barrier();
#pragma unroll
      for (int p = 0; p < PPL; ++p) s[p] = CT(0);
      for (int q = 0; q < nw; ++q) {
#pragma unroll
        for (int p = 0; p < PPL; ++p) s[p] += sb[q * TP + lane * PPL + p];
      }
    }

    CT wv[PPL];
    if constexpr (WEIGHTED) {
      if (PPL >= 4 && fast) {
#pragma unroll
        for (int p = 0; p < PPL; p += 4) {
          const f32x4_a4 t = *reinterpret_cast<const f32x4_a4*>(w + x0 + p);
          wv[p] = t.x; if (p + 1 < PPL) wv[p + 1] = t.y;
          if (p + 2 < PPL) wv[p + 2] = t.z; if (p + 3 < PPL) wv[p + 3] = t.w;
        }
      } else {
#pragma unroll
        for (int p = 0; p < PPL; ++p) {
          const CT t = CT(w[min(x0 + p, m - 1)]);
          wv[p] = (x0 + p < m) ? t : CT(0);
        }
      }
#pragma unroll
      for (int p = 0; p < PPL; ++p) s[p] *= wv[p];      // s now holds w * s
    }
#pragma unroll
    for (int r = 0; r < MPW; ++r) {
      CT tm = CT(0), ta = CT(0);
#pragma unroll
      for (int p = 0; p < PPL; ++p) {
        CT uv;
        if constexpr (KEEP_RAW) uv = extract_ct<MODE, T, CT>(raw[r].v[p], ex);
        else uv = u[r][p];
        tm += WEIGHTED ? wv[p] * uv : uv;
        ta += s[p] * uv;
      }
      accm[r] += tm;
      acca[r] += ta;
    }
    ++it;
  };
  if constexpr (!SFROM || sizeof(T) == 1) {
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) step(tile, std::false_type());
  } else {
    const int64_t nfull = m / TP;
    for (int64_t tile = blockIdx.x; tile < nfull; tile += gridDim.x) step(tile, std::true_type());
    // The ragged tile (the last of its workgroup), two members at a time: no sums
    // meet here, so nothing else has to stay in registers.  (In one body with the
    // whole tiles its loads and shifts are the kernel's registers, and the loaded
    // values, coming from two branches, are copied as they arrive: the weighted
    // FP32 row pass took 129, three waves per SIMD, mean_weighted of n = 33 on 3.5M
    // points 204 us; 190 so.)
    constexpr int NQ = 2;
    auto ragged = [&](auto shortc) {
      const int64_t x0 = nfull * TP + (int64_t)lane * PPL;
      const CT* sg = reinterpret_cast<const CT*>(sglob);
      CT s[PPL], wv[PPL];
#pragma unroll
      for (int p = 0; p < PPL; ++p) {
        const int64_t x = min(x0 + p, m - 1);
        const CT ts = sg[x], tw = WEIGHTED ? CT(w[x]) : CT(1);
        wv[p] = (x0 + p < m) ? tw : CT(0);
        s[p] = (x0 + p < m) ? (WEIGHTED ? ts * tw : ts) : CT(0);
      }
#pragma unroll
      for (int r0 = 0; r0 < MPW; r0 += NQ) {
        Vec16<T> v[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const T* row = U + (int64_t)min(mbase + r0 + q, n - 1) * ld;
          if constexpr (decltype(shortc)::value) v[q] = load16_guarded(row, x0, m);
          else v[q] = TailLoad<T>(x0, m)(row);
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          CT tm = CT(0), ta = CT(0);
#pragma unroll
          for (int p = 0; p < PPL; ++p) {
            CT uv = extract_ct<MODE, T, CT>(v[q].v[p], ex);
            if constexpr (!KEEP_RAW) uv = (x0 + p < m) ? uv : CT(0);
            tm += WEIGHTED ? wv[p] * uv : uv;
            ta += s[p] * uv;
          }
          accm[r0 + q] += tm;
          acca[r0 + q] += ta;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (nfull < ntiles && blockIdx.x == (unsigned)(nfull % gridDim.x)) {
      if (m >= PPL) ragged(std::false_type());
      else ragged(std::true_type());   // (rows shorter than a vector)
    }
  }

  const int ng = gridDim.x;
#pragma unroll
  for (int r = 0; r < MPW; ++r) {
    const double a = wave_sum((double)accm[r]);
    const double b = wave_sum((double)acca[r]);
    const int i = mbase + r;
    if (lane == 0 && i < n) {
      part[(size_t)i * ng + blockIdx.x] = a;
      part[((size_t)n + i) * ng + blockIdx.x] = b;
    }
  }
}

// ---------------------------------------------------------------------------
// Pipelined soft path (rows aligned to LB bytes, N <= NWMAX * MPW): the same sums
// as pidmean_soft_kernel, with a register double buffer.  Workgroup b takes
// the full tiles b, b + G, b + 2G, ... (G = grid); while one tile's column
// sums go through LDS and its members' sums are accumulated, the loads of
// the next tile are in flight.  The loop runs over pairs of tiles with no
// branch around a load, so the compiler's wait counts keep the other buffer
// outstanding: a tile past the workgroup's last one is read with an offset
// beyond the buffer's range, which the hardware answers with zeros and no
// memory access, and it adds nothing.  Rows past n re-read the wave's last
// row, and their copies are taken off the column sum.  The ragged last tile
// is taken afterwards, with guarded loads, by the workgroup it falls to.
// Soft masks keep the raw vectors and widen them twice; fields keep the
// extracted probabilities.
// part layout: [2][n][grid] doubles (m, then A).
template <typename T, int MODE, int MPW, int LB, bool WEIGHTED, int NWMAX>
__global__ __launch_bounds__(64 * NWMAX) void pidmean_pipe_kernel(
    const T* __restrict__ U, int64_t ld, int n, int64_t m, const float* __restrict__ w,
    Extract ex, double* __restrict__ part) {
  using CT = ComputeT<T>;
  using V = VecB<T, LB>;
  constexpr int PPL = V::N;
  constexpr int TP = 64 * PPL;
  constexpr bool KEEP_RAW = (MODE == MODE_NONE);
  constexpr uint32_t OOB = 0x80000000u;   // beyond every buffer range used here
  extern __shared__ __align__(16) unsigned char smem_raw[];
  CT* sbuf = reinterpret_cast<CT*>(smem_raw);
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int nw = blockDim.x >> 6;
  const int mbase = wave * MPW;
  const int G = gridDim.x;
  const int b = blockIdx.x;
  const int64_t nfull = m / TP;
  const int64_t K = (nfull > b) ? (nfull - 1 - b) / G + 1 : 0;   // full tiles of this workgroup

  // One buffer resource per wave, based at its first row; row r sits at
  // scalar offset min(r, rl) * ld, the points at a 32-bit per-lane offset.
  // The host has checked that every offset fits in 31 bits.
  const int rl = min(n - 1, mbase + MPW - 1) - mbase;            // last valid row of the wave
  const CT dup = (CT)(MPW - 1 - rl);                               // copies of row rl beyond it
  const __amdgpu_buffer_rsrc_t rsU = buffer_rsrc(
      U + (int64_t)mbase * ld, (uint32_t)(((int64_t)rl * ld + m) * (int64_t)sizeof(T)));
  const __amdgpu_buffer_rsrc_t rsW = buffer_rsrc(w, (uint32_t)(m * (int64_t)sizeof(float)));
  const uint32_t ldb0 = (uint32_t)(ld * (int64_t)sizeof(T));     // row stride in bytes
  const uint32_t xb = (uint32_t)b * TP + (uint32_t)(lane * PPL);
  const uint32_t xg = (uint32_t)G * TP;

  V bufA[MPW], bufB[MPW];
  float wA[WEIGHTED ? PPL : 1], wB[WEIGHTED ? PPL : 1];
  auto load_tile = [&](V* buf, float* wb, int64_t k) {
    const bool ok = k < K;
    const uint32_t x = xb + (uint32_t)k * xg;
    const uint32_t vo = ok ? x * (uint32_t)sizeof(T) : OOB;
    // row offsets recomputed per tile (a scalar multiply each) rather than
    // kept in scalar registers across the loop
    uint32_t ldb = ldb0;
    asm volatile("" : "+s"(ldb));
#pragma unroll
    for (int r = 0; r < MPW; ++r) buf[r] = bufload_nt<T, LB>(rsU, vo, (uint32_t)min(r, rl) * ldb);
    if constexpr (WEIGHTED) {
      // wave 0 reads the tile's weights (shared through LDS); the other
      // waves issue the same loads past the buffer's end (no memory access,
      // the same instructions, so the wait counts stay the same)
      constexpr int WB = PPL * 4 < 16 ? PPL * 4 : 16;   // bytes per weight load
      const uint32_t wo = (ok && wave == 0) ? x * 4u : OOB;
#pragma unroll
      for (int o = 0; o < PPL; o += WB / 4) {
        const VecB<float, WB> t = bufload_nt<float, WB>(rsW, wo + 4u * o, 0u);
#pragma unroll
        for (int p = 0; p < WB / 4; ++p) wb[o + p] = t.v[p];
      }
    }
  };

  // Per-lane sums run over at most 16 tiles; then each wave folds them
  // (fixed butterfly) into FP64 accumulators of its members in LDS, placed
  // after the two column-sum halves.  Lane 0 owns the wave's accumulators.
  CT accm[MPW], acca[MPW];
#pragma unroll
  for (int r = 0; r < MPW; ++r) { accm[r] = CT(0); acca[r] = CT(0); }
  double* lacc = reinterpret_cast<double*>(sbuf + (size_t)2 * nw * TP) + (size_t)wave * MPW * 2;
  float* wsh = reinterpret_cast<float*>(reinterpret_cast<double*>(sbuf + (size_t)2 * nw * TP) + (size_t)nw * MPW * 2);
                                                          // [2][TP] weights of the tile (wave 0's loads)
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < 2 * MPW; ++r) lacc[r] = 0.0;
  }
  auto fold = [&]() {
#pragma unroll
    for (int r = 0; r < MPW; ++r) {
      const CT a = wave_sum(accm[r]);
      const CT c = wave_sum(acca[r]);
      if (lane == 0) { lacc[2 * r] += (double)a; lacc[2 * r + 1] += (double)c; }
      accm[r] = CT(0);
      acca[r] = CT(0);
    }
  };

  // One tile: column sums of the wave's members -> LDS half `parity`; after
  // the barrier every lane adds the NW partials for its points (fixed order)
  // and accumulates m_i and A_i of its members.  tv[p] = 0 marks a point past
  // the end (its raw value reads as zero; fields would turn it into
  // Phi(-c/sigma)); soft masks need no factor.
  auto process = [&](V* buf, const float* wb, int parity, const CT* tv) {
    CT u[KEEP_RAW ? 1 : MPW][PPL];
    CT sp[PPL];
#pragma unroll
    for (int p = 0; p < PPL; ++p) sp[p] = CT(0);
#pragma unroll
    for (int r = 0; r < MPW; ++r) {
#pragma unroll
      for (int p = 0; p < PPL; ++p) {
        CT val = extract_ct<MODE, T, CT>(buf[r].v[p], ex);
        if constexpr (!KEEP_RAW) { val *= tv[p]; u[r][p] = val; }
        sp[p] += val;
      }
    }
    // take off the copies of row rl read for rows past n
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      CT last;
      if constexpr (KEEP_RAW) last = extract_ct<MODE, T, CT>(buf[MPW - 1].v[p], ex);
      else last = u[MPW - 1][p];
      sp[p] -= dup * last;
    }
    if constexpr (KEEP_RAW) {
#pragma unroll
      for (int r = 0; r < MPW; ++r) opaque(buf[r]);   // widen again below
    }
    CT* sb = sbuf + (size_t)parity * nw * TP;
#pragma unroll
    for (int p = 0; p < PPL; ++p) sb[wave * TP + lane * PPL + p] = sp[p];
    if constexpr (WEIGHTED) {
      if (wave == 0) {
#pragma unroll
        for (int p = 0; p < PPL; ++p) wsh[(size_t)parity * TP + lane * PPL + p] = wb[p];
      }
    }
    lds_barrier();
    float wl[WEIGHTED ? PPL : 1];
    if constexpr (WEIGHTED) {
#pragma unroll
      for (int p = 0; p < PPL; ++p) wl[p] = wsh[(size_t)parity * TP + lane * PPL + p];
    }
    CT s[PPL];
#pragma unroll
    for (int p = 0; p < PPL; ++p) s[p] = CT(0);
    for (int q = 0; q < nw; ++q) {
#pragma unroll
      for (int p = 0; p < PPL; ++p) s[p] += sb[q * TP + lane * PPL + p];
    }
    if constexpr (WEIGHTED) {
#pragma unroll
      for (int p = 0; p < PPL; ++p) s[p] *= (CT)wl[p];   // s now holds w * s
    }
#pragma unroll
    for (int r = 0; r < MPW; ++r) {
      CT tm = CT(0), ta = CT(0);
#pragma unroll
      for (int p = 0; p < PPL; ++p) {
        CT uv;
        if constexpr (KEEP_RAW) uv = extract_ct<MODE, T, CT>(buf[r].v[p], ex);
        else uv = u[r][p];
        if constexpr (WEIGHTED) tm += (CT)wl[p] * uv;
        else tm += uv;
        ta += s[p] * uv;
      }
      accm[r] += tm;
      acca[r] += ta;
    }
  };

  // pairs of tiles; when K is odd the second tile of the last pair is past
  // the end and adds zeros
  load_tile(bufA, wA, 0);
  __builtin_amdgcn_sched_barrier(0);   // prologue loads in the loop's order (A, then B)
  load_tile(bufB, wB, 1);
  for (int64_t k = 0; k < K; k += 2) {
    CT one[PPL], second[PPL];
#pragma unroll
    for (int p = 0; p < PPL; ++p) { one[p] = CT(1); second[p] = (k + 1 < K) ? CT(1) : CT(0); }
    process(bufA, wA, 0, one);
    load_tile(bufA, wA, k + 2);
    process(bufB, wB, 1, second);
    load_tile(bufB, wB, k + 3);
    if ((k & 15) == 14 && k + 2 < K) fold();   // every 16 tiles, if more follow
  }
  // ragged last tile (LDS half 0 follows the loop's last tile, which used 1)
  if ((m % TP) != 0 && b == (int)(nfull % G)) {
    const int64_t x0 = nfull * TP + (int64_t)lane * PPL;
#pragma unroll
    for (int r = 0; r < MPW; ++r)
      bufA[r] = loadB_guarded<T, LB>(U + (int64_t)(mbase + min(r, rl)) * ld, x0, m);
    if constexpr (WEIGHTED) {
#pragma unroll
      for (int p = 0; p < PPL; ++p) wA[p] = w[(x0 + p < m) ? x0 + p : m - 1] * ((x0 + p < m) ? 1.0f : 0.0f);
    }
    CT pf[PPL];   // entries past m add nothing (fields would map 0 to Phi(-c/sigma))
#pragma unroll
    for (int p = 0; p < PPL; ++p) pf[p] = (x0 + p < m) ? CT(1) : CT(0);
    process(bufA, wA, 0, pf);
  }

  fold();
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < MPW; ++r) {
      const int i = mbase + r;
      if (i < n) {
        part[(size_t)i * G + b] = lacc[2 * r];
        part[((size_t)n + i) * G + b] = lacc[2 * r + 1];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// DMA-staged soft path (soft masks; rows 16-byte aligned, M * sizeof(T) a
// multiple of 16, N <= 8 * RPW).  Tiles hold TPP = 128 / sizeof(T) points of
// every row.  Each wave owns RPW rows and streams its 128-byte row segments of
// each tile straight into a ring of NBUF LDS slots (16 bytes per lane, eight
// rows per instruction), so NBUF - 1 tiles are in flight without holding
// registers, and no other wave reads them.  Per tile, a lane reads its point
// of the wave's rows from LDS for the wave's column sums, which go through
// LDS (one barrier), and again for m_i and A_i.  Loads of tiles past the
// workgroup's share, of rows past N and of points past M use an offset
// beyond the buffer's range: they write zeros and read no memory, so the
// loop has no branch around a load and the wait counts are constants.
// Lane sums run over at most 16 tiles and are then folded (fixed butterfly)
// into FP64 accumulators in LDS.  part layout: [2][n][grid] doubles.
template <typename T, bool WEIGHTED, int RPW, int NBUF>
__global__ __launch_bounds__(512) void pidmean_dma_kernel(
    const T* __restrict__ U, int64_t ld, int n, int64_t m, const float* __restrict__ w,
    double* __restrict__ part) {
  using CT = ComputeT<T>;
  constexpr int SEG = 128;                  // bytes of a row per tile
  constexpr int TPP = SEG / (int)sizeof(T); // points per tile
  constexpr int LPP = 64 / TPP;             // lanes per point
  constexpr int RPL = RPW / LPP;            // rows per lane
  constexpr int RPI = 64 * 16 / SEG;        // rows per load instruction (8)
  constexpr int DPT = RPW / RPI + (WEIGHTED ? 1 : 0);   // load instructions per tile and wave
  constexpr uint32_t OOB = 0x80000000u;
  static_assert(RPW % RPI == 0 && RPW % LPP == 0, "row split");
  static_assert((NBUF - 2) * DPT <= 63, "wait count");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int nw = blockDim.x >> 6;
  const int mbase = wave * RPW;
  const int nrows = min(RPW, n - mbase);    // valid rows of this wave (>= 1)
  const int G = gridDim.x;
  const int b = blockIdx.x;
  const int64_t ntiles = (m + TPP - 1) / TPP;
  const int64_t K = (ntiles > b) ? (ntiles - 1 - b) / G + 1 : 0;

  // LDS: raw ring [NBUF][nw][RPW][SEG], weights [NBUF][nw][64] floats,
  // column-sum partials [2][nw][TPP], FP64 accumulators [nw][RPW][2]
  unsigned char* raw = smem_raw;
  float* wts = reinterpret_cast<float*>(raw + (size_t)NBUF * nw * RPW * SEG);
  CT* psum = reinterpret_cast<CT*>(wts + (WEIGHTED ? (size_t)NBUF * nw * 64 : 0));
  double* lacc = reinterpret_cast<double*>(psum + (size_t)2 * nw * TPP) + (size_t)wave * RPW * 2;
  auto slot_raw = [&](int64_t k) -> unsigned char* {
    return raw + ((size_t)(k % NBUF) * nw + wave) * RPW * SEG;
  };
  auto slot_w = [&](int64_t k) -> float* { return wts + ((size_t)(k % NBUF) * nw + wave) * 64; };

  // resources based at the wave's first row; the host has checked that all
  // offsets stay below 2^31
  const BufRes rsU = make_bufres(U + (int64_t)mbase * ld, (uint32_t)(((int64_t)(nrows - 1) * ld + m) * (int64_t)sizeof(T)));
  const BufRes rsW = make_bufres(w, (uint32_t)(m * (int64_t)sizeof(float)));
  const uint32_t ldb = (uint32_t)(ld * (int64_t)sizeof(T));
  const int lrow = lane >> 3;               // row within a load instruction
  const uint32_t lbyte = (uint32_t)(lane & 7) * 16u;

  auto issue = [&](int64_t k) {
    const int64_t t = b + k * G;
    const bool tok = k < K;
    const uint32_t xb = (uint32_t)(t * SEG) + lbyte;                  // byte of the point in a row
    const bool pok = tok && (int64_t)(t * TPP) + (lane & 7) * (16 / (int)sizeof(T)) < m;
    unsigned char* dst = slot_raw(k);
#pragma unroll
    for (int j = 0; j < RPW / RPI; ++j) {
      const int r = j * RPI + lrow;
      const uint32_t vo = (pok && r < nrows) ? (uint32_t)r * ldb + xb : OOB;
      dma_to_lds<16>(rsU, dst + (size_t)j * RPI * SEG, vo);
    }
    if constexpr (WEIGHTED) {
      const int64_t x = t * TPP + lane;
      const uint32_t vo = (tok && lane < TPP && x < m) ? (uint32_t)(x * 4) : OOB;
      dma_to_lds<4>(rsW, slot_w(k), vo);
    }
  };

  CT accm[RPL], acca[RPL];
#pragma unroll
  for (int i = 0; i < RPL; ++i) { accm[i] = CT(0); acca[i] = CT(0); }
  if (lane == 0) {
    for (int r = 0; r < 2 * RPW; ++r) lacc[r] = 0.0;
  }
  const int pt = lane % TPP;                // this lane's point in a tile
  const int hr = lane / TPP;                // and its first row
  // members of a lane: rows hr + LPP * i; fold the TPP lanes of each row
  auto fold = [&]() {
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      CT a = accm[i], c = acca[i];
#pragma unroll
      for (int o = TPP / 2; o >= 1; o >>= 1) { a += __shfl_xor(a, o, 64); c += __shfl_xor(c, o, 64); }
      if (pt == 0) {
        const int r = hr + LPP * i;
        lacc[2 * r] += (double)a;
        lacc[2 * r + 1] += (double)c;
      }
      accm[i] = CT(0);
      acca[i] = CT(0);
    }
  };

#pragma unroll
  for (int k = 0; k < NBUF - 1; ++k) issue(k);
  for (int64_t k = 0; k < K; ++k) {
    vm_wait<(NBUF - 2) * DPT>();            // this wave's loads of tile k have landed
    const unsigned char* rt = slot_raw(k);
    const int64_t x = (b + k * G) * TPP + pt;
    const bool pv = x < m;
    CT sp = CT(0);
#pragma unroll
    for (int i = 0; i < RPL; ++i)
      sp += to_ct<CT>(*reinterpret_cast<const T*>(rt + (size_t)(hr + LPP * i) * SEG + (size_t)pt * sizeof(T)));
    // the wave's rows (lanes pt, pt + TPP, ...)
    if constexpr (std::is_same<CT, float>::value) {
      sp = sum_from<TPP>(sp);
    } else {
#pragma unroll
      for (int o = TPP; o < 64; o <<= 1) sp += __shfl_xor(sp, o, 64);
    }
    CT* ps = psum + (size_t)(k & 1) * nw * TPP;
    if (hr == 0) ps[wave * TPP + pt] = pv ? sp : CT(0);
    lds_barrier();
    issue(k + NBUF - 1);                    // into the slot this wave finished with
    CT s = CT(0);
    for (int q = 0; q < nw; ++q) s += ps[q * TPP + pt];
    CT wv = CT(1);
    if constexpr (WEIGHTED) { wv = pv ? (CT)slot_w(k)[pt] : CT(0); s *= wv; }
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      CT u = to_ct<CT>(*reinterpret_cast<const T*>(rt + (size_t)(hr + LPP * i) * SEG + (size_t)pt * sizeof(T)));
      u = pv ? u : CT(0);
      accm[i] += WEIGHTED ? wv * u : u;
      acca[i] += s * u;
    }
    if ((k & 15) == 15 && k + 1 < K) fold();
  }
  fold();
  vm_wait<0>();                             // no load into LDS outlives the workgroup
  if (lane == 0) {
    for (int r = 0; r < nrows; ++r) {
      part[(size_t)(mbase + r) * G + b] = lacc[2 * r];
      part[((size_t)n + mbase + r) * G + b] = lacc[2 * r + 1];
    }
  }
}

// ---------------------------------------------------------------------------
// Column sums over the members for the two-pass cases: s(x) = sum_j u_j(x)
// and, for all-pairs depths without the matrix, t(x) = sum_j coef_j u_j(x).
// Block (bx, g) owns 64 * PPL points (16 bytes of every row per lane) and the
// members [g chunk, (g + 1) chunk); its 4 waves take the members q, q + 4, ...
// of that range in ascending order, four rows in flight, and add their sums
// in order q = 0..3; the member groups' sums are added in order g = 0, 1, ...
// by colsum_combine.
template <typename T, int MODE, bool SCALED>
__global__ __launch_bounds__(256) void colsum_part_kernel(const T* __restrict__ U, int64_t ld, int n, int64_t m,
                                                          Extract ex, const ComputeT<T>* __restrict__ coef,
                                                          int chunk, void* __restrict__ part_v) {
  using CT = ComputeT<T>;
  using AT = CT;
  constexpr int PPL = Vec16<T>::N;
  __shared__ AT part[4][64 * PPL];
  const int lane = threadIdx.x & 63;
  const int q = threadIdx.x >> 6;
  const int64_t x0 = (int64_t)blockIdx.x * (64 * PPL) + (int64_t)lane * PPL;
  const int i0 = blockIdx.y * chunk, i1 = min(n, i0 + chunk);
  AT t[PPL];
#pragma unroll
  for (int p = 0; p < PPL; ++p) t[p] = AT(0);
  auto add = [&](int i, const Vec16<T>& v) {
    const CT c = SCALED ? coef[i] : CT(1);
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      const CT u = extract_ct<MODE, T, CT>(v.v[p], ex);
      t[p] += SCALED ? c * u : u;
    }
  };
  // vector loads of four rows in flight, at any row address; the ragged last
  // tile's are shifted, and rows shorter than a vector take element loads, one row
  // at a time (with four, their registers are the kernel's: 16-bit input 49 -> 96,
  // five waves per SIMD instead of eight)
  auto sum = [&](auto rows, auto load) {
    int i = i0 + q;
    if constexpr (decltype(rows)::value == 4) {
      for (; i + 12 < i1; i += 16) {
        const Vec16<T> a0 = load(i), a1 = load(i + 4), a2 = load(i + 8), a3 = load(i + 12);
        add(i, a0); add(i + 4, a1); add(i + 8, a2); add(i + 12, a3);
      }
    }
    for (; i < i1; i += 4) add(i, load(i));
  };
  constexpr std::integral_constant<int, 1> one;
  constexpr std::integral_constant<int, 4> four;
  if ((int64_t)(blockIdx.x + 1) * (64 * PPL) <= m) {
    sum(four, [&](int i) { return load16_nt_any(U + (int64_t)i * ld + x0); });
  } else if (m >= PPL) {
    const TailLoad<T> tail(x0, m);
    sum(one, [&](int i) { return tail(U + (int64_t)i * ld); });
  } else {
    sum(one, [&](int i) { return load16_guarded(U + (int64_t)i * ld, x0, m); });
  }
#pragma unroll
  for (int p = 0; p < PPL; ++p) part[q][lane * PPL + p] = t[p];
  __syncthreads();
  AT* out = reinterpret_cast<AT*>(part_v) + (size_t)blockIdx.y * m;
  for (int e = threadIdx.x; e < 64 * PPL; e += 256) {
    const int64_t x = (int64_t)blockIdx.x * (64 * PPL) + e;
    if (x < m) out[x] = ((part[0][e] + part[1][e]) + part[2][e]) + part[3][e];
  }
}

template <typename AT>
__global__ __launch_bounds__(256) void colsum_combine(const AT* __restrict__ part, int groups, int64_t m,
                                                      AT* __restrict__ out) {
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < m; x += (int64_t)gridDim.x * blockDim.x) {
    AT s = part[x];
    for (int g = 1; g < groups; ++g) s += part[(size_t)g * m + x];
    out[x] = s;
  }
}

// ---------------------------------------------------------------------------
// Fixed-order reduction of the per-workgroup partials: one block per member
// and quantity (grid.y = 2: m, then A); thread t sums the partials
// t, t+256, ... in ascending order, then a fixed tree over the 256 threads.
__global__ __launch_bounds__(256) void pidmean_reduce(const double* __restrict__ part, int nparts, int n,
                                                      double* __restrict__ out) {
  __shared__ double red[256];
  const int i = blockIdx.x, q = blockIdx.y, t = threadIdx.x;
  const size_t base = ((size_t)q * n + i) * nparts;
  double s = 0.0;
  for (int b = t; b < nparts; b += 256) s += part[base + b];
  red[t] = s;
  __syncthreads();
  for (int o = 128; o >= 1; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  if (t == 0) out[(size_t)q * n + i] = red[0];
}

// ---------------------------------------------------------------------------
// All-pairs depths in O(N M) (no inclusion matrix).  With G_ji = sum_x w u_j u_i
// (Sec. 3.2 / 3.4),
//   IN_out(i) = (1/N) sum_j G_ji / m_j = (1/N) sum_x w u_i(x) t(x),
//   t(x) = sum_j u_j(x) / m_j   (terms with m_j = 0 are 0),
// so IN_out needs one column sum weighted by the inverse masses and one row
// dot product; IN_in(i) = S_i / (N m_i) is the PID-mean IN_in (Sec. 4.1).

// Inverse masses (0 for m = 0) in the compute type of the passes.
template <typename CT>
__global__ __launch_bounds__(256) void inv_mass_kernel(const double* __restrict__ mass, int n,
                                                       CT* __restrict__ coef) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) coef[i] = mass[i] > 0.0 ? (CT)(1.0 / mass[i]) : CT(0);
}

// red = [m (n), B (n)] with B_i = sum_x w u_i t; in_in from the PID-mean pass.
__global__ __launch_bounds__(256) void pairs_linear_ratios(const double* __restrict__ red,
                                                           const double* __restrict__ in_in_pm, int n,
                                                           double* __restrict__ m_out, double* __restrict__ in_in,
                                                           double* __restrict__ in_out, double* __restrict__ depth) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double ii = in_in_pm[i];
  const double oo = red[n + i] / (double)n;
  if (m_out) m_out[i] = red[i];
  if (in_in) in_in[i] = ii;
  if (in_out) in_out[i] = oo;
  if (depth) depth[i] = ii < oo ? ii : oo;
}

// ---------------------------------------------------------------------------
// The same in three passes over the data where PID-mean takes two (large N):
// the masses come out of the column-sum pass, and both row sums, A_i = sum_x w
// u_i s and B_i = sum_x w u_i t, out of one row pass.  Every FP32 chain is that
// of the kernels above (column sums: colsum_part_kernel; per-lane sums over
// the tiles b, b + G, ... of a row workgroup: pidmean_soft_kernel), so the
// results are the same bit for bit.  Seven launches instead of
// twelve.  FP16 n = 2048 on 256^2 (268 MB): 219 -> 169 us a call, of
// which 59, 42 and 48 us are the passes (this first one has only 1024 waves
// there: the tiles of a lane's chain cannot be split), 28 us the small
// launches; n = 400 on 400^2 134 -> 97, FP32 n = 700 on 512^2 504 -> 401.

// Column sums s and masses.  Block (b, g): the tiles b, b + G, ... (G =
// gridDim.x, the row pass's grid) of the members [g chunk, (g + 1) chunk);
// wave q takes the members q, q + 4, ... and keeps their lanes' sums over the
// tiles in LDS.  Eight rows are added while the next eight (of this tile or
// the next) are in flight, at any row address; a ragged last tile is read by
// shifted loads (m >= Vec16<T>::N).
template <typename T, bool WEIGHTED>
__global__ __launch_bounds__(256) void colsum_mass_kernel(const T* __restrict__ U, int64_t ld, int n, int64_t m,
                                                          const float* __restrict__ w, int chunk, int64_t ntiles,
                                                          ComputeT<T>* __restrict__ out_v,
                                                          double* __restrict__ mpart) {
  using CT = ComputeT<T>;
  constexpr int PPL = Vec16<T>::N, TP = 64 * PPL, R = 8;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  CT* part = reinterpret_cast<CT*>(smem_raw);                     // [2][4][TP]
  const int lane = threadIdx.x & 63;
  const int q = wave_id();
  const int i0 = blockIdx.y * chunk, i1 = min(n, i0 + chunk);
  const int nm = max(0, (i1 - i0 - q + 3) / 4);                   // members of this wave
  const int nk = max(1, (nm + R - 1) / R);                        // steps of a tile
  CT* acc = part + 8 * TP + (size_t)q * (((chunk + 3) / 4 + R - 1) / R * R) * 64 + lane;
  for (int k = 0; k < nk * R; ++k) acc[k * 64] = CT(0);
  CT* out = out_v + (size_t)blockIdx.y * m;
  const int G = gridDim.x;
  const int nt = (int)((ntiles - blockIdx.x + G - 1) / G);        // tiles of this block (>= 1)
  const T* row0 = U + (int64_t)min(i0 + q, n - 1) * ld;

  // loads of step (j, c): the members 8 c .. 8 c + 7 of the wave on its tile j
  // (past the last one: read again, added as zeros)
  auto load = [&](Vec16<T> (&a)[R], int j, int c) {
    const TailLoad<T> at(((int64_t)blockIdx.x + (int64_t)min(j, nt - 1) * G) * TP + (int64_t)lane * PPL, m);
#pragma unroll
    for (int r = 0; r < R; ++r)
      a[r] = load16_nt_any(row0 + (int64_t)(4 * max(0, min(R * c + r, nm - 1))) * ld + at.xs);
    asm volatile("" ::: "memory");   // (issued here, not sunk to where they are used)
  };
  CT t[PPL], wv[PPL];
  auto step = [&](Vec16<T> (&a)[R], int j, int c) {
    const int64_t tile = (int64_t)blockIdx.x + (int64_t)j * G;
    const int64_t x0 = tile * TP + (int64_t)lane * PPL;
    if constexpr (WEIGHTED) {
      if (c == 0) {
#pragma unroll
        for (int p = 0; p < PPL; ++p) {
          const CT x = CT(w[min(x0 + p, m - 1)]);
          wv[p] = (x0 + p < m) ? x : CT(0);
        }
      }
    }
    if ((tile + 1) * TP > m) {
      const TailLoad<T> at(x0, m);
#pragma unroll
      for (int r = 0; r < R; ++r) a[r] = at.fix(a[r]);   // (zeros past m)
    }
#pragma unroll
    for (int p = 0; p < PPL; ++p) t[p] = c == 0 ? CT(0) : t[p];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (R * c + r >= nm) a[r] = Vec16<T>{};
      CT tm = CT(0);
#pragma unroll
      for (int p = 0; p < PPL; ++p) {
        const CT u = to_ct<CT>(a[r].v[p]);
        t[p] += u;
        tm += WEIGHTED ? wv[p] * u : u;
      }
      acc[(R * c + r) * 64] += tm;
    }
    if (c == nk - 1) {   // the tile's sums, waves in order
      CT* pb = part + (j & 1) * 4 * TP;
#pragma unroll
      for (int p = 0; p < PPL; ++p) pb[q * TP + lane * PPL + p] = t[p];
      lds_barrier();     // (the other buffer's readers are past it)
      for (int e = threadIdx.x; e < TP; e += 256) {
        const int64_t x = tile * TP + e;
        if (x < m) out[x] = ((pb[e] + pb[TP + e]) + pb[2 * TP + e]) + pb[3 * TP + e];
      }
    }
  };
  Vec16<T> a[R], b[R];
  auto next = [&](int& j, int& c) {
    if (++c == nk) {
      c = 0;
      ++j;
    }
  };
#pragma unroll
  for (int p = 0; p < PPL; ++p) t[p] = CT(0);
  int j = 0, c = 0;
  load(a, 0, 0);
  for (;;) {
    int j2 = j, c2 = c;
    next(j2, c2);
    load(b, j2, c2);
    step(a, j, c);
    if (j2 == nt) break;
    j = j2;
    c = c2;
    next(j, c);
    load(a, j, c);
    step(b, j2, c2);
    if (j == nt) break;
  }
  for (int k0 = 0; k0 < nm; k0 += R) {   // (R sums side by side: one after the other is 6 lane moves deep each)
    double s[R];
#pragma unroll
    for (int r = 0; r < R; ++r) s[r] = wave_sum((double)acc[(k0 + r) * 64]);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (lane == 0 && k0 + r < nm) mpart[(size_t)(i0 + q + 4 * (k0 + r)) * G + blockIdx.x] = s[r];
  }
}

// Sum of a member's row of partials by one wave, in the order of
// pidmean_reduce (256 strands, then its tree); in lane 0.
__device__ __forceinline__ double wave_parts_sum(const double* __restrict__ row, int nparts) {
  const int lane = threadIdx.x & 63;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 4; ++k)
    for (int b = lane + 64 * k; b < nparts; b += 256) s[k] += row[b];
  double v = (s[0] + s[2]) + (s[1] + s[3]);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}

// Blocks [0, cblocks): the member groups' column sums in order (as
// colsum_combine); the others: masses and their inverses, a member per wave.
template <typename AT>
__global__ __launch_bounds__(256) void linear_mid_kernel(const AT* __restrict__ cpart, int groups, int64_t m,
                                                         AT* __restrict__ s_out, int cblocks,
                                                         const double* __restrict__ mpart, int nparts, int n,
                                                         double* __restrict__ mass, AT* __restrict__ coef) {
  if ((int)blockIdx.x < cblocks) {
    for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < m; x += (int64_t)cblocks * 256) {
      AT s = cpart[x];
      for (int g = 1; g < groups; ++g) s += cpart[(size_t)g * m + x];
      s_out[x] = s;
    }
    return;
  }
  const int i = ((int)blockIdx.x - cblocks) * 4 + wave_id();
  if (i >= n) return;
  const double v = wave_parts_sum(mpart + (size_t)i * nparts, nparts);
  if ((threadIdx.x & 63) == 0) {
    mass[i] = v;
    coef[i] = v > 0.0 ? (AT)(1.0 / v) : AT(0);
  }
}

// Row sums A and B; part [2][n][gridDim.x].  Geometry and loads as
// pidmean_soft_kernel in its two-pass form.
template <typename T, int MPW, bool WEIGHTED>
__global__ __launch_bounds__(512) void rows_two_kernel(const T* __restrict__ U, int64_t ld, int n, int64_t m,
                                                       const float* __restrict__ w, int64_t ntiles,
                                                       const ComputeT<T>* __restrict__ sv,
                                                       const ComputeT<T>* __restrict__ tv, double* __restrict__ part) {
  using CT = ComputeT<T>;
  constexpr int PPL = Vec16<T>::N, TP = 64 * PPL;
  const int lane = threadIdx.x & 63;
  const int mbase = (blockIdx.y * (blockDim.x >> 6) + wave_id()) * MPW;
  CT acca[MPW], accb[MPW];
#pragma unroll
  for (int r = 0; r < MPW; ++r) { acca[r] = CT(0); accb[r] = CT(0); }
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t x0 = tile * TP + (int64_t)lane * PPL;
    const bool fast = (tile + 1) * TP <= m;
    const TailLoad<T> at(x0, m);
    Vec16<T> v[MPW];
    CT s[PPL], t[PPL];
#pragma unroll
    for (int r = 0; r < MPW; ++r) v[r] = load16_nt_any(U + (int64_t)min(mbase + r, n - 1) * ld + at.xs);
    if (fast) {
      __builtin_memcpy(s, sv + x0, sizeof(s));
      __builtin_memcpy(t, tv + x0, sizeof(t));
    } else {
#pragma unroll
      for (int p = 0; p < PPL; ++p) {
        const CT a = sv[min(x0 + p, m - 1)], b = tv[min(x0 + p, m - 1)];
        s[p] = (x0 + p < m) ? a : CT(0);
        t[p] = (x0 + p < m) ? b : CT(0);
      }
    }
    if constexpr (WEIGHTED) {
#pragma unroll
      for (int p = 0; p < PPL; ++p) {
        const CT x = CT(w[min(x0 + p, m - 1)]);
        s[p] *= x;
        t[p] *= x;
      }
    }
    auto sums = [&](bool cut) {
#pragma unroll
      for (int r = 0; r < MPW; ++r) {
        const Vec16<T> vr = cut ? at.fix(v[r]) : v[r];
        CT ta = CT(0), tb = CT(0);
#pragma unroll
        for (int p = 0; p < PPL; ++p) {
          const CT u = to_ct<CT>(vr.v[p]);
          ta += s[p] * u;
          tb += t[p] * u;
        }
        acca[r] += ta;
        accb[r] += tb;
      }
    };
    if (fast) sums(false);
    else sums(true);
  }
  const int ng = gridDim.x;
#pragma unroll
  for (int r = 0; r < MPW; ++r) {
    const double a = wave_sum((double)acca[r]);
    const double b = wave_sum((double)accb[r]);
    const int i = mbase + r;
    if (lane == 0 && i < n) {
      part[(size_t)i * ng + blockIdx.x] = a;
      part[((size_t)n + i) * ng + blockIdx.x] = b;
    }
  }
}

// A member per wave: A_i and B_i from their partials, then the ratios.
__global__ __launch_bounds__(256) void linear_finish_kernel(const double* __restrict__ part, int nparts, int n,
                                                            const double* __restrict__ mass, pid_out o) {
#pragma clang fp contract(off)
  const int i = blockIdx.x * 4 + wave_id();
  if (i >= n) return;
  const double a = wave_parts_sum(part + (size_t)i * nparts, nparts);
  const double b = wave_parts_sum(part + (size_t)(n + i) * nparts, nparts);
  if ((threadIdx.x & 63) != 0) return;
  const double mm = mass[i];
  const double ii = (mm > 0.0) ? a / ((double)n * mm) : 0.0;
  const double oo = b / (double)n;
  if (o.mass) o.mass[i] = mm;
  if (o.in_in) o.in_in[i] = ii;
  if (o.in_out) o.in_out[i] = oo;
  if (o.depth) o.depth[i] = ii < oo ? ii : oo;
}

// ---------------------------------------------------------------------------
// Host side: plan, workspace and launch.

template <typename T, int MODE, int MPW, bool W, int NWMAX>
static void launch_soft_one(const MeanPlan& p, const pid_ensemble& e, const Extract& ex,
                            int nwaves, const void* sglob, double* part, hipStream_t st, const KernelTimer& tm) {
  const size_t lds = (size_t)2 * nwaves * (64 * Vec16<T>::N) * sizeof(ComputeT<T>);
  hipExtLaunchKernelGGL((pidmean_soft_kernel<T, MODE, MPW, W, false, NWMAX>), dim3(p.grid), dim3(64 * nwaves),
                        (uint32_t)lds, st, tm.start(), tm.stop(), 0u, reinterpret_cast<const T*>(e.data), e.ld, (int)e.n, e.m, e.weights, ex,
                     p.ntiles, sglob, part);
}

template <typename T, int MODE, int MPW>
static void launch_soft_t(const MeanPlan& p, const pid_ensemble& e, const Extract& ex,
                          const void* sglob, double* part, hipStream_t st) {
  const T* U = reinterpret_cast<const T*>(e.data);
  const bool wtd = e.weights != nullptr;
  KernelTimer tm("pidmean", st, /*by_launch=*/true);   // one kernel per call
  if (p.pipe_lb) {   // the plan picks the pipelined kernel only where it is instantiated
    if constexpr (MODE != MODE_STEP && !std::is_same<T, uint8_t>::value && !(sizeof(T) == 8 && MPW == 32) &&
                  !(sizeof(T) == 2 && (MODE == MODE_GAUSS || MODE == MODE_MODEL)) && MPW != 16) {
      constexpr int LB = (MPW == 4) ? 16 : (MPW == 8 ? 8 : 4);
      constexpr int NWM = (MPW == 32) ? 8 : 16;
      if (wtd)
        hipExtLaunchKernelGGL((pidmean_pipe_kernel<T, MODE, MPW, LB, true, NWM>), dim3(p.pipe_grid),
                              dim3(64 * p.nwaves), (uint32_t)p.lds_bytes, st, tm.start(), tm.stop(), 0u, U, e.ld, (int)e.n, e.m, e.weights, ex, part);
      else
        hipExtLaunchKernelGGL((pidmean_pipe_kernel<T, MODE, MPW, LB, false, NWM>), dim3(p.pipe_grid),
                              dim3(64 * p.nwaves), (uint32_t)p.lds_bytes, st, tm.start(), tm.stop(), 0u, U, e.ld, (int)e.n, e.m, e.weights, ex, part);
    }
    return;
  }
  if constexpr (MPW != 32) {
    dim3 grid(p.grid, p.two_pass ? p.groups : 1);
    dim3 block(64 * p.nwaves);
    if (p.two_pass) {
      if (wtd)
        hipExtLaunchKernelGGL((pidmean_soft_kernel<T, MODE, MPW, true, true, 8>), grid, block, 0u, st, tm.start(), tm.stop(), 0u, U,
                           e.ld, (int)e.n, e.m, e.weights, ex, p.ntiles, sglob, part);
      else
        hipExtLaunchKernelGGL((pidmean_soft_kernel<T, MODE, MPW, false, true, 8>), grid, block, 0u, st, tm.start(), tm.stop(), 0u, U,
                           e.ld, (int)e.n, e.m, e.weights, ex, p.ntiles, sglob, part);
      return;
    }
    // single pass; 16 waves only where N needs them.  The plan gives U8 and
    // FP64 input at most 8 waves, so their 16-wave variants are not built (a
    // larger block would fail at launch, reported by the caller's check).
    if constexpr (sizeof(T) == 4 || sizeof(T) == 2) {
      if (p.nwaves > 8) {
        if (wtd) launch_soft_one<T, MODE, MPW, true, 16>(p, e, ex, p.nwaves, sglob, part, st, tm);
        else launch_soft_one<T, MODE, MPW, false, 16>(p, e, ex, p.nwaves, sglob, part, st, tm);
        return;
      }
    }
    if (wtd) launch_soft_one<T, MODE, MPW, true, 8>(p, e, ex, p.nwaves, sglob, part, st, tm);
    else launch_soft_one<T, MODE, MPW, false, 8>(p, e, ex, p.nwaves, sglob, part, st, tm);
  }
}

template <typename T, int MODE>
static void dispatch_mpw(const MeanPlan& p, const pid_ensemble& e, const Extract& ex,
                         const void* sglob, void* part, hipStream_t st) {
  switch (p.mpw) {
    case 4: launch_soft_t<T, MODE, 4>(p, e, ex, sglob, (double*)part, st); break;
    case 8: launch_soft_t<T, MODE, 8>(p, e, ex, sglob, (double*)part, st); break;
    case 32: launch_soft_t<T, MODE, 32>(p, e, ex, sglob, (double*)part, st); break;
    default: launch_soft_t<T, MODE, 16>(p, e, ex, sglob, (double*)part, st); break;
  }
}

template <typename T>
static void dispatch_mode(const MeanPlan& p, const pid_ensemble& e, int iso_kind, const Extract& ex,
                          const void* sglob, void* part, hipStream_t st) {
  switch (iso_kind) {
    case PID_ISO_GAUSSIAN: dispatch_mpw<T, MODE_GAUSS>(p, e, ex, sglob, part, st); break;
    case PID_ISO_STEP: dispatch_mpw<T, MODE_STEP>(p, e, ex, sglob, part, st); break;
    case PID_ISO_RAMP: case PID_ISO_TENT: case PID_ISO_DENSITY:
      if constexpr (has_models<T>()) dispatch_mpw<T, MODE_MODEL>(p, e, ex, sglob, part, st);
      break;
    default: dispatch_mpw<T, MODE_NONE>(p, e, ex, sglob, part, st); break;
  }
}

template <typename T, int MODE, bool SCALED>
static void launch_colsum_g(const pid_ensemble& e, const Extract& ex, int groups, const void* coef, void* gpart,
                            void* sout, hipStream_t st) {
  using CT = ComputeT<T>;
  using AT = CT;
  constexpr int PPL = Vec16<T>::N;
  const T* U = reinterpret_cast<const T*>(e.data);
  const dim3 grid((unsigned)((e.m + 64 * PPL - 1) / (64 * PPL)), (unsigned)groups);
  const int chunk = (int)((e.n + groups - 1) / groups);
  KernelTimer tm("pidmean_colsum", st);
  void* dst = groups > 1 ? gpart : sout;
  hipLaunchKernelGGL((colsum_part_kernel<T, MODE, SCALED>), grid, 256, 0, st, U, e.ld, (int)e.n, e.m, ex,
                     (const CT*)coef, chunk, dst);
  if (groups > 1) {
    const int cgrid = (int)std::min<int64_t>((e.m + 255) / 256, device_cu_count() * 8);
    hipLaunchKernelGGL(colsum_combine<AT>, cgrid, 256, 0, st, (const AT*)gpart, groups, e.m, (AT*)sout);
  }
}

template <typename T>
static void launch_colsum(const MeanPlan& p, const pid_ensemble& e, int iso_kind, const Extract& ex,
                          void* sout, void* gpart, hipStream_t st) {
  const int g = p.colsum_groups;
  if (iso_kind == PID_ISO_GAUSSIAN) {
    launch_colsum_g<T, MODE_GAUSS, false>(e, ex, g, nullptr, gpart, sout, st);
  } else if (iso_mode(iso_kind) == MODE_MODEL) {
    if constexpr (has_models<T>()) launch_colsum_g<T, MODE_MODEL, false>(e, ex, g, nullptr, gpart, sout, st);
  } else if (iso_kind == PID_ISO_STEP) {
    launch_colsum_g<T, MODE_STEP, false>(e, ex, g, nullptr, gpart, sout, st);
  } else {
    launch_colsum_g<T, MODE_NONE, false>(e, ex, g, nullptr, gpart, sout, st);
  }
}

static hipError_t launch_mean_finalize(const MeanPlan& p, const pid_ensemble& e, void* part, void* red,
                                       int nparts, const pid_out& out, hipStream_t st) {
  KernelTimer tm("pidmean_finalize", st);
  dim3 rgrid((unsigned)e.n, 2);
  hipLaunchKernelGGL(pidmean_reduce, rgrid, 256, 0, st, (const double*)part, nparts, (int)e.n, (double*)red);
  launch_mean_finish((const double*)red, e.n, out, st);
  return hipGetLastError();
}

template <typename T>
static void launch_dma(const MeanPlan& p, const pid_ensemble& e, double* part, hipStream_t st) {
  const T* U = reinterpret_cast<const T*>(e.data);
  KernelTimer tm("pidmean", st, /*by_launch=*/true);
  auto go = [&](auto kern) {
    (void)allow_dynamic_lds((const void*)kern);   // set on the first launch of each kernel
    hipExtLaunchKernelGGL(kern, dim3(p.dma_grid), dim3(64 * p.dma_nwaves), (uint32_t)p.dma_lds, st, tm.start(),
                          tm.stop(), 0u, U, e.ld, (int)e.n, e.m,
                       e.weights, part);
  };
  const bool wtd = e.weights != nullptr;
  if (wtd) go(pidmean_dma_kernel<T, true, 32, 4>);
  else go(pidmean_dma_kernel<T, false, 32, 4>);
}

hipError_t launch_pid_mean(const MeanPlan& plan, const pid_ensemble& e, int iso_kind,
                           const ExtractHost& exh, const pid_out& out, void* ws, hipStream_t st) {
  if (plan.bits) return launch_mask_bits_mean(e, iso_kind, exh, out, ws, st);
  Extract ex = __builtin_bit_cast(Extract, exh);
  Carve c(ws);
  void* part = c.take<double>((size_t)std::max(std::max(plan.grid, plan.pipe_grid), plan.dma_grid) * 2 * e.n);
  void* red = c.take<double>((size_t)2 * e.n);
  void* sbuf = plan.two_pass ? (void*)c.take<double>((size_t)e.m) : nullptr;
  void* gpart = plan.two_pass ? (void*)c.take<double>((size_t)e.m * (size_t)plan.colsum_groups) : nullptr;
  const int eb = elem_bytes_of(e.dtype);
  const bool vec = ((reinterpret_cast<uintptr_t>(e.data) & 15) == 0) && ((e.ld * eb) % 16 == 0) &&
                   (e.weights == nullptr || (reinterpret_cast<uintptr_t>(e.weights) & 15) == 0);
  // the pipelined kernel needs aligned rows and buffer offsets (one wave's
  // rows, the weights) below 2^31; otherwise the unpipelined kernel runs
  MeanPlan p = plan;
  if (p.dma_rpw) {
    const bool fits = ((int64_t)(p.dma_rpw - 1) * e.ld + e.m) * eb < (INT64_C(1) << 31) &&
                      e.m * (int64_t)sizeof(float) < (INT64_C(1) << 31);
    if (vec && fits) {
      switch (e.dtype) {
        case PID_F64: launch_dma<double>(p, e, (double*)part, st); break;
        case PID_F32: launch_dma<float>(p, e, (double*)part, st); break;
        case PID_F16: launch_dma<f16>(p, e, (double*)part, st); break;
        default: launch_dma<bf16_t>(p, e, (double*)part, st); break;
      }
      hipError_t err = hipGetLastError();
      if (err != hipSuccess) return err;
      return launch_mean_finalize(p, e, part, red, p.dma_grid, out, st);
    }
  }
  if (p.pipe_lb) {
    const bool fits = ((int64_t)(p.mpw - 1) * e.ld + e.m) * eb < (INT64_C(1) << 31) &&
                      e.m * (int64_t)sizeof(float) < (INT64_C(1) << 31);
    if (!(vec && fits)) { p.pipe_lb = 0; p.mpw = p.fb_mpw; p.nwaves = p.fb_nwaves; }
  }
  const int nparts = p.pipe_lb ? p.pipe_grid : p.grid;
  switch (e.dtype) {
    case PID_F64:
      if (p.two_pass) launch_colsum<double>(p, e, iso_kind, ex, sbuf, gpart, st);
      dispatch_mode<double>(p, e, iso_kind, ex, sbuf, part, st); break;
    case PID_F32:
      if (p.two_pass) launch_colsum<float>(p, e, iso_kind, ex, sbuf, gpart, st);
      dispatch_mode<float>(p, e, iso_kind, ex, sbuf, part, st); break;
    case PID_F16:
      if (p.two_pass) launch_colsum<f16>(p, e, iso_kind, ex, sbuf, gpart, st);
      dispatch_mode<f16>(p, e, iso_kind, ex, sbuf, part, st); break;
    case PID_BF16:
      if (p.two_pass) launch_colsum<bf16_t>(p, e, iso_kind, ex, sbuf, gpart, st);
      dispatch_mode<bf16_t>(p, e, iso_kind, ex, sbuf, part, st); break;
    default:
      if (p.two_pass) launch_colsum<uint8_t>(p, e, iso_kind, ex, sbuf, gpart, st);
      dispatch_mode<uint8_t>(p, e, iso_kind, ex, sbuf, part, st); break;
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  return launch_mean_finalize(p, e, part, red, nparts, out, st);
}


// ---------------------------------------------------------------------------
// All-pairs depths without the inclusion matrix: the PID-mean pass (masses,
// IN_in), then t = sum_j u_j / m_j into memory, then B_i = sum_x w u_i t with
// the two-pass row kernel (soft arithmetic, also for binary input).
template <typename T>
static void launch_linear_t(const pid_ensemble& e, int iso_kind, const Extract& ex, const MeanPlan& p3,
                            void* coef, int tg, void* tpart, void* tbuf, double* part, hipStream_t st) {
  if (iso_kind == PID_ISO_GAUSSIAN) launch_colsum_g<T, MODE_GAUSS, true>(e, ex, tg, coef, tpart, tbuf, st);
  else if (iso_kind == PID_ISO_STEP) launch_colsum_g<T, MODE_STEP, true>(e, ex, tg, coef, tpart, tbuf, st);
  else if (iso_mode(iso_kind) == MODE_MODEL) {
    if constexpr (has_models<T>()) launch_colsum_g<T, MODE_MODEL, true>(e, ex, tg, coef, tpart, tbuf, st);
  } else launch_colsum_g<T, MODE_NONE, true>(e, ex, tg, coef, tpart, tbuf, st);
  if (iso_kind == PID_ISO_GAUSSIAN) dispatch_mpw<T, MODE_GAUSS>(p3, e, ex, tbuf, part, st);
  else if (iso_kind == PID_ISO_STEP) dispatch_mpw<T, MODE_STEP>(p3, e, ex, tbuf, part, st);
  else if (iso_mode(iso_kind) == MODE_MODEL) {
    if constexpr (has_models<T>()) dispatch_mpw<T, MODE_MODEL>(p3, e, ex, tbuf, part, st);
  } else dispatch_mpw<T, MODE_NONE>(p3, e, ex, tbuf, part, st);
}

// Column sums and masses, t, then both row sums (see colsum_mass_kernel).
constexpr size_t kColsumMassLds = 131072;
template <typename T>
static size_t colsum_mass_lds(int chunk) {
  return (8 * 64 * (size_t)Vec16<T>::N + 4 * (size_t)(((chunk + 3) / 4 + 7) / 8 * 8) * 64) * sizeof(ComputeT<T>);
}

template <typename T>
static void launch_linear_three(const pid_ensemble& e, const Extract& ex, const MeanPlan& p, int groups, void* cpart,
                                void* s, double* mpart, double* mass, void* coef, void* tpart, void* t, double* part,
                                hipStream_t st) {
  using CT = ComputeT<T>;
  constexpr int MPW = sizeof(T) == 2 ? 8 : 16;
  const T* U = reinterpret_cast<const T*>(e.data);
  const int chunk = (int)((e.n + groups - 1) / groups);
  {
    KernelTimer tm("pidmean_colsum", st);
    const size_t lds = colsum_mass_lds<T>(chunk);
    auto go = [&](auto k) {
      (void)allow_dynamic_lds((const void*)k);
      hipLaunchKernelGGL(k, dim3((unsigned)p.grid, (unsigned)groups), 256, lds, st, U, e.ld, (int)e.n, e.m, e.weights,
                         chunk, p.ntiles, (CT*)(groups > 1 ? cpart : s), mpart);
    };
    if (e.weights) go(colsum_mass_kernel<T, true>);
    else go(colsum_mass_kernel<T, false>);
    const int cb = groups > 1 ? (int)std::min<int64_t>((e.m + 255) / 256, device_cu_count() * 8) : 0;
    hipLaunchKernelGGL(linear_mid_kernel<CT>, cb + (int)((e.n + 3) / 4), 256, 0, st, (const CT*)cpart, groups, e.m,
                       (CT*)s, cb, mpart, p.grid, (int)e.n, mass, (CT*)coef);
  }
  launch_colsum_g<T, MODE_NONE, true>(e, ex, groups, coef, tpart, t, st);
  KernelTimer tm("pidmean", st);
  const dim3 grid((unsigned)p.grid, (unsigned)p.groups);
  if (e.weights)
    hipLaunchKernelGGL((rows_two_kernel<T, MPW, true>), grid, 512, 0, st, U, e.ld, (int)e.n, e.m, e.weights,
                       p.ntiles, (const CT*)s, (const CT*)t, part);
  else
    hipLaunchKernelGGL((rows_two_kernel<T, MPW, false>), grid, 512, 0, st, U, e.ld, (int)e.n, e.m, e.weights,
                       p.ntiles, (const CT*)s, (const CT*)t, part);
}

hipError_t launch_pairs_linear(const pid_ensemble& e, int iso_kind, const ExtractHost& exh, const pid_out& out,
                               void* ws, hipStream_t st) {
  const MeanPlan p1 = mean_plan(e.n, e.m, e.dtype, iso_kind, e.weights != nullptr);
  const MeanPlan p3 = rows_plan(e.n, e.m, e.dtype);
  Carve c(ws);
  void* ws1 = c.take<char>(mean_workspace(p1, e.n, e.m));
  double* mass = c.take<double>((size_t)e.n);
  double* inin = c.take<double>((size_t)e.n);
  void* coef = c.take<double>((size_t)e.n);
  void* tbuf = c.take<double>((size_t)e.m);
  const int tg = colsum_groups(e.n, e.m, elem_bytes_of(e.dtype));
  void* tpart = c.take<double>((size_t)e.m * (size_t)tg);
  double* part = c.take<double>((size_t)p3.grid * 2 * e.n);
  double* red = c.take<double>((size_t)2 * e.n);
  Extract ex = __builtin_bit_cast(Extract, exh);
  // Three passes for soft masks where PID-mean takes two with the row pass's
  // geometry (n > 256; FP64 n > 128) and the members of a group fit the LDS of
  // colsum_mass_kernel.
  const int chunk = (int)((e.n + tg - 1) / tg);
  bool done = false;
  auto three = [&](auto tag) {
    using T = decltype(tag);
    if (!p1.two_pass || p1.binary || p1.grid != p3.grid || p1.groups != p3.groups || p1.mpw != p3.mpw ||
        p1.nwaves != p3.nwaves || p3.nwaves != 8 || p3.mpw != (sizeof(T) == 2 ? 8 : 16) || p1.colsum_groups != tg ||
        e.m < Vec16<T>::N || colsum_mass_lds<T>(chunk) > kColsumMassLds)
      return;
    Carve c1(ws1);   // the pieces of the PID-mean workspace
    double* mpart = c1.take<double>((size_t)p1.grid * 2 * e.n);
    (void)c1.take<double>((size_t)2 * e.n);
    void* s = c1.take<double>((size_t)e.m);
    void* cpart = c1.take<double>((size_t)e.m * (size_t)tg);
    launch_linear_three<T>(e, ex, p3, tg, cpart, s, mpart, mass, coef, tpart, tbuf, part, st);
    done = true;
  };
  if (iso_kind == PID_ISO_NONE) {
    switch (e.dtype) {
      case PID_F64: three(double()); break;
      case PID_F32: three(float()); break;
      case PID_F16: three(f16()); break;
      case PID_BF16: three(bf16_t()); break;
      default: break;
    }
  }
  if (done) {
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    KernelTimer tm("pidmean_finalize", st);
    hipLaunchKernelGGL(linear_finish_kernel, (int)((e.n + 3) / 4), 256, 0, st, part, p3.grid, (int)e.n, mass, out);
    return hipGetLastError();
  }
  // pass 1: masses and IN_in
  pid_out o1{};
  o1.mass = mass;
  o1.in_in = inin;
  hipError_t err = launch_pid_mean(p1, e, iso_kind, exh, o1, ws1, st);
  if (err != hipSuccess) return err;
  // coefficients 1 / m_j
  const bool dbl = e.dtype == PID_F64;
  if (dbl)
    hipLaunchKernelGGL(inv_mass_kernel<double>, (int)((e.n + 255) / 256), 256, 0, st, mass, (int)e.n, (double*)coef);
  else
    hipLaunchKernelGGL(inv_mass_kernel<float>, (int)((e.n + 255) / 256), 256, 0, st, mass, (int)e.n, (float*)coef);
  // passes 2 and 3: t, then B
  switch (e.dtype) {
    case PID_F64: launch_linear_t<double>(e, iso_kind, ex, p3, coef, tg, tpart, tbuf, part, st); break;
    case PID_F32: launch_linear_t<float>(e, iso_kind, ex, p3, coef, tg, tpart, tbuf, part, st); break;
    case PID_F16: launch_linear_t<f16>(e, iso_kind, ex, p3, coef, tg, tpart, tbuf, part, st); break;
    case PID_BF16: launch_linear_t<bf16_t>(e, iso_kind, ex, p3, coef, tg, tpart, tbuf, part, st); break;
    default: launch_linear_t<uint8_t>(e, iso_kind, ex, p3, coef, tg, tpart, tbuf, part, st); break;
  }
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  KernelTimer tm("pidmean_finalize", st);
  dim3 rgrid((unsigned)e.n, 2);
  hipLaunchKernelGGL(pidmean_reduce, rgrid, 256, 0, st, part, p3.grid, (int)e.n, red);
  hipLaunchKernelGGL(pairs_linear_ratios, (int)((e.n + 255) / 256), 256, 0, st, red, inin, (int)e.n, out.mass,
                     out.in_in, out.in_out, out.depth);
  return hipGetLastError();
}

}  // namespace pidk

namespace pidk {

// ---------------------------------------------------------------------------
// PID-mean against a reliability-weighted mean contour (Sec. 4.1, the
// optional weighting of the point-wise mean):
//   ubar = s_r / R,  s_r(x) = sum_j r_j u_j(x),  R = sum_j r_j,
//   A_i = sum_x w u_i(x) s_r(x)  =>  u_i <_p ubar = A_i / (R m_i),
//   m(ubar) = sum_j r_j m_j / R  =>  ubar <_p u_i = A_i / sum_j r_j m_j.
// Two streaming passes: s_r into the workspace (the column-sum kernel with
// the weights as coefficients), then m_i and A_i by the two-pass row kernel.

template <typename CT>
__global__ __launch_bounds__(256) void member_coef_kernel(const double* __restrict__ r, int n, CT* __restrict__ q) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) q[i] = (CT)r[i];
}

// One block: R and sum_j r_j m_j by a fixed tree, then the ratios.  R <= 0
// (no positive weight) gives zero depths.
__global__ __launch_bounds__(256) void pidmean_weighted_ratios(const double* __restrict__ red,
                                                               const double* __restrict__ r, int n,
                                                               double* __restrict__ m_out,
                                                               double* __restrict__ in_in,
                                                               double* __restrict__ in_out,
                                                               double* __restrict__ depth) {
#pragma clang fp contract(off)
  __shared__ double sr[256], sm[256];
  const int t = threadIdx.x;
  double a = 0.0, b = 0.0;
  for (int i = t; i < n; i += 256) {
    a += r[i];
    b += r[i] * red[i];
  }
  sr[t] = a;
  sm[t] = b;
  __syncthreads();
  for (int o = 128; o >= 1; o >>= 1) {
    if (t < o) { sr[t] += sr[t + o]; sm[t] += sm[t + o]; }
    __syncthreads();
  }
  const double R = sr[0], Mq = sm[0];
  for (int i = t; i < n; i += 256) {
    const double mm = red[i], A = red[n + i];
    const double ii = (mm > 0.0 && R > 0.0) ? A / (R * mm) : 0.0;
    const double oo = (Mq > 0.0 && R > 0.0) ? A / Mq : 0.0;
    if (m_out) m_out[i] = mm;
    if (in_in) in_in[i] = ii;
    if (in_out) in_out[i] = oo;
    if (depth) depth[i] = ii < oo ? ii : oo;
  }
}

template <typename T>
static void launch_weighted_t(const pid_ensemble& e, int iso_kind, const Extract& ex, const MeanPlan& p3,
                              const void* coef, int tg, void* tpart, void* sbuf, double* part, hipStream_t st) {
  if (iso_kind == PID_ISO_GAUSSIAN) launch_colsum_g<T, MODE_GAUSS, true>(e, ex, tg, coef, tpart, sbuf, st);
  else if (iso_kind == PID_ISO_STEP) launch_colsum_g<T, MODE_STEP, true>(e, ex, tg, coef, tpart, sbuf, st);
  else if (iso_mode(iso_kind) == MODE_MODEL) {
    if constexpr (has_models<T>()) launch_colsum_g<T, MODE_MODEL, true>(e, ex, tg, coef, tpart, sbuf, st);
  } else launch_colsum_g<T, MODE_NONE, true>(e, ex, tg, coef, tpart, sbuf, st);
  if (iso_kind == PID_ISO_GAUSSIAN) dispatch_mpw<T, MODE_GAUSS>(p3, e, ex, sbuf, part, st);
  else if (iso_kind == PID_ISO_STEP) dispatch_mpw<T, MODE_STEP>(p3, e, ex, sbuf, part, st);
  else if (iso_mode(iso_kind) == MODE_MODEL) {
    if constexpr (has_models<T>()) dispatch_mpw<T, MODE_MODEL>(p3, e, ex, sbuf, part, st);
  } else dispatch_mpw<T, MODE_NONE>(p3, e, ex, sbuf, part, st);
}

hipError_t launch_pid_mean_weighted(const pid_ensemble& e, int iso_kind, const ExtractHost& exh,
                                    const double* member_w, const pid_out& out, void* ws, hipStream_t st) {
  const MeanPlan p3 = rows_plan(e.n, e.m, e.dtype);
  Carve c(ws);
  void* coef = c.take<double>((size_t)e.n);
  void* sbuf = c.take<double>((size_t)e.m);
  const int tg = colsum_groups(e.n, e.m, elem_bytes_of(e.dtype));
  void* tpart = c.take<double>((size_t)e.m * (size_t)tg);
  double* part = c.take<double>((size_t)p3.grid * 2 * e.n);
  double* red = c.take<double>((size_t)2 * e.n);
  const int cg = (int)((e.n + 255) / 256);
  if (e.dtype == PID_F64) hipLaunchKernelGGL(member_coef_kernel<double>, cg, 256, 0, st, member_w, (int)e.n, (double*)coef);
  else hipLaunchKernelGGL(member_coef_kernel<float>, cg, 256, 0, st, member_w, (int)e.n, (float*)coef);
  Extract ex = __builtin_bit_cast(Extract, exh);
  switch (e.dtype) {
    case PID_F64: launch_weighted_t<double>(e, iso_kind, ex, p3, coef, tg, tpart, sbuf, part, st); break;
    case PID_F32: launch_weighted_t<float>(e, iso_kind, ex, p3, coef, tg, tpart, sbuf, part, st); break;
    case PID_F16: launch_weighted_t<f16>(e, iso_kind, ex, p3, coef, tg, tpart, sbuf, part, st); break;
    case PID_BF16: launch_weighted_t<bf16_t>(e, iso_kind, ex, p3, coef, tg, tpart, sbuf, part, st); break;
    default: launch_weighted_t<uint8_t>(e, iso_kind, ex, p3, coef, tg, tpart, sbuf, part, st); break;
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  KernelTimer tm("pidmean_finalize", st);
  dim3 rgrid((unsigned)e.n, 2);
  hipLaunchKernelGGL(pidmean_reduce, rgrid, 256, 0, st, part, p3.grid, (int)e.n, red);
  hipLaunchKernelGGL(pidmean_weighted_ratios, 1, 256, 0, st, red, member_w, (int)e.n, out.mass, out.in_in,
                     out.in_out, out.depth);
  return hipGetLastError();
}

}  // namespace pidk
