// Gram kernel for values that are multiplied as they are stored (FP16 masks
// under the FP16 scheme, BF16 masks under the BF16 scheme, U8 0/1 masks under
// the INT8 scheme, no model and no point weights): the staged slabs are the
// MFMA operands, so there is no conversion pass and no second tile.
//
// For 16-bit values the splits, the slabs (128 bytes of a row = 64 points),
// their order within a split, the MFMA instruction and the k order are those of
// gram_dma_kernel, so every FP32 partial is the same bit for bit; what differs
// is who computes it.  (INT8 partials are exact in any order.)
#pragma once
#include "gram_cover.h"

namespace pidk {

template <int MT>
using AccElem = typename std::conditional<MT == MT_I8, int, float>::type;

// Sum of a chunk's points: FP32 in order (16-bit values), or the exact count.
template <typename Tin>
__device__ __forceinline__ double chunk_mass(const Vec16<Tin>& v) {
  if constexpr (sizeof(Tin) == 1) {
    const uint4 q = __builtin_bit_cast(uint4, v);
    uint32_t c = __builtin_amdgcn_udot4(q.x, 0x01010101u, 0u, false);
    c = __builtin_amdgcn_udot4(q.y, 0x01010101u, c, false);
    c = __builtin_amdgcn_udot4(q.z, 0x01010101u, c, false);
    c = __builtin_amdgcn_udot4(q.w, 0x01010101u, c, false);
    return (double)c;
  } else {
    float ms = to_float(v.v[0]);
#pragma unroll
    for (int e = 1; e < Vec16<Tin>::N; ++e) ms = ms + to_float(v.v[e]);
    return (double)ms;
  }
}

// A workgroup's share of one split: the sub-tiles of row blocks [I0, I0 + na)
// against column blocks [J0, J0 + nb), or, on the diagonal, the upper
// sub-tiles of the blocks [I0, I0 + na).
struct RawUnit {
  int I0, na, J0, nb;
  bool diag;
};

// Units of BIG geometry (super-blocks of 8 row blocks; an off-diagonal pair is
// two units of 8 x 4 blocks) in the order J = 0, 1, ...: J * halves(J) off-
// diagonal units, then the diagonal one.  Every super-block but the last has
// 8 row blocks, hence two halves, so the units before J number J * J.
// Units of the small geometry: super-blocks of 4 row blocks, pairs I <= J.
__host__ __device__ inline int raw_units(bool big, int nbt) {
  if (big) {
    const int nsup = (nbt + 7) / 8, last = nbt - 8 * (nsup - 1);
    return (nsup - 1) * (nsup - 1) + (nsup - 1) * (last > 4 ? 2 : 1) + 1;
  }
  const int nsup = (nbt + 3) / 4;
  return nsup * (nsup + 1) / 2;
}

__device__ __forceinline__ RawUnit raw_unit(bool big, int nbt, int t) {
  RawUnit u;
  if (big) {
    int J = 0;
    while ((J + 1) * (J + 1) <= t) ++J;
    const int nj = min(8, nbt - 8 * J), halves = nj > 4 ? 2 : 1;
    const int r = t - J * J;
    u.diag = r == J * halves;
    if (u.diag) {
      u.I0 = u.J0 = 8 * J;
      u.na = u.nb = nj;
    } else {
      u.I0 = 8 * (r / halves);
      u.na = 8;
      u.J0 = 8 * J + 4 * (r % halves);
      u.nb = min(4, nbt - u.J0);
    }
  } else {
    int J = 0;
    while ((J + 1) * (J + 2) / 2 <= t) ++J;
    const int I = t - J * (J + 1) / 2;
    u.diag = I == J;
    u.I0 = 4 * I;
    u.J0 = 4 * J;
    u.na = min(4, nbt - u.I0);
    u.nb = min(4, nbt - u.J0);
  }
  return u;
}

// Big: 8 waves, up to 384 staged rows (48 KB per slab, a ring of three; the
// diagonal units stage 256 rows in a ring of four); small: 4 waves, up to 256
// staged rows in a ring of two (128 rows in a ring of four), so that two
// workgroups share a CU.  A wave multiplies 2x2 groups of sub-tiles: four
// fragment reads from LDS feed four MFMAs.  What bounds it is the lines in
// flight: a CU keeps about 64 requests of 128 bytes outstanding, and the units
// stage more rows than a split has (each is read once from HBM, the rest from
// the L2): for n = 512 on 1024^2 by these units 447 us, MFMA busy 26 %.
template <bool BIG>
struct RawGeom {
  static constexpr int NW = BIG ? 8 : 4;
  static constexpr int RI = BIG ? 256 : 128;        // rows of the I side (LDS row of the first J row)
  static constexpr int ROFF = BIG ? 384 : 256;      // staged rows, off the diagonal
  static constexpr int NBOFF = BIG ? 3 : 2;         // ring slots, off the diagonal
  static constexpr int NBDIAG = 4;                  // and on it
  static constexpr int LDS = BIG ? 3 * 384 * 128 : 2 * 256 * 128;
  static_assert(NBOFF * ROFF * 128 <= LDS && NBDIAG * RI * 128 <= LDS, "ring");
};

template <typename Tin, int MT, bool BIG>
__global__ __launch_bounds__(64 * RawGeom<BIG>::NW, 2) void gram_raw_kernel(GramArgs a, int units) {
  using GM = RawGeom<BIG>;
  static_assert(raw_operand<Tin, MT>(), "values multiplied as they are");
  constexpr int SEG = 128;                    // bytes of a row per slab
  constexpr int EB = sizeof(Tin);
  constexpr int EPC = 16 / EB;                // points per 16-byte chunk
  constexpr int KS = SEG / EB;                // points per slab
  constexpr int NW = GM::NW;
  constexpr uint32_t OOB = 0x80000000u;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();

  // XCD-first decode of the block index: the units of one split share an L2
  const int b = blockIdx.x;
  const int q = b >> 3;
  const int split = (q / units) * 8 + (b & 7);
  const RawUnit un = raw_unit(BIG, a.nbt, q % units);
  const int cnt = (a.slabs > split) ? (int)((a.slabs - 1 - split) / a.nsplit + 1) : 0;

  // The slab's rows land as they are, 128 bytes a row; lane l of a load
  // instruction (8 rows) fetches chunk (l & 7) ^ (row / 2 & 7) of its row, so
  // that any 16 consecutive lanes of a fragment read (one chunk of 16 rows)
  // cover the 64 banks once.
  const int lr = lane >> 3;
  const int chunk = (lane & 7) ^ ((4 * wave + (lr >> 1)) & 7);   // (row = 8 (wave + NW i) + lr)
  const uint32_t ldb = (uint32_t)(a.ld * EB);
  const int plim = (int)a.m - chunk * EPC;    // chunk in range: first point of the slab < plim

  // fragment addresses: row (lane & 31) of a block, chunk 2 kk + (lane >> 5)
  const int frow = (lane & 31) * SEG;
  int foff[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) foff[kk] = frow + (((2 * kk + (lane >> 5)) ^ ((lane >> 1) & 7)) << 4);

  // LW: load instructions per wave and slab; NG: 2x2 groups of this wave (DG:
  // diagonal ones, whose lower sub-tile is left out); NB: ring slots; MASS:
  // also the row sums of the staged rows (rows of the I side).
  auto work = [&](auto lwc, auto ngc, auto dgc, auto nbc, auto massc, const int (&r0)[2], const int (&c0)[2]) {
    constexpr int LW = decltype(lwc)::value, NG = decltype(ngc)::value, NB = decltype(nbc)::value;
    constexpr bool DG = decltype(dgc)::value, MASS = decltype(massc)::value;
    constexpr int SLOT = LW * NW * 8 * SEG;
    constexpr int NGA = NG > 0 ? NG : 1;
    static_assert((NB - 2) * LW <= 63, "wait count");
    // resources of the wave's load instructions: 8 consecutive rows each
    BufRes rs[LW];
    uint32_t vrow[LW];
#pragma unroll
    for (int i = 0; i < LW; ++i) {
      const int row = 8 * (wave + NW * i);    // LDS row
      const int g = (row < GM::RI) ? 32 * un.I0 + row : 32 * un.J0 + row - GM::RI;
      const int blocks = (row < GM::RI) ? un.na : un.nb;
      const int lim = (row < GM::RI) ? row : row - GM::RI;
      const int nv = (lim < 32 * blocks) ? max(0, min(8, a.n - g)) : 0;
      const Tin* base = reinterpret_cast<const Tin*>(a.U) + (int64_t)(nv > 0 ? g : 0) * a.ld;
      rs[i] = make_bufres(base, (uint32_t)(((int64_t)max(nv - 1, 0) * a.ld + a.m) * EB));
      vrow[i] = (lr < nv) ? (uint32_t)lr * ldb + (uint32_t)chunk * 16u : OOB;
    }
    auto issue = [&](int j, int slot) {
      const int64_t s = split + (int64_t)j * a.nsplit;
      const bool ok = j < cnt;
      const uint32_t sbyte = ok ? (uint32_t)(s * SEG) : 0u;
      const bool pok = ok && (int)(s * KS) < plim;
#pragma unroll
      for (int i = 0; i < LW; ++i)
        dma_to_lds<16>(rs[i], lds + slot * SLOT + (wave + NW * i) * 8 * SEG, pok ? vrow[i] : OOB, sbyte);
    };
    constexpr int MC = MASS ? GM::RI / (8 * NW) : 1;   // mass chunks per thread
    double accm[MC];
#pragma unroll
    for (int ci = 0; ci < MC; ++ci) accm[ci] = 0.0;
    AccVec<MT> acc[NGA][4];
#pragma unroll
    for (int g = 0; g < NGA; ++g)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[g][t][r] = 0;

#pragma unroll
    for (int j = 0; j < NB - 1; ++j) issue(j, j);
    int cur = 0;
    for (int j = 0; j < cnt; ++j) {
      vm_wait<(NB - 2) * LW>();
      lds_barrier();     // every wave's rows of slab j are in LDS, and slab j - 1 has been read
      issue(j + NB - 1, cur == 0 ? NB - 1 : cur - 1);
      const unsigned char* sl = lds + cur * SLOT;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        uint4 fa[4][2][1], fb[4][2][1];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            fa[kk][h][0] = *reinterpret_cast<const uint4*>(sl + (r0[g] + h) * (32 * SEG) + foff[kk]);
            if constexpr (!DG) fb[kk][h][0] = *reinterpret_cast<const uint4*>(sl + c0[g] * SEG + h * (32 * SEG) + foff[kk]);
          }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          if constexpr (DG) {
            mfma_step<MT>(acc[g][0], fa[kk][0], fa[kk][0]);
            mfma_step<MT>(acc[g][1], fa[kk][0], fa[kk][1]);
            mfma_step<MT>(acc[g][3], fa[kk][1], fa[kk][1]);
          } else {
            mfma_step<MT>(acc[g][0], fa[kk][0], fb[kk][0]);
            mfma_step<MT>(acc[g][1], fa[kk][0], fb[kk][1]);
            mfma_step<MT>(acc[g][2], fa[kk][1], fb[kk][0]);
            mfma_step<MT>(acc[g][3], fa[kk][1], fb[kk][1]);
          }
        }
      }
      if constexpr (MASS) {
        // a thread's chunks belong to the same rows in every slab: FP32 over
        // the chunk's points, then FP64 slab by slab
        Vec16<Tin> raw[MC];
#pragma unroll
        for (int ci = 0; ci < MC; ++ci) {
          const int row = (threadIdx.x >> 3) + 8 * NW * ci;
          raw[ci] = *reinterpret_cast<const Vec16<Tin>*>(sl + row * SEG + (((lane & 7) ^ ((row >> 1) & 7)) << 4));
        }
#pragma unroll
        for (int ci = 0; ci < MC; ++ci) {
          accm[ci] += chunk_mass(raw[ci]);
        }
      }
      cur = (cur == NB - 1) ? 0 : cur + 1;
    }
    vm_wait<0>();        // no load into LDS outlives the workgroup

    // partial sub-tiles
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int rb = r0[g] + (t >> 1), cb = (DG ? r0[g] : (c0[g] - (un.diag ? 0 : GM::RI)) / 32) + (t & 1);
        if ((DG && t == 2) || rb >= un.na || cb >= un.nb) continue;
        const int R = un.I0 + rb, C = un.J0 + cb;
        AccElem<MT>* p = reinterpret_cast<AccElem<MT>*>(a.part) + ((size_t)split * a.np + (size_t)(C * (C + 1) / 2 + R)) * 1024;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          p[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 32 + (lane & 31)] = acc[g][t][r];
      }
    if constexpr (MASS) {
#pragma unroll
      for (int ci = 0; ci < MC; ++ci) {
        double t = accm[ci];
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) t += __shfl_xor(t, o, 64);
        const int row = (threadIdx.x >> 3) + 8 * NW * ci;
        const int gr = 32 * un.I0 + row;
        if ((lane & 7) == 0 && row < 32 * un.na && gr < a.n) a.part_mass[(size_t)split * a.n + gr] = t;
      }
    }
  };
  // (c0 is given as the LDS row of the first column block)
  constexpr auto one = std::integral_constant<int, 1>();
  constexpr auto no = std::false_type();
  constexpr auto yes = std::true_type();
  constexpr auto lwo = std::integral_constant<int, GM::ROFF / (8 * NW)>();
  constexpr auto lwd = std::integral_constant<int, GM::RI / (8 * NW)>();
  constexpr auto nbo = std::integral_constant<int, GM::NBOFF>();
  constexpr auto nbd = std::integral_constant<int, GM::NBDIAG>();
  if (!un.diag) {
    const int nr = GM::RI / 64;   // row pairs
    const int r[2] = {2 * (wave % nr), 0}, c[2] = {GM::RI + 64 * (wave / nr), 0};
    work(lwo, one, no, nbo, no, r, c);
  } else if constexpr (BIG) {
    if (wave < 6) {   // pairs of block pairs (0,1) (0,2) (1,2) (0,3) (1,3) (2,3)
      const int gb = (wave >= 3) ? 3 : (wave >= 1 ? 2 : 1);
      const int r[2] = {2 * (wave - gb * (gb - 1) / 2), 0}, c[2] = {64 * gb, 0};
      work(lwd, one, no, nbd, yes, r, c);
    } else {          // two diagonal groups
      const int r[2] = {4 * (wave - 6), 4 * (wave - 6) + 2}, c[2] = {0, 0};
      work(lwd, std::integral_constant<int, 2>(), yes, nbd, yes, r, c);
    }
  } else {
    if (wave == 0) {
      const int r[2] = {0, 0}, c[2] = {64, 0};
      work(lwd, one, no, nbd, yes, r, c);
    } else if (wave < 3) {
      const int r[2] = {2 * (wave - 1), 0}, c[2] = {0, 0};
      work(lwd, one, yes, nbd, yes, r, c);
    } else {
      const int r[2] = {0, 0}, c[2] = {0, 0};
      work(lwd, std::integral_constant<int, 0>(), no, nbd, yes, r, c);
    }
  }
}

// One super-tile of at most RI = 64 or 128 rows: SPI = 256 / RI slabs
// share the 32 KB of a ring slot, so that as many bytes stay in flight, and as
// much is read between two barriers, for few rows as for many.  A wave
// multiplies sub-tiles wave, wave + NW, ... of the triangle, slab by slab.
template <typename Tin, int MT, int RI>
__global__ __launch_bounds__(512, 2) void gram_raw_tri_kernel(GramArgs a) {
  static_assert(raw_operand<Tin, MT>(), "values multiplied as they are");
  constexpr int EB = sizeof(Tin), SEG = 128, EPC = 16 / EB, KS = SEG / EB, NB = 4, NW = 8;
  constexpr int LW = 32 / NW;                 // load instructions per wave and slot
  constexpr int SPI = 256 / RI;               // slabs per ring slot
  constexpr int SLOT = 256 * SEG;
  constexpr int NT = ((RI / 32) * (RI / 32 + 1) / 2 + NW - 1) / NW;   // sub-tiles per wave
  constexpr int CPT = 32 / NW;                // chunks per thread and slot
  constexpr int MC = RI / (8 * NW);           // rows per thread (its chunks belong to these in every slab)
  static_assert(MC >= 1, "a thread's chunks of a row lie in different slabs");
  constexpr uint32_t OOB = 0x80000000u;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int split = blockIdx.x;
  const int cnt = (a.slabs > split) ? (int)((a.slabs - 1 - split) / a.nsplit + 1) : 0;
  const int iters = (cnt + SPI - 1) / SPI;

  // load instruction q = wave + 8 i: rows 8q mod RI .. + 7 of slab 8q / RI of
  // the slot; chunks swizzled as in gram_raw_kernel
  const int lr = lane >> 3;
  const int chunk = (lane & 7) ^ ((4 * wave + (lr >> 1)) & 7);
  const uint32_t ldb = (uint32_t)(a.ld * EB);
  const int plim = (int)a.m - chunk * EPC;
  BufRes rs[LW];
  uint32_t vrow[LW];
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int g = (8 * (wave + NW * i)) % RI;
    const int nv = max(0, min(8, a.n - g));
    const Tin* base = reinterpret_cast<const Tin*>(a.U) + (int64_t)(nv > 0 ? g : 0) * a.ld;
    rs[i] = make_bufres(base, (uint32_t)(((int64_t)max(nv - 1, 0) * a.ld + a.m) * EB));
    vrow[i] = (lr < nv) ? (uint32_t)lr * ldb + (uint32_t)chunk * 16u : OOB;
  }
  auto issue = [&](int it, int slot) {
#pragma unroll
    for (int i = 0; i < LW; ++i) {
      const int j = it * SPI + (8 * (wave + NW * i)) / RI;
      const int64_t s = split + (int64_t)j * a.nsplit;
      const bool ok = j < cnt;
      const uint32_t sbyte = ok ? (uint32_t)(s * SEG) : 0u;
      const bool pok = ok && (int)(s * KS) < plim;
      dma_to_lds<16>(rs[i], lds + slot * SLOT + (wave + NW * i) * 8 * SEG, pok ? vrow[i] : OOB, sbyte);
    }
  };
  const int T = a.nbt * (a.nbt + 1) / 2;
  int ir[NT], ic[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int k = min(wave + NW * t, T - 1);
    int c = 0;
    while ((c + 1) * (c + 2) / 2 <= k) ++c;
    ic[t] = c;
    ir[t] = k - c * (c + 1) / 2;
  }
  const int nt = wave >= T ? 0 : (T - 1 - wave) / NW + 1;
  const int frow = (lane & 31) * SEG;
  int foff[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) foff[kk] = frow + (((2 * kk + (lane >> 5)) ^ ((lane >> 1) & 7)) << 4);

  AccVec<MT> acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0;
  double accm[MC];
#pragma unroll
  for (int c = 0; c < MC; ++c) accm[c] = 0.0;

#pragma unroll
  for (int it = 0; it < NB - 1; ++it) issue(it, it);
  int cur = 0;
  for (int it = 0; it < iters; ++it) {
    vm_wait<(NB - 2) * LW>();
    lds_barrier();       // every wave's rows of this slot are in LDS, and the previous slot has been read
    issue(it + NB - 1, cur == 0 ? NB - 1 : cur - 1);
    const unsigned char* sl = lds + cur * SLOT;
    // (slabs past the split's share read as zeros and add nothing)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t < nt) {
#pragma unroll
        for (int sp = 0; sp < SPI; ++sp) {
          uint4 fa[4][1], fb[4][1];
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            fa[kk][0] = *reinterpret_cast<const uint4*>(sl + (sp * RI + ir[t] * 32) * SEG + foff[kk]);
            fb[kk][0] = *reinterpret_cast<const uint4*>(sl + (sp * RI + ic[t] * 32) * SEG + foff[kk]);
          }
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) mfma_step<MT>(acc[t], fa[kk], fb[kk]);
        }
      }
    }
    // masses: FP32 over a chunk's points, FP64 slab by slab
    Vec16<Tin> raw[CPT];
#pragma unroll
    for (int ci = 0; ci < CPT; ++ci) {
      const int row = (threadIdx.x >> 3) + 8 * NW * ci;   // of the slot: slab row / RI
      raw[ci] = *reinterpret_cast<const Vec16<Tin>*>(sl + row * SEG + (((lane & 7) ^ ((row >> 1) & 7)) << 4));
    }
#pragma unroll
    for (int ci = 0; ci < CPT; ++ci) {
      accm[ci % MC] += chunk_mass(raw[ci]);
    }
    cur = (cur == NB - 1) ? 0 : cur + 1;
  }
  vm_wait<0>();          // no load into LDS outlives the workgroup

#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t < nt) {
      AccElem<MT>* p = reinterpret_cast<AccElem<MT>*>(a.part) +
                 ((size_t)split * a.np + (size_t)(ic[t] * (ic[t] + 1) / 2 + ir[t])) * 1024;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        p[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 32 + (lane & 31)] = acc[t][r];
    }
  }
#pragma unroll
  for (int c = 0; c < MC; ++c) {
    double t = accm[c];
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) t += __shfl_xor(t, o, 64);
    const int row = (threadIdx.x >> 3) + 8 * NW * c;
    if ((lane & 7) == 0 && row < a.n) a.part_mass[(size_t)split * a.n + row] = t;
  }
}

// Units by such a design, 5 to 20 row blocks: a CU keeps about 64 requests of
// 128 bytes outstanding, so its time is the rows it stages, and a split's time
// those of its largest unit.  16 waves of NT sub-tiles each (a wave reads its
// row block's fragments again only where the row block changes): with 8 waves
// of 2x2 groups, half the fragment reads, the reads and products of a slab
// follow one another (n = 512 on 1024^2 511 us, n = 448 on 640^2 228 against
// 165).  MC x 128 rows are summed; LW load instructions per wave and slab (a
// unit of fewer rows uses fewer).  Whole calls, gram_raw_kernel and this one:
// n = 288 on 640^2 166 -> 98 us, n = 400 on 704x640 322 -> 159, n = 384 on
// 960^2 489 -> 268, n = 512 on 1024^2 460 -> 397 (1.07 GB); beside the
// converting kernel n = 256 on 1024^2 148 -> 132.
template <typename Tin, int MT, int LW, int NT, int MC>
__global__ __launch_bounds__(1024) void gram_raw_cover_kernel(GramArgs a, RawCover cv) {
  static_assert(raw_operand<Tin, MT>(), "values multiplied as they are");
  constexpr int EB = sizeof(Tin), SEG = 128, EPC = 16 / EB, KS = SEG / EB, NB = 4, NW = 16;
  constexpr uint32_t OOB = 0x80000000u;
  extern __shared__ __align__(16) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();

  // XCD-first decode of the block index: the units of one split share an L2
  const int b = blockIdx.x;
  const int q = b >> 3;
  const int split = (q / cv.units) * 8 + (b & 7);
  const int un = q % cv.units;
  const int cnt = (a.slabs > split) ? (int)((a.slabs - 1 - split) / a.nsplit + 1) : 0;
  const int nblk = cv.nblk[un], npair = cv.npair[un], nmass = cv.nmass[un];
  const int slot = nblk * 32 * SEG;

  // load instruction wave + 16 i: 8 consecutive rows; chunks swizzled as in
  // gram_raw_kernel
  const int lr = lane >> 3;
  const int chunk = (lane & 7) ^ ((4 * wave + (lr >> 1)) & 7);
  const uint32_t ldb = (uint32_t)(a.ld * EB);
  const int plim = (int)a.m - chunk * EPC;
  const int lw = (4 * nblk - wave + NW - 1) / NW;   // of this wave: LW - 2 .. LW
  BufRes rs[LW];
  uint32_t vrow[LW];
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int k = wave + NW * i;
    const int g = 32 * cv.blk[un][min(k >> 2, kCoverBlocks - 1)] + 8 * (k & 3);
    const int nv = (k < 4 * nblk) ? max(0, min(8, a.n - g)) : 0;
    const Tin* base = reinterpret_cast<const Tin*>(a.U) + (int64_t)(nv > 0 ? g : 0) * a.ld;
    rs[i] = make_bufres(base, (uint32_t)(((int64_t)max(nv - 1, 0) * a.ld + a.m) * EB));
    vrow[i] = (lr < nv) ? (uint32_t)lr * ldb + (uint32_t)chunk * 16u : OOB;
  }
  auto issue = [&](int j, int sl) {
    const int64_t s = split + (int64_t)j * a.nsplit;
    const bool ok = j < cnt;
    const uint32_t sbyte = ok ? (uint32_t)(s * SEG) : 0u;
    const bool pok = ok && (int)(s * KS) < plim;
#pragma unroll
    for (int i = 0; i < LW; ++i)
      if (i < lw) dma_to_lds<16>(rs[i], lds + sl * slot + (wave + NW * i) * 8 * SEG, pok ? vrow[i] : OOB, sbyte);
  };
  // this wave's sub-tiles: neighbours in the list, mostly of one row block
  const int t0 = wave * npair / NW, nt = (wave + 1) * npair / NW - t0;   // (<= NT)
  int ir[NT], ic[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int k = cv.pair[un][min(t0 + t, kCoverPairs - 1)];
    ir[t] = k & 15;
    ic[t] = k >> 4;
  }
  const int frow = (lane & 31) * SEG;
  int foff[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) foff[kk] = frow + (((2 * kk + (lane >> 5)) ^ ((lane >> 1) & 7)) << 4);

  AccVec<MT> acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0;
  double accm[MC];
#pragma unroll
  for (int c = 0; c < MC; ++c) accm[c] = 0.0;

  // Even waves fetch three slabs ahead, odd ones two: what is in flight comes
  // from two places of each row, which a row stride of a large power of two
  // would otherwise put on few memory channels (n = 512 on 1024^2: 458 us
  // all three ahead, 397 so; all else the same within 3 %).
  const int la = NB - 1 - (wave & 1);
  const int left = (la - 1) * lw;      // loads of this wave that may stay in flight past slab j's
  for (int j = 0; j < la; ++j) issue(j, j);
  int cur = 0;
  for (int j = 0; j < cnt; ++j) {
    switch (left) {
      case 1: vm_wait<1>(); break;
      case 2: vm_wait<2>(); break;
      case 3: vm_wait<3>(); break;
      case 4: vm_wait<4>(); break;
      case 6: vm_wait<6>(); break;
      default: vm_wait<0>();
    }
    lds_barrier();     // every wave's rows of slab j are in LDS, and slab j - 1 has been read
    issue(j + la, (cur + la) & (NB - 1));
    const unsigned char* sl = lds + cur * slot;
    uint4 fa[4][1], fb[4][1];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t < nt) {
        if (t == 0 || ir[t] != ir[t > 0 ? t - 1 : 0]) {
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) fa[kk][0] = *reinterpret_cast<const uint4*>(sl + ir[t] * (32 * SEG) + foff[kk]);
        }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) fb[kk][0] = *reinterpret_cast<const uint4*>(sl + ic[t] * (32 * SEG) + foff[kk]);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) mfma_step<MT>(acc[t], fa[kk], fb[kk]);
      }
    }
    // masses: FP32 over a chunk's points, FP64 slab by slab
#pragma unroll
    for (int c = 0; c < MC; ++c) {
      if (wave + 16 * c < 4 * nmass) {   // (8 rows per wave)
        const int row = (threadIdx.x >> 3) + 128 * c;
        accm[c] += chunk_mass(*reinterpret_cast<const Vec16<Tin>*>(sl + row * SEG + (((lane & 7) ^ ((row >> 1) & 7)) << 4)));
      }
    }
    cur = (cur == NB - 1) ? 0 : cur + 1;
  }
  vm_wait<0>();        // no load into LDS outlives the workgroup

#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t < nt) {
      const int R = cv.blk[un][ir[t]], C = cv.blk[un][ic[t]];   // R <= C
      AccElem<MT>* p = reinterpret_cast<AccElem<MT>*>(a.part) + ((size_t)split * a.np + (size_t)(C * (C + 1) / 2 + R)) * 1024;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        p[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 32 + (lane & 31)] = acc[t][r];
    }
  }
#pragma unroll
  for (int c = 0; c < MC; ++c) {
    double t = accm[c];
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) t += __shfl_xor(t, o, 64);
    const int row = (threadIdx.x >> 3) + 128 * c;
    if ((lane & 7) == 0 && row < 32 * nmass) {
      const int gr = 32 * cv.blk[un][row >> 5] + (row & 31);
      if (gr < a.n) a.part_mass[(size_t)split * a.n + gr] = t;
    }
  }
}

template <typename Tin, int MT>
void launch_gram_raw(const GramArgs& ga, hipStream_t st, const KernelTimer& tm) {
  static_assert(raw_operand<Tin, MT>(), "values multiplied as they are");
  auto go = [&](auto k, int grid, int threads, size_t lds, auto... more) {
    (void)allow_dynamic_lds((const void*)k);
    hipExtLaunchKernelGGL(k, dim3((unsigned)grid), dim3(threads), (uint32_t)lds, st, tm.start(), tm.stop(), 0u, ga,
                          more...);
  };
  // Up to 4 row blocks: slabs share a ring slot.  FP16 masks, whole call
  // against the converting kernel: n = 33 on 192^3 514 -> 120 us (3.9 TB/s),
  // n = 64 on 128^3 139 -> 65, n = 128 on 192^3 640 -> 390 (4.7 TB/s).
  constexpr size_t ring = 4 * 256 * 128;
  if (ga.nbt <= 2) return go(gram_raw_tri_kernel<Tin, MT, 64>, ga.nsplit, 512, ring);
  if (ga.nbt <= 4) return go(gram_raw_tri_kernel<Tin, MT, 128>, ga.nsplit, 512, ring);
  const RawCover* cv = raw_cover(ga.nbt, ga.nsplit);
  // Units by a covering design where a split is long enough to pay for their
  // larger ends: 8 and more row blocks in a unit lose to the small units below
  // at 32 slabs a split (n = 512 on 256^2 42.1 -> 44.7 us) and win at 50
  // (on 320^2 83.8 -> 65.7), fewer are level at 8 (n = 384 on 160^2 25.7 ->
  // 27.0; on 256^2, 21 slabs, 32.8 -> 32.0).  One unit (up to 8 row blocks) has
  // no others to lose to.  U8, this and the big units below: n = 136 on 160^3
  // 128 and 145 us, on 216^3 267 and 300; n = 256 on 128^3 121 and 150, on
  // 160^3 245 and 247, on 176^3 334 and 299: which is ahead from 5 row blocks on
  // goes by the row stride (the channels its rows meet on), not by the length
  // of the splits (at most one per CU; 64 to 308 slabs in these).
  if (cv && (cv->units == 1 || ga.slabs >= (int64_t)(cv->maxblk >= 8 ? 48 : 12) * ga.nsplit)) {
    auto cover = [&](auto lw, auto nt, auto mc) {
      go(gram_raw_cover_kernel<Tin, MT, decltype(lw)::value, decltype(nt)::value, decltype(mc)::value>,
         cv->units * ga.nsplit, 1024, (size_t)4 * cv->maxblk * 4096, *cv);
    };
    constexpr std::integral_constant<int, 1> c1;
    constexpr std::integral_constant<int, 2> c2;
    constexpr std::integral_constant<int, 3> c3;
    if (cv->maxmass > 4) return cover(c2, c3, c2);
    if (cv->maxblk > 8) return cover(c3, c3, c1);
    if (cv->maxpair <= 16) return cover(c2, c1, c1);
    if (cv->maxpair <= 32) return cover(c2, c2, c1);
    return cover(c2, c3, c1);
  }
  // Else the small units while all of them are resident at once (two per CU,
  // 256 CUs), else the big ones, which stage fewer rows per split: n = 1000 on
  // 256^2 386 -> 151 small and 176 big, n = 2048 on 256^2 1044 -> 405 and 385.
  const int us = raw_units(false, ga.nbt), ub = raw_units(true, ga.nbt);
  const bool big = us * ga.nsplit > 512;
  if (big) go(gram_raw_kernel<Tin, MT, true>, ub * ga.nsplit, 64 * RawGeom<true>::NW, RawGeom<true>::LDS, ub);
  else go(gram_raw_kernel<Tin, MT, false>, us * ga.nsplit, 64 * RawGeom<false>::NW, RawGeom<false>::LDS, us);
}

}  // namespace pidk
