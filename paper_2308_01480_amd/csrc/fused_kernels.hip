// The fused Krylov product Y = A (A^T Z) of float32 / float64 unfoldings of up to 512 rows
// (Algorithm 3, step 4), with Z in registers.
//
// What bounds it: the float32 / float64 matrix cores and HBM about equally (288 x 331,776
// float32 at 18 columns, padded to 32: 12.2 GFLOP, 79 us; 382 MB, 78 us at the rate of a large
// copy).  k_fused keeps Z in LDS, so one work-group of four waves fills a CU and every load,
// LDS read and barrier of its chain is exposed: 262 us.  Here a tile column block of W = A_J^T Z
// belongs to four of eight waves, each of which keeps its own rows of Z in registers; without Z
// two work-groups share a CU and every SIMD has four waves to choose from (155 us).  The four
// partials are summed once per tile: summed by every wave as it reads W, the four times as many
// LDS reads cost more than the barrier they save (174 us).
//
// The sums keep k_fused's order: k-step ks of W goes to partial ks mod 4, the four partials are
// added in order, a row block's products run tile by tile, and work-groups take the same tiles.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "stream_tiles.h"

namespace ttr {

constexpr int kFrWaves = 8;
constexpr int kFrThreads = 64 * kFrWaves;

// Pitch of a partial W row: four rows apart (the k-steps' lane groups) fall on distinct banks.
template <typename T> constexpr int fr_pitch(int S) { return S % 32 == 16 ? S : S + 16; }
// Vector registers the kernel keeps live: Z, the two products' sums, the tile in flight, and
// about 36 for operands and addresses.  128 let two work-groups share a CU, 256 one.
template <typename T, int SB, int KPW>
constexpr int fr_regs() {
  constexpr int words = sizeof(T) / 4, TT = tile_cols_t<T>(), NO = TT == 32 ? SB : (SB + 1) / 2;
  constexpr int stage = (16 * KPW * (TT * (int)sizeof(T) / 16) + kFrThreads - 1) / kFrThreads * 4;
  return words * (KPW * NO + (KPW + kFrWaves - 1) / kFrWaves * SB * 4 + NO * 4 + SB) + stage + 36;
}
constexpr int kFrRegs = 244;

template <typename T, int SB, int KPW>
constexpr size_t fr_lds_bytes(int apitch) {
  return ((size_t)16 * KPW * apitch + (size_t)4 * tile_cols_t<T>() * fr_pitch<T>(SB * 16)) * sizeof(T);
}
// Row pitch of the A tile.  Wide rows (44 words) keep column c at (c % 4) TT/4 + c / 4, so that
// the TT / 4 operands of a lane in the second product (columns 4 ks + q) are contiguous 16-byte
// loads and sixteen rows fall on distinct banks; they are taken where they do not cost a
// resident work-group (288 rows float32 at 32 columns 174 -> 168 us, float64 361 -> 347 us;
// 512 rows at 16 columns would go from 60 to 68 us, 96 rows at 32 from 82 to 90).
template <typename T, int SB, int KPW>
constexpr bool fr_wide() {
  const int by_regs = fr_regs<T, SB, KPW>() <= 64 ? 4 : fr_regs<T, SB, KPW>() <= 128 ? 2 : 1;
  const int narrow = (int)(kLdsBytes / fr_lds_bytes<T, SB, KPW>(tile_cols_t<T>() + 1));
  const int wide = (int)(kLdsBytes / fr_lds_bytes<T, SB, KPW>(176 / (int)sizeof(T)));
  return wide >= 1 && wide >= (narrow < by_regs ? narrow : by_regs);
}

// KPW: k-steps of each partial (rows / 16, rounded up to an even count; the rows beyond m_pad
// stay zero in LDS).  Waves w and w + 4 form partial w mod 4 of different output blocks of W:
// float32 tiles (two blocks of 16 columns) split by tile columns, float64 ones by columns of Z.
template <typename T, int SB, int KPW, int EU>
__global__ __launch_bounds__(kFrThreads, EU) void k_fused_r(const T* __restrict__ A, int64_t m, int64_t n, int m_pad,
                                                            const T* __restrict__ Zg, T* __restrict__ part,
                                                            int64_t tiles_per_group, int64_t ntiles) {
  using M = Mma<T>;
  constexpr int TT = tile_cols_t<T>(), TB = TT / 16, S = SB * 16, PW = fr_pitch<T>(S), KS = TT / 4;
  constexpr bool WIDE = fr_wide<T, SB, KPW>();
  constexpr int AP = WIDE ? 176 / (int)sizeof(T) : TT + 1;
  auto apos = [](int c) { return WIDE ? (c % 4) * KS + c / 4 : c; };
  constexpr int VEC = 16 / (int)sizeof(T);
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  constexpr int NO = TB == 2 ? SB : (SB + 1) / 2;      // output blocks of W per wave
  constexpr int APW = (KPW + kFrWaves - 1) / kFrWaves;  // row blocks of Y per wave
  constexpr int ROWS = 16 * KPW;
  extern __shared__ __align__(16) unsigned char smem[];
  T* As = reinterpret_cast<T*>(smem);  // ROWS x AP
  T* Wp = As + ROWS * AP;              // four partials, TT x PW each
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 15, q = lane >> 4;
  const int kp = wave & 3, half = wave >> 2;
  const int64_t g = blockIdx.x;
  const int64_t t0 = g * tiles_per_group;
  const int64_t t1 = t0 + tiles_per_group < ntiles ? t0 + tiles_per_group : ntiles;

  for (int e = m_pad * AP + threadIdx.x; e < ROWS * AP; e += kFrThreads) As[e] = T(0);
  T zr[KPW][NO];
#pragma unroll
  for (int i = 0; i < KPW; ++i) {
    const int row = 4 * (kp + 4 * i) + q;
#pragma unroll
    for (int o = 0; o < NO; ++o) {
      const int sb = TB == 2 ? o : 2 * o + half;
      zr[i][o] = (row < m_pad && sb < SB) ? Zg[row * S + sb * 16 + j] : T(0);
    }
  }
  typename M::acc acc2[APW][SB];
#pragma unroll
  for (int i = 0; i < APW; ++i)
#pragma unroll
    for (int sb = 0; sb < SB; ++sb) acc2[i][sb] = M::zero();

  constexpr int VPR = TT * (int)sizeof(T) / 16;
  TileRegs<T, (ROWS * VPR + kFrThreads - 1) / kFrThreads, kFrThreads> regs;
  if (t0 < t1) regs.fetch(A, m, n, 0, m_pad, t0 * TT);
  const int acol = apos((TB == 2 ? 16 * half : 0) + j);
  for (int64_t t = t0; t < t1; ++t) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < (ROWS * VPR + kFrThreads - 1) / kFrThreads; ++i) {
      const int idx = (int)threadIdx.x + i * kFrThreads, rr = idx / VPR, cv = idx % VPR;
      if (idx < m_pad * VPR) {
        const vec_t v = __builtin_bit_cast(vec_t, regs.v[i]);
#pragma unroll
        for (int e = 0; e < VEC; ++e) As[rr * AP + apos(VEC * cv + e)] = v[e];
      }
    }
    __syncthreads();
    if (t + 1 < t1) regs.fetch(A, m, n, 0, m_pad, (t + 1) * TT);
    typename M::acc acc1[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) acc1[o] = M::zero();
#pragma unroll
    for (int i = 0; i < KPW; ++i) {
      const T a = As[(4 * (kp + 4 * i) + q) * AP + acol];
#pragma unroll
      for (int o = 0; o < NO; ++o) acc1[o] = M::mma(a, zr[i][o], acc1[o]);
    }
    T* Wme = Wp + kp * TT * PW;
#pragma unroll
    for (int o = 0; o < NO; ++o) {
      const int sb = TB == 2 ? o : 2 * o + half, c0 = TB == 2 ? 16 * half : 0;
      if (sb < SB)
#pragma unroll
        for (int r = 0; r < 4; ++r) Wme[(c0 + M::orow(lane, r)) * PW + sb * 16 + j] = acc1[o][r];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < TT * S; e += kFrThreads) {
      T* w = Wp + (e / S) * PW + e % S;
      w[0] = ((w[0] + w[TT * PW]) + w[2 * TT * PW]) + w[3 * TT * PW];
    }
    __syncthreads();
    T b[KS][SB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int sb = 0; sb < SB; ++sb) b[ks][sb] = Wp[(4 * ks + q) * PW + sb * 16 + j];
#pragma unroll
    for (int i = 0; i < APW; ++i) {
      const int ab = wave + kFrWaves * i;
      if (ab < KPW) {
        const T* src = As + (ab * 16 + j) * AP + (WIDE ? q * KS : q);
        T av[KS];
        if constexpr (WIDE) {
#pragma unroll
          for (int h = 0; h < KS / VEC; ++h)
            *reinterpret_cast<vec_t*>(av + VEC * h) = *reinterpret_cast<const vec_t*>(src + VEC * h);
        } else {
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) av[ks] = src[4 * ks];
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int sb = 0; sb < SB; ++sb) acc2[i][sb] = M::mma(av[ks], b[ks][sb], acc2[i][sb]);
      }
    }
  }
  T* out = part + g * (int64_t)m_pad * S;
#pragma unroll
  for (int i = 0; i < APW; ++i) {
    const int ab = wave + kFrWaves * i;
    if (ab * 16 < m_pad) {
#pragma unroll
      for (int sb = 0; sb < SB; ++sb)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(int64_t)(ab * 16 + M::orow(lane, r)) * S + sb * 16 + j] = acc2[i][sb][r];
    }
  }
}

// Compiled k-steps: rows / 16 rounded up to one of these.
constexpr int kFrSteps[] = {2, 4, 6, 8, 10, 12, 14, 16, 18, 20, 24, 28, 32};

// Whether this form takes m_pad rows (a multiple of 16) at the padded width S: one-pass shapes
// (fused_fits), less those where several work-groups of the form with Z in LDS share a CU and are
// as fast or faster: float64 while one takes at most half the LDS (112 x 200,000 at 16 columns 53
// against 69 us, 288 x 331,776 at 32 390 against 366), float32 up to 64 rows (64 x 300,000 at 32
// 49.4 against 50.6 us, 112 x 200,000 at 16 45.6 against 39.5).
template <typename T>
constexpr bool fr_rows(int64_t m_pad, int S) {
  constexpr int DT = sizeof(T) == 8 ? TTR_F64 : TTR_F32;
  const size_t z_in_lds = fused_lds_bytes(m_pad, S, DT);
  if (m_pad > kFusedMaxRows || z_in_lds > kLdsBytes) return false;
  return DT == TTR_F64 ? z_in_lds > kLdsBytes / 2 : m_pad > 64;
}

// Whether any of the row counts that KPW k-steps serve is taken.
template <typename T, int SB, int KPW>
constexpr bool fr_used() {
  int below = 0;
  for (int k : kFrSteps)
    if (k < KPW) below = k;
  for (int blocks = below + 1; blocks <= KPW; ++blocks)
    if (fr_rows<T>(16 * blocks, SB * 16)) return true;
  return false;
}

template <typename T, int SB, int KPW>
static hipError_t launch_fr(const StreamArgs& a) {
  if constexpr (fr_used<T, SB, KPW>()) {
    static_assert(fr_regs<T, SB, KPW>() <= kFrRegs, "registers");
    constexpr int TT = tile_cols_t<T>(), S = SB * 16;
    constexpr int EU = fr_regs<T, SB, KPW>() <= 128 ? 4 : 2;
    const int64_t ntiles = (a.n + TT - 1) / TT;
    const int64_t G = groups_for(ntiles, kMaxGroups);
    const int64_t tpg = (ntiles + G - 1) / G, gu = (ntiles + tpg - 1) / tpg;
    const size_t lds = fr_lds_bytes<T, SB, KPW>(fr_wide<T, SB, KPW>() ? 176 / (int)sizeof(T) : TT + 1);
    if (lds > kLdsBytes || !part_fits(a, gu, a.m_pad * S, sizeof(T))) return hipErrorInvalidValue;
    auto kern = k_fused_r<T, SB, KPW, EU>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) { (void)hipGetLastError(); return e; }
    if ((e = mark_event(a.ev_begin, a.stream)) != hipSuccess) return e;
    for (int rep = 0; rep < a.reps; ++rep) {
      hipLaunchKernelGGL(kern, dim3((unsigned)gu), dim3(kFrThreads), lds, a.stream, (const T*)a.A, a.m, a.n, (int)a.m_pad,
                         (const T*)a.Z, (T*)a.part, tpg, ntiles);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if ((e = mark_event(a.ev_end, a.stream)) != hipSuccess) return e;
    return launch_reduce_rows((const T*)a.part, gu, a.m_pad * (int64_t)S, (int)a.m, S, a.s, a.y, a.ldy, a.stream);
  }
  return hipErrorInvalidValue;
}

template <typename T, int SB>
static hipError_t fr_launch(const StreamArgs& a) {
  const int blocks = (int)(a.m_pad / 16);
#define TTR_FR(K) \
  if (blocks <= K) return launch_fr<T, SB, K>(a);
  TTR_FR(2) TTR_FR(4) TTR_FR(6) TTR_FR(8) TTR_FR(10) TTR_FR(12) TTR_FR(14) TTR_FR(16) TTR_FR(18) TTR_FR(20) TTR_FR(24)
  TTR_FR(28) TTR_FR(32)
#undef TTR_FR
  return hipErrorInvalidValue;
}

template <typename T>
static hipError_t fr_width(const StreamArgs& a) {
  switch (a.S / 16) {
    case 1: return fr_launch<T, 1>(a);
    case 2: return fr_launch<T, 2>(a);
    case 3: return fr_launch<T, 3>(a);
    case 4: return fr_launch<T, 4>(a);
  }
  return hipErrorInvalidValue;
}

bool fused_r_takes(const StreamArgs& a) {
  return a.dtype == TTR_F32 ? fr_rows<float>(a.m_pad, a.S) : a.dtype == TTR_F64 && fr_rows<double>(a.m_pad, a.S);
}

hipError_t launch_fused_r(const StreamArgs& a) {
  if (!fused_r_takes(a)) return hipErrorInvalidValue;
  return a.dtype == TTR_F32 ? fr_width<float>(a) : fr_width<double>(a);
}

}  // namespace ttr
