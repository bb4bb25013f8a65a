// Block orthonormalisation of one Krylov block (Algorithm 3, steps 4-5) in five row-parallel
// launches (three without a previous basis):
//
//   project   h = Q^T Y, ||Y||_F^2                                   Q: m x js, Y: m x s
//   update    P = Y - Q h;  h2 = Q^T P
//   update    P <- P - Q h2;  Gm = P^T P
//   tgram     pivoted Cholesky T1 = E R_11^{-1} of Gm (rank-revealing first pass);
//             U = P T1;  G2 = U^T U
//   out       T2 = R^{-1} of the Cholesky of G2 (second pass);  Q_j = U T2, also rounded into
//             the zero-padded stream copy
//
// This is block classical Gram-Schmidt run twice (P = Y - Q Q^T Y, then P -= Q Q^T P),
// followed by the rank-revealing QR of the projected block.
//
// What bounds it: latency (10 MFLOP and 2 MB for a 960 x 30 block).  Every kernel splits the
// m rows into chunks of RB rows; work-group g takes chunks g, g + G, ..., stages each chunk in
// LDS with all of its global loads in flight at once, forms its products with float64
// matrix-core instructions and writes one partial.  The G partials are summed in group order
// by every work-group of the next launch for itself (G <= kOrthMaxGroups: at most 0.3 MB from
// L2), which also repeats the s x s factorisation: nothing waits for a last work-group, its
// fences and one more round trip, and no transform travels through memory.  Tall blocks have
// more groups and a separate summing launch after each step.  With the step's sums and
// factorisation in an elected last work-group of each launch a 960 x 30 block against 90
// columns took 164 us, now 131 us; an 8192 x 40 block alone 280 us on the 15 groups it was
// given, now 125 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "convert.h"
#include "kernels.h"
#include "qr_tail.h"
#include "wave_ops.h"

namespace ttr {

typedef double d4_t __attribute__((ext_vector_type(4)));

constexpr int kOrthThreads = 256;
constexpr int kOrthWaves = kOrthThreads / 64;

__device__ inline d4_t mma64(double a, double b, d4_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ inline d4_t zero4() { return d4_t{0.0, 0.0, 0.0, 0.0}; }

// Rows and columns of a staged chunk over the threads: 8 rows x 32 columns at a time.
constexpr int kStageRows = 8, kStageCols = 32;

// Stages rows [r0, r0 + RB) x columns [0, kc) of src (ld lds) into Ds (pitch ldd), zero
// for rows >= r1.  Sixteen loads of a thread are issued before its LDS stores.
template <int NR, int NC>
__device__ inline void stage_rows_t(const double* __restrict__ src, int64_t lds, int kc, int64_t r0, int64_t r1,
                                    double* __restrict__ Ds, int ldd) {
  const int tr = (int)threadIdx.x / kStageCols, tc = (int)threadIdx.x % kStageCols;
  const double* p = src + (r0 + tr) * lds + tc;
  for (int c0 = 0; c0 < kc; c0 += kStageCols * NC) {
    double v[NR][NC];
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const int c = c0 + tc + kStageCols * j;
        v[i][j] = (c < kc && r0 + tr + kStageRows * i < r1) ? p[(int64_t)kStageRows * i * lds + c0 + kStageCols * j] : 0.0;
      }
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const int c = c0 + tc + kStageCols * j;
        if (c < kc) Ds[(tr + kStageRows * i) * ldd + c] = v[i][j];
      }
  }
}

__device__ inline void stage_rows(const double* __restrict__ src, int64_t lds, int kc, int64_t r0, int64_t r1, int RB,
                                  double* __restrict__ Ds, int ldd) {
  if (RB == 64) stage_rows_t<8, 2>(src, lds, kc, r0, r1, Ds, ldd);
  else if (RB == 32) stage_rows_t<4, 4>(src, lds, kc, r0, r1, Ds, ldd);
  else stage_rows_t<2, 4>(src, lds, kc, r0, r1, Ds, ldd);  // RB = 16
}

// Copies len entries of W into Ws.
__device__ inline void stage_matrix(const double* __restrict__ W, int len, double* __restrict__ Ws) {
  for (int e = threadIdx.x; e < len; e += kOrthThreads) Ws[e] = W[e];
}

__device__ inline void store_rows_global(const double* __restrict__ Ds, int ldd, int kb, int64_t r0, int64_t r1, int RB,
                                         double* __restrict__ dst, int64_t ldo) {
  for (int lr = (int)threadIdx.x / kStageCols; lr < RB; lr += kStageRows)
    for (int c = (int)threadIdx.x % kStageCols; c < kb; c += kStageCols)
      if (r0 + lr < r1) dst[(r0 + lr) * ldo + c] = Ds[lr * ldd + c];
}

// acc[t] (tile t = wave + kOrthWaves * i of the ka x kb output, 16 x 16 each) +=
// Xs^T Ys over the RB staged rows (pitches ldx, ldy; rows beyond the chunk are zero).
template <int MAXT>
__device__ inline void tn_tiles(const double* __restrict__ Xs, int ldx, int ka, const double* __restrict__ Ys, int ldy,
                                int kb, int RB, d4_t (&acc)[MAXT]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ta = (ka + 15) / 16, tb = (kb + 15) / 16;
  const int i16 = lane & 15, k4 = lane >> 4;
#pragma unroll
  for (int t = 0; t < MAXT; ++t) {
    const int tile = wave + kOrthWaves * t;
    if (tile >= ta * tb) break;
    const int a = (tile / tb) * 16 + i16, b = (tile % tb) * 16 + i16;
    const bool aok = a < ka, bok = b < kb;
    d4_t c = acc[t];
    for (int k0 = 0; k0 < RB; k0 += 16) {
      double xa[4], yv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int row = k0 + 4 * u + k4;
        xa[u] = aok ? Xs[row * ldx + a] : 0.0;
        yv[u] = bok ? Ys[row * ldy + b] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) c = mma64(xa[u], yv[u], c);
    }
    acc[t] = c;
  }
}

// Ds (RB x kb, pitch ldd) = base - Xs W (SUB, base = Ds itself) or Xs W, with Xs the
// staged RB x ka rows (pitch ldx) and W (ka x kb, pitch kb) in LDS or global memory.
// Every output element is read (as base) and written by the same lane.
template <bool SUB>
__device__ inline void nn_rows(const double* __restrict__ Xs, int ldx, int ka, const double* W, int kb, int RB,
                               double* Ds, int ldd) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tb = (kb + 15) / 16;
  const int i16 = lane & 15, k4 = lane >> 4;
  for (int tile = wave; tile < (RB / 16) * tb; tile += kOrthWaves) {
    const int rt = tile / tb, ct = tile % tb;
    const int lrow = rt * 16 + i16;
    const int col = ct * 16 + i16;
    d4_t c = zero4();
    for (int k0 = 0; k0 < ka; k0 += 16) {
      double xa[4], wb[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + 4 * u + k4;
        xa[u] = k < ka ? Xs[lrow * ldx + k] : 0.0;
        wb[u] = (k < ka && col < kb) ? W[k * kb + col] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) c = mma64(xa[u], wb[u], c);
    }
    if (col < kb) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int lr = rt * 16 + k4 + 4 * r;
        Ds[lr * ldd + col] = SUB ? Ds[lr * ldd + col] - c[r] : c[r];
      }
    }
  }
}

// Writes the tiles of acc into out (ka x kb, row-major).
template <int MAXT>
__device__ inline void store_tiles(const d4_t (&acc)[MAXT], int ka, int kb, double* __restrict__ out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ta = (ka + 15) / 16, tb = (kb + 15) / 16;
#pragma unroll
  for (int t = 0; t < MAXT; ++t) {
    const int tile = wave + kOrthWaves * t;
    if (tile >= ta * tb) break;
    const int b = (tile % tb) * 16 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int a = (tile / tb) * 16 + (lane >> 4) + 4 * r;
      if (a < ka && b < kb) out[(int64_t)a * kb + b] = acc[t][r];
    }
  }
}

// out[e] = sum over the G partials part[g * len + e], in group order, by one work-group.
__device__ inline void sum_partials(const double* __restrict__ part, int G, int len, double* __restrict__ out) {
  constexpr int U = 3;
  for (int e0 = 0; e0 < len; e0 += U * kOrthThreads) {
    double v[U][kOrthMaxGroups];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * kOrthThreads + (int)threadIdx.x;
#pragma unroll
      for (int g = 0; g < kOrthMaxGroups; ++g) v[u][g] = (e < len && g < G) ? part[(int64_t)g * len + e] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * kOrthThreads + (int)threadIdx.x;
      double acc = 0.0;
#pragma unroll
      for (int g = 0; g < kOrthMaxGroups; ++g) acc += v[u][g];
      if (e < len) out[e] = acc;
    }
  }
}

__device__ inline double block_total(double v) {
  __shared__ double red[kOrthWaves];
  v = sum64(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

// How a launch finds the sums of the previous one: partials to sum itself (part, G groups) or
// sums formed by k_orth_sum (sums).  `in_lds`: the sums are kept in this launch's LDS.
struct OrthSums {
  const double* part = nullptr;
  int G = 0;
  const double* sums = nullptr;
  int in_lds = 0;
};

// The len sums, in Ws (LDS) or where they are.  The caller synchronises.
__device__ inline const double* fetch_sums(const OrthSums& in, int len, double* Ws) {
  if (!in.sums) { sum_partials(in.part, in.G, len, Ws); return Ws; }
  if (!in.in_lds) return in.sums;
  stage_matrix(in.sums, len, Ws);
  return Ws;
}

// ---------------------------------------------------------------------------------
// project: partials of h (js x s) = Q^T Y and of ||Y||_F^2.
// LDS: Q rows (RB x js+1), Y rows (RB x s+1).
// ---------------------------------------------------------------------------------
template <int MAXT>
__global__ __launch_bounds__(kOrthThreads) void k_orth_project(OrthArgs a, const double* __restrict__ Y, int64_t ldy,
                                                               int RB, double* __restrict__ part) {
  extern __shared__ __align__(16) double dsm[];
  const int lq = a.js + 1, ly = a.s + 1;
  double* Qs = dsm;
  double* Ys = Qs + RB * lq;
  d4_t acc[MAXT];
#pragma unroll
  for (int t = 0; t < MAXT; ++t) acc[t] = zero4();
  double nrm = 0.0;
  const int64_t nchunks = (a.m + RB - 1) / RB;
  for (int64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
    const int64_t r0 = ch * RB, r1 = r0 + RB < a.m ? r0 + RB : a.m;
    stage_rows(a.Q, a.ldq, a.js, r0, r1, RB, Qs, lq);
    stage_rows(Y, ldy, a.s, r0, r1, RB, Ys, ly);
    __syncthreads();
    tn_tiles<MAXT>(Qs, lq, a.js, Ys, ly, a.s, RB, acc);
    for (int lr = (int)threadIdx.x / kStageCols; lr < RB; lr += kStageRows)
      for (int c = (int)threadIdx.x % kStageCols; c < a.s; c += kStageCols) {
        const double v = Ys[lr * ly + c];
        nrm = fma(v, v, nrm);
      }
    __syncthreads();
  }
  store_tiles<MAXT>(acc, a.js, a.s, part + (int64_t)blockIdx.x * a.js * a.s);
  const double t = block_total(nrm);
  if (threadIdx.x == 0) a.norm_part[blockIdx.x] = t;
}

// ---------------------------------------------------------------------------------
// update: P = S - Q W (js >= 1, written to a.P) or P = S; then the partials of h2 = Q^T P
// (NEXT_PROJ, with *ref = ||Y||_F^2 from the partial norms) or of Gm = P^T P.
// LDS: W (js x s, unless it is read from memory), Q rows (RB x js+1), P rows (RB x s+1).
// ---------------------------------------------------------------------------------
template <int MAXT, bool NEXT_PROJ>
__global__ __launch_bounds__(kOrthThreads) void k_orth_update(OrthArgs a, const double* __restrict__ S, int64_t lds_,
                                                              int RB, OrthSums in, double* __restrict__ part) {
  extern __shared__ __align__(16) double dsm[];
  const int lq = a.js + 1, lp = a.s + 1;
  double* Ws = dsm;
  double* Qs = Ws + (in.in_lds ? a.js * a.s : 0);
  double* Ps = Qs + (a.js > 0 ? RB * lq : 0);
  const double* Wp = a.js > 0 ? fetch_sums(in, a.js * a.s, Ws) : nullptr;
  if (NEXT_PROJ && blockIdx.x == 0 && threadIdx.x < 64) {
    double t = 0.0;
    for (int g = threadIdx.x; g < in.G; g += 64) t += a.norm_part[g];
    t = sum64(t);
    if (threadIdx.x == 0) *a.ref = t;
  }
  d4_t acc[MAXT];
#pragma unroll
  for (int t = 0; t < MAXT; ++t) acc[t] = zero4();
  bool bad = false;
  const int64_t nchunks = (a.m + RB - 1) / RB;
  for (int64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
    const int64_t r0 = ch * RB, r1 = r0 + RB < a.m ? r0 + RB : a.m;
    if (a.js > 0) stage_rows(a.Q, a.ldq, a.js, r0, r1, RB, Qs, lq);
    stage_rows(S, lds_, a.s, r0, r1, RB, Ps, lp);
    __syncthreads();
    if (a.status)
      for (int lr = (int)threadIdx.x / kStageCols; lr < RB; lr += kStageRows)
        for (int c = (int)threadIdx.x % kStageCols; c < a.s; c += kStageCols) bad |= !isfinite(Ps[lr * lp + c]);
    if (a.js > 0) {
      nn_rows<true>(Qs, lq, a.js, Wp, a.s, RB, Ps, lp);
      __syncthreads();
      store_rows_global(Ps, lp, a.s, r0, r1, RB, a.P, a.ldp);
    }
    if (NEXT_PROJ) tn_tiles<MAXT>(Qs, lq, a.js, Ps, lp, a.s, RB, acc);
    else tn_tiles<MAXT>(Ps, lp, a.s, Ps, lp, a.s, RB, acc);
    __syncthreads();
  }
  const int ka = NEXT_PROJ ? a.js : a.s;
  store_tiles<MAXT>(acc, ka, a.s, part + (int64_t)blockIdx.x * ka * a.s);
  if (bad) *a.status = 1;
}

// ---------------------------------------------------------------------------------
// tgram: T1 of the pivoted Cholesky of Gm (pivots <= coef * (*ref) dropped; ref = trace(Gm)
// when ref_from_gram), kept1;  U = P T1 (written to a.U);  partials of G2 = U^T U.
// LDS: T1 (s x s), Gm and then R_11 (SMAX x SMAX), P and U rows (RB x s+1 each).
// ---------------------------------------------------------------------------------
template <int SMAX>
__global__ __launch_bounds__(kOrthThreads) void k_orth_tgram(OrthArgs a, const double* __restrict__ P, int64_t ldp,
                                                             int RB, OrthSums in, double* __restrict__ part) {
  extern __shared__ __align__(16) double dsm[];
  __shared__ QrTailSmem<SMAX> sm;
  __shared__ int kept;
  const int s = a.s, lp = s + 1;
  double* Ts = dsm;
  double* Gs = Ts + s * s;
  double* Ps = Gs + SMAX * SMAX;
  double* Us = Ps + RB * lp;
  const int64_t nchunks = (a.m + RB - 1) / RB;
  // the first chunk's rows travel while the transform is formed
  if (blockIdx.x < nchunks) {
    const int64_t r0 = (int64_t)blockIdx.x * RB, r1 = r0 + RB < a.m ? r0 + RB : a.m;
    stage_rows(P, ldp, s, r0, r1, RB, Ps, lp);
  }
  fetch_sums(in, s * s, Gs);
  __syncthreads();
  double thr;
  if (a.ref_from_gram) {
    double tr = 0.0;
    for (int i = 0; i < s; ++i) tr += Gs[i * s + i];
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.ref = tr;
    thr = a.coef * tr;
  } else {
    thr = a.coef * (*a.ref);
  }
  qrcp_block<SMAX>(Gs, s, s, thr, Ts, &kept, Gs, sm);
  __syncthreads();
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) *a.kept1 = kept;
    if (a.Tprod)
      for (int e = threadIdx.x; e < s * s; e += kOrthThreads) a.T1[e] = Ts[e];
  }
  d4_t acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = zero4();
  for (int64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
    const int64_t r0 = ch * RB, r1 = r0 + RB < a.m ? r0 + RB : a.m;
    if (ch != blockIdx.x) {
      stage_rows(P, ldp, s, r0, r1, RB, Ps, lp);
      __syncthreads();
    }
    nn_rows<false>(Ps, lp, s, Ts, s, RB, Us, lp);
    __syncthreads();
    store_rows_global(Us, lp, s, r0, r1, RB, a.U, a.ldu);
    tn_tiles<4>(Us, lp, s, Us, lp, s, RB, acc);
    __syncthreads();
  }
  store_tiles<4>(acc, s, s, part + (int64_t)blockIdx.x * s * s);
}

// ---------------------------------------------------------------------------------
// out: T2 = R^{-1} of the Cholesky of G2 over the first kept1 columns (pivots <= thresh2
// dropped, survivors packed), kept2, Tprod = T1 T2 when asked; Q_j = U T2 into a.Qout (ld ldqo)
// and, when zs is given, rounded into the stream copy zs (m_pad x Sz, dtype zdt; rows >= m and
// columns >= s are zero).  LDS: T2 (s x s), G2 and then R (SMAX x SMAX), U rows, Q rows (RB x
// s+1 each).
// ---------------------------------------------------------------------------------
template <int SMAX, typename TZ>
__global__ __launch_bounds__(kOrthThreads) void k_orth_out(OrthArgs a, int RB, OrthSums in) {
  extern __shared__ __align__(16) double dsm[];
  __shared__ QrTailSmem<SMAX> sm;
  __shared__ int kept;
  const int s = a.s, lp = s + 1;
  double* Ts = dsm;
  double* Gs = Ts + s * s;
  double* Us = Gs + SMAX * SMAX;
  double* Os = Us + RB * lp;
  const int64_t rows_z = a.zs ? a.m_pad : a.m;
  const int64_t nchunks = (rows_z + RB - 1) / RB;
  // the first chunk's rows travel while the transform is formed
  {
    const int64_t r0 = (int64_t)blockIdx.x * RB, r1 = r0 + RB < a.m ? r0 + RB : a.m;
    stage_rows(a.U, a.ldu, s, r0, r1, RB, Us, lp);
  }
  fetch_sums(in, s * s, Gs);
  __syncthreads();
  chol_inv_block<SMAX>(Gs, s, s, *a.kept1, a.thresh2, Ts, &kept, Gs, sm);
  __syncthreads();
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) *a.kept2 = kept;
    if (a.Tprod)
      for (int e = threadIdx.x; e < s * s; e += kOrthThreads) {
        const int i = e / s, j = e % s;
        double acc2 = 0.0;
        for (int l = 0; l < s; ++l) acc2 = fma(a.T1[i * s + l], Ts[l * s + j], acc2);
        a.Tprod[e] = acc2;
      }
  }
  for (int64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
    const int64_t r0 = ch * RB, r1 = r0 + RB < a.m ? r0 + RB : a.m;
    if (ch != blockIdx.x) {
      stage_rows(a.U, a.ldu, s, r0, r1, RB, Us, lp);
      __syncthreads();
    }
    nn_rows<false>(Us, lp, s, Ts, s, RB, Os, lp);
    __syncthreads();
    store_rows_global(Os, lp, s, r0, r1, RB, a.Qout, a.ldqo);
    if (a.zs) {
      TZ* z = static_cast<TZ*>(a.zs);
      for (int lr = (int)threadIdx.x / kStageCols; lr < RB; lr += kStageRows)
        for (int c = (int)threadIdx.x % kStageCols; c < a.Sz; c += kStageCols) {
          const int64_t row = r0 + lr;
          if (row < a.m_pad) z[row * a.Sz + c] = (row < a.m && c < s) ? round_from_f64<TZ>(Os[lr * lp + c]) : TZ(0);
        }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------
// Separate sums: out[e] = sum over the G row-group partials part[g * len + e] for e < len.
// Tall blocks: each output's G partials are summed by eight thread slices over contiguous
// group ranges, combined in slice order.  k_orth_sum_few: in group order (sum_partials) for the
// few groups of a shorter block whose sums do not fit beside its rows in LDS.
// ---------------------------------------------------------------------------------
constexpr int kRedSegO = 8;
constexpr int kRedOutsO = kOrthThreads / kRedSegO;

__global__ __launch_bounds__(kOrthThreads) void k_orth_sum(const double* __restrict__ part, int G, int len,
                                                           double* __restrict__ out) {
  __shared__ double red[kRedSegO][kRedOutsO];
  const int o = threadIdx.x % kRedOutsO, seg = threadIdx.x / kRedOutsO;
  const int e = blockIdx.x * kRedOutsO + o;
  const int per = (G + kRedSegO - 1) / kRedSegO;
  const int g0 = seg * per, g1 = g0 + per < G ? g0 + per : G;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (e < len) {
    int g = g0;
    for (; g + 4 <= g1; g += 4)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += part[(int64_t)(g + u) * len + e];
    for (int u = 0; g < g1; ++g, ++u) acc[u] += part[(int64_t)g * len + e];
  }
  red[seg][o] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (seg == 0 && e < len) {
    double t = red[0][o];
#pragma unroll
    for (int k = 1; k < kRedSegO; ++k) t += red[k][o];
    out[e] = t;
  }
}

__global__ __launch_bounds__(kOrthThreads) void k_orth_sum_few(const double* __restrict__ part, int G, int len,
                                                               double* __restrict__ out) {
  const int e = blockIdx.x * kOrthThreads + threadIdx.x;
  if (e >= len) return;
  double acc = 0.0;
#pragma unroll
  for (int g = 0; g < kOrthMaxGroups; ++g) acc += g < G ? part[(int64_t)g * len + e] : 0.0;
  out[e] = acc;
}

__global__ void k_zero_int(int* p) { *p = 0; }

// ---------------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------------
hipError_t zero_int(int* p, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(1), 0, st, p);
  return hipGetLastError();
}

template <typename F>
static hipError_t orth_set_lds(F kernel, size_t bytes) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}

// Largest row chunk RB in {64, 32, 16} whose dynamic LDS (doubles: fixed + RB * per_row) fits
// beside `reserve` bytes; 0 if none does.  The chunk sizes and the group count fix the order
// of every sum over the rows, so the reserves are constants of the rule and not the present
// kernels' own (smaller) needs: a pivoted Cholesky that kept R twice, its scalars and its Gram.
static int pick_rows(size_t fixed, size_t per_row, size_t reserve, size_t* bytes) {
  for (int rb = 64; rb >= 16; rb /= 2) {
    const size_t b = (fixed + (size_t)rb * per_row) * sizeof(double);
    if (b + reserve + 1024 <= (size_t)kLdsBytes) { *bytes = b; return rb; }
  }
  return 0;
}
static size_t tail_reserve(int s) {
  const size_t S = (size_t)(s + 15) / 16 * 16;
  return (3 * S + 2 * S * (S + 1) + S * S) * sizeof(double) + 3 * S * sizeof(int);
}
static int orth_groups(int64_t rows, int RB, bool big) {
  const int64_t c = (rows + RB - 1) / RB;
  return (int)std::max<int64_t>(1, std::min<int64_t>(c, big ? kOrthBigGroups : kOrthMaxGroups));
}
static bool part_ok(const OrthArgs& a, int G, int ka) {
  return (size_t)G * (size_t)ka * a.s * sizeof(double) <= a.part_bytes;
}

// The sums of a launch's partials for the next one: tall blocks, a single partial buffer (the
// next launch would overwrite what it reads) and sums that the next launch cannot keep in LDS
// take a launch of their own (into `out`).
static hipError_t orth_sums(const OrthArgs& a, const double* part, int G, int len, bool fits, double* out, OrthSums* in) {
  *in = OrthSums();
  in->part = part;
  in->G = G;
  in->in_lds = fits ? 1 : 0;
  if (!a.big && fits && a.two_parts) return hipSuccess;
  if (!out) return hipErrorInvalidValue;
  in->sums = out;
  if (a.big)
    hipLaunchKernelGGL(k_orth_sum, dim3((unsigned)((len + kRedOutsO - 1) / kRedOutsO)), dim3(kOrthThreads), 0, a.st,
                       part, G, len, out);
  else
    hipLaunchKernelGGL(k_orth_sum_few, dim3((unsigned)((len + kOrthThreads - 1) / kOrthThreads)), dim3(kOrthThreads), 0,
                       a.st, part, G, len, out);
  return hipGetLastError();
}

template <int MAXT>
static hipError_t project_t(const OrthArgs& a, const double* Y, int64_t ldy, double* part, int* G) {
  size_t lds = 0;
  const int RB = pick_rows(0, (size_t)(a.js + 1) + (a.s + 1), 0, &lds);
  if (!RB) return hipErrorInvalidValue;
  *G = orth_groups(a.m, RB, a.big);
  if (!part_ok(a, *G, a.js) || *G > a.norm_cap) return hipErrorInvalidValue;
  const hipError_t e = orth_set_lds(k_orth_project<MAXT>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_orth_project<MAXT>, dim3(*G), dim3(kOrthThreads), lds, a.st, a, Y, ldy, RB, part);
  return hipGetLastError();
}

// `part` holds the previous partials (Gin groups of js x s); this launch's go to `out`.
template <int MAXT, bool NP>
static hipError_t update_t(const OrthArgs& a, const double* S, int64_t lds_, const double* part, int Gin, double* sums,
                           double* out, int* G) {
  const size_t reserve = (NP || a.big) ? 0 : tail_reserve(a.s);
  const size_t per_row = (size_t)(a.js > 0 ? a.js + 1 : 0) + (a.s + 1);
  size_t lds = 0;
  bool fits = true;
  int RB = pick_rows((size_t)a.js * a.s, per_row, reserve, &lds);
  if (!RB) { fits = false; RB = pick_rows(0, per_row, reserve, &lds); }
  *G = orth_groups(a.m, RB ? RB : 16, a.big);
  if (!RB || !part_ok(a, *G, NP ? a.js : a.s)) return hipErrorInvalidValue;
  OrthSums in;
  hipError_t e = hipSuccess;
  if (a.js > 0 && (e = orth_sums(a, part, Gin, a.js * a.s, fits, sums, &in)) != hipSuccess) return e;
  if ((e = orth_set_lds(k_orth_update<MAXT, NP>, lds)) != hipSuccess) return e;
  hipLaunchKernelGGL((k_orth_update<MAXT, NP>), dim3(*G), dim3(kOrthThreads), lds, a.st, a, S, lds_, RB, in, out);
  return hipGetLastError();
}

template <int SMAX>
static hipError_t tgram_t(const OrthArgs& a, const double* P, int64_t ldp, const double* part, int Gin, double* out,
                          int* G) {
  size_t lds = 0;
  const size_t ss = (size_t)a.s * a.s;
  const int RB = pick_rows(ss, 2 * (size_t)(a.s + 1), a.big ? 0 : tail_reserve(a.s), &lds);
  if (!RB) return hipErrorInvalidValue;
  *G = orth_groups(a.m, RB, a.big);
  if (!part_ok(a, *G, a.s)) return hipErrorInvalidValue;
  OrthSums in;
  hipError_t e = orth_sums(a, part, Gin, a.s * a.s, true, a.gsum, &in);
  if (e != hipSuccess) return e;
  lds += (size_t)SMAX * SMAX * sizeof(double);  // Gm and R_11 beside the rule's T1 and rows
  if (lds + sizeof(QrTailSmem<SMAX>) + 1024 > (size_t)kLdsBytes) return hipErrorInvalidValue;
  if ((e = orth_set_lds(k_orth_tgram<SMAX>, lds)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_orth_tgram<SMAX>, dim3(*G), dim3(kOrthThreads), lds, a.st, a, P, ldp, RB, in, out);
  return hipGetLastError();
}

// The output has no partials: one work-group per 16-row chunk, up to 256.
template <int SMAX, typename TZ>
static hipError_t out_t(const OrthArgs& a, const OrthSums& in) {
  constexpr int RB = 16;
  const size_t lds = ((size_t)a.s * a.s + (size_t)SMAX * SMAX + (size_t)RB * 2 * (a.s + 1)) * sizeof(double);
  const hipError_t e = orth_set_lds(k_orth_out<SMAX, TZ>, lds);
  if (e != hipSuccess) return e;
  const int64_t chunks = ((a.zs ? a.m_pad : a.m) + RB - 1) / RB;
  hipLaunchKernelGGL((k_orth_out<SMAX, TZ>), dim3((unsigned)std::min<int64_t>(chunks, 256)), dim3(kOrthThreads), lds, a.st,
                     a, RB, in);
  return hipGetLastError();
}

// tgram and out at the compiled width SMAX >= s.
template <int SMAX>
static hipError_t qr_t(const OrthArgs& a, const double* P, int64_t ldp, const double* part, int Gin, double* other) {
  int G = 0;
  hipError_t e = tgram_t<SMAX>(a, P, ldp, part, Gin, other, &G);
  if (e != hipSuccess) return e;
  OrthSums in;
  if ((e = orth_sums(a, other, G, a.s * a.s, true, a.gsum, &in)) != hipSuccess) return e;
  if (!a.zs || a.zdt == TTR_F64) return out_t<SMAX, double>(a, in);
  if (a.zdt == TTR_F32) return out_t<SMAX, float>(a, in);
  return out_t<SMAX, __bf16>(a, in);
}

hipError_t orth_step(const OrthArgs& args, const double* Y, int64_t ldy) {
  OrthArgs a = args;
  const int s = a.s, js = a.js;
  if (a.m <= 0 || s < 1 || s > 64 || js < 0 || js > kMaxSmall || !Y || !a.part || !a.U || !a.kept1 || !a.kept2 || !a.ref ||
      !a.Qout)
    return hipErrorInvalidValue;
  if (js > 0 && (!a.Q || !a.P || !a.norm_part)) return hipErrorInvalidValue;
  if (a.Tprod && !a.T1) return hipErrorInvalidValue;
  if (a.zs && (a.m_pad < a.m || a.Sz < s)) return hipErrorInvalidValue;
  // two partial buffers in turn when the scratch holds two: a launch that sums the previous
  // partials itself reads one while it writes the other
  const size_t half = a.part_bytes / 2 / 256 * 256;
  a.two_parts = !a.big && (size_t)orth_groups(a.m, 16, false) * std::max(js, s) * s * sizeof(double) <= half;
  if (a.two_parts) a.part_bytes = half;
  double* pa = a.part;
  double* pb = a.two_parts ? a.part + half / sizeof(double) : a.part;
  hipError_t e = hipSuccess;
  const double* P = Y;
  int64_t ldp = ldy;
  int G = 0;
  if (js > 0) {
    const int tiles = ((js + 15) / 16) * ((s + 15) / 16);
    if (tiles > 16 * kOrthWaves) return hipErrorInvalidValue;
    e = tiles <= 4 * kOrthWaves ? project_t<4>(a, Y, ldy, pa, &G)
        : tiles <= 8 * kOrthWaves ? project_t<8>(a, Y, ldy, pa, &G) : project_t<16>(a, Y, ldy, pa, &G);
    if (e != hipSuccess) return e;
    const int G1 = G;
    e = tiles <= 4 * kOrthWaves   ? update_t<4, true>(a, Y, ldy, pa, G1, a.h, pb, &G)
        : tiles <= 8 * kOrthWaves ? update_t<8, true>(a, Y, ldy, pa, G1, a.h, pb, &G)
                                  : update_t<16, true>(a, Y, ldy, pa, G1, a.h, pb, &G);
    if (e != hipSuccess) return e;
    P = a.P;
    ldp = a.ldp;
    std::swap(pa, pb);
  }
  int G2 = 0;
  e = update_t<4, false>(a, P, ldp, pa, G, a.h2, pb, &G2);
  if (e != hipSuccess) return e;
  switch ((s + 7) / 8) {
    case 1: return qr_t<8>(a, P, ldp, pb, G2, pa);
    case 2: return qr_t<16>(a, P, ldp, pb, G2, pa);
    case 3: return qr_t<24>(a, P, ldp, pb, G2, pa);
    case 4: return qr_t<32>(a, P, ldp, pb, G2, pa);
    case 5: return qr_t<40>(a, P, ldp, pb, G2, pa);
    case 6: return qr_t<48>(a, P, ldp, pb, G2, pa);
    case 7: return qr_t<56>(a, P, ldp, pb, G2, pa);
    default: return qr_t<64>(a, P, ldp, pb, G2, pa);
  }
}

}  // namespace ttr
