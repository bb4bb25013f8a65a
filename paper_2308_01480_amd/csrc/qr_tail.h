// Work-group (256-thread) factorisations of a small s x s Gram matrix (s <= SMAX <= 64)
// that turn a block into an orthonormal basis: the rank-revealing pivoted Cholesky (first
// pass) and the Cholesky inverse (second pass).  Lane l of every wave holds row l of the
// Schur complement, wave w its columns [w SMAX/4, (w+1) SMAX/4), so one elimination step
// costs each wave a quarter of the row update and a single barrier.  Every work-group of the
// block orthonormalisation that needs a transform runs them for itself.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "wave_ops.h"

namespace ttr {

// The largest of v over the wave (DPP maxima over 16 lanes, then the four row maxima).
template <int CTRL>
__device__ inline uint32_t dpp_max_u32(uint32_t v) {
  const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
  return v > o ? v : o;
}
__device__ inline uint32_t wave_max_u32(uint32_t v) {
  v = dpp_max_u32<0xB1>(v);   // lane ^ 1
  v = dpp_max_u32<0x4E>(v);   // lane ^ 2
  v = dpp_max_u32<0x141>(v);  // mirror within 8
  v = dpp_max_u32<0x140>(v);  // mirror within 16
  v = dpp_max_u32<0x142>(v);  // row 0 into 1, 2 into 3 (lane 15 of the row before)
  v = dpp_max_u32<0x143>(v);  // rows 0-1 into 2-3 (lane 31)
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
// The lane of the largest v > 0 over the wave, ties to the lowest lane; -1 if there is none.
// Positive values are ordered as their bit patterns: the high words are compared first, the
// low words only when two high words are equal.
__device__ inline int wave_argmax_positive(double v) {
  const bool in = v > 0.0;
  const uint32_t hi = in ? (uint32_t)__double2hiint(v) : 0u;
  const uint32_t mh = wave_max_u32(hi);
  uint64_t hit = __ballot(in && hi == mh);
  if (hit & (hit - 1)) {
    const bool c = in && hi == mh;
    const uint32_t ml = wave_max_u32(c ? (uint32_t)__double2loint(v) : 0u);
    hit = __ballot(c && (uint32_t)__double2loint(v) == ml);
  }
  return hit ? __builtin_ctzll(hit) : -1;
}

// Shared memory of the work-group factorisations below, beside the SMAX x SMAX matrix
// Rt that the caller places.
template <int SMAX>
struct alignas(16) QrTailSmem {
  alignas(16) double prow[2][SMAX];  // pivot row, double buffered across steps
  double rinv[SMAX];
  int rowid[SMAX];  // row of pivot j
  int pos[SMAX];    // pivot position of row l, SMAX if it was not taken
};

// Column c of X = Rt^{-1} (Rt upper triangular k x k, pitch SMAX, zero beyond k; rinv[i] =
// 1 / Rt[i][i] or 0) by back substitution with the column in registers:
// x[i] = -(sum_{l > i} Rt[i][l] x[l]) rinv[i] for i < c, x[c] = rinv[c].  The sum of row i
// starts with the newest entry x[i + 1], so a column is one chain of k^2 / 2 dependent
// products (about 17 cycles each).
template <int SMAX>
__device__ inline void tri_inverse_col(const double* Rt, const double* rinv, int c, double (&x)[SMAX]) {
#pragma unroll
  for (int i = SMAX - 1; i >= 0; --i) {
    double acc = 0.0;
#pragma unroll
    for (int l = i + 1; l < SMAX; ++l) acc = fma(Rt[i * SMAX + l], x[l], acc);
    const double ri = rinv[i];
    x[i] = i > c ? 0.0 : (i == c ? ri : -acc * ri);
  }
}

// Rank-revealing first pass: pivoted Cholesky of the s x s block Gram (pitch ldg).  Step j
// picks the largest remaining diagonal (ties to the smaller index; every wave finds the
// same pivot from its identical copy of the diagonal), the pivot row is exchanged through
// LDS and the remaining rows are updated; it stops at the first pivot <= thr or
// <= s 2^-52 d_0.  T (s x s, in LDS) = E R_11^{-1}: row rowid[i], column c holds
// (R_11^{-1})[i][c]; *kept = k, the number of pivots taken.  Rt (SMAX x SMAX) receives R_11 in
// pivot order and may be Gm's own memory.  All 256 threads call it; the caller synchronises
// before it reads T or *kept.
//
// What bounds it: one dependent chain per step in every wave (argmax, reciprocal root, LDS
// exchange, update).  Every lane forms the reciprocal root of its own diagonal beside the
// argmax, and nothing is stored in the loop: a pivoted row is not updated again, so lane l
// still holds its row of R, unscaled, at the end.  Both factorisations
// and inverses of a 30-column block take 39 us by themselves (44 us with the root after the
// exchange, a float64 argmax, and rows stored in the loop); 18 columns 23 us (38 us at the
// next multiple of sixteen).
template <int SMAX>
__device__ inline void qrcp_block(const double* Gm, int ldg, int s, double thr, double* T, int* kept, double* Rt,
                                  QrTailSmem<SMAX>& sm) {
  constexpr int CW = SMAX / 4;
  const int tid = threadIdx.x, l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), c0 = w * CW;
  const int lc = l < SMAX ? l : SMAX - 1;
  double r[CW];
#pragma unroll
  for (int t = 0; t < CW; ++t) r[t] = (l < s && c0 + t < s) ? Gm[l * ldg + c0 + t] : 0.0;
  double diag = l < s ? Gm[l * ldg + l] : 0.0;  // zero once pivoted
  if (tid < SMAX) { sm.rinv[tid] = 0.0; sm.pos[tid] = SMAX; }
  double floor = thr, mydiag = 0.0, myrinv = 0.0;
  int k = 0, mypos = SMAX;
  for (; k < s; ++k) {
    const double root = rsqrt_nr(diag);
    const int pv = wave_argmax_positive(diag);
    if (pv < 0) break;
    const double best = lane_value(diag, pv);
    if (k == 0) {  // the larger of the two; a NaN threshold stays, so that nothing passes it
      const double low = (double)s * 0x1p-52 * best;
      floor = thr < low ? low : thr;
    }
    if (!__builtin_amdgcn_readfirstlane(best > floor)) break;
    double* pb = sm.prow[k & 1];
    if (l == pv) {
#pragma unroll
      for (int t = 0; t < CW; ++t) pb[c0 + t] = r[t];
    }
    const double rinv = lane_value(root, pv);
    __syncthreads();
    const double pl = pb[lc];
    double pc[CW];
#pragma unroll
    for (int t = 0; t < CW; ++t) pc[t] = pb[c0 + t];
    // rows already pivoted (and lanes beyond s) take a zero factor: no divergent update
    const bool live = diag > 0.0 && l != pv;
    const double rl = live ? pl * rinv : 0.0;
    const double f = -rl * rinv;
#pragma unroll
    for (int t = 0; t < CW; ++t) r[t] = fma(f, pc[t], r[t]);
    mydiag = l == pv ? diag : mydiag;
    myrinv = l == pv ? rinv : myrinv;
    mypos = l == pv ? k : mypos;
    diag = live ? fma(-rl, rl, diag) : 0.0;
  }
  __syncthreads();  // Gm has been read, pos has been cleared
  if (w == 0 && mypos < SMAX) {
    sm.pos[l] = mypos;
    sm.rowid[mypos] = l;
    sm.rinv[mypos] = myrinv;
  }
  for (int e = tid; e < SMAX * SMAX; e += 256) Rt[e] = 0.0;
  for (int e = tid; e < s * s; e += 256) T[e] = 0.0;
  __syncthreads();
  if (mypos < SMAX) {
#pragma unroll
    for (int t = 0; t < CW; ++t) {
      const int p = sm.pos[c0 + t];
      if (p < SMAX && p >= mypos) Rt[mypos * SMAX + p] = (p == mypos ? mydiag : r[t]) * myrinv;
    }
  }
  __syncthreads();
  // column l of R_11^{-1} in registers (wave 0)
  if (w == 0) {
    double x[SMAX];
    tri_inverse_col<SMAX>(Rt, sm.rinv, l, x);
    if (l < k) {
#pragma unroll
      for (int i = 0; i < SMAX; ++i)
        if (i <= l) T[sm.rowid[i] * s + l] = x[i];
    }
    if (l == 0) *kept = k;
  }
}

// Second orthonormalisation pass: Gm (s x s, pitch ldg) = Q^T Q of a basis whose first
// k_in columns are non-zero and nearly orthonormal.  Cholesky of that leading block,
// Gm = R^T R; a column whose pivot is <= thresh is dropped (its row of R is zero, so it
// takes no part in the remaining factorisation).  T (s x s) = R^{-1} with the surviving
// columns packed first, zeros after; *kept_out = their number.  Every lane keeps its own
// diagonal and its reciprocal root is formed while the pivot row is exchanged; the rows of R
// are stored at the end, as in qrcp_block.  Rt may be Gm's own memory.  All 256 threads call it.
template <int SMAX>
__device__ inline void chol_inv_block(const double* Gm, int ldg, int s, int k_in, double thresh, double* T, int* kept_out,
                                      double* Rt, QrTailSmem<SMAX>& sm) {
  constexpr int CW = SMAX / 4;
  const int tid = threadIdx.x, l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), c0 = w * CW;
  const int lc = l < SMAX ? l : SMAX - 1;
  const int k = __builtin_amdgcn_readfirstlane(k_in < s ? k_in : s);
  double r[CW];
#pragma unroll
  for (int t = 0; t < CW; ++t) r[t] = (l < k && c0 + t < k) ? Gm[l * ldg + c0 + t] : 0.0;
  double diag = l < k ? Gm[l * ldg + l] : 0.0;
  double myrinv = 0.0, mydiag = 0.0;
  for (int j = 0; j < k; ++j) {
    double* pb = sm.prow[j & 1];
    if (l == j) {
#pragma unroll
      for (int t = 0; t < CW; ++t) pb[c0 + t] = r[t];
    }
    const double root = diag > thresh ? rsqrt_nr(diag) : 0.0;
    const double rinv = lane_value(root, j);
    __syncthreads();
    const double pl = pb[lc];
    double pc[CW];
#pragma unroll
    for (int t = 0; t < CW; ++t) pc[t] = pb[c0 + t];
    const double rl = (l > j && l < k) ? pl * rinv : 0.0;
    const double f = -rl * rinv;  // zero for rows at or above j and for dropped pivots
#pragma unroll
    for (int t = 0; t < CW; ++t) r[t] = fma(f, pc[t], r[t]);
    myrinv = l == j ? rinv : myrinv;
    mydiag = l == j ? diag : mydiag;
    diag = fma(f, pl, diag);
  }
  __syncthreads();  // Gm has been read
#pragma unroll
  for (int t = 0; t < CW; ++t) {
    const int c = c0 + t;
    if (l < SMAX) Rt[l * SMAX + c] = (l < k && c < k && c >= l) ? (c == l ? mydiag : r[t]) * myrinv : 0.0;
  }
  for (int e = tid; e < s * s; e += 256) T[e] = 0.0;
  if (w == 0 && l < SMAX) sm.rinv[l] = myrinv;
  __syncthreads();
  if (w == 0) {
    // packed positions of the surviving columns
    const bool kl = myrinv != 0.0;
    const uint64_t kb = __ballot(kl);
    if (l == 0) *kept_out = __popcll(kb);
    const int pc = __popcll(kb & ((1ull << l) - 1ull));
    double x[SMAX];
    tri_inverse_col<SMAX>(Rt, sm.rinv, l, x);
    if (kl) {
#pragma unroll
      for (int i = 0; i < SMAX; ++i)
        if (i <= l && ((kb >> i) & 1)) T[i * s + pc] = x[i];
    }
  }
}

}  // namespace ttr
