// Leading eigenpairs of small symmetric float64 matrices: the Rayleigh-Ritz matrix and the
// saturated Grams of the sweep, and the stand-alone ttr_sym_eig_top.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "eig_layout.h"
#include "kernels.h"
#include "qr_tail.h"
#include "wave_ops.h"

namespace ttr {

// ----------------------------------------------------------------------------------
// Leading eigenpairs of a symmetric n x n matrix (n <= kTopMaxN, r wanted pairs), for
// the Rayleigh-Ritz and saturated Gram steps that only keep the top r directions.
// 1. Householder reduction T = Q^T A Q to tridiagonal form.  A lives in registers:
//    entry (i, j) belongs to thread (i mod 16, j mod 16) of a 16 x 16 grid, so the
//    product A v is summed across the 16 lanes of one row group inside a wave (DPP).
//    The reflectors are kept in LDS, packed.
// 2. The r largest eigenvalues of T by multisection: gl lanes per eigenvalue count the
//    eigenvalues below gl interior points of the current interval (sign changes of
//    the leading principal minors of T - x I, rescaled by powers of two) and keep the
//    sub-interval that holds the wanted index.
// 3. Eigenvectors of T from twisted factorisations of T - lambda I (one forward and
//    one backward recurrence per vector), then two Cholesky-QR passes over all r
//    vectors (clustered eigenvalues give an orthonormal basis of the cluster).
// 4. Back-transformation z = Q y with the stored reflectors.
// Output: vals[0..r) decreasing, vecs[:, 0..r) (leading dimension n) unit vectors;
// a value at or below n 2^-52 vals[0] counts as unresolved and gets a zero value and a
// zero vector; vals[r..n) = 0.
// ----------------------------------------------------------------------------------
constexpr int kTopMaxN = 128;
constexpr int kTopMaxR = 64;
constexpr int kTopThreads = 256;

typedef double de_t __attribute__((ext_vector_type(2)));  // (d_i, e_{i-1}^2), the second 0 for i = 0

// Number of eigenvalues of the tridiagonal T below x: sign changes of p_i = det(T_i - x I),
// p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}, renormalised by a power of two every 4 steps; an
// exact zero counts as a sign change (tiny pivot).  One chain per lane, bound by the number of
// instructions: a change is the exclusive-or of two sign bits, zeros are looked for once per
// four steps (and the four repeated with them replaced; a NaN takes the same way), the next four rows are loaded ahead.
__device__ __forceinline__ int sturm_count(const de_t* __restrict__ de, int n, double x) {
  double pm = 1.0, p = de[0][0] - x;
  if (p == 0.0) p = -0x1p-1000;
  uint32_t c = (uint32_t)__double2hiint(p) >> 31;
  auto careful = [&](de_t v) {
    double pn = fma(v[0] - x, p, -v[1] * pm);
    if (pn == 0.0) pn = -0x1p-1000 * p;
    c += (pn < 0.0) != (p < 0.0);
    pm = p;
    p = pn;
  };
  int i = 1;
  if (i + 3 < n) {
    de_t a0 = de[1], a1 = de[2], a2 = de[3], a3 = de[4];
    for (;;) {
      const bool more = i + 7 < n;
      const int nx = more ? i + 4 : i;
      const de_t b0 = de[nx], b1 = de[nx + 1], b2 = de[nx + 2], b3 = de[nx + 3];
      const double p1 = fma(a0[0] - x, p, -a0[1] * pm);
      const double p2 = fma(a1[0] - x, p1, -a1[1] * p);
      const double p3 = fma(a2[0] - x, p2, -a2[1] * p1);
      const double p4 = fma(a3[0] - x, p3, -a3[1] * p2);
      if (__any(!(fabs(p1) > 0.0) || !(fabs(p2) > 0.0) || !(fabs(p3) > 0.0) || !(fabs(p4) > 0.0))) {
        careful(a0); careful(a1); careful(a2); careful(a3);
      } else {
        const uint32_t h0 = __double2hiint(p), h1 = __double2hiint(p1), h2 = __double2hiint(p2), h3 = __double2hiint(p3),
                       h4 = __double2hiint(p4);
        c += ((h0 ^ h1) >> 31) + ((h1 ^ h2) >> 31);
        c += ((h2 ^ h3) >> 31) + ((h3 ^ h4) >> 31);
        pm = p3;
        p = p4;
      }
      const int ex = max(__builtin_amdgcn_frexp_exp(p), __builtin_amdgcn_frexp_exp(pm));
      p = ldexp(p, -ex);
      pm = ldexp(pm, -ex);
      i += 4;
      if (!more) break;
      a0 = b0; a1 = b1; a2 = b2; a3 = b3;
    }
  }
  for (; i < n; ++i) careful(de[i]);
  return (int)c;
}

// Packed reflector storage: v_k (entries k+1..n-1) starts at refl_off(k).
__device__ inline int refl_off(int k, int n) { return k * (n - 1) - (k * (k - 1)) / 2; }

// Pivot used for the LDL^T / UDU^T recurrences: magnitudes below `tiny` become +-tiny.
__device__ inline double guard_pivot(double x, double tiny) { return fabs(x) < tiny ? (x < 0.0 ? -tiny : tiny) : x; }

// One panel of the Householder tridiagonalisation in k_eig_top: steps k = 16 KB + kc,
// kc = 0..15, with the register column KB a compile-time index.  Rows and columns below
// 16 KB are finished: their register blocks (a, b < KB) are neither read nor updated.
template <int NB, int KB>
__device__ inline void tri_panel(double (&A)[NB][NB], int n, double (*colb)[kTopMaxN], double (*pb)[kTopMaxN],
                                 double* __restrict__ Vs, double* __restrict__ dd, double* __restrict__ ee,
                                 double* __restrict__ taus) {
  constexpr int TG = 16;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int tr = tid / TG, tc = tid % TG;
  for (int kc = 0; kc < TG; ++kc) {
    const int k = KB * TG + kc;
    if (k + 2 >= n) break;
    double* col = colb[k & 1];
    double* p = pb[k & 1];
    if (tc == kc) {
#pragma unroll
      for (int a = KB; a < NB; ++a) col[tr + TG * a] = A[a][KB];
    }
    __syncthreads();
    double cr[NB], cc[NB];
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      cr[a] = col[tr + TG * a];
      cc[a] = col[tc + TG * a];
    }
    const int i1 = k + 1 + lane, i2 = i1 + 64;
    const double c1 = col[i1 < kTopMaxN ? i1 : 0], c2 = col[i2 < kTopMaxN ? i2 : 0];
    const double x0 = col[k + 1];
    // ||x(2:)||^2 over rows k+2 .. n-1 (c1 of lane 0 is x0 itself)
    double s = (lane > 0 && i1 < n ? c1 * c1 : 0.0) + (i2 < n ? c2 * c2 : 0.0);
    s = sum64(s);
    double tau = 0.0, beta = x0, scale = 0.0;
    if (s > 0.0) {
      const double nrm = sqrt(fma(x0, x0, s));
      beta = x0 >= 0.0 ? -nrm : nrm;
      tau = (beta - x0) * rcp_nr(beta);
      scale = rcp_nr(x0 - beta);
    }
    double vr[NB], vc[NB], w[NB];
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      const int i = tr + TG * a, j = tc + TG * a;
      vr[a] = i == k + 1 ? 1.0 : ((i > k + 1 && i < n) ? cr[a] * scale : 0.0);
      vc[a] = j == k + 1 ? 1.0 : ((j > k + 1 && j < n) ? cc[a] * scale : 0.0);
    }
#pragma unroll
    for (int a = KB; a < NB; ++a) {
      double t = 0.0;
#pragma unroll
      for (int b = KB; b < NB; ++b) t = fma(A[a][b], vc[b], t);
      w[a] = sum16(t);
    }
    if (tc == 0) {
#pragma unroll
      for (int a = KB; a < NB; ++a) p[tr + TG * a] = tau * w[a];
    }
    const double v1 = lane == 0 ? 1.0 : c1 * scale, v2 = c2 * scale;
    if (wid == 0) {
      const int o = refl_off(k, n) - (k + 1);
      if (i1 < n) Vs[o + i1] = v1;
      if (i2 < n) Vs[o + i2] = v2;
      if (lane == 0) { taus[k] = tau; ee[k] = beta; dd[k] = col[k]; }
    }
    __syncthreads();
    double pr[NB], pc[NB];
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      pr[a] = p[tr + TG * a];
      pc[a] = p[tc + TG * a];
    }
    const double q1 = p[i1 < kTopMaxN ? i1 : 0], q2 = p[i2 < kTopMaxN ? i2 : 0];
    const double sk = (i1 < n ? v1 * q1 : 0.0) + (i2 < n ? v2 * q2 : 0.0);
    const double K = 0.5 * tau * sum64(sk);
    double wc[NB];
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      const int i = tr + TG * a, j = tc + TG * a;
      w[a] = (i > k && i < n) ? fma(-K, vr[a], pr[a]) : 0.0;
      wc[a] = (j > k && j < n) ? fma(-K, vc[a], pc[a]) : 0.0;
    }
#pragma unroll
    for (int a = KB; a < NB; ++a)
#pragma unroll
      for (int b = KB; b < NB; ++b) A[a][b] -= vr[a] * wc[b] + w[a] * vc[b];
  }
}

template <int NB, int KB>
struct TriPanels {
  __device__ static void run(double (&A)[NB][NB], int n, double (*colb)[kTopMaxN], double (*pb)[kTopMaxN],
                             double* Vs, double* dd, double* ee, double* taus) {
    if (16 * KB + 2 >= n) return;
    tri_panel<NB, KB>(A, n, colb, pb, Vs, dd, ee, taus);
    TriPanels<NB, KB + 1>::run(A, n, colb, pb, Vs, dd, ee, taus);
  }
};
template <int NB>
struct TriPanels<NB, NB> {
  __device__ static void run(double (&)[NB][NB], int, double (*)[kTopMaxN], double (*)[kTopMaxN], double*, double*,
                             double*, double*) {}
};

// Back-transformation panel KB of k_eig_top: y <- H_k y for k = 16 KB + 15 down to 16 KB
// (k <= n - 3).  Rows below 16 KB are untouched by these reflectors, so only register
// blocks a >= KB take part, and only block KB (rows on both sides of k) and the last block
// (rows beyond n) need a mask.  Two reflectors at a time:
// H_{k-1} H_k y = y - f1 v_k - f2 v_{k-1}, f1 = tau_k v_k^T y,
// f2 = tau_{k-1} (v_{k-1}^T y - (v_{k-1}^T v_k) f1); the three dot products of a pair are
// summed over the 16 lanes of a column group together.
// Reflector v_k (entries k+1..n-1, v_k[k+1] = 1) read by the back-transformation: packed in
// LDS behind each other.
struct ReflPacked {
  const double* Vs;
  int n;
  __device__ double operator()(int k, int i) const { return Vs[refl_off(k, n) - (k + 1) + i]; }
};
constexpr int kBigPitch = 256;

template <int NB, int CB2, int KB, class Refl>
__device__ inline void back_panel(double (&yv)[NB][CB2], const Refl& refl, const double* __restrict__ taus, int n,
                                  int rg) {
  constexpr int TG = 16;
  auto load_v = [&](int k, double (&v)[NB]) {
#pragma unroll
    for (int a = KB; a < NB; ++a) {
      const int i = rg + TG * a;
      if (a == KB || a == NB - 1) {
        const int ic = i <= k ? k + 1 : (i < n ? i : n - 1);
        const double x = refl(k, ic);
        v[a] = (i > k && i < n) ? x : 0.0;
      } else {
        v[a] = refl(k, i);
      }
    }
  };
  int k = min(TG * KB + TG - 1, n - 3);
  if (k < TG * KB) return;
  if (((k - TG * KB) & 1) == 0) {  // odd count: one reflector first
    double va[NB];
    load_v(k, va);
    const double t0 = taus[k];
#pragma unroll
    for (int b = 0; b < CB2; ++b) {
      double x1 = 0.0;
#pragma unroll
      for (int a = KB; a < NB; ++a) x1 = fma(va[a], yv[a][b], x1);
      const double f = t0 * sum16(x1);
#pragma unroll
      for (int a = KB; a < NB; ++a) yv[a][b] = fma(-f, va[a], yv[a][b]);
    }
    --k;
  }
  // the next pair's reflectors are loaded while the current pair is applied
  double va[NB], vb[NB];
  if (k > TG * KB) {
    load_v(k, va);
    load_v(k - 1, vb);
  }
  for (; k > TG * KB; k -= 2) {
    const bool more = k - 2 > TG * KB;
    double na[NB], nb[NB];
    if (more) {
      load_v(k - 2, na);
      load_v(k - 3, nb);
    }
    const double ta = taus[k], tb = taus[k - 1];
    double cp = 0.0;
#pragma unroll
    for (int a = KB; a < NB; ++a) cp = fma(vb[a], va[a], cp);
    double d1[CB2], d2[CB2];
#pragma unroll
    for (int b = 0; b < CB2; ++b) {
      double x1 = 0.0, x2 = 0.0;
#pragma unroll
      for (int a = KB; a < NB; ++a) {
        x1 = fma(va[a], yv[a][b], x1);
        x2 = fma(vb[a], yv[a][b], x2);
      }
      d1[b] = sum16(x1);
      d2[b] = sum16(x2);
    }
    const double cab = sum16(cp);
#pragma unroll
    for (int b = 0; b < CB2; ++b) {
      const double f1 = ta * d1[b];
      const double f2 = tb * fma(-cab, f1, d2[b]);
#pragma unroll
      for (int a = KB; a < NB; ++a) yv[a][b] = fma(-f2, vb[a], fma(-f1, va[a], yv[a][b]));
    }
    if (more) {
#pragma unroll
      for (int a = KB; a < NB; ++a) {
        va[a] = na[a];
        vb[a] = nb[a];
      }
    }
  }
}

template <int NB, int CB2, int KB, class Refl>
struct BackPanels {
  __device__ static void run(double (&yv)[NB][CB2], const Refl& refl, const double* taus, int n, int rg) {
    back_panel<NB, CB2, KB>(yv, refl, taus, n, rg);
    BackPanels<NB, CB2, KB - 1, Refl>::run(yv, refl, taus, n, rg);
  }
};
template <int NB, int CB2, class Refl>
struct BackPanels<NB, CB2, -1, Refl> {
  __device__ static void run(double (&)[NB][CB2], const Refl&, const double*, int, int) {}
};

// Gershgorin bounds of T = (dd, ee) for the multisection, widened by rounding, and ||T||; the
// same bits in every wave.
struct TriBounds { double lo, hi, nrm; };
__device__ __forceinline__ TriBounds tri_bounds(const double* __restrict__ dd, const double* __restrict__ ee, int n) {
  const int lane = threadIdx.x & 63;
  double glo = 1e308, ghi = -1e308;
  for (int i = lane; i < n; i += 64) {
    const double el = i > 0 ? fabs(ee[i - 1]) : 0.0, er = i + 1 < n ? fabs(ee[i]) : 0.0;
    glo = fmin(glo, dd[i] - el - er);
    ghi = fmax(ghi, dd[i] + el + er);
  }
  TriBounds t;
  t.lo = min64(glo);
  t.hi = max64(ghi);
  t.nrm = fmax(fmax(fabs(t.lo), fabs(t.hi)), 0x1p-1000);
  const double fudge = 4.0 * (double)n * 0x1p-52 * t.nrm;
  t.lo -= fudge;
  t.hi += fudge;
  return t;
}

// Lanes per eigenvalue of the multisection: the most (at most 16) that bisect all r values in
// one round of four waves, 64 / gl groups in each.
static int multisect_lanes(int r) {
  int gl = 16;
  while (gl > 2 && (kTopThreads / 64) * (64 / gl) < r) --gl;
  return gl;
}

// lam[j - first], j = first + (group of this lane) < last: the j-th largest eigenvalue of T by
// multisection, gl lanes per value counting the eigenvalues below gl interior points.  Groups
// never straddle a wave: 64 / gl per wave, the last lanes of a wave idle.
__device__ __forceinline__ void multisect(const de_t* __restrict__ de, int n, const TriBounds& tb, int gl, int first, int last,
                                 double* __restrict__ lam) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const double tol = 4.0 * 0x1p-52 * tb.nrm;
  const double frac = 1.0 / (double)(gl + 1);
  const unsigned gmask = (gl >= 32) ? 0xFFFFFFFFu : ((1u << gl) - 1u);
  const int gpw = 64 / gl, gi = lane / gl, g = lane % gl;
  for (int j0 = first; j0 < last; j0 += nw * gpw) {
    const int j = j0 + wid * gpw + gi;
    if (gi < gpw && j < last) {
      const int idx = n - 1 - j;  // ascending index of the j-th largest eigenvalue
      double lo = tb.lo, hi = tb.hi;
      for (int it = 0; it < 96 && hi - lo > tol; ++it) {
        const double h = (hi - lo) * frac;
        const int c = sturm_count(de, n, lo + h * (double)(g + 1));
        const uint64_t ball = __ballot(c <= idx);
        const unsigned bits = (unsigned)(ball >> (gi * gl)) & gmask;
        const int top = bits ? 31 - __clz(bits) : -1;  // last point with <= idx values below it
        const double nlo = top >= 0 ? lo + h * (double)(top + 1) : lo;
        const double nhi = top < gl - 1 ? lo + h * (double)(top + 2) : hi;
        lo = nlo;
        hi = nhi;
      }
      if (g == 0) lam[j - first] = 0.5 * (lo + hi);
    }
  }
}

// Eigenvectors of T for the values j0 .. j0 + cnt - 1 (< r), column j - y0 of Y (pitch yp).
// Lane pair (2t, 2t+1) factors T - lambda I = L D L^T (forward) and = U R U^T (backward).  An
// isolated value takes the twisted vector: at the index k with the smallest |gamma_k| =
// |D_k + R_k - (d_k - lambda)|, z_k = 1, z_i = -L_i z_{i+1} (i < k), z_{i+1} = -U_i z_i (i >= k).
// A value within 1e-3 ||T|| of a neighbour instead takes two solves with L D L^T from a hashed
// right-hand side, so that the vectors of a cluster span its eigenspace.  Y's column holds R
// first.  lam holds the values from number l0 on; SD, SL, SU: n x bv; twist, inv: cnt entries.
//
// What bounds it: chains of n dependent steps per lane, so every loop loads the next four rows
// before it works on the present ones, zeros that need the three-term relation are looked for
// by a wave vote, and the final scaling runs on all threads.
__device__ __forceinline__ void tri_vectors(int n, int r, int j0, int cnt, int bv, const double* __restrict__ dd,
                                   const double* __restrict__ ee, const double* __restrict__ lam, int l0, double nrm,
                                   double* __restrict__ Y, int yp, int y0, double* __restrict__ SD,
                                   double* __restrict__ SL, double* __restrict__ SU, int* __restrict__ twist,
                                   double* __restrict__ inv) {
  const int tid = threadIdx.x, NT = blockDim.x;
  const double tiny = 0x1p-52 * nrm, cthr = 1e-3 * nrm;
  const int t = tid >> 1, side = tid & 1, j = j0 + t, yc = j - y0;
  const bool act = t < cnt && j < r;
  const double lj = act ? lam[j - l0] : 0.0;
  const bool clust =
      act && ((j > 0 && lam[j - 1 - l0] - lj < cthr) || (j + 1 < r && lj - lam[j + 1 - l0] < cthr));
  if (act && (side == 0 || !clust)) {
    // both lanes of a pair run the same instructions: side 0 forward (L, D: p = D),
    // side 1 backward (U, R: p = R, R kept in Y)
    double* Xo = side ? SU : SL;
    double* Po = side ? Y : SD;
    const int ps = side ? yp : bv, pc = side ? yc : t, sg = side ? -1 : 1;
    int ie = side ? n - 2 : 0;  // off-diagonal entry of the step; the diagonal one it updates is ie + (side ? 0 : 1)
    const int dof = side ? 0 : 1;
    double P = guard_pivot(dd[side ? n - 1 : 0] - lj, tiny);
    Po[(side ? n - 1 : 0) * ps + pc] = P;
    double e4[4], d4[4];
    auto load = [&](int i0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = min(max(i0 + sg * u, 0), n - 2 > 0 ? n - 2 : 0);
        e4[u] = ee[i];
        d4[u] = dd[i + dof];
      }
    };
    if (n > 1) load(ie);
    for (int st = 0; st + 1 < n; st += 4) {
      double ec[4], dc[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) { ec[u] = e4[u]; dc[u] = d4[u]; }
      load(ie + 4 * sg);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (st + u + 1 < n) {
          const double x = ec[u] * rcp_nr(P);
          Xo[ie * bv + t] = x;
          P = guard_pivot(fma(-x, ec[u], dc[u] - lj), tiny);
          Po[(ie + dof) * ps + pc] = P;
          ie += sg;
        }
      }
    }
  }
  __syncthreads();
  if (act && !clust) {
    // smallest |gamma_k|, the first of equal ones: each lane of the pair looks at half of the rows
    const int h = (n + 1) / 2, ka = side ? h : 0, kb = side ? n : h;
    int kbest = ka;
    double gbest = 1e308;
    for (int k = ka; k < kb; k += 4) {
      double gk[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int kk = min(k + u, n - 1);
        gk[u] = fabs(SD[kk * bv + t] + Y[kk * yp + yc] - (dd[kk] - lj));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k + u < kb && gk[u] < gbest) { gbest = gk[u]; kbest = k + u; }
    }
    const double go = __shfl_xor(gbest, 1, 64);
    const int ko = __shfl_xor(kbest, 1, 64);
    // side 0 holds the smaller indices: it wins ties; nothing below 1e308 leaves index 0
    if (side == 0) twist[t] = go < gbest ? ko : (gbest < 1e308 ? kbest : 0);
  }
  __syncthreads();
  if (act && !clust) {
    // side 0: z_i = -L_i z_{i+1} for i = kt-1 .. 0; side 1: z_{i+1} = -U_i z_i for
    // i = kt .. n-2 (a zero z takes the three-term relation instead)
    const int kt = twist[t];
    const double* X = side ? SU : SL;
    const int cs = side ? n - 1 - kt : kt, sg = side ? 1 : -1;
    int i = side ? kt : kt - 1;
    if (side == 0) Y[kt * yp + yc] = 1.0;
    double nn = side ? 0.0 : 1.0;
    double zp = 1.0, zpp = 0.0;
    double x4[4];
    auto load = [&](int i0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) x4[u] = X[min(max(i0 + sg * u, 0), n - 1) * bv + t];
    };
    load(i);
    for (int st = 0; st < cs; st += 4) {
      double xc[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) xc[u] = x4[u];
      load(i + 4 * sg);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (st + u < cs) {
          double z = -xc[u] * zp;
          if (__any(zp == 0.0)) {
            const bool nb = side ? i > 0 : i + 1 < n - 1;
            const int inb = side ? (i > 0 ? i - 1 : 0) : i + 1;
            if (zp == 0.0 && ee[i] != 0.0 && nb) z = -(ee[inb] / ee[i]) * zpp;
          }
          Y[(side ? i + 1 : i) * yp + yc] = z;
          nn = fma(z, z, nn);
          zpp = zp;
          zp = z;
          i += sg;
        }
      }
    }
    const double s = 1.0 / sqrt(nn + __shfl_xor(nn, 1, 64));
    if (side == 0) inv[t] = s;
  }
  if (act && clust && side == 0) {
    // x = (L D L^T)^{-1} b twice, in column yc of Y; b_i in [0.5, 1.5) from a hash of (i, j),
    // then the first solution scaled to unit length
    double scale = 1.0;
    for (int it = 0; it < 2; ++it) {
      double yv = 0.0;
      for (int i0 = 0; i0 < n; i0 += 4) {
        double l4[4], b4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = min(i0 + u, n - 1);
          l4[u] = SL[(i > 0 ? i - 1 : 0) * bv + t];
          const uint32_t hsh = (uint32_t)(i * 2654435761u) ^ (uint32_t)((j + 1) * 40503u);
          b4[u] = it == 0 ? 0.5 + (double)((hsh >> 8) & 0xFFFF) * (1.0 / 65536.0) : Y[i * yp + yc] * scale;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (i0 + u < n) {
            yv = i0 + u == 0 ? b4[u] : fma(-l4[u], yv, b4[u]);
            Y[(i0 + u) * yp + yc] = yv;
          }
        }
      }
      double xv = 0.0, nn = 0.0;
      for (int i0 = n - 1; i0 >= 0; i0 -= 4) {
        double l4[4], y4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = max(i0 - u, 0);
          l4[u] = SL[i * bv + t];
          y4[u] = Y[i * yp + yc] * rcp_nr(SD[i * bv + t]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (i0 - u >= 0) {
            xv = i0 - u == n - 1 ? y4[u] : fma(-l4[u], xv, y4[u]);
            Y[(i0 - u) * yp + yc] = xv;
            nn = fma(xv, xv, nn);
          }
        }
      }
      scale = nn > 0.0 ? 1.0 / sqrt(nn) : 0.0;
    }
    inv[t] = scale;
  }
  __syncthreads();
  const int nc = min(cnt, r - j0);
  for (int e = tid; e < n * nc; e += NT) {
    const int i = e / nc, c = e - i * nc;
    Y[i * yp + j0 - y0 + c] *= inv[c];
  }
  __syncthreads();
}

// Whether any of the r values lies in a cluster (their vectors then take two Cholesky-QR passes).
__device__ inline bool any_cluster(const double* __restrict__ lam, int r, double nrm) {
  const double cthr = 1e-3 * nrm;
  bool any = false;
  for (int j = 0; j + 1 < r; ++j) any |= lam[j] - lam[j + 1] < cthr;
  return any;
}

// Cholesky-QR of the n x r columns of Ys (pitch r + 1), `passes` times: Gram (one thread per
// entry), Cholesky on four waves (lane l holds row l, each wave a quarter of the columns), then
// every row of Ys solved against R in registers.  Dependent columns give zeros (rdiag = 0).  The
// solve loads RMAX entries from the start of every row of R: the shared memory behind Gm holds
// them (chol_qr_doubles).
template <int RMAX>
__device__ __forceinline__ void chol_qr(int n, int r, int passes, double* __restrict__ Ys, double* __restrict__ Gm,
                               double* __restrict__ Xi, double* __restrict__ rdiag, double (*colx)[64]) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, NT = blockDim.x;
  const int rp = r + 1;
  for (int pass = 0; pass < passes; ++pass) {
    for (int e = tid; e < r * (r + 1) / 2; e += NT) {
      int c1 = 0, rem = e;
      while (rem >= r - c1) { rem -= r - c1; ++c1; }
      const int c2 = c1 + rem;
      double sacc = 0.0;
#pragma unroll 8
      for (int i = 0; i < n; ++i) sacc = fma(Ys[i * rp + c1], Ys[i * rp + c2], sacc);
      Gm[c1 * rp + c2] = sacc;
    }
    __syncthreads();
    {  // R (upper, rows in Gm), 1 / R_jj in Xi[j]: lane l holds row l, wave w < 4 the columns
       // [w CW, (w+1) CW); the pivot row comes from lane k of each wave, the pivot column
       // (= row, by symmetry) through LDS from the wave that owns it
      constexpr int CW = RMAX / 4;
      const int c0 = wid * CW;
      double row[CW];
#pragma unroll
      for (int t = 0; t < CW; ++t) {
        const int c = c0 + t;
        row[t] = (wid < 4 && lane < r && c < r) ? (c >= lane ? Gm[lane * rp + c] : Gm[c * rp + lane]) : 0.0;
      }
      for (int k = 0; k < r; ++k) {
        double* cb = colx[k & 1];
        if (wid < 4 && k >= c0 && k < c0 + CW) {
          double cv = 0.0;
#pragma unroll
          for (int t = 0; t < CW; ++t) cv = (c0 + t == k) ? row[t] : cv;
          cb[lane] = cv;
        }
        __syncthreads();
        if (wid < 4) {
          const double d = cb[k];
          const double cl = cb[lane];
          const bool ok = d > 1e-20;
          const double rinv = ok ? rsqrt_nr(d) : 0.0;
          const double rl = (ok && lane > k && lane < r) ? cl * rinv : 0.0;
          const double f = -rl * rinv;
#pragma unroll
          for (int t = 0; t < CW; ++t) row[t] = fma(f, lane_value(row[t], k), row[t]);
          if (wid == 0 && lane > k && lane < r) Gm[k * rp + lane] = rl;
          if (tid == 0) { Xi[k] = rinv; rdiag[k] = ok ? d * rinv : 0.0; }
        }
      }
    }
    __syncthreads();
    for (int i = tid; i < n; i += NT) {  // y R = y_old, row by row (dependent columns give zeros)
      double y[RMAX];
#pragma unroll
      for (int jj = 0; jj < RMAX; ++jj) y[jj] = jj < r ? Ys[i * rp + jj] : 0.0;
#pragma unroll
      for (int c = 0; c < RMAX; ++c)
        if (c < r) {
          y[c] *= Xi[c];
#pragma unroll
          for (int jj = c + 1; jj < RMAX; ++jj) y[jj] = fma(-y[c], Gm[c * rp + jj], y[jj]);
          // row by row of R: all of them loaded ahead do not fit in the registers
          if constexpr (RMAX > 16) __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
      for (int jj = 0; jj < RMAX; ++jj)
        if (jj < r) Ys[i * rp + jj] = y[jj];
    }
    __syncthreads();
  }
}

// Parts 2-4 of the leading-eigenpair solver of k_eig_top, on the tridiagonal T = (dd, ee) of
// step 1 with its Householder reflectors (taus, refl).  Runs on kTopThreads threads; every
// array is shared memory except vecs, vals.
template <int NB, int RMAX, class Refl>
__device__ __forceinline__ void eig_top_tail(int n, int r, int bv, int gl, const double* __restrict__ dd,
                                    const double* __restrict__ ee, de_t* __restrict__ de,
                                    const double* __restrict__ taus, const Refl& refl, double* __restrict__ lam,
                                    double* __restrict__ rdiag, double (*colx)[64], int* __restrict__ twist,
                                    double* __restrict__ inv, double* __restrict__ Ys, double* __restrict__ Gm,
                                    double* __restrict__ Xi, double* __restrict__ SD, double* __restrict__ SL,
                                    double* __restrict__ SU, double* __restrict__ vecs, double* __restrict__ vals) {
  constexpr int TG = 16, NT = kTopThreads;
  const int tid = threadIdx.x, lane = tid & 63;
  const int rp = r + 1;
  for (int i = tid; i < n; i += NT) de[i] = de_t{dd[i], i > 0 ? ee[i - 1] * ee[i - 1] : 0.0};
  const TriBounds tb = tri_bounds(dd, ee, n);
  __syncthreads();
  // ---- 2. the r largest eigenvalues of T ----
  multisect(de, n, tb, gl, 0, r, lam);
  __syncthreads();
  // ---- 3. eigenvectors of T, orthonormalised ----
  const bool any_clust = any_cluster(lam, r, tb.nrm);
  for (int jb = 0; jb < r; jb += bv) tri_vectors(n, r, jb, bv, bv, dd, ee, lam, 0, tb.nrm, Ys, rp, 0, SD, SL, SU, twist, inv);
  chol_qr<RMAX>(n, r, any_clust ? 2 : 1, Ys, Gm, Xi, rdiag, colx);
  // ---- 4. back-transformation z = Q y with the stored reflectors, last first.  Thread
  //      (row group rg = lane % 16, column group cg = tid / 16) keeps rows rg + 16 a and
  //      columns cg + 16 b of y in registers; the dot products of a reflector with a column
  //      are summed over the 16 lanes of the column group (DPP), so no barrier is needed. ----
  constexpr int CB2 = RMAX / 16;
  const int rg = lane & 15, cg = tid >> 4;
  const double res = (double)n * 0x1p-52 * fmax(lam[0], 0.0);
  double yv[NB][CB2];
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < CB2; ++b) {
      const int i = rg + TG * a, c = cg + 16 * b;
      yv[a][b] = (c < r && i < n) ? Ys[i * rp + c] : 0.0;
    }
  // Reflectors are applied two at a time, panel by panel (k = 16 KB + 15 .. 16 KB): see
  // back_panel.
  BackPanels<NB, CB2, NB - 1, Refl>::run(yv, refl, taus, n, rg);
#pragma unroll
  for (int b = 0; b < CB2; ++b) {
    const int c = cg + 16 * b;
    if (c < r) {
      const bool keep = rdiag[c] > 0.0 && lam[c] > res;
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        const int i = rg + TG * a;
        if (i < n) vecs[i * n + c] = keep ? yv[a][b] : 0.0;
      }
      if (rg == 0) vals[c] = keep ? lam[c] : 0.0;
    }
  }
  for (int j = r + tid; j < n; j += NT) vals[j] = 0.0;
}

template <int NB, int RMAX>
__global__ __launch_bounds__(kTopThreads) void k_eig_top(const double* __restrict__ a_in, int n, int r,
                                                         double* __restrict__ vecs, double* __restrict__ vals, int bv,
                                                         int gl) {
  constexpr int TG = 16;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double colb[2][kTopMaxN], pb[2][kTopMaxN];
  __shared__ double dd[kTopMaxN], ee[kTopMaxN], taus[kTopMaxN];
  __shared__ de_t de[kTopMaxN];
  __shared__ double lam[kTopMaxR], rdiag[kTopMaxR], inv[kTopMaxR], colx[2][64];
  __shared__ int twist[kTopMaxR];
  const int tid = threadIdx.x;
  const int tr = tid / TG, tc = tid % TG;
  const int rp = r + 1;
  double* Vs = reinterpret_cast<double*>(smem);            // packed reflectors
  double* Ys = Vs + ((n * (n - 1) / 2 + 1) & ~1);          // n x rp eigenvectors of T, then of A
  double* Gm = Ys + n * rp;                                // r x rp Gram / R factor
  double* Xi = Gm + r * rp;                                // 1 / R_jj
  double* SD = Xi + r * rp;                                // twisted factorisations, [i * bv + t]
  double* SL = SD + n * bv;
  double* SU = SL + n * bv;

  // ---- 1. tridiagonalisation: every LDS operand of a step is read in one batch ----
  double A[NB][NB];
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int i = tr + TG * a, j = tc + TG * b;
      A[a][b] = (i < n && j < n) ? a_in[i * n + j] : 0.0;
    }
  TriPanels<NB, 0>::run(A, n, colb, pb, Vs, dd, ee, taus);
  {
    const int k0 = n >= 2 ? n - 2 : 0;
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int i = tr + TG * a, j = tc + TG * b;
        if (i == j && i >= k0 && i < n) dd[i] = A[a][b];
        if (n >= 2 && i == n - 1 && j == n - 2) ee[n - 2] = A[a][b];
      }
  }
  __syncthreads();
  eig_top_tail<NB, RMAX>(n, r, bv, gl, dd, ee, de, taus, ReflPacked{Vs, n}, lam, rdiag, colx, twist, inv, Ys, Gm, Xi,
                         SD, SL, SU, vecs, vals);
}

template <int NB, int RMAX>
static hipError_t launch_eig_top_r(const double* a, int n, int r, double* vecs, double* vals, hipStream_t st, int bv) {
  const size_t lds = eig_top_lds(n, r, bv);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_eig_top<NB, RMAX>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) { (void)hipGetLastError(); return e; }
  hipLaunchKernelGGL((k_eig_top<NB, RMAX>), dim3(1), dim3(kTopThreads), lds, st, a, n, r, vecs, vals, bv,
                     multisect_lanes(r));
  return hipGetLastError();
}

template <int NB>
static hipError_t launch_eig_top(const double* a, int n, int r, double* vecs, double* vals, hipStream_t st, int bv) {
  if (r <= 16) return launch_eig_top_r<NB, 16>(a, n, r, vecs, vals, st, bv);
  if (r <= 32) return launch_eig_top_r<NB, 32>(a, n, r, vecs, vals, st, bv);
  return launch_eig_top_r<NB, 64>(a, n, r, vecs, vals, st, bv);
}

// ----------------------------------------------------------------------------------
// Leading eigenpairs for kTopMaxN < n <= kMaxSmall (the Rayleigh-Ritz matrix of wide
// Krylov spaces, e.g. w = 200): the matrix no longer fits one work-group's registers or
// LDS, so step 1 runs on a copy in global memory (L2-resident: at most 512 KB) and the
// other steps follow on the tridiagonal form.
//
// k_tridiag_big: Householder tridiagonalisation (lower form, as in step 1 of k_eig_top)
// by 1024 threads.  Step k's rank-2 update A -= v w^T + w v^T is applied lazily, fused
// with step k+1's product p = tau A v: one pass over the trailing block per step.  The
// first k0 steps keep the matrix in global memory (L2-resident, rows of pitch kBigPitch;
// wave w owns rows i = w (mod 16), lane l columns l + 64 c).  From step k0 on the trailing
// block's lower triangle (rows and columns >= k0, packed by rows) fits in LDS and the
// product is split in two passes: rows (the update, and sum_{j <= i} A_ij v_j) then
// columns (sum_{i > j} A_ij v_j).  Eight lanes own the pair of rows (and of columns)
// k + 1 + a and n - 1 - a, whose lengths add up to the same count for every a, and sum
// them in a fixed order.  Row k (the symmetric copy of column k) is formed with the
// pending update, gives d_k, e_k and the reflector, which is stored in W[k][k+1..n) for
// the back-transformation.  W: n rows of pitch kBigPitch, then d, e, tau (kBigPitch each).
//
// n - 2 dependent steps bound it, each three barriers, a square root and a division, and two
// passes over the triangle at LDS and issue rate.  n = 200: 880 us with every wave repeating
// the scalars of a step and single columns at the ends of rows; 795 us with idle waves kept to
// the barriers, (v, w) in one load and masked last rounds.  Eight columns or rows a round in
// place of four took the registers to 128 and gave nothing.
// ----------------------------------------------------------------------------------
constexpr int kTriThreads = 1024;

__device__ inline double block_sum_tri(double v, double* red, int tid) {
  v = sum64(v);
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < kTriThreads / 64; ++w) t += red[w];  // fixed order: every thread the same sum
  __syncthreads();
  return t;
}

// An entry of the pending update; both of a pair come with one load.
struct alignas(16) vw_t { double v, w; };

// Offset of (i, j), j <= i, in the packed lower triangle of the block that starts at k0.
__device__ inline int tri_off(int i, int j, int k0) {
  const int a = i - k0;
  return a * (a + 1) / 2 + (j - k0);
}

// Step-k start shared by both storage forms: the reflector from xs (row k with the
// pending update), stored as d_k, e_k, tau_k and W[k][k+1..n); vc <- v.  Returns tau.
__device__ inline double tri_reflector(int n, int k, double* xs, double* red, double* s_sc, double* dg, double* eg,
                                       double* tg, double* W, vw_t* vc) {
  const int tid = threadIdx.x;
  double sq = 0.0;
  for (int i = k + 2 + tid; i < n; i += kTriThreads) sq += xs[i] * xs[i];
  sq = block_sum_tri(sq, red, tid);
  if (tid == 0) {
    const double x0 = xs[k + 1];
    double tau = 0.0, beta = x0, scale = 0.0;
    if (sq > 0.0) {
      const double nrm = sqrt(fma(x0, x0, sq));
      beta = x0 >= 0.0 ? -nrm : nrm;
      tau = (beta - x0) / beta;
      scale = 1.0 / (x0 - beta);
    }
    s_sc[0] = tau; s_sc[1] = scale;
    dg[k] = xs[k];
    eg[k] = beta;
    tg[k] = tau;
  }
  __syncthreads();
  const double tau = s_sc[0], scale = s_sc[1];
  for (int i = k + 1 + tid; i < n; i += kTriThreads) {
    const double v = i == k + 1 ? 1.0 : xs[i] * scale;
    vc[i].v = v;
    W[(int64_t)k * kBigPitch + i] = v;  // reflector k
  }
  if (tid == 0) vc[k].v = 0.0;
  __syncthreads();
  return tau;
}

// w = p - (tau/2 v^T p) v on the w of vw (holding p), then the pending update becomes (v, w).
__device__ inline void tri_finish_w(int n, int k, double tau, vw_t* vw, double* red) {
  const int tid = threadIdx.x;
  double kv = 0.0;
  for (int i = k + 1 + tid; i < n; i += kTriThreads) kv += vw[i].v * vw[i].w;
  const double K = 0.5 * tau * block_sum_tri(kv, red, tid);
  for (int i = k + 1 + tid; i < n; i += kTriThreads) vw[i].w = fma(-K, vw[i].v, vw[i].w);
  if (tid == 0) vw[k].w = 0.0;
  __syncthreads();
}

// Row pass of one LDS step for the pair of rows i1 <= i2 (i1 == i2: one row): the pending
// update A_ij -= v_i w_j + w_i v_j over j = k+1..i, written back, and sum_j A_ij c_j with
// the new reflector c_j = x_j scale (c_{k+1} = 1; x = row k, xs).  Lane q of eight takes
// j = k+1+q (mod 8); the vector entries (v_j, w_j) of a column are one load and serve both rows.
// Bound by instruction issue and the LDS round trips: all loads of a round are issued before its
// stores, and the last round is masked (its loads clamped to the row) rather than finished one
// column at a time.
template <int U, bool MASK, bool BOTH, bool FIRST>
__device__ __forceinline__ void tri_round(double* ra, double* rb, int j, int last, int kk, bool two, vw_t ca, vw_t cb,
                                          const vw_t* vw, const double* xs, double scale, double& pa, double& pb) {
  double av[U], bv[U], xv[U];
  vw_t wv[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int jc = MASK ? min(j + 8 * u, last) : j + 8 * u;
    if (BOTH) av[u] = ra[jc];
    bv[u] = rb[jc];
    wv[u] = vw[jc];
    xv[u] = xs[jc];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int jj = j + 8 * u;
    if (!MASK || jj <= last) {
      double c = xv[u] * scale;
      if (FIRST && u == 0) c = jj == kk ? 1.0 : c;
      if (BOTH) {
        const double x = av[u] - ca.v * wv[u].w - ca.w * wv[u].v;
        ra[jj] = x;
        pa = fma(x, c, pa);
      }
      if (!BOTH || two) {
        const double y = bv[u] - cb.v * wv[u].w - cb.w * wv[u].v;
        rb[jj] = y;
        pb = fma(y, c, pb);
      }
    }
  }
}

__device__ __forceinline__ void tri_row_pair(double* T, int k0, int k, int i1, int i2, int q, const vw_t* vw,
                                             const double* xs, double scale, double& p1, double& p2) {
  double* ra = T + (i1 - k0) * (i1 - k0 + 1) / 2 - k0;  // element (i1, j) at ra[j]
  double* rb = T + (i2 - k0) * (i2 - k0 + 1) / 2 - k0;
  const bool two = i2 != i1;
  const vw_t ca = vw[i1], cb = vw[i2];
  double pa = 0.0, pb = 0.0;
  const int j0 = k + 1 + q;
  // columns of both rows: column k + 1 is the first of lane 0
  int j = j0;
  if (j <= i1) {
    tri_round<4, true, true, true>(ra, rb, j, i1, k + 1, two, ca, cb, vw, xs, scale, pa, pb);
    for (j += 32; j + 24 <= i1; j += 32)
      tri_round<4, false, true, false>(ra, rb, j, i1, k + 1, two, ca, cb, vw, xs, scale, pa, pb);
    if (j <= i1) tri_round<4, true, true, false>(ra, rb, j, i1, k + 1, two, ca, cb, vw, xs, scale, pa, pb);
  }
  if (two) {  // the rest of row i2
    j = j0 + ((i1 - j0 + 8) >> 3) * 8;
    for (; j + 24 <= i2; j += 32)
      tri_round<4, false, false, false>(ra, rb, j, i2, k + 1, two, ca, cb, vw, xs, scale, pa, pb);
    if (j <= i2) tri_round<4, true, false, false>(ra, rb, j, i2, k + 1, two, ca, cb, vw, xs, scale, pa, pb);
  }
  p1 = pa;
  p2 = pb;
}

// Column pass for column j: sum_{r > j} A_rj v_r, lane q of eight taking r = j+1+q (mod 8), four
// rows per round, then the rest.
__device__ __forceinline__ double tri_col_pass(const double* T, int k0, int n, int j, int q, const vw_t* vc) {
  double part = 0.0;
  int r = j + 1 + q;
  int off = tri_off(r, j, k0);  // off(r + 8) = off(r) + 8 (r - k0) + 36
  for (; r + 24 < n; r += 32) {
    const int o1 = off + 8 * (r - k0) + 36;
    const int o2 = o1 + 8 * (r + 8 - k0) + 36;
    const int o3 = o2 + 8 * (r + 16 - k0) + 36;
    const double t0 = T[off], t1 = T[o1], t2 = T[o2], t3 = T[o3];
    const double c0 = vc[r].v, c1 = vc[r + 8].v, c2 = vc[r + 16].v, c3 = vc[r + 24].v;
    part = fma(t0, c0, part);
    part = fma(t1, c1, part);
    part = fma(t2, c2, part);
    part = fma(t3, c3, part);
    off = o3 + 8 * (r + 24 - k0) + 36;
  }
  if (r < n) {  // one to three rows
    const int o1 = r + 8 < n ? off + 8 * (r - k0) + 36 : off;
    const int o2 = r + 16 < n ? o1 + 8 * (r + 8 - k0) + 36 : off;
    const double t0 = T[off], t1 = T[o1], t2 = T[o2];
    const double c0 = vc[r].v, c1 = vc[min(r + 8, n - 1)].v, c2 = vc[min(r + 16, n - 1)].v;
    part = fma(t0, c0, part);
    if (r + 8 < n) part = fma(t1, c1, part);
    if (r + 16 < n) part = fma(t2, c2, part);
  }
  return part;
}

__global__ __launch_bounds__(kTriThreads) void k_tridiag_big(const double* __restrict__ a_in, int n,
                                                            double* __restrict__ W, int k0) {
  extern __shared__ double T[];  // packed lower triangle of rows / columns >= k0
  __shared__ vw_t vws[2][kBigPitch];
  __shared__ double xs[kBigPitch];
  __shared__ double red[kTriThreads / 64], redK[kTriThreads / 64];
  __shared__ double s_sc[2], s_x0[1];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  double* dg = W + (int64_t)n * kBigPitch;
  double* eg = dg + kBigPitch;
  double* tg = eg + kBigPitch;
  for (int e = tid; e < n * kBigPitch; e += kTriThreads) {
    const int i = e / kBigPitch, j = e % kBigPitch;
    W[e] = j < n ? a_in[(int64_t)i * n + j] : 0.0;
  }
  for (int i = tid; i < kBigPitch; i += kTriThreads) vws[0][i] = vw_t{0.0, 0.0};
  if (tid < kTriThreads / 64) redK[tid] = 0.0;
  __syncthreads();
  int cur = 0;  // vws[cur]: the update pending from the previous step
  int k = 0;
  for (; k + 2 < n && k < k0; ++k) {
    const vw_t* vp = vws[cur];
    for (int i = k + tid; i < n; i += kTriThreads)
      xs[i] = W[(int64_t)k * kBigPitch + i] - vp[k].v * vp[i].w - vp[k].w * vp[i].v;
    __syncthreads();
    vw_t* vc = vws[cur ^ 1];
    const double tau = tri_reflector(n, k, xs, red, s_sc, dg, eg, tg, W, vc);
    // fused: pending update of the trailing block, then p_i = tau sum_j A_ij v_j
    for (int i = k + 1 + wid; i < n; i += kTriThreads / 64) {
      double* row = W + (int64_t)i * kBigPitch;
      const double vpi = vp[i].v, wpi = vp[i].w;
      double part = 0.0;
#pragma unroll
      for (int c = 0; c < kBigPitch / 64; ++c) {
        const int j = lane + 64 * c;
        if (j > k && j < n) {
          const double a = row[j] - vpi * vp[j].w - wpi * vp[j].v;
          row[j] = a;
          part = fma(a, vc[j].v, part);
        }
      }
      part = sum64(part);
      if (lane == 0) vc[i].w = tau * part;  // p, turned into w below
    }
    __syncthreads();
    tri_finish_w(n, k, tau, vc, red);
    cur ^= 1;
  }
  if (k + 2 < n) {
    // the trailing block (rows and columns >= k = k0) moves to LDS, without the pending update
    for (int i = k + wid; i < n; i += kTriThreads / 64)
      for (int j = k + lane; j <= i; j += 64) T[tri_off(i, j, k0)] = W[(int64_t)i * kBigPitch + j];
    __syncthreads();
  }
  // LDS steps.  At the start of step k, vws[cur] holds v of step k - 1 and, as w, its
  // p = tau A v; its w = p - K v, K = kscale * (sum of redK), is completed by the owner of
  // each entry in phase X (K = 0 on entry: w itself is there).  A wave whose rows are used up
  // keeps only the barriers: its sums are zeros, and it takes no issue slots from the others.
  double kscale = 0.0;
  for (; k + 2 < n; ++k) {
    const int N = n - k - 1;  // rows and columns k + 1 .. n - 1
    if (wid * 64 >= N + 1 && wid * 8 >= (N + 1) / 2) {
      if (lane == 0) red[wid] = 0.0;
      __syncthreads();
      if (lane == 0) redK[wid] = 0.0;
      __syncthreads();
      __syncthreads();
      cur ^= 1;
      continue;
    }
    vw_t* vp = vws[cur];
    vw_t* vc = vws[cur ^ 1];
    double ks = 0.0;
#pragma unroll
    for (int w = 0; w < kTriThreads / 64; ++w) ks += redK[w];  // fixed order
    const double K = kscale * ks;
    // phase X: thread i - k forms w_i and row k's entry x_i with the pending update
    const int i = k + tid;
    const double vk = vp[k].v, wk = fma(-K, vk, vp[k].w);
    double x = 0.0, sq = 0.0;
    if (i < n) {
      const double vi = vp[i].v;
      const double wi = fma(-K, vi, vp[i].w);
      if (i > k) vp[i].w = wi;  // w_k stays p_k in LDS: every thread reads it above
      x = T[tri_off(i, k, k0)] - vk * wi - wk * vi;
      if (i >= k + 2) sq = x * x;
      if (i == k + 1) s_x0[0] = x;
      if (i == k) dg[k] = x;
      xs[i] = x;
    }
    sq = sum64(sq);
    if (lane == 0) red[wid] = sq;
    __syncthreads();
    // the reflector, by every thread from the same sums (row k fills at most kBigPitch / 64 waves)
    double sqs = 0.0;
#pragma unroll
    for (int w = 0; w < kBigPitch / 64; ++w) sqs += red[w];
    const double x0 = s_x0[0];
    double tau = 0.0, beta = x0, scale = 0.0;
    if (sqs > 0.0) {
      const double nrm = sqrt(fma(x0, x0, sqs));
      beta = x0 >= 0.0 ? -nrm : nrm;
      tau = (beta - x0) / beta;
      scale = 1.0 / (x0 - beta);
    }
    if (tid == 0) { eg[k] = beta; tg[k] = tau; }
    // v_i = x_i scale (v_{k+1} = 1): kept by its owner for the column pass and the next
    // step (visible after the row pass's barrier); the row pass forms it from xs itself
    if (i < n) {
      const double v = i == k ? 0.0 : (i == k + 1 ? 1.0 : x * scale);
      vc[i].v = v;
      if (i > k) W[(int64_t)k * kBigPitch + i] = v;  // reflector k
    }
    const int a = tid >> 3, q = tid & 7;
    const int i1 = k + 1 + a, i2 = n - 1 - a;  // i1 == i2: the middle row of an odd N
    const bool act = a < (N + 1) / 2, two = i2 != i1;
    double p1 = 0.0, p2 = 0.0;
    if (act) tri_row_pair(T, k0, k, i1, i2, q, vp, xs, scale, p1, p2);
    p1 = sum8(p1);
    p2 = sum8(p2);
    if (act && q == 0) {
      vc[i1].w = p1;
      if (two) vc[i2].w = p2;
    }
    __syncthreads();
    double c1 = 0.0, c2 = 0.0;
    if (act) {
      c1 = tri_col_pass(T, k0, n, i1, q, vc);
      if (two) c2 = tri_col_pass(T, k0, n, i2, q, vc);
    }
    c1 = sum8(c1);
    c2 = sum8(c2);
    double kv = 0.0;
    if (act && q == 0) {
      const double pa = tau * (vc[i1].w + c1);
      vc[i1].w = pa;
      kv = vc[i1].v * pa;
      if (two) {
        const double pb = tau * (vc[i2].w + c2);
        vc[i2].w = pb;
        kv = fma(vc[i2].v, pb, kv);
      }
    }
    kv = sum64(kv);
    if (lane == 0) redK[wid] = kv;
    kscale = 0.5 * tau;
    __syncthreads();
    cur ^= 1;
  }
  // the last 2 x 2 block with the update of the last step
  if (tid == 0) {
    const vw_t* vp = vws[cur];
    double ks = 0.0;
    for (int w = 0; w < kTriThreads / 64; ++w) ks += redK[w];
    const double K = kscale * ks;
    const int a = n - 2, b = n - 1;
    const double wa = fma(-K, vp[a].v, vp[a].w), wb = fma(-K, vp[b].v, vp[b].w);
    const bool lds = k0 <= a;
    const double aa = lds ? T[tri_off(a, a, k0)] : W[(int64_t)a * kBigPitch + a];
    const double bb = lds ? T[tri_off(b, b, k0)] : W[(int64_t)b * kBigPitch + b];
    const double ba = lds ? T[tri_off(b, a, k0)] : W[(int64_t)b * kBigPitch + a];
    dg[a] = aa - 2.0 * vp[a].v * wa;
    dg[b] = bb - 2.0 * vp[b].v * wb;
    eg[a] = ba - vp[b].v * wa - wb * vp[a].v;
    tg[a] = 0.0;
    tg[b] = 0.0;
  }
}

// Static LDS of k_tridiag_big (vectors, sums, scalars) and its first LDS step: the smallest
// k0 whose trailing lower triangle (n - k0 rows) fits in the rest of the LDS.
constexpr size_t kTriStaticBytes = (5 * kBigPitch + 2 * (kTriThreads / 64) + 3) * sizeof(double);
static void tri_lds_plan(int n, int* k0, size_t* bytes) {
  const size_t budget = (kLdsBytes - kTriStaticBytes - 256) / sizeof(double);
  int m0 = n;
  while (m0 > 0 && (size_t)m0 * (m0 + 1) / 2 > budget) --m0;
  *k0 = n - m0;
  *bytes = (size_t)m0 * (m0 + 1) / 2 * sizeof(double);
}

// ----------------------------------------------------------------------------------
// Steps 2-4 on the tridiagonal form of k_tridiag_big, two launches.
//
// k_tri_vectors: work-groups 0 .. ne-1 find kVecPer eigenvalues each (and one neighbour on
// either side, which the cluster rule looks at) and their eigenvectors of T, the rest form the
// T factor of one compact-WY panel each.  As one work-group with everything in its LDS the 32
// vectors of n = 200 went through in three batches and the panels' inner products in another
// launch on one CU.  n = 200, r = 32: 340 + 172 us so, 234 + 172 us now with the Cholesky-QR
// in the second.
//
// The back-transformation is vecs <- Q vecs with Q = H_0 H_1 ... H_{n-3} in panels of kWyPanel
// reflectors applied last panel first.  Panel p (reflectors k0 = 16 p ...) is P = I - V T V^T
// with T upper triangular: T_jj = tau_j and column j above the diagonal -tau_j T (V_{<j}^T v_j)
// (row a of T in lane a).  Row a of panel p's T goes to the free front of a row of W (reflector
// k occupies columns k + 1 .. of row k).
//
// k_back_wy: one work-group of 1024 threads takes the vectors of T through the Cholesky-QR and
// then the panels, three small products each over Y held in LDS: X = V^T Y, X <- T X,
// Y <- Y - V X; the next panel's reflectors are loaded while one is applied.
// ----------------------------------------------------------------------------------
constexpr int kVecPer = 8;
constexpr int kVecThreads = 256;
constexpr int kWyThreads = 1024;
constexpr int kWyPairs = kWyPanel * (kWyPanel - 1) / 2;

__device__ inline int64_t wy_t_row(int pn, int a, int n) {
  // rows 0 .. 15 hold fewer than 16 free entries: panel 0 uses the columns behind the last rows'
  return pn > 0 ? (int64_t)(pn * kWyPanel + a) * kBigPitch : (int64_t)(n - kWyPanel + a) * kBigPitch + kWyPanel;
}

__global__ __launch_bounds__(kVecThreads) void k_tri_vectors(double* __restrict__ W, int n, int r, int ne, int gl,
                                                             double* __restrict__ vecs, double* __restrict__ vals) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double dd[kBigPitch], ee[kBigPitch];
  __shared__ de_t de[kBigPitch];
  __shared__ double lam[kVecPer + 2], inv[kVecPer];
  __shared__ int twist[kVecPer];
  const int tid = threadIdx.x;
  const double* dg = W + (int64_t)n * kBigPitch;
  if ((int)blockIdx.x < ne) {
    double* Y = reinterpret_cast<double*>(smem);  // n x kVecPer, then the factorisations
    double* SD = Y + n * kVecPer;
    double* SL = SD + n * kVecPer;
    double* SU = SL + n * kVecPer;
    for (int i = tid; i < n; i += kVecThreads) {
      dd[i] = dg[i];
      ee[i] = i + 1 < n ? dg[kBigPitch + i] : 0.0;
    }
    __syncthreads();
    for (int i = tid; i < n; i += kVecThreads) de[i] = de_t{dd[i], i > 0 ? ee[i - 1] * ee[i - 1] : 0.0};
    const TriBounds tb = tri_bounds(dd, ee, n);
    __syncthreads();
    const int j0 = blockIdx.x * kVecPer, first = max(j0 - 1, 0), last = min(j0 + kVecPer + 1, r);
    multisect(de, n, tb, gl, first, last, lam);  // lam[j - first] is eigenvalue j
    __syncthreads();
    tri_vectors(n, r, j0, kVecPer, kVecPer, dd, ee, lam, first, tb.nrm, Y, kVecPer, j0, SD, SL, SU, twist, inv);
    const int nc = min(kVecPer, r - j0);
    for (int e = tid; e < n * nc; e += kVecThreads) {
      const int i = e / nc, c = e - i * nc;
      vecs[(int64_t)i * n + j0 + c] = Y[i * kVecPer + c];
    }
    if (tid < nc) vals[j0 + tid] = lam[j0 + tid - first];
    if (blockIdx.x == 0 && tid == 0) W[(int64_t)(n + 2) * kBigPitch + kBigPitch - 1] = tb.nrm;  // tau_{255} is never used
    return;
  }
  // T factor of panel pn: inner products v_{k0+a} . v_{k0+b} over rows i > k0 + b, then row a of
  // T in lane a: T_aj = -tau_j sum_{b=a}^{j-1} T_ab G_bj (j > a)
  constexpr int P = kWyPanel;
  const int pn = (int)blockIdx.x - ne, k0 = pn * P, kc = min(P, n - 2 - k0);
  double* V = reinterpret_cast<double*>(smem);  // kc x n, reflector by reflector
  double* Gs = V + P * n;
  const double* taus = W + (int64_t)(n + 2) * kBigPitch;
  for (int e = tid; e < kc * n; e += kVecThreads) {
    const int k = e / n, i = e - k * n;
    V[e] = i > k0 + k ? W[(int64_t)(k0 + k) * kBigPitch + i] : 0.0;
  }
  __syncthreads();
  if (tid < kWyPairs) {
    int q = tid, b = 1;
    while (q >= b) { q -= b; ++b; }  // pair (a = q, b), a < b
    double g = 0.0;
    if (b < kc) {
      const double* va = V + q * n;
      const double* vb = V + b * n;
#pragma unroll 8
      for (int i = k0 + b + 1; i < n; ++i) g = fma(va[i], vb[i], g);
    }
    Gs[tid] = g;
  }
  __syncthreads();
  if (tid < P) {
    const int a = tid;
    double trow[P];
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const double tj = j < kc ? taus[k0 + j] : 0.0;
      double v = 0.0;
      if (j == a) {
        v = tj;
      } else if (j > a) {
        double acc = 0.0;
#pragma unroll
        for (int b = 0; b < j; ++b)
          if (b >= a) acc = fma(trow[b], Gs[j * (j - 1) / 2 + b], acc);
        v = -tj * acc;
      }
      trow[j] = v;
    }
    if (a < kc) {
      double* out = W + wy_t_row(pn, a, n);
#pragma unroll
      for (int j = 0; j < P; ++j) out[j] = trow[j];
    }
  }
}

static size_t tri_vectors_lds(int n) {
  return std::max((size_t)4 * n * kVecPer, (size_t)kWyPanel * n + kWyPairs) * sizeof(double);
}

template <int RMAX>
__global__ __launch_bounds__(kWyThreads) void k_back_wy(const double* __restrict__ W, int n, int r,
                                                        double* __restrict__ vecs, double* __restrict__ vals) {
  constexpr int P = kWyPanel;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double lam[kTopMaxR], rdiag[kTopMaxR], colx[2][64], Ts[P * P];
  const int rp = r + 1;
  const int npan = (n - 3) / P + 1;  // reflectors 0 .. n - 3
  double* Ys = reinterpret_cast<double*>(smem);  // n x rp
  double* Vp = Ys + n * rp;                      // n x (P + 1): the current panel, zero where v is
  double* Xs = Vp + n * (P + 1);                 // P x rp
  double* Gm = Xs + P * rp;                      // r x rp Gram / R factor
  double* Xi = Gm + r * rp;                      // 1 / R_jj
  const int tid = threadIdx.x;
  for (int e = tid; e < n * r; e += kWyThreads) Ys[(e / r) * rp + e % r] = vecs[(int64_t)(e / r) * n + e % r];
  for (int j = tid; j < r; j += kWyThreads) lam[j] = vals[j];
  // the panel's reflectors: entry i of reflector j by thread (i = tid / 16 + 64 u, j = tid % 16)
  constexpr int VU = kBigPitch * P / kWyThreads;
  double vn[VU], tn = 0.0;
  auto load_panel = [&](int pn) {
    const int k0 = pn * P, kc = min(P, n - 2 - k0), j = tid % P, k = k0 + j;
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int i = tid / P + (kWyThreads / P) * u;
      vn[u] = (j < kc && i > k && i < n) ? W[(int64_t)k * kBigPitch + i] : 0.0;
    }
    if (tid < P * P) tn = tid / P < kc ? W[wy_t_row(pn, tid / P, n) + tid % P] : 0.0;
  };
  load_panel(npan - 1);
  const double nrm = W[(int64_t)(n + 2) * kBigPitch + kBigPitch - 1];
  __syncthreads();
  chol_qr<RMAX>(n, r, any_cluster(lam, r, nrm) ? 2 : 1, Ys, Gm, Xi, rdiag, colx);
  const double res0 = (double)n * 0x1p-52 * fmax(lam[0], 0.0);
  for (int e = tid; e < n * r; e += kWyThreads) {
    const int i = e / r, c = e % r;
    if (!(rdiag[c] > 0.0 && lam[c] > res0)) Ys[i * rp + c] = 0.0;
  }
  for (int pn = npan - 1; pn >= 0; --pn) {
    const int k0 = pn * P;
    const int kc = min(P, n - 2 - k0);  // reflectors of this panel
    __syncthreads();
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int i = tid / P + (kWyThreads / P) * u;
      if (i < n) Vp[i * (P + 1) + tid % P] = vn[u];
    }
    if (tid < P * P) Ts[tid] = tn;
    if (pn > 0) load_panel(pn - 1);
    __syncthreads();
    {  // X = V^T Y: two lanes per entry (alternate rows), summed by one lane exchange
      const int ent = tid >> 1, h = tid & 1;
      const int j = ent / RMAX, c = ent % RMAX;
      double acc = 0.0;
      if (j < kc && c < r) {
#pragma unroll 8
        for (int i = k0 + 1 + j + h; i < n; i += 2) acc = fma(Vp[i * (P + 1) + j], Ys[i * rp + c], acc);
      }
      acc += dpp_mov<0xB1>(acc);
      if (h == 0 && j < P && c < r) Xs[j * rp + c] = acc;
    }
    __syncthreads();
    double x2 = 0.0;
    const int j2 = tid / RMAX, c2 = tid % RMAX;
    if (j2 < kc && c2 < r) {
      const double* T = Ts + j2 * P;
#pragma unroll
      for (int b = 0; b < P; ++b)
        if (b >= j2 && b < kc) x2 = fma(T[b], Xs[b * rp + c2], x2);
    }
    __syncthreads();
    if (j2 < P && c2 < r) Xs[j2 * rp + c2] = x2;
    __syncthreads();
    for (int e = tid; e < (n - k0 - 1) * r; e += kWyThreads) {
      const int i = k0 + 1 + e / r, c = e % r;
      double acc = Ys[i * rp + c];
#pragma unroll
      for (int j = 0; j < P; ++j) acc = fma(-Vp[i * (P + 1) + j], Xs[j * rp + c], acc);
      Ys[i * rp + c] = acc;
    }
  }
  __syncthreads();
  for (int e = tid; e < n * r; e += kWyThreads) vecs[(int64_t)(e / r) * n + e % r] = Ys[(e / r) * rp + e % r];
  for (int c = tid; c < n; c += kWyThreads) vals[c] = (c < r && rdiag[c] > 0.0 && lam[c] > res0) ? lam[c] : 0.0;
}

template <int RMAX>
static hipError_t launch_eig_top_big(const double* a, int n, int r, double* vecs, double* vals, double* work,
                                     hipStream_t st) {
  int k0 = 0;
  size_t tri_bytes = 0;
  tri_lds_plan(n, &k0, &tri_bytes);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_tridiag_big),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)tri_bytes);
  if (e != hipSuccess) { (void)hipGetLastError(); return e; }
  hipLaunchKernelGGL(k_tridiag_big, dim3(1), dim3(kTriThreads), tri_bytes, st, a, n, work, k0);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const size_t lds = tri_vectors_lds(n);
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_tri_vectors), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)lds);
  if (e != hipSuccess) { (void)hipGetLastError(); return e; }
  const int ne = (r + kVecPer - 1) / kVecPer, npan = (n - 3) / kWyPanel + 1;
  hipLaunchKernelGGL(k_tri_vectors, dim3(ne + npan), dim3(kVecThreads), lds, st, work, n, r, ne, multisect_lanes(r), vecs,
                     vals);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const size_t wy = back_wy_lds(n, r);
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_back_wy<RMAX>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)wy);
  if (e != hipSuccess) { (void)hipGetLastError(); return e; }
  hipLaunchKernelGGL((k_back_wy<RMAX>), dim3(1), dim3(kWyThreads), wy, st, work, n, r, vecs, vals);
  return hipGetLastError();
}

hipError_t sym_eig_top(const double* a, int n, int r, double* vecs, double* vals, double* work, hipStream_t st) {
  if (n <= 0 || r <= 0) return hipErrorInvalidValue;
  if (r > n) r = n;
  // largest batch of twisted factorisations that fits next to the static arrays (~12 KB)
  const size_t budget = kLdsBytes - 14 * 1024;
  int bv = r < kTopThreads / 2 ? r : kTopThreads / 2;
  while (bv > 1 && eig_top_lds(n, r, bv) > budget) --bv;
  if (n > kTopMaxN && n <= kBigPitch && r <= 32 && work) {
    if (r <= 16) return launch_eig_top_big<16>(a, n, r, vecs, vals, work, st);
    return launch_eig_top_big<32>(a, n, r, vecs, vals, work, st);
  }
  if (n > kTopMaxN || r > kTopMaxR || eig_top_lds(n, r, bv) > budget) {
    const hipError_t e = sym_eig(a, n, vecs, vals, work, st);
    if (e != hipSuccess || r == n) return e;
    return axpby(1, n - r, 0.0, nullptr, 0, 0.0, vals + r, n, nullptr, st);  // vals[r..n) = 0
  }
  switch ((n + 15) / 16) {
    case 1: return launch_eig_top<1>(a, n, r, vecs, vals, st, bv);
    case 2: return launch_eig_top<2>(a, n, r, vecs, vals, st, bv);
    case 3: return launch_eig_top<3>(a, n, r, vecs, vals, st, bv);
    case 4: return launch_eig_top<4>(a, n, r, vecs, vals, st, bv);
    case 5: return launch_eig_top<5>(a, n, r, vecs, vals, st, bv);
    case 6: return launch_eig_top<6>(a, n, r, vecs, vals, st, bv);
    case 7: return launch_eig_top<7>(a, n, r, vecs, vals, st, bv);
    default: return launch_eig_top<8>(a, n, r, vecs, vals, st, bv);
  }
}

}  // namespace ttr
