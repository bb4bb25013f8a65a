// Small dense float64 kernels of the sweep: the m x w and w x w side of every mode
// (projections between Krylov blocks, Gram matrices, SVQB orthonormalisation,
// Rayleigh-Ritz, completion).
#include <hip/hip_runtime.h>

#include "common.h"
#include "convert.h"
#include "kernels.h"
#include "wave_ops.h"

namespace ttr {

template <typename T> __device__ inline double ld_as_double(const T* p, int64_t i) { return (double)p[i]; }

// ----------------------------------------------------------------------------------
// C = alpha X^T Y + beta C (or split-K partials), 16 x 16 output tile per work-group.
// ----------------------------------------------------------------------------------
// Split-K: at most kTnMaxChunks row chunks of at least kTnRowsPerChunk rows each (one
// 64-row LDS block per work-group at the sweep's m = 960, so a work-group waits for one
// round of loads).
constexpr int kTnRowsPerChunk = 64;
constexpr int kTnMaxChunks = 15;

template <typename TX, typename TY, typename TC>
__global__ __launch_bounds__(256) void k_gemm_tn(int64_t m, int ka, int kb, const TX* __restrict__ X, int64_t ldx,
                                                 const TY* __restrict__ Y, int64_t ldy, double alpha, double beta,
                                                 TC* __restrict__ C, int64_t ldc, double* __restrict__ part,
                                                 int64_t rows_per_chunk) {
  __shared__ double Xs[64][17];
  __shared__ double Ys[64][17];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int a0 = blockIdx.x * 16, b0 = blockIdx.y * 16;
  const int64_t r0 = (int64_t)blockIdx.z * rows_per_chunk;
  const int64_t r1 = r0 + rows_per_chunk < m ? r0 + rows_per_chunk : m;
  // four interleaved partial sums (rows rr = 4i + q go to q), added in a fixed order
  double acc4[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t rb = r0; rb < r1; rb += 64) {
    for (int e = threadIdx.x; e < 64 * 16; e += 256) {
      const int rr = e >> 4, cc = e & 15;
      const int64_t row = rb + rr;
      Xs[rr][cc] = (row < r1 && a0 + cc < ka) ? (double)X[row * ldx + a0 + cc] : 0.0;
      Ys[rr][cc] = (row < r1 && b0 + cc < kb) ? (double)Y[row * ldy + b0 + cc] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int rr = 0; rr < 64; rr += 4)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc4[q] = fma(Xs[rr + q][ty], Ys[rr + q][tx], acc4[q]);
    __syncthreads();
  }
  const double acc = (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]);
  const int a = a0 + ty, b = b0 + tx;
  if (a < ka && b < kb) {
    if (part) {
      part[(int64_t)blockIdx.z * ka * kb + (int64_t)a * kb + b] = acc;
    } else {
      const double old = beta != 0.0 ? (double)C[(int64_t)a * ldc + b] : 0.0;
      C[(int64_t)a * ldc + b] = (TC)(alpha * acc + beta * old);
    }
  }
}

template <typename TC>
__global__ __launch_bounds__(256) void k_gemm_tn_finish(const double* __restrict__ part, int chunks, int ka, int kb,
                                                        double alpha, double beta, TC* __restrict__ C, int64_t ldc) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= ka * kb) return;
  const int a = idx / kb, b = idx % kb;
  double acc = 0.0;
  for (int z = 0; z < chunks; ++z) acc += part[(int64_t)z * ka * kb + idx];
  const double old = beta != 0.0 ? (double)C[(int64_t)a * ldc + b] : 0.0;
  C[(int64_t)a * ldc + b] = (TC)(alpha * acc + beta * old);
}

template <typename TX, typename TY>
static hipError_t gemm_tn_t(int64_t m, int ka, int kb, const TX* X, int64_t ldx, const TY* Y, int64_t ldy,
                            double alpha, double beta, void* C, int cdt, int64_t ldc, double* scratch,
                            hipStream_t st) {
  int64_t chunks = (m + kTnRowsPerChunk - 1) / kTnRowsPerChunk;
  if (chunks > kTnMaxChunks) chunks = kTnMaxChunks;
  if (chunks < 1 || scratch == nullptr) chunks = 1;
  const int64_t rpc = (m + chunks - 1) / chunks;
  const dim3 grid((ka + 15) / 16, (kb + 15) / 16, (unsigned)chunks);
  const bool split = chunks > 1;
  if (cdt == TTR_F64) {
    hipLaunchKernelGGL((k_gemm_tn<TX, TY, double>), grid, dim3(256), 0, st, m, ka, kb, X, ldx, Y, ldy, alpha, beta,
                       (double*)C, ldc, split ? scratch : nullptr, rpc);
    if (split)
      hipLaunchKernelGGL((k_gemm_tn_finish<double>), dim3((ka * kb + 255) / 256), dim3(256), 0, st, scratch,
                         (int)chunks, ka, kb, alpha, beta, (double*)C, ldc);
  } else {
    hipLaunchKernelGGL((k_gemm_tn<TX, TY, float>), grid, dim3(256), 0, st, m, ka, kb, X, ldx, Y, ldy, alpha, beta,
                       (float*)C, ldc, split ? scratch : nullptr, rpc);
    if (split)
      hipLaunchKernelGGL((k_gemm_tn_finish<float>), dim3((ka * kb + 255) / 256), dim3(256), 0, st, scratch,
                         (int)chunks, ka, kb, alpha, beta, (float*)C, ldc);
  }
  return hipGetLastError();
}

template <typename TX>
static hipError_t gemm_tn_x(int64_t m, int ka, int kb, const TX* X, int64_t ldx, const void* Y, int ydt,
                            int64_t ldy, double alpha, double beta, void* C, int cdt, int64_t ldc, double* scratch,
                            hipStream_t st) {
  if (ydt == TTR_F64) return gemm_tn_t(m, ka, kb, X, ldx, (const double*)Y, ldy, alpha, beta, C, cdt, ldc, scratch, st);
  if (ydt == TTR_F32) return gemm_tn_t(m, ka, kb, X, ldx, (const float*)Y, ldy, alpha, beta, C, cdt, ldc, scratch, st);
  return gemm_tn_t(m, ka, kb, X, ldx, (const __bf16*)Y, ldy, alpha, beta, C, cdt, ldc, scratch, st);
}

hipError_t gemm_tn(int64_t m, int ka, int kb, const void* X, int xdt, int64_t ldx, const void* Y, int ydt,
                   int64_t ldy, double alpha, double beta, void* C, int cdt, int64_t ldc, double* scratch,
                   hipStream_t st) {
  if (ka <= 0 || kb <= 0) return hipSuccess;
  if (xdt == TTR_F64) return gemm_tn_x(m, ka, kb, (const double*)X, ldx, Y, ydt, ldy, alpha, beta, C, cdt, ldc, scratch, st);
  if (xdt == TTR_F32) return gemm_tn_x(m, ka, kb, (const float*)X, ldx, Y, ydt, ldy, alpha, beta, C, cdt, ldc, scratch, st);
  return gemm_tn_x(m, ka, kb, (const __bf16*)X, ldx, Y, ydt, ldy, alpha, beta, C, cdt, ldc, scratch, st);
}

// Symmetric part of the summed split-K partials, C (k x k) = (S + S^T) / 2: work-group
// (bx, by) sums the 16 x 16 tile (bx, by) and its mirror tile (by, bx), both along rows,
// and meets the mirror's transpose through LDS.
__global__ __launch_bounds__(256) void k_gemm_tn_finish_sym(const double* __restrict__ part, int chunks, int k,
                                                            double* __restrict__ C, int64_t ldc) {
  __shared__ double mir[16][17];
  const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
  const int a0 = blockIdx.y * 16, b0 = blockIdx.x * 16;
  const int64_t kk = (int64_t)k * k;
  double s1 = 0.0, s2 = 0.0;
  if (a0 + ty < k && b0 + tx < k)
    for (int z = 0; z < chunks; ++z) s1 += part[z * kk + (int64_t)(a0 + ty) * k + b0 + tx];
  if (b0 + ty < k && a0 + tx < k)
    for (int z = 0; z < chunks; ++z) s2 += part[z * kk + (int64_t)(b0 + ty) * k + a0 + tx];
  mir[ty][tx] = s2;  // S[b0 + ty][a0 + tx]
  __syncthreads();
  if (a0 + ty < k && b0 + tx < k) C[(int64_t)(a0 + ty) * ldc + b0 + tx] = 0.5 * (s1 + mir[tx][ty]);
}

hipError_t gemm_tn_sym(int64_t m, int k, const double* X, int64_t ldx, const double* Y, int64_t ldy, double* C,
                       int64_t ldc, double* scratch, hipStream_t st) {
  if (k <= 0) return hipSuccess;
  if (ldc != k) return hipErrorInvalidValue;
  int64_t chunks = (m + kTnRowsPerChunk - 1) / kTnRowsPerChunk;
  if (chunks > kTnMaxChunks) chunks = kTnMaxChunks;
  if (chunks < 2 || scratch == nullptr) {
    // one chunk: the product, then the symmetric part in place
    const hipError_t e = gemm_tn_t(m, k, k, X, ldx, Y, ldy, 1.0, 0.0, C, TTR_F64, ldc, nullptr, st);
    if (e != hipSuccess) return e;
    return symmetrize(C, k, st);
  }
  const int64_t rpc = (m + chunks - 1) / chunks;
  const dim3 grid((k + 15) / 16, (k + 15) / 16, (unsigned)chunks);
  const dim3 grid2((k + 15) / 16, (k + 15) / 16);
  hipLaunchKernelGGL((k_gemm_tn<double, double, double>), grid, dim3(256), 0, st, m, k, k, X, ldx, Y, ldy, 1.0, 0.0,
                     C, ldc, scratch, rpc);
  hipLaunchKernelGGL(k_gemm_tn_finish_sym, grid2, dim3(256), 0, st, scratch, (int)chunks, k, C, ldc);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------------
// C = alpha X W + beta C, 16 rows x 16 columns per work-group, one output per thread; the
// inner dimension in chunks of 128 whose X rows and W block are loaded in one round; a chunk
// ends at the last 16 that hold data.  Latency bounds it (inner sizes of 20 to 54 mostly): with
// every chunk walked to 128 and the leading columns counted one load after another 7.1 us at
// 24^5's sizes.
// ----------------------------------------------------------------------------------
constexpr int kNnRows = 16, kNnK = 128;

// Number of leading entries of v[0 .. n) that are > 0, by one wave, the same in all of them.
__device__ inline int leading_positive(const double* __restrict__ v, int n) {
  const int lane = threadIdx.x & 63;
  for (int base = 0; base < n; base += 64) {
    const uint64_t no = ~__ballot(base + lane < n && v[min(base + lane, n - 1)] > 0.0);
    if (no) return base + __ffsll((unsigned long long)no) - 1;
  }
  return n;
}

// colvals (optional): only the leading columns c with colvals[c] > 0 of W are used, the
// rest read as zero, and their count goes to *ncols.
template <typename TX>
__global__ __launch_bounds__(256) void k_gemm_nn(int64_t m, int ka, int kb, const TX* __restrict__ X, int64_t ldx,
                                                 const double* __restrict__ W, int64_t ldw, double alpha,
                                                 double beta, double* __restrict__ C, int64_t ldc,
                                                 const double* __restrict__ colvals, int* __restrict__ ncols) {
  __shared__ double Xs[kNnRows][kNnK + 1];
  __shared__ double Ws[kNnK][17];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int64_t r0 = (int64_t)blockIdx.y * kNnRows;
  const int c0 = blockIdx.x * 16;
  int kc = kb;
  if (colvals) {
    kc = leading_positive(colvals, kb);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *ncols = kc;
  }
  // four interleaved partial sums (k = 4i + q go to q), added in a fixed order
  double acc4[4] = {0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < ka; k0 += kNnK) {
    const int kn = min(ka - k0, kNnK), groups = (kn + 15) / 16;
    // X: sixteen columns of sixteen rows per round; W: sixteen rows
#pragma unroll
    for (int u = 0; u < kNnK / 16; ++u)
      if (u < groups) {
        const int kk = 16 * u + tx, wk = 16 * u + ty;
        Xs[ty][kk] = (r0 + ty < m && kk < kn) ? (double)X[(r0 + ty) * ldx + k0 + kk] : 0.0;
        Ws[wk][tx] = (wk < kn && c0 + tx < kc) ? W[(int64_t)(k0 + wk) * ldw + c0 + tx] : 0.0;
      }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kNnK / 16; ++u)
      if (u < groups) {
#pragma unroll
        for (int kk = 16 * u; kk < 16 * u + 16; kk += 4)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc4[q] = fma(Xs[ty][kk + q], Ws[kk + q][tx], acc4[q]);
      }
    __syncthreads();
  }
  const int c = c0 + tx;
  const int64_t row = r0 + ty;
  if (c < kb && row < m) {
    const double acc = (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]);
    const double old = beta != 0.0 ? C[row * ldc + c] : 0.0;
    C[row * ldc + c] = alpha * acc + beta * old;
  }
}

hipError_t gemm_nn(int64_t m, int ka, int kb, const void* X, int xdt, int64_t ldx, const double* W, int64_t ldw,
                   double alpha, double beta, double* C, int64_t ldc, hipStream_t st) {
  if (m <= 0 || kb <= 0) return hipSuccess;
  const dim3 grid((unsigned)((kb + 15) / 16), (unsigned)((m + kNnRows - 1) / kNnRows));
  if (xdt == TTR_F64)
    hipLaunchKernelGGL(k_gemm_nn<double>, grid, dim3(256), 0, st, m, ka, kb, (const double*)X, ldx, W, ldw, alpha,
                       beta, C, ldc, nullptr, nullptr);
  else if (xdt == TTR_F32)
    hipLaunchKernelGGL(k_gemm_nn<float>, grid, dim3(256), 0, st, m, ka, kb, (const float*)X, ldx, W, ldw, alpha,
                       beta, C, ldc, nullptr, nullptr);
  else
    hipLaunchKernelGGL(k_gemm_nn<__bf16>, grid, dim3(256), 0, st, m, ka, kb, (const __bf16*)X, ldx, W, ldw, alpha,
                       beta, C, ldc, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t gemm_nn_ritz(int64_t m, int w, int r, const double* X, int64_t ldx, const double* vecs,
                        const double* vals, double* C, int64_t ldc, int* nv, hipStream_t st) {
  if (m <= 0 || r <= 0 || r > w) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((r + 15) / 16), (unsigned)((m + kNnRows - 1) / kNnRows));
  hipLaunchKernelGGL(k_gemm_nn<double>, grid, dim3(256), 0, st, m, w, r, X, ldx, vecs, (int64_t)w, 1.0, 0.0, C, ldc,
                     vals, nv);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------------
// C (m1 x m2, ldc) = alpha X (m1 x a, ldx) Y^T (Y: m2 x a, ldy) + beta C, float64.
// 16 x 16 output tile per work-group, contraction in chunks of 16.
// ----------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_gemm_nt(int64_t m1, int64_t m2, int a, const double* __restrict__ X,
                                                 int64_t ldx, const double* __restrict__ Y, int64_t ldy,
                                                 double alpha, double beta, double* __restrict__ C, int64_t ldc) {
  __shared__ double Xs[16][17];
  __shared__ double Ys[16][17];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int64_t i0 = (int64_t)blockIdx.y * 16, j0 = (int64_t)blockIdx.x * 16;
  double acc = 0.0;
  for (int k0 = 0; k0 < a; k0 += 16) {
    Xs[ty][tx] = (i0 + ty < m1 && k0 + tx < a) ? X[(i0 + ty) * ldx + k0 + tx] : 0.0;
    Ys[ty][tx] = (j0 + ty < m2 && k0 + tx < a) ? Y[(j0 + ty) * ldy + k0 + tx] : 0.0;
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) acc += Xs[ty][kk] * Ys[tx][kk];
    __syncthreads();
  }
  const int64_t i = i0 + ty, j = j0 + tx;
  if (i < m1 && j < m2) {
    const double old = beta != 0.0 ? C[i * ldc + j] : 0.0;
    C[i * ldc + j] = alpha * acc + beta * old;
  }
}

hipError_t gemm_nt(int64_t m1, int64_t m2, int a, const double* X, int64_t ldx, const double* Y, int64_t ldy,
                   double alpha, double beta, double* C, int64_t ldc, hipStream_t st) {
  if (m1 <= 0 || m2 <= 0) return hipSuccess;
  const dim3 grid((unsigned)((m2 + 15) / 16), (unsigned)((m1 + 15) / 16));
  hipLaunchKernelGGL(k_gemm_nt, grid, dim3(256), 0, st, m1, m2, a, X, ldx, Y, ldy, alpha, beta, C, ldc);
  return hipGetLastError();
}

// Y (rows x cols, ldy) = alpha X (ldx) + beta Y; columns >= *ncols_keep (if given) of the
// result are zeroed.
__global__ __launch_bounds__(256) void k_axpby(int64_t rows, int cols, double alpha, const double* __restrict__ X,
                                               int64_t ldx, double beta, double* __restrict__ Y, int64_t ldy,
                                               const int* __restrict__ keep) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const int64_t i = idx / cols;
  const int j = (int)(idx % cols);
  double v = (X ? alpha * X[i * ldx + j] : 0.0) + (beta != 0.0 ? beta * Y[i * ldy + j] : 0.0);
  if (keep && j >= *keep) v = 0.0;
  Y[i * ldy + j] = v;
}

hipError_t axpby(int64_t rows, int cols, double alpha, const double* X, int64_t ldx, double beta, double* Y,
                 int64_t ldy, const int* keep, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  const int64_t total = rows * cols;
  hipLaunchKernelGGL(k_axpby, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, rows, cols, alpha, X, ldx,
                     beta, Y, ldy, keep);
  return hipGetLastError();
}

// Out (s x s) = copyltu(alpha M) = tril(alpha M) + tril(alpha M, -1)^T (out of place).
__global__ __launch_bounds__(256) void k_copyltu(const double* __restrict__ M, int s, double alpha,
                                                 double* __restrict__ out) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= s * s) return;
  const int i = idx / s, j = idx % s;
  out[idx] = alpha * (i >= j ? M[i * s + j] : M[j * s + i]);
}

hipError_t copyltu(const double* M, int s, double alpha, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_copyltu, dim3((s * s + 255) / 256), dim3(256), 0, st, M, s, alpha, out);
  return hipGetLastError();
}

// S (n x n) <- K + K^T (out of place).
__global__ __launch_bounds__(256) void k_sym_sum(const double* __restrict__ K, int64_t n, double* __restrict__ S) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n * n) return;
  const int64_t i = idx / n, j = idx % n;
  S[idx] = K[i * n + j] + K[j * n + i];
}

hipError_t sym_sum(const double* K, int64_t n, double* S, hipStream_t st) {
  const int64_t total = n * n;
  hipLaunchKernelGGL(k_sym_sum, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, K, n, S);
  return hipGetLastError();
}

// Adjoint of the top-r eigenvectors of a symmetric w x w matrix (gauge-invariant use:
// only kept x discarded pairs).  Inputs: U (w x w, column j = eigenvector j of the
// resolved part, zero columns for unresolved directions), lam (w, decreasing, zero for
// unresolved), Ub (w x r, adjoint of U[:, :r]), nvalid (*nv <= r kept columns).
// Out: Mb (w x w) = sym( sum_i v_i u_i^T ), with
//   v_i = sum_{j >= r resolved} u_j (u_j . ub_i) / (lam_i - lam_j)
//       + (ub_i - U_res U_res^T ub_i) / lam_i                    (unresolved: lam_j = 0).
// k_eig_adjoint_v: one work-group per kept i, v_i to column i of V (w x r); k_eig_adjoint_m: Mb,
// one thread per entry.  Chains of dependent memory reads bound both.  w = 54, r = 12: one
// work-group for everything, its columns one after another, took 108 us.
constexpr int kAdjThreads = 256;

__device__ inline int adj_kept(const int* nv, int r) { return *nv < r ? *nv : r; }

__global__ __launch_bounds__(kAdjThreads) void k_eig_adjoint_v(const double* __restrict__ U,
                                                               const double* __restrict__ lam, int w, int r,
                                                               const double* __restrict__ Ub,
                                                               const int* __restrict__ nv, double* __restrict__ V) {
  __shared__ double proj[kAdjThreads], coef[kAdjThreads], ub[kAdjThreads];
  const int tid = threadIdx.x, i = blockIdx.x;
  if (i >= adj_kept(nv, r)) return;
  if (tid < w) ub[tid] = Ub[tid * r + i];
  __syncthreads();
  const int nres = leading_positive(lam, w);
  const double li = lam[i];
  if (tid < nres) {  // u_j . ub_i for every resolved j
    double acc = 0.0;
#pragma unroll 8
    for (int l = 0; l < w; ++l) acc += U[l * w + tid] * ub[l];
    proj[tid] = acc;
    coef[tid] = tid >= r ? acc / (li - lam[tid]) : 0.0;
  }
  __syncthreads();
  if (tid < w) {
    double res = ub[tid], v = 0.0;
#pragma unroll 8
    for (int j = 0; j < nres; ++j) {
      const double uj = U[tid * w + j];
      res -= uj * proj[j];
      v += uj * coef[j];
    }
    V[tid * r + i] = v + res / li;
  }
}

// Mb = sym(V U_kept^T)
__global__ __launch_bounds__(kAdjThreads) void k_eig_adjoint_m(const double* __restrict__ U, int w, int r,
                                                               const int* __restrict__ nv,
                                                               const double* __restrict__ V, double* __restrict__ Mb) {
  const int e = blockIdx.x * kAdjThreads + threadIdx.x;
  if (e >= w * w) return;
  const int a = e / w, b = e % w, kept = adj_kept(nv, r);
  double x = 0.0, y = 0.0;
#pragma unroll 4
  for (int i = 0; i < kept; ++i) {
    x += V[a * r + i] * U[b * w + i];
    y += V[b * r + i] * U[a * w + i];
  }
  Mb[e] = 0.5 * (x + y);
}

hipError_t eig_adjoint(const double* U, const double* lam, int w, int r, const double* Ub, const int* nv, double* V,
                       double* Mb, hipStream_t st) {
  if (w > kAdjThreads) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_eig_adjoint_v, dim3(r), dim3(kAdjThreads), 0, st, U, lam, w, r, Ub, nv, V);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_eig_adjoint_m, dim3((w * w + kAdjThreads - 1) / kAdjThreads), dim3(kAdjThreads), 0, st, U, w, r,
                     nv, V, Mb);
  return hipGetLastError();
}

// lb[i] = -1/2 lam_i^{-3/2} (Vr^T Wb)_{ii} and Vb = Wb diag(lam^{-1/2}) for the
// n < m saturated mode (W = V_r diag(lam^{-1/2})).  One work-group.
__global__ __launch_bounds__(256) void k_scale_adjoint(const double* __restrict__ Vr, int n, int r,
                                                       const double* __restrict__ lam, const double* __restrict__ Wb,
                                                       double* __restrict__ Vb, double* __restrict__ lb) {
  const int tid = threadIdx.x;
  for (int i = tid; i < r; i += blockDim.x) {
    double acc = 0.0;
    for (int l = 0; l < n; ++l) acc += Vr[l * n + i] * Wb[l * r + i];
    lb[i] = lam[i] > 0.0 ? -0.5 * acc / (lam[i] * sqrt(lam[i])) : 0.0;
  }
  for (int e = tid; e < n * r; e += blockDim.x) {
    const int i = e % r;
    Vb[e] = lam[i] > 0.0 ? Wb[e] / sqrt(lam[i]) : 0.0;
  }
}

hipError_t scale_adjoint(const double* Vr, int n, int r, const double* lam, const double* Wb, double* Vb, double* lb,
                         hipStream_t st) {
  hipLaunchKernelGGL(k_scale_adjoint, dim3(1), dim3(256), 0, st, Vr, n, r, lam, Wb, Vb, lb);
  return hipGetLastError();
}

// Mb (n x n) += sum_{i < r} lb_i u_i u_i^T  (eigenvalue part of an eigen adjoint).
__global__ __launch_bounds__(256) void k_add_eigval_adjoint(const double* __restrict__ U, int n, int r,
                                                            const double* __restrict__ lb, double* __restrict__ Mb) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * n) return;
  const int a = e / n, b = e % n;
  double acc = 0.0;
  for (int i = 0; i < r; ++i) acc += lb[i] * U[a * n + i] * U[b * n + i];
  Mb[e] += acc;
}

hipError_t add_eigval_adjoint(const double* U, int n, int r, const double* lb, double* Mb, hipStream_t st) {
  hipLaunchKernelGGL(k_add_eigval_adjoint, dim3((n * n + 255) / 256), dim3(256), 0, st, U, n, r, lb, Mb);
  return hipGetLastError();
}

// Sum of squares of a large array in float64: per-block partials then a fixed-order finish.
template <typename T>
__global__ __launch_bounds__(256) void k_sumsq_big(const T* __restrict__ x, int64_t n, double* __restrict__ part) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const double v = (double)x[i];
    acc += v * v;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void k_sum_finish(const double* __restrict__ part, int nb, double sign_a,
                                                    const double* __restrict__ other, double* __restrict__ out) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int i = threadIdx.x; i < nb; i += 256) acc += part[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sign_a * red[0] + (other ? *other : 0.0);
}

// *out = sign * sum(x^2) + (*other if given); `part` holds 1024 doubles.
hipError_t sumsq_big(const void* x, int dt, int64_t n, double sign, const double* other, double* part, double* out,
                     hipStream_t st) {
  const int nb = 1024;
  if (dt == TTR_F64)
    hipLaunchKernelGGL(k_sumsq_big<double>, dim3(nb), dim3(256), 0, st, (const double*)x, n, part);
  else if (dt == TTR_F32)
    hipLaunchKernelGGL(k_sumsq_big<float>, dim3(nb), dim3(256), 0, st, (const float*)x, n, part);
  else
    hipLaunchKernelGGL(k_sumsq_big<__bf16>, dim3(nb), dim3(256), 0, st, (const __bf16*)x, n, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_sum_finish, dim3(1), dim3(256), 0, st, part, nb, sign, other, out);
  return hipGetLastError();
}

// dX = 2 X + dX (element-wise, X and dX of the same dtype: float64 or float32).
template <typename T>
__global__ __launch_bounds__(256) void k_two_x_plus(const T* __restrict__ x, T* __restrict__ dx, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    dx[i] = (T)(2.0 * (double)x[i] + (double)dx[i]);
}

hipError_t two_x_plus(const void* x, void* dx, int dt, int64_t n, hipStream_t st) {
  if (dt == TTR_F64) hipLaunchKernelGGL(k_two_x_plus<double>, dim3(2048), dim3(256), 0, st, (const double*)x, (double*)dx, n);
  else hipLaunchKernelGGL(k_two_x_plus<float>, dim3(2048), dim3(256), 0, st, (const float*)x, (float*)dx, n);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------------
// Eigen-decomposition of a symmetric positive semi-definite n x n Gram matrix G.
//
// 1. Pivoted Cholesky: P^T G P = R^T R (R upper triangular, k x n), stopping when the
//    largest remaining diagonal falls to n * 2^-52 of the largest initial one (what
//    is left is rounding noise of G).  This is the R factor of a column-pivoted QR of
//    any F with F^T F = G, so
// 2. one-sided (Hestenes) Jacobi on the k rows of R (Drmac and Veselic's preconditioned
//    Jacobi SVD) converges in a few sweeps: rows p, q are rotated until
//    r_p . r_q <= tol ||r_p|| ||r_q|| for every pair.  The converged rows are sigma_j u_j
//    with u_j (in pivoted coordinates) the eigenvectors of G and sigma_j^2 its
//    eigenvalues.
// Pairs follow the round-robin (circle) ordering: in round k of a sweep over npad
// (even) indices, pair 0 is (k, npad-1) and pair i >= 1 is ((k+i) mod (npad-1),
// (k-i) mod (npad-1)); every pair meets once per sweep.  A group of G lanes (G | 16,
// inside one DPP row) handles one pair; lane g owns entries g, g+G, ... of both rows
// (at most RPL each, held in registers during the round).  The three dot products are
// summed across the group with DPP permutes (row mirror, half-row mirror, quad
// butterflies), which pair values symmetrically so every lane of the group obtains the
// bitwise same sums and rotation.  Output: vals[j] = sigma_j^2 decreasing, vecs column j
// the matching unit eigenvector; the n - k unresolved directions get zero columns and
// zero values.
// ----------------------------------------------------------------------------------
constexpr int kEigMaxSweeps = 40;


__device__ inline double group_sum(double v, int G) {
  if (G >= 16) v += dpp_mov<0x140>(v);  // row_mirror: lane i <-> 15 - i
  if (G >= 8) v += dpp_mov<0x141>(v);   // row_half_mirror: lane i <-> 7 - i (within 8)
  if (G >= 4) v += dpp_mov<0x4E>(v);    // quad_perm [2,3,0,1]
  if (G >= 2) v += dpp_mov<0xB1>(v);    // quad_perm [1,0,3,2]
  return v;
}

template <int NT, int G, int RPL, bool IN_LDS>
__global__ __launch_bounds__(NT) void k_eig_psd(const double* __restrict__ g_in, int n, double* __restrict__ vecs,
                                                double* __restrict__ vals, double* __restrict__ work) {
  // Rows have pitch LDA = G * RPL >= n and are zero beyond column n, so every lane
  // reads and writes its RPL entries of a row without bounds checks.
  constexpr int LDA = G * RPL;
  // entries of a row pair that a lane holds at a time: all of them, or a part, read again for the
  // rotation (both rows of 32 entries were more than the registers of a 1024-thread work-group:
  // n = 200 55.3 ms with the rest spilled)
  constexpr int CH = RPL <= 8 ? RPL : 16;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int rowid[kMaxSmall];   // row of A holding R row j
  __shared__ int remain[kMaxSmall];  // indices not yet eliminated
  __shared__ int gone[kMaxSmall];    // nonzero: eliminated
  __shared__ int s_piv, s_nrem, rotated;
  __shared__ double s_d;
  __shared__ double norms[kMaxSmall + 1];
  double* A = IN_LDS ? reinterpret_cast<double*>(smem) : work;  // n rows of pitch LDA
  const int tid = threadIdx.x, lane = tid & 63;
  for (int e = tid; e < n * LDA; e += NT) {
    const int i = e / LDA, l = e % LDA;
    A[e] = l < n ? g_in[i * n + l] : 0.0;
  }
  for (int i = tid; i < n; i += NT) { remain[i] = i; gone[i] = 0; }
  if (tid == 0) s_nrem = n;
  __syncthreads();
  // Products of two eigenvalues leave the range of float64 from about 2^512 (2^-512) on: such a
  // matrix is scaled by an even power of two, so that its largest diagonal entry is about one.
  int scale = 0;
  {
    double top = 0.0;
    for (int i = lane; i < n; i += 64) top = fmax(top, A[i * LDA + i]);
    top = max64(top);
    if (top < INFINITY) scale = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_frexp_exp(top)) / 2 * 2;
    if (scale > -400 && scale < 400) scale = 0;
    if (scale != 0) {
      __syncthreads();  // every wave has read the diagonal
      for (int e = tid; e < n * LDA; e += NT) A[e] = ldexp(A[e], -scale);
      __syncthreads();
    }
  }

  // ---- pivoted Cholesky of the Schur complements, in place and without row swaps:
  // step j picks the remaining index pv with the largest diagonal, turns row pv into
  // R_j = S[pv, :] / sqrt(S[pv, pv]) (zero on eliminated columns) and updates the
  // remaining block.  Sum_j R_j^T R_j = G on the resolved part. ----
  int k = 0;
  double d0 = 0.0;
  for (int j = 0; j < n; ++j) {
    const int nrem = s_nrem;
    if (tid < 64) {  // wave 0: argmax over the remaining diagonal, ties by smaller index
      double best = -1.0;
      int bi = 1 << 30, bt = 0;
      for (int t = lane; t < nrem; t += 64) {
        const int i = remain[t];
        const double d = A[i * LDA + i];
        if (d > best || (d == best && i < bi)) { best = d; bi = i; bt = t; }
      }
      const double top = max64(best);
      int pi = best == top ? bi : 1 << 30;
      for (int off = 32; off > 0; off >>= 1) pi = min(pi, __shfl_xor(pi, off, 64));
      if (j == 0) d0 = top;
      const bool ok = nrem > 0 && top > 0.0 && top > (double)n * 0x1p-52 * d0;
      if (ok && bi == pi) {  // the lane that holds it
        remain[bt] = remain[nrem - 1];
        gone[bi] = 1;
        rowid[j] = bi;
        s_nrem = nrem - 1;
      }
      if (lane == 0) {
        s_piv = ok ? pi : -1;
        s_d = top;
      }
    }
    __syncthreads();
    const int pv = s_piv;
    if (pv < 0) break;
    k = j + 1;
    const double rinv = 1.0 / sqrt(s_d);
    const int nr = s_nrem;
    // R_j: diagonal entry sqrt(d), remaining columns scaled, eliminated columns zero
    for (int l = tid; l < n; l += NT) {
      const double v = A[pv * LDA + l];
      A[pv * LDA + l] = l == pv || gone[l] == 0 ? v * rinv : 0.0;
    }
    __syncthreads();
    for (int t = tid >> 5; t < nr; t += NT / 32) {
      const int i = remain[t];
      const double f = A[pv * LDA + i];
      for (int c = tid & 31; c < nr; c += 32) {
        const int l = remain[c];
        A[i * LDA + l] -= f * A[pv * LDA + l];
      }
    }
    __syncthreads();
  }
  // rows of unresolved indices hold Schur-complement noise: clear them
  for (int t = 0; t < s_nrem; ++t) {
    const int i = remain[t];
    for (int l = tid; l < LDA; l += NT) A[i * LDA + l] = 0.0;
  }
  __syncthreads();

  // ---- Hestenes on the k rows R_j (rows rowid[j] of A) ----
  const int npad = k + (k & 1);
  const int npairs = npad / 2;
  const int pair = tid / G, gl = tid % G;
  const bool active = pair < npairs && k > 1;
  const double tol = 1e-15 * (double)n;
  for (int sweep = 0; sweep < kEigMaxSweeps && k > 1; ++sweep) {
    int mine = 0;
    if (NT > 64) {
      if (tid == 0) rotated = 0;
      __syncthreads();
    }
    int p = 0, q = 0;
    if (active) { p = pair == 0 ? 0 : pair; q = pair == 0 ? npad - 1 : npad - 1 - pair; }
    for (int r = 0; r < npad - 1; ++r) {
      if (active && p < k && q < k) {
        double* rp = A + rowid[p] * LDA + gl;
        double* rq = A + rowid[q] * LDA + gl;
        double x[CH], y[CH];
        double al = 0.0, be = 0.0, ga = 0.0;
        auto load = [&](int h) {
#pragma unroll
          for (int t = 0; t < CH; ++t) { x[t] = rp[(h + t) * G]; y[t] = rq[(h + t) * G]; }
        };
        auto dots = [&] {
#pragma unroll
          for (int t = 0; t < CH; ++t) { al += x[t] * x[t]; be += y[t] * y[t]; ga += x[t] * y[t]; }
        };
        load(0);
        dots();
#pragma unroll 1
        for (int h = CH; h < RPL; h += CH) { load(h); dots(); }
        al = group_sum(al, G); be = group_sum(be, G); ga = group_sum(ga, G);
        // estimates and Newton steps in place of divisions and roots, in the range where they hold
        const double pr = al * be;
        const bool wide = pr > 0x1p-960 ? fabs(ga) * rsqrt_nr(pr) > tol : fabs(ga) > tol * sqrt(pr);
        if (al > 0.0 && be > 0.0 && wide) {
          const double zeta = fabs(ga) > 0x1p-500 ? (be - al) * rcp_nr(2.0 * ga) : (be - al) / (2.0 * ga);
          double t;
          if (fabs(zeta) > 1e150) {
            t = 0.5 / zeta;
          } else {
            const double z1 = 1.0 + zeta * zeta;
            t = rcp_nr(fabs(zeta) + z1 * rsqrt_nr(z1));
            t = zeta >= 0.0 ? t : -t;
          }
          const double c = rsqrt_nr(1.0 + t * t), s = c * t;
#pragma unroll 1
          for (int h = 0; h < RPL; h += CH) {
            if (CH < RPL) load(h);
#pragma unroll
            for (int u = 0; u < CH; ++u) {
              rp[(h + u) * G] = c * x[u] - s * y[u];
              rq[(h + u) * G] = s * x[u] + c * y[u];
            }
          }
          mine = 1;
        }
      }
      __syncthreads();
      if (active) {  // next round: every index except npad-1 advances by one (mod npad-1)
        p = (p == npad - 1) ? p : (p + 1 == npad - 1 ? 0 : p + 1);
        q = (q == npad - 1) ? q : (q + 1 == npad - 1 ? 0 : q + 1);
      }
    }
    int any;
    if (NT == 64) {
      any = __any(mine);
    } else {
      if (mine) rotated = 1;
      __syncthreads();
      any = rotated;
      __syncthreads();
    }
    if (!any) break;
  }
  // ---- values sigma^2 (decreasing, ties by index), unit vectors; unresolved: zero ----
  for (int j = tid; j < n; j += NT) {
    double s2 = 0.0;
    if (j < k) {
      const double* rj = A + rowid[j] * LDA;
#pragma unroll 8
      for (int i = 0; i < n; ++i) s2 += rj[i] * rj[i];
    }
    norms[j] = s2;
  }
  __syncthreads();
  for (int j = tid; j < n; j += NT) {
    const double nj = norms[j];
    int rank = 0;
#pragma unroll 8
    for (int i = 0; i < n; ++i) {
      const double ni = norms[i];
      rank += (ni > nj) || (ni == nj && i < j);
    }
    vals[rank] = ldexp(nj, scale);
    const double inv = nj > 0.0 ? 1.0 / sqrt(nj) : 0.0;
    const double* rj = A + (j < k ? rowid[j] : 0) * LDA;
#pragma unroll 8
    for (int i = 0; i < n; ++i) vecs[(int64_t)i * n + rank] = j < k ? rj[i] * inv : 0.0;
  }
}

template <int NT, int G, int RPL, bool IN_LDS>
static hipError_t launch_eig(const double* a, int n, double* vecs, double* vals, double* work, hipStream_t st) {
  const size_t lds = IN_LDS ? (size_t)n * G * RPL * 8 : 0;
  if (IN_LDS) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_eig_psd<NT, G, RPL, IN_LDS>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) { (void)hipGetLastError(); return e; }
  }
  hipLaunchKernelGGL((k_eig_psd<NT, G, RPL, IN_LDS>), dim3(1), dim3(NT), lds, st, a, n, vecs, vals, work);
  return hipGetLastError();
}

hipError_t sym_eig(const double* a, int n, double* vecs, double* vals, double* work, hipStream_t st) {
  if (n <= 0 || n > kMaxSmall) return hipErrorInvalidValue;
  // (threads, lanes per pair, entries per lane): lanes x entries = row pitch >= n,
  // lanes x pairs <= threads.
  if (n <= 16) return launch_eig<64, 8, 2, true>(a, n, vecs, vals, work, st);
  if (n <= 32) return launch_eig<64, 4, 8, true>(a, n, vecs, vals, work, st);
  if (n <= 64) return launch_eig<256, 8, 8, true>(a, n, vecs, vals, work, st);
  if (n <= 128) return launch_eig<1024, 16, 8, true>(a, n, vecs, vals, work, st);
  return launch_eig<1024, 8, 32, false>(a, n, vecs, vals, work, st);
}

// ----------------------------------------------------------------------------------
// SVQB transform, Ritz / saturated selection.
// ----------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_svqb(const double* __restrict__ vecs, const double* __restrict__ vals, int n,
                                              const double* __restrict__ ref, double coef, double* __restrict__ T,
                                              int* __restrict__ kept) {
  const double thr = coef * (ref ? *ref : vals[0]);
  int k = 0;
  while (k < n && vals[k] > thr) ++k;
  for (int e = threadIdx.x; e < n * n; e += blockDim.x) {
    const int j = e % n;
    T[e] = j < k ? vecs[e] / sqrt(vals[j]) : 0.0;
  }
  if (threadIdx.x == 0) *kept = k;
}

hipError_t svqb_transform(const double* vecs, const double* vals, int n, const double* ref, double coef, double* T,
                          int* kept, hipStream_t st) {
  hipLaunchKernelGGL(k_svqb, dim3(1), dim3(256), 0, st, vecs, vals, n, ref, coef, T, kept);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_sat(const double* __restrict__ vecs, const double* __restrict__ vals, int m,
                                             int r, double tau, double* __restrict__ G, int* __restrict__ nv) {
  double tot = 0.0;
  for (int j = 0; j < r && j < m; ++j) tot += vals[j];
  const double thr = tau * tau * tot;
  int k = 0;
  while (k < r && k < m && vals[k] > thr) ++k;
  for (int e = threadIdx.x; e < m * r; e += blockDim.x) {
    const int i = e / r, j = e % r;
    G[e] = j < k ? vecs[(int64_t)i * m + j] : 0.0;
  }
  if (threadIdx.x == 0) *nv = k;
}

hipError_t sat_select(const double* vecs, const double* vals, int m, int r, double tau, double* G, int* nv,
                      hipStream_t st) {
  hipLaunchKernelGGL(k_sat, dim3(1), dim3(256), 0, st, vecs, vals, m, r, tau, G, nv);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------------
// Completion: for i = 0, 1, ... v = e_i - G_c (G_c^T e_i); v -= G_c (G_c^T v); accept
// v / ||v|| when ||v||^2 > 1/(4m), until r columns.  One work-group; v in `work`.
// ----------------------------------------------------------------------------------
__device__ inline double block_sum(double v, double* red) {
  const int tid = threadIdx.x;
  red[tid] = v;
  __syncthreads();
  for (int off = blockDim.x / 2; off > 0; off >>= 1) {
    if (tid < off) red[tid] += red[tid + off];
    __syncthreads();
  }
  const double out = red[0];
  __syncthreads();
  return out;
}

__global__ __launch_bounds__(256) void k_complete(double* __restrict__ G, int64_t m, int r, const int* __restrict__ nv,
                                                  double* __restrict__ v) {
  __shared__ double red[256];
  __shared__ double coef[64];
  int col = *nv;
  if (col >= r) return;
  const double thresh = 1.0 / (4.0 * (double)m);
  for (int64_t cand = 0; cand < m && col < r; ++cand) {
    // v = e_cand - G_c G_c^T e_cand  (G_c^T e_cand = row cand of G)
    if (threadIdx.x < 64) coef[threadIdx.x] = (int)threadIdx.x < col ? G[cand * r + threadIdx.x] : 0.0;
    __syncthreads();
    for (int64_t i = threadIdx.x; i < m; i += blockDim.x) {
      double acc = (i == cand) ? 1.0 : 0.0;
      for (int c = 0; c < col; ++c) acc -= G[i * r + c] * coef[c];
      v[i] = acc;
    }
    __syncthreads();
    // second pass: v -= G_c (G_c^T v)
    for (int c = 0; c < col; ++c) {
      double part = 0.0;
      for (int64_t i = threadIdx.x; i < m; i += blockDim.x) part += G[i * r + c] * v[i];
      const double sum = block_sum(part, red);
      if (threadIdx.x == 0) coef[c] = sum;
    }
    __syncthreads();
    double part = 0.0;
    for (int64_t i = threadIdx.x; i < m; i += blockDim.x) {
      double acc = v[i];
      for (int c = 0; c < col; ++c) acc -= G[i * r + c] * coef[c];
      v[i] = acc;
      part += acc * acc;
    }
    const double nv2 = block_sum(part, red);
    if (nv2 > thresh) {
      const double inv = 1.0 / sqrt(nv2);
      for (int64_t i = threadIdx.x; i < m; i += blockDim.x) G[i * r + col] = v[i] * inv;
      ++col;
    }
    __syncthreads();
  }
}

hipError_t complete_columns(double* G, int64_t m, int r, const int* nv, double* work, hipStream_t st) {
  if (r > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_complete, dim3(1), dim3(256), 0, st, G, m, r, nv, work);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------------
// Conversions, symmetrisation, identity.
// ----------------------------------------------------------------------------------
template <typename TI, typename TO>
__global__ __launch_bounds__(256) void k_convert(const TI* __restrict__ in, int64_t rows, int cols, int64_t ldi,
                                                 TO* __restrict__ out, int64_t rows_pad, int cols_pad, int64_t ldo) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows_pad * cols_pad) return;
  const int64_t i = idx / cols_pad;
  const int j = (int)(idx % cols_pad);
  out[i * ldo + j] = round_from_f64<TO>((i < rows && j < cols) ? (double)in[i * ldi + j] : 0.0);
}

template <typename TI>
static hipError_t convert_from(const TI* in, int64_t rows, int cols, int64_t ldi, void* out, int odt,
                               int64_t rows_pad, int cols_pad, int64_t ldo, hipStream_t st) {
  const int64_t total = rows_pad * cols_pad;
  const dim3 grid((unsigned)((total + 255) / 256));
  if (odt == TTR_F64)
    hipLaunchKernelGGL((k_convert<TI, double>), grid, dim3(256), 0, st, in, rows, cols, ldi, (double*)out, rows_pad,
                       cols_pad, ldo);
  else if (odt == TTR_F32)
    hipLaunchKernelGGL((k_convert<TI, float>), grid, dim3(256), 0, st, in, rows, cols, ldi, (float*)out, rows_pad,
                       cols_pad, ldo);
  else
    hipLaunchKernelGGL((k_convert<TI, __bf16>), grid, dim3(256), 0, st, in, rows, cols, ldi, (__bf16*)out, rows_pad,
                       cols_pad, ldo);
  return hipGetLastError();
}

hipError_t convert_pad(const void* in, int idt, int64_t rows, int cols, int64_t ldi, void* out, int odt,
                       int64_t rows_pad, int cols_pad, int64_t ldo, hipStream_t st) {
  if (rows_pad <= 0 || cols_pad <= 0) return hipSuccess;
  if (idt == TTR_F64) return convert_from((const double*)in, rows, cols, ldi, out, odt, rows_pad, cols_pad, ldo, st);
  if (idt == TTR_F32) return convert_from((const float*)in, rows, cols, ldi, out, odt, rows_pad, cols_pad, ldo, st);
  return convert_from((const __bf16*)in, rows, cols, ldi, out, odt, rows_pad, cols_pad, ldo, st);
}

__global__ __launch_bounds__(256) void k_symmetrize(double* __restrict__ a, int n) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n * n) return;
  const int i = idx / n, j = idx % n;
  if (i < j) {
    const double v = 0.5 * (a[i * n + j] + a[j * n + i]);
    a[i * n + j] = v;
    a[j * n + i] = v;
  }
}

// status |= 1 when any of the n float64 values is NaN or infinite (every writer stores the
// same value, so the race between them is benign).
__global__ __launch_bounds__(256) void k_flag_nonfinite(const double* __restrict__ v, int64_t n,
                                                        int* __restrict__ status) {
  bool bad = false;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    bad |= !isfinite(v[i]);
  if (__any(bad) && (threadIdx.x & 63) == 0) *status = 1;
}

hipError_t flag_nonfinite(const double* v, int64_t n, int* status, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 256);
  hipLaunchKernelGGL(k_flag_nonfinite, dim3((unsigned)blocks), dim3(256), 0, st, v, n, status);
  return hipGetLastError();
}

__global__ void k_set_scalar(double* __restrict__ p, double v) { *p = v; }

hipError_t set_scalar(double* p, double v, hipStream_t st) {
  hipLaunchKernelGGL(k_set_scalar, dim3(1), dim3(1), 0, st, p, v);
  return hipGetLastError();
}

hipError_t symmetrize(double* a, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_symmetrize, dim3((n * n + 255) / 256), dim3(256), 0, st, a, n);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_identity(double* __restrict__ a, int64_t m) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= m * m) return;
  a[idx] = (idx / m == idx % m) ? 1.0 : 0.0;
}

hipError_t identity(double* a, int64_t m, hipStream_t st) {
  hipLaunchKernelGGL(k_identity, dim3((unsigned)((m * m + 255) / 256)), dim3(256), 0, st, a, m);
  return hipGetLastError();
}

}  // namespace ttr
