// Streaming reconstruction error of a tensor train (Section 4 metrics): ||X - Xhat||^2,
// ||X||^2 and max |Xhat|, all in float64.
//
// The modes are split at s: R (r_s x inner) is the contraction of cores s+1..d (formed once by
// the caller), L (outer x r_s) the left interface rows G_1[i_1] .. G_s[i_s].  X is read as an
// outer x inner matrix and compared with Xhat = L R tile by tile, Xhat formed on the float64
// matrix cores and never written.
//
// What bounds it: X read once (1.0 GB of a 48^5 float32 tensor: 0.2 ms at the 4.9 TB/s of a
// large copy) and 2 r_s float64 flops per entry (10 GFLOP at r_s = 20: 0.16 ms on the matrix
// cores).  One thread per entry with scalar products read all of R through L2 for every row of
// L (2.85 ms).  A wave here owns 64 rows of L and walks column tiles: an R tile is loaded once
// into registers for those 64 rows.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "wave_ops.h"

namespace ttr {

namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef double d2_t __attribute__((ext_vector_type(2)));

constexpr int kErrRows = 128;      // rows of X per work-group (64 when outer is that small)
constexpr int kErrGroups = 2048;   // work-groups wanted: 256 CUs, a few resident on each

struct TTErrArgs {
  int s;
  int64_t dims[TTR_MAX_D];
  int64_t ranks[TTR_MAX_D + 1];
  const double* cores[TTR_MAX_D];
};

// VEC consecutive entries of X per lane (16-byte loads of float32 and float64).
template <typename TX> struct XVec;
template <> struct XVec<double> { static constexpr int N = 2; typedef double V __attribute__((ext_vector_type(2))); };
template <> struct XVec<float> { static constexpr int N = 4; typedef float V __attribute__((ext_vector_type(4))); };
template <> struct XVec<__bf16> { static constexpr int N = 4; typedef __bf16 V __attribute__((ext_vector_type(4))); };

}  // namespace

// Work-group (rb, cb): rows rb * rows_wg .. of X, columns cb * chunk ..; its four waves are
// rows_wg / 64 row groups times 4 / (rows_wg / 64) interleaved column-tile groups.  The column
// chunk is the fast index of blockIdx, so that with a multiple of eight chunks each XCD's L2
// keeps its own share of R.
//
// A column tile is 16 VEC columns: lane (j, q) = (lane % 16, lane / 16) holds columns
// VEC j .. VEC j + VEC - 1, and the t-th matrix-core product takes columns VEC j + t, so X is
// read in whole vectors.  Result element v of a product is row q + 4 v.
template <typename TX, int KS>
__global__ __launch_bounds__(256) void k_tt_error(const TX* __restrict__ x, int64_t outer, int64_t inner,
                                                  TTErrArgs args, const double* __restrict__ R, int rows_wg,
                                                  int pitch, int64_t nchunks, int64_t chunk, int aligned,
                                                  double* __restrict__ part) {
  constexpr int VEC = XVec<TX>::N;
  typedef typename XVec<TX>::V xv_t;
  extern __shared__ double lds[];
  __shared__ int64_t dig[kErrRows];
  __shared__ double red[12];
  const int tid = threadIdx.x;
  const int64_t row0 = ((int64_t)blockIdx.x / nchunks) * rows_wg;
  const int64_t cbeg = ((int64_t)blockIdx.x % nchunks) * chunk;
  const int64_t cend = cbeg + chunk < inner ? cbeg + chunk : inner;
  const int rs = (int)args.ranks[args.s];

  // left interface rows: L_0 = G_1[i_1], L_k = L_{k-1} G_{k+1}[i_{k+1}], two LDS buffers in turn
  double* cur = lds;
  double* nxt = args.s > 1 ? lds + (size_t)rows_wg * pitch : lds;
  int64_t below = 1;
  for (int k = 1; k < args.s; ++k) below *= args.dims[k];
  for (int k = 0; k < args.s; ++k) {
    const int ra = (int)args.ranks[k], rb = (int)args.ranks[k + 1];
    const int64_t I = args.dims[k];
    const double* __restrict__ Gk = args.cores[k];
    if (tid < rows_wg) dig[tid] = row0 + tid < outer ? ((row0 + tid) / below) % I : 0;
    __syncthreads();
    for (int e = tid; e < rows_wg * rb; e += 256) {
      const int row = e / rb, b = e - row * rb;
      const double* g = Gk + dig[row] * rb + b;
      double v;
      if (k == 0) {
        v = g[0];
      } else {
        v = 0.0;
#pragma unroll 4
        for (int a = 0; a < ra; ++a) v += cur[row * pitch + a] * g[(int64_t)a * I * rb];
      }
      nxt[row * pitch + b] = row0 + row < outer ? v : 0.0;
    }
    __syncthreads();
    double* t = cur; cur = nxt; nxt = t;
    if (k + 1 < args.s) below /= args.dims[k + 1];
  }
  for (int e = tid; e < rows_wg * (4 * KS - rs); e += 256) {
    const int row = e / (4 * KS - rs), b = rs + e % (4 * KS - rs);
    cur[row * pitch + b] = 0.0;
  }
  __syncthreads();

  const int lane = tid & 63, wave = tid >> 6, j = lane & 15, q = lane >> 4;
  const int nrg = rows_wg / 64, rg = wave % nrg, cg = wave / nrg, ncg = 4 / nrg;
  const int64_t wrow = row0 + 64 * rg;
  const double* __restrict__ Lw = cur + (size_t)64 * rg * pitch;
  double e2 = 0.0, x2 = 0.0, xinf = 0.0;
  if (wrow < outer) {
    for (int64_t c0 = cbeg + (int64_t)16 * VEC * cg; c0 < cend; c0 += (int64_t)16 * VEC * ncg) {
      const int64_t col = c0 + VEC * j;
      const bool whole = c0 + 16 * VEC <= inner;
      xv_t xr[4][4];
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t row = wrow + 16 * rb + q + 4 * v;
          xv_t val;
#pragma unroll
          for (int t = 0; t < VEC; ++t) val[t] = (TX)0.0f;
          if (row < outer) {
            const TX* src = x + row * inner + col;
            if (whole && aligned) {
              val = *reinterpret_cast<const xv_t*>(src);
            } else {
#pragma unroll
              for (int t = 0; t < VEC; ++t)
                if (col + t < inner) val[t] = src[t];
            }
          }
          xr[rb][v] = val;
        }
      double b[KS][VEC];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int k = 4 * ks + q;
        const double* src = R + (int64_t)k * inner + col;
#pragma unroll
        for (int t = 0; t < VEC; ++t) b[ks][t] = 0.0;
        if (k < rs) {
          if (whole && aligned) {
#pragma unroll
            for (int t = 0; t < VEC; t += 2) {
              const d2_t p = *reinterpret_cast<const d2_t*>(src + t);
              b[ks][t] = p[0];
              b[ks][t + 1] = p[1];
            }
          } else {
#pragma unroll
            for (int t = 0; t < VEC; ++t)
              if (col + t < inner) b[ks][t] = src[t];
          }
        }
      }
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        if (wrow + 16 * rb >= outer) break;
        d4_t acc[VEC];
#pragma unroll
        for (int t = 0; t < VEC; ++t) acc[t] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const double a = Lw[(16 * rb + j) * pitch + 4 * ks + q];
#pragma unroll
          for (int t = 0; t < VEC; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[ks][t], acc[t], 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int t = 0; t < VEC; ++t) {
            const double xv = (double)xr[rb][v][t];  // zero, as Xhat, beyond the last row / column
            const double df = xv - acc[t][v];
            e2 += df * df;
            x2 += xv * xv;
            xinf = fmax(xinf, fabs(acc[t][v]));
          }
      }
    }
    // Xhat beyond the last row / column is zeros times entries of a core: NaN, not zero, where an
    // entry is infinite.  Then the errors are summed again over the entries that there are.
    // (Masks in the sums above: 388 to 392 us for 48^5 float32 in place of 382.)
    if ((inner % (16 * VEC) != 0 || wrow + 64 > outer) && __any(e2 != e2)) {
      e2 = 0.0;
#pragma unroll 1
      for (int64_t c0 = cbeg + (int64_t)16 * VEC * cg; c0 < cend; c0 += (int64_t)16 * VEC * ncg)
#pragma unroll 1
        for (int e = 0; e < 16 * VEC; ++e) {
          const int lr = q + 4 * (e / VEC);
          const int64_t row = wrow + lr, col = c0 + VEC * j + e % VEC;
          if (row < outer && col < inner) {
            double xh = 0.0;
            for (int k = 0; k < rs; ++k) xh = fma(Lw[lr * pitch + k], R[(int64_t)k * inner + col], xh);
            const double df = (double)x[row * inner + col] - xh;
            e2 += df * df;
          }
        }
    }
  }
  e2 = sum64(e2);
  x2 = sum64(x2);
  xinf = max64(xinf);
  if (lane == 0) { red[3 * wave] = e2; red[3 * wave + 1] = x2; red[3 * wave + 2] = xinf; }
  __syncthreads();
  if (tid == 0) {
    part[(int64_t)blockIdx.x * 3 + 0] = (red[0] + red[3]) + (red[6] + red[9]);
    part[(int64_t)blockIdx.x * 3 + 1] = (red[1] + red[4]) + (red[7] + red[10]);
    part[(int64_t)blockIdx.x * 3 + 2] = fmax(fmax(red[2], red[5]), fmax(red[8], red[11]));
  }
}

__global__ __launch_bounds__(256) void k_tt_error_finish(const double* __restrict__ part, int64_t groups,
                                                         double* __restrict__ out3) {
  __shared__ double r0[256], r1[256], r2[256];
  const int tid = threadIdx.x;
  // fixed assignment of work-groups to threads, then a fixed tree
  const int64_t per = (groups + 255) / 256;
  double a = 0.0, b = 0.0, c = 0.0;
  for (int64_t o = tid * per; o < (tid + 1) * per && o < groups; ++o) {
    a += part[o * 3]; b += part[o * 3 + 1]; c = fmax(c, part[o * 3 + 2]);
  }
  r0[tid] = a; r1[tid] = b; r2[tid] = c;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (tid < off) { r0[tid] += r0[tid + off]; r1[tid] += r1[tid + off]; r2[tid] = fmax(r2[tid], r2[tid + off]); }
    __syncthreads();
  }
  if (tid == 0) { out3[0] = r0[0]; out3[1] = r1[0]; out3[2] = r2[0]; }
}

// C (m x n) = A (m x k) B (k x n) row-major float64, k <= 64: the right part R, core by core.
// A wave forms 16 rows x 64 columns on the matrix cores, a work-group 64 x 64; A and B come
// straight from L2 (at 48^5 and rank 20: 960 x 20 times 20 x 2304, 18 MB written).  The general
// small product spent 75 us there on chunks of 128 inner indices, 108 of them padding.
__global__ __launch_bounds__(256) void k_tt_right(int64_t m, int k, int64_t n, const double* __restrict__ A,
                                                  const double* __restrict__ B, double* __restrict__ C) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 15, q = lane >> 4;
  const int64_t r0 = ((int64_t)blockIdx.x * 4 + wave) * 16, c0 = (int64_t)blockIdx.y * 64;
  if (r0 >= m) return;
  const int64_t row = r0 + j;
  d4_t acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int k0 = 0; k0 < k; k0 += 4) {
    const int kk = k0 + q;
    const double a = (kk < k && row < m) ? A[row * k + kk] : 0.0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t c = c0 + 16 * t + j;
      const double b = (kk < k && c < n) ? B[(int64_t)kk * n + c] : 0.0;
      acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[t], 0, 0, 0);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t r = r0 + q + 4 * v, c = c0 + 16 * t + j;
      if (r < m && c < n) C[r * n + c] = acc[t][v];
    }
}

hipError_t tt_right_product(int64_t m, int k, int64_t n, const double* A, const double* B, double* C, hipStream_t st) {
  const int64_t gx = (m + 63) / 64, gy = (n + 63) / 64;  // n <= 2^20: an inner block
  if (m <= 0 || n <= 0 || k <= 0 || gx >= (1 << 24) || gy > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_tt_right, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, st, m, k, n, A, B, C);
  return hipGetLastError();
}

template <typename TX, int KS>
static hipError_t launch_tt_error(const TX* x, int64_t outer, int64_t inner, const TTErrArgs& args, const double* R,
                                  double* part, int64_t part_groups, double* out3, hipStream_t st) {
  constexpr int VEC = XVec<TX>::N, TC = 16 * VEC;
  const int rows_wg = outer <= 64 ? 64 : kErrRows;
  const int64_t rblocks = (outer + rows_wg - 1) / rows_wg, tiles = (inner + TC - 1) / TC;
  // column chunks: about kErrGroups work-groups in all, a multiple of eight of them when there
  // are that many (one share of R per XCD), never more partials than the scratch holds
  int64_t want = std::max<int64_t>(1, std::min<int64_t>({kErrGroups / rblocks, tiles, part_groups / rblocks}));
  if (want >= 8) want = want / 8 * 8;
  const int64_t chunk = (tiles + want - 1) / want * TC;
  const int64_t nchunks = (inner + chunk - 1) / chunk;
  // a launch of 2^32 threads is not refused by the runtime, only partly run
  if (rblocks * nchunks > part_groups || rblocks * nchunks >= (1 << 24)) return hipErrorInvalidValue;
  int rmax = 4 * KS;
  for (int k = 1; k <= args.s; ++k) rmax = std::max(rmax, (int)args.ranks[k]);
  const int pitch = rmax + 1;
  const size_t bytes = (size_t)(args.s > 1 ? 2 : 1) * rows_wg * pitch * 8;
  const hipError_t el = hipFuncSetAttribute(reinterpret_cast<const void*>(k_tt_error<TX, KS>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (el != hipSuccess) { (void)hipGetLastError(); return el; }
  const int aligned = inner % VEC == 0 && inner % 2 == 0 && reinterpret_cast<uintptr_t>(x) % (VEC * sizeof(TX)) == 0 &&
                      reinterpret_cast<uintptr_t>(R) % 16 == 0;
  hipLaunchKernelGGL((k_tt_error<TX, KS>), dim3((unsigned)(rblocks * nchunks)), dim3(256), bytes, st, x, outer, inner,
                     args, R, rows_wg, pitch, nchunks, chunk, aligned, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_tt_error_finish, dim3(1), dim3(256), 0, st, part, rblocks * nchunks, out3);
  return hipGetLastError();
}

// k-steps of four compiled: the smallest that covers r_s (ranks are at most 64).
template <typename TX>
static hipError_t tt_error_t(const TX* x, int64_t outer, int64_t inner, const TTErrArgs& args, const double* R,
                             double* part, int64_t pg, double* out3, hipStream_t st) {
  const int ks = (int)(args.ranks[args.s] + 3) / 4;
  if (ks <= 1) return launch_tt_error<TX, 1>(x, outer, inner, args, R, part, pg, out3, st);
  if (ks <= 2) return launch_tt_error<TX, 2>(x, outer, inner, args, R, part, pg, out3, st);
  if (ks <= 3) return launch_tt_error<TX, 3>(x, outer, inner, args, R, part, pg, out3, st);
  if (ks <= 4) return launch_tt_error<TX, 4>(x, outer, inner, args, R, part, pg, out3, st);
  if (ks <= 5) return launch_tt_error<TX, 5>(x, outer, inner, args, R, part, pg, out3, st);
  if (ks <= 6) return launch_tt_error<TX, 6>(x, outer, inner, args, R, part, pg, out3, st);
  if (ks <= 8) return launch_tt_error<TX, 8>(x, outer, inner, args, R, part, pg, out3, st);
  if (ks <= 12) return launch_tt_error<TX, 12>(x, outer, inner, args, R, part, pg, out3, st);
  if (ks <= 16) return launch_tt_error<TX, 16>(x, outer, inner, args, R, part, pg, out3, st);
  return hipErrorInvalidValue;
}

hipError_t tt_error_blocks(const void* x, int xdt, int64_t outer, int64_t inner, int s_split, const int64_t* dims,
                           const int64_t* ranks, const double* const* cores, const double* R, double* part,
                           int64_t part_groups, double* out3, hipStream_t st) {
  TTErrArgs args;
  args.s = s_split;
  for (int k = 0; k < TTR_MAX_D; ++k) {
    args.dims[k] = k < s_split ? dims[k] : 1;
    args.cores[k] = k < s_split ? cores[k] : nullptr;
  }
  for (int k = 0; k <= TTR_MAX_D; ++k) args.ranks[k] = k <= s_split ? ranks[k] : 1;
  if (xdt == TTR_F64) return tt_error_t((const double*)x, outer, inner, args, R, part, part_groups, out3, st);
  if (xdt == TTR_F32) return tt_error_t((const float*)x, outer, inner, args, R, part, part_groups, out3, st);
  return tt_error_t((const __bf16*)x, outer, inner, args, R, part, part_groups, out3, st);
}

}  // namespace ttr
