// Matrix-core traits and tile staging shared by the float64 / float32 streaming kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ttr {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef double d4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));

// ----------------------------------------------------------------------------------
// Matrix-core traits.  For 16x16x4 (float32/float64) lane l supplies A[l%16][l/16]
// and B[l/16][l%16]; the 16x16 result lands as 4 values per lane in column l%16 and
// rows orow(l, r).  For 16x16x32 bfloat16 lane l supplies 8 consecutive k values
// 8*(l/16) .. 8*(l/16)+7 of row (A) / column (B) l%16.
// ----------------------------------------------------------------------------------
template <typename T> struct Mma;
template <> struct Mma<float> {
  typedef f4_t acc;
  typedef float scalar;
  static constexpr int K = 4;
  __device__ static acc zero() { return acc{0.f, 0.f, 0.f, 0.f}; }
  __device__ static acc mma(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int orow(int lane, int r) { return 4 * (lane >> 4) + r; }
};
template <> struct Mma<double> {
  typedef d4_t acc;
  typedef double scalar;
  static constexpr int K = 4;
  __device__ static acc zero() { return acc{0.0, 0.0, 0.0, 0.0}; }
  __device__ static acc mma(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int orow(int lane, int r) { return (lane >> 4) + 4 * r; }
};

template <typename T> __device__ __host__ constexpr int tile_cols_t() { return sizeof(T) == 8 ? 16 : 32; }

// Sixteen bytes from a pointer that is aligned to its element only: rows of odd length put
// every row at another offset, and the vector loads of global memory take any of them.  (Four
// scalar loads in their place: 378 us for the carry of a 250 x 1000003 float32 unfolding.)
template <typename T>
__device__ __forceinline__ u4_t load16(const T* p) {
  u4_t v;
  __builtin_memcpy(&v, p, sizeof(v));
  return v;
}

// ----------------------------------------------------------------------------------
// Tile staging.  A tile is `rows` (multiple of 16) x TT columns starting at (row0, col0).
// fetch() issues the global loads into registers (16-byte vectors when the tile is
// whole, guarded scalar loads otherwise); commit() writes them to LDS
// with row pitch TT+1.  Rows >= m and columns >= n are zero.
// ----------------------------------------------------------------------------------
template <typename T, int MAXV, int NTH = kThreads, int TTC = tile_cols_t<T>()>
struct TileRegs {
  static constexpr int VEC = 16 / sizeof(T);
  static constexpr int TT = TTC;
  static constexpr int VPR = TT / VEC;
  u4_t v[MAXV];

  // WHOLE: the compiler is told to expect whole tiles, and lays the loop out for them (results are
  // the same; which kernels gain by it is measured beside their calls).
  template <bool WHOLE = false>
  __device__ void fetch(const T* __restrict__ A, int64_t m, int64_t n, int64_t row0, int rows, int64_t col0) {
    if (WHOLE ? __builtin_expect(col0 + TT <= n, 1) : col0 + TT <= n) fetch_full(A, m, n, row0, rows, col0);
    else fetch_guarded(A, m, n, row0, rows, col0);
  }

  // Whole tile: lane (r, cv) loads rows r, r + RSTEP, ... with one
  // 16-byte vector each; the row stride is uniform, so addresses stay per-lane base +
  // scalar offset.
  __device__ void fetch_full(const T* __restrict__ A, int64_t m, int64_t n, int64_t row0, int rows, int64_t col0) {
    constexpr int RSTEP = NTH / VPR;
    const int r_in = (int)threadIdx.x / VPR, cv = (int)threadIdx.x % VPR;
    const T* base = A + (row0 + r_in) * n + col0 + cv * VEC;
    const int64_t lim = (m - row0 < (int64_t)rows ? m - row0 : (int64_t)rows) - r_in;  // valid i * RSTEP < lim
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      u4_t val = u4_t{0u, 0u, 0u, 0u};
      if ((int64_t)i * RSTEP < lim) val = load16(base + (int64_t)i * RSTEP * n);
      v[i] = val;
    }
  }

  __device__ void fetch_guarded(const T* __restrict__ A, int64_t m, int64_t n, int64_t row0, int rows, int64_t col0) {
    const int nv = rows * VPR;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      const int idx = (int)threadIdx.x + i * NTH;
      u4_t val = u4_t{0u, 0u, 0u, 0u};
      if (idx < nv) {
        const int rr = idx / VPR, cv = idx % VPR;
        const int64_t row = row0 + rr;
        if (row < m) {
          const T* src = A + row * n + col0 + (int64_t)cv * VEC;
          T tmp[VEC];
#pragma unroll
          for (int e = 0; e < VEC; ++e) tmp[e] = (col0 + cv * VEC + e < n) ? src[e] : T(0);
          val = *reinterpret_cast<u4_t*>(tmp);
        }
      }
      v[i] = val;
    }
  }

  // Row pitch TT, the blocks of 16 columns of row r permuted by an exclusive or with swz(r).
  template <class Swz>
  __device__ void commit_swizzled(T* __restrict__ As, int rows, Swz swz) const {
    const int nv = rows * VPR;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      const int idx = (int)threadIdx.x + i * NTH;
      if (idx < nv) {
        const int rr = idx / VPR, col = idx % VPR * VEC;
        *reinterpret_cast<u4_t*>(As + rr * TT + (col ^ swz(rr))) = v[i];
      }
    }
  }

  template <int PAD = 1>
  __device__ void commit(T* __restrict__ As, int rows) const {
    constexpr int AP = TT + PAD;
    const int nv = rows * VPR;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      const int idx = (int)threadIdx.x + i * NTH;
      if (idx < nv) {
        const int rr = idx / VPR, cv = idx % VPR;
        T tmp[VEC];
        *reinterpret_cast<u4_t*>(tmp) = v[i];
#pragma unroll
        for (int e = 0; e < VEC; ++e) As[rr * AP + cv * VEC + e] = tmp[e];
      }
    }
  }
};

__device__ inline bool ptr_aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace ttr
