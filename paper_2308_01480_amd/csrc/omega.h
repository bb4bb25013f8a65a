// Entries of the Gaussian test matrices Omega_k (Algorithm 3, step 3) on the device:
// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC 2011) keyed by (seed, k) with counter
// (beta, g, 0, 0) feeds the eight entries c = 8g .. 8g+7 of row beta: word j = (c % 8) / 2
// splits into two 23-bit uniforms u (low half) and v (high half), and the Box-Muller
// transform sqrt(-2 ln u) (cos 2 pi v, sin 2 pi v) gives entries 8g + 2j and 8g + 2j + 1.
// The transform is defined as a fixed sequence of correctly rounded float32 operations (no
// fused multiply-add), so that any implementation following the same sequence draws the same
// bits.  Here the one division and the square root are the hardware's float32 reciprocal (root)
// estimate with one fused correction: both depend on the 23 bits of u alone, and over all 2^23
// of them the results equal the correctly rounded ones.
//
// What bounds it: vector ALU.  A wave draws 512 entries in about 2110 cycles, 890 of them
// Philox; with the division and the root in float64, quadrants found by comparisons and
// uniforms scaled before use it took 2630.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "convert.h"

namespace ttr {

// The 128-bit product of a 64-bit word and a 64-bit constant from four 32 x 32 -> 64
// products, each partial sum kept below 2^64: lo = (p2 mod 2^32) 2^32 + (p0 mod 2^32), hi = p3.
__device__ inline void mulhilo64(uint64_t a, uint64_t b, uint64_t* hi, uint64_t* lo) {
  const uint64_t aL = (uint32_t)a, aH = a >> 32, bL = (uint32_t)b, bH = b >> 32;
  const uint64_t p0 = aL * bL;
  const uint64_t p1 = aH * bL + (p0 >> 32);
  const uint64_t p2 = aL * bH + (uint32_t)p1;
  *hi = aH * bH + ((p1 >> 32) + (p2 >> 32));
  *lo = (p2 << 32) | (uint32_t)p0;
}

__device__ inline void philox4x64_10(uint64_t (&x)[4], uint64_t k0, uint64_t k1) {
  const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    uint64_t hi0, lo0, hi1, lo1;
    mulhilo64(x[0], M0, &hi0, &lo0);
    mulhilo64(x[2], M1, &hi1, &lo1);
    const uint64_t y0 = hi1 ^ x[1] ^ k0, y2 = hi0 ^ x[3] ^ k1;
    x[0] = y0; x[1] = lo1; x[2] = y2; x[3] = lo0;
    k0 += W0; k1 += W1;
  }
}

// sqrt(-2 ln u) of u = ((w >> 9) + 1/2) 2^-23: u 2^23 = 2^e f with f in [sqrt 1/2, sqrt 2], the
// atanh series of ln f to t^11, t = (f - 1) / (f + 1), plus (e - 23) ln 2.
__device__ __attribute__((always_inline)) inline float radius32(uint32_t w) {
#pragma clang fp contract(off)
  const uint32_t bits = __float_as_uint((float)(w >> 9) + 0.5f);
  const int e = (int)(bits - 0x3F3504F4u) >> 23;  // f > 0x1.6a09e6p+0 takes the next exponent
  const float f = __uint_as_float(bits - ((uint32_t)e << 23));
  const float num = f - 1.0f, den = f + 1.0f;
  const float rc = __builtin_amdgcn_rcpf(den);
  const float t0 = num * rc;
  const float t = __builtin_fmaf(__builtin_fmaf(-den, t0, num), rc, t0);
  const float t2 = t * t;
  float p = 0x1.745d18p-4f * t2 + 0x1.c71c72p-4f;
  p = p * t2 + 0x1.24924ap-3f;
  p = p * t2 + 0x1.99999ap-3f;
  p = p * t2 + 0x1.555556p-2f;
  p = p * t2 + 1.0f;
  const float y = -2.0f * ((float)(e - 23) * 0x1.62e430p-1f + (t + t) * p);
  const float rs = __builtin_amdgcn_rsqf(y);
  const float r0 = y * rs;
  return __builtin_fmaf(__builtin_fmaf(-r0, r0, y), 0.5f * rs, r0);
}

// (cos 2 pi v, sin 2 pi v) of v = ((w >> 9) + 1/2) 2^-23: the quadrant is the word's two top
// bits, the fraction of 4 v the 21 bits below; Taylor polynomials of sin x (to x^13) and cos x
// (to x^14) on x in [0, pi/2).
__device__ __attribute__((always_inline)) inline void cossin32(uint32_t w, float* cs, float* sn) {
#pragma clang fp contract(off)
  const float x = ((float)((w >> 9) & 0x1FFFFFu) + 0.5f) * (0x1.921fb6p+0f * 0x1p-21f);
  const float x2 = x * x;
  float sp = 0x1.612462p-33f * x2 + -0x1.ae6456p-26f;
  sp = sp * x2 + 0x1.71de3ap-19f;
  sp = sp * x2 + -0x1.a01a02p-13f;
  sp = sp * x2 + 0x1.111112p-7f;
  sp = sp * x2 + -0x1.555556p-3f;
  sp = sp * x2 + 1.0f;
  const float s = x * sp;
  float cp = -0x1.93974ap-37f * x2 + 0x1.1eed8ep-29f;
  cp = cp * x2 + -0x1.27e4fcp-22f;
  cp = cp * x2 + 0x1.a01a02p-16f;
  cp = cp * x2 + -0x1.6c16c2p-10f;
  cp = cp * x2 + 0x1.555556p-5f;
  cp = cp * x2 + -0.5f;
  const float c = cp * x2 + 1.0f;
  // quadrants 0..3: (c, s), (-s, c), (-c, -s), (s, -c)
  const bool odd = (w & 0x40000000u) != 0;
  *cs = __uint_as_float(__float_as_uint(odd ? s : c) ^ ((w ^ (w << 1)) & 0x80000000u));
  *sn = __uint_as_float(__float_as_uint(odd ? c : s) ^ (w & 0x80000000u));
}

// The eight entries c = 8g .. 8g+7 of row beta of Omega_k.
__device__ __attribute__((always_inline)) inline void omega8(uint64_t seed, int k, int64_t beta, int g,
                                                             float (&z)[8]) {
#pragma clang fp contract(off)
  uint64_t x[4] = {(uint64_t)beta, (uint64_t)g, 0ull, 0ull};
  philox4x64_10(x, seed, (uint64_t)k);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float r = radius32((uint32_t)x[j]);
    float cs, sn;
    cossin32((uint32_t)(x[j] >> 32), &cs, &sn);
    z[2 * j] = r * cs;
    z[2 * j + 1] = r * sn;
  }
}

}  // namespace ttr

namespace ttr {

// Item id of a tile of `rows` rows (a compile-time power of two): consecutive lanes take
// consecutive rows of one group of eight columns, so no runtime division, neighbouring
// addresses in a transposed tile, and, from 64 rows on, one group for the whole wave (waves
// start at multiples of 64 items), whose share of the second Philox round is scalar.
__device__ __attribute__((always_inline)) inline int omega_group(int id, int rows) {
  const int g = id / rows;
  return rows % 64 == 0 ? __builtin_amdgcn_readfirstlane(g) : g;
}

// Rows [beta0, beta0 + rows) of Omega_k (zero beyond row n), entries c < 8 ceil(s / 8)
// (zero for c >= s), rounded once to T and written into LDS by `nthr` threads (tid =
// 0 .. nthr-1 among them): entry (b, c) goes to Om[b * rs + c * cs] (rs = pitch, cs = 1
// for a row-major tile; rs = 1, cs = pitch for a transposed one).
template <typename T>
__device__ __attribute__((always_inline)) inline void omega_tile(uint64_t seed, int k, int64_t beta0, int rows,
                                                                 int64_t n, int s, T* __restrict__ Om, int rs, int cs,
                                                                 int tid, int nthr) {
  const int g8 = (s + 7) / 8;
  for (int id = tid; id < rows * g8; id += nthr) {
    const int g = omega_group(id, rows), b = id % rows;
    float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (beta0 + b < n) omega8(seed, k, beta0 + b, g, z);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int c = 8 * g + j;
      // z is a float32: its round to nearest even into T equals that of (double)z
      Om[b * rs + c * cs] = c < s ? (T)z[j] : T(0);
    }
  }
}

}  // namespace ttr
