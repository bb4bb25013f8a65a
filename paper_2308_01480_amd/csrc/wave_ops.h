// Cross-lane reductions of float64 values inside one 64-lane wavefront (DPP row
// operations and lane reads): no LDS and no barriers.
#pragma once

#include <hip/hip_runtime.h>

namespace ttr {

template <int CTRL>
__device__ inline double dpp_mov(double v) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xF, 0xF, false);
  hi = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// Sums over aligned lane groups; every lane of the group obtains the same bits.
__device__ inline double sum8(double v) {
  v += dpp_mov<0xB1>(v);   // lane ^ 1
  v += dpp_mov<0x4E>(v);   // lane ^ 2
  v += dpp_mov<0x141>(v);  // mirror within 8
  return v;
}
__device__ inline double sum16(double v) {
  v += dpp_mov<0xB1>(v);   // lane ^ 1
  v += dpp_mov<0x4E>(v);   // lane ^ 2
  v += dpp_mov<0x141>(v);  // mirror within 8
  v += dpp_mov<0x140>(v);  // mirror within 16
  return v;
}
__device__ inline double lane_value(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}
// Row broadcasts (lane 15 of a row into the next row, lane 31 into the upper half) leave
// ((row 0 + row 1) + (row 2 + row 3)) of the rows' sums in lane 63.
template <int CTRL>
__device__ inline double dpp_row_bcast(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ inline double sum64(double v) {
  v = sum16(v);
  v += dpp_row_bcast<0x142>(v);
  v += dpp_row_bcast<0x143>(v);
  return lane_value(v, 63);
}
__device__ inline double min64(double v) {
  v = fmin(v, dpp_mov<0xB1>(v));
  v = fmin(v, dpp_mov<0x4E>(v));
  v = fmin(v, dpp_mov<0x141>(v));
  v = fmin(v, dpp_mov<0x140>(v));
  return fmin(fmin(lane_value(v, 0), lane_value(v, 16)), fmin(lane_value(v, 32), lane_value(v, 48)));
}
__device__ inline double max64(double v) { return -min64(-v); }
// 1/x to full precision from the hardware estimate and two Newton steps (|x| >= DBL_MIN).
__device__ inline double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// 1/sqrt(x) for x > 0: the hardware estimate refined by three Newton steps (quadratic
// convergence from the estimate's relative error to float64 rounding level).
__device__ inline double rsqrt_nr(double x) {
  double r = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
  r = r * fma(-hx * r, r, 1.5);
  r = r * fma(-hx * r, r, 1.5);
  r = r * fma(-hx * r, r, 1.5);
  return r;
}

}  // namespace ttr
