// Dynamic LDS of the leading-eigenpair kernels, in doubles (host code).
#pragma once

#include <algorithm>
#include <cstddef>

namespace ttr {

constexpr int kWyPanel = 16;  // reflectors of one compact-WY panel

// Compiled width of the row solve in the Cholesky-QR for r columns.
inline int chol_qr_width(int r) { return r <= 16 ? 16 : r <= 32 ? 32 : 64; }

// The Cholesky-QR's Gram / R factor (r rows of pitch r + 1) and 1 / R_jj behind it (room for
// as many).  The row solve loads whole rows of R at its compiled width, entries that it then
// leaves unused beyond column r: the last row ends (r - 1)(r + 1) + width doubles after the
// factor's start, which for r <= 2 is more than the two arrays hold.
inline size_t chol_qr_doubles(int r) {
  return std::max((size_t)2 * r * (r + 1), (size_t)(r - 1) * (r + 1) + chol_qr_width(r));
}

// k_eig_top: packed reflectors, Y (n rows of pitch r + 1), the Cholesky-QR's arrays and, behind
// their first 2 r (r + 1) entries, bv twisted factorisations (D, L, U).
inline size_t eig_top_factor_at(int n, int r) { return (size_t)((n * (n - 1) / 2 + 1) & ~1) + (size_t)n * (r + 1); }
inline size_t eig_top_lds(int n, int r, int bv) {
  const size_t used = (size_t)2 * r * (r + 1) + (size_t)3 * bv * n;
  return (eig_top_factor_at(n, r) + std::max(used, chol_qr_doubles(r))) * sizeof(double) + 16;
}

// k_back_wy: Y, one panel of reflectors (n rows of pitch 17), its products (16 rows of pitch
// r + 1), the Cholesky-QR's arrays.
inline size_t back_wy_factor_at(int n, int r) {
  return (size_t)n * (r + 1) + (size_t)n * (kWyPanel + 1) + (size_t)kWyPanel * (r + 1);
}
inline size_t back_wy_lds(int n, int r) { return (back_wy_factor_at(n, r) + chol_qr_doubles(r)) * sizeof(double); }

}  // namespace ttr
