// MRT change of basis (section 5) as compile-time constants, and its
// products with a site's nine values.
//
// The matrices are rebuilt from their velocity polynomials in tensor order;
// the inverses come from Gauss-Jordan elimination with partial pivoting.  As
// kernel arguments the 162 entries had to be fetched through the scalar
// cache in several dependent batches by every wavefront, more than the
// scalar registers hold; as literals they cost nothing, and the zeros (22 of
// 81 in M1, more in M2) no instruction.  The products add the remaining terms
// in the same order with the same roundings.  512^2 step kernel on one box:
// FP32 9.8 -> 6.6 us, FP64 18.4 -> 9.7 us; FP32 adjoint kernel 16.0 -> 10.8.
#pragma once

#include <hip/hip_runtime.h>

namespace lbm {

struct MrtTable { double M[81], Minv[81]; };

constexpr double c_abs(double x) { return x < 0.0 ? -x : x; }

// basis: 0 M1 (rows rho, e, epsilon, j_x, q_x, j_y, q_y, p_xx, p_xy), 1 M2.
constexpr MrtTable mrt_table(int basis) {
  MrtTable t{};
  for (int i = 0; i < 9; ++i) {
    const double vx = (i % 3) - 1, vy = (i / 3) - 1, v2 = vx * vx + vy * vy;
    const double m1[9] = {1, -4 + 3 * v2, 4 - 10.5 * v2 + 4.5 * v2 * v2, vx, (-5 + 3 * v2) * vx,
                          vy, (-5 + 3 * v2) * vy, vx * vx - vy * vy, vx * vy};
    const double m2[9] = {1, vx, vy, v2, vx * vx - vy * vy, vx * vy, vx * vx * vy, vx * vy * vy,
                          vx * vx * vy * vy};
    for (int k = 0; k < 9; ++k) t.M[k * 9 + i] = basis == 0 ? m1[k] : m2[k];
  }
  double a[9][18] = {};
  for (int r = 0; r < 9; ++r)
    for (int c = 0; c < 18; ++c) a[r][c] = c < 9 ? t.M[r * 9 + c] : (c - 9 == r ? 1.0 : 0.0);
  for (int c = 0; c < 9; ++c) {
    int p = c;
    for (int r = c + 1; r < 9; ++r)
      if (c_abs(a[r][c]) > c_abs(a[p][c])) p = r;
    for (int k = 0; k < 18; ++k) {
      const double s = a[c][k];
      a[c][k] = a[p][k];
      a[p][k] = s;
    }
    const double piv = a[c][c];
    for (int k = 0; k < 18; ++k) a[c][k] /= piv;
    for (int r = 0; r < 9; ++r) {
      if (r == c) continue;
      const double f = a[r][c];
      if (f != 0.0)
        for (int k = 0; k < 18; ++k) a[r][k] -= f * a[c][k];
    }
  }
  for (int r = 0; r < 9; ++r)
    for (int c = 0; c < 9; ++c) t.Minv[r * 9 + c] = a[r][c + 9];
  return t;
}

// out = M v (INV: Minv v), or with TR the transpose's product.
template <class R, int BASIS, bool INV, bool TR>
__device__ __forceinline__ void mrt_mul(const R v[9], R out[9]) {
  constexpr MrtTable t = mrt_table(BASIS);
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    R s = R(0);
#pragma unroll
    for (int j = 0; j < 9; ++j) {
      const int e = TR ? j * 9 + k : k * 9 + j;
      const double c = INV ? t.Minv[e] : t.M[e];
      if (c != 0.0) s = fma((R)c, v[j], s);
    }
    out[k] = s;
  }
}
template <class R, bool INV, bool TR>
__device__ __forceinline__ void mrt_mul(int basis, const R v[9], R out[9]) {
  if (basis == 0) mrt_mul<R, 0, INV, TR>(v, out);
  else mrt_mul<R, 1, INV, TR>(v, out);
}

}  // namespace lbm
