// The filter of one Fourier mode (file comment of kernels_fft.hip), shared by
// k_mode_apply and k_cols.
#ifndef REXII_MODE_FILTER_H
#define REXII_MODE_FILTER_H

#include <hip/hip_runtime.h>

#include "kernels_fft.h"

namespace rexii {

// Canonical wavenumber of k on an axis of n points: the smallest index
// with the same s^2 (centred differences: sin^2(2 pi k / n) has period n/2
// and is symmetric about n/4 for even n, symmetric about n/2 for odd n;
// Fourier differentiation: s^2 depends on |signed k|, the Nyquist mode's
// derivative is 0).  theta, and with it the coefficients of r(t A(k)),
// depends on the mode only through these two numbers.
__host__ __device__ inline int canon_index(int k, int n, int deriv) {
  if (deriv == 0 && n % 2 == 0) {
    const int h = n / 2, kc = k % h;
    return kc < h - kc ? kc : h - kc;
  }
  if (deriv != 0 && 2 * k == n) return 0;
  return k < n - k ? k : n - k;
}

// Symmetric tables (square grids: s_x and s_y are the same function, so the
// pairs (a, b) and (b, a) share theta): entries e = b (b + 1) / 2 + a, a <= b.
__host__ __device__ inline int tri_index(int a, int b) { return a <= b ? b * (b + 1) / 2 + a : a * (a + 1) / 2 + b; }

// f <- a0 f + C1 X f + C2 X^2 f for mode (kx, ky), X = t A(k) with the mode's
// own (signed) symbols.
__device__ __forceinline__ void mode_filter(const ModeFilter& m, int kx, int ky, double2 (&f)[3]) {
  const int ca = canon_index(kx, m.nx, m.deriv), cb = canon_index(ky, m.ny, m.deriv);
  const int e = m.sym ? tri_index(ca, cb) : cb * m.cnx + ca;
  double2 c;
  if (m.ns <= 1) {
    c = m.coef[e];
  } else {
    // the splits' unscaled sums, added in split order (as k_mode_coef_sum)
    double c1 = 0.0, c2 = 0.0;
    for (int q = 0; q < m.ns; ++q) {
      const double2 v = m.coef[size_t(q) * m.ne + e];
      c1 += v.x;
      c2 += v.y;
    }
    c = make_double2(m.scale * c1, m.scale * c2);
  }
  const double sx = m.sxt[kx], sy = m.syt[ky];
  // X v with X = t A(k); -i a (x + i y) = (a y, -a x)
  const double hx = m.t * m.H * sx, hy = m.t * m.H * sy, gx = m.t * m.g * sx, gy = m.t * m.g * sy, tf = m.t * m.fc;
  auto apply = [&](const double2 (&v)[3], double2 (&o)[3]) {
    o[0] = make_double2(hx * v[1].y + hy * v[2].y, -(hx * v[1].x + hy * v[2].x));
    o[1] = make_double2(gx * v[0].y + tf * v[2].x, -gx * v[0].x + tf * v[2].y);
    o[2] = make_double2(gy * v[0].y - tf * v[1].x, -gy * v[0].x - tf * v[1].y);
  };
  double2 x1[3], x2[3];
  apply(f, x1);
  apply(x1, x2);
#pragma unroll
  for (int q = 0; q < 3; ++q)
    f[q] = make_double2(m.a0 * f[q].x + c.x * x1[q].x + c.y * x2[q].x, m.a0 * f[q].y + c.x * x1[q].y + c.y * x2[q].y);
}

}  // namespace rexii

#endif
