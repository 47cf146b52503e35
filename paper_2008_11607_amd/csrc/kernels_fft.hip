// Fourier-space REXII for a constant depth (the paper solves its test
// problem this way, per Fourier mode, Sec. 4).
//
// After a 2D FFT of (eta, u, v), mode k carries the 3 x 3 symbol
//   A(k) = [[0, -i H s_x, -i H s_y], [-i g s_x, 0, f_c], [-i g s_y, -f_c, 0]],
// with s = n sin(2 pi k / n) for centred differences, or s = 2 pi k (signed
// k, the odd derivative of the Nyquist mode taken as 0) for Fourier
// differentiation.  Its eigenvalues are 0 and +-i omega,
// omega^2 = f_c^2 + g H (s_x^2 + s_y^2), so for X = t A(k) and theta = t omega
// any function r of X is the quadratic that interpolates r on {0, +-i theta}
// (Theorem 1 of the paper, matrix functions through the eigenvalues):
//   r(X) = c0 I + c1 X + c2 X^2.
// For one pole, r(x) = w / (x - z), the Newton divided differences on the
// nodes (0, i theta, -i theta) are w/(-z), w/(z (i theta - z)) and
// -w/(z (z^2 + theta^2)), which give
//   c1 = -w / (z^2 + theta^2),  c2 = (-w / z) / (z^2 + theta^2).
// The result must be real (eq. modifiedRexiMatrixReducedSum takes the real
// part); since A(-k) = conj(A(k)) and F(-k) = conj(F(k)) for a real state,
// the real part in physical space is, per mode, the same quadratic with
// Re c0, Re c1, Re c2.  So the half spectrum of a real-to-complex FFT is
// filtered with real coefficients and a complex-to-real FFT returns u.
//
// Per term of the sum the filter needs Re(c1) and Re(c2) at theta^2:
// with z^2 = a + i b and s = a + theta^2,
//   Re(-w e) = -(w_r s + w_i b) / (s^2 + b^2),  e = 1/(z^2 + theta^2),
// and the two poles of one term of the reduced sum have equal a and b^2
// (z_2 = -conj(z_1)), so they share the denominator s^2 + b^2 and are
// merged into one table entry (a, b^2, A1, B1, A2, B2):
//   Re c1 += (A1 s + B1) / (s^2 + b^2),  Re c2 += (A2 s + B2) / (s^2 + b^2).
// theta^2 depends on the mode only through s_x^2 and s_y^2, which repeat
// along each axis, so the sums are formed once per distinct pair
// (k_mode_coef) and a second kernel applies the quadratic to every mode
// (k_mode_apply).  On square grids the pair is unordered (s_x and s_y are
// the same function), which halves the table again.
#include <hip/hip_runtime.h>
#include <rocfft/rocfft.h>

#include <cmath>
#include <map>
#include <mutex>
#include <string>
#include <tuple>

#include "kernels.h"
#include "kernels_fft.h"
#include "mode_filter.h"
#include "rexii_internal.h"

namespace rexii {

constexpr int kModeWaves = 16;  // most waves (term slices) per block
constexpr int kTermDoubles = 6;

// 1/x to full FP64 precision: hardware reciprocal estimate and two
// Newton-Raphson steps r <- r + r (1 - x r) (each squares the relative error).
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// s * s + b with b read from a scalar register (one VOP3 instruction; the
// compiler otherwise copies b into vector registers for a VOP2 fmac).
__device__ __forceinline__ double sq_plus(double s, double b) {
  double d;
  asm("v_fma_f64 %0, %1, %1, %2" : "=v"(d) : "v"(s), "s"(b));
  return d;
}

// s for wavenumber index k of an axis of n points (see file comment); the
// kernels read it from a table the host fills once per grid.
double axis_symbol(int k, int n, int deriv) {
  if (deriv == 0) return double(n) * std::sin(2.0 * M_PI * double(k) / double(n));
  const int ks = (2 * k == n) ? 0 : (2 * k < n ? k : k - n);
  return 2.0 * M_PI * double(ks);
}

// The four running sums of a range of terms: (A s + B) / d is accumulated as
// (s/d) A + (1/d) B, one table operand per FMA and four independent chains.
struct TermAcc {
  double c1a = 0.0, c1b = 0.0, c2a = 0.0, c2b = 0.0;
  __device__ __forceinline__ void one(const double* q, double s, double i1) {
    const double e1 = i1 * s;
    c1a = fma(e1, q[2], c1a);
    c1b = fma(i1, q[3], c1b);
    c2a = fma(e1, q[4], c2a);
    c2b = fma(i1, q[5], c2b);
  }
};

// Adds the terms [lo, hi) at theta^2 = th2 + lo2 (lo2: rounding of th2 where
// it is known, else 0), but those in the lane's [nl, nh).  The range is
// wave-uniform, so the entries arrive through scalar loads.
template <bool LOW, bool SKIP = false>
__device__ __forceinline__ void term_range(const double* __restrict__ tab, int lo, int hi, double th2, double lo2,
                                           TermAcc& c, int nl = 0, int nh = 0) {
  // Four terms share one reciprocal: 1/d1 = (d2 d3 d4) / (d1 d2 d3 d4).
  // d >= b^2 = (2 h^2 mu n)^2 for n >= 1 and d >= a^2 = (h mu)^4 for n = 0, and
  // d < 4 (theta^2 + (h N)^2)^2, so the product stays in range for any h above
  // 1e-3 and theta below 1e18.
  auto sum = [&](const double* q) { return LOW ? (q[0] + th2) + lo2 : q[0] + th2; };
  auto add = [&](const double* q, int j, double s, double i1) {
    c.one(q, s, SKIP && j >= nl && j < nh ? 0.0 : i1);
  };
  auto pair = [&](const double* q, int j) {
    const double s1 = sum(q), s2 = sum(q + kTermDoubles);
    const double d1 = sq_plus(s1, q[1]), d2 = sq_plus(s2, q[kTermDoubles + 1]);
    const double r = recip(d1 * d2);
    add(q, j, s1, r * d2);
    add(q + kTermDoubles, j + 1, s2, r * d1);
  };
  auto quad = [&](const double* q, int j) {
    const double s1 = sum(q), s2 = sum(q + kTermDoubles);
    const double s3 = sum(q + 2 * kTermDoubles), s4 = sum(q + 3 * kTermDoubles);
    const double d1 = sq_plus(s1, q[1]), d2 = sq_plus(s2, q[kTermDoubles + 1]);
    const double d3 = sq_plus(s3, q[2 * kTermDoubles + 1]), d4 = sq_plus(s4, q[3 * kTermDoubles + 1]);
    const double p12 = d1 * d2, p34 = d3 * d4;
    const double r = recip(p12 * p34);
    const double r12 = r * p34, r34 = r * p12;
    add(q, j, s1, r12 * d2);
    add(q + kTermDoubles, j + 1, s2, r12 * d1);
    add(q + 2 * kTermDoubles, j + 2, s3, r34 * d4);
    add(q + 3 * kTermDoubles, j + 3, s4, r34 * d3);
  };
  int j = lo;
  for (; j + 7 < hi; j += 8) {  // unrolled by hand: the loads of two quads issue together
    const double* q = tab + size_t(j) * kTermDoubles;
    quad(q, j);
    quad(q + 4 * kTermDoubles, j + 4);
  }
  for (; j + 1 < hi; j += 2) pair(tab + size_t(j) * kTermDoubles, j);
  if (j < hi) {
    const double* q = tab + size_t(j) * kTermDoubles;
    const double s1 = sum(q);
    add(q, j, s1, recip(sq_plus(s1, q[1])));
  }
}

// Re c1 and Re c2 at theta^2 = th2 over the terms [w per, (w + 1) per) of
// the table (per = ceil(nterm / nw)).
__device__ __forceinline__ void term_sums(const double* __restrict__ tab, int nterm, int w, int nw, double th2,
                                          double& c1, double& c2) {
  const int per = (nterm + nw - 1) / nw;
  const int lo = min(nterm, w * per), hi = min(nterm, lo + per);
  TermAcc c;
  term_range<false>(tab, lo, hi, th2, 0.0, c);
  c1 = c.c1a + c.c1b;
  c2 = c.c2a + c.c2b;
}

// 0..n/4 (centred, even n), 0..(n-1)/2 (odd n), 0..n/2-1 (Fourier
// differentiation, even n: the Nyquist mode has index 0)
int canon_count(int n, int deriv) { return n % 2 ? (n + 1) / 2 : deriv ? n / 2 : n / 4 + 1; }

// The pole sums per distinct frequency: coef[cy * cnx + cx] = scale (Re c1,
// Re c2) at theta^2 = t^2 (f_c^2 + g H (s_x^2 + s_y^2)) for the canonical
// wavenumbers (cx, cy).  tab: nterm entries of kTermDoubles.  Block: 64
// entries (one per lane) x nw waves; grid row s (blockIdx.y) takes split s of
// the terms, wave w of the block slice w of that split, and the slices are
// added in wave order through (nw - 1) x 1 KB of dynamic LDS.  With one
// split the block writes scale (c1, c2) to coef; with several it writes its
// unscaled sums to part[s][e] and k_mode_coef_sum adds the splits in order.
__device__ inline void tri_coords(int e, int& a, int& b) {
  b = int((sqrt(8.0 * double(e) + 1.0) - 1.0) * 0.5);
  if ((b + 1) * (b + 2) / 2 <= e) ++b;
  if (b * (b + 1) / 2 > e) --b;
  a = e - b * (b + 1) / 2;
}

__global__ __launch_bounds__(64 * kModeWaves) void k_mode_coef(double2* __restrict__ coef,
                                                               double2* __restrict__ part, int cnx, int cny, int sym,
                                                               const double* __restrict__ sxt,
                                                               const double* __restrict__ syt, double t, double g,
                                                               double H, double fc, double scale,
                                                               const double* __restrict__ tab, int nterm) {
  extern __shared__ double red[];
  const int ne = sym ? cnx * (cnx + 1) / 2 : cnx * cny;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int nw = int(blockDim.x >> 6);
  const int ns = int(gridDim.y), sp = int(blockIdx.y);
  const int per_s = (nterm + ns - 1) / ns;
  const int lo_s = min(nterm, sp * per_s), cnt_s = min(nterm, lo_s + per_s) - lo_s;
  const int e = int(blockIdx.x) * 64 + lane;
  const bool live = e < ne;
  int cx = 0, cy = 0;
  if (live) {
    if (sym) {
      tri_coords(e, cx, cy);
    } else {
      cx = e % cnx;
      cy = e / cnx;
    }
  }
  const double sx = sxt[cx], sy = syt[cy];
  const double th2 = t * t * fma(g * H, fma(sx, sx, sy * sy), fc * fc);
  double c1, c2;
  term_sums(tab + size_t(lo_s) * kTermDoubles, cnt_s, w, nw, th2, c1, c2);
  if (nw > 1) {
    if (w > 0) {
      red[(w - 1) * 128 + lane] = c1;
      red[(w - 1) * 128 + 64 + lane] = c2;
    }
    __syncthreads();
    if (w != 0) return;
    for (int v = 1; v < nw; ++v) {
      c1 += red[(v - 1) * 128 + lane];
      c2 += red[(v - 1) * 128 + 64 + lane];
    }
  }
  if (!live) return;
  if (ns == 1)
    coef[e] = make_double2(scale * c1, scale * c2);
  else
    part[size_t(sp) * ne + e] = make_double2(c1, c2);
}

// coef[e] = scale sum_s part[s][e], splits added in index order.
__global__ __launch_bounds__(256) void k_mode_coef_sum(double2* __restrict__ coef, const double2* __restrict__ part,
                                                       int ne, int ns, double scale) {
  const int e = int(blockIdx.x) * 256 + threadIdx.x;
  if (e >= ne) return;
  double c1 = 0.0, c2 = 0.0;
  for (int s = 0; s < ns; ++s) {
    const double2 v = part[size_t(s) * ne + e];
    c1 += v.x;
    c2 += v.y;
  }
  coef[e] = make_double2(scale * c1, scale * c2);
}

// ---------------------------------------------------------------------------
// Pole sums by near and far terms.
//
// As functions of s = theta^2 the terms are analytic but for poles at
// s = -z^2 = (y^2 - d^2) +- 2 i d y, y = h j, d = h |mu|.  theta in [0, theta_max]
// is cut into boxes; for the s of one box the terms whose poles lie outside
// the ellipse with foci at the box's ends and semi-axes (kFarA, kFarB) half
// widths (sum rho = 3.2) are summed as one polynomial: their sum is formed at
// kCheb Chebyshev points of the box and interpolated (each term's error is
// rho^-kCheb = 7e-17 of the term).  The few terms inside (y within about
// 1.76 half widths of the box's centre in theta) are added directly.  So
// nbox kCheb theta values meet the whole table instead of every distinct one,
// and each of those meets (near terms + a polynomial).
//
// Box edges in theta: 0, 4, 8, 16, .. up to tg = 4 2^k >= w, then steps of w:
// c1 ~ 1/theta and c2 ~ 1/theta^2 vary by no more than 4 within a box beyond
// the first, so the interpolation's error is relative to the values there.
// The polynomial's variable is s, not theta: theta^2 - s_c is exact to the
// rounding of theta^2, a rounded theta (5e-13 at 5000) is used only to pick
// the box.
// ---------------------------------------------------------------------------
constexpr double kFarA = 1.75625, kFarB = 1.44375;  // (rho +- 1/rho) / 2, rho = 3.2

__device__ __forceinline__ int far_box(const FarBoxes& fb, double th) {
  int b;
  if (th < fb.tg) {
    b = th < 4.0 ? 0 : ilogb(th) - 1;
  } else {
    b = fb.k + 1 + int((th - fb.tg) * fb.inv_w);
  }
  return min(max(b, 0), fb.nbox - 1);
}

// Centre and half width of box b in s.
__device__ __forceinline__ void far_span(const FarBoxes& fb, int b, double& sc, double& sd) {
  const double lo = b == 0 ? 0.0 : b <= fb.k ? ldexp(4.0, b - 1) : fb.tg + (b - fb.k - 1) * fb.w;
  const double hi = b <= fb.k ? ldexp(4.0, b) : lo + fb.w;
  sc = 0.5 * fma(lo, lo, hi * hi);
  sd = 0.5 * (hi - lo) * (hi + lo);
}

// The near terms [lo, hi) of a box: with v = y^2 the pole is inside the
// ellipse where (v - p)^2 / al^2 + 4 d^2 v / be^2 < 1, p = d^2 + sc; one
// term more on either side covers the rounding of the roots.
__device__ __forceinline__ void far_window(const FarBoxes& fb, double sc, double sd, int nterm, int& lo, int& hi) {
  const double al = kFarA * sd, p = fma(fb.d, fb.d, sc);
  const double q = p - 2.0 * fb.d * fb.d * ((kFarA / kFarB) * (kFarA / kFarB));
  const double disc = fma(q, q, fma(-p, p, al * al));
  lo = hi = 0;
  if (!(disc > 0.0)) return;
  const double r = sqrt(disc), vh = q + r, vl = q - r;
  if (!(vh > 0.0)) {
    // every y > 0 is far; n = 0 has its pole at v = 0
    hi = p * p < al * al ? 1 : 0;
    return;
  }
  lo = vl > 0.0 ? min(nterm, max(0, int(sqrt(vl) * fb.inv_h) - 1)) : 0;
  hi = int(min(double(nterm), sqrt(vh) * fb.inv_h + 2.0));
}

// Far sums at the Chebyshev points.  Lanes 0..31 and 32..63 of every wave
// hold the points of two neighbouring boxes; the term slices are split over
// the block's waves and the grid's rows as in k_mode_coef.  node[s][b][i].
__global__ __launch_bounds__(64 * kModeWaves) void k_mode_far(double2* __restrict__ node, FarBoxes fb,
                                                              const double* __restrict__ tab, int nterm) {
  extern __shared__ double red[];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int nw = int(blockDim.x >> 6);
  const int slices = int(gridDim.y) * nw, sl = int(blockIdx.y) * nw + w;
  const int per = (nterm + slices - 1) / slices;
  const int lo = min(nterm, sl * per), hi = min(nterm, lo + per);
  const int b = int(blockIdx.x) * 2 + (lane >> 5), i = lane & 31;
  const int bb = min(b, fb.nbox - 1);
  double sc, sd;
  far_span(fb, bb, sc, sd);
  int nl, nh;
  far_window(fb, sc, sd, nterm, nl, nh);
  const double x = cospi((2 * i + 1) * (0.5 / kCheb));
  const double th2 = fma(sd, x, sc), lo2 = fma(sd, x, sc - th2);  // the point and its rounding
  // the range that is near for either box
  const int l0 = __builtin_amdgcn_readlane(nl, 0), l1 = __builtin_amdgcn_readlane(nl, 32);
  const int h0 = __builtin_amdgcn_readlane(nh, 0), h1 = __builtin_amdgcn_readlane(nh, 32);
  const int ul = l0 < h0 ? (l1 < h1 ? min(l0, l1) : l0) : l1;
  const int uh = l0 < h0 ? (l1 < h1 ? max(h0, h1) : h0) : max(l1, h1);
  TermAcc c;
  term_range<true>(tab, lo, min(hi, ul), th2, lo2, c);
  term_range<true, true>(tab, max(lo, ul), min(hi, uh), th2, lo2, c, nl, nh);
  term_range<true>(tab, max(lo, uh), hi, th2, lo2, c);
  double c1 = c.c1a + c.c1b, c2 = c.c2a + c.c2b;
  if (nw > 1) {
    if (w > 0) {
      red[(w - 1) * 128 + lane] = c1;
      red[(w - 1) * 128 + 64 + lane] = c2;
    }
    __syncthreads();
    if (w != 0) return;
    for (int v = 1; v < nw; ++v) {
      c1 += red[(v - 1) * 128 + lane];
      c2 += red[(v - 1) * 128 + 64 + lane];
    }
  }
  if (b < fb.nbox) node[(size_t(blockIdx.y) * fb.nbox + b) * kCheb + i] = make_double2(c1, c2);
}

// Chebyshev coefficients of one box per block from its node sums (splits
// added in order): c_k = (2 - [k = 0]) / kCheb sum_i f_i cos(pi k (2i+1) / (2 kCheb)).
__global__ __launch_bounds__(4 * kCheb) void k_mode_cheb(double2* __restrict__ cheb, const double2* __restrict__ node,
                                                         int nbox, int ns) {
  __shared__ double ct[4 * kCheb];
  __shared__ double2 part[4 * kCheb];
  const int b = int(blockIdx.x), i = threadIdx.x & (kCheb - 1), g = threadIdx.x / kCheb;
  ct[threadIdx.x] = cospi(double(threadIdx.x) * (0.5 / kCheb));
  double2 f = make_double2(0.0, 0.0);
  for (int s = g; s < ns; s += 4) {
    const double2 v = node[(size_t(s) * nbox + b) * kCheb + i];
    f.x += v.x;
    f.y += v.y;
  }
  part[threadIdx.x] = f;
  __syncthreads();
  if (g == 0) {
    for (int q = 1; q < 4; ++q) {
      f.x += part[q * kCheb + i].x;
      f.y += part[q * kCheb + i].y;
    }
    part[i] = f;
  }
  __syncthreads();
  if (g > 0) return;
  double2 c = make_double2(0.0, 0.0);
  for (int m = 0; m < kCheb; ++m) {
    const double t = ct[(i * (2 * m + 1)) & (4 * kCheb - 1)];
    c.x = fma(part[m].x, t, c.x);
    c.y = fma(part[m].y, t, c.y);
  }
  const double sc = (i == 0 ? 1.0 : 2.0) / kCheb;
  cheb[size_t(b) * kCheb + i] = make_double2(sc * c.x, sc * c.y);
}

// coef[e] = scale (far polynomial + near terms) at the entry's theta.
__global__ __launch_bounds__(64) void k_mode_near(double2* __restrict__ coef, const double2* __restrict__ cheb,
                                                  FarBoxes fb, int cnx, int cny, int sym,
                                                  const double* __restrict__ sxt, const double* __restrict__ syt,
                                                  double t, double g, double H, double fc, double scale,
                                                  const double* __restrict__ tab, int nterm) {
  const int ne = sym ? cnx * (cnx + 1) / 2 : cnx * cny;
  const int e = int(blockIdx.x) * 64 + int(threadIdx.x);
  if (e >= ne) return;
  int cx, cy;
  if (sym) {
    tri_coords(e, cx, cy);
  } else {
    cx = e % cnx;
    cy = e / cnx;
  }
  const double sx = sxt[cx], sy = syt[cy];
  const double th2 = t * t * fma(g * H, fma(sx, sx, sy * sy), fc * fc);
  const int b = far_box(fb, sqrt(th2));
  double sc, sd;
  far_span(fb, b, sc, sd);
  int nl, nh;
  far_window(fb, sc, sd, nterm, nl, nh);
  const double x2 = 2.0 * ((th2 - sc) / sd);
  const double2* cb = cheb + size_t(b) * kCheb;
  double u1 = 0.0, u2 = 0.0, v1 = 0.0, v2 = 0.0;   // Clenshaw, both sums
#pragma unroll 8
  for (int k = kCheb - 1; k >= 1; --k) {
    const double2 c = cb[k];
    const double nu = fma(x2, u1, c.x - u2), nv = fma(x2, v1, c.y - v2);
    u2 = u1;
    u1 = nu;
    v2 = v1;
    v1 = nv;
  }
  const double2 c0 = cb[0];
  const double f1 = fma(0.5 * x2, u1, c0.x - u2), f2 = fma(0.5 * x2, v1, c0.y - v2);
  TermAcc c;
  const double2* tb = reinterpret_cast<const double2*>(tab);
  int j = nl;
  for (; j + 3 < nh; j += 4) {
    double q[4][6];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const double2 v = tb[size_t(j + m) * 3 + r];
        q[m][2 * r] = v.x;
        q[m][2 * r + 1] = v.y;
      }
    const double s1 = q[0][0] + th2, s2 = q[1][0] + th2, s3 = q[2][0] + th2, s4 = q[3][0] + th2;
    const double d1 = fma(s1, s1, q[0][1]), d2 = fma(s2, s2, q[1][1]);
    const double d3 = fma(s3, s3, q[2][1]), d4 = fma(s4, s4, q[3][1]);
    const double p12 = d1 * d2, p34 = d3 * d4;
    const double r = recip(p12 * p34);
    const double r12 = r * p34, r34 = r * p12;
    c.one(q[0], s1, r12 * d2);
    c.one(q[1], s2, r12 * d1);
    c.one(q[2], s3, r34 * d4);
    c.one(q[3], s4, r34 * d3);
  }
  for (; j < nh; ++j) {
    const double* q = tab + size_t(j) * kTermDoubles;
    const double s = q[0] + th2;
    c.one(q, s, recip(fma(s, s, q[1])));
  }
  coef[e] = make_double2(scale * (f1 + (c.c1a + c.c1b)), scale * (f2 + (c.c2a + c.c2b)));
}

// F: [3][ny][nxh] half spectra, filtered in place.
__global__ __launch_bounds__(256) void k_mode_apply(double2* __restrict__ F, ModeFilter mf) {
  const int nxh = mf.nx / 2 + 1;
  const int nm = nxh * mf.ny;
  const int m = int(blockIdx.x) * 256 + threadIdx.x;
  if (m >= nm) return;
  double2 f[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) f[q] = F[size_t(q) * nm + m];
  mode_filter(mf, m % nxh, m / nxh, f);
#pragma unroll
  for (int q = 0; q < 3; ++q) F[size_t(q) * nm + m] = f[q];
}

// u = f; flags[b] = 1 if block b met a value that is not finite, else 0
// (every block writes its word, so nothing has to be cleared first).
__global__ __launch_bounds__(256) void k_copy_check(const double* __restrict__ f, double* __restrict__ u, size_t n,
                                                    int* __restrict__ flags) {
  bool bad = false;
  for (size_t i = blockIdx.x * size_t(blockDim.x) + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x) {
    const double v = f[i];
    u[i] = v;
    bad = bad || !isfinite(v);
  }
  const int any = __syncthreads_or(bad ? 1 : 0);
  if (threadIdx.x == 0) flags[blockIdx.x] = any;
}

// Shape of k_mode_coef: waves per block (kCoefWaves, fewer when a wave would
// get under 64 terms) and term splits (grid rows): blocks up to about
// kCoefBlocks (32 per CU) while every wave keeps at least kMinTermsPerWave
// terms.  Measured (pole-sum stage, events; waves x splits) on square grids
// with the unordered table: 512^2 at t rho 1000 (132 entry blocks, 2034
// terms) 8 x 4: 16.8 us, 8 x 8: 16.1, 4 x 8: 16.0, 4 x 16: 21.0, 2 x 16:
// 21.1, 8 x 2: 19.6; 2048^2 at t rho 5000 (2060 entry blocks, 10034 terms)
// 8 x 4: 533 us, 8 x 2: 508, 8 x 1: 528, 4 x 4: 475, 4 x 8: 471, 2 x 8: 475.
constexpr int kCoefWaves = 4;
constexpr int kCoefBlocks = 8192;
constexpr int kMinTermsPerWave = 32;
// Where k_cols reads the coefficients (whole = true) the splits would be added
// for each of a thread's modes one after the other: splits only where the
// waves of the blocks leave more than half the SIMDs empty.  512^2: 8 splits,
// sums + columns 15 + 27 us, one split of 16 waves 19 + 16.
constexpr int kWholeWaves = 2048;
constexpr int kFarWaves = 4096;  // k_mode_far: waves wanted on the chip (4 per SIMD)
// Split sums of at most this many bytes are added by k_mode_apply as it reads
// them (they stay in L2); larger ones by k_mode_coef_sum first.
constexpr size_t kSplitsInApplyBytes = size_t(2) << 20;

void mode_coef_shape(int entries, int nterm, bool whole, int* nw_out, int* ns_out) {
  const int blocks = (entries + 63) / 64;
  int nw = 1, ns = 1;
  if (whole) {
    while (nw < kModeWaves && nterm >= 64 * nw) nw *= 2;
    while (ns < 64 && blocks * ns * nw < kWholeWaves && nterm >= 2 * ns * nw * kMinTermsPerWave) ns *= 2;
  } else {
    while (nw < kCoefWaves && nterm >= 128 * nw) nw *= 2;
    while (ns < 64 && blocks * ns < kCoefBlocks && nterm >= 2 * ns * nw * kMinTermsPerWave) ns *= 2;
  }
  *nw_out = nw;
  *ns_out = ns;
}

int mode_entries(int cnx, int cny, int sym) { return sym ? cnx * (cnx + 1) / 2 : cnx * cny; }

// Boxes for theta in [0, thmax] and whether they pay.  Work in units of one
// term at one theta: direct, entries x nterm; boxed, nodes x nterm for the far
// sums (32 thmax / w + the graded boxes) plus entries x (near terms of a box,
// 1.76 w / h, at kNearCost: their loads are per lane, 48 bytes a term, where
// the direct sums read the table through scalar loads) and two launches more
// (kFarLaunches); w minimises the two sums.  Measured (pole-sum stage, events;
// direct -> boxed): 2048^2, t rho 5000 (131841 entries, 10034 terms) 510 -> 76
// us, at kNearCost 1.5 88; 1501 x 1201, t rho 2000 (451351, 4034) 648 -> 68;
// 1000^2, h = 0.2, t rho 1500 (31626, 7534) 121 -> 45; 701 x 310, t rho 1000
// (27378, 2034) 34 -> 25; 512^2, t rho 1000 (8385, 2034) stays direct, 14.
// Error against long double sums (c1 theta, c2 theta^2; rms, t rho 1000):
// direct 1.5e-16, 3.0e-16, boxed 2.2e-16, 3.4e-16, beside the rounding of
// theta^2 itself (theta eps / 2 of the result, 5e-14).
constexpr double kNearCost = 3.0;
constexpr double kFarLaunches = 2.0e7;

FarBoxes far_boxes(double thmax, double h, double d, int entries, int nterm) {
  FarBoxes fb{};
  if (!(h > 0.0 && d > 0.0 && thmax > 0.0 && thmax < 1e7)) return fb;
  const double near = kFarA / h * kNearCost;
  double w = std::sqrt(kCheb * thmax * nterm / (near * entries));
  if (!(w >= 1.0)) w = 1.0;
  int k = 0;
  double tg = 4.0;
  while (tg < w) {
    tg *= 2.0;
    ++k;
  }
  const int uni = thmax > tg ? int((thmax - tg) / w) + 1 : 0;
  const int nbox = k + 1 + uni;
  const double cost = double(kCheb) * nbox * nterm + double(entries) * (near * w + 2.0 * kCheb) + kFarLaunches;
  if (cost > 0.8 * double(entries) * nterm) return fb;
  fb.w = w;
  fb.inv_w = 1.0 / w;
  fb.tg = tg;
  fb.d = d;
  fb.inv_h = 1.0 / h;
  fb.k = k;
  fb.nbox = nbox;
  return fb;
}

void far_shape(int nbox, int nterm, int* nw_out, int* ns_out) {
  const int blocks = (nbox + 1) / 2;
  int nw = 1;
  while (nw < kCoefWaves && nterm >= 128 * nw) nw *= 2;
  int ns = 1;
  while (ns < 64 && blocks * ns * nw < kFarWaves && nterm >= 2 * ns * nw * kMinTermsPerWave) ns *= 2;
  *nw_out = nw;
  *ns_out = ns;
}

size_t far_doubles2(const FarBoxes& fb, int nterm) {
  if (fb.nbox == 0) return 0;
  int nw = 1, ns = 1;
  far_shape(fb.nbox, nterm, &nw, &ns);
  return size_t(ns + 1) * fb.nbox * kCheb;
}

void launch_mode_boxed(double2* coef, double2* far, const FarBoxes& fb, int cnx, int cny, int sym, const double* sxt,
                       const double* syt, double t, double g, double H, double fc, double scale, const double* tab,
                       int nterm, hipStream_t s) {
  const int ne = mode_entries(cnx, cny, sym);
  int nw = 1, ns = 1;
  far_shape(fb.nbox, nterm, &nw, &ns);
  double2* cheb = far;
  double2* node = far + size_t(fb.nbox) * kCheb;
  const size_t lds = size_t(nw - 1) * 128 * sizeof(double);
  hipLaunchKernelGGL(k_mode_far, dim3(unsigned((fb.nbox + 1) / 2), unsigned(ns)), dim3(64 * nw), lds, s, node, fb,
                     tab, nterm);
  hipLaunchKernelGGL(k_mode_cheb, dim3(unsigned(fb.nbox)), dim3(4 * kCheb), 0, s, cheb, node, fb.nbox, ns);
  hipLaunchKernelGGL(k_mode_near, dim3(unsigned((ne + 63) / 64)), dim3(64), 0, s, coef, cheb, fb, cnx, cny, sym, sxt,
                     syt, t, g, H, fc, scale, tab, nterm);
}

bool mode_sum_in_apply(int entries, int ns) { return ns > 1 && size_t(ns) * entries * 16 <= kSplitsInApplyBytes; }

void launch_mode_coef(double2* coef, double2* part, int cnx, int cny, int sym, const double* sxt, const double* syt,
                      double t, double g, double H, double fc, double scale, const double* tab, int nterm, int nw,
                      int ns, hipStream_t s) {
  const int ne = mode_entries(cnx, cny, sym);
  const size_t lds = size_t(nw - 1) * 128 * sizeof(double);
  hipLaunchKernelGGL(k_mode_coef, dim3(unsigned((ne + 63) / 64), unsigned(ns)), dim3(64 * nw), lds, s, coef, part,
                     cnx, cny, sym, sxt, syt, t, g, H, fc, scale, tab, nterm);
  if (ns > 1 && !mode_sum_in_apply(ne, ns))
    hipLaunchKernelGGL(k_mode_coef_sum, dim3(unsigned((ne + 255) / 256)), dim3(256), 0, s, coef, part, ne, ns, scale);
}

void launch_mode_apply(double2* F, const ModeFilter& mf, hipStream_t s) {
  const long nm = long(mf.nx / 2 + 1) * mf.ny;
  hipLaunchKernelGGL(k_mode_apply, dim3(unsigned((nm + 255) / 256)), dim3(256), 0, s, F, mf);
}

int copy_check_blocks(size_t n) {
  const size_t b = (n + 255) / 256;
  return int(b < 1 ? 1 : (b > size_t(kCopyCheckMaxBlocks) ? size_t(kCopyCheckMaxBlocks) : b));
}

void launch_copy_check(const double* f, double* u, size_t n, int* flags, hipStream_t s) {
  hipLaunchKernelGGL(k_copy_check, dim3(unsigned(copy_check_blocks(n))), dim3(256), 0, s, f, u, n, flags);
}

// ---------------------------------------------------------------------------
// rocFFT plans: batch of 3 real 2D transforms, [3][ny][nx] real <->
// [3][ny][nx/2+1] complex, not in place, FP64.  Cached per (device, nx, ny)
// for the life of the process.
// ---------------------------------------------------------------------------
namespace {
struct FftPair {
  rocfft_plan fwd = nullptr, inv = nullptr;
  size_t work = 0;
};
std::mutex g_fft_mu;
std::map<std::tuple<int, int, int>, FftPair> g_fft;
bool g_fft_setup = false;

std::string fft_msg(const char* what, rocfft_status s) { return std::string(what) + " failed (rocfft status " + std::to_string(int(s)) + ")"; }
}  // namespace

rexii_status rocfft_ensure_setup() {
  std::lock_guard<std::mutex> lk(g_fft_mu);
  if (!g_fft_setup) {
    const rocfft_status s = rocfft_setup();
    if (s != rocfft_status_success) return set_error(REXII_ERR_HIP, fft_msg("rocfft_setup", s));
    g_fft_setup = true;
  }
  return REXII_OK;
}

rexii_status fft_plans(int nx, int ny, size_t* work_bytes, void** fwd, void** inv, bool create) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return set_error(REXII_ERR_HIP, "hipGetDevice failed");
  std::lock_guard<std::mutex> lk(g_fft_mu);
  if (!create) {
    const auto found = g_fft.find(std::make_tuple(dev, nx, ny));
    if (found == g_fft.end())
      return set_error(REXII_ERR_INVALID_ARG,
                       "no FFT plan for this grid on this device yet: call rexii_fourier_workspace_size "
                       "(or rexii_apply_fourier) for it first; creating a plan allocates device memory");
    if (work_bytes) *work_bytes = found->second.work;
    if (fwd) *fwd = found->second.fwd;
    if (inv) *inv = found->second.inv;
    return REXII_OK;
  }
  if (!g_fft_setup) {
    const rocfft_status s = rocfft_setup();
    if (s != rocfft_status_success) return set_error(REXII_ERR_HIP, fft_msg("rocfft_setup", s));
    g_fft_setup = true;
  }
  const auto key = std::make_tuple(dev, nx, ny);
  auto it = g_fft.find(key);
  if (it == g_fft.end()) {
    FftPair p;
    const size_t len[2] = {size_t(nx), size_t(ny)};  // fastest dimension first
    rocfft_status s = rocfft_plan_create(&p.fwd, rocfft_placement_notinplace, rocfft_transform_type_real_forward,
                                         rocfft_precision_double, 2, len, 3, nullptr);
    if (s != rocfft_status_success) return set_error(REXII_ERR_HIP, fft_msg("rocfft_plan_create (forward)", s));
    s = rocfft_plan_create(&p.inv, rocfft_placement_notinplace, rocfft_transform_type_real_inverse,
                           rocfft_precision_double, 2, len, 3, nullptr);
    if (s != rocfft_status_success) {
      rocfft_plan_destroy(p.fwd);
      return set_error(REXII_ERR_HIP, fft_msg("rocfft_plan_create (inverse)", s));
    }
    size_t w1 = 0, w2 = 0;
    rocfft_plan_get_work_buffer_size(p.fwd, &w1);
    rocfft_plan_get_work_buffer_size(p.inv, &w2);
    p.work = w1 > w2 ? w1 : w2;
    it = g_fft.emplace(key, p).first;
  }
  if (work_bytes) *work_bytes = it->second.work;
  if (fwd) *fwd = it->second.fwd;
  if (inv) *inv = it->second.inv;
  return REXII_OK;
}

// Batch of `batch` complex 2D transforms [batch][ny][nx], in place, FP64,
// forward and inverse (unnormalised); cached per (device, nx, ny, batch).
namespace {
std::map<std::tuple<int, int, int, int>, FftPair> g_fft_c2c;
}

rexii_status fft_plans_c2c(int nx, int ny, int batch, size_t* work_bytes, void** fwd, void** inv) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return set_error(REXII_ERR_HIP, "hipGetDevice failed");
  const rexii_status su = rocfft_ensure_setup();
  if (su != REXII_OK) return su;
  std::lock_guard<std::mutex> lk(g_fft_mu);
  const auto key = std::make_tuple(dev, nx, ny, batch);
  auto it = g_fft_c2c.find(key);
  if (it == g_fft_c2c.end()) {
    FftPair p;
    const size_t len[2] = {size_t(nx), size_t(ny)};
    rocfft_status s = rocfft_plan_create(&p.fwd, rocfft_placement_inplace, rocfft_transform_type_complex_forward,
                                         rocfft_precision_double, 2, len, size_t(batch), nullptr);
    if (s != rocfft_status_success) return set_error(REXII_ERR_HIP, fft_msg("rocfft_plan_create (c2c forward)", s));
    s = rocfft_plan_create(&p.inv, rocfft_placement_inplace, rocfft_transform_type_complex_inverse,
                           rocfft_precision_double, 2, len, size_t(batch), nullptr);
    if (s != rocfft_status_success) {
      rocfft_plan_destroy(p.fwd);
      return set_error(REXII_ERR_HIP, fft_msg("rocfft_plan_create (c2c inverse)", s));
    }
    size_t w1 = 0, w2 = 0;
    rocfft_plan_get_work_buffer_size(p.fwd, &w1);
    rocfft_plan_get_work_buffer_size(p.inv, &w2);
    p.work = w1 > w2 ? w1 : w2;
    it = g_fft_c2c.emplace(key, p).first;
  }
  if (work_bytes) *work_bytes = it->second.work;
  if (fwd) *fwd = it->second.fwd;
  if (inv) *inv = it->second.inv;
  return REXII_OK;
}

rexii_status fft_execute(void* plan, void* in, void* out, void* work, size_t work_bytes, hipStream_t s) {
  rocfft_execution_info info = nullptr;
  rocfft_status st = rocfft_execution_info_create(&info);
  if (st != rocfft_status_success) return set_error(REXII_ERR_HIP, fft_msg("rocfft_execution_info_create", st));
  st = rocfft_execution_info_set_stream(info, s);
  if (st == rocfft_status_success && work_bytes > 0) st = rocfft_execution_info_set_work_buffer(info, work, work_bytes);
  if (st == rocfft_status_success) {
    void* ib[1] = {in};
    void* ob[1] = {out};
    st = rocfft_execute(static_cast<rocfft_plan>(plan), ib, ob, info);
  }
  rocfft_execution_info_destroy(info);
  if (st != rocfft_status_success) return set_error(REXII_ERR_HIP, fft_msg("rocfft_execute", st));
  return REXII_OK;
}

// ---------------------------------------------------------------------------
// Static device scratch of rexii_apply_fourier_noalloc: one copy of this
// array per GPU, held until the process ends.  In host code its name is
// only a host-side stand-in; the device address comes from
// hipGetSymbolAddress (per device, with that device current) and only that
// address is handed to kernels and library calls.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[REXII_STATIC_SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mu;
std::map<int, void*> g_scratch;  // device -> address of its copy of scratch
}  // namespace

rexii_status static_scratch(void** ptr) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return set_error(REXII_ERR_HIP, "hipGetDevice failed");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  auto it = g_scratch.find(dev);
  if (it == g_scratch.end()) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
      return set_error(REXII_ERR_HIP, std::string("hipGetSymbolAddress(scratch) failed: ") + hipGetErrorString(e));
    if (reinterpret_cast<uintptr_t>(p) & 255)
      return set_error(REXII_ERR_HIP, "static scratch is not 256-byte aligned");
    it = g_scratch.emplace(dev, p).first;
  }
  *ptr = it->second;
  return REXII_OK;
}

}  // namespace rexii

// built with this file: one translation unit
#include "kernels_fft2d.hip"
