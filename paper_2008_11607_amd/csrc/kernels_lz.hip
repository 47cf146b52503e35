// Shared-Krylov (multi-shift) REXII: every shifted system of the pole sum
// is (tA - z_k I) x_k = f with the same right-hand side, and Krylov spaces
// are shift invariant, K_m(tA - z I, f) = K_m(A, f).  One Lanczos process
// therefore serves all poles:
//   A V_m = V_m T_m + beta_m v_{m+1} e_m^T,
//   r(tA) f ~ ||f||_W V_m Re sum_k w_k (t T_m - z_k I)^{-1} e_1.
// With W = diag(g, H, H) the operator (any depth field, flux form) satisfies
// W A = -(W A)^T, so A is skew-adjoint in <x, y>_W = x^T W y: the Lanczos
// recurrence has no diagonal term and is real,
//   w_j = A v_j + beta_{j-1} v_{j-1},  beta_j = ||w_j||_W,  v_{j+1} = w_j / beta_j,
// and T_m is real skew-tridiagonal (T[j+1][j] = beta_j = -T[j][j+1]).
//
// Pass 1 yields beta_1..beta_m and keeps as many of the vectors as the
// workspace holds; the small problems are solved on the GPU (k_lz_small);
// pass 2 is u = sum_j y_j v_j over the kept vectors (k_lz_gather, 24 bytes a
// point and vector) and, for the others, the same steps once more with
// u += y_j v_j (128 bytes a point and step).  Every step twice and the small
// problem on the host took 44.1 ms at 512^2, t rho = 1000 (17.3 ms now) and
// 27.1 ms for the 2048^2 depth field at t rho = 100 (13.3 ms now, the sum of
// 160 vectors 2.8 ms at 5.8 TB/s).  The reductions are in a fixed
// order, so repeated steps reproduce pass 1 bit for bit.
//
// Storage: the vectors are kept unnormalised, buf_j = beta_{j-1} v_j
// (buf_1 = f, beta_0 = ||f||_W); step j reads buf_j and buf_{j-1} and writes
// w_j = buf_{j+1}, to a place of its own or over buf_{j-1}.
#include <hip/hip_runtime.h>

#include "kernels_lz.h"
#include "device_util.h"

namespace rexii {

constexpr int kLzTX = 64;   // tile columns (one per lane)
constexpr int kLzRows = 8;  // rows per thread (a sliding window of three rows)
constexpr int kLzNT = 256;  // threads: 64 x 4
constexpr int kLzTY = kLzRows * (kLzNT / kLzTX);  // 32 rows per tile

__device__ __forceinline__ double block_sum_lz(double v, double* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < kLzNT / 64; ++k) s += sh[k];
  return s;  // valid in thread 0
}

// One Lanczos step for every state r (blockIdx.y) of the batch.
//   cur = buf_j, prev = buf_{j-1}, out = w_j (may be prev); states lie
//   stride doubles apart.
//   beta[r * ldb + j - 1] = beta_{j-1} (beta_0 = ||f||_W), beta[.. + j - 2].
//   j == 1: no prev term (prev is not read).
//   part[r * nblk + block] = this block's sum of g w_eta^2 + H (w_u^2 + w_v^2)
//     (skipped when part == nullptr).
//   y != nullptr (pass 2): u += (y[r * ldy + j - 1] / beta_{j-1}) buf_j.
//   last: pass 2's final step (w_m is not needed: nothing is written).
__global__ __launch_bounds__(kLzNT) void k_lz_step(const double* __restrict__ cur, const double* prev, double* out,
                                                   size_t stride, const double* __restrict__ H, double H0, double g,
                                                   double fc,
                                                   int nx, int ny, int j, const double* __restrict__ beta, int ldb,
                                                   double* __restrict__ part, const double* __restrict__ y, int ldy,
                                                   double* __restrict__ u, int last) {
  __shared__ double sh[kLzNT / 64];
  const int r = blockIdx.y;
  const size_t n = size_t(nx) * ny;
  const double* c = cur + size_t(r) * stride;
  const double* pv = prev + size_t(r) * stride;
  double* ov = out + size_t(r) * stride;
  const double* br = beta + size_t(r) * ldb;
  const double sc = 1.0 / br[j - 1];                                  // v_j = sc * buf_j
  const double sp = (j >= 2) ? br[j - 1] / br[j - 2] : 0.0;          // beta_{j-1} v_{j-1} = sp * buf_{j-1}
  const double yv = y ? y[size_t(r) * ldy + j - 1] : 0.0;
  const double yc = (yv != 0.0) ? yv * sc : 0.0;  // a zero state has beta_0 = 0 and y = 0
  double* ur = u ? u + size_t(r) * 3 * n : nullptr;
  const int tiles_x = (nx + kLzTX - 1) / kLzTX;
  const int i = (blockIdx.x % tiles_x) * kLzTX + (threadIdx.x & 63);
  const int j0 = (blockIdx.x / tiles_x) * kLzTY + (threadIdx.x >> 6) * kLzRows;
  const double hx = 0.5 * nx, hy = 0.5 * ny;
  double acc = 0.0;
  if (i < nx && j0 < ny) {
    const int ie = (i + 1 == nx) ? 0 : i + 1, iw = (i == 0) ? nx - 1 : i - 1;
    const double* ce = c;
    const double* cu = c + n;
    const double* cv = c + 2 * n;
    // rows jj - 1, jj, jj + 1 of eta, v and the depth in registers: each
    // row is loaded once per thread and slides down the window
    auto row = [&](int jj) { return size_t(jj < 0 ? jj + ny : (jj >= ny ? jj - ny : jj)) * nx + i; };
    const size_t q0 = row(j0 - 1), q1 = row(j0);
    double eS = ce[q0], eC = ce[q1], vS = cv[q0], vC = cv[q1];
    double HS = H ? H[q0] : H0, HC = H ? H[q1] : H0;
    for (int k = 0; k < kLzRows; ++k) {
      const int jj = j0 + k;
      if (jj >= ny) break;
      const size_t p = size_t(jj) * nx + i, qn = row(jj + 1);
      const size_t pe = size_t(jj) * nx + ie, pw = size_t(jj) * nx + iw;
      const double eN = ce[qn], vN = cv[qn], HN = H ? H[qn] : H0;
      const double He = H ? H[pe] : H0, Hw = H ? H[pw] : H0;
      const double b0 = eC, b1 = cu[p], b2 = vC;
      // A buf_j (flux form, centred differences)
      const double ae = -(hx * (He * cu[pe] - Hw * cu[pw]) + hy * (HN * vN - HS * vS));
      const double au = -g * hx * (ce[pe] - ce[pw]) + fc * b2;
      const double av = -g * hy * (eN - eS) - fc * b1;
      if (ur && yc != 0.0) {  // y_j = 0 beyond a state's own Krylov dimension
        ur[p] += yc * b0;
        ur[n + p] += yc * b1;
        ur[2 * n + p] += yc * b2;
      }
      if (!last) {
        double w0 = sc * ae, w1 = sc * au, w2 = sc * av;
        if (j >= 2) {
          w0 += sp * pv[p];
          w1 += sp * pv[n + p];
          w2 += sp * pv[2 * n + p];
        }
        ov[p] = w0;
        ov[n + p] = w1;
        ov[2 * n + p] = w2;
        acc += g * w0 * w0 + HC * (w1 * w1 + w2 * w2);
      }
      eS = eC;
      eC = eN;
      vS = vC;
      vC = vN;
      HS = HC;
      HC = HN;
    }
  }
  if (!part) return;
  const double s = block_sum_lz(acc, sh);
  if (threadIdx.x == 0) part[size_t(r) * gridDim.x + blockIdx.x] = s;
}

// ||f||_W partial sums of each state (for beta_0), and buf_1 = f.
__global__ __launch_bounds__(kLzNT) void k_lz_start(const double* __restrict__ f, double* __restrict__ buf,
                                                    size_t stride, const double* __restrict__ H, double H0, double g, int nx,
                                                    int ny, double* __restrict__ part, int* __restrict__ flag) {
  __shared__ double sh[kLzNT / 64];
  const int r = blockIdx.y;
  const size_t n = size_t(nx) * ny;
  const double* fr = f + size_t(r) * 3 * n;
  double* br = buf + size_t(r) * stride;
  const int tiles_x = (nx + kLzTX - 1) / kLzTX;
  const int i = (blockIdx.x % tiles_x) * kLzTX + (threadIdx.x & 63);
  const int j0 = (blockIdx.x / tiles_x) * kLzTY + (threadIdx.x >> 6) * kLzRows;
  double acc = 0.0;
  bool bad = false;
  if (i < nx) {
    for (int k = 0; k < kLzRows; ++k) {
      const int jj = j0 + k;
      if (jj >= ny) break;
      const size_t p = size_t(jj) * nx + i;
      const double a = fr[p], b = fr[n + p], c = fr[2 * n + p];
      br[p] = a;
      br[n + p] = b;
      br[2 * n + p] = c;
      const double Hp = H ? H[p] : H0;
      acc += g * a * a + Hp * (b * b + c * c);
      bad = bad || !isfinite(a) || !isfinite(b) || !isfinite(c);
    }
  }
  if (bad) atomicOr(flag, 1);
  const double s = block_sum_lz(acc, sh);
  if (threadIdx.x == 0) part[size_t(r) * gridDim.x + blockIdx.x] = s;
}

// beta[r * ldb + slot] = sqrt(sum of part[r][0..nblk)) in a fixed order
// (one block per state).
__global__ __launch_bounds__(kLzNT) void k_lz_norm(const double* __restrict__ part, int nblk,
                                                   double* __restrict__ beta, int ldb, int slot) {
  __shared__ double sh[kLzNT / 64];
  const int r = blockIdx.x;
  double s = 0.0;
  for (int k = threadIdx.x; k < nblk; k += kLzNT) s += part[size_t(r) * nblk + k];
  s = block_sum_lz(s, sh);
  if (threadIdx.x == 0) beta[size_t(r) * ldb + slot] = sqrt(s);
}

// u = sum_j coef[j] buf_{j+1}, j < m, the vectors n3 doubles apart: memory
// bound, eight vectors' loads in flight per thread, added in order.
template <typename V>
__global__ __launch_bounds__(256) void k_lz_gather(const double* __restrict__ vecs, size_t n3, int m,
                                                   const double* __restrict__ coef, double* __restrict__ u) {
  constexpr int kW = sizeof(V) / 8, kU = 8;
  const size_t i = (size_t(blockIdx.x) * 256 + threadIdx.x) * kW;
  if (i >= n3) return;
  double acc[kW];
#pragma unroll
  for (int w = 0; w < kW; ++w) acc[w] = 0.0;
  auto add = [&](V v, double c) {
    const double* d = reinterpret_cast<const double*>(&v);
#pragma unroll
    for (int w = 0; w < kW; ++w) acc[w] += c * d[w];
  };
  int j = 0;
  for (; j + kU <= m; j += kU) {
    V v[kU];
#pragma unroll
    for (int k = 0; k < kU; ++k) v[k] = *reinterpret_cast<const V*>(vecs + size_t(j + k) * n3 + i);
#pragma unroll
    for (int k = 0; k < kU; ++k) add(v[k], coef[j + k]);
  }
  for (; j < m; ++j) add(*reinterpret_cast<const V*>(vecs + size_t(j) * n3 + i), coef[j]);
#pragma unroll
  for (int w = 0; w < kW; ++w) u[i + w] = acc[w];
}

// The small problem: y = beta_0 Re sum_k w_k (t T - z_k I)^{-1} e_1 for the
// m x m skew tridiagonal T (T[j+1][j] = b[j] = -T[j][j+1], 1-based).  One lane
// per conjugate pair of poles (z_2 = -conj(z_1): with D = diag((-1)^(j-1)),
// D T D = -T, so (tT - z_2)^{-1} e_1 = -D conj((tT - z_1)^{-1} e_1)).
// Elimination from the last row up needs no pivoting (the Hermitian part of
// tT - z is -Re(z) I) and leaves a one-term recurrence for x:
//   delta_m = -z, delta_j = -z + (t b_j)^2 / delta_{j+1},
//   x_1 = 1 / delta_1, x_{j+1} = -t b_j x_j / delta_{j+1}.
// Bound: the serial chain of one reciprocal a row (about 130 cycles): 1184
// rows and 2062 pairs take 0.2 ms here and took 3.5 ms on 16 host threads.
// part[block][j] = the block's sum over its 64 pairs.
constexpr int kSmU = 8;   // rows whose loads are in flight together
__global__ __launch_bounds__(64) void k_lz_small(const double* __restrict__ b, int m, double t,
                                                 const LzPair* __restrict__ pairs, int npair, double2* inv,
                                                 double* __restrict__ part) {
  const int lane = threadIdx.x;
  const int q = blockIdx.x * 64 + lane;
  LzPair pr;
  pr.z = make_double2(1.0, 0.0);
  pr.w1 = pr.w2 = make_double2(0.0, 0.0);
  if (q < npair) pr = pairs[q];
  double2* iv = inv + size_t(blockIdx.x) * 64 * m + lane;   // row j at iv[64 (j - 1)]
  double2 dl = make_double2(-pr.z.x, -pr.z.y), x = make_double2(0.0, 0.0);
  auto recip = [&](double2 v) {
    const double r = 1.0 / (v.x * v.x + v.y * v.y);
    return make_double2(v.x * r, -v.y * r);
  };
  x = recip(dl);
  iv[size_t(64) * (m - 1)] = x;
  for (int j1 = m - 1; j1 >= 1; j1 -= kSmU) {
    double bb[kSmU];
#pragma unroll
    for (int k = 0; k < kSmU; ++k) bb[k] = b[j1 - k > 1 ? j1 - k : 1];
#pragma unroll
    for (int k = 0; k < kSmU; ++k) {
      const int j = j1 - k;
      if (j < 1) break;
      const double s = t * bb[k], s2 = s * s;
      dl = make_double2(s2 * x.x - pr.z.x, s2 * x.y - pr.z.y);
      x = recip(dl);
      iv[size_t(64) * (j - 1)] = x;
    }
  }
  // x holds 1 / delta_1; odd and even rows (1-based) take the second pole's
  // term with opposite signs
  const double c1r = pr.w1.x - pr.w2.x, c1i = -pr.w1.y - pr.w2.y;
  const double c2r = pr.w1.x + pr.w2.x, c2i = pr.w2.y - pr.w1.y;
  double* pp = part + size_t(blockIdx.x) * m;
  for (int j0 = 1; j0 <= m; j0 += kSmU) {
    double2 id[kSmU];
    double bb[kSmU];
#pragma unroll
    for (int k = 0; k < kSmU; ++k) {
      const int j = j0 + k + 1 <= m ? j0 + k + 1 : m;   // row after j0 + k
      id[k] = iv[size_t(64) * (j - 1)];
      bb[k] = b[j - 1];
    }
#pragma unroll
    for (int k = 0; k < kSmU; ++k) {
      const int j = j0 + k;
      if (j > m) break;
      const double v = ((k & 1) == 0) ? c1r * x.x + c1i * x.y : c2r * x.x + c2i * x.y;   // j0 is odd
      const double s = wave_total63(v);
      if (lane == 63) pp[j - 1] = s;
      const double sub = -t * bb[k];
      x = make_double2(sub * (x.x * id[k].x - x.y * id[k].y), sub * (x.x * id[k].y + x.y * id[k].x));
    }
  }
}

// y_j = b_0 sum of the blocks' parts; coef_j = y_j / b_{j-1} (y also as the
// weights of repeated steps); out = (|y|^2, |last 8 of y|^2).
__global__ __launch_bounds__(1024) void k_lz_ysum(const double* __restrict__ part, int nblk, int m,
                                                  const double* __restrict__ b, double* __restrict__ y,
                                                  double* __restrict__ coef, double* __restrict__ out) {
  __shared__ double sh[32];
  double tot = 0.0, tail = 0.0;
  for (int j = threadIdx.x; j < m; j += 1024) {
    double s = 0.0;
    for (int k = 0; k < nblk; ++k) s += part[size_t(k) * m + j];
    s *= b[0];
    y[j] = s;
    coef[j] = s / b[j];
    tot += s * s;
    if (j >= m - 8) tail += s * s;
  }
  tot = wave_total63(tot);
  tail = wave_total63(tail);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) {
    sh[w] = tot;
    sh[16 + w] = tail;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, c = 0.0;
    for (int k = 0; k < 16; ++k) {
      a += sh[k];
      c += sh[16 + k];
    }
    out[0] = a;
    out[1] = c;
  }
}

int lz_blocks(int nx, int ny) { return ((nx + kLzTX - 1) / kLzTX) * ((ny + kLzTY - 1) / kLzTY); }

void launch_lz_start(const double* f, double* buf, size_t stride, const double* H, double H0, double g, int nx, int ny,
                     int nrhs, double* part, int* flag, double* beta, int ldb, hipStream_t s) {
  const int nb = lz_blocks(nx, ny);
  hipLaunchKernelGGL(k_lz_start, dim3(nb, nrhs), dim3(kLzNT), 0, s, f, buf, stride, H, H0, g, nx, ny, part, flag);
  hipLaunchKernelGGL(k_lz_norm, dim3(nrhs), dim3(kLzNT), 0, s, part, nb, beta, ldb, 0);
}

void launch_lz_step(const double* cur, const double* prev, double* out, size_t stride, const double* H, double H0,
                    double g, double fc, int nx, int ny, int nrhs, int j, double* beta, int ldb, double* part,
                    const double* y, int ldy, double* u, int last, hipStream_t s) {
  const int nb = lz_blocks(nx, ny);
  hipLaunchKernelGGL(k_lz_step, dim3(nb, nrhs), dim3(kLzNT), 0, s, cur, prev, out, stride, H, H0, g, fc, nx, ny, j,
                     beta, ldb, part, y, ldy, u, last);
  if (part) hipLaunchKernelGGL(k_lz_norm, dim3(nrhs), dim3(kLzNT), 0, s, part, nb, beta, ldb, j);
}

void launch_lz_gather(const double* vecs, size_t n3, int m, const double* coef, double* u, hipStream_t s) {
  // pairs of doubles where every vector starts on a 16-byte boundary
  const bool two = (n3 % 2 == 0) && ((reinterpret_cast<uintptr_t>(vecs) | reinterpret_cast<uintptr_t>(u)) % 16 == 0);
  const size_t items = two ? n3 / 2 : n3;
  const dim3 grid(unsigned((items + 255) / 256));
  if (two)
    hipLaunchKernelGGL(k_lz_gather<double2>, grid, dim3(256), 0, s, vecs, n3, m, coef, u);
  else
    hipLaunchKernelGGL(k_lz_gather<double>, grid, dim3(256), 0, s, vecs, n3, m, coef, u);
}

size_t lz_small_bytes(int m, int npair) {
  const size_t nb = (size_t(npair) + 63) / 64;
  return nb * 64 * m * sizeof(double2) + nb * m * sizeof(double) + 512;
}
void launch_lz_small(const double* b, int m, double t, const LzPair* pairs, int npair, void* scratch, double* y,
                     double* coef, double* out, hipStream_t s) {
  const int nb = (npair + 63) / 64;
  double2* inv = static_cast<double2*>(scratch);
  double* part = reinterpret_cast<double*>(inv + size_t(nb) * 64 * m);
  hipLaunchKernelGGL(k_lz_small, dim3(nb), dim3(64), 0, s, b, m, t, pairs, npair, inv, part);
  hipLaunchKernelGGL(k_lz_ysum, dim3(1), dim3(1024), 0, s, part, nb, m, b, y, coef, out);
}

}  // namespace rexii
