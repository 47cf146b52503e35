// Two-dimensional real transforms of the Fourier path, three launches for
// the whole of "transform, filter, transform back":
//   k_rows_fwd  two real rows as one complex FFT along x, written transposed:
//               G[kx][field][y] (kx <= nx/2); checks the input on the way;
//   k_cols      one kx, the three fields: FFT along y, the filter of every
//               mode, inverse FFT along y, in place;
//   k_rows_inv  the inverse of k_rows_fwd.
// So a state is read once and written once and its spectrum moves twice in
// either direction; the filter needs all three fields of a mode, which the
// column's thread holds in registers.
//
// One FFT of M = 2^m points is worked by M/8 threads, eight points each:
// radix-8 steps in registers with exchanges through LDS between them (index
// padded by one in eight: every step's accesses are spread over the banks).
// Forward runs by decimation in frequency, natural order in (thread t holds
// t + i M/8), digit-reversed positions 8 t + i out; inverse the other way
// round, so neither order is ever sorted.  A length n that is no power of two
// is a convolution with the chirp exp(i pi j^2 / n) of M >= 2 n - 1 points
// (Bluestein 1970): forward, times the chirp's transform, inverse.
//
// What bounds them: at 2048^2 (rows 64 us, columns 77, rows 46; rocFFT, the
// copy and a filter pass took 36 + 148 + 38 + 146) memory, 200 MB a launch,
// and the few waves a CU holds beside 36 KB buffers; for chirp lengths LDS
// and latency (M = 4096: eight steps of 128 KB in and out a row; 1501 x 1201:
// 76, 135 and 64 us against 618 + 20 + 626 of rocFFT); at 512^2 and below the
// chain of the column's steps (9, 15, 6 us at 512^2).  Accuracy: as rocFFT's to
// a few eps (a chirp length passes two transforms).
#include <hip/hip_runtime.h>

#include <cmath>
#include <vector>

#include "kernels_fft.h"
#include "mode_filter.h"

namespace rexii {

namespace {

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 conj2(double2 a) { return make_double2(a.x, -a.y); }
// S i a
template <int S>
__device__ __forceinline__ double2 rot(double2 a) {
  return S > 0 ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// X_q = sum_j x_j exp(S 2 pi i j q / 4), in place
template <int S>
__device__ __forceinline__ void dft4(double2& a, double2& b, double2& c, double2& d) {
  const double2 s0 = cadd(a, c), s1 = csub(a, c), t0 = cadd(b, d), t1 = rot<S>(csub(b, d));
  a = cadd(s0, t0);
  b = cadd(s1, t1);
  c = csub(s0, t0);
  d = csub(s1, t1);
}

template <int S>
__device__ __forceinline__ void dft8(double2 (&v)[8]) {
  constexpr double h = 0.70710678118654752440;
  double2 a0 = cadd(v[0], v[4]), a1 = cadd(v[1], v[5]), a2 = cadd(v[2], v[6]), a3 = cadd(v[3], v[7]);
  double2 b0 = csub(v[0], v[4]), b1 = csub(v[1], v[5]), b2 = csub(v[2], v[6]), b3 = csub(v[3], v[7]);
  const double2 r1 = rot<S>(b1), r3 = rot<S>(b3);
  b1 = make_double2(h * (b1.x + r1.x), h * (b1.y + r1.y));  // times exp(S i pi / 4)
  b2 = rot<S>(b2);
  b3 = make_double2(h * (r3.x - b3.x), h * (r3.y - b3.y));  // times exp(S 3 i pi / 4)
  dft4<S>(a0, a1, a2, a3);
  dft4<S>(b0, b1, b2, b3);
  v[0] = a0;
  v[1] = b0;
  v[2] = a1;
  v[3] = b1;
  v[4] = a2;
  v[5] = b2;
  v[6] = a3;
  v[7] = b3;
}

// the last step of 2, 4 or 8 points on the thread's eight positions
template <int S>
__device__ __forceinline__ void dft_last(double2 (&v)[8], int l) {
  if (l == 3) {
    dft8<S>(v);
  } else if (l == 2) {
    dft4<S>(v[0], v[1], v[2], v[3]);
    dft4<S>(v[4], v[5], v[6], v[7]);
  } else {
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
      const double2 a = cadd(v[i], v[i + 1]), b = csub(v[i], v[i + 1]);
      v[i] = a;
      v[i + 1] = b;
    }
  }
}

__device__ __forceinline__ int pad(int i) { return i + (i >> 3); }

// v[q] *= w_L^(j q) (conjugated for S > 0) from the step's table w_L^j,
// w_L^2j, w_L^4j (h = L/8 entries of each: the lanes' loads are contiguous;
// strided loads from one table of w_M cost as much as the LDS exchange); the
// other powers are products.
template <int S>
__device__ __forceinline__ void twiddle(double2 (&v)[8], const double2* __restrict__ tw, int h, int j) {
  double2 w1 = tw[j], w2 = tw[h + j], w4 = tw[2 * h + j];
  if (S > 0) {
    w1 = conj2(w1);
    w2 = conj2(w2);
    w4 = conj2(w4);
  }
  const double2 w3 = cmul(w1, w2), w5 = cmul(w1, w4), w6 = cmul(w2, w4);
  v[1] = cmul(v[1], w1);
  v[2] = cmul(v[2], w2);
  v[3] = cmul(v[3], w3);
  v[4] = cmul(v[4], w4);
  v[5] = cmul(v[5], w5);
  v[6] = cmul(v[6], w6);
  v[7] = cmul(v[7], cmul(w3, w4));
}

// Forward transform: v natural (t + q M/8) in, positions 8 t + q out.  The
// caller's LDS writes before it must be behind a barrier if they are not the
// thread's own natural entries; after it the thread has read its own
// positions last.
__device__ __forceinline__ void fft_dif(double2 (&v)[8], double2* buf, int t, int lm, const double2* __restrict__ tw) {
  int l = lm;
  for (; l > 3; l -= 3) {
    const int l8 = l - 3, j = t & ((1 << l8) - 1), base = ((t >> l8) << l) + j;
    if (l < lm) {
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = buf[pad(base + (q << l8))];
    }
    dft8<-1>(v);
    twiddle<-1>(v, tw, 1 << l8, j);
    tw += 3 << l8;
#pragma unroll
    for (int q = 0; q < 8; ++q) buf[pad(base + (q << l8))] = v[q];
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = buf[pad(8 * t + q)];
  dft_last<-1>(v, l);
}

// Inverse (unscaled): positions 8 t + q in, natural t + q M/8 out, which the
// thread has read last.
__device__ __forceinline__ void fft_dit(double2 (&v)[8], double2* buf, int t, int lm, const double2* __restrict__ tw) {
  int l = lm - 3 * ((lm - 1) / 3);
  tw += 3 * (((1 << lm) - (1 << l)) / 7);   // the steps' tables, last step first
  dft_last<1>(v, l);
#pragma unroll
  for (int q = 0; q < 8; ++q) buf[pad(8 * t + q)] = v[q];
  __syncthreads();
  for (l += 3; l <= lm; l += 3) {
    const int l8 = l - 3, j = t & ((1 << l8) - 1), base = ((t >> l8) << l) + j;
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = buf[pad(base + (q << l8))];
    tw -= 3 << l8;
    twiddle<1>(v, tw, 1 << l8, j);
    dft8<1>(v);
    if (l < lm) {
#pragma unroll
      for (int q = 0; q < 8; ++q) buf[pad(base + (q << l8))] = v[q];
      __syncthreads();
    }
  }
}

// frequency at position p, and position of frequency k
__device__ __forceinline__ int freq_at(int p, int lm) {
  int k = 0, s = 0, l = lm;
  for (; l > 3; l -= 3) {
    k += (p >> (l - 3)) << s;
    p &= (1 << (l - 3)) - 1;
    s += 3;
  }
  return k + (p << s);
}
__device__ __forceinline__ int pos_of(int k, int lm) {
  int p = 0, l = lm;
  for (; l > 3; l -= 3) {
    p += (k & 7) << (l - 3);
    k >>= 3;
  }
  return p + k;
}

// The chirp convolution of v (already times the chirp, zero from n on):
// natural in, natural out.
__device__ __forceinline__ void convolve(double2 (&v)[8], double2* buf, int t, const FftAxis& ax) {
  fft_dif(v, buf, t, ax.lm, ax.tw);
  const int tpf = 1 << (ax.lm - 3);
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = cmul(v[q], ax.bhat[q * tpf + t]);
  fft_dit(v, buf, t, ax.lm, ax.tw);
}

// Blocks are handed to the 8 XCDs in turn; four neighbouring row pairs share
// the 128-byte lines of G they write and read, so each run of 32 blocks gives
// four neighbours to every XCD and its L2 holds the line for all four.
__device__ __forceinline__ int neighbour_block(int b, int nb) {
  const int g = b & ~31;
  if (g + 32 > nb) return b;
  return g + (b & 7) * 4 + ((b >> 3) & 3);
}

}  // namespace

template <bool BLU>
__global__ __launch_bounds__(1024) void k_rows_fwd(const double* __restrict__ f, double2* __restrict__ G, FftAxis ax,
                                                  int ny, int first, int npairs, int* __restrict__ flags) {
  extern __shared__ double2 lds[];
  const int n = ax.n, tpf = 1 << (ax.lm - 3);
  const int t = int(threadIdx.x) & (tpf - 1), sub = int(threadIdx.x) >> (ax.lm - 3);
  double2* buf = lds + size_t(sub) * (9 * tpf);
  const int blk = neighbour_block(int(blockIdx.x), int(gridDim.x));
  const int pr = blk * (int(blockDim.x) >> (ax.lm - 3)) + sub;
  const bool live = pr < npairs;
  const int npy = (ny + 1) / 2, pair = first + pr;
  const int fld = live ? pair / npy : 0, y0 = live ? 2 * (pair % npy) : 0;
  const bool two = live && y0 + 1 < ny;
  const double* ra = f + (size_t(fld) * ny + y0) * n;
  const double* rb = ra + n;
  double2 v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int j = t + i * tpf;
    v[i] = make_double2(live && j < n ? ra[j] : 0.0, two && j < n ? rb[j] : 0.0);
  }
  bool bad = false;
#pragma unroll
  for (int i = 0; i < 8; ++i) bad = bad || !isfinite(v[i].x) || !isfinite(v[i].y);
  if (BLU) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = t + i * tpf;
      if (j < n) v[i] = cmul(v[i], ax.chirp[j]);
    }
    convolve(v, buf, t, ax);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = t + i * tpf;
      if (j < n) buf[pad(j)] = cmul(v[i], ax.chirp[j]);
    }
  } else {
    fft_dif(v, buf, t, ax.lm, ax.tw);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) buf[pad(freq_at(8 * t + i, ax.lm))] = v[i];
  }
  const int any = __syncthreads_or(bad ? 1 : 0);
  if (threadIdx.x == 0) flags[blk] = any;
  // The two rows' spectra from Z = A + i B: A = (Z(k) + conj Z(-k)) / 2,
  // B = (Z(k) - conj Z(-k)) / 2i.  Rows run fastest over the threads: the
  // block's rows of one k are neighbours in G.
  const int fpb = int(blockDim.x) >> (ax.lm - 3), lr = 31 - __clz(2 * fpb), rows = 1 << lr;
  const int yy = int(threadIdx.x) & (rows - 1), ks = int(blockDim.x) >> lr;
  const int wp = blk * fpb + (yy >> 1);
  if (wp >= npairs) return;
  const int of = (first + wp) / npy, oy = 2 * ((first + wp) % npy) + (yy & 1);
  if (oy >= ny) return;
  const double2* zb = lds + size_t(yy >> 1) * (9 * tpf);
  for (int k = int(threadIdx.x) >> lr; k <= n / 2; k += ks) {
    const double2 z = zb[pad(k)], y = zb[pad(k ? n - k : 0)];
    const double2 a = make_double2(0.5 * (z.x + y.x), 0.5 * (z.y - y.y));
    const double2 c = make_double2(0.5 * (z.y + y.y), 0.5 * (y.x - z.x));
    G[(size_t(k) * 3 + of) * ny + oy] = make_double2((yy & 1) ? c.x : a.x, (yy & 1) ? c.y : a.y);
  }
}

__device__ __forceinline__ void reduce_flags(const int* __restrict__ flags, int nflags, int* __restrict__ word) {
  int any = 0;
  for (int b = int(threadIdx.x); b < nflags; b += int(blockDim.x)) any |= flags[b];
  any = __syncthreads_or(any);
  if (threadIdx.x == 0) *word = any;
}

// One column a block, one exchange buffer, the fields in turn; the spectra of
// the three fields wait in registers (powers of two: 8 points a thread) or,
// for a chirp, in G itself, each thread's own entries (in registers they
// cost the second block on the CU: 169 against 100 VGPRs).
// word: 1 if any of the nflags words of k_rows_fwd is set, else 0.
__global__ __launch_bounds__(512, 3) void k_cols(double2* __restrict__ G, FftAxis ax, ModeFilter mf,
                                              const int* __restrict__ flags, int nflags, int* __restrict__ word) {
  extern __shared__ double2 lds[];
  const int n = ax.n, tpf = 1 << (ax.lm - 3), t = int(threadIdx.x), col = int(blockIdx.x);
  double2* g = G + size_t(col) * 3 * n;
  double2 r[3][8];
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int i = 0; i < 8; ++i) r[q][i] = g[size_t(q) * n + t + i * tpf];
  if (blockIdx.x == 0) reduce_flags(flags, nflags, word);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (q > 0) __syncthreads();
    double2 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = r[q][i];
    fft_dif(v, lds, t, ax.lm, ax.tw);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[q][i] = v[i];
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    // always true; as a branch it keeps the eight modes apart, which at once
    // do not fit the registers
    const int ky = freq_at(8 * t + i, ax.lm);
    if (ky < n) {
      double2 m[3] = {r[0][i], r[1][i], r[2][i]};
      mode_filter(mf, col, ky, m);
      r[0][i] = m[0];
      r[1][i] = m[1];
      r[2][i] = m[2];
    }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (q > 0) __syncthreads();
    double2 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = r[q][i];
    fft_dit(v, lds, t, ax.lm, ax.tw);
#pragma unroll
    for (int i = 0; i < 8; ++i) g[size_t(q) * n + t + i * tpf] = v[i];
  }
}

__global__ __launch_bounds__(512, 4) void k_cols_chirp(double2* __restrict__ G, FftAxis ax, ModeFilter mf,
                                                       const int* __restrict__ flags, int nflags,
                                                       int* __restrict__ word) {
  extern __shared__ double2 lds[];
  constexpr int RN = 4;   // n <= M/2
  const int n = ax.n, tpf = 1 << (ax.lm - 3), t = int(threadIdx.x), col = int(blockIdx.x);
  double2* g = G + size_t(col) * 3 * n;
  if (blockIdx.x == 0) reduce_flags(flags, nflags, word);
  double2 v[8];
  // S = -1: the transform; 1: the inverse as the conjugate of the transform of the conjugate
  auto transform = [&](int q, bool inverse) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = t + i * tpf;
      v[i] = make_double2(0.0, 0.0);
      if (i < RN && j < n) {
        double2 x = g[size_t(q) * n + j];
        if (inverse) x.y = -x.y;
        v[i] = cmul(x, ax.chirp[j]);
      }
    }
    convolve(v, lds, t, ax);
#pragma unroll
    for (int i = 0; i < RN; ++i) {
      const int j = t + i * tpf;
      if (j < n) {
        double2 x = cmul(v[i], ax.chirp[j]);
        if (inverse) x.y = -x.y;
        g[size_t(q) * n + j] = x;
      }
    }
  };
  for (int q = 0; q < 3; ++q) transform(q, false);
  for (int i = 0; i < RN; ++i) {
    const int j = t + i * tpf;
    if (j < n) {
      double2 m[3] = {g[j], g[size_t(n) + j], g[size_t(2) * n + j]};
      mode_filter(mf, col, j, m);
      g[j] = m[0];
      g[size_t(n) + j] = m[1];
      g[size_t(2) * n + j] = m[2];
    }
  }
  for (int q = 0; q < 3; ++q) transform(q, true);
}

// k_cols with a group of M/8 threads and an exchange buffer for each field:
// a third of the chain of transforms, three times the waves.
template <bool BLU>
__global__ __launch_bounds__(768) void k_cols3(double2* __restrict__ G, FftAxis ax, int nxh, ModeFilter mf,
                                               const int* __restrict__ flags, int nflags, int* __restrict__ word) {
  extern __shared__ double2 lds[];
  const int n = ax.n, tpf = 1 << (ax.lm - 3);
  const int t = int(threadIdx.x) & (tpf - 1), slot = int(threadIdx.x) >> (ax.lm - 3);
  const int q = slot % 3, cpb = int(blockDim.x) / (3 * tpf);
  const int col = int(blockIdx.x) * cpb + slot / 3;
  const bool live = col < nxh;
  double2* buf = lds + size_t(slot) * (9 * tpf);
  double2* g = G + (size_t(live ? col : 0) * 3 + q) * n;
  double2 v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int j = t + i * tpf;
    v[i] = j < n ? g[j] : make_double2(0.0, 0.0);
  }
  if (blockIdx.x == 0) reduce_flags(flags, nflags, word);
  if (BLU) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = t + i * tpf;
      if (j < n) v[i] = cmul(v[i], ax.chirp[j]);
    }
    convolve(v, buf, t, ax);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = t + i * tpf;
      if (j < n) v[i] = cmul(v[i], ax.chirp[j]);
    }
  } else {
    fft_dif(v, buf, t, ax.lm, ax.tw);
  }
  // the other fields of the thread's modes; each group filters them and keeps its own
  auto at = [&](int i) { return pad(BLU ? t + i * tpf : 8 * t + i); };
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (!BLU || t + i * tpf < n) buf[at(i)] = v[i];
  __syncthreads();
  const double2* b0 = buf - size_t(q) * (9 * tpf);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int ky = BLU ? t + i * tpf : freq_at(8 * t + i, ax.lm);
    if (live && ky < n) {
      double2 m[3] = {b0[at(i)], b0[9 * tpf + at(i)], b0[18 * tpf + at(i)]};
      mode_filter(mf, col, ky, m);
      v[i].x = q == 0 ? m[0].x : q == 1 ? m[1].x : m[2].x;
      v[i].y = q == 0 ? m[0].y : q == 1 ? m[1].y : m[2].y;
    }
  }
  __syncthreads();
  if (BLU) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = t + i * tpf;
      v[i] = j < n ? cmul(conj2(v[i]), ax.chirp[j]) : make_double2(0.0, 0.0);
    }
    convolve(v, buf, t, ax);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = t + i * tpf;
      if (live && j < n) g[j] = conj2(cmul(v[i], ax.chirp[j]));
    }
  } else {
    fft_dit(v, buf, t, ax.lm, ax.tw);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (live) g[t + i * tpf] = v[i];
  }
}

template <bool BLU>
__global__ __launch_bounds__(1024) void k_rows_inv(const double2* __restrict__ G, double* __restrict__ u, FftAxis ax,
                                                  int ny, int npairs) {
  extern __shared__ double2 lds[];
  const int n = ax.n, tpf = 1 << (ax.lm - 3);
  const int t = int(threadIdx.x) & (tpf - 1), sub = int(threadIdx.x) >> (ax.lm - 3);
  double2* buf = lds + size_t(sub) * (9 * tpf);
  const int blk = neighbour_block(int(blockIdx.x), int(gridDim.x));
  const int pair = blk * (int(blockDim.x) >> (ax.lm - 3)) + sub;
  const bool live = pair < npairs;
  const int npy = (ny + 1) / 2;
  const int fld = live ? pair / npy : 0, y0 = live ? 2 * (pair % npy) : 0;
  const bool two = live && y0 + 1 < ny;
  // Z = A + i B over all k from the half spectra of two real rows (the
  // imaginary parts at k = 0 and n/2 are 0), the block's pairs fastest over
  // the threads
  const int fpb = int(blockDim.x) >> (ax.lm - 3), lf = 31 - __clz(fpb);
  const int lp = int(threadIdx.x) & (fpb - 1), wp = blk * fpb + lp, ks = int(blockDim.x) >> lf;
  if (wp < npairs) {
    const int of = wp / npy, oy = 2 * (wp % npy);
    const bool both = oy + 1 < ny;
    double2* zb = lds + size_t(lp) * (9 * tpf);
    for (int k = int(threadIdx.x) >> lf; k <= n / 2; k += ks) {
      const double2* p = G + (size_t(k) * 3 + of) * ny + oy;
      double2 a = p[0], c = both ? p[1] : make_double2(0.0, 0.0);
      const bool self = k == 0 || 2 * k == n;
      if (self) a.y = c.y = 0.0;
      const double2 z = make_double2(a.x - c.y, a.y + c.x), y = make_double2(a.x + c.y, c.x - a.y);
      zb[pad(BLU ? k : pos_of(k, ax.lm))] = z;
      if (!self) zb[pad(BLU ? n - k : pos_of(n - k, ax.lm))] = y;
    }
  }
  __syncthreads();
  double2 v[8];
  if (BLU) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = t + i * tpf;
      v[i] = make_double2(0.0, 0.0);
      if (j < n) v[i] = cmul(conj2(buf[pad(j)]), ax.chirp[j]);
    }
    convolve(v, buf, t, ax);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = t + i * tpf;
      if (j < n) v[i] = conj2(cmul(v[i], ax.chirp[j]));
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = buf[pad(8 * t + i)];
    fft_dit(v, buf, t, ax.lm, ax.tw);
  }
  if (!live) return;
  double* ua = u + (size_t(fld) * ny + y0) * n;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int j = t + i * tpf;
    if (j < n) {
      ua[j] = v[i].x;
      if (two) ua[n + j] = v[i].y;
    }
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Points of the FFT that a length takes: itself for a power of two, else the
// chirp's.  0: not done here (a power of two up to 4096 or a length up to
// 2048: the exchange buffer of 4096 points is 72 KB, two blocks a CU).
int fft_points(int n) {
  if (n < 16) return 0;
  int M = 16;
  if ((n & (n - 1)) == 0) return n <= 4096 ? n : 0;
  if (n > 2048) return 0;
  while (M < 2 * n - 1) M *= 2;
  return M;
}

static size_t twiddle_count(int M) {
  size_t c = 0;
  for (; M > 8; M /= 8) c += 3 * size_t(M / 8);
  return c;
}

size_t fft_axis_doubles(int n) {
  const int M = fft_points(n);
  if (M == 0) return 0;
  return size_t(2) * (twiddle_count(M) + (M == n ? 0 : M + n));
}

namespace {
// plain recursive transform for the chirp's table (host, once per length)
struct LC {
  long double x, y;
};
void host_fft(LC* a, LC* tmp, int n, const LC* w, int ws) {
  if (n == 1) return;
  const int h = n / 2;
  for (int i = 0; i < h; ++i) {
    tmp[i] = a[2 * i];
    tmp[h + i] = a[2 * i + 1];
  }
  host_fft(tmp, a, h, w, 2 * ws);
  host_fft(tmp + h, a + h, h, w, 2 * ws);
  for (int i = 0; i < h; ++i) {
    const LC e = tmp[i], o = tmp[h + i], c = w[i * ws];
    const LC p = {o.x * c.x - o.y * c.y, o.x * c.y + o.y * c.x};
    a[i] = {e.x + p.x, e.y + p.y};
    a[h + i] = {e.x - p.x, e.y - p.y};
  }
}
}  // namespace

// [tw: per step L = M, M/8, ..: w_L^j, w_L^2j, w_L^4j, j < L/8] [chirp: exp(-i pi j^2 / n), j < n] [bhat: the transform of
// the conjugate chirp / M, at position 8 t + q stored at q M/8 + t]
void fft_axis_fill(int n, double* out) {
  const int M = fft_points(n);
  if (M == 0) return;
  const long double pi = 3.14159265358979323846264338327950288L;
  std::vector<LC> w(M);
  for (int k = 0; k < M; ++k) {
    w[k] = {cosl(2.0L * pi * k / M), -sinl(2.0L * pi * k / M)};
  }
  double* tw = out;
  for (int L = M; L > 8; L /= 8)
    for (int e = 1; e <= 4; e *= 2)
      for (int j = 0; j < L / 8; ++j) {
        const LC& c = w[size_t(j) * e * (M / L)];
        *tw++ = double(c.x);
        *tw++ = double(c.y);
      }
  if (M == n) return;
  double* chirp = out + 2 * twiddle_count(M);
  double* bhat = chirp + 2 * size_t(n);
  std::vector<LC> b(M, LC{0.0L, 0.0L}), tmp(M);
  for (int j = 0; j < n; ++j) {
    const long long e = (static_cast<long long>(j) * j) % (2LL * n);
    const long double c = cosl(pi * e / n), s = sinl(pi * e / n);
    chirp[2 * j] = double(c);
    chirp[2 * j + 1] = double(-s);
    b[j] = {c, s};
    if (j > 0) b[M - j] = {c, s};
  }
  host_fft(b.data(), tmp.data(), M, w.data(), 1);
  int lm = 0;
  while ((1 << lm) < M) ++lm;
  for (int p = 0; p < M; ++p) {
    int k = 0, s = 0, r = p;
    for (int l = lm; l > 3; l -= 3) {
      k += (r >> (l - 3)) << s;
      r &= (1 << (l - 3)) - 1;
      s += 3;
    }
    k += r << s;
    const size_t at = size_t(p & 7) * (M / 8) + (p >> 3);
    bhat[2 * at] = double(b[k].x / M);
    bhat[2 * at + 1] = double(b[k].y / M);
  }
}

FftAxis fft_axis(int n, const double* tab) {
  FftAxis a{};
  const int M = fft_points(n);
  a.n = n;
  while ((1 << a.lm) < M) ++a.lm;
  a.tw = reinterpret_cast<const double2*>(tab);
  a.chirp = a.tw + twiddle_count(M);
  a.bhat = a.chirp + n;
  return a;
}

namespace {
// 4 pairs are 8 rows, one 128-byte line of G for each k.  2048^2, forward
// rows: one pair a block 74 us, two (512 threads) 64, four (1024) 67.
constexpr int kRowPairs = 4;
constexpr int kRowThreads = 512;
// k_cols3 up to 2^these points.  2048 points, columns stage, k_cols ->
// k_cols3: power of two (2048^2) 77 -> 109 us, one block of 12 waves a CU
// against three of 4; chirp (1000^2) 73 -> 62.
constexpr int kCols3MaxLog = 10, kCols3ChirpMaxLog = 11;
size_t fft_lds(const FftAxis& a, int ffts) { return size_t(ffts) * (size_t(9) << (a.lm - 3)) * sizeof(double2); }
bool is_chirp(const FftAxis& a) { return (1 << a.lm) != a.n; }

// Row pairs per block: at least a wave, then up to kRowPairs while the chip
// has two blocks a CU.
int row_pairs(const FftAxis& a, int pairs) {
  const int tpf = 1 << (a.lm - 3);
  int p = tpf < 64 ? 64 / tpf : 1;
  while (p < kRowPairs && 2 * p * tpf <= kRowThreads && pairs >= 2 * p * 512) p *= 2;
  return p;
}

template <class K>
hipError_t allow_lds(K k, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
}
}  // namespace

int rows_blocks(const FftAxis& ax, int pairs) {
  const int p = row_pairs(ax, pairs);
  return (pairs + p - 1) / p;
}

hipError_t launch_rows_fwd(const double* f, double2* G, const FftAxis& ax, int ny, int first, int pairs, int* flags,
                           hipStream_t s) {
  const int p = row_pairs(ax, pairs);
  const size_t lds = fft_lds(ax, p);
  auto k = is_chirp(ax) ? k_rows_fwd<true> : k_rows_fwd<false>;
  const hipError_t e = allow_lds(k, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(unsigned(rows_blocks(ax, pairs))), dim3(unsigned(p << (ax.lm - 3))), lds, s, f, G, ax, ny,
                     first, pairs, flags);
  return hipSuccess;
}

hipError_t launch_cols(double2* G, const FftAxis& ax, int nxh, const ModeFilter& mf, const int* flags, int nflags,
                       int* word, hipStream_t s) {
  const int tpf = 1 << (ax.lm - 3);
  if (ax.lm <= (is_chirp(ax) ? kCols3ChirpMaxLog : kCols3MaxLog)) {
    const int c = 3 * tpf < 64 ? 64 / (3 * tpf) : 1;   // columns per block
    const size_t lds = fft_lds(ax, 3 * c);
    auto k = is_chirp(ax) ? k_cols3<true> : k_cols3<false>;
    const hipError_t e = allow_lds(k, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(unsigned((nxh + c - 1) / c)), dim3(unsigned(3 * c * tpf)), lds, s, G, ax, nxh, mf, flags,
                       nflags, word);
    return hipSuccess;
  }
  const size_t lds = fft_lds(ax, 1);
  auto k = is_chirp(ax) ? k_cols_chirp : k_cols;
  const hipError_t e = allow_lds(k, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(unsigned(nxh)), dim3(unsigned(tpf)), lds, s, G, ax, mf, flags, nflags, word);
  return hipSuccess;
}

hipError_t launch_rows_inv(const double2* G, double* u, const FftAxis& ax, int ny, hipStream_t s) {
  const int pairs = 3 * ((ny + 1) / 2), p = row_pairs(ax, pairs);
  const size_t lds = fft_lds(ax, p);
  auto k = is_chirp(ax) ? k_rows_inv<true> : k_rows_inv<false>;
  const hipError_t e = allow_lds(k, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(unsigned(rows_blocks(ax, pairs))), dim3(unsigned(p << (ax.lm - 3))), lds, s, G, u, ax, ny,
                     pairs);
  return hipSuccess;
}

}  // namespace rexii
