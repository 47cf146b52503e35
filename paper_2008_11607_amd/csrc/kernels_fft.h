// Launchers of the Fourier-space path (kernels_fft.hip).
#ifndef REXII_KERNELS_FFT_H
#define REXII_KERNELS_FFT_H

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace rexii {

// Fourier-space path (constant depth).  tab holds nterm merged terms
// (a, b^2, A1, B1, A2, B2); deriv 0: centred-difference symbols, 1: Fourier
// differentiation.
// canon_count: number of distinct canonical wavenumbers on
// an axis of n points (modes with the same canonical pair share theta).
int canon_count(int n, int deriv);
// coef [cny][cnx] = scale (Re c1, Re c2) per canonical pair; nw waves per
// block, the terms in ns splits (part: ns x entries double2 when ns > 1).
void mode_coef_shape(int entries, int nterm, bool whole, int* nw, int* ns);
// sxt, syt: the axis symbols s(k) of the x wavenumbers 0..nx/2 and the y
// wavenumbers 0..ny-1 (axis_symbol), device.
double axis_symbol(int k, int n, int deriv);
// sym = 1 (square grids): the table holds the unordered pairs a <= b only,
// cnx (cnx + 1) / 2 entries (mode_entries).
int mode_entries(int cnx, int cny, int sym);
// With ns > 1 the splits go to part; k_mode_coef_sum adds them into coef,
// unless mode_sum_in_apply(entries, ns): then k_mode_apply adds them (pass
// it part and ns).
void launch_mode_coef(double2* coef, double2* part, int cnx, int cny, int sym, const double* sxt, const double* syt,
                      double t, double g, double H, double fc, double scale, const double* tab, int nterm, int nw,
                      int ns, hipStream_t s);
bool mode_sum_in_apply(int entries, int ns);
// Pole sums with the far terms of each box of theta as one polynomial
// (kernels_fft.hip).  nbox = 0: the direct sums are the better way.
constexpr int kCheb = 32;  // Chebyshev points per box: half a wave
struct FarBoxes {
  double w, inv_w, tg;  // uniform boxes: width, first edge
  double d, inv_h;      // poles at theta = +-h j +- i d
  int k, nbox;          // graded boxes 0..k, boxes in all
};
// For theta in [0, thmax], terms j with poles z = -d + i h j.
FarBoxes far_boxes(double thmax, double h, double d, int entries, int nterm);
void far_shape(int nbox, int nterm, int* nw, int* ns);  // waves per block, term splits
size_t far_doubles2(const FarBoxes& fb, int nterm);  // double2 of scratch
void launch_mode_boxed(double2* coef, double2* far, const FarBoxes& fb, int cnx, int cny, int sym, const double* sxt,
                       const double* syt, double t, double g, double H, double fc, double scale, const double* tab,
                       int nterm, hipStream_t s);
// What the filter of a mode needs: the coefficients (ns <= 1: scaled entries;
// ns > 1: ns x ne unscaled split sums, added in order and multiplied by
// scale) and the axis symbols.
struct ModeFilter {
  const double2* coef;
  int ns, ne;
  double scale;
  int cnx, sym, nx, ny, deriv;
  const double *sxt, *syt;
  double t, g, H, fc, a0;
};
// F [3][ny][nx/2+1] <- a0 F + C1 t A F + C2 (t A)^2 F
void launch_mode_apply(double2* F, const ModeFilter& mf, hipStream_t s);

// Own transforms (kernels_fft2d.hip).  fft_points: 0 if a length is not done
// there; fft_axis_doubles/fill: its table (twiddles and chirp), to be handed
// to fft_axis as a device copy.
struct FftAxis {
  int n, lm;  // length, log2 of the points of its FFT
  const double2 *tw, *chirp, *bhat;
};
int fft_points(int n);
size_t fft_axis_doubles(int n);
void fft_axis_fill(int n, double* out);
FftAxis fft_axis(int n, const double* tab);
int rows_blocks(const FftAxis& ax, int pairs);
// Row pairs [first, first + pairs) of the 3 (ny+1)/2 of a state; one word per
// block in flags (rows_blocks of them).
hipError_t launch_rows_fwd(const double* f, double2* G, const FftAxis& ax, int ny, int first, int pairs, int* flags,
                           hipStream_t s);
hipError_t launch_cols(double2* G, const FftAxis& ax, int nxh, const ModeFilter& mf, const int* flags, int nflags,
                       int* word, hipStream_t s);
hipError_t launch_rows_inv(const double2* G, double* u, const FftAxis& ax, int ny, hipStream_t s);

// u = f and one finiteness word per block: flags[copy_check_blocks(n)]
// (at most kCopyCheckMaxBlocks), each 0 or 1.
constexpr int kCopyCheckMaxBlocks = 2048;
int copy_check_blocks(size_t n);
void launch_copy_check(const double* f, double* u, size_t n, int* flags, hipStream_t s);

}  // namespace rexii

#endif
