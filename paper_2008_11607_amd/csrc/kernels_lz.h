// Launchers of the shared-Krylov (multi-shift) path (kernels_lz.hip).
// States are [3][ny][nx] FP64, a batch's states `stride` doubles apart; beta
// is [nrhs][ldb] with beta_0 = ||f||_W and beta_j = ||w_j||_W; part is
// [nrhs][lz_blocks()] block partial sums.
#ifndef REXII_KERNELS_LZ_H
#define REXII_KERNELS_LZ_H

#include <hip/hip_runtime.h>
#include <stddef.h>

#include "kernels.h"

namespace rexii {

// Two poles z, -conj(z) of a term with their weights.
struct LzPair {
  double2 z, w1, w2;
};

// A launch of Lanczos steps with the vectors on the chip (k_lz_chip).
constexpr int kLzChipMaxG = 256;
struct LzChip {
  int nx, ny, nrhs;
  int G, Sc, nt, rt, lds;   // blocks a state, runs a column, threads, rows a run, LDS bytes
  int gpx, rec_stride;      // groups per XCD (a state then lies on one) or 0; words between records
  int groups, ctl_words;
  ChipWaits waits;
  int j0, steps;            // first step (1-based) and their number
  int kept, ldb;            // vectors kept in memory (place of buf_j: see run_multishift), row of beta
  size_t stride;            // doubles between states
  double g, fc, H0;
  const double* H;          // depth field or nullptr
  double* vecs;
  double* beta;
  unsigned long long* rec;
  unsigned long long* ring;
  int* ctl;
  int* flag;                // kChipGaveUp, kChipLate
};
bool lz_chip_config(int nx, int ny, int nrhs, bool depth, int cus, LzChip* c);
size_t lz_chip_bytes(const LzChip& c);
void lz_chip_mailboxes(LzChip& c, void* mem, hipStream_t s);
void launch_lz_chip(const LzChip& c, hipStream_t s);

int lz_blocks(int nx, int ny);
// buf = f, beta[r][0] = ||f_r||_W, flag[0] |= 1 on a non-finite value of f.
void launch_lz_start(const double* f, double* buf, size_t stride, const double* H, double H0, double g, int nx, int ny,
                     int nrhs, double* part, int* flag, double* beta, int ldb, hipStream_t s);
// Lanczos step j (1-based) on cur = buf_j, prev = buf_{j-1}; out (which may
// be prev) receives buf_{j+1}; with part, beta[r][j] = ||w_j||_W is formed;
// with y and u, u += y_j v_j; last: only the accumulation.
void launch_lz_step(const double* cur, const double* prev, double* out, size_t stride, const double* H, double H0,
                    double g, double fc, int nx, int ny, int nrhs, int j, double* beta, int ldb, double* part,
                    const double* y, int ldy, double* u, int last, hipStream_t s);
// u = sum_{j < m} coef[j] vecs[j], vectors of n3 doubles.
void launch_lz_gather(const double* vecs, size_t n3, int m, const double* coef, double* u, hipStream_t s);
// The small problem of one state: b = its beta row, y[j], coef[j] = y_j / b_{j-1}
// and out = (|y|^2, |last 8 of y|^2), 64 nb pairs at a time; scratch:
// lz_small_bytes(m, nb), 256-byte aligned.
size_t lz_small_bytes(int m, int nb);
void launch_lz_small(const double* b, int m, double t, const LzPair* pairs, int npair, int nb, void* scratch, double* y,
                     double* coef, double* out, hipStream_t s);

}  // namespace rexii

#endif
