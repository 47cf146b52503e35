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
// problem on the host took 44.1 ms at 512^2, t rho = 1000 (17.3 ms with the
// vectors kept, 12.0 with the steps on the chip, below) and 27.1 ms for the
// 2048^2 depth field at t rho = 100 (13.3 to 15.4 ms now, the sum of 160
// vectors 2.8 ms at 5.8 TB/s).  The reductions are in a fixed order, so
// repeated steps reproduce pass 1 bit for bit (a step whose vector is not kept
// is k_lz_step in both passes).
//
// Storage: the vectors are kept unnormalised, buf_j = beta_{j-1} v_j
// (buf_1 = f, beta_0 = ||f||_W); step j reads buf_j and buf_{j-1} and writes
// w_j = buf_{j+1}, to a place of its own or over buf_{j-1}.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "kernels_lz.h"
#include "chip_sync.h"

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

// ---------------------------------------------------------------------------
// Lanczos steps with the vectors on the chip.  A group of G blocks holds a
// state: a block has a strip of grid rows, a thread a column's run of RT (or
// RT - 1) rows with buf_j and buf_{j-1} (and the depth) in registers; LDS
// holds eta and H u for the east and west neighbours and the runs' edge rows
// of H v.  A launch runs `steps` steps from the vectors in memory; a step
// writes buf_{j+1} there (the basis: only steps whose vector is kept run here,
// so the two vectors a launch starts from outlive it), posts eta and H v of the strip's edge
// rows and one partial norm, and waits once for the other blocks, as the
// chip COCG kernel does.  Four mailbox buffers: the words of sync i are
// emptied after sync i + 1 and known to be gone at the end of i + 2, before
// the record of i + 3 is posted; nobody looks for i + 4 before it has that.
//
// Bound: the exchange.  One launch of k_lz_step and one of k_lz_norm a step
// took 14 us at 512^2 and 12 us at 64^2, a step here 7.5 and 2.4 us (whole
// calls: 512^2, t rho 1000 17.3 -> 12.0 ms; 64^2, t rho 100 4.0 -> 0.9 ms).
// ---------------------------------------------------------------------------
template <int RT, bool DEPTH>
__global__ __launch_bounds__(512, 2) void k_lz_chip(LzChip c) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lz_lds[];
  __shared__ double red[8];
  __shared__ double bc[3];      // 1 / beta_j, beta_j / beta_{j-1}, beta_j
  __shared__ int sh[8];
  constexpr int PR = RT | 1;
  const int tid = int(threadIdx.x), nt = int(blockDim.x), lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6;
  const int nx = c.nx, ny = c.ny, G = c.G;
  const bool local = c.gpx > 0;
  int st = int(blockIdx.x), rank = 0, gid = st;
  if (tid == 0) sh[5] = 0;      // a wait gave up
  if (G > 1) {
    GroupPlace gp;
    bool late = false;
    if (!join_group(c.ctl, G, c.gpx, c.nrhs, c.waits, sh, gp, late)) {
      if (late && tid == 0) atomicOr(c.flag, kChipLate);
      return;
    }
    gid = gp.gid;
    rank = gp.rank;
    st = local ? (gid - gp.xcd * c.gpx) * 8 + gp.xcd : gid;
  }
  const size_t n = size_t(nx) * ny, n3 = 3 * n;
  double* vec = c.vecs + size_t(st) * c.stride;
  double* br = c.beta + size_t(st) * c.ldb;
  auto place = [&](int j) { return vec + size_t(j <= c.kept ? j - 1 : c.kept + ((j - c.kept - 1) & 1)) * n3; };
  // ---- the block's rows ya .. ya + R - 1 and the thread's run of them
  const int ya = int((long long)rank * ny / G), R = int((long long)(rank + 1) * ny / G) - ya;
  const int s = tid / nx;
  const bool valid = s < c.Sc;
  const int col = valid ? tid - s * nx : 0, seg = valid ? s : 0;
  auto first_row = [&](int q) { return int((long long)q * R / c.Sc); };
  const int r0 = first_row(seg);
  const bool full = first_row(seg + 1) - r0 == RT;
  const bool rtop = valid && G > 1 && seg == 0, rbot = valid && G > 1 && seg == c.Sc - 1;
  const int su = (seg == 0) ? c.Sc - 1 : seg - 1, sd = (seg == c.Sc - 1) ? 0 : seg + 1;
  const int item = seg * nx + col, iu = su * nx + col, id = sd * nx + col;
  const int base = item * PR;
  const int west = (seg * nx + (col == 0 ? nx - 1 : col - 1)) * PR, east = (seg * nx + (col + 1 == nx ? 0 : col + 1)) * PR;
  const int utop = iu * PR + first_row(su + 1) - first_row(su) - 1, ubot = id * PR;
  const int items = c.Sc * nx;
  double* E = reinterpret_cast<double*>(lz_lds);
  double* U = E + size_t(items) * PR;
  double* VT = U + size_t(items) * PR;   // H v of a run's first row
  double* VB = VT + items;               // ... and of its last
  const int y0 = ya + r0;
  auto gofs = [&](int i) {               // grid point of row i (-1 .. RT) of the run
    int y = y0 + i;
    y = (y < 0) ? y + ny : (y >= ny ? y - ny : y);
    return unsigned(y * nx + col);
  };
  unsigned long long* rec = c.rec + size_t(gid) * 4 * G * c.rec_stride;
  unsigned long long* ring = c.ring + size_t(gid) * 16 * G * nx;   // [4][G][top eta, H v, bottom eta, H v][nx]
  const int up_rank = (rank == 0) ? G - 1 : rank - 1, dn_rank = (rank + 1 == G) ? 0 : rank + 1;
  const double hx = 0.5 * nx, hy = 0.5 * ny, g = c.g, fc = c.fc;

  double A[3][RT], B[3][RT], H[DEPTH ? RT : 1];
  double et = 0.0, vt = 0.0, eb = 0.0, vb = 0.0;   // ring rows: eta and H v above and below
  {
    const double* cu = place(c.j0);
    const double* pv = place(c.j0 > 1 ? c.j0 - 1 : 1);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const bool in = valid && (i < RT - 1 || full);
      const unsigned q = in ? gofs(i) : 0u;
      if (DEPTH) H[i] = in ? c.H[q] : 0.0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        A[k][i] = in ? cu[k * n + q] : 0.0;
        B[k][i] = (in && c.j0 > 1) ? pv[k * n + q] : 0.0;
      }
    }
    if (rtop) {
      const unsigned q = gofs(-1);
      et = cu[q];
      vt = (DEPTH ? c.H[q] : c.H0) * cu[2 * n + q];
    }
    if (rbot) {
      const unsigned q = gofs(full ? RT : RT - 1);
      eb = cu[q];
      vb = (DEPTH ? c.H[q] : c.H0) * cu[2 * n + q];
    }
  }
  auto depth = [&](int i) { return DEPTH ? H[DEPTH ? i : 0] : c.H0; };
  // eta, H u and the edge rows of H v of a vector into LDS
  auto share = [&](const double (&v)[3][RT]) __attribute__((always_inline)) {
    if (!valid) return;
#pragma unroll
    for (int i = 0; i < RT; ++i)
      if (i < RT - 1 || full) {
        E[base + i] = v[0][i];
        U[base + i] = depth(i) * v[1][i];
      }
    VT[item] = depth(0) * v[2][0];
    VB[item] = (full || RT == 1) ? depth(RT - 1) * v[2][RT - 1] : depth(RT > 1 ? RT - 2 : 0) * v[2][RT > 1 ? RT - 2 : 0];
  };
  share(A);
  double bj1 = br[c.j0 - 1], sc = 1.0 / bj1, sp = (c.j0 >= 2) ? bj1 / br[c.j0 - 2] : 0.0;
  __syncthreads();
  unsigned sync_no = 0;
  bool bad = false;
  // step j: cu = buf_j, pv = buf_{j-1}, replaced by buf_{j+1}
  auto step = [&](const double (&cu)[3][RT], double (&pv)[3][RT], int j) __attribute__((always_inline)) {
    const unsigned buf = sync_no & 3u, obuf = (sync_no + 3u) & 3u;
    double acc = 0.0;
    if (valid) {
      double eS = rtop ? et : E[utop], vS = rtop ? vt : VB[iu];
      const double eL = rbot ? eb : E[ubot], vL = rbot ? vb : VT[id];
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        double eN, vN;
        if (i == RT - 1) {
          eN = eL;
          vN = vL;
        } else {
          eN = cu[0][i + 1];
          vN = depth(i + 1) * cu[2][i + 1];
          if (i == RT - 2) {
            eN = full ? eN : eL;
            vN = full ? vN : vL;
          }
        }
        const double ae = -(hx * (U[east + i] - U[west + i]) + hy * (vN - vS));
        const double au = -g * hx * (E[east + i] - E[west + i]) + fc * cu[2][i];
        const double av = -g * hy * (eN - eS) - fc * cu[1][i];
        eS = cu[0][i];
        vS = depth(i) * cu[2][i];
        double w0 = sc * ae + sp * pv[0][i], w1 = sc * au + sp * pv[1][i], w2 = sc * av + sp * pv[2][i];
        if (i == RT - 1 && !full) w0 = w1 = w2 = 0.0;
        pv[0][i] = w0;
        pv[1][i] = w1;
        pv[2][i] = w2;
        acc += g * w0 * w0 + depth(i) * (w1 * w1 + w2 * w2);
      }
    }
    acc = wave_total63(acc);
    if (lane == 63) red[wid] = acc;
    __syncthreads();  // every neighbour value has been read
    share(pv);
    if (G > 1) {
      unsigned long long* rx = ring + (size_t(buf) * G + rank) * 4 * nx + col;
      if (rtop) {
        post(rx, pv[0][0], local);
        post(rx + nx, depth(0) * pv[2][0], local);
      }
      if (rbot) {
        const int l = RT > 1 ? RT - 2 : 0;
        post(rx + 2 * nx, full ? pv[0][RT - 1] : pv[0][l], local);
        post(rx + 3 * nx, full ? depth(RT - 1) * pv[2][RT - 1] : depth(l) * pv[2][l], local);
      }
    }
    if (wid == 0) {
      double v = 0.0;
      for (int k = 0; k < nw; ++k) v += red[k];
      if (G > 1) {
        unsigned long long* rb = rec + size_t(buf) * G * c.rec_stride;
        if (lane == 0) post(rb + size_t(rank) * c.rec_stride, v, local);
        v = 0.0;
        for (int b0 = 0; b0 < G; b0 += 64) {
          const unsigned long long* th = rb + size_t(b0 + lane < G ? b0 + lane : 0) * c.rec_stride;
          unsigned long long w;
          unsigned k = 0;
          while (!__all((w = ald(th)) != kNoWord)) {
            if (++k > kRunPolls) {
              sh[5] = 1;
              break;
            }
          }
          const double t = wave_total63(b0 + lane < G ? __longlong_as_double((long long)w) : 0.0);
          v += lane_value(t, 63);
        }
      }
      const double b = sqrt(v);
      if (lane == 0) {
        bc[0] = 1.0 / b;
        bc[1] = b / bj1;
        bc[2] = b;
        if (rank == 0) br[j] = b;
      }
    }
    if (G > 1) {
      const unsigned long long* rup = ring + (size_t(buf) * G + up_rank) * 4 * nx + 2 * nx + col;
      const unsigned long long* rdn = ring + (size_t(buf) * G + dn_rank) * 4 * nx + col;
      unsigned k = 0;
      if (rtop) {
        unsigned long long a, b;
        while ((a = ald(rup)) == kNoWord || (b = ald(rup + nx)) == kNoWord) {
          if (++k > kRunPolls) {
            sh[5] = 1;
            break;
          }
        }
        et = __longlong_as_double((long long)a);
        vt = __longlong_as_double((long long)ald(rup + nx));
      }
      if (rbot) {
        unsigned long long a, b;
        while ((a = ald(rdn)) == kNoWord || (b = ald(rdn + nx)) == kNoWord) {
          if (++k > kRunPolls) {
            sh[5] = 1;
            break;
          }
        }
        eb = __longlong_as_double((long long)a);
        vb = __longlong_as_double((long long)ald(rdn + nx));
      }
      stores_done();  // the words emptied after the sync before (long done)
    }
    __syncthreads();
    ++sync_no;
    sc = bc[0];
    sp = bc[1];
    bj1 = bc[2];
    if (G > 1) {
      if (tid == 0) mst(rec + (size_t(obuf) * G + rank) * c.rec_stride, kNoWord, local);
      unsigned long long* rx = ring + (size_t(obuf) * G + rank) * 4 * nx + col;
      if (rtop) {
        mst(rx, kNoWord, local);
        mst(rx + nx, kNoWord, local);
      }
      if (rbot) {
        mst(rx + 2 * nx, kNoWord, local);
        mst(rx + 3 * nx, kNoWord, local);
      }
      bad = uni(sh[5]) != 0;
    }
    // the vector, for the basis and the next launch: written here, a whole
    // step before the next loads that a wavefront waits for (loads complete
    // after the stores issued before them)
    if (valid) {
      double* ov = place(j + 1);
#pragma unroll
      for (int i = 0; i < RT; ++i)
        if (i < RT - 1 || full) {
          const unsigned q = gofs(fresh(i));
          __builtin_nontemporal_store(pv[0][i], ov + q);
          __builtin_nontemporal_store(pv[1][i], ov + n + q);
          __builtin_nontemporal_store(pv[2][i], ov + 2 * n + q);
        }
    }
  };
  for (int k = 0; k < c.steps && !bad; k += 2) {
    step(A, B, c.j0 + k);
    if (k + 1 >= c.steps || bad) break;
    step(B, A, c.j0 + k + 1);
  }
  if (bad) {
    if (tid == 0) atomicOr(c.flag, kChipGaveUp);
    return;
  }
  // ---- the mailboxes empty for the next launch
  if (G > 1) {
    stores_done();
    __syncthreads();
    if (tid == 0) {
      int* gc = c.ctl + kChipCtlHead + gid * kChipCtlGroup;
      __hip_atomic_fetch_add(&gc[2], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      unsigned k = 0;
      while (ldc(&gc[2]) < G) {
        if (++k > kRunPolls) {
          atomicOr(c.flag, kChipGaveUp);
          break;
        }
      }
    }
    __syncthreads();
    if (tid < 4) ast(rec + (size_t(tid) * G + rank) * c.rec_stride, kNoWord);
    for (int k = tid; k < 16 * nx; k += nt) ast(ring + (size_t(k / (4 * nx)) * G + rank) * 4 * nx + k % (4 * nx), kNoWord);
  }
}

// Zeroes the control words and the flag before a launch.
__global__ __launch_bounds__(256) void k_lz_ctl(int* ctl, int words, int* flag) {
  for (int k = threadIdx.x; k < words; k += 256) ctl[k] = 0;
  if (threadIdx.x == 0) flag[0] = 0;
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
// part[block][j] = the block's sum over its 64 pairs, added to what earlier
// pairs left there (again).
constexpr int kSmU = 8;   // rows whose loads are in flight together
__global__ __launch_bounds__(64) void k_lz_small(const double* __restrict__ b, int m, double t,
                                                 const LzPair* __restrict__ pairs, int npair, double2* inv,
                                                 double* __restrict__ part, int again) {
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
      if (lane == 63) pp[j - 1] = again ? pp[j - 1] + s : s;
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

namespace {
using LzChipFn = void (*)(LzChip);
constexpr int kLzMaxRT = 10;
template <bool D>
LzChipFn lz_chip_fn(int rt) {
  static const LzChipFn f[kLzMaxRT] = {k_lz_chip<1, D>, k_lz_chip<2, D>, k_lz_chip<3, D>, k_lz_chip<4, D>,
                                       k_lz_chip<5, D>, k_lz_chip<6, D>, k_lz_chip<7, D>, k_lz_chip<8, D>,
                                       k_lz_chip<9, D>, k_lz_chip<10, D>};
  return f[rt - 1];
}
}  // namespace

// Launch shape of k_lz_chip; false where no shape fits or k_lz_step is the
// faster.  Estimates in us, from steps timed on MI355X: a thread's row takes
// about 40 VALU instructions, a step 250 more; the exchange beyond them about
// 1.2 us + 2 ns a column on one XCD and 1.3 us + 9 ns a column + 4 ns a block across (64^2:
// 2.4 us a step in all, 256^2: 4.2, 512^2: 7.5, much the same for 64 to 128
// blocks); the vector's write is bound by about 0.55 TB/s per XCD.  k_lz_step
// and k_lz_norm: 10 us + 80 bytes a point at 5 TB/s (14 us at 512^2).
bool lz_chip_config(int nx, int ny, int nrhs, bool depth, int cus, LzChip* c) {
  double best = 10.0 + 80.0 * nx * double(ny) * nrhs / 5e6;
  bool found = false;
  for (int Sc = 1; Sc * nx <= 512; ++Sc) {
    const int nt = (Sc * nx + 63) / 64 * 64;
    for (int rt = 1; rt <= kLzMaxRT; ++rt) {
      const int G = (ny + Sc * rt - 1) / (Sc * rt);
      if ((ny + G * Sc - 1) / (G * Sc) != rt || ny < G * Sc || G > kLzChipMaxG) continue;
      if (G > 1 && ny / G < 1) continue;
      const size_t lds = (size_t(2) * (rt | 1) + 2) * Sc * nx * 8;
      if (lds > size_t(kChipMaxLds)) continue;
      const void* f = reinterpret_cast<const void*>(depth ? lz_chip_fn<true>(rt) : lz_chip_fn<false>(rt));
      if (lds > 48 * 1024 &&
          hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kChipMaxLds) != hipSuccess) {
        (void)hipGetLastError();
        continue;
      }
      int occ = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, f, nt, lds) != hipSuccess || occ < 1) {
        (void)hipGetLastError();
        continue;
      }
      for (int loc = 0; loc < 2; ++loc) {
        const int gpx = (nrhs + 7) / 8, fit = (cus / 8) * occ / G;   // groups an XCD has to take, and can at once
        if (loc && (G == 1 || fit < 1)) continue;
        if (!loc && cus * occ < G) continue;
        const double turns = loc ? std::ceil(double(gpx) / fit) : std::ceil(double(nrhs) / (cus * occ / G));
        const int per_cu = loc ? (G * std::min(fit, gpx) + cus / 8 - 1) / (cus / 8)
                               : (G * std::min(nrhs, cus * occ / G) + cus - 1) / cus;   // blocks that share a CU
        const double valu = per_cu * ((nt / 64 + 3) / 4) * 4.0 * (rt * 40.0 + 250.0) / 2370.0;
        const double wr = 24.0 * nx * double(ny) / 0.55e6 * (loc ? std::min(fit, gpx) : std::max(1.0, double(nrhs) / turns) / std::min(8.0, double(G)));
        // (one wavefront a SIMD waits out its own latencies: 1.5 times as long)
        const double own = (nt * per_cu <= 256 ? 1.5 : 1.0) * valu + (G == 1 ? 0.9 : loc ? 1.2 + 0.002 * nx : 1.3 + 0.009 * nx + 0.004 * G);
        const double t = turns * (std::max(own, wr) + 0.2 * std::min(own, wr));
        if (t < best) {
          best = t;
          found = true;
          c->nx = nx;
          c->ny = ny;
          c->nrhs = nrhs;
          c->G = G;
          c->Sc = Sc;
          c->nt = nt;
          c->rt = rt;
          c->lds = int(lds);
          c->gpx = loc ? gpx : 0;
          c->rec_stride = loc ? kChipRec : 1;
          c->groups = loc ? 8 * gpx : nrhs;
          c->ctl_words = kChipCtlHead + kChipCtlGroup * c->groups;
        }
      }
    }
  }
  return found;
}
size_t lz_chip_bytes(const LzChip& c) {
  const size_t rec = size_t(c.groups) * 4 * c.G * c.rec_stride * 8, ring = size_t(c.groups) * 16 * c.G * c.nx * 8;
  return (c.G > 1 ? ring + rec : 0) + size_t(c.ctl_words) * 4 + 1024;
}
// Lays the mailboxes out in mem (256-byte aligned) and empties them.
void lz_chip_mailboxes(LzChip& c, void* mem, hipStream_t s) {
  const size_t rec = (size_t(c.groups) * 4 * c.G * c.rec_stride * 8 + 255) / 256 * 256;
  const size_t ring = size_t(c.groups) * 16 * c.G * c.nx * 8;
  char* p = static_cast<char*>(mem);
  c.ctl = reinterpret_cast<int*>(p);
  p += (size_t(c.ctl_words) * 4 + 255) / 256 * 256;
  c.rec = reinterpret_cast<unsigned long long*>(p);
  c.ring = reinterpret_cast<unsigned long long*>(p + rec);
  if (c.G == 1) return;
  double none;
  memset(&none, 0xff, sizeof(none));
  launch_fill_value(reinterpret_cast<double*>(c.rec), (rec + ring) / 8, none, s);
}
void launch_lz_chip(const LzChip& c, hipStream_t s) {
  hipLaunchKernelGGL(k_lz_ctl, dim3(1), dim3(256), 0, s, c.ctl, c.ctl_words, c.flag);
  hipLaunchKernelGGL(c.H ? lz_chip_fn<true>(c.rt) : lz_chip_fn<false>(c.rt), dim3(c.groups * c.G), dim3(c.nt), c.lds, s,
                     c);
}

size_t lz_small_bytes(int m, int nb) {
  return size_t(nb) * 64 * m * sizeof(double2) + size_t(nb) * m * sizeof(double) + 512;
}
void launch_lz_small(const double* b, int m, double t, const LzPair* pairs, int npair, int nb, void* scratch, double* y,
                     double* coef, double* out, hipStream_t s) {
  double2* inv = static_cast<double2*>(scratch);
  double* part = reinterpret_cast<double*>(inv + size_t(nb) * 64 * m);
  for (int q = 0; q < npair; q += 64 * nb) {
    const int left = npair - q, blocks = std::min(nb, (left + 63) / 64);
    hipLaunchKernelGGL(k_lz_small, dim3(blocks), dim3(64), 0, s, b, m, t, pairs + q, left, inv, part, q > 0 ? 1 : 0);
  }
  hipLaunchKernelGGL(k_lz_ysum, dim3(1), dim3(1024), 0, s, part, nb, m, b, y, coef, out);
}

}  // namespace rexii
