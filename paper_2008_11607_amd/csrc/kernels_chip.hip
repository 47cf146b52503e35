// COCG inner iterations of the slot engine with the solve held on the chip.
//
// The pass kernels (kernels.hip) stream r, p and d of every live slot through
// HBM once per step.  Here a group of G blocks takes one slot at a time and
// runs up to K inner steps with r, d and q = K p in registers and p in LDS,
// so that a step moves only the strips' edge rows and one record of sums
// per block.  The stencil has stride 2, so rows of one parity form periodic
// chains of their own (two of length ny / 2 for even ny, one of length ny
// for odd ny); a strip is a run of chain rows, and its halo is one chain row
// on either side.
//
// One step, with alpha, beta from the previous one (the recurrences and the
// summation formulas of the pass kernels):
//   d += alpha p, r -= alpha q, p = r + beta p     own points, and r, p of
//                                                  the two ring rows (their q
//                                                  comes from the neighbours)
//   q = (L - zeta) p and the nine partial sums
//   post q of the strip's edge rows, then the block's sums; wait for the
//   sums of all G blocks; alpha, beta, stop test (every block by itself)
// so a step waits once for the other blocks.
//
// Bound: VALU issue (44 instructions a point and step and 280 a wavefront in
// FP32, 42 and 240 in FP64, counted) plus one exchange between the blocks a
// step: 1.8 us a step for 64^2 in FP64 (one block, no exchange), 4.5 us for
// 256^2 in FP64 (16 blocks of one XCD), 5.8 us for 512^2 in FP32 (32 blocks),
// 7.5 us for 512^2 in FP64 (64 blocks across XCDs), and 15 to 60 us a launch;
// 1.9 and 3.3 us of the middle two are VALU.  Measured whole calls, passes ->
// chip: 64^2 t rho 100 FP64 7.3 -> 1.3 ms, 130 x 66 with velocities t rho 150
// 55 -> 12.8 ms, 256^2 t rho 300 FP64 241 to 274 -> 77 to 79 ms, 512^2 t rho
// 250 mixed, tol 1e-7 513 to 537 -> 210 to 214 ms (the passes run at 5.5 TB/s
// of HBM there, and end their last rounds earlier).  Tried and left out: two
// blocks of 256 threads a CU (10 to 25% slower), four wavefronts a SIMD at 128
// registers (spills), the edge rows' state in LDS (3 to 6% slower), sleeps in
// the waits and raised wave priority (no change).
//
// Communication between the blocks of a group: agent-scope stores and loads.
// A mailbox word (a sum of a block's record, or part of an edge value) holds
// kNoWord until it is posted, so a reader needs no flag beside it.  Records
// and edge rows use three buffers in turn: a block puts kNoWord back into
// what it posted in sync i once it has every record of sync i + 1 (all have
// read the words of i by then) and before it posts its record of i + 2, and
// nobody looks for the words of i + 3 before it has the record of i + 2.
//
// Waits end: a group starts only when all its blocks are on the chip (its
// members are taken in the order in which blocks start, and no other launch
// of this kind runs beside it), and every wait counts its polls and gives up
// past a limit, a group that has not started by cancelling itself (its slots
// run in the next launch).
#include <climits>

#include "kernels.h"
#include "chip_sync.h"

namespace rexii {

namespace {

// Sums of v[0..9) over each row of 16 lanes, to dst[0..9) of the row (in
// LDS).  FP32: nine trees of four DPP adds.  FP64 moves two registers a
// step, so lanes share the nine values out: after the steps over lane bits
// 0, 1 and 2 a lane holds the value of those three bits and the ninth.
__device__ __forceinline__ void row_sums(float (&v)[kNDots], double* dst) {
#pragma unroll
  for (int k = 0; k < kNDots; ++k) {
    v[k] += dpp_f32<0xb1, 0xf>(v[k]);
    v[k] += dpp_f32<0x4e, 0xf>(v[k]);
    v[k] += dpp_f32<0x124, 0xf>(v[k]);
    v[k] += dpp_f32<0x128, 0xf>(v[k]);
  }
  if ((threadIdx.x & 15) == 0) {
#pragma unroll
    for (int k = 0; k < kNDots; ++k) dst[k] = double(v[k]);
  }
}
__device__ __forceinline__ void row_sums(double (&v)[kNDots], double* dst) {
  const int lane = int(threadIdx.x);
  const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
  double u[4], w[2], n = v[8] + dpp_f64<0xb1, 0xf>(v[8]);
#pragma unroll
  for (int k = 0; k < 4; ++k) u[k] = (b0 ? v[k + 4] : v[k]) + dpp_f64<0xb1, 0xf>(b0 ? v[k] : v[k + 4]);
#pragma unroll
  for (int k = 0; k < 2; ++k) w[k] = (b1 ? u[k + 2] : u[k]) + dpp_f64<0x4e, 0xf>(b1 ? u[k] : u[k + 2]);
  n += dpp_f64<0x4e, 0xf>(n);
  double x = (b2 ? w[1] : w[0]) + dpp_f64<0x124, 0xf>(b2 ? w[0] : w[1]);
  n += dpp_f64<0x124, 0xf>(n);
  x += dpp_f64<0x128, 0xf>(x);
  n += dpp_f64<0x128, 0xf>(n);
  if ((lane & 8) == 0) dst[(lane & 1) * 4 + (lane & 2) + ((lane >> 2) & 1)] = x;
  if ((lane & 15) == 8) dst[8] = n;
}

struct ChipCtl {       // in LDS: what one thread or wavefront tells the block
  double2 al, be, rr;  // wavefront 0: alpha and beta of the next step, r^T r
  int act;             // 1: the inner solve has ended
  int bad;             // a wait gave up
  int slot;
};

}  // namespace

// Threads own columns: item j of thread t is column-segment t + j NT of the
// block's nx x (Sc cpb), rows j0 .. j0 + cnt - 1 of its chain with
// cnt = RT or RT - 1.  In LDS an item's rows lie together (pitch RT or
// RT + 1, odd), so that a row is an immediate offset from the item's place
// and lanes fall into different banks.
//
// The operator is scaled by 1 / cx: q = K p / cx, so alpha is cx times the
// alpha of K, and d is updated with alpha / cx.
template <typename T, int Q, int RT>
__device__ __forceinline__ void chip_run(const Eng& e, const Chip& c, unsigned char* lds_raw) {
  using V = typename C2<T>::t;
  constexpr int kRows = sizeof(T) == 4 ? 4 : 2;  // rows whose LDS reads are in flight together
  constexpr int kGr = (RT + kRows - 1) / kRows;
  constexpr int PR = chip_pitch(RT);
  __shared__ double red[64 * kNDots];  // sums of the rows of 16 lanes
  __shared__ ChipCtl ctl;
  V* P = reinterpret_cast<V*>(lds_raw);
  const int tid = int(threadIdx.x), nt = int(blockDim.x);
  const int lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = nt >> 6;
  const int nx = c.nx, ny = c.ny, L = c.L, G = c.G;

  // ---- group formation: groups fill in the order in which blocks start
  int gid = int(blockIdx.x), rank = 0;
  int* gc = nullptr;
  const bool local = c.gpx > 0;
  if (tid == 0) ctl.bad = 0;
  if (G > 1) {
    GroupPlace gp;
    bool late = false;
    if (!join_group(c.ctl, G, c.gpx, INT_MAX, c.waits, reinterpret_cast<int*>(red), gp, late)) {
      if (late && tid == 0) atomicOr(&e.counter[2], kChipLate);
      return;
    }
    gid = gp.gid;
    rank = gp.rank;
    gc = c.ctl + kChipCtlHead + gid * kChipCtlGroup;
  }
  // ---- geometry of the block's strip and of the thread's items
  const bool ringed = c.Gc > 1;
  const int ch0 = (G == 1) ? 0 : rank / c.Gc;         // first chain of the block
  const int strip = (G == 1) ? 0 : rank - ch0 * c.Gc;
  const int ja = int((long long)strip * L / c.Gc);     // chain rows ja .. jb - 1
  const int R = int((long long)(strip + 1) * L / c.Gc) - ja;
  const int segs = c.Sc * ((G == 1) ? c.nch : 1);
  int base[Q], left[Q], right[Q], top[Q], bot[Q], grow[Q], col[Q];
  bool valid[Q], full[Q], rtop[Q], rbot[Q];
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    const int ci = tid + j * nt;
    const int s = ci / nx;
    valid[j] = s < segs;
    const int cx_ = valid[j] ? ci - s * nx : 0;
    const int sv = valid[j] ? s : 0;
    const int cl = sv / c.Sc, k = sv - cl * c.Sc;      // local chain, segment in it
    auto first_row = [&](int q) { return int((long long)q * R / c.Sc); };
    const int r0 = first_row(k);
    full[j] = first_row(k + 1) - r0 == RT;
    col[j] = cx_;
    const int row0 = sv * nx;                          // item of column 0
    base[j] = (row0 + cx_) * PR;
    left[j] = (row0 + ((cx_ >= 2) ? cx_ - 2 : cx_ - 2 + nx)) * PR;
    right[j] = (row0 + ((cx_ + 2 < nx) ? cx_ + 2 : cx_ + 2 - nx)) * PR;
    rtop[j] = valid[j] && ringed && k == 0;
    rbot[j] = valid[j] && ringed && k == c.Sc - 1;
    const int ku = (k == 0) ? c.Sc - 1 : k - 1, kd = (k == c.Sc - 1) ? 0 : k + 1;
    top[j] = ((cl * c.Sc + ku) * nx + cx_) * PR + first_row(ku + 1) - first_row(ku) - 1;
    bot[j] = ((cl * c.Sc + kd) * nx + cx_) * PR;
    grow[j] = (ch0 + cl) + 2 * (ja + r0);              // grid row before the wrap
  }
  auto gaddr = [&](int gr0, int cj, int i) {           // grid point of row i (i = -1 .. RT) of an item
    int y = gr0 + 2 * i;
    y = (y < 0) ? y + ny : y;
    y = (y >= ny) ? y - ny : y;
    y = (y >= ny) ? y - ny : y;
    return unsigned(y * nx + cj);
  };
  // mailboxes of the group: records [3][G][kChipRec], edge rows [3][G][2][nx]
  unsigned long long* rec = c.rec + size_t(gid) * 3 * G * kChipRec;
  V* ring = reinterpret_cast<V*>(c.ring) + size_t(gid) * 3 * G * 2 * nx;
  const int up_rank = ch0 * c.Gc + ((strip == 0) ? c.Gc - 1 : strip - 1);
  const int dn_rank = ch0 * c.Gc + ((strip + 1 == c.Gc) ? 0 : strip + 1);

  unsigned sync_no = 0;   // syncs done so far, over all slots
  unsigned seq = 0;       // slots taken so far
  for (;;) {
    // ---- the group's next slot
    if (tid == 0) {
      int s = -1;
      if (rank == 0) {
        for (;;) {
          const int i = __hip_atomic_fetch_add(&c.ctl[1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (i >= e.B) break;
          if (ldc(&e.slots[i].status) == kInner) {
            s = i;
            break;
          }
        }
        if (G > 1)
          ast(reinterpret_cast<unsigned long long*>(gc + 4),
              (static_cast<unsigned long long>(seq + 1) << 32) | unsigned(s + 1));
      } else {
        unsigned n = 0;
        unsigned long long w;
        while (unsigned((w = ald(reinterpret_cast<unsigned long long*>(gc + 4))) >> 32) != seq + 1) {
          if (++n > c.waits.run_polls) {
            ctl.bad = 1;
            break;
          }
        }
        s = int(unsigned(w)) - 1;
      }
      ctl.slot = s;
    }
    __syncthreads();
    const int slot = uni(ctl.slot);
    if (uni(ctl.bad) != 0) {
      if (tid == 0) atomicOr(&e.counter[2], kChipGaveUp);
      return;
    }
    if (slot < 0) break;
    ++seq;
    const Slot* S = &e.slots[slot];
    const SlotWords sw(S);
    const int par = sw.i32(SLOT_OFF(parity));
    const int it0 = sw.i32(SLOT_OFF(it_inner)), itt0 = sw.i32(SLOT_OFF(it_total));
    const int rounds = sw.i32(SLOT_OFF(rounds)), max_it = sw.i32(SLOT_OFF(max_it));
    const double in_tol2 = sw.f64(SLOT_OFF(in_tol2));
    const double cx64 = sw.f64(SLOT_OFF(cx)), icx = 1.0 / cx64;
    const double2 zeta64 = sw.c64(SLOT_OFF(zeta));
    double2 al64 = sw.c64(SLOT_OFF(alpha)), be64 = sw.c64(SLOT_OFF(beta)), rr64 = make_double2(0.0, 0.0);
    al64.x *= cx64;
    al64.y *= cx64;
    const V nzeta = mk<V>(-zeta64.x * icx, -zeta64.y * icx);
    const T ry = T(sw.f64(SLOT_OFF(cy)) * icx);
    const size_t sb = size_t(slot) * e.cap;
    V* gr = reinterpret_cast<V*>(par ? e.r1 : e.r0) + sb;
    V* gp = reinterpret_cast<V*>(par ? e.p1 : e.p0) + sb;
    V* gd = reinterpret_cast<V*>(e.d) + sb;
    // ---- the slot's vectors: r, d in registers, p in LDS
    V r[Q][RT], d[Q][RT], q[Q][RT];
    V rt[Q], rb[Q], pt[Q], pb[Q];   // ring rows (first and last segment of a strip)
    const bool first = it0 == 0, fold = first && rounds >= 2;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      rt[j] = rb[j] = pt[j] = pb[j] = zero2<V>();
      const int gr0 = fresh(grow[j]), cj = fresh(col[j]), bj = fresh(base[j]);
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        if (i % kRows == 0) asm volatile("" ::: "memory");
        r[j][i] = d[j][i] = q[j][i] = zero2<V>();
        if (valid[j] && (i < RT - 1 || full[j])) {
          const unsigned g = gaddr(gr0, cj, i);
          r[j][i] = gr[g];
          P[bj + i] = gp[g];
          if (fold) {
            const V dv = gd[g];
            double2 xv = e.x64[sb + g];
            xv.x += double(dv.x);
            xv.y += double(dv.y);
            e.x64[sb + g] = xv;
          }
          if (!first) d[j][i] = gd[g];
        }
      }
      if (rtop[j]) {
        const unsigned g = gaddr(gr0, cj, -1);
        rt[j] = gr[g];
        pt[j] = gp[g];
      }
      if (rbot[j]) {
        const unsigned g = gaddr(gr0, cj, full[j] ? RT : RT - 1);
        rb[j] = gr[g];
        pb[j] = gp[g];
      }
    }
    __syncthreads();
    int steps = 0, act = 0;
    for (;;) {
      // ---- q = (L - zeta) p / cx and the sums
      const unsigned buf = sync_no % 3u, obuf = (sync_no + 2u) % 3u;
      T a[kNDots];
#pragma unroll
      for (int k = 0; k < kNDots; ++k) a[k] = T(0);
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        if (!valid[j]) continue;
        // (the LDS reads are in bounds for every item: a select, no branch)
        const V lt = P[top[j]], lb = P[bot[j]];
        V up = sel(rtop[j], pt[j], lt);
        const V hb = sel(rbot[j], pb[j], lb);
        V cur = P[base[j]];
        V we[2][kRows], ea[2][kRows], so[2][kRows];
        auto fetch = [&](int g) {
#pragma unroll
          for (int u = 0; u < kRows; ++u) {
            const int i = g * kRows + u;
            if (i >= RT) break;
            we[g & 1][u] = P[left[j] + i];
            ea[g & 1][u] = P[right[j] + i];
            if (i < RT - 1) so[g & 1][u] = P[base[j] + i + 1];
          }
        };
        fetch(0);
#pragma unroll
        for (int g = 0; g < kGr; ++g) {
          if (g + 1 < kGr) fetch(g + 1);
          asm volatile("" ::: "memory");
#pragma unroll
          for (int u = 0; u < kRows; ++u) {
            const int i = g * kRows + u;
            if (i >= RT) break;
            const V w = we[g & 1][u], x = ea[g & 1][u];
            const V nxt = (i == RT - 1) ? hb : (i == RT - 2 ? sel(full[j], so[g & 1][u], hb) : so[g & 1][u]);
            V v;
            v.x = fma1(ry, fma1(T(-2), cur.x, nxt.x + up.x), fma1(T(-2), cur.x, x.x + w.x));
            v.y = fma1(ry, fma1(T(-2), cur.y, nxt.y + up.y), fma1(T(-2), cur.y, x.y + w.y));
            v = cfma(nzeta, cur, v);
            if (i == RT - 1) {
              v = sel(full[j], v, zero2<V>());
              cur = sel(full[j], cur, zero2<V>());
            }
            const V rv = r[j][i];
            // (fused by hand: left to the compiler each of these costs a
            // product and a sum more)
            a[0] = fms(cur.x, v.x, cur.y, v.y, a[0]);
            a[1] = fma2(cur.x, v.y, cur.y, v.x, a[1]);
            a[2] = fms(v.x, rv.x, v.y, rv.y, a[2]);
            a[3] = fma2(v.x, rv.y, v.y, rv.x, a[3]);
            a[4] = fms(v.x, v.x, v.y, v.y, a[4]);
            a[5] = fma1(v.x, v.y, a[5]);
            a[6] = fms(rv.x, rv.x, rv.y, rv.y, a[6]);
            a[7] = fma1(rv.x, rv.y, a[7]);
            a[8] = fma2(rv.x, rv.x, rv.y, rv.y, a[8]);
            // formed here, not sunk to a later use (with the operands of
            // every row kept until then)
            pin(v.x);
            pin(v.y);
            q[j][i] = v;
            up = cur;
            cur = nxt;
          }
#pragma unroll
          for (int k = 0; k < kNDots; ++k) pin(a[k]);
        }
      }
      // ---- post the edge rows, then the block's sums
      if (G > 1) stores_done();  // the words emptied after the last sync
      if (ringed) {
        V* rtx = ring + (size_t(buf) * G + rank) * 2 * nx;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          if (rtop[j]) post(rtx + col[j], q[j][0], local);
          if (rbot[j]) post(rtx + nx + col[j], sel(full[j], q[j][RT - 1], q[j][RT - 2]), local);
        }
      }
      row_sums(a, red + (tid >> 4) * kNDots);
      __syncthreads();
      if (wid == 0) {
        // block sums: lane 4 k + j adds sum k of the rows of lanes 16 j of
        // every wavefront, then the four lanes of a sum
        double v = 0.0;
        const int k = lane >> 2;
        if (k < kNDots)
          for (int w = 0; w < nw; ++w) v += red[(4 * w + (lane & 3)) * kNDots + k];
        v = quad_sum(v);
        if (G > 1 && k < kNDots && (lane & 3) == 0) post(rec + (size_t(buf) * G + rank) * kChipRec + k, v, local);
        red[lane] = v;
      }
      // the neighbours' edge rows: first look
      V qt[Q], qb[Q];
      const V* rrx = ring + size_t(buf) * G * 2 * nx;
      const V* rup = rrx + size_t(up_rank) * 2 * nx + nx;
      const V* rdn = rrx + size_t(dn_rank) * 2 * nx;
      if (ringed) {
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          qt[j] = qb[j] = zero2<V>();
          if (rtop[j]) qt[j] = take(rup + col[j]);
          if (rbot[j]) qb[j] = take(rdn + col[j]);
        }
      }
      if (wid == 0) {
        double v = 0.0;
        if (G > 1) {
          // the group's sums: lane 4 k + j adds sum k of blocks j, j + 4, ...
          const int k = min(lane >> 2, kNDots - 1);
          for (int g0 = 0; g0 < G; g0 += 32) {
            const unsigned long long* theirs = rec + (size_t(buf) * G + g0) * kChipRec + k;
            unsigned long long w[8];
            unsigned n = 0;
            for (;;) {
              bool have = true;
#pragma unroll
              for (int u = 0; u < 8; ++u) {
                const int b = 4 * u + (lane & 3);
                w[u] = (g0 + b < G) ? ald(theirs + size_t(b) * kChipRec) : 0ull;
              }
#pragma unroll
              for (int u = 0; u < 8; ++u) have = have && w[u] != kNoWord;
              if (__all(have)) break;
              if (++n > c.waits.run_polls) {
                ctl.bad = 1;
                break;
              }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) v += __longlong_as_double((long long)w[u]);
          }
          v = quad_sum(v);
        } else {
          v = red[lane];
        }
        // alpha and beta of the next step, or the end of the inner solve:
        // with w = 1 / (p^T q), alpha = r^T r w and
        // beta = 1 - 2 q^T r w + (q^T q w) (r^T r w)
        int act0 = 0;
        if (steps > 0) {
          const double2 pq = make_double2(lane_value(v, 0), lane_value(v, 4));
          const double2 qr = make_double2(lane_value(v, 8), lane_value(v, 12));
          const double2 qq = make_double2(lane_value(v, 16), 2.0 * lane_value(v, 20));
          const double2 rr = make_double2(lane_value(v, 24), 2.0 * lane_value(v, 28));
          const double n2 = lane_value(v, 32);
          const bool good = __all(lane >= 4 * kNDots || isfinite(v)) && (fabs(pq.x) + fabs(pq.y) > 0.0) &&
                            (fabs(rr.x) + fabs(rr.y) > 0.0);
          rr64 = rr;
          if (!good || n2 <= in_tol2 || itt0 + steps >= max_it) {
            act0 = 1;
          } else {
            const double iden = 1.0 / (pq.x * pq.x + pq.y * pq.y);
            const double2 w = make_double2(pq.x * iden, -pq.y * iden);
            const double2 al = cmul(rr, w), bq = cmul(cmul(qq, w), al), br = cmul(qr, w);
            al64 = al;
            be64 = make_double2(1.0 - 2.0 * br.x + bq.x, bq.y - 2.0 * br.y);
          }
        }
        if (lane == 0) {
          ctl.al = al64;
          ctl.be = be64;
          ctl.act = act0;
        }
      }
      if (ringed) {
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          unsigned n = 0;
          while (rtop[j] && !there(qt[j])) {
            qt[j] = take(rup + col[j]);
            if (++n > c.waits.run_polls) {
              ctl.bad = 1;
              break;
            }
          }
          while (rbot[j] && !there(qb[j])) {
            qb[j] = take(rdn + col[j]);
            if (++n > c.waits.run_polls) {
              ctl.bad = 1;
              break;
            }
          }
        }
      }
      __syncthreads();
      ++sync_no;
      if (G > 1) {
        // everybody has read the words posted in the sync before: empty them
        if (tid < kNDots) mst(rec + (size_t(obuf) * G + rank) * kChipRec + tid, kNoWord, local);
        if (ringed) {
          V* rtx = ring + (size_t(obuf) * G + rank) * 2 * nx;
#pragma unroll
          for (int j = 0; j < Q; ++j) {
            if (rtop[j]) empty(rtx + col[j], local);
            if (rbot[j]) empty(rtx + nx + col[j], local);
          }
        }
        if (uni(ctl.bad) != 0) {
          act = 2;
          break;
        }
      }
      act = uni(ctl.act);
      if (act != 0 || steps >= c.K) break;
      ++steps;
      // ---- the next step's vectors
      const double2 au = uni(ctl.al), bu = uni(ctl.be);
      const V nal = mk<V>(-au.x, -au.y), be = mk<V>(bu.x, bu.y);
      const V ad = mk<V>(au.x * icx, au.y * icx);
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        if (!valid[j]) continue;
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          if (i % kRows == 0) asm volatile("" ::: "memory");
          if (i < RT - 1 || full[j]) {
            const V pc = P[base[j] + i];
            d[j][i] = cfma(ad, pc, d[j][i]);
            r[j][i] = cfma(nal, q[j][i], r[j][i]);
            pin(d[j][i].x);
            pin(d[j][i].y);
            P[base[j] + i] = cfma(be, pc, r[j][i]);
          }
        }
      }
      if (ringed) {
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          rt[j] = cfma(nal, qt[j], rt[j]);
          pt[j] = cfma(be, pt[j], rt[j]);
          rb[j] = cfma(nal, qb[j], rb[j]);
          pb[j] = cfma(be, pb[j], rb[j]);
        }
      }
      __syncthreads();
    }
    if (act == 2) {
      if (tid == 0) atomicOr(&e.counter[2], kChipGaveUp);
      return;
    }
    // ---- back to memory: d, and r and p if the inner solve goes on
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      if (!valid[j]) continue;
      const int gr0 = fresh(grow[j]), cj = fresh(col[j]), bj = fresh(base[j]);
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        if (i % kRows == 0) asm volatile("" ::: "memory");
        if (i < RT - 1 || full[j]) {
          const unsigned g = gaddr(gr0, cj, i);
          gd[g] = d[j][i];
          if (act == 0) {
            gr[g] = r[j][i];
            gp[g] = P[bj + i];
          }
        }
      }
    }
    if (rank == 0 && tid == 0) {
      Slot* Z = &e.slots[slot];
      Z->it_inner = it0 + steps;
      Z->it_total = itt0 + steps;
      Z->visits = ldc(&Z->visits) + 1;
      Z->chip_its = ldc(&Z->chip_its) + steps;
      Z->alpha = make_double2(al64.x * icx, al64.y * icx);
      Z->beta = be64;
      Z->dcp = Z->alpha;   // should the passes take the next step: d += alpha p
      if (steps > 0) Z->rr = rr64;
      if (act == 1) Z->status = kInnerDone;
    }
    __syncthreads();
  }
  // ---- leave the group's mailboxes empty for the next launch, once every
  // block has read the last words
  if (G > 1) {
    stores_done();
    __syncthreads();
    if (tid == 0) {
      __hip_atomic_fetch_add(&gc[2], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      unsigned n = 0;
      while (ldc(&gc[2]) < G) {
        if (++n > c.waits.run_polls) {
          atomicOr(&e.counter[2], kChipGaveUp);
          break;
        }
      }
    }
    __syncthreads();
    if (tid < 3 * kChipRec) ast(rec + (size_t(tid / kChipRec) * G + rank) * kChipRec + tid % kChipRec, kNoWord);
    if (ringed)
      for (int k = tid; k < 6 * nx; k += nt) empty(ring + (size_t(k / (2 * nx)) * G + rank) * 2 * nx + k % (2 * nx), false);
  }
}
template <typename T, int Q, int RT, int NT, int W>
__global__ __launch_bounds__(NT, W) void k_chip(Eng e, Chip c) {
  extern __shared__ __attribute__((aligned(16))) unsigned char chip_lds[];
  chip_run<T, Q, RT>(e, c, chip_lds);
}

namespace {

struct ChipFn {
  ChipVariant v;
  void (*fn)(Eng, Chip);
};
#define CHIP(T, Q, RT, NT, W) {{Q, RT, NT}, k_chip<T, Q, RT, NT, W>}
// 512 threads leave 256 registers a thread; r, d and q take 6 (FP32) or 12
// (FP64) a point, so 23 or 8 rows of one column.  Two columns a thread (Q = 2)
// serve rows of 513 to 1024 points, which one column of 512 threads cannot
// hold, and 512^2, where 8 rows of two columns put a solve on 32 blocks as 16
// rows of one do: only the FP32 shape of 8 rows was built, so grids of more
// than 512 columns with more than 512 rows (64 blocks), and every FP64 grid
// past 512 columns, are streamed.
const ChipFn kChipF32[] = {
    CHIP(float, 1, 2, 512, 2),
    CHIP(float, 1, 3, 512, 2),
    CHIP(float, 1, 4, 512, 2),
    CHIP(float, 1, 5, 512, 2),
    CHIP(float, 1, 6, 512, 2),
    CHIP(float, 1, 7, 512, 2),
    CHIP(float, 1, 8, 512, 2),
    CHIP(float, 1, 9, 512, 2),
    CHIP(float, 1, 10, 512, 2),
    CHIP(float, 1, 11, 512, 2),
    CHIP(float, 1, 12, 512, 2),
    CHIP(float, 1, 13, 512, 2),
    CHIP(float, 1, 14, 512, 2),
    CHIP(float, 1, 15, 512, 2),
    CHIP(float, 1, 16, 512, 2),
    CHIP(float, 1, 17, 512, 2),
    CHIP(float, 1, 18, 512, 2),
    CHIP(float, 1, 19, 512, 2),
    CHIP(float, 1, 20, 512, 2),
    CHIP(float, 1, 21, 512, 2),
    CHIP(float, 1, 22, 512, 2),
    CHIP(float, 1, 23, 512, 2),
    CHIP(float, 2, 8, 512, 2),
};
const ChipFn kChipF64[] = {
    CHIP(double, 1, 2, 512, 2),
    CHIP(double, 1, 3, 512, 2),
    CHIP(double, 1, 4, 512, 2),
    CHIP(double, 1, 5, 512, 2),
    CHIP(double, 1, 6, 512, 2),
    CHIP(double, 1, 7, 512, 2),
    CHIP(double, 1, 8, 512, 2),
};
#undef CHIP
const ChipFn& chip_fn(int is_f32, int k) { return is_f32 ? kChipF32[k] : kChipF64[k]; }

}  // namespace

int chip_variants(int is_f32) {
  return int(is_f32 ? sizeof(kChipF32) / sizeof(kChipF32[0]) : sizeof(kChipF64) / sizeof(kChipF64[0]));
}
ChipVariant chip_variant(int is_f32, int k) { return chip_fn(is_f32, k).v; }
int chip_occupancy(int is_f32, int k, int nt, int lds) {
  const void* f = reinterpret_cast<const void*>(chip_fn(is_f32, k).fn);
  if (lds > 48 * 1024 && hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kChipMaxLds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  int occ = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, f, nt, lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return occ;
}
void launch_chip(const Eng& e, const Chip& c, hipStream_t s) {
  hipLaunchKernelGGL(chip_fn(e.d_is_f32, c.variant).fn, dim3(c.ngroups * c.G), dim3(c.nt), c.lds, s, e, c);
}

}  // namespace rexii
