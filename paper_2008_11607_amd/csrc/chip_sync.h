// Words that blocks of one launch exchange while they run, and small helpers
// of the kernels that keep a solve on the chip (kernels_chip.hip,
// kernels_lz.hip).  A mailbox word holds kNoWord until it is posted.
#ifndef REXII_CHIP_SYNC_H
#define REXII_CHIP_SYNC_H

#include "device_util.h"

namespace rexii {

constexpr unsigned long long kNoWord = ~0ull;   // a NaN pattern no sum produces
// Polls for a word of a running group, seconds (it is microseconds away): ends
// what cannot go on.  k_lz_chip takes the constant (as a launch parameter it
// cost 1.6% at 512^2, as 2^20 or 2^22 2 to 8%), k_chip the launch parameter
// (the constant cost 4% at 256^2 in FP64): the code around the waits differs.
constexpr unsigned kRunPolls = 1u << 23;

__device__ __forceinline__ unsigned long long ald(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ast(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Mailbox stores.  A group on one XCD shares its L2: L1 is write-through and
// the readers' agent-scope loads pass their L1, so a store that goes no
// further than L2 is enough (a sync with 2 x 512 edge words, 32 blocks:
// 1.95 us against 3.07 us with stores through to memory).
__device__ __forceinline__ void mst(unsigned long long* p, unsigned long long v, bool local) {
  if (local)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void post(float2* p, float2 v, bool local) {
  mst(reinterpret_cast<unsigned long long*>(p),
      (static_cast<unsigned long long>(__float_as_uint(v.y)) << 32) | __float_as_uint(v.x), local);
}
__device__ __forceinline__ void post(double2* p, double2 v, bool local) {
  mst(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v.x), local);
  mst(reinterpret_cast<unsigned long long*>(p) + 1, (unsigned long long)__double_as_longlong(v.y), local);
}
__device__ __forceinline__ float2 take(const float2* p) {
  const unsigned long long w = ald(reinterpret_cast<const unsigned long long*>(p));
  return make_float2(__uint_as_float(unsigned(w)), __uint_as_float(unsigned(w >> 32)));
}
__device__ __forceinline__ double2 take(const double2* p) {
  const unsigned long long* q = reinterpret_cast<const unsigned long long*>(p);
  return make_double2(__longlong_as_double((long long)ald(q)), __longlong_as_double((long long)ald(q + 1)));
}
__device__ __forceinline__ void post(unsigned long long* p, double v, bool local) {
  const unsigned long long w = (unsigned long long)__double_as_longlong(v);
  mst(p, w == kNoWord ? 0x7ff8000000000000ull : w, local);
}
__device__ __forceinline__ void empty(float2* p, bool local) {
  mst(reinterpret_cast<unsigned long long*>(p), kNoWord, local);
}
__device__ __forceinline__ void empty(double2* p, bool local) {
  mst(reinterpret_cast<unsigned long long*>(p), kNoWord, local);
  mst(reinterpret_cast<unsigned long long*>(p) + 1, kNoWord, local);
}
__device__ __forceinline__ bool there(float2 v) {
  return (__float_as_uint(v.x) & __float_as_uint(v.y)) != 0xffffffffu;
}
__device__ __forceinline__ bool there(double2 v) {
  return (unsigned long long)__double_as_longlong(v.x) != kNoWord &&
         (unsigned long long)__double_as_longlong(v.y) != kNoWord;
}
// every earlier store of this wavefront has been acknowledged
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The value, unknown to loop-invariant code motion: addresses formed from it
// are formed at use instead of being kept in registers across the step loop.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

template <typename T>
__device__ __forceinline__ void pin(T& v) {
  asm volatile("" : "+v"(v));
}

template <typename V>
__device__ __forceinline__ V zero2() {
  V v;
  v.x = 0;
  v.y = 0;
  return v;
}
template <typename V>
__device__ __forceinline__ V sel(bool c, V a, V b) {
  V v;
  v.x = c ? a.x : b.x;
  v.y = c ? a.y : b.y;
  return v;
}

__device__ __forceinline__ float fma1(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma1(double a, double b, double c) { return __builtin_fma(a, b, c); }
// c + a b + d e and c + a b - d e
template <typename T>
__device__ __forceinline__ T fma2(T a, T b, T d, T e, T c) {
  return fma1(d, e, fma1(a, b, c));
}
template <typename T>
__device__ __forceinline__ T fms(T a, T b, T d, T e, T c) {
  return fma1(-d, e, fma1(a, b, c));
}
// c + a b, complex
template <typename V>
__device__ __forceinline__ V cfma(V a, V b, V c) {
  V r;
  r.x = fma1(-a.y, b.y, fma1(a.x, b.x, c.x));
  r.y = fma1(a.y, b.x, fma1(a.x, b.y, c.y));
  return r;
}

__device__ __forceinline__ double quad_sum(double v) {
  v += dpp_f64<0xb1, 0xf>(v);
  v += dpp_f64<0x4e, 0xf>(v);
  return v;
}
__device__ __forceinline__ double lane_value(double v, int l) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = unsigned(__builtin_amdgcn_readlane(int(unsigned(b)), l));
  const unsigned hi = unsigned(__builtin_amdgcn_readlane(int(unsigned(b >> 32)), l));
  return __longlong_as_double((long long)((static_cast<unsigned long long>(hi) << 32) | lo));
}

// A block's place among the groups of a launch.  Groups fill in the order in
// which blocks start (of any XCD, or with gpx > 0 of one XCD each, gpx groups
// per XCD): a block waits only for blocks that start as soon as others leave,
// provided that no other launch of this kind holds CUs (the host gives such
// launches of a process one after the other; against another process the
// limit of the wait helps).
// ctl: [8 + x] tickets, then per group at kChipCtlHead + g kChipCtlGroup:
// [0] arrivals, [1] state (0 forming, 1 ready, 2 cancelled).  Returns false
// for a block beyond the groups, for one of a group without work (with
// gpx > 0 group k of XCD x works on item 8 k + x of `items`; the others do
// not wait for each other), for a group that did not fill (late) and for a
// block that is to be dropped.
struct GroupPlace {
  int gid, rank, xcd;
};
__device__ __forceinline__ bool join_group(int* ctl, int G, int gpx, int items, const ChipWaits& waits, int* sh,
                                           GroupPlace& gp, bool& late) {
  if (threadIdx.x == 0) {
    int x = 0;
    if (gpx > 0) asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(x));
    x &= 7;
    const int ticket = __hip_atomic_fetch_add(&ctl[8 + x], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int k = ticket / G;
    const bool over = gpx > 0 && (k >= gpx || 8 * k + x >= items);
    const int g = x * gpx + k;
    int* w = ctl + kChipCtlHead + (over ? 0 : g) * kChipCtlGroup;
    if (!over && __hip_atomic_fetch_add(&w[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == G - 1 &&
        g != waits.late_group)
      atomicCAS(&w[1], 0, 1);
    unsigned n = 0;
    int st = 2, lt = 0;
    while (!over && (st = ldc(&w[1])) == 0) {
      if (++n > waits.form_polls && atomicCAS(&w[1], 0, 2) == 0) lt = 1;
      __builtin_amdgcn_s_sleep(2);
    }
    sh[0] = (waits.run_polls == 0 && ticket - k * G == G - 1) ? 2 : st;
    sh[1] = g;
    sh[2] = ticket - k * G;
    sh[3] = x;
    sh[4] = lt;
  }
  __syncthreads();
  const bool ok = uni(sh[0]) == 1;
  gp.gid = uni(sh[1]);
  gp.rank = uni(sh[2]);
  gp.xcd = uni(sh[3]);
  late = uni(sh[4]) != 0;
  __syncthreads();
  return ok;
}

}  // namespace rexii

#endif
