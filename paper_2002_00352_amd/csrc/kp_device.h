// Device helpers shared by the sweep kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "kp_internal.h"

__device__ __forceinline__ int popc64(uint64_t x) { return __popcll(x); }

__device__ __forceinline__ uint64_t dkey(double v) {
  return (uint64_t)__double_as_longlong(v);
}
__device__ __forceinline__ double kdbl(uint64_t k) { return __longlong_as_double((long long)k); }

// Exponential bucket of a breakpoint around the previous multiplier: 0 inside
// (center - delta, center + delta), else sign * (1 + floor(log2(|d| / delta)))
// capped at 31; delta is a power of two, so the log is an exponent difference.
// Monotone non-decreasing in v.
__device__ __forceinline__ int exp_bucket(double v, double center, double delta) {
  double d = v - center;
  double a = fabs(d);
  if (!(a >= delta)) return 0;
  int ea = (int)((dkey(a) >> 52) & 0x7FF);
  int ed = (int)((dkey(delta) >> 52) & 0x7FF);
  int id = 1 + (ea - ed);
  id = id > 31 ? 31 : id;
  return d < 0.0 ? -id : id;
}

// An interval that holds every breakpoint of exponential bucket id (the
// bucket test rounds v - center, by far less than the widening here); the
// outermost buckets are open.
__device__ __forceinline__ void bucket_bounds(double center, double delta, int id, double &lo, double &hi) {
  const int a = id < 0 ? -id : id;
  const double far_ = ldexp(delta, a), near_ = a ? ldexp(delta, a - 1) : 0.0;
  const double slack = (center + far_) * 0x1p-48;
  if (id == 0) { lo = center - far_; hi = center + far_; }
  else if (id > 0) { lo = center + near_; hi = a >= 31 ? INFINITY : center + far_; }
  else { lo = a >= 31 ? 0.0 : center - far_; hi = center - near_; }
  lo = fmax(lo - slack, 0.0);
  hi = fmax(hi + slack, 0.0);
}

// ---- exact sums (XSum) ----
// x = sign (hi 2^-24 + lo 2^-56) with hi = floor(|x| 2^24) and lo the rest in
// units of 2^-56 (|x| < 2^39): s - floor(s) is exact for s >= 0, and the
// scalings by powers of two are exact, so lo is an integer on the grid.
__device__ __forceinline__ void xs_parts(double x, long long &h, long long &l) {
  const double s = fabs(x) * 0x1p24;
  const double f = floor(s);
  const double r = (s - f) * 0x1p32;
  long long hi = (long long)f;
  long long lo = (long long)rint(r);
  if (lo == 0x100000000ll) { lo = 0; hi += 1; }
  if (x < 0.0) { hi = -hi; lo = -lo; }
  h = hi;
  l = lo;
}
__device__ __forceinline__ XSum xs_of(double x) {
  XSum r;
  xs_parts(x, r.hi, r.lo);
  return r;
}
__device__ __forceinline__ XSum xs_plus(XSum a, XSum b) {
  XSum r;
  r.hi = a.hi + b.hi;
  r.lo = a.lo + b.lo;
  return r;
}
__device__ __forceinline__ XSum xs_minus(const XSum &a, const XSum &b) {
  XSum r;
  r.hi = a.hi - b.hi;
  r.lo = a.lo - b.lo;
  return r;
}
__device__ __forceinline__ void xs_add(XSum &a, double x) { a = xs_plus(a, xs_of(x)); }
__device__ __forceinline__ XSum xs_zero() {
  XSum r;
  r.hi = 0;
  r.lo = 0;
  return r;
}
__device__ __forceinline__ bool xs_nonzero(const XSum &a) { return a.hi != 0 || a.lo != 0; }
// Integer adds: the same total whatever order the lanes and blocks add in.
__device__ __forceinline__ void xs_atomic_add_sum(XSum *dst, const XSum &v) {
  if (v.hi) atomicAdd((unsigned long long *)&dst->hi, (unsigned long long)v.hi);
  if (v.lo) atomicAdd((unsigned long long *)&dst->lo, (unsigned long long)v.lo);
}
__device__ __forceinline__ void xs_atomic_add(XSum *dst, double x) { xs_atomic_add_sum(dst, xs_of(x)); }
// The nearest doubles to the parts, added (exact when the total needs no
// more than 53 bits, e.g. on the 2^-24 grid below 2^29).
__device__ __forceinline__ double xs_to_double(const XSum &a) {
  const long long H = a.hi + (a.lo >> 32);
  const long long L = a.lo & 0xFFFFFFFFll;
  const double h = (double)H * 0x1p-24;
  const double l = (double)L * 0x1p-56;
  return h + l;
}
// a > B exactly, for B >= 0 (B's own bits below 2^-56 are kept in the
// comparison).
__device__ __forceinline__ bool xs_gt(const XSum &a, double B) {
  if (!(B < 0x1p38)) return xs_to_double(a) > B;   // outside the exact range (budgets below 2^38)
  const long long H = a.hi + (a.lo >> 32);
  const long long L = a.lo & 0xFFFFFFFFll;
  const double sB = B * 0x1p24;
  const double fB = floor(sB);
  const double rB = (sB - fB) * 0x1p32;
  const long long HB = (long long)fB;
  return H > HB || (H == HB && (double)L > rB);
}

// Non-zero when v >= 0 is off the grid of SweepArgs::gmag / ginv (a sum of
// multiples of the unit g below g 2^53 is exact in FP64); the sweeps OR the
// answers of all they sum and report them at the end.
__device__ __forceinline__ uint32_t off_grid(double v, double gmag) {
  const double up = v + gmag;
  return up - gmag != v ? 1u : 0u;
}
__device__ __forceinline__ uint32_t off_grid(float v, float ginv) {
  return __float_as_uint(__builtin_amdgcn_fractf(v * ginv));
}
__device__ __forceinline__ void report_off_grid(const SweepArgs &a, uint32_t off) {
  if (__ballot(off != 0) && (threadIdx.x & 63) == 0) atomicOr(a.off, 1u);
}

// Bin of a post-processing key: the number of the nb - 1 ascending
// splitters below it.
__device__ __forceinline__ int fx_bin_of(const uint64_t *split, int nb, uint64_t key) {
  int lo = 0, hi = nb - 1;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (split[mid] < key) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Breakpoint arithmetic of the walks.  For lines z_a = c_a - lambda b_a and
// z_b = c_b - lambda b_b with b_a > b_b, the crossing is
// fl(fl(c_a - c_b) / fl(b_a - b_b)) and line a ranks above line b for lambda
// below it; a line's zero crossing is fl(c_a / b_a).  cr_gt decides
// fl(num / den) > t for den > 0 from exact fma residual signs and divides
// only when the quotient lies within one ulp of t, so that the decisions
// agree with the divided crossings bit for bit.
__device__ __forceinline__ bool cr_gt(double num, double den, double t) {   // t >= 0
  const double r = fma(-t, den, num);            // sign of num - t*den, exact
  if (!(r > 0.0)) return false;                  // quotient <= t
  const double up = kdbl(dkey(t) + 1);           // next double above t
  const double r2 = fma(-up, den, num);
  if (r2 >= 0.0) return true;                    // quotient >= up
  return num / den > t;
}
// The laminar sets in LDS, as chains from an item's smallest set up: the
// breakpoint phases look for the innermost full set that holds an item all
// the time, in code where lanes diverge; read from the kernel's arguments
// (scalar loads, each waited for, over all the sets) those looks were most of
// a walk's time.  Up to three sets (top-Q; two groups and a total) are held in
// scalar registers instead: three tests cost less than a chain of dependent
// LDS reads (N = 5e6, M = 10, K = 20, three sets: 9.4 -> 8.4 ms for four
// iterations), and more of them would push the scalar registers out.
struct SetNode {
  uint64_t mask;
  int cap, up;
};
// FEW: how many sets are held in registers.  3 in the lean kernel up to 16
// items; 1 in the others, whose scalar registers already spill (M = 20 with
// 11 sets lost 4 %, batches 1 %; ragged CSR costs gained nothing).
template <int FEW>
struct SetTreeN {
  const SetNode *node;
  const int16_t *first;
  int L;
  int cap[FEW];         // up to that many sets: in registers (scalar ones, the same for every lane)
  uint64_t m[FEW];
  // the members of S in the innermost full set that holds o (0: none is full)
  __device__ __forceinline__ uint64_t circuit(uint64_t S, int o) const {
    if (L <= FEW) {
      uint64_t c = 0;
      #pragma unroll
      for (int l = FEW - 1; l >= 0; --l)   // (subsets come first: the innermost one last)
        if ((m[l] >> o & 1) && popc64(S & m[l]) >= cap[l]) c = S & m[l];
      return c;
    }
    for (int l = first[o]; l >= 0;) {
      const SetNode n = node[l];
      if (popc64(S & n.mask) >= n.cap) return S & n.mask;
      l = n.up;
    }
    return 0;
  }
};
using SetTree = SetTreeN<1>;
__host__ __device__ __forceinline__ size_t set_tree_bytes(int L, int M) {
  return (((size_t)L * sizeof(SetNode) + 15) & ~(size_t)15) + (((size_t)M * 2 + 15) & ~(size_t)15);
}
// Copy T into mem (set_tree_bytes of LDS); the block synchronises afterwards.
template <int FEW = 1>
__device__ __forceinline__ SetTreeN<FEW> set_tree_load(void *mem, const TreeDev &T, int M, int tid, int nthreads) {
  SetNode *n = (SetNode *)mem;
  int16_t *f = (int16_t *)((unsigned char *)mem + (((size_t)T.L * sizeof(SetNode) + 15) & ~(size_t)15));
  for (int l = tid; l < T.L; l += nthreads) { n[l].mask = T.mask[l]; n[l].cap = T.cap[l]; n[l].up = T.up[l]; }
  for (int j = tid; j < M; j += nthreads) f[j] = T.first[j];
  SetTreeN<FEW> t;
  t.node = n;
  t.first = f;
  t.L = T.L;
  #pragma unroll
  for (int l = 0; l < FEW; ++l) {
    t.m[l] = l < T.L ? T.mask[l] : 0ull;
    t.cap[l] = l < T.L ? T.cap[l] : 0;
  }
  return t;
}

// Laminar-matroid greedy over the ranked items: accept an eligible item when
// no node containing it is full.  Equivalent to Alg.1 (both return the unique
// maximum-weight independent set under the strict order (p~ desc, j asc)).
__device__ __forceinline__ uint64_t greedy_mask(const uint8_t *perm, int M, uint64_t eligible,
                                                const SetTree &T) {
  uint64_t S = 0, blocked = 0;
  for (int r = 0; r < M && (eligible & ~blocked); ++r) {
    const int j = perm[r];
    const uint64_t bit = 1ull << j;
    if ((eligible & ~blocked) & bit) {
      S |= bit;
      eligible &= ~bit;
      for (int l = T.first[j]; l >= 0;) {
        const SetNode n = T.node[l];
        if (popc64(S & n.mask) >= n.cap) blocked |= n.mask;
        l = n.up;
      }
    }
  }
  return S;
}

// The same from the kernel's arguments (evaluations: no chains in LDS).
__device__ __forceinline__ uint64_t greedy_mask(const uint8_t *perm, int M, uint64_t eligible,
                                                const TreeDev &T) {
  uint64_t S = 0, blocked = 0;
  for (int r = 0; r < M; ++r) {
    const int j = perm[r];
    const uint64_t bit = 1ull << j;
    if ((eligible & bit) && !(blocked & bit)) {
      S |= bit;
      for (int l = 0; l < T.L; ++l) {
        const uint64_t m = T.mask[l];
        if ((m & bit) && popc64(S & m) >= T.cap[l]) blocked |= m;
      }
    }
  }
  return S;
}

// Bin or emit one breakpoint (v1, v2) of knapsack k according to its search
// mode: the first pass bins every breakpoint into exponential buckets around
// lambda_k^t and emits the central ones; later passes emit one bucket or key
// range, record a bucket's key hull, or bin a key range linearly.  Emitted
// events go to the block's staging region (published by publish_block).
__device__ __forceinline__ void record_event(const SweepArgs &a, const KWalk &ks, int k, double best,
                                             double v2, int mode, XSum *hs, uint32_t *hc,
                                             unsigned long long *hmin, unsigned long long *hmax,
                                             uint32_t *kcnt, uint32_t *kovf, uint32_t *nstage,
                                             int bid) {
  const uint64_t key = dkey(best);
  bool emit = false;
  if (mode == KS_EXP && hs) {
    const int id = exp_bucket(best, ks.center, ks.delta);
    xs_atomic_add(&hs[k * KP_NB + 32 + id], v2);
    atomicAdd(&hc[k * KP_NB + 32 + id], 1u);
    emit = (id >= -KP_CENTRAL_W && id <= KP_CENTRAL_W);
  } else if (mode == KS_EMIT_BUCKET || mode == KS_HULL_BUCKET) {
    if (exp_bucket(best, ks.center, ks.delta) == ks.bstar) {
      atomicMin(&hmin[k], (unsigned long long)key);
      atomicMax(&hmax[k], (unsigned long long)key);
      emit = (mode == KS_EMIT_BUCKET);
    }
  } else if (mode == KS_REFINE) {
    if (hs && key >= ks.klo && key <= ks.khi) {
      const int bin = (int)((key - ks.klo) >> ks.shift);
      xs_atomic_add(&hs[k * KP_NB + bin], v2);
      atomicAdd(&hc[k * KP_NB + bin], 1u);
    }
  } else {  // KS_EMIT_RANGE, KS_WINDOW
    emit = (key >= ks.klo && key <= ks.khi);
    if (emit && mode == KS_EMIT_RANGE) {
      atomicMin(&hmin[k], (unsigned long long)key);
      atomicMax(&hmax[k], (unsigned long long)key);
    }
  }
  if (emit) {
    const uint32_t slot = atomicAdd(nstage, 1u);
    if (slot < a.stage_cap) {
      const size_t e = (size_t)bid * a.stage_cap + slot;
      a.stage_v1[e] = best;
      a.stage_v2[e] = v2;
      a.stage_k[e] = (uint16_t)k;
      atomicAdd(&kcnt[k], 1u);
    } else {
      kovf[k] = 1u;
    }
  }
}

// Does a knapsack in search state m need another pass over its users?
__device__ __forceinline__ bool walk_mode(int m) {
  return m == KS_EXP || m == KS_EMIT_BUCKET || m == KS_HULL_BUCKET || m == KS_REFINE ||
         m == KS_EMIT_RANGE || m == KS_WINDOW;
}

// A knapsack's search state in this pass: sampled passes take the knapsacks
// that search a sample, the others the rest.
__device__ __forceinline__ int pass_mode(const SweepArgs &a, int k) {
  const KState &s = a.st[k];
  if (((s.flags & KS_FLAG_SAMPLE) != 0) != (a.sampled != 0)) return KS_DONE;
  // (a pass without histograms leaves the searches that bin to another one)
  return a.no_hist && (s.mode == KS_EXP || s.mode == KS_REFINE) ? (int)KS_DONE : s.mode;
}

// End of a sweep block: add its histograms to the global ones, reserve space
// for its staged events with one atomic per knapsack and copy them there.
// Every thread of the block calls this.
__device__ __forceinline__ void publish_block(const SweepArgs &a, int K, XSum *hs, uint32_t *hc,
                                              unsigned long long *hmin, unsigned long long *hmax,
                                              uint32_t *kcnt, uint32_t *kpos, uint32_t *kovf,
                                              uint32_t *nstage, int tid, int nthreads, int bid,
                                              const XSum *kcorr = nullptr) {
  for (int t = tid; hc && t < K * KP_NB; t += nthreads) {
    if (hc[t]) {
      xs_atomic_add_sum(&a.hist_sum[t], hs[t]);
      atomicAdd(&a.hist_cnt[t], hc[t]);
    }
  }
  for (int k = tid; k < K; k += nthreads) {
    if (kcnt[k]) kpos[k] = atomicAdd(&a.st[k].n_emit, kcnt[k]);
    if (kovf[k]) atomicOr(&a.st[k].overflow, 1);
    if (kcorr && xs_nonzero(kcorr[k])) xs_atomic_add_sum(&a.st[k].corr, kcorr[k]);
    if (hmin[k] != ~0ull) {
      atomicMin((unsigned long long *)&a.st[k].hull_lo, hmin[k]);
      atomicMax((unsigned long long *)&a.st[k].hull_hi, hmax[k]);
    }
    kcnt[k] = 0u;
  }
  __syncthreads();
  const uint32_t ns = *nstage < a.stage_cap ? *nstage : a.stage_cap;
  for (uint32_t t = tid; t < ns; t += nthreads) {
    const size_t e = (size_t)bid * a.stage_cap + t;
    const int k = a.stage_k[e];
    const uint32_t dst = kpos[k] + atomicAdd(&kcnt[k], 1u);
    if (dst < a.emit_cap) {
      a.emit_v1[(size_t)k * a.emit_cap + dst] = a.stage_v1[e];
      a.emit_v2[(size_t)k * a.emit_cap + dst] = a.stage_v2[e];
    } else {
      atomicOr(&a.st[k].overflow, 1);
    }
  }
}

// Relative tolerance of the decisions taken from moved lines: values computed
// as z - d b differ from the lines that the breakpoint arithmetic uses by a
// few 2^-53 of |z| + (lambda_k + t) b, so what is farther apart than 2^-44 of
// those magnitudes is decided the same way by both.
#define KP_LINE_TOL 0x1p-44

// No moving item of a (user, knapsack) pair is selected at lambda^t (S0 & A
// empty): does none come in at or above tlo?  Items only rise as lambda_k
// falls, so one that is below zero, or below the lowest member of its circuit
// (all of them fixed lines), at tlo has no breakpoint above it.
template <class TR, class ZV, class BV>
__device__ __forceinline__ bool pair_idle(const TR &T, uint64_t A, uint64_t S0, ZV zv, BV bv, double lk, double tlo) {
  const double d = tlo - lk, mt = lk + tlo;
  for (uint64_t m = A; m; m &= m - 1) {
    const int o = __ffsll((long long)m) - 1;
    const double zo = zv(o), bo = bv(o), so = d * bo;
    const double vo = zo - so, to = KP_LINE_TOL * (fabs(zo) + mt * bo);
    if (vo < -to) continue;
    uint64_t circ = T.circuit(S0, o);
    if (!circ) return false;
    for (; circ; circ &= circ - 1) {
      const double zs = zv(__ffsll((long long)circ) - 1);
      if (!(zs - vo > to + KP_LINE_TOL * fabs(zs))) return false;
    }
  }
  return true;
}

// One (user, knapsack) pair of a breakpoint phase: its breakpoints in
// [ks.tlo, ks.thi], from the top.
//
// The state of the walk is the greedy set S; the next breakpoint below is the
// highest crossing of an item outside S with zero (a free item) or with a
// member of the innermost full set that holds it (Alg.1's exchange);
// fma-residual comparisons decide which is highest.  Above every breakpoint S
// is the greedy set T of the items that do not move with k: S0, the one at
// lambda^t, without its moving members and with the best fixed items that
// come in for them.  Where the range has an upper end the walk starts there:
// each moving item, positive at thi, is added to T or exchanged for the
// lowest member of its circuit (the matroid greedy does not depend on the
// order of insertion), and a set that is still the greedy one at tlo has no
// breakpoint in between -- for most pairs these two looks at the moving items
// are all.  Decisions within rounding of a tie are not taken from moved
// lines: such a pair is walked from the top.  (Walking every pair from the
// top in every pass cost 3-4.5 ms a pass of 3e5 users with M = 23, K = 12.)
//
// The two parts are separate functions because most pairs end with the first:
// a wave whose lanes all take the second costs a fraction of one where a few
// lanes do.
//
// A: the items moving with k, zv(j): p~_j, bv(j): item j's cost in k (0
// outside A), rk(r): the item of rank r by (p~ desc, index asc), pos: the
// items with p~ > 0.  Returns 0 when no breakpoint lies in the range (*above:
// a window's consumption just above thi), else the start of the walk: 1 with
// *So the greedy set at thi, 2 with *So the set T above every breakpoint.
template <class TR, class ZV, class BV, class RK>
__device__ __forceinline__ int pair_start(const TR &tr, uint64_t A, uint64_t S0, uint64_t pos, ZV zv, BV bv, RK rk, double lk,
                                          const KWalk &ks, uint64_t *So, double *above_out) {
  const bool window = ks.mode == KS_WINDOW;
  const double tlo = ks.tlo, thi = ks.thi;
  uint64_t T = S0 & ~A;
  {
    // every moving member gone lets at most one fixed item in
    int left = popc64(S0 & A);
    uint64_t cand = pos & ~A & ~S0;
    for (int r = 0; left > 0 && cand; ++r) {
      const int j = rk(r);
      if (!(cand >> j & 1)) continue;
      cand &= ~(1ull << j);
      if (!tr.circuit(T, j)) { T |= 1ull << j; --left; }
    }
  }
  uint64_t S = T;
  bool at = thi < INFINITY;   // S is the greedy set at thi
  if (at) {
    const double d = thi - lk, mt = lk + thi;
    uint64_t cc = 0;           // the circuit that the lowest member below belongs to
    int s1 = -1;
    double v1 = 0.0, z1 = 0.0, b1 = 0.0, t1 = 0.0;
    bool amb = false;          // another, different line within rounding of it
    for (uint64_t m = A; m; m &= m - 1) {
      const int o = __ffsll((long long)m) - 1;
      const double zo = zv(o), bo = bv(o), so = d * bo;
      const double vo = zo - so, to = KP_LINE_TOL * (fabs(zo) + mt * bo);
      if (vo < -to) continue;
      if (!(vo > to)) { at = false; break; }
      const uint64_t circ = tr.circuit(S, o);
      if (!circ) { S |= 1ull << o; continue; }
      if (circ != cc) {
        cc = circ;
        s1 = -1;
        amb = false;
        for (uint64_t c = circ; c; c &= c - 1) {
          const int s = __ffsll((long long)c) - 1;
          const double zs = zv(s), bs = bv(s), ss = d * bs;
          const double vs = zs - ss, ts = KP_LINE_TOL * (fabs(zs) + mt * bs);
          if (s1 >= 0 && zs == z1 && bs == b1) { s1 = s; continue; }   // one line: the higher index is lower
          if (s1 < 0 || vs < v1) {
            amb = s1 >= 0 && v1 - vs <= t1 + ts;
            s1 = s; v1 = vs; z1 = zs; b1 = bs; t1 = ts;
          } else if (vs - v1 <= t1 + ts) {
            amb = true;
          }
        }
      }
      if (zo == z1 && bo == b1) {
        if (o > s1) continue;
      } else {
        const double diff = vo - v1;
        if (fabs(diff) <= to + t1) { at = false; break; }
        if (diff < 0.0) continue;
      }
      if (amb) { at = false; break; }
      S = (S | (1ull << o)) & ~(1ull << s1);
      cc = 0;
    }
    if (!at) S = T;
  }
  if (at) {
    double above = 0.0;
    if (window)
      for (uint64_t m = S & A; m; m &= m - 1) above = above + bv(__ffsll((long long)m) - 1);
    // does any moving item outside S come in at or above tlo?
    const double d = tlo - lk, mt = lk + tlo;
    bool quiet = true;
    uint64_t cc = 0;
    double vmin = 0.0, tmax = 0.0;   // lowest value at tlo over that circuit, largest tolerance
    for (uint64_t m = A & ~S; quiet && m; m &= m - 1) {
      const int o = __ffsll((long long)m) - 1;
      const double zo = zv(o), bo = bv(o), so = d * bo;
      const double vo = zo - so, to = KP_LINE_TOL * (fabs(zo) + mt * bo);
      if (vo < -to) continue;
      const uint64_t circ = tr.circuit(S, o);
      if (!circ) { quiet = false; break; }
      if (circ != cc) {
        cc = circ;
        vmin = INFINITY;
        tmax = 0.0;
        for (uint64_t c = circ; c; c &= c - 1) {
          const int s = __ffsll((long long)c) - 1;
          const double zs = zv(s), bs = bv(s), ss = d * bs;
          vmin = fmin(vmin, zs - ss);
          tmax = fmax(tmax, KP_LINE_TOL * (fabs(zs) + mt * bs));
        }
      }
      if (vmin - vo > to + tmax) continue;
      for (uint64_t c = circ; c; c &= c - 1) {
        const int s = __ffsll((long long)c) - 1;
        const double bs = bv(s);
        if (bs >= bo) continue;   // stays above o all the way down
        const double zs = zv(s), ss = d * bs;
        if (!(zs - ss - vo > to + KP_LINE_TOL * (fabs(zs) + mt * bs))) { quiet = false; break; }
      }
    }
    if (quiet) { *above_out = above; return 0; }
  }
  *So = S;
  return at ? 1 : 2;
}

// The walk of a pair from the set S (at: the greedy set at thi, else the one
// above every breakpoint) down to tlo; emit(v1, v2) takes a breakpoint in the
// range.  *above: a window's consumption just above thi.  Returns false when
// the walk runs past its event limit.
template <class TR, class ZV, class BV, class EM>
__device__ __forceinline__ bool pair_walk(int M, const TR &tr, uint64_t A, uint64_t S, bool at, ZV zv, BV bv, double lk, const KWalk &ks, EM emit,
                                          double *above_out) {
  const bool window = ks.mode == KS_WINDOW;
  const double tlo = ks.tlo, thi = ks.thi;
  double above = 0.0;
  if (at && window)
    for (uint64_t m = S & A; m; m &= m - 1) above = above + bv(__ffsll((long long)m) - 1);
  const int maxev = M * M + M + 8;
  for (int ev = 0;; ++ev) {
    if (ev >= maxev) return false;
    double best = 0.0;
    int bo = -1, bs = -1;
    for (uint64_t cand = A & ~S; cand; cand &= cand - 1) {
      const int o = __ffsll((long long)cand) - 1;
      const double bo_d = bv(o);
      const double add_o = lk * bo_d;
      const double co = zv(o) + add_o;
      uint64_t circ = tr.circuit(S, o);
      // compared with the running maximum through cr_gt: a division only
      // for a crossing that beats it
      if (!circ) {
        if (co > 0.0 && cr_gt(co, bo_d, best)) { best = co / bo_d; bo = o; bs = -1; }
      } else {
        for (; circ; circ &= circ - 1) {
          const int s = __ffsll((long long)circ) - 1;
          const double bs_d = bv(s);
          if (bs_d < bo_d) {
            const double add_s = lk * bs_d;
            const double cs = zv(s) + add_s;
            const double num = co - cs;
            const double den = bo_d - bs_d;
            if (cr_gt(num, den, best)) { best = num / den; bo = o; bs = s; }
          }
        }
      }
    }
    if (bo < 0 || best < tlo) break;   // every later breakpoint is lower
    const double v2 = bs >= 0 ? bv(bo) - bv(bs) : bv(bo);
    S = (S | (1ull << bo)) & ~(bs >= 0 ? (1ull << bs) : 0ull);
    if (window && best > thi) above = above + v2;
    else emit(best, v2);
  }
  *above_out = above;
  return true;
}

// Window filter (one user): the smallest distance between two of its lines
// that can turn positive within h of lambda_k^t, or between such a line and
// zero, must exceed h * bmax (plus a rounding margin): lines move against
// each other by at most |b_a - b_b| <= bmax per unit of lambda_k.  gmin and
// gscale come from the user's p~ in rank order (lines below -H, H the widest
// window's bound, never turn positive).
__device__ __forceinline__ bool window_calm(double gmin, double gscale, double h, double bmax,
                                           double lk) {
  const double need = h * bmax * (1.0 + 0x1p-30) + 0x1p-36 * (1.0 + gscale + lk * bmax + h * bmax);
  return gmin > need;
}
