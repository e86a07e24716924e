// The threshold search of the SCD calls (Alg.4's reduce, Sec. 5.2's buckets):
// the per-knapsack state machine that runs between sweep passes, the exact
// selection among the emitted breakpoints, and the search's first and last
// steps for single and batched instances.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "kp_device.h"

hipError_t kp_launch_reduce_tab(const void *tab, int n, hipStream_t stream);   // kp_kernels.hip

// ---------------------------------------------------------------------------
// SCD threshold search
// ---------------------------------------------------------------------------
// The rest of a window state from its edges (l: lambda_k^t).
__device__ __forceinline__ void set_window(KState &s, double l) {
  s.mode = KS_WINDOW;
  s.klo = dkey(s.wlo);
  s.khi = dkey(s.whi);
  s.tlo = s.wlo;
  s.thi = s.whi;
  const double up = s.whi - l, dn = l - s.wlo;
  s.hw = fmax(fabs(up), fabs(dn));
  s.far = l < s.wlo || l > s.whi;
}

// The window a search starts with, from the multiplier's history: around
// lambda_k^t, 1.25x the last step wide, when that step was small against
// lambda_k^t; else, when the multiplier alternates (it returns close to
// lambda_k^{t-1}: the drift |lambda^t - lambda^{t-2}| is under 1/8 of the
// last step), around lambda_k^{t-1}, 1.25x the drift wide.  hw is the
// farthest window edge from lambda_k^t (the filters bound the lines'
// movement by it).  step, prev, drift < 0 or NaN: unknown.
// Half-widths are at least 2^-20 of the centre: near convergence a
// multiplier's step or its 2-cycle drift can shrink to almost nothing and
// then move by more than that once, and a window that misses costs a full
// pass, while a few hundred more listed users cost little.
__device__ __forceinline__ void choose_window(KState &s, double step, double prev, double drift) {
  double c = 0.0, h = 0.0;
  if (step > 0.0 && KP_WIN_MULT * step <= KP_WIN_MAX_REL * s.center) {
    c = s.center;
    h = fmax(KP_WIN_MULT * step, s.center * 0x1p-20);
  } else if (step > 0.0 && drift >= 0.0 && prev >= 0.0 && drift * 8.0 <= step) {
    const double floor_ = (prev > 0x1p-20 ? prev : 0x1p-20) * 0x1p-20;
    c = prev;
    h = KP_WIN_MULT * (drift > floor_ ? drift : floor_);
  } else {
    return;
  }
  s.whi = c + h;
  s.wlo = c - h > 0.0 ? c - h : 0.0;
  set_window(s, s.center);
}

// The start of a search without a window.  frac > 0: the search runs on that
// share of the users first and turns into a window around the sample's
// threshold (k_sample_window).  frac == 0: the instance is small, its pass
// emits every breakpoint and the threshold is selected among them (one pass;
// the exponential buckets took two or three).  frac < 0, or the other starts
// failed: exponential buckets over every breakpoint.
__device__ __forceinline__ void search_start(KState &s) {
  s.far = 0;
  s.tlo = 0.0;
  s.thi = INFINITY;
  s.klo = 0;
  s.khi = ~0ull;
  s.n_emit = 0;
  s.overflow = 0;
  s.fab = xs_zero();
  s.err = 0.0;
  s.hull_lo = ~0ull;
  s.hull_hi = 0;
  s.corr = xs_zero();
  const uint32_t tried = s.flags & KS_FLAG_TRIED;
  if (tried || s.frac < 0.0) {
    s.mode = KS_EXP;
    s.flags = tried;
  } else {
    s.mode = KS_EMIT_RANGE;
    s.wlo = 0.0;
    // (KS_FLAG_WINDOW: the threshold is 0 when the increments do not exceed
    // the budget)
    s.flags = s.frac > 0.0 ? KS_FLAG_SAMPLE : (KS_FLAG_TRIED | KS_FLAG_WINDOW);
  }
}

// The half-width of the central exponential bucket around multiplier l, a
// power of two: hint (above the last step; <= 0: none) when that is small
// against l; else 2^-10 of l, and at l = 0 (or below 2^-20) 2^-20, so that the
// base-2 buckets around 0 reach 2^11 before they are capped.  (A multiplier
// that alternates between 0 and 2.5 had a central bucket of 4 with three
// quarters of the breakpoints in it: dense M = K = 10, 3e5 users, windows off,
// 9.5 ms a sweep, now 5.0.)
__device__ __forceinline__ double bucket_width(double l, double hint) {
  if (hint > 0.0 && hint <= 0.0625 * l) return hint;
  return l > 0x1p-20 ? ldexp(1.0, ilogb(l) - 10) : 0x1p-20;
}

__global__ void k_scd_init(KState *st, int K, const double *lam_in, const uint8_t *kmask,
                           double *hist, int hinted_in, int window, int interp, double frac) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  KState s;
  s.mode = (kmask && !kmask[k]) ? KS_DONE : KS_EXP;
  s.bstar = 0;
  s.shift = 0;
  s.overflow = 0;
  s.n_emit = 0;
  s.flags = 0;
  s.center = lam_in[k];
  // hist: [K] bucket widths and [K] last steps (valid when hinted_in), then
  // [K] lambda^{t-1} and [K] lambda^{t-2} (NaN while unknown), shifted here
  // once per iteration, and [K] the multipliers last returned
  // A multiplier that the last call did not return (by more than 1/16 of
  // its last step) starts a new trajectory: its windows and its past multipliers would
  // be stale.
  const bool same = hist && hinted_in && fabs(lam_in[k] - hist[4 * K + k]) <= 0.0625 * hist[K + k];
  const double *delta_hint = same ? hist : nullptr;
  double d = delta_hint ? delta_hint[k] : 0.0;
  const bool hinted = d > 0.0;
  double prev = -1.0, drift = -1.0;
  if (hist) {
    prev = same ? hist[2 * K + k] : NAN;
    const double prev2 = same ? hist[3 * K + k] : NAN;
    drift = fabs(lam_in[k] - prev2);   // NaN while unknown
    hist[3 * K + k] = prev;
    hist[2 * K + k] = lam_in[k];
  }
  if (interp) {
    // interpolated reduce: a fixed fine central bucket, 2^-20 of the
    // multiplier (of 2^-20 when it is smaller), a power of two
    const double base = lam_in[k] > 0x1p-20 ? lam_in[k] : 0x1p-20;
    d = ldexp(1.0, ilogb(base) - 20);
  } else {
    d = bucket_width(lam_in[k], d);
  }
  s.delta = d;
  s.fab = xs_zero();
  s.result = lam_in[k];
  s.klo = 0;
  s.khi = ~0ull;
  s.hull_lo = ~0ull;
  s.hull_hi = 0;
  s.wlo = 0.0;
  s.whi = 0.0;
  s.hw = 0.0;
  s.corr = xs_zero();
  s.err = 0.0;
  s.eoff = 0;
  s.ecap = 0;
  s.ncomp = 0;
  s.sel_lo = 0;
  s.sel_hi = 0;
  s.sel_fab = xs_zero();
  s.sel_bin = -1;
  s.far = 0;
  s.tlo = 0.0;
  s.thi = INFINITY;
  s.frac = frac;
  if (interp) {
    s.flags = KS_FLAG_INTERP;
  } else if (s.mode == KS_EXP) {
    if (window && hinted) choose_window(s, delta_hint[K + k], prev, drift);
    if (s.mode == KS_EXP) search_start(s);
  }
  st[k] = s;
}

// err rounded up to the units of the exact sums
__device__ __forceinline__ XSum err_units(double err) {
  XSum e = xs_of(err);
  if (err > 0.0) e.lo += 1;
  return e;
}

__device__ __forceinline__ int bits_needed(uint64_t x) { return x ? 64 - __clzll((long long)x) : 0; }

__device__ __forceinline__ void set_refine(KState &s, uint64_t lo, uint64_t hi) {
  s.klo = lo;
  s.khi = hi;
  const int nb = bits_needed(hi - lo);
  s.shift = nb > 6 ? nb - 6 : 0;   // (hi - lo) >> shift < 64
  s.mode = KS_REFINE;
}

// Sum over the lanes at or above this one (a suffix scan of the wave).
__device__ __forceinline__ XSum wave_suffix(XSum v, int lane) {
  #pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const long long h = __shfl_down(v.hi, d, 64), l = __shfl_down(v.lo, d, 64);
    if (lane + d < 64) { v.hi += h; v.lo += l; }
  }
  return v;
}
__device__ __forceinline__ XSum shfl_xs(const XSum &v, int src) {
  XSum r;
  r.hi = __shfl(v.hi, src, 64);
  r.lo = __shfl(v.lo, src, 64);
  return r;
}

// After a pass: pick the bin holding the threshold and choose the next step.
// One wave per knapsack, lane b holding bin b: the running sums from the top
// are a suffix scan over the lanes and the bin a ballot (the sums are exact,
// so neither depends on an order); one thread per knapsack walking its 64
// bins through global memory took 5-16 us a pass, this 3-4.
__global__ void __launch_bounds__(64) k_scd_locate(KState *st, int K, const double *B, const double *R,
                                                   const int *rinst, XSum *hist_sum, uint32_t *hist_cnt,
                                                   uint32_t emit_cap, SumCheck sc, int nohist, int *pending,
                                                   unsigned int *win) {
  const int k = blockIdx.x, lane = threadIdx.x;
  if (k == 0 && lane == 0) { pending[0] = 0; pending[1] = 0; }   // counted again by the selection
  if (st[k].mode == KS_DONE) return;
  // (a pass without histograms left these searches out)
  if (nohist && (st[k].mode == KS_EXP || st[k].mode == KS_REFINE)) return;
  KState s = st[k];
  if (s.ecap) emit_cap = s.ecap;   // batched: this knapsack's own buffer
  const double Bk = B[k];
  const int in = rinst ? rinst[k] : 0;
  const unsigned int off = sc.off[in];
  XSum h = xs_zero();
  uint32_t cnt = 0;
  if (s.mode == KS_EXP || s.mode == KS_REFINE) {
    h = hist_sum[(size_t)k * KP_NB + lane];
    cnt = hist_cnt[(size_t)k * KP_NB + lane];
    if (cnt) {
      hist_sum[(size_t)k * KP_NB + lane] = xs_zero();
      hist_cnt[(size_t)k * KP_NB + lane] = 0u;
    }
  }
  // running sums down to each bin, and the highest bin at which they exceed B_k
  const XSum run = wave_suffix(h, lane);
  const XSum at = s.mode == KS_REFINE ? xs_plus(s.fab, run) : run;
  const uint64_t over = __ballot(cnt != 0 && xs_gt(at, Bk));
  if (s.mode == KS_EXP) {
    const XSum total = shfl_xs(run, 0);
    if (!xs_gt(total, Bk)) {
      s.mode = KS_DONE;
      s.result = 0.0;
    } else {
      const int bin = over ? 63 - __clzll((long long)over) : 1;
      const XSum hb = shfl_xs(h, bin);
      const uint32_t nb = __shfl(cnt, bin, 64);
      const XSum cum = xs_minus(shfl_xs(run, bin), hb);
      s.bstar = bin - 32;
      s.fab = cum;
      if (s.flags & KS_FLAG_INTERP) {
        // Sec. 5.2's approximate reduce: the bucket's increments spread
        // linearly over its interval [lo, hi] (lo clamped at 0)
        const int id = bin - 32;
        const double c = s.center, d = s.delta;
        double lo, hi;
        if (id == 0) { lo = c - d; hi = c + d; }
        else if (id > 0) { lo = c + ldexp(d, id - 1); hi = c + ldexp(d, id); }
        else { lo = c - ldexp(d, -id); hi = c - ldexp(d, -id - 1); }
        lo = fmax(lo, 0.0);
        const double frac = (Bk - xs_to_double(cum)) / xs_to_double(hb);
        const double width = hi - lo;
        const double prod = frac * width;
        const double v = hi - prod;
        s.mode = KS_DONE;
        s.result = fmax(v, lo);
      } else {
        const bool central = s.bstar >= -KP_CENTRAL_W && s.bstar <= KP_CENTRAL_W;
        if (central && !s.overflow) {
          s.mode = KS_SELECT_BUCKET;
        } else {
          s.mode = nb <= emit_cap / 2 ? KS_EMIT_BUCKET : KS_HULL_BUCKET;
          s.n_emit = 0;
          s.overflow = 0;
          s.hull_lo = ~0ull;
          s.hull_hi = 0;
        }
      }
    }
  } else if (s.mode == KS_EMIT_BUCKET || s.mode == KS_HULL_BUCKET) {
    if (s.mode == KS_EMIT_BUCKET && !s.overflow) {
      s.mode = KS_SELECT_BUCKET;
    } else {
      set_refine(s, s.hull_lo, s.hull_hi);
    }
  } else if (s.mode == KS_REFINE) {
    const int bin = over ? 63 - __clzll((long long)over) : 0;   // (exact sums: some bin exceeds)
    const uint32_t nb = __shfl(cnt, bin, 64);
    s.fab = xs_plus(s.fab, xs_minus(shfl_xs(run, bin), shfl_xs(h, bin)));
    const uint64_t lo = s.klo + ((uint64_t)bin << s.shift);
    const uint64_t hi0 = lo + ((((uint64_t)1) << s.shift) - 1);
    const uint64_t hi = hi0 < s.khi ? hi0 : s.khi;
    if (lo == hi) {
      s.mode = KS_DONE;
      s.result = kdbl(lo);
    } else if (nb <= emit_cap / 2) {
      s.klo = lo;
      s.khi = hi;
      s.mode = KS_EMIT_RANGE;
      s.n_emit = 0;
      s.overflow = 0;
    } else {
      set_refine(s, lo, hi);
    }
  } else if (s.mode == KS_EMIT_RANGE) {
    if (s.flags & KS_FLAG_SAMPLE) {   // (a sample's search waits for its own pass)
    } else if (!s.overflow) {
      s.mode = KS_SELECT_RANGE;
      if (s.flags & KS_FLAG_WINDOW) {   // every breakpoint was emitted: their keys
        s.klo = s.hull_lo;
        s.khi = s.hull_hi;
      }
    } else if (s.flags & KS_FLAG_WINDOW) {
      search_start(s);                  // too many to emit: buckets
    } else {
      set_refine(s, s.klo, s.khi);
    }
  } else if (s.mode == KS_WINDOW) {
    // consumption just above the window, summed over users
    // consumption of knapsack k (batched: R of instance rinst[k] sits after
    // the R, g, P columns of the instances before it)
    const double Rk = R[k + 2 * in];
    const XSum above = xs_plus(xs_of(Rk), s.corr);
    const double lim = sc.per ? sc.per[3 * in] : sc.lim;
    if (win && lane == 0) { atomicAdd(&win[0], 1u); atomicAdd(&win[3], s.n_emit); }
    bool over = s.overflow || xs_gt(above, Bk);   // the threshold lies above the window
    s.err = 0.0;
    if (off != 0 || !(Rk < lim)) {
      const double rel = sc.per ? sc.per[3 * in + 1] : sc.rel, ab = sc.per ? sc.per[3 * in + 2] : sc.abs;
      s.err = rel * fmax(fmax(Rk, Bk), xs_to_double(above)) + ab;
      const XSum e = err_units(s.err);
      if (!s.overflow && xs_gt(xs_plus(above, e), Bk) && !xs_gt(xs_minus(above, e), Bk)) {
        over = true;                    // on its edge, as far as R tells: buckets
        s.flags |= KS_FLAG_TRIED;
      }
    }
    if (over) {
      if (win && lane == 0) atomicAdd(&win[1], 1u);
      search_start(s);
    } else {
      s.mode = KS_SELECT_RANGE;         // [klo, khi] is the window
      s.fab = above;
      s.flags |= KS_FLAG_WINDOW;
    }
  }
  // where the breakpoints that the next pass looks for lie
  if (s.mode == KS_EMIT_BUCKET || s.mode == KS_HULL_BUCKET) {
    bucket_bounds(s.center, s.delta, s.bstar, s.tlo, s.thi);
  } else if (s.mode == KS_REFINE || s.mode == KS_EMIT_RANGE) {
    s.tlo = kdbl(s.klo);
    s.thi = s.khi < 0x7FF0000000000000ull ? kdbl(s.khi) : INFINITY;
  }
  s.ncomp = 0;
  if (lane == 0) st[k] = s;
}

// ---- exact selection of the threshold among the emitted breakpoints ----
// The largest breakpoint at which the running sum from above exceeds B_k.
// One block takes up to SEL_SMALL events by itself; more of them are first
// binned by key over many blocks (k_sel_hist), and the events of the bin that
// holds the threshold compacted (k_sel_compact).  Reading them with one block
// cost up to 2.8 ms of a sweep (1e6 events); a single block that sorted 4096
// events and scanned them with one thread 0.1-0.9 ms even on small problems.
#define SEL_NT 1024
#define SEL_FEW 256        // candidates compared all with all

__device__ __forceinline__ bool sel_mode(int m) { return m == KS_SELECT_BUCKET || m == KS_SELECT_RANGE; }

// The keys a selection looks at: the range, or an interval that holds every
// breakpoint of exponential bucket bstar (widened by more than the rounding
// of the bucket test).
__device__ __forceinline__ void sel_keys(const KState &s, uint64_t &lo, uint64_t &hi) {
  if (s.flags & KS_FLAG_SAMPLE) {
    lo = s.hull_lo;
    hi = s.hull_hi;
    return;
  }
  if (s.mode == KS_SELECT_RANGE) {
    lo = s.klo;
    hi = s.khi;
    return;
  }
  double l, h;
  bucket_bounds(s.center, s.delta, s.bstar, l, h);
  lo = dkey(l);
  hi = dkey(h);
}
__device__ __forceinline__ bool sel_takes(const KState &s, bool bucket, uint64_t lo, uint64_t hi, double v,
                                          uint64_t &key) {
  key = dkey(v);
  return key >= lo && key <= hi && !(bucket && exp_bucket(v, s.center, s.delta) != s.bstar);
}
__device__ __forceinline__ int sel_shift(uint64_t lo, uint64_t hi, int bits) {
  const int nb = bits_needed(hi - lo);
  return nb > bits ? nb - bits : 0;   // (hi - lo) >> shift < 2^bits
}

// The highest of NBIN bins (in LDS) at which Fab plus the sums from the top
// exceeds B_k, by a block of NTH threads: *bin (-1: none) and *cum, the sum
// above it.  part: LDS [NTH / 64 + 1].
template <int NBIN, int NTH>
__device__ __forceinline__ void sel_pick(const XSum *hsum, const uint32_t *hcnt, const XSum &Fab, double Bk,
                                         XSum *part, int *bin, XSum *cum) {
  constexpr int PER = (NBIN + NTH - 1) / NTH;
  constexpr int TH = NBIN / PER;              // threads that hold bins
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid == 0) *bin = -1;
  XSum mine = xs_zero();
  if (tid < TH)
    for (int i = 0; i < PER; ++i) mine = xs_plus(mine, hsum[tid * PER + i]);
  const XSum run = wave_suffix(mine, lane);   // this thread's bins and those above them in the wave
  if (lane == 0 && tid < TH) part[wv] = run;
  __syncthreads();
  if (tid < TH) {
    XSum above = xs_plus(Fab, xs_minus(run, mine));
    for (int w = wv + 1; w * 64 < TH; ++w) above = xs_plus(above, part[w]);
    if (!xs_gt(above, Bk) && xs_gt(xs_plus(above, mine), Bk)) {   // (one thread at most: the sums rise)
      for (int i = PER - 1; i >= 0; --i) {
        const int b = tid * PER + i;
        const XSum next = xs_plus(above, hsum[b]);
        if (hcnt[b] && xs_gt(next, Bk)) { *bin = b; *cum = above; break; }
        above = next;
      }
    }
  }
  __syncthreads();
}

#define SH_NT 512
__global__ void __launch_bounds__(SH_NT) k_sel_hist(const KState *st, const double *V1, const double *V2,
                                                    uint32_t emit_cap, SelWs w, int sample) {
  const int k = blockIdx.x, tid = threadIdx.x;
  const int mode = st[k].mode;
  // (sample: the sampled searches' emitted breakpoints, whatever their count)
  if (sample ? !(st[k].flags & KS_FLAG_SAMPLE) || mode != KS_EMIT_RANGE || st[k].n_emit == 0
             : !sel_mode(mode) || st[k].n_emit <= SEL_SMALL)
    return;
  __shared__ KState s;
  __shared__ XSum hs[SEL_BINS];
  __shared__ uint32_t hc[SEL_BINS];
  if (tid == 0) s = st[k];
  for (int t = tid; t < SEL_BINS; t += SH_NT) { hs[t] = xs_zero(); hc[t] = 0u; }
  __syncthreads();
  const size_t eo = s.ecap ? (size_t)s.eoff : (size_t)k * emit_cap;
  if (s.ecap) emit_cap = s.ecap;
  const uint32_t n = s.n_emit < emit_cap ? s.n_emit : emit_cap;
  const bool bucket = mode == KS_SELECT_BUCKET;
  uint64_t lo, hi;
  sel_keys(s, lo, hi);
  const int shift = sel_shift(lo, hi, SEL_BITS);
  #pragma unroll 4
  for (uint32_t e = blockIdx.y * SH_NT + tid; e < n; e += gridDim.y * SH_NT) {
    const double v = V1[eo + e], inc = V2[eo + e];
    uint64_t key;
    if (!sel_takes(s, bucket, lo, hi, v, key)) continue;
    const int b = (int)((key - lo) >> shift);
    xs_atomic_add(&hs[b], inc);
    atomicAdd(&hc[b], 1u);
  }
  __syncthreads();
  for (int t = tid; t < SEL_BINS; t += SH_NT) {
    if (!hc[t]) continue;
    xs_atomic_add_sum(&w.hsum[(size_t)k * SEL_BINS + t], hs[t]);
    atomicAdd(&w.hcnt[(size_t)k * SEL_BINS + t], hc[t]);
  }
}

__global__ void __launch_bounds__(SH_NT) k_sel_compact(KState *st, const double *B, const double *V1,
                                                       const double *V2, uint32_t emit_cap, SelWs w) {
  const int k = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int mode = st[k].mode;
  if (!sel_mode(mode) || st[k].n_emit <= SEL_SMALL) return;
  __shared__ KState s;
  __shared__ XSum hs[SEL_BINS];
  __shared__ uint32_t hc[SEL_BINS];
  __shared__ XSum part[SH_NT / 64 + 1];
  __shared__ int bin;
  __shared__ XSum cum;
  if (tid == 0) s = st[k];
  for (int t = tid; t < SEL_BINS; t += SH_NT) {
    hs[t] = w.hsum[(size_t)k * SEL_BINS + t];
    hc[t] = w.hcnt[(size_t)k * SEL_BINS + t];
  }
  __syncthreads();
  sel_pick<SEL_BINS, SH_NT>(hs, hc, s.fab, B[k], part, &bin, &cum);
  uint64_t lo, hi;
  sel_keys(s, lo, hi);
  const int shift = sel_shift(lo, hi, SEL_BITS);
  const uint64_t blo = lo + ((uint64_t)(bin < 0 ? 0 : bin) << shift);
  const uint64_t bhi0 = blo + ((((uint64_t)1) << shift) - 1);
  const uint64_t bhi = bhi0 < hi ? bhi0 : hi;
  if (blockIdx.y == 0 && tid == 0) {   // (the other blocks read none of these)
    st[k].sel_bin = bin;
    st[k].sel_lo = blo;
    st[k].sel_hi = bhi;
    if (bin >= 0) st[k].sel_fab = cum;
  }
  if (bin < 0 || hc[bin] > SEL_COMP) return;   // (too many for the list: the last step reads them all)
  const size_t eo = s.ecap ? (size_t)s.eoff : (size_t)k * emit_cap;
  if (s.ecap) emit_cap = s.ecap;
  const uint32_t n = s.n_emit < emit_cap ? s.n_emit : emit_cap;
  const bool bucket = mode == KS_SELECT_BUCKET;
  for (uint32_t e0 = blockIdx.y * SH_NT; e0 < n; e0 += gridDim.y * SH_NT) {
    const uint32_t e = e0 + tid;
    uint64_t key = 0;
    const bool take = e < n && sel_takes(s, bucket, blo, bhi, V1[eo + e], key);
    const uint64_t m = __ballot(take);
    if (!m) continue;
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&st[k].ncomp, (uint32_t)__popcll(m));
    base = __shfl(base, 0, 64);
    const uint32_t slot = base + (uint32_t)__popcll(m & ((1ull << lane) - 1));
    if (take && slot < SEL_COMP) {
      w.c1[(size_t)k * SEL_COMP + slot] = kdbl(key);
      w.c2[(size_t)k * SEL_COMP + slot] = V2[eo + e];
    }
  }
}

// The total over the block (part: LDS [SEL_NT / 64]), to every thread.
__device__ __forceinline__ XSum block_total(XSum v, XSum *part) {
  v = wave_suffix(v, threadIdx.x & 63);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  XSum t = xs_zero();
  #pragma unroll 1
  for (int q = 0; q < SEL_NT / 64; ++q) t = xs_plus(t, part[q]);
  return t;
}

__global__ void __launch_bounds__(SEL_NT) k_sel_final(KState *st, const double *B, const double *V1,
                                                      const double *V2, uint32_t emit_cap, SelWs w, int binned,
                                                      int *pending, unsigned int *win) {
  const int k = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int mode = st[k].mode;
  if (!sel_mode(mode)) {
    if (tid == 0 && mode != KS_DONE) atomicAdd(pending, 1);
    return;
  }
  constexpr int KEEP = 2048;           // events kept in LDS
  __shared__ KState s;
  __shared__ XSum hs[256];
  __shared__ uint32_t hc[256];
  __shared__ XSum part[SEL_NT / 64 + 1];
  __shared__ uint64_t lkey[KEEP];
  __shared__ double lval[KEEP];
  __shared__ int bin;
  __shared__ XSum cum;
  __shared__ uint32_t cnt, fill, kunsure;
  __shared__ unsigned long long kmin, kmax, kres;
  if (tid == 0) s = st[k];
  __syncthreads();
  const double Bk = B[k];
  const bool big = s.n_emit > SEL_SMALL;
  if (big && !binned) {   // left for the binning steps
    if (tid == 0) { atomicAdd(pending, 1); atomicAdd(pending + 1, 1); }
    return;
  }
  size_t eo = s.ecap ? (size_t)s.eoff : (size_t)k * emit_cap;
  if (s.ecap) emit_cap = s.ecap;
  uint32_t n = s.n_emit < emit_cap ? s.n_emit : emit_cap;
  const double *E1 = V1 + eo, *E2 = V2 + eo;
  bool bucket = mode == KS_SELECT_BUCKET;
  uint64_t lo, hi;
  XSum Fab = s.fab;
  bool below = false;                  // a window's increments do not take the sum past B_k
  // err > 0: whether a result holds whatever R lost to rounding (else exact
  // buckets decide); sure: that the increments fit the budget
  const bool chk = s.err > 0.0;
  const XSum ex = err_units(s.err);
  bool sure = !chk;
  if (big) {
    for (int t = tid; t < SEL_BINS; t += SEL_NT) {
      w.hsum[(size_t)k * SEL_BINS + t] = xs_zero();
      w.hcnt[(size_t)k * SEL_BINS + t] = 0u;
    }
    lo = s.sel_lo;
    hi = s.sel_hi;
    if (s.sel_bin >= 0) Fab = s.sel_fab;
    below = s.sel_bin < 0;
    if (s.ncomp && s.ncomp <= SEL_COMP) {
      E1 = w.c1 + (size_t)k * SEL_COMP;
      E2 = w.c2 + (size_t)k * SEL_COMP;
      n = s.ncomp;
      bucket = false;
    }
  } else {
    sel_keys(s, lo, hi);
    if (s.flags & KS_FLAG_WINDOW) {
      XSum v = xs_zero();
      for (uint32_t e = tid; e < n; e += SEL_NT) xs_add(v, E2[e]);
      v = wave_suffix(v, lane);
      if (lane == 0) part[tid >> 6] = v;
      __syncthreads();
      XSum tot = Fab;
      for (int q = 0; q < SEL_NT / 64; ++q) tot = xs_plus(tot, part[q]);
      below = !xs_gt(tot, Bk);
      if (chk) sure = !xs_gt(xs_plus(tot, ex), Bk);
      __syncthreads();
    }
  }
  if ((s.flags & KS_FLAG_WINDOW) && below) {
    if (chk && big && s.wlo == 0.0) {
      XSum v = xs_zero();
      #pragma unroll 1
      for (uint32_t e = tid; e < s.n_emit; e += SEL_NT) xs_add(v, (V2 + eo)[e]);
      const XSum tot = xs_plus(s.fab, block_total(v, part));
      sure = !xs_gt(xs_plus(tot, ex), Bk);
    }
    if (tid == 0) {
      if (s.wlo == 0.0 && sure) {       // every breakpoint is in the window
        st[k].result = 0.0;
        st[k].mode = KS_DONE;
      } else {
        KState r = s;                   // below the window: search again
        if (s.wlo == 0.0) r.flags |= KS_FLAG_TRIED;
        else if (win) atomicAdd(&win[2], 1u);
        search_start(r);
        st[k] = r;
        atomicAdd(pending, 1);
      }
    }
    return;
  }
  // narrow the key range until few candidates are left
  bool inlds = false;
  for (int it = 0; it < 80; ++it) {
    if (tid == 0) { cnt = 0; kmin = ~0ull; kmax = 0ull; fill = 0; }
    if (tid < 256) { hs[tid] = xs_zero(); hc[tid] = 0u; }
    __syncthreads();
    uint32_t c = 0;
    uint64_t mn = ~0ull, mx = 0;
    #pragma unroll 4
    for (uint32_t e = tid; e < n; e += SEL_NT) {
      uint64_t key = 0;
      bool ok;
      if (inlds) { key = lkey[e]; ok = key >= lo && key <= hi; }
      else ok = sel_takes(s, bucket, lo, hi, E1[e], key);
      if (ok) { ++c; mn = key < mn ? key : mn; mx = key > mx ? key : mx; }
    }
    #pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      c += __shfl_xor(c, d, 64);
      const uint64_t a = (uint64_t)__shfl_xor((long long)mn, d, 64), b = (uint64_t)__shfl_xor((long long)mx, d, 64);
      mn = a < mn ? a : mn;
      mx = b > mx ? b : mx;
    }
    if (lane == 0 && c) { atomicAdd(&cnt, c); atomicMin(&kmin, mn); atomicMax(&kmax, mx); }
    __syncthreads();
    if (!inlds && cnt <= KEEP) {
      for (uint32_t e = tid; e < n; e += SEL_NT) {
        uint64_t key;
        if (!sel_takes(s, bucket, lo, hi, E1[e], key)) continue;
        const uint32_t q = atomicAdd(&fill, 1u);
        lkey[q] = key;
        lval[q] = E2[e];
      }
      inlds = true;
      __syncthreads();
      n = cnt;
    }
    if (cnt <= SEL_FEW || kmin >= kmax) break;
    lo = kmin;
    hi = kmax;
    const int shift = sel_shift(lo, hi, 8);
    for (uint32_t e = tid; e < n; e += SEL_NT) {
      uint64_t key;
      double v2;
      if (inlds) {
        key = lkey[e];
        if (key < lo || key > hi) continue;
        v2 = lval[e];
      } else {
        if (!sel_takes(s, bucket, lo, hi, E1[e], key)) continue;
        v2 = E2[e];
      }
      const int b = (int)((key - lo) >> shift);
      xs_atomic_add(&hs[b], v2);
      atomicAdd(&hc[b], 1u);
    }
    __syncthreads();
    sel_pick<256, SEL_NT>(hs, hc, Fab, Bk, part, &bin, &cum);
    const int b = bin < 0 ? 0 : bin;   // (exact sums: some bin exceeds)
    if (bin >= 0) Fab = cum;
    const uint64_t nlo = lo + ((uint64_t)b << shift);
    const uint64_t nhi = nlo + ((((uint64_t)1) << shift) - 1);
    lo = nlo;
    hi = nhi < hi ? nhi : hi;
    __syncthreads();
  }
  // the candidates, compared all with all (or all equal: kmin)
  if (tid == 0) { kres = kmin; fill = 0; kunsure = 0; }
  __syncthreads();
  const bool few = cnt <= SEL_FEW && kmin < kmax;
  if (few) {
    XSum *fv = hs;   // [256]
    __shared__ uint64_t fk[SEL_FEW];
    for (uint32_t e = tid; e < n; e += SEL_NT) {
      const uint64_t key = lkey[e];
      if (key < lo || key > hi) continue;
      const uint32_t q = atomicAdd(&fill, 1u);
      fk[q] = key;
      fv[q] = xs_of(lval[e]);
    }
    __syncthreads();
    if (tid < (int)fill) {
      const uint64_t key = fk[tid];
      XSum at = Fab;
      for (uint32_t q = 0; q < fill; ++q)
        if (fk[q] >= key) at = xs_plus(at, fv[q]);
      if (xs_gt(at, Bk)) atomicMax(&kres, (unsigned long long)key);
      // no running sum, nor the one above them all, may lie that close to the budget
      if (chk && (xs_gt(xs_plus(at, ex), Bk) != xs_gt(xs_minus(at, ex), Bk) || xs_gt(xs_plus(Fab, ex), Bk))) kunsure = 1;
    }
    __syncthreads();
  }
  if (chk) {
    if (!few) {
      // every candidate has the same key: the sum with them must exceed the
      // budget, and the one above them not (one event is the rule near
      // convergence: a wave adds up to 64)
      const bool small = inlds && n <= 64;
      XSum v = xs_zero();
      if (!small || tid < 64) {
        for (uint32_t e = tid; e < n; e += SEL_NT) {
          uint64_t key = 0;
          if (inlds) key = lkey[e];
          if (inlds ? key >= lo && key <= hi : sel_takes(s, bucket, lo, hi, E1[e], key)) xs_add(v, inlds ? lval[e] : E2[e]);
        }
        v = small ? wave_suffix(v, lane) : v;
      }
      if (!small) v = block_total(v, part);
      if (tid == 0 && (!xs_gt(xs_minus(xs_plus(Fab, v), ex), Bk) || xs_gt(xs_plus(Fab, ex), Bk))) kunsure = 1;
      __syncthreads();
    }
    if (kunsure) {
      if (tid == 0) {
        KState r = s;
        r.flags |= KS_FLAG_TRIED;
        search_start(r);
        st[k] = r;
        atomicAdd(pending, 1);
      }
      return;
    }
  }
  if (tid == 0) {
    st[k].result = kdbl(kres);
    st[k].mode = KS_DONE;
  }
}

__global__ void k_scd_finish(const KState *st, int K, const double *lam_in, double *lam_out,
                             double *delta_next) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  const double nl = st[k].result;
  lam_out[k] = nl;
  if (delta_next) {
    // next search: the bucket width, a power of two above this step, and the
    // step itself (bounded below) for the window
    const double step = fabs(nl - lam_in[k]);
    const double floor_ = (nl > 0x1p-20 ? nl : 0x1p-20) * 0x1p-30;
    const double w = step > floor_ ? step : floor_;
    delta_next[k] = ldexp(1.0, ilogb(w) + 1);
    delta_next[K + k] = w;
    delta_next[4 * K + k] = nl;
  }
}

// The window a sampled search turns into: every breakpoint of the sample was
// emitted and binned by key (2048 bins of about 2 % each over the keys'
// span), and the window runs from the bin where the sample's running sum
// exceeds its budget by the share KP_SAMPLE_DEV / sqrt(n) of it, n the
// breakpoints above the threshold, down to where it falls short of it by as
// much.  A sum of n increments of independent users deviates by about
// 1.3 / sqrt(n) of itself (increments of a spread like the uniform's), so that
// is 3.5 deviations: 2 of 6950 windows missed (dense and two costs per item,
// 4e4 to 1e6 users), none of 2000 with every item twice.  Users that are alike
// within a tile of 64 deviate more (56 % of 1000 windows on such rows missed,
// 16 % of 500 on dense costs) and go on with buckets.  A sample with too
// few breakpoints above the threshold opens the window over everything, when
// the emission buffer can be expected to hold all users' breakpoints; a sample
// that overflowed it tells that it cannot, and the search goes on with
// buckets at once (a window over everything emitted and dropped every
// breakpoint first: 21 ms of 91 for 2e5 users with M = 32, K = 16, Q = 20).
// Exactness does not depend on any of it: a window's search is decided
// exactly over all users, and a miss falls back to the buckets.
#define KP_SAMPLE_DEV 4.5
#define SW_NT 256
__global__ void __launch_bounds__(SW_NT) k_sample_window(KState *st, const double *B, uint32_t emit_cap, SelWs w) {
  const int k = blockIdx.x, tid = threadIdx.x;
  if (!(st[k].flags & KS_FLAG_SAMPLE) || st[k].mode != KS_EMIT_RANGE) return;
  __shared__ KState s;
  __shared__ XSum hs[SEL_BINS];
  __shared__ uint32_t hc[SEL_BINS];
  __shared__ XSum part[SW_NT / 64 + 1];
  __shared__ int bin, b0;
  __shared__ XSum cum;
  __shared__ uint32_t above;
  if (tid == 0) { s = st[k]; above = 0; }
  __syncthreads();
  const bool any = s.n_emit != 0;
  for (int t = tid; any && t < SEL_BINS; t += SW_NT) {
    hs[t] = w.hsum[(size_t)k * SEL_BINS + t];
    hc[t] = w.hcnt[(size_t)k * SEL_BINS + t];
    w.hsum[(size_t)k * SEL_BINS + t] = xs_zero();
    w.hcnt[(size_t)k * SEL_BINS + t] = 0u;
  }
  __syncthreads();
  double wlo = 0.0, whi = INFINITY;
  bool buckets = s.overflow != 0;
  if (any && !buckets) {
    const double Bs = B[k] * s.frac;
    const int shift = sel_shift(s.hull_lo, s.hull_hi, SEL_BITS);
    sel_pick<SEL_BINS, SW_NT>(hs, hc, xs_zero(), Bs, part, &bin, &cum);
    if (tid == 0) b0 = bin;
    __syncthreads();
    uint32_t c = 0;
    for (int t = tid; t < SEL_BINS; t += SW_NT)
      if (t >= b0) c += hc[t];
    if (c) atomicAdd(&above, c);
    __syncthreads();
    if (above >= 16u) {
      const double dev = fmin(0.5, KP_SAMPLE_DEV / sqrt((double)above));
      sel_pick<SEL_BINS, SW_NT>(hs, hc, xs_zero(), Bs * (1.0 - dev), part, &bin, &cum);
      // the top of that bin; nothing exceeds it: no threshold above the lowest breakpoint
      const int bh = bin;
      __syncthreads();
      sel_pick<SEL_BINS, SW_NT>(hs, hc, xs_zero(), Bs * (1.0 + dev), part, &bin, &cum);
      const int bl = bin;
      const uint64_t one = 1;
      if (bh < 0) {
        whi = kdbl(s.hull_lo);
      } else {
        const uint64_t key = s.hull_lo + ((uint64_t)(bh + 1) << shift);
        whi = kdbl(key < s.hull_hi ? key : s.hull_hi);
      }
      if (bl >= 0) {
        const uint64_t key = s.hull_lo + ((uint64_t)bl << shift);
        wlo = kdbl(key - one);
      }
    } else {
      buckets = (double)s.n_emit > s.frac * (double)(s.ecap ? s.ecap : emit_cap);
    }
  }
  if (buckets) {
    if (tid == 0) {
      s.flags |= KS_FLAG_TRIED;
      search_start(s);
      st[k] = s;
    }
    return;
  }
  if (tid == 0) {
    const double l = s.center;   // lambda_k^t
    s.flags = KS_FLAG_TRIED;
    s.n_emit = 0;
    s.overflow = 0;
    s.fab = xs_zero();
    s.hull_lo = ~0ull;
    s.hull_hi = 0;
    s.corr = xs_zero();
    s.wlo = wlo;
    s.whi = whi;
    set_window(s, l);
    if (whi < INFINITY) {   // a miss continues with buckets around it
      s.center = 0.5 * (wlo + whi);
      s.delta = ldexp(1.0, ilogb(fmax(whi - wlo, whi * 0x1p-20)));
    }
    st[k] = s;
  }
}

// Knapsacks starting with a window and those needing another search mode.
// out[0]: knapsacks searching with a window, out[1]: with another search
// mode, out[2]: windows that do not contain lambda_k^t (alternation windows),
// or with reach > 0 windows that extend farther than reach lambda_k^t from it;
// out[3] is cleared (the dense window pass's probe counts into it)
__global__ void k_count_modes(const KState *st, int K, double reach, int *out) {
  __shared__ int c[3];
  if (threadIdx.x < 3) c[threadIdx.x] = 0;
  __syncthreads();
  for (int k = threadIdx.x; k < K; k += blockDim.x) {
    const KState &s = st[k];
    if (s.mode == KS_WINDOW) {
      atomicAdd(&c[0], 1);
      // (result: lambda_k^t until the search ends)
      if (reach > 0.0 ? !(s.hw <= reach * s.result) : s.far != 0) atomicAdd(&c[2], 1);
    } else if (s.mode != KS_DONE) {
      atomicAdd(&c[1], 1);
    }
  }
  __syncthreads();
  if (threadIdx.x < 3) out[threadIdx.x] = c[threadIdx.x];
  if (threadIdx.x == 3) out[3] = 0;
}

__global__ void k_scd_init_flat(KState *st, int Kf, const double *const *lam_in, const int *kinst,
                                const int *klocal, double *hint, int window, const uint64_t *eoff,
                                const uint32_t *ecap, const double *frac, unsigned int *off) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= Kf) return;
  if (klocal[f] == 0) off[kinst[f]] = 0u;
  const double l = lam_in[kinst[f]][klocal[f]];
  KState s;
  s.mode = KS_EXP;
  s.bstar = 0;
  s.shift = 0;
  s.overflow = 0;
  s.n_emit = 0;
  s.flags = 0;
  s.center = l;
  s.delta = bucket_width(l, hint ? hint[f] : 0.0);
  s.fab = xs_zero();
  s.result = l;
  s.klo = 0;
  s.khi = ~0ull;
  s.hull_lo = ~0ull;
  s.hull_hi = 0;
  s.wlo = 0.0;
  s.whi = 0.0;
  s.hw = 0.0;
  s.corr = xs_zero();
  s.err = 0.0;
  s.eoff = eoff ? eoff[f] : 0;
  s.ecap = ecap ? ecap[f] : 0;
  s.ncomp = 0;
  s.sel_lo = 0;
  s.sel_hi = 0;
  s.sel_fab = xs_zero();
  s.sel_bin = -1;
  s.far = 0;
  s.tlo = 0.0;
  s.thi = INFINITY;
  // a window from the multiplier's history (as the single-instance search);
  // the history columns shift once per iteration, here
  if (hint) {
    // (a multiplier that the last step did not return: no window, no past)
    const bool same = hint[f] > 0.0 && fabs(l - hint[4 * Kf + f]) <= 0.0625 * hint[Kf + f];
    const double prev = same ? hint[2 * Kf + f] : NAN;
    const double drift = same ? fabs(l - hint[3 * Kf + f]) : NAN;
    hint[3 * Kf + f] = prev;
    hint[2 * Kf + f] = l;
    if (window && same) choose_window(s, hint[Kf + f], prev, drift);
  }
  s.frac = frac[f];
  if (s.mode == KS_EXP) search_start(s);
  st[f] = s;
}

// Batched: flags[s] = 1 if instance s has a knapsack that needs another
// pass over its users (knapsacks koff[s] .. koff[s+1]-1 of the flat state).
__global__ void k_inst_active(const KState *st, const int *koff, int n, int *flags) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  int on = 0;
  for (int f = koff[s]; f < koff[s + 1]; ++f) on |= walk_mode(st[f].mode) ? 1 : 0;
  flags[s] = on;
}

__global__ void k_scd_finish_flat(const KState *st, int Kf, double *const *lam_out, const int *kinst,
                                  const int *klocal, double *hint) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= Kf) return;
  const double nl = st[f].result;
  lam_out[kinst[f]][klocal[f]] = nl;
  if (hint) {
    // the next iteration's bucket width: the power of two above this step
    const double step = fabs(nl - hint[2 * Kf + f]);   // (that column holds this iteration's lambda_in)
    const double floor_ = (nl > 0x1p-20 ? nl : 0x1p-20) * 0x1p-30;
    const double w = step > floor_ ? step : floor_;
    hint[f] = ldexp(1.0, ilogb(w) + 1);
    hint[Kf + f] = w;
    hint[4 * Kf + f] = nl;
  }
}


hipError_t kp_launch_batched_aux(int which, const void *tab, int n, KState *st, const void *lam_ptrs,
                                 const int *kinst, const int *klocal, double *hint, const uint64_t *eoff,
                                 const uint32_t *ecap, const double *frac, unsigned int *off, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  if (which == 0) return kp_launch_reduce_tab(tab, n, stream);
  if (which == 1 || which == 3) {   // 3: with a window where the last step allows
    hipLaunchKernelGGL(k_scd_init_flat, dim3((n + 63) / 64), dim3(64), 0, stream, st, n,
                       (const double *const *)lam_ptrs, kinst, klocal, hint,
                       which == 3 ? 1 : 0, eoff, ecap, frac, off);
  } else {
    hipLaunchKernelGGL(k_scd_finish_flat, dim3((n + 63) / 64), dim3(64), 0, stream, (const KState *)st,
                       n, (double *const *)lam_ptrs, kinst, klocal, hint);
  }
  return hipGetLastError();
}

hipError_t kp_launch_inst_active(const KState *st, const int *koff, int n, int *flags, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_inst_active, dim3((n + 63) / 64), dim3(64), 0, stream, st, koff, n, flags);
  return hipGetLastError();
}

hipError_t kp_launch_scd_init(KState *st, int K, const double *lam_in, const uint8_t *kmask,
                              double *hist, int hinted, int window, int interp, double frac,
                              hipStream_t stream) {
  hipLaunchKernelGGL(k_scd_init, dim3((K + 63) / 64), dim3(64), 0, stream, st, K, lam_in, kmask,
                     hist, hinted, window, interp, frac);
  return hipGetLastError();
}

__global__ void k_fill_i32(int *dst, int n, int v) {
  if ((int)threadIdx.x < n) dst[threadIdx.x] = v;
}
static hipError_t kp_launch_fill_i32(int *dst, int n, int v, hipStream_t stream) {
  hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, stream, dst, n, v);
  return hipGetLastError();
}

// Workspace of the selection for K knapsacks; its histograms start cleared.
size_t kp_sel_bytes(int K) {
  return (size_t)K * (SEL_BINS * (sizeof(XSum) + 4) + SEL_COMP * 16);
}
size_t kp_sel_clear_bytes(int K) { return (size_t)K * SEL_BINS * (sizeof(XSum) + 4); }
SelWs kp_sel_ws(void *mem, int K) {
  SelWs w;
  w.hsum = (XSum *)mem;
  w.hcnt = (uint32_t *)(w.hsum + (size_t)K * SEL_BINS);
  w.c1 = (double *)(w.hcnt + (size_t)K * SEL_BINS);
  w.c2 = w.c1 + (size_t)K * SEL_COMP;
  return w;
}

// After a pass: locate, then select.  blocks: blocks per knapsack of the
// binning steps; 0 leaves the knapsacks with more events than one block
// selects from in their selecting state (pending[1] counts them) for
// kp_launch_scd_select_many: the binning kernels, each 4-5 us even with
// nothing to bin, then cost nothing in the passes that emit little.
hipError_t kp_launch_scd_locate_select(KState *st, int K, const double *B, const double *R,
                                       const int *rinst, XSum *hist_sum, uint32_t *hist_cnt,
                                       const double *ev1, const double *ev2, uint32_t emit_cap,
                                       const SelWs &w, int blocks, const SumCheck &sc, int nohist, int *pending,
                                       unsigned int *win, hipStream_t stream) {
  hipLaunchKernelGGL(k_scd_locate, dim3(K), dim3(64), 0, stream, st, K, B, R, rinst, hist_sum,
                     hist_cnt, emit_cap, sc, nohist, pending, win);
  if (blocks > 0) {
    hipLaunchKernelGGL(k_sel_hist, dim3(K, blocks), dim3(SH_NT), 0, stream, st, ev1, ev2, emit_cap, w, 0);
    hipLaunchKernelGGL(k_sel_compact, dim3(K, blocks), dim3(SH_NT), 0, stream, st, B, ev1, ev2, emit_cap, w);
  }
  hipLaunchKernelGGL(k_sel_final, dim3(K), dim3(SEL_NT), 0, stream, st, B, ev1, ev2, emit_cap, w,
                     blocks > 0 ? 1 : 0, pending, win);
  return hipGetLastError();
}

hipError_t kp_launch_scd_select_many(KState *st, int K, const double *B, const double *ev1, const double *ev2,
                                     uint32_t emit_cap, const SelWs &w, int blocks, int *pending,
                                     unsigned int *win, hipStream_t stream) {
  hipError_t e = kp_launch_fill_i32(pending, 2, 0, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_sel_hist, dim3(K, blocks), dim3(SH_NT), 0, stream, st, ev1, ev2, emit_cap, w, 0);
  hipLaunchKernelGGL(k_sel_compact, dim3(K, blocks), dim3(SH_NT), 0, stream, st, B, ev1, ev2, emit_cap, w);
  hipLaunchKernelGGL(k_sel_final, dim3(K), dim3(SEL_NT), 0, stream, st, B, ev1, ev2, emit_cap, w, 1, pending, win);
  return hipGetLastError();
}

hipError_t kp_launch_count_modes(const KState *st, int K, double reach, int *out, hipStream_t stream) {
  hipLaunchKernelGGL(k_count_modes, dim3(1), dim3(256), 0, stream, st, K, reach, out);
  return hipGetLastError();
}

hipError_t kp_launch_scd_finish(const KState *st, int K, const double *lam_in, double *lam_out,
                                double *delta_next, hipStream_t stream) {
  hipLaunchKernelGGL(k_scd_finish, dim3((K + 63) / 64), dim3(64), 0, stream, st, K, lam_in,
                     lam_out, delta_next);
  return hipGetLastError();
}

// The sampled searches' emitted breakpoints to windows (the sample's sweep
// ran): blocks per knapsack that bin them.
hipError_t kp_launch_sample_window(KState *st, int K, const double *B, const double *ev1, const double *ev2,
                                   uint32_t emit_cap, const SelWs &w, int blocks, hipStream_t stream) {
  hipLaunchKernelGGL(k_sel_hist, dim3(K, blocks), dim3(SH_NT), 0, stream, st, ev1, ev2, emit_cap, w, 1);
  hipLaunchKernelGGL(k_sample_window, dim3(K), dim3(SW_NT), 0, stream, st, B, emit_cap, w);
  return hipGetLastError();
}
