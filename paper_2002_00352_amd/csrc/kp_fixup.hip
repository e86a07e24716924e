// Post-processing for feasibility (Sec. 5.4): the candidates (users whose
// solution consumes a violated knapsack) are taken in (G_i asc, i asc) order
// and the shortest prefix whose reset covers every violated knapsack is
// reset.  Nothing is sorted but the last thousand users around the boundary:
// splitters drawn from a sample of the G values cut the key range into bins,
// one pass adds every candidate's costs on the violated knapsacks into
// per-bin exact sums, and the bin in which the last knapsack becomes covered
// is found from the bins' prefix sums.  A pass over the bin bytes resets the
// users of the earlier bins and lists that bin's users; a list of more than
// FX_LAST users is cut again the same way, and one block sorts what is left,
// finds the shortest covering prefix and resets it.  (A radix sort of the
// sample and of the bin's users took 97 launches of three kernels: 2.9 of
// 5.2 ms of GPU time in the solve of 1e4 users; fix-up of 1e7 sparse users
// 3.49 -> 1.41 ms.)  Coverage compares
// exact sums (two-limb fixed point) with B_k: the consumption a reset leaves
// is a real sum, so the reset set does not depend on any summation order.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>
#include <algorithm>
#include <functional>
#include "kp_device.h"

#define FX_NT 256
#define FX_IPT 16                       // users per thread of a chunk
#define FX_CHUNK (FX_NT * FX_IPT)
#define FX_NONE 0xFFu                   // bin byte of a user that is not a candidate
#define FX_LDS_MAX (48 * 1024)          // per-block accumulators above this live in global memory
#define FX_SAMPLE 2048                  // users sampled for the splitters
#define FX_LAST 1024                    // users the last block takes

struct FixState {
  int bstar;            // bin in which the last violated knapsack is covered (-1: none violated)
  uint32_t nstar;       // users in it (listed)
  uint32_t napp;        // users appended to the list (atomic)
  int eq;               // every sampled key is eqk: bins below, at and above it
  unsigned long long eqk;
  unsigned long long nreset;   // users reset
};

struct FixArgs {
  ProbDev pr;
  uint8_t *x;             // [N*M] selection at lambda; the reset clears rows
  const double *lam;      // [K]
  const int *kv;          // [K] slot of a violated knapsack, or -1
  const int *vk;          // [nv] knapsack of each slot
  const double *Bv;       // [nv] their budgets
  int nv, nb;
  int d;                  // CSR: entries in every row (row r's start at r * d), or 0
  uint64_t *split;        // [nb - 1] ascending splitter keys
  uint8_t *bin;           // [N] bin of every user (FX_NONE: not a candidate)
  XSum *hsum;             // [nb][nv] exact consumption per bin (cleared between levels)
  uint32_t *hcnt;         // [nb] candidates per bin (cleared between levels)
  FixState *fs;
  XSum *tot;              // [nv] consumption of all candidates
  XSum *cthr;             // [nv] consumption of the users before the current bin
  int *act;               // [nv] slot covered inside the current bin
  XSum *rem;              // [K + 1] removed consumption and profit
  // the users looked at: all of them (list null), or a list and its keys
  const uint32_t *list;
  const uint64_t *lkey;
  uint32_t nlist;
  int byidx;              // list: every key is equal, the users' indices order them
  uint32_t *olist;        // the list the current bin's users are appended to
  uint64_t *okey;
};

// the cost entries (k, b) of item row r in storage order (d > 0: every CSR
// row holds d entries)
template <class F>
__device__ __forceinline__ void fx_row(const ProbDev &pr, int d, int64_t r, F f) {
  if (pr.fmt == 0) {   // dense rows
    const float *bb = pr.b + r * pr.K;
    for (int k = 0; k < pr.K; ++k) f(k, bb[k]);
  } else if (d > 0) {
    const int64_t e0 = r * d;
    for (int t = 0; t < d; ++t) f((int)pr.col[e0 + t], pr.val[e0 + t]);
  } else {
    const int64_t e1 = pr.rowptr[r + 1];
    for (int64_t e = pr.rowptr[r]; e < e1; ++e) f((int)pr.col[e], pr.val[e]);
  }
}

// the selected items of user i: its x bytes read without a branch in between
// (a branch per item made every load wait for the one before)
__device__ __forceinline__ uint64_t fx_sel(const FixArgs &f, int64_t i) {
  const uint8_t *xr = f.x + i * f.pr.M;
  uint64_t m = 0;
  #pragma unroll 8
  for (int j = 0; j < f.pr.M; ++j) m |= (uint64_t)(xr[j] != 0) << j;
  return m;
}

// G_i, the sum of p~ over the selected items in ascending index order (p~ as
// the sweep forms it: the stored costs in order, a product then a
// subtraction), and whether user i consumes a violated knapsack
__device__ __forceinline__ bool fx_user(const FixArgs &f, int64_t i, double &G) {
  const int M = f.pr.M, K = f.pr.K;
  bool cand = false;
  double g = 0.0;
  for (uint64_t m = fx_sel(f, i); m; m &= m - 1) {
    const int64_t r = i * M + __ffsll((long long)m) - 1;
    double acc = (double)f.pr.p[r];
    fx_row(f.pr, f.d, r, [&](int k, float c) {
      if ((unsigned)k >= (unsigned)K) return;
      const double prod = f.lam[k] * (double)c;
      acc = acc - prod;
      cand = cand || (c > 0.0f && f.kv[k] >= 0);
    });
    g = g + acc;
  }
  G = g;
  return cand;
}

// exact consumption of knapsack k by user i's selection
__device__ __forceinline__ XSum fx_use(const FixArgs &f, int64_t i, int k) {
  XSum s = xs_zero();
  for (uint64_t m = fx_sel(f, i); m; m &= m - 1) {
    const int64_t r = i * f.pr.M + __ffsll((long long)m) - 1;
    if (f.pr.fmt == 0) {
      s = xs_plus(s, xs_of((double)f.pr.b[r * f.pr.K + k]));
      continue;
    }
    fx_row(f.pr, f.d, r, [&](int kk, float c) {
      if (kk == k) s = xs_plus(s, xs_of((double)c));
    });
  }
  return s;
}

// the order of a list's entry at this level
__device__ __forceinline__ uint64_t fx_key(const FixArgs &f, uint32_t e) {
  return f.byidx ? (uint64_t)f.list[e] : f.lkey[e];
}
__device__ __forceinline__ int fx_bin(const FixArgs &f, const uint64_t *sp, int eq, uint64_t eqk, uint64_t key) {
  if (eq) return key < eqk ? 0 : key == eqk ? 1 : 2;
  return fx_bin_of(sp, f.nb, key);
}

__global__ void k_fix_init(FixArgs f) {
  const size_t n = (size_t)f.nb * f.nv;
  const size_t t0 = blockIdx.x * (size_t)blockDim.x + threadIdx.x, st = (size_t)gridDim.x * blockDim.x;
  for (size_t t = t0; t < n; t += st) f.hsum[t] = xs_zero();
  for (size_t t = t0; t < (size_t)f.nb; t += st) f.hcnt[t] = 0u;
  for (size_t t = t0; t < (size_t)f.nv; t += st) { f.cthr[t] = xs_zero(); f.act[t] = 1; }
  for (size_t t = t0; t <= (size_t)f.pr.K; t += st) f.rem[t] = xs_zero();
  if (t0 == 0) { f.fs->bstar = -1; f.fs->nstar = 0; f.fs->napp = 0; f.fs->eq = 0; f.fs->eqk = 0; f.fs->nreset = 0; }
}

// splitters: the quantiles q / nb of a strided sample's keys, sorted in LDS
// (all keys in bin 0 when the sample holds no candidate); for a list whose
// sampled keys are all equal, that key instead
__global__ void __launch_bounds__(1024) k_fix_splits(FixArgs f) {
  __shared__ uint64_t key[FX_SAMPLE];
  __shared__ uint32_t cnt;
  const int tid = threadIdx.x;
  if (tid == 0) cnt = 0;
  __syncthreads();
  const int64_t n = f.list ? (int64_t)f.nlist : f.pr.N;
  const int64_t ns = n < FX_SAMPLE ? n : FX_SAMPLE, stride = ns ? n / ns : 1;
  for (int64_t s = tid; s < ns; s += 1024) {
    uint64_t k;
    if (f.list) {
      k = fx_key(f, (uint32_t)(s * stride));
    } else {
      double G;
      if (!fx_user(f, s * stride, G)) continue;
      k = dkey(G + 0.0);
    }
    key[atomicAdd(&cnt, 1u)] = k;
  }
  __syncthreads();
  const uint32_t m = cnt;
  uint32_t P2 = 2;
  while (P2 < m) P2 <<= 1;
  for (uint32_t t = m + tid; t < P2; t += 1024) key[t] = ~0ull;
  __syncthreads();
  for (uint32_t size = 2; size <= P2; size <<= 1) {
    for (uint32_t stp = size >> 1; stp > 0; stp >>= 1) {
      for (uint32_t t = tid; t < P2; t += 1024) {
        const uint32_t o = t ^ stp;
        if (o > t) {
          const uint64_t a = key[t], b = key[o];
          if (((t & size) == 0) == (a > b)) { key[t] = b; key[o] = a; }
        }
      }
      __syncthreads();
    }
  }
  for (int q = tid; q < f.nb - 1; q += 1024) f.split[q] = m ? key[((uint64_t)(q + 1) * m) / f.nb] : ~0ull;
  if (tid == 0) {
    // a list's splitters must leave something above them to make progress
    const bool eq = f.list && m && key[0] == key[m - 1];
    f.fs->eq = eq ? 1 : 0;
    f.fs->eqk = eq ? key[0] : 0;
    if (f.list && !eq && f.split[0] == key[m - 1]) {   // a heavy top value: cut below it
      uint32_t q = m - 1;
      while (q > 0 && key[q] == key[m - 1]) --q;
      f.split[0] = key[q];
    }
  }
}

// every user (bin byte) or list entry: per-bin candidate counts and exact
// consumption of the violated knapsacks still open (block accumulators in LDS
// when they fit, added to the global ones at the end; the grid strides over
// chunks)
__global__ void __launch_bounds__(FX_NT) k_fix_bins(FixArgs f, int lds) {
  extern __shared__ __align__(16) unsigned char fsm[];
  const int nb = f.nb, nv = f.nv, K = f.pr.K, M = f.pr.M;
  XSum *hs = lds ? (XSum *)fsm : f.hsum;
  uint32_t *hc = lds ? (uint32_t *)(fsm + (size_t)nb * nv * sizeof(XSum)) : f.hcnt;
  uint64_t *sp = (uint64_t *)(fsm + (lds ? (size_t)nb * nv * sizeof(XSum) + (size_t)nb * 4 + 8 : 0));
  if (lds) {
    for (int t = threadIdx.x; t < nb * nv; t += FX_NT) hs[t] = xs_zero();
    for (int t = threadIdx.x; t < nb; t += FX_NT) hc[t] = 0u;
  }
  for (int t = threadIdx.x; t < nb - 1; t += FX_NT) sp[t] = f.split[t];
  __syncthreads();
  const int eq = f.fs->eq;
  const uint64_t eqk = f.fs->eqk;
  const int64_t n = f.list ? (int64_t)f.nlist : f.pr.N;
  for (int64_t e = blockIdx.x * (int64_t)FX_NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * FX_NT) {
    const int64_t i = f.list ? (int64_t)f.list[e] : e;
    int b = 0;
    if (f.list) {
      b = fx_bin(f, sp, eq, eqk, fx_key(f, (uint32_t)e));
    } else {
      double G;
      const bool cand = fx_user(f, i, G);
      if (cand) b = fx_bin_of(sp, nb, dkey(G + 0.0));
      f.bin[i] = cand ? (uint8_t)b : (uint8_t)FX_NONE;
      if (!cand) continue;
    }
    atomicAdd(&hc[b], 1u);
    XSum *row = hs + (size_t)b * nv;
    for (uint64_t m = fx_sel(f, i); m; m &= m - 1) {
      fx_row(f.pr, f.d, i * M + __ffsll((long long)m) - 1, [&](int k, float c) {
        if ((unsigned)k >= (unsigned)K || !(c > 0.0f)) return;
        const int v = f.kv[k];
        if (v >= 0 && f.act[v]) xs_atomic_add(&row[v], (double)c);
      });
    }
  }
  if (!lds) return;
  __syncthreads();
  for (int t = threadIdx.x; t < nb * nv; t += FX_NT)
    if (xs_nonzero(hs[t])) xs_atomic_add_sum(&f.hsum[t], hs[t]);
  for (int t = threadIdx.x; t < nb; t += FX_NT)
    if (hc[t]) atomicAdd(&f.hcnt[t], hc[t]);
}

__device__ __forceinline__ XSum fx_scan_up(XSum v, int lane) {   // sum of the lanes up to this one
  #pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const long long h = __shfl_up(v.hi, d, 64), l = __shfl_up(v.lo, d, 64);
    if (lane >= d) { v.hi += h; v.lo += l; }
  }
  return v;
}

// per open slot: the first bin whose prefix covers it, exactly (covered:
// total - removed <= B); the boundary's bin is the largest.  A wave per slot,
// a lane per bin (one thread per slot walking the bins took 30-45 us).
#define FL_NT 1024
__global__ void __launch_bounds__(FL_NT) k_fix_locate(FixArgs f, int level) {
  __shared__ int bst;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid == 0) bst = -1;
  __syncthreads();
  const int nb = f.nb;
  for (int v = wv; v < f.nv; v += FL_NT / 64) {
    int vb = -1;
    if (f.act[v]) {
      XSum T = f.tot[v];
      if (level == 0) {
        XSum s = xs_zero();
        for (int b = lane; b < nb; b += 64) s = xs_plus(s, f.hsum[(size_t)b * f.nv + v]);
        for (int d = 32; d > 0; d >>= 1) { s.hi += __shfl_xor(s.hi, d, 64); s.lo += __shfl_xor(s.lo, d, 64); }
        T = s;
        if (lane == 0) f.tot[v] = T;
      }
      const double Bk = f.Bv[v];
      if (level > 0 || xs_gt(T, Bk)) {
        XSum S = f.cthr[v];   // removed before the bins of this chunk of 64
        for (int b0 = 0; b0 < nb && vb < 0; b0 += 64) {
          const int b = b0 + lane;
          const XSum h = b < nb ? f.hsum[(size_t)b * f.nv + v] : xs_zero();
          const XSum in = xs_plus(S, fx_scan_up(h, lane));
          const uint64_t ok = __ballot(b < nb && !xs_gt(xs_minus(T, in), Bk));
          int at = ok ? __ffsll((long long)ok) - 1 : -1;
          if (!ok && b0 + 64 >= nb) at = nb - 1 - b0;   // (the last bin covers: exact sums)
          if (at >= 0) {
            vb = b0 + at;
            const XSum ex = xs_minus(in, h);
            XSum c;
            c.hi = __shfl(ex.hi, at, 64);
            c.lo = __shfl(ex.lo, at, 64);
            if (lane == 0) f.cthr[v] = c;
          } else {
            S.hi = __shfl(in.hi, 63, 64);
            S.lo = __shfl(in.lo, 63, 64);
          }
        }
      }
    }
    if (lane == 0) {
      f.act[v] = vb;   // (turned into a flag below)
      atomicMax(&bst, vb);
    }
  }
  __syncthreads();
  for (int v = tid; v < f.nv; v += FL_NT) f.act[v] = bst >= 0 && f.act[v] == bst ? 1 : 0;
  if (tid == 0) {
    unsigned long long before = 0;
    for (int b = 0; b < bst; ++b) before += f.hcnt[b];
    f.fs->bstar = bst;
    f.fs->nstar = bst >= 0 ? f.hcnt[bst] : 0u;
    f.fs->napp = 0u;
    f.fs->nreset += before;
  }
  __syncthreads();
  for (size_t t = tid; t < (size_t)nb * f.nv; t += FL_NT) f.hsum[t] = xs_zero();
  for (int t = tid; t < nb; t += FL_NT) f.hcnt[t] = 0u;
}

// clear item row r of a reset user; its consumption goes to rem, its profit
// to the thread's own sum
__device__ __forceinline__ void fx_clear(const FixArgs &f, int64_t r, XSum *rem, XSum &profit) {
  if (!f.x[r]) return;
  f.x[r] = 0;
  xs_add(profit, (double)f.pr.p[r]);
  fx_row(f.pr, f.d, r, [&](int k, float c) {
    if ((unsigned)k < (unsigned)f.pr.K && c != 0.0f) xs_atomic_add(&rem[k], (double)c);
  });
}
__device__ __forceinline__ void fx_profit(const FixArgs &f, XSum profit, int lane) {
  for (int d = 32; d > 0; d >>= 1) { profit.hi += __shfl_xor(profit.hi, d, 64); profit.lo += __shfl_xor(profit.lo, d, 64); }
  if (lane == 0 && xs_nonzero(profit)) xs_atomic_add_sum(&f.rem[f.pr.K], profit);
}

// Chunks of 256 ipt users (or list entries; ipt 16 reads the bin bytes 16 at a
// time, 1 spreads a small instance over the compute units): those of the bins before the
// boundary's are reset, those of its bin appended to the next list.  Both are
// queued in LDS first, so that a wave takes 64 users (item rows) that need
// the work instead of the few among 64 that do.
__global__ void __launch_bounds__(FX_NT) k_fix_split_off(FixArgs f, int ipt, int lds) {
  extern __shared__ __align__(16) unsigned char fsm[];
  __shared__ uint16_t qr[FX_CHUNK], qs[FX_CHUNK];
  __shared__ uint32_t nr, nq, base;
  __shared__ uint64_t sp[128];
  const int tid = threadIdx.x, K = f.pr.K, M = f.pr.M;
  const int bst = f.fs->bstar;
  if (bst < 0) return;
  XSum *rem = lds ? (XSum *)fsm : f.rem;
  if (lds)
    for (int t = tid; t < K; t += FX_NT) rem[t] = xs_zero();
  const int eq = f.fs->eq;
  const uint64_t eqk = f.fs->eqk;
  for (int t = tid; t < f.nb - 1; t += FX_NT) sp[t] = f.split[t];
  XSum profit = xs_zero();
  const int64_t n = f.list ? (int64_t)f.nlist : f.pr.N;
  const int64_t chunk = (int64_t)FX_NT * ipt, nch = (n + chunk - 1) / chunk;
  for (int64_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
    __syncthreads();
    if (tid == 0) { nr = 0; nq = 0; }
    __syncthreads();
    const int64_t e0 = ch * chunk;
    const int c0 = tid * FX_IPT;
    if (f.list || ipt < FX_IPT) {
      for (int q = 0; q < ipt; ++q) {
        const int c = q * FX_NT + tid;
        if (e0 + c >= n) break;
        const int bin = f.list ? 0 : (int)f.bin[e0 + c];
        if (bin == (int)FX_NONE) continue;
        const int b = f.list ? fx_bin(f, sp, eq, eqk, fx_key(f, (uint32_t)(e0 + c))) : bin;
        if (b < bst) qr[atomicAdd(&nr, 1u)] = (uint16_t)c;
        else if (b == bst) qs[atomicAdd(&nq, 1u)] = (uint16_t)c;
      }
    } else {
      uint8_t bb[FX_IPT];
      if (e0 + c0 + FX_IPT <= n) {
        const uint4 w = *(const uint4 *)(f.bin + e0 + c0);
        const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
        for (int q = 0; q < FX_IPT; ++q) bb[q] = (uint8_t)(ws[q >> 2] >> (8 * (q & 3)));
      } else {
        for (int q = 0; q < FX_IPT; ++q) bb[q] = e0 + c0 + q < n ? f.bin[e0 + c0 + q] : (uint8_t)FX_NONE;
      }
      for (int q = 0; q < FX_IPT; ++q) {
        if (bb[q] == FX_NONE) continue;
        if ((int)bb[q] < bst) qr[atomicAdd(&nr, 1u)] = (uint16_t)(c0 + q);
        else if ((int)bb[q] == bst) qs[atomicAdd(&nq, 1u)] = (uint16_t)(c0 + q);
      }
    }
    __syncthreads();
    if (tid == 0 && nq) base = atomicAdd(&f.fs->napp, nq);
    __syncthreads();
    for (uint32_t t = tid; t < nq; t += FX_NT) {
      const int64_t e = e0 + qs[t];
      const int64_t i = f.list ? (int64_t)f.list[e] : e;
      uint64_t key;
      if (f.list) {
        key = f.lkey[e];
      } else {
        double G;
        fx_user(f, i, G);
        key = dkey(G + 0.0);
      }
      f.olist[base + t] = (uint32_t)i;
      f.okey[base + t] = key;
    }
    const uint32_t rows = nr * (uint32_t)M;
    for (uint32_t t = tid; t < rows; t += FX_NT) {
      const uint32_t u = t / (uint32_t)M;
      const int64_t e = e0 + qr[u];
      const int64_t i = f.list ? (int64_t)f.list[e] : e;
      fx_clear(f, i * M + (t - u * (uint32_t)M), rem, profit);
    }
  }
  fx_profit(f, profit, tid & 63);
  if (!lds) return;
  __syncthreads();
  for (int t = tid; t < K; t += FX_NT)
    if (xs_nonzero(rem[t])) xs_atomic_add_sum(&f.rem[t], rem[t]);
}

// The last users around the boundary (a list of at most FX_LAST): sorted by
// (key, index); per open slot the shortest prefix that covers it, the longest
// of which is reset.  A longer list is left for another level.
__global__ void __launch_bounds__(FX_LAST) k_fix_last(FixArgs f) {
  __shared__ uint64_t key[FX_LAST];
  __shared__ uint32_t idx[FX_LAST];
  __shared__ XSum part[FX_LAST / 64];
  __shared__ uint32_t first, tstar;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint32_t n = f.fs->bstar < 0 ? 0u : f.fs->nstar;
  if (n == 0 || n > FX_LAST) return;
  key[tid] = tid < (int)n ? f.okey[tid] : ~0ull;
  idx[tid] = tid < (int)n ? f.olist[tid] : 0xFFFFFFFFu;
  if (tid == 0) tstar = 0;
  __syncthreads();
  uint32_t P2 = 2;
  while (P2 < n) P2 <<= 1;
  for (uint32_t size = 2; size <= P2; size <<= 1) {
    for (uint32_t stp = size >> 1; stp > 0; stp >>= 1) {
      const uint32_t t = tid, o = t ^ stp;
      if (t < P2 && o > t) {
        const uint64_t a = key[t], b = key[o];
        const uint32_t ia = idx[t], ib = idx[o];
        const bool gt = a > b || (a == b && ia > ib);
        if (((t & size) == 0) == gt) { key[t] = b; key[o] = a; idx[t] = ib; idx[o] = ia; }
      }
      __syncthreads();
    }
  }
  for (int v = 0; v < f.nv; ++v) {
    if (!f.act[v]) continue;   // (the same for every thread)
    if (tid == 0) first = n - 1;
    const XSum in = fx_scan_up(tid < (int)n ? fx_use(f, (int64_t)idx[tid], f.vk[v]) : xs_zero(), lane);
    if (lane == 63) part[wv] = in;
    __syncthreads();
    XSum S = xs_plus(f.cthr[v], in);
    for (int w = 0; w < wv; ++w) S = xs_plus(S, part[w]);
    if (tid < (int)n && !xs_gt(xs_minus(f.tot[v], S), f.Bv[v])) atomicMin(&first, (uint32_t)tid);
    __syncthreads();
    if (tid == 0 && first + 1 > tstar) tstar = first + 1;
    __syncthreads();
  }
  __syncthreads();
  const uint32_t rows = tstar * (uint32_t)f.pr.M;
  XSum profit = xs_zero();
  for (uint32_t t = tid; t < rows; t += FX_LAST) {
    const uint32_t u = t / (uint32_t)f.pr.M;
    fx_clear(f, (int64_t)idx[u] * f.pr.M + (t - u * (uint32_t)f.pr.M), f.rem, profit);
  }
  fx_profit(f, profit, lane);
  if (tid == 0) f.fs->nreset += tstar;
}

__global__ void k_fix_final(FixArgs f, const double *R, const double *P, double *R_out, double *P_out,
                            int64_t *n_reset) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  const int K = f.pr.K;
  if (c > K) return;
  const double s = xs_to_double(f.rem[c]);
  if (c < K) {
    R_out[c] = R[c] - s;
  } else {
    *P_out = *P - s;
    *n_reset = (int64_t)f.fs->nreset;
  }
}

// bins of the post-processing: the most (a power of two, 4 to 128) whose sums
// over nv slots fit in budget bytes (4: whatever they take)
int kp_fixup_bins(int nv, size_t budget) {
  int nb = 128;
  while (nb > 4 && (size_t)nb * nv * sizeof(XSum) > budget) nb >>= 1;
  return nb;
}

namespace {
struct FxLayout {
  size_t bin, split, hsum, hcnt, fs, tot, cthr, act, rem, key[2], idx[2], total;
};
FxLayout fx_layout(int64_t N, int nv, int K) {
  FxLayout L;
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
  // the bin arrays at their largest (at most 128 bins and 40 KB of sums, or
  // four rows), so that a layout never outgrows the one for more slots
  L.bin = take((size_t)N + 16);
  L.split = take(128 * 8);
  L.hsum = take(std::max<size_t>(40 * 1024, 4 * (size_t)nv * sizeof(XSum)));
  L.hcnt = take(128 * 4);
  L.fs = take(sizeof(FixState));
  L.tot = take((size_t)nv * sizeof(XSum));
  L.cthr = take((size_t)nv * sizeof(XSum));
  L.act = take((size_t)nv * 4);
  L.rem = take((size_t)(K + 1) * sizeof(XSum));
  for (int q = 0; q < 2; ++q) {
    L.key[q] = take((size_t)N * 8 + 8);
    L.idx[q] = take((size_t)N * 4 + 4);
  }
  L.total = off;
  return L;
}
}  // namespace

size_t kp_fixup_scratch_bytes(int64_t N, int nv, int K) { return fx_layout(N, nv, K).total; }

// kv / vk / Bv: device arrays of the violated slots; nb: bins (4 to 128; more
// than four: nb * nv sums within 40 KB); pinned: 64 bytes of pinned host
// memory; persist_all: blocks of the user passes at most; bins_pass: launches the per-user
// bin pass (k_fix_bins when empty).  Synchronizes the stream once, and once
// per level that a large list takes.
hipError_t kp_launch_fixup_pipeline(ProbDev pr, int row_d, uint8_t *x, const double *lam, const int *kv,
                                    const int *vk, const double *Bv, int nv, int nb, const double *R,
                                    const double *P,
                                    double *R_out, double *P_out, int64_t *n_reset, void *scratch,
                                    hipStream_t stream, uint32_t *pinned, int persist_all,
                                    const std::function<hipError_t(const FixBins &)> &bins_pass) {
  const int64_t N = pr.N;
  const int K = pr.K;
  const FxLayout L = fx_layout(N, nv, K);
  char *w = (char *)scratch;
  FixArgs f;
  memset(&f, 0, sizeof f);
  f.pr = pr;
  f.d = pr.fmt == 0 ? 0 : row_d;
  f.x = x;
  f.lam = lam;
  f.kv = kv;
  f.vk = vk;
  f.Bv = Bv;
  f.nv = nv;
  if (nb < 4 || nb > 128 || (nb > 4 && (size_t)nb * nv * sizeof(XSum) > 40 * 1024)) return hipErrorInvalidValue;
  f.nb = nb;
  f.split = (uint64_t *)(w + L.split);
  f.bin = (uint8_t *)(w + L.bin);
  f.hsum = (XSum *)(w + L.hsum);
  f.hcnt = (uint32_t *)(w + L.hcnt);
  f.fs = (FixState *)(w + L.fs);
  f.tot = (XSum *)(w + L.tot);
  f.cthr = (XSum *)(w + L.cthr);
  f.act = (int *)(w + L.act);
  f.rem = (XSum *)(w + L.rem);
  f.olist = (uint32_t *)(w + L.idx[0]);
  f.okey = (uint64_t *)(w + L.key[0]);
  const size_t lb = (size_t)nb * nv * sizeof(XSum) + (size_t)nb * 4 + 8 + (size_t)nb * 8;
  const int bins_lds = lb <= FX_LDS_MAX;
  const size_t lb_used = bins_lds ? lb : (size_t)nb * 8;
  const int rem_lds = (size_t)K * sizeof(XSum) <= FX_LDS_MAX / 2;
  const size_t lr = rem_lds ? (size_t)K * sizeof(XSum) : 0;
  hipLaunchKernelGGL(k_fix_init, dim3(16), dim3(256), 0, stream, f);
  hipError_t e;
  for (int level = 0;; ++level) {
    const int64_t n = f.list ? (int64_t)f.nlist : N;
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n + FX_NT - 1) / FX_NT, persist_all));
    const int ipt = n >= (int64_t)persist_all * FX_CHUNK ? FX_IPT : 1;
    const int chunks = (int)std::max<int64_t>(1, std::min<int64_t>((n + FX_NT * ipt - 1) / (FX_NT * ipt), persist_all));
    hipLaunchKernelGGL(k_fix_splits, dim3(1), dim3(1024), 0, stream, f);
    if (level == 0 && bins_pass) {
      FixBins fb;
      fb.bin = f.bin;
      fb.kv = kv;
      fb.split = f.split;
      fb.hsum = f.hsum;
      fb.hcnt = f.hcnt;
      fb.nb = f.nb;
      fb.nv = nv;
      if ((e = bins_pass(fb)) != hipSuccess) return e;
    } else {
      hipLaunchKernelGGL(k_fix_bins, dim3(blocks), dim3(FX_NT), lb_used, stream, f, bins_lds);
    }
    hipLaunchKernelGGL(k_fix_locate, dim3(1), dim3(FL_NT), 0, stream, f, level);
    hipLaunchKernelGGL(k_fix_split_off, dim3(chunks), dim3(FX_NT), lr, stream, f, ipt, rem_lds);
    hipLaunchKernelGGL(k_fix_last, dim3(1), dim3(FX_LAST), 0, stream, f);
    if ((e = hipMemcpyAsync(pinned, f.fs, sizeof(FixState), hipMemcpyDeviceToHost, stream)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(stream)) != hipSuccess) return e;
    FixState hs;
    memcpy(&hs, pinned, sizeof hs);
    if (hs.bstar < 0 || hs.nstar <= FX_LAST) break;
    // a longer list: cut again (in the order of the indices once every key
    // of the list is known to be equal)
    if (level > 256) return hipErrorUnknown;   // (every level takes users off the list)
    f.byidx = f.byidx || (f.list && hs.eq && hs.bstar == 1);
    f.list = f.olist;
    f.lkey = f.okey;
    f.nlist = hs.nstar;
    f.olist = (uint32_t *)(w + L.idx[(level + 1) & 1]);
    f.okey = (uint64_t *)(w + L.key[(level + 1) & 1]);
  }
  hipLaunchKernelGGL(k_fix_final, dim3((K + 1 + 255) / 256), dim3(256), 0, stream, f, R, P, R_out, P_out,
                     n_reset);
  return hipGetLastError();
}
