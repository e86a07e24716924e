// gfx950 kernels of the per-user subproblem sweep.
//
// One block (256 threads, four wave64s) processes tiles of U users at a time:
//   phase 0  the tile's costs b are staged in LDS as a dense [U][M][K] tile
//            (coalesced 16-byte loads for dense b, a per-row scatter for CSR),
//   phase A  one thread per item row computes the cost-adjusted profit
//            p~ = p - sum_k lambda_k b_k  (FP64, k ascending, no FMA),
//   phase B1 one thread per user ranks its items by (p~ desc, index asc) and
//            runs the hierarchical greedy (Alg.1, as the equivalent laminar
//            matroid greedy on bitmasks),
//   phase B2 reduces consumption and, for SCD, looks at every (user, knapsack)
//            pair: those that a filter does not settle are queued, dealt over
//            the block and walked along the user's consumption step function
//            in lambda_k over the pass's range (the breakpoints of Alg.3/4),
//            which are binned or emitted.
// R, g and P are summed in a fixed order: per (user,k) values go to LDS and
// are added in user order, per block into a private slot, and slots are
// added in block order by a second kernel.  The threshold search's sums
// (histogram bins, window corrections) are exact two-limb integers added
// with integer atomics, so their order does not matter.  This file also
// holds the batched sweep, the statistics' reductions and the input checks
// (the threshold search's state machine: kp_search.hip; the post-processing:
// kp_fixup.hip).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>
#include <type_traits>
#include <algorithm>
#include <functional>
#include "kp_internal.h"

#define NT 256

#include "kp_device.h"

// ---------------------------------------------------------------------------
// the sweep kernel
// ---------------------------------------------------------------------------
typedef float v4f __attribute__((ext_vector_type(4)));
#define CH 8      // prefetched 16-byte chunks of dense costs per thread and tile
#define PCH 4     // prefetched profits (and CSR row offsets) per thread and tile
#define ECH 8     // prefetched CSR entries per thread and tile

// Register-resident copy of one tile's inputs, loaded one tile ahead so the
// loads overlap the previous tile's compute.
struct Prefetch {
  v4f b4[CH];
  float pv[PCH];
  int64_t rp[PCH];      // CSR: rowptr of the rows this thread scores
  int64_t rp_end;       // CSR: rowptr one past the tile (valid in thread 0)
  int32_t ec[ECH];      // CSR entries of the tile, cooperative layout
  float ev[ECH];
};

template <int FMT>
__device__ __forceinline__ void issue_rows(Prefetch &f, const ProbDev &pr, int64_t u0, int nr, int K,
                                           int tid, int aligned) {
  // profits (all formats) and, for CSR, the row offsets
  #pragma unroll
  for (int i = 0; i < PCH; ++i) {
    const int r = tid + i * NT;
    if (r < nr) {
      f.pv[i] = __builtin_nontemporal_load(pr.p + u0 * pr.M + r);
      if (FMT == 1) f.rp[i] = pr.rowptr[u0 * pr.M + r];
    }
  }
  if (FMT == 1 && tid == 0) f.rp_end = pr.rowptr[u0 * pr.M + nr];
  if (FMT == 0 && aligned) {
    const float *src = pr.b + u0 * (int64_t)pr.M * K;
    const int n4 = (nr * K) >> 2;
    const v4f *s4 = (const v4f *)src;
    #pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int t = tid + i * NT;
      if (t < n4) f.b4[i] = __builtin_nontemporal_load(s4 + t);
    }
  }
}

__device__ __forceinline__ void issue_entries(Prefetch &f, const ProbDev &pr, int64_t e0, int64_t e1,
                                              int tid) {
  #pragma unroll
  for (int i = 0; i < ECH; ++i) {
    const int64_t e = e0 + tid + (int64_t)i * NT;
    if (e < e1) {
      f.ec[i] = __builtin_nontemporal_load(pr.col + e);
      f.ev[i] = __builtin_nontemporal_load(pr.val + e);
    }
  }
}

// A window that does not contain lambda_k^t, dense costs, at most one binding
// set (mask m1, cap c1): the lines moved to the window's centre c,
// z'_j = p~_j - (c - lambda_k^t) b_jk.  Over the window (radius r around c) a
// line moves by at most r b_jk, so the selection at c stays the same when
// the selected lines stay farther than r bmax (plus a rounding margin) from
// the others of the set and from zero.  In two parts.  First pass: zmax, the selection outside the set (whose moving
// members must keep their sign: the smallest |z'| among those that may be
// positive is checked against the bound), and the set's positive members
// with their smallest z' and the best other members (all of them; moving
// ones).  Lines at or below -Hs
// never turn positive in the window (Hs may be an upper bound of the
// window's reach: the tests only grow more cautious).
struct FarPass {
  double zmax = 0.0, nearz = INFINITY;
  bool anyn = false;
  uint64_t sel = 0, posm = 0;
  double minpos = INFINITY, bestneg = -INFINITY, bestnegA = -INFINITY;
};
__device__ __forceinline__ void far_item(FarPass &f, double z, int j, bool moving, bool member, double Hs) {
  if (z > -Hs) f.zmax = fmax(f.zmax, fabs(z));
  if (member) {
    if (z > 0.0) {
      f.posm |= 1ull << j;
      f.minpos = fmin(f.minpos, z);
    } else {
      f.bestneg = fmax(f.bestneg, z);
      if (moving) f.bestnegA = fmax(f.bestnegA, z);
    }
  } else {
    if (moving && z > -Hs) { f.nearz = fmin(f.nearz, fabs(z)); f.anyn = true; }
    if (z > 0.0) f.sel |= 1ull << j;
  }
}
// The rest of the test from its first pass (Hs: the exact reach r bmk plus
// margin): at most c1 positive members -- T is all of them, the best member
// left out the best of the others; more -- T by passes over the set.
__device__ __forceinline__ bool far_finish(const FarPass &f, const double *zu, const float *bu, int M, int K,
                                           int k, uint64_t A, double lk, double dl, double r, double bmk,
                                           double Hs, uint64_t m1, int c1, double *cw) {
  const double bound = r * bmk * (1.0 + 0x1p-30) + 0x1p-36 * (1.0 + f.zmax + Hs + (lk + fabs(dl) + r) * bmk);
  if (f.anyn && !(f.nearz > bound)) return false;   // may change sign
  auto moved = [&](int j) -> double {
    const double b = (A >> j & 1) ? (double)bu[j * K + k] : 0.0;
    const double s = dl * b;
    return zu[j] - s;
  };
  uint64_t sel = f.sel;
  const int npos = popc64(f.posm);
  if (npos <= c1) {
    // at most c1 positive members: T is all of them, the best member left
    // out the best of the others (the same tests as below, no more passes)
    if (npos == c1 && f.bestneg > -Hs && !(f.minpos - f.bestneg > bound)) return false;
    if (npos > 0 && !(f.minpos > bound)) return false;
    if (npos < c1 && !(f.bestnegA < -bound)) return false;
    sel |= f.posm;
    double sum = 0.0;
    for (uint64_t m = sel & A; m; m &= m - 1) {
      const int j = __ffsll((long long)m) - 1;
      sum = sum + (double)bu[j * K + k];
    }
    *cw = sum;
    return true;
  }
  // more: T, the c1 best positive members (z' desc, index asc), taken two
  // per pass over the set (the second best of a pass is the best once the
  // first has joined T)
  uint64_t inT = 0;
  int nt = 0;
  double minT = INFINITY;
  for (;;) {
    double v1 = -INFINITY, v2 = -INFINITY;
    int j1 = -1, j2 = -1;
    #pragma unroll 4
    for (int j = 0; j < M; ++j) {
      if (!(m1 >> j & 1) || (inT >> j & 1)) continue;
      const double z = moved(j);
      if (z > v1) { v2 = v1; j2 = j1; v1 = z; j1 = j; }
      else if (z > v2) { v2 = z; j2 = j; }
    }
    bool done = false;
    for (int h = 0; h < 2 && !done; ++h) {
      const double best = h == 0 ? v1 : v2;
      const int bj = h == 0 ? j1 : j2;
      if (bj < 0) { done = true; break; }
      if (nt < c1 && best > 0.0) {
        inT |= 1ull << bj;
        minT = best;
        ++nt;
        continue;
      }
      // bj: the best member outside T
      if (nt == c1 && best > -Hs && !(minT - best > bound)) return false;
      done = true;
    }
    if (done) break;
  }
  if (nt > 0 && !(minT > bound)) return false;
  if (nt < c1) {
    // room is left: no moving member outside T may turn positive
    #pragma unroll 4
    for (int j = 0; j < M; ++j) {
      if (!(m1 >> j & 1) || (inT >> j & 1) || !(A >> j & 1)) continue;
      if (!(moved(j) < -bound)) return false;
    }
  }
  sel |= inT;
  double sum = 0.0;
  for (uint64_t m = sel & A; m; m &= m - 1) {
    const int j = __ffsll((long long)m) - 1;
    sum = sum + (double)bu[j * K + k];
  }
  *cw = sum;
  return true;
}

// MX, KX: the item and knapsack counts when they are fixed at compile time
// (dense costs with M = K = 10, or M = 20 and K = 50), else 0: the loops
// over the items and the knapsacks then have constant trip counts (c2 SCD
// step 3.50 -> 3.25 ms; c4 SCD 28.4 -> 27.6 ms, DD 9.02 -> 8.58 ms).
template <int FMT, bool SCD, int MX = 0, int KX = 0>
__device__ __forceinline__ void sweep_body(const SweepArgs &a, const TileGeom &g, const int bid,
                                           const int nblk, unsigned char *smem) {
  const int tid = threadIdx.x;
  const int M = MX ? MX : g.M, K = KX ? KX : g.K, U = g.U;
  const int R = U * M;             // item rows per tile
  const int Q = U * K;             // (user, knapsack) pairs per tile
  // ---- LDS carve-up (byte offsets are multiples of 16) ----
  size_t off = 0;
  auto carve = [&](size_t bytes) { unsigned char *p = smem + off; off += (bytes + 15) & ~(size_t)15; return p; };
  float *bt = (float *)carve((size_t)R * K * 4);          // [U][M][K]
  double *pt = (double *)carve((size_t)R * 8);            // [U][M]
  uint8_t *perm = (uint8_t *)carve((size_t)R);            // [U][M] rank -> item
  uint64_t *Sm = (uint64_t *)carve((size_t)U * 8);        // greedy set at lambda^t
  uint64_t *Pm = (uint64_t *)carve((size_t)U * 8);        // items with p~ > 0
  int8_t *tau = (int8_t *)carve(SCD ? (size_t)U * 2 : 0); // per user: the threshold elements (at most one set)
  uint64_t *Am = (uint64_t *)carve(SCD && FMT == 1 ? (size_t)Q * 8 : 0);  // CSR: items with an entry, per (user, knapsack)
  double *vk = (double *)carve((size_t)Q * 8);            // per (user,k) consumption
  uint32_t *nwq = (uint32_t *)carve(SCD ? 16 : 0);            // pairs left to look at, to walk
  double *uPG = (double *)carve((size_t)U * 16);          // per user P_i, G_i
  double *acc = (double *)carve((size_t)(K + 2) * 8);     // block running sums
  double *lam = (double *)carve((size_t)K * 8);           // lambda^t staged once per block
  float *pl = (float *)carve((size_t)R * 4);              // staged profits
  int32_t *rpl = (int32_t *)carve((size_t)(R + 1) * 4);   // CSR: row offsets relative to the tile
  // CSR: staged entries (SCD: at most 64 knapsacks, a byte each; 255: malformed)
  void *eclv = carve(FMT == 1 ? (size_t)NT * ECH * (SCD ? 1 : 4) : 0);
  int32_t *ecl = (int32_t *)eclv;
  uint8_t *ecb = (uint8_t *)eclv;
  float *evl = (float *)carve(FMT == 1 ? (size_t)NT * ECH * 4 : 0);
  // the (user, knapsack) pairs left to look at, those with a breakpoint to
  // find (bit 15: from the top) and the sets their walks start with; CSR: over
  // the staged entries, which the scores have consumed by then
  auto qcarve = [&](size_t bytes, size_t &at) {
    if (FMT == 0) return carve(bytes);
    unsigned char *p = (unsigned char *)evl + at;
    at += (bytes + 15) & ~(size_t)15;
    return p;
  };
  size_t qat = 0;
  uint64_t *wS = (uint64_t *)qcarve(SCD ? (size_t)Q * 8 : 0, qat);
  uint16_t *wq = (uint16_t *)qcarve(SCD ? (size_t)Q * 2 : 0, qat);
  uint16_t *wq2 = (uint16_t *)qcarve(SCD ? (size_t)Q * 2 : 0, qat);
  if (FMT == 1 && qat > (size_t)NT * ECH * 4) carve(qat - (size_t)NT * ECH * 4);   // (beyond them)
  int64_t *ebase = (int64_t *)carve(16);                  // CSR: first entry of the next tile
  KWalk *kst = SCD ? (KWalk *)carve((size_t)K * sizeof(KWalk)) : nullptr;
  XSum *hs = nullptr;
  uint32_t *hc = nullptr;
  const bool hist = !a.no_hist;   // histograms (exponential buckets, refinement bins) in LDS
  int *kmode = nullptr;
  uint32_t *kcnt = nullptr, *kpos = nullptr, *kovf = nullptr, *nstage = nullptr;
  unsigned long long *hmin = nullptr, *hmax = nullptr;
  double *kwide = nullptr, *ugap = nullptr;
  XSum *kxs = nullptr;
  if (SCD) {
    kwide = (double *)carve(16);                   // the widest window
    kxs = (XSum *)carve((size_t)K * sizeof(XSum)); // window corrections
    ugap = (double *)carve((size_t)U * 16);        // per user: gap and scale of the window filter
    if (hist) {
      hs = (XSum *)carve((size_t)K * KP_NB * sizeof(XSum));
      hc = (uint32_t *)carve((size_t)K * KP_NB * 4);
    }
    kmode = (int *)carve((size_t)K * 4);
    kcnt = (uint32_t *)carve((size_t)K * 4);
    kpos = (uint32_t *)carve((size_t)K * 4);
    kovf = (uint32_t *)carve((size_t)K * 4);
    hmin = (unsigned long long *)carve((size_t)K * 8);
    hmax = (unsigned long long *)carve((size_t)K * 8);
    nstage = (uint32_t *)carve(16);
  }
  SetTree tr;
  if (SCD) tr = set_tree_load(carve(set_tree_bytes(a.tree.L, M)), a.tree, M, tid, NT);
  for (int t = tid; t < K + 2; t += NT) acc[t] = 0.0;
  for (int t = tid; t < K; t += NT) lam[t] = a.lam[t];
  if (SCD) {
    for (int t = tid; t < K; t += NT) kst[t] = a.st[t];
    if (hist)
      for (int t = tid; t < K * KP_NB; t += NT) { hs[t] = xs_zero(); hc[t] = 0u; }
    for (int t = tid; t < K; t += NT) {
      kmode[t] = pass_mode(a, t);
      kcnt[t] = 0u;
      kpos[t] = 0u;
      kovf[t] = 0u;
      hmin[t] = ~0ull;
      hmax[t] = 0ull;
      kxs[t] = xs_zero();
    }
    if (tid == 0) {
      *nstage = 0u;
      double m = 0.0;
      for (int k = 0; k < K; ++k)
        if (pass_mode(a, k) == KS_WINDOW) m = a.st[k].hw > m ? a.st[k].hw : m;
      kwide[0] = m;
    }
  }
  const int64_t N = a.pr.N;
  if (SCD && !a.want_stats) {
    __syncthreads();
    __shared__ int busy;
    if (tid == 0) busy = 0;
    __syncthreads();
    for (int t = tid; t < K; t += NT)
      if (walk_mode(kmode[t])) busy = 1;
    __syncthreads();
    if (!busy) return;
  }

  // ---- software pipeline: prefetch tile bid ----
  // some cost is off the grid on which FP64 sums are exact (CSR: every entry of
  // the pass with the statistics; dense: the consumptions and the costs of
  // the pairs looked at, M times fewer than all)
  // (the units in vector registers: read from the kernel's arguments they cost
  // a scalar load and a wait at every use)
  uint32_t offg = 0;
  double gmag = SCD && a.want_stats ? a.gmag : 0.0;
  float ginv = SCD && (FMT == 0 || a.want_stats) ? a.ginv : 0.0f;
  if (SCD) __asm__ volatile("" : "+v"(ginv));
  if (SCD && FMT == 0) __asm__ volatile("" : "+v"(gmag));
  Prefetch f;
  int64_t tile = bid;
  if (tile < a.ntiles) {
    const int64_t u0 = SCD ? (tile * a.tstride + a.toff) * U : tile * (int64_t)U;
    const int nu = (int)((N - u0) < U ? (N - u0) : U);
    issue_rows<FMT>(f, a.pr, u0, nu * M, K, tid, g.aligned);
    if (FMT == 1) {
      if (tid == 0) { ebase[0] = a.pr.rowptr[u0 * M]; ebase[1] = f.rp_end; }
      __syncthreads();
      issue_entries(f, a.pr, ebase[0], ebase[1], tid);
    }
  }

  for (; tile < a.ntiles; tile += nblk) {
    const int64_t u0 = SCD ? (tile * a.tstride + a.toff) * U : tile * (int64_t)U;
    const int nu = (int)((N - u0) < U ? (N - u0) : U);     // users in this tile
    const int nr = nu * M;
    __syncthreads();   // previous tile's readers are done with the LDS tile
    // ---- store the prefetched tile into LDS ----
    int64_t e_first = 0;
    int n_ent = 0;
    bool full = false;
    #pragma unroll
    for (int i = 0; i < PCH; ++i) {
      const int r = tid + i * NT;
      if (r < nr) pl[r] = f.pv[i];
    }
    if (FMT == 0) {
      const float *src = a.pr.b + u0 * (int64_t)M * K;
      const int nf = nr * K;
      if (g.aligned) {
        const int n4 = nf >> 2;
        v4f *d4 = (v4f *)bt;
        #pragma unroll
        for (int i = 0; i < CH; ++i) {
          const int t = tid + i * NT;
          if (t < n4) d4[t] = f.b4[i];
        }
        // beyond the prefetched chunks, and the ragged tail: direct loads
        const v4f *s4 = (const v4f *)src;
        for (int t = tid + CH * NT; t < n4; t += NT) d4[t] = s4[t];
        for (int t = (n4 << 2) + tid; t < nf; t += NT) bt[t] = src[t];
      } else {
        for (int t = tid; t < nf; t += NT) bt[t] = src[t];
      }
    } else {
      e_first = ebase[0];
      n_ent = (int)(ebase[1] - ebase[0]);
      #pragma unroll
      for (int i = 0; i < PCH; ++i) {
        const int r = tid + i * NT;
        if (r < nr) rpl[r] = (int32_t)(f.rp[i] - e_first);
      }
      if (tid == 0) rpl[nr] = n_ent;
      #pragma unroll
      for (int i = 0; i < ECH; ++i) {
        const int t = tid + i * NT;
        if (t < n_ent && t < NT * ECH) {
          if (SCD) ecb[t] = (uint8_t)((unsigned)f.ec[i] < 255u ? f.ec[i] : 255);
          else ecl[t] = f.ec[i];
          evl[t] = f.ev[i];
        }
      }
      for (int t = tid; t < R * K; t += NT) bt[t] = 0.0f;
      // rows with an entry in most knapsacks are looked at as dense ones: their
      // items' bits cost an LDS atomic each, and walking them one by one lost
      // to the plain loop (M = 16, K = 8, full rows, 2e5 users: a sweep with
      // windows 0.30 -> 0.26 ms, with windows away from lambda^t 0.73 -> 0.45)
      full = SCD && 2 * n_ent > nr * K;
      if (SCD && !full)
        for (int t = tid; t < Q; t += NT) Am[t] = 0ull;
    }
    // ---- issue the next tile's loads (they land during this tile's compute) ----
    const int64_t ntile = tile + nblk;
    int64_t nu0 = 0;
    int nnr = 0;
    if (ntile < a.ntiles) {
      nu0 = SCD ? (ntile * a.tstride + a.toff) * U : ntile * (int64_t)U;
      nnr = (int)((N - nu0) < U ? (N - nu0) : U) * M;
      issue_rows<FMT>(f, a.pr, nu0, nnr, K, tid, g.aligned);
    }
    // at most one (pruned) set, e.g. top-Q: every row decides its own
    // selection in the rank phase; the users' masks start empty
    const bool fastsel = a.tree.L <= 1;
    if (fastsel && tid < nu) Sm[tid] = 0ull;
    // with at most one set the threshold elements follow from two items per
    // user, found by the rank phase: [0] the set's lowest selected member
    // (set full) and [1] its best positive member left out
    const bool fastau = SCD && fastsel;
    if (fastau && tid < nu) { tau[2 * tid] = -1; tau[2 * tid + 1] = -1; }
    if (SCD && tid == 0) { nwq[0] = 0u; nwq[1] = 0u; nwq[2] = full ? 1u : 0u; }
    // window filter, per user: [0] the smallest gap (a minimum over the
    // rows, taken on the bits of non-negative doubles), [1] the largest cost
    // (a maximum over the rows, on the bits of a non-negative float)
    if (SCD && tid < nu) {
      ((unsigned long long *)ugap)[2 * tid] = (unsigned long long)__double_as_longlong(1e300);
      ((unsigned int *)ugap)[4 * tid + 2] = 0u;
    }
    __syncthreads();
    // ---- phase A: scores ----
    if (FMT == 0) {
      for (int r = tid; r < nr; r += NT) {
        double accp = (double)pl[r];
        const float *br = bt + (size_t)r * K;
        #pragma unroll 4
        for (int k = 0; k < K; ++k) {
          const double prod = lam[k] * (double)br[k];
          accp = accp - prod;
        }
        pt[r] = accp;
      }
    } else {
      // CSR: scatter each row's stored entries into the dense tile and score
      // over the stored columns in ascending order (skipping zeros is
      // bit-identical: acc - lambda*0 == acc)
      for (int r = tid; r < nr; r += NT) {
        const int e0 = rpl[r], e1 = rpl[r + 1];
        double accp = (double)pl[r];
        for (int e = e0; e < e1; ++e) {
          int k;
          float v;
          if (e < NT * ECH) { k = SCD ? (int)ecb[e] : ecl[e]; v = evl[e]; }
          else { k = a.pr.col[e_first + e]; v = a.pr.val[e_first + e]; }   // tile beyond the staging
          if ((unsigned)k >= (unsigned)K) continue;   // malformed column: ignored (kp_validate_inputs reports it)
          bt[(size_t)r * K + k] = v;
          if (SCD) offg |= off_grid(v, ginv);
          if (SCD && !full && v > 0.0f) {
            const int u = r / M;
            atomicOr((unsigned long long *)&Am[u * K + k], 1ull << (r - u * M));
          }
          const double prod = lam[k] * (double)v;
          accp = accp - prod;
        }
        pt[r] = accp;
      }
    }
    __syncthreads();
    // ---- phase B1a: rank of every item of every user (one thread per row) ----
    const uint64_t m1 = a.tree.L == 1 ? a.tree.mask[0] : 0ull;
    const int c1 = a.tree.L == 1 ? a.tree.cap[0] : 0;
    for (int r = tid; r < nr; r += NT) {
      const int u = r / M, j = r - u * M;
      const double *z = pt + u * M;
      const double zj = z[j];
      int rank = 0, rank1 = 0;
      #pragma unroll 4
      for (int jj = 0; jj < M; ++jj) {
        const double zz = z[jj];
        const int beats = (zz > zj) || (zz == zj && jj < j);
        rank += beats;
        rank1 += beats & (int)(m1 >> jj & 1);
      }
      perm[u * M + rank] = (uint8_t)j;
      if (SCD && kwide[0] > 0.0) {
        // largest positive cost of the row (0 if none): the maximum below
        // is taken over the users' rows as unsigned bits, which order like
        // the floats for positive values
        const float *br = bt + (size_t)r * K;
        float mx = 0.0f;
        #pragma unroll 4
        for (int k = 0; k < K; ++k) mx = br[k] > mx ? br[k] : mx;
        if (mx > 0.0f) atomicMax((unsigned int *)ugap + 4 * u + 2, __float_as_uint(mx));
      }
      // Alg.1 with at most one set: a positive item is kept unless it is in
      // the set behind cap better members of it (those are positive too)
      if (fastsel && zj > 0.0 && (!(m1 >> j & 1) || rank1 < c1))
        atomicOr((unsigned long long *)&Sm[u], 1ull << j);
      if (fastau && zj > 0.0 && (m1 >> j & 1)) {
        if (rank1 == c1 - 1) tau[2 * u] = (int8_t)j;
        else if (rank1 == c1) tau[2 * u + 1] = (int8_t)j;
      }
    }
    // CSR: the next tile's entry range is known now that its row offsets have
    // landed; start those loads too
    if (FMT == 1 && ntile < a.ntiles) {
      if (tid == 0) { ebase[0] = f.rp[0]; ebase[1] = f.rp_end; }
    }
    __syncthreads();
    if (FMT == 1 && ntile < a.ntiles) issue_entries(f, a.pr, ebase[0], ebase[1], tid);
    // ---- phase B1b: the greedy, one thread per user ----
    if (tid < nu) {
      const int u = tid;
      const double *z = pt + u * M;
      uint64_t pos = 0;
      #pragma unroll 4
      for (int j = 0; j < M; ++j) if (z[j] > 0.0) pos |= 1ull << j;
      uint64_t S;
      if (fastsel) S = Sm[u];
      else if (SCD) S = greedy_mask(perm + u * M, M, pos, tr);
      else S = greedy_mask(perm + u * M, M, pos, a.tree);
      Sm[u] = S;
      Pm[u] = pos;
      // sums over the selected items in ascending index order
      double Pi = 0.0, Gi = 0.0;
      const float *pp = pl + u * M;
      for (uint64_t m = S; m; m &= m - 1) {
        const int j = __ffsll((long long)m) - 1;
        Pi = Pi + (double)pp[j];
        Gi = Gi + z[j];
      }
      uPG[2 * u] = Pi;
      uPG[2 * u + 1] = Gi;
      if (a.x_out) {
        uint8_t *xo = a.x_out + (u0 + u) * M;
        for (int j = 0; j < M; ++j) xo[j] = (uint8_t)(S >> j & 1);
      }
    }
    if (SCD && kwide[0] > 0.0) {
      // window filter, one thread per rank position: the smallest gap
      // between a user's p~ in rank order and between them and zero, over
      // the lines that can turn positive inside the widest window (ranks
      // descend, so those are a prefix of the ranks); two identical lines
      // (equal p~ and equal costs in every knapsack, e.g. the copies of a
      // categorical item) never cross
      const double hm = kwide[0];
      for (int q = tid; q < nr; q += NT) {
        const int u = q / M, rr = q - u * M;
        const float bm = __uint_as_float(((const unsigned int *)ugap)[4 * u + 2]);
        const double H = hm * (double)bm * (1.0 + 0x1p-30) + 0x1p-36 * (1.0 + (double)bm * hm);
        const double *z = pt + u * M;
        const int jv = perm[u * M + rr];
        const double v = z[jv];
        if (!(v > -H)) continue;
        double c = fabs(v);
        if (rr > 0) {
          const int jp = perm[u * M + rr - 1];
          const double prev = z[jp];
          bool same = prev == v;
          const float *ba = bt + ((size_t)u * M + jp) * K, *bb = bt + ((size_t)u * M + jv) * K;
          for (int k = 0; same && k < K; ++k) same = ba[k] == bb[k];
          if (!same) c = prev - v < c ? prev - v : c;
        }
        atomicMin((unsigned long long *)ugap + 2 * u, (unsigned long long)__double_as_longlong(c));
      }
    }
    __syncthreads();
    // ---- phase B2: one thread per (user, knapsack): its consumption, and
    // whether it can have a breakpoint in the pass's range.  The pairs left
    // are queued and walked by as many threads as there are pairs: without the
    // queue every wave took the walk's time for the few of its lanes that
    // needed one (pairs looked at: 11-26 % of them, walked: 3-12 %) ----
    auto look = [&](auto dense) {
      constexpr bool DN = decltype(dense)::value;   // dense costs, or CSR rows with an entry in most knapsacks
      for (int q = tid; q < nu * K; q += NT) {
        const int u = q / K, k = q - u * K;
        const uint64_t S0 = Sm[u];
        const float *bu = bt + (size_t)u * M * K;
        double v = 0.0;
        uint64_t A = 0;     // SCD: moving lines, b_jk > 0
        float bmk = 0.0f;   // SCD: their largest cost
        // a window away from lambda_k^t with at most one binding set: the
        // far-window test's first pass runs in the same pass over the items
        // (its cut at -Hs taken with the user's largest cost over every
        // knapsack, an upper bound of bmk: only more cautious); on CSR rows up
        // to a cap of 8: its passes over the set grow with the cap (M = 32,
        // K = 16, cap 20, 2e5 users: 2.0 ms a sweep without it, 2.3 with)
        bool fused = false, fused_ok = false;
        double fused_cw = 0.0;
        // a user with no line above -H (its gap record untouched) is calm in
        // every window: only its consumption is needed (A stays empty, so no
        // test or walk follows)
        const bool settled = SCD && kmode[k] == KS_WINDOW && kwide[0] > 0.0 && !(ugap[2 * u] < 1e300);
        if (settled) {
          for (uint64_t m = S0; m; m &= m - 1) v = v + (double)bu[(__ffsll((long long)m) - 1) * K + k];
        } else if (SCD) {
          double fr = 0.0, fdl = 0.0;
          if (DN && kmode[k] == KS_WINDOW && kst[k].far && a.tree.L <= 1 && kwide[0] > 0.0 &&
              (FMT == 0 || a.tree.L == 0 || a.tree.cap[0] <= 8)) {
            const double wlo = kst[k].wlo, whi = kst[k].whi;
            const double c = 0.5 * (wlo + whi);
            fr = fmax(whi - c, c - wlo);
            fdl = c - lam[k];
            fused = fabs(fdl) > fr;
          }
          if (fused) {
            const double *zu = pt + u * M;
            const double lk = lam[k];
            const uint64_t m1 = a.tree.L == 1 ? a.tree.mask[0] : 0ull;
            const double bmu = (double)__uint_as_float(((const unsigned int *)ugap)[4 * u + 2]);
            const double Hup = fr * bmu * (1.0 + 0x1p-30) + 0x1p-36 * (1.0 + (lk + fabs(fdl) + fr) * bmu);
            FarPass f;
            #pragma unroll 4
            for (int j = 0; j < M; ++j) {
              const float bj = bu[j * K + k];
              if (S0 >> j & 1) v = v + (double)bj;
              const bool mov = bj > 0.0f;
              if (mov) A |= 1ull << j;
              bmk = bj > bmk ? bj : bmk;
              const double b = mov ? (double)bj : 0.0;
              const double sh = fdl * b;
              far_item(f, zu[j] - sh, j, mov, (m1 >> j & 1) != 0, Hup);
            }
            const double Hs = fr * (double)bmk * (1.0 + 0x1p-30) + 0x1p-36 * (1.0 + (lk + fabs(fdl) + fr) * (double)bmk);
            fused_ok = far_finish(f, zu, bu, M, K, k, A, lk, fdl, fr, (double)bmk, Hs, m1,
                                  a.tree.L == 1 ? a.tree.cap[0] : 0, &fused_cw);
          } else if (!DN) {
            // the stored entries only, in ascending item order
            A = Am[q];
            for (uint64_t m = A; m; m &= m - 1) {
              const int j = __ffsll((long long)m) - 1;
              const float bj = bu[j * K + k];
              if (S0 >> j & 1) v = v + (double)bj;
              bmk = bj > bmk ? bj : bmk;
            }
          } else {
            #pragma unroll 4
            for (int j = 0; j < M; ++j) {
              const float bj = bu[j * K + k];
              if (S0 >> j & 1) v = v + (double)bj;
              if (bj > 0.0f) A |= 1ull << j;
              bmk = bj > bmk ? bj : bmk;
            }
          }
        } else {
          // the selected items only, in ascending index order
          for (uint64_t m = S0; m; m &= m - 1) v = v + (double)bu[(__ffsll((long long)m) - 1) * K + k];
        }
        vk[q] = v;
        if (SCD) {
          if (FMT == 0) offg |= off_grid(v, gmag);
          const int mode = kmode[k];
          if (walk_mode(mode)) {
            const double lk = lam[k];
            const double *zu = pt + u * M;
            bool walk = A != 0;
            if (walk && mode == KS_WINDOW) {
              // no breakpoint of this user inside the window: nothing to emit
              // and its consumption just above the window is v_ik (no correction)
              double cw = fused_cw;
              // the filter's scale: |top p~| + H, with H from the user's
              // largest cost and the widest window
              const float bmu = __uint_as_float(((const unsigned int *)ugap)[4 * u + 2]);
              const double hm = kwide[0];
              const double Hu = hm * (double)bmu * (1.0 + 0x1p-30) + 0x1p-36 * (1.0 + (double)bmu * hm);
              const double gscale = fabs(zu[perm[u * M]]) + Hu;
              if (window_calm(ugap[2 * u], gscale, kst[k].hw, (double)bmk, lk)) {
                walk = false;
              } else if (fused && fused_ok) {
                // no breakpoint inside the window: its consumption just above
                // the window is the window's set's
                walk = false;
                if (cw != v) {
                  xs_atomic_add_sum(&kxs[k], xs_minus(xs_of(cw), xs_of(v)));
                }
              }
            }
            if (walk && (S0 & A) == 0 &&
                pair_idle(tr, A, S0, [&](int j) -> double { return zu[j]; },
                          [&](int j) -> double { return (double)bu[j * K + k]; }, lk, kst[k].tlo)) {
              walk = false;   // (in a window its consumption stays 0)
            }
            if (walk) wq[atomicAdd(nwq, 1u)] = (uint16_t)q;
          }
        }
      }
    };
    // (full: read back from LDS at each use instead of held in scarce scalar registers)
    auto is_full = [&]() -> bool { return FMT == 1 && __builtin_amdgcn_readfirstlane((int)nwq[2]) != 0; };
    if (FMT == 0 || is_full()) look(std::true_type());
    else look(std::false_type());
    __syncthreads();
    if (SCD) {
      const int nw = (int)nwq[0];
      // (dealt over the waves in turn: a wave's time is its slowest lane's)
      for (int i = (tid & 63) * (NT / 64) + (tid >> 6); i < nw; i += NT) {
        const int q = wq[i];
        const int u = q / K, k = q - u * K;
        const int mode = kmode[k];
        const KWalk &ks = kst[k];
        const double lk = lam[k], v = vk[q];
        const double *zu = pt + u * M;
        const float *bu = bt + (size_t)u * M * K;
        const uint64_t S0 = Sm[u];
        uint64_t A = 0;
        if (FMT == 1 && !is_full()) {
          A = Am[q];
        } else {
          #pragma unroll 4
          for (int j = 0; j < M; ++j) {
            const float bj = bu[j * K + k];
            if (bj > 0.0f) A |= 1ull << j;
            offg |= off_grid(bj, ginv);
          }
        }
        double above = 0.0;   // window: the consumption just above it
        if (fastau && (A & (A - 1)) == 0) {
          // one moving line: its only breakpoint is where it crosses its
          // threshold element (a horizontal line) or the zero level: the
          // lowest selected member when it is out, the best member left
          // out when it is in (set full), else zero
          const int o = __ffsll((long long)A) - 1;
          const int th = (!(m1 >> o & 1) || tau[2 * u] < 0) ? -1 : (int)tau[2 * u + ((S0 >> o & 1) ? 1 : 0)];
          const double bo_d = (double)bu[o * K + k];
          const double add_o = lk * bo_d;
          const double co = zu[o] + add_o;
          const double num = th < 0 ? co : co - zu[th];
          // divided only where the quotient can lie in the pass's range
          if (num > 0.0 && num >= ks.tlo * bo_d * (1.0 - 0x1p-40)) {
            const bool over = mode == KS_WINDOW && num > ks.thi * bo_d * (1.0 + 0x1p-40);
            const double best = over ? INFINITY : num / bo_d;
            if (mode == KS_WINDOW && best > ks.thi) above = bo_d;
            else if (best >= ks.tlo) record_event(a, ks, k, best, bo_d, mode, hs, hc, hmin, hmax, kcnt, kovf, nstage, bid);
          }
        } else {
          uint64_t Sw = 0;
          const int st = pair_start(
              tr, A, S0, Pm[u], [&](int j) -> double { return zu[j]; },
              [&](int j) -> double { return (A >> j & 1) ? (double)bu[j * K + k] : 0.0; },
              [&](int r) -> int { return (int)perm[u * M + r]; }, lk, ks, &Sw, &above);
          if (st) {
            const uint32_t w = atomicAdd(&nwq[1], 1u);
            wq2[w] = (uint16_t)(q | (st == 2 ? 0x8000 : 0));
            wS[w] = Sw;
            continue;
          }
        }
        if (mode == KS_WINDOW && above != v) {
          xs_atomic_add_sum(&kxs[k], xs_minus(xs_of(above), xs_of(v)));
        }
      }
      __syncthreads();
      const int nw2 = (int)nwq[1];
      for (int i = (tid & 63) * (NT / 64) + (tid >> 6); i < nw2; i += NT) {
        const int q = wq2[i] & 0x7FFF;
        const int u = q / K, k = q - u * K;
        const int mode = kmode[k];
        const KWalk &ks = kst[k];
        const double *zu = pt + u * M;
        const float *bu = bt + (size_t)u * M * K;
        uint64_t A = 0;
        if (FMT == 1 && !is_full()) {
          A = Am[q];
        } else {
          #pragma unroll 4
          for (int j = 0; j < M; ++j)
            if (bu[j * K + k] > 0.0f) A |= 1ull << j;
        }
        double above = 0.0;
        const bool ok = pair_walk(
            M, tr, A, wS[i], !(wq2[i] & 0x8000),
            [&](int j) -> double { return zu[j]; },
            [&](int j) -> double { return (A >> j & 1) ? (double)bu[j * K + k] : 0.0; }, lam[k], ks,
            [&](double v1, double v2) {
              record_event(a, ks, k, v1, v2, mode, hs, hc, hmin, hmax, kcnt, kovf, nstage, bid);
            },
            &above);
        if (!ok) atomicAdd(a.err, 1ull);
        if (mode == KS_WINDOW && above != vk[q]) {
          xs_atomic_add_sum(&kxs[k], xs_minus(xs_of(above), xs_of(vk[q])));
        }
      }
      __syncthreads();
    }
    // ---- fixed-order sums of the tile into the block accumulators ----
    if (a.want_stats) {
      for (int k = tid; k < K; k += NT) {
        double s = 0.0;
        #pragma unroll 4
        for (int u = 0; u < nu; ++u) s = s + vk[u * K + k];
        acc[k] = acc[k] + s;
      }
      if (tid == NT - 1) {
        double sp = 0.0, sg = 0.0;
        for (int u = 0; u < nu; ++u) { sp = sp + uPG[2 * u]; sg = sg + uPG[2 * u + 1]; }
        acc[K] = acc[K] + sg;
        acc[K + 1] = acc[K + 1] + sp;
      }
    }
  }
  __syncthreads();
  if (a.want_stats) {
    for (int t = tid; t < K + 2; t += NT) a.partials[(size_t)bid * (K + 2) + t] = acc[t];
  }
  if (SCD) report_off_grid(a, offg);
  if (SCD) publish_block(a, K, hs, hc, hmin, hmax, kcnt, kpos, kovf, nstage, tid, NT, bid, kxs);
}


template <int FMT, bool SCD, int MX = 0, int KX = 0>
__global__ void __launch_bounds__(NT) k_sweep(const SweepArgs a, const TileGeom g) {
  extern __shared__ __align__(16) unsigned char smem[];
  sweep_body<FMT, SCD, MX, KX>(a, g, blockIdx.x, gridDim.x, smem);
}

// the general kernel for a shape (dense costs with M = K = 10, or M = 20
// and K = 50: the counts compiled in)
static const void *sweep_fn(int fmt, bool scd, int M, int K) {
  if (fmt == 0 && M == 10 && K == 10)
    return scd ? (const void *)k_sweep<0, true, 10, 10> : (const void *)k_sweep<0, false, 10, 10>;
  if (fmt == 0 && M == 20 && K == 50)
    return scd ? (const void *)k_sweep<0, true, 20, 50> : (const void *)k_sweep<0, false, 20, 50>;
  if (fmt == 0) return scd ? (const void *)k_sweep<0, true> : (const void *)k_sweep<0, false>;
  return scd ? (const void *)k_sweep<1, true> : (const void *)k_sweep<1, false>;
}

// Batched: blocks [block_off[s], block_off[s+1]) work on instance s, whose
// arguments are copied into LDS; one launch covers every instance.  n_dev:
// the instance count read from the device (a split made there; blocks past
// the last instance's range exit at once), else n_inst.
// at most 168 VGPRs: three waves per SIMD
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(3, 8))) k_sweep_batched(const SweepArgs *descs, const TileGeom *geoms,
                                                      const int *block_off, int n_inst, const int *n_dev) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ SweepArgs sa;
  __shared__ TileGeom sg;
  __shared__ int inst;
  if (n_dev) {
    n_inst = *n_dev;
    if (n_inst <= 0 || (int)blockIdx.x >= block_off[n_inst]) return;
  }
  if (threadIdx.x == 0) {
    int lo = 0, hi = n_inst - 1;
    while (lo < hi) {   // last s with block_off[s] <= blockIdx.x
      const int mid = (lo + hi + 1) >> 1;
      if (block_off[mid] <= (int)blockIdx.x) lo = mid; else hi = mid - 1;
    }
    inst = lo;
  }
  __syncthreads();
  const int s = inst;
  {
    const int *src = (const int *)(descs + s);
    int *dst = (int *)&sa;
    for (int t = threadIdx.x; t < (int)(sizeof(SweepArgs) / 4); t += NT) dst[t] = src[t];
    if (threadIdx.x == 0) sg = geoms[s];
  }
  __syncthreads();
  const int bid = blockIdx.x - block_off[s];
  const int nblk = block_off[s + 1] - block_off[s];
  if (sa.pr.fmt == 0) sweep_body<0, true>(sa, sg, bid, nblk, smem);
  else sweep_body<1, true>(sa, sg, bid, nblk, smem);
}

// ---------------------------------------------------------------------------
// second-level reduction of the block partials (fixed order), dual value
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_reduce_stats(const double *partials, int nblk, int K,
                                                      const double *lam, const double *B,
                                                      double *R, double *g, double *P) {
  // one block per output column (K consumptions, then sum G_i, then sum P_i);
  // every thread adds a fixed strided subset, then a fixed tree: deterministic
  __shared__ double red[256];
  const int c = blockIdx.x, t = threadIdx.x;
  double s = 0.0;
  for (int b = t; b < nblk; b += 256) s = s + partials[(size_t)b * (K + 2) + c];
  red[t] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) red[t] = red[t] + red[t + w];
    __syncthreads();
  }
  if (t != 0) return;
  s = red[0];
  if (c < K) {
    if (R) R[c] = s;
  } else if (c == K) {
    // g = sum_i G_i + sum_k lambda_k B_k
    double tt = s;
    for (int k = 0; k < K; ++k) { const double lb = lam[k] * B[k]; tt = tt + lb; }
    if (g) *g = tt;
  } else {
    if (P) *P = s;
  }
}

// ---------------------------------------------------------------------------
// Pre-solving by sampling (Sec. 5.3): the sub-instance of the sampled users
// ---------------------------------------------------------------------------
// dst[s * rowlen + c] = src[users[s] * rowlen + c]
__global__ void k_gather_rows(const float *src, float *dst, const int64_t *users, int64_t n,
                              int64_t rowlen) {
  const int64_t total = n * rowlen;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t s = e / rowlen, c = e - s * rowlen;
    dst[e] = src[users[s] * rowlen + c];
  }
}

// stored entries of every sampled item row
__global__ void k_gather_len(const int64_t *rowptr, const int64_t *users, int64_t n, int M,
                             int64_t *len) {
  const int64_t total = n * M;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t s = e / M, j = e - s * M;
    const int64_t r = users[s] * M + j;
    len[e] = rowptr[r + 1] - rowptr[r];
  }
}

// out[0] = 0, out[i + 1] = len[0] + ... + len[i]  (one block; chunk per thread,
// then a scan of the chunk sums in LDS)
__global__ void __launch_bounds__(1024) k_scan_i64(const int64_t *len, int64_t *out, int64_t n) {
  __shared__ int64_t part[1024];
  const int t = threadIdx.x;
  const int64_t chunk = (n + 1023) / 1024;
  const int64_t lo = t * chunk < n ? t * chunk : n;
  const int64_t hi = lo + chunk < n ? lo + chunk : n;
  int64_t sum = 0;
  for (int64_t i = lo; i < hi; ++i) sum += len[i];
  part[t] = sum;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int64_t v = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int64_t run = part[t] - sum;
  if (t == 0) out[0] = 0;
  for (int64_t i = lo; i < hi; ++i) { run += len[i]; out[i + 1] = run; }
}

// copy the sampled item rows' entries (rows are short: one thread per row)
__global__ void k_gather_csr(const int64_t *rowptr, const int32_t *col, const float *val,
                             const int64_t *users, int64_t n, int M, const int64_t *subptr,
                             int32_t *scol, float *sval) {
  const int64_t total = n * M;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t s = e / M, j = e - s * M;
    const int64_t r = users[s] * M + j;
    int64_t o = subptr[e];
    for (int64_t q = rowptr[r]; q < rowptr[r + 1]; ++q, ++o) {
      scol[o] = col[q];
      sval[o] = val[q];
    }
  }
}

// ---------------------------------------------------------------------------
// DD step (Eq.14) and the dual gradient
// ---------------------------------------------------------------------------
__global__ void k_dd_update(int K, double alpha, const double *R, const double *B, double *lam) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  const double d = R[k] - B[k];
  const double stp = alpha * d;
  const double nl = lam[k] + stp;
  lam[k] = nl > 0.0 ? nl : 0.0;
}

__global__ void k_dual_backward(int K, const double *R, const double *B, const double *gout,
                                double *glam) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  const double d = B[k] - R[k];
  glam[k] = gout[0] * d;
}

// ---------------------------------------------------------------------------
// input validation pass
// ---------------------------------------------------------------------------
__global__ void k_validate(const float *v, int64_t n, unsigned int *flags) {
  // flags[0]: non-finite seen, flags[1]: negative seen
  unsigned int nf = 0, ng = 0;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
       t += (int64_t)gridDim.x * blockDim.x) {
    const float x = v[t];
    nf |= !isfinite(x);
    ng |= (x < 0.0f);
  }
  if (nf) atomicOr(&flags[0], 1u);
  if (ng) atomicOr(&flags[1], 1u);
}

__global__ void k_validate_csr(const int64_t *rowptr, const int32_t *col, int64_t nrows, int K,
                               unsigned int *flags) {
  unsigned int bad = 0;
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < nrows;
       r += (int64_t)gridDim.x * blockDim.x) {
    const int64_t e0 = rowptr[r], e1 = rowptr[r + 1];
    if (e1 < e0) { bad = 1; continue; }
    int prev = -1;
    for (int64_t e = e0; e < e1; ++e) {
      const int c = col[e];
      if (c <= prev || c >= K) bad = 1;
      prev = c;
    }
  }
  if (bad) atomicOr(&flags[2], 1u);
}

// ---------------------------------------------------------------------------
// batched helpers: statistics by column table, flat per-(instance, k) init
// and finish
// ---------------------------------------------------------------------------
struct ColDesc {
  const double *partials;  // [nblk][K + 2] of the instance
  const double *lam;       // [K]
  const double *B;         // [K]
  double *out;             // destination of this column
  int nblk, K, col, pad;
};

__global__ void __launch_bounds__(256) k_reduce_stats_tab(const ColDesc *tab) {
  __shared__ double red[256];
  const ColDesc d = tab[blockIdx.x];
  const int t = threadIdx.x;
  double s = 0.0;
  for (int b = t; b < d.nblk; b += 256) s = s + d.partials[(size_t)b * (d.K + 2) + d.col];
  red[t] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) red[t] = red[t] + red[t + w];
    __syncthreads();
  }
  if (t != 0) return;
  s = red[0];
  if (d.col == d.K) {
    for (int k = 0; k < d.K; ++k) { const double lb = d.lam[k] * d.B[k]; s = s + lb; }
  }
  *d.out = s;
}

hipError_t kp_launch_reduce_tab(const void *tab, int n, hipStream_t stream) {
  hipLaunchKernelGGL(k_reduce_stats_tab, dim3(n), dim3(256), 0, stream, (const ColDesc *)tab);
  return hipGetLastError();
}

hipError_t kp_launch_sweep_batched(const SweepArgs *descs, const TileGeom *geoms, const int *block_off,
                                   int n_inst, int total_blocks, size_t lds, hipStream_t stream,
                                   const int *n_dev) {
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void *)k_sweep_batched,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_sweep_batched, dim3(total_blocks), dim3(NT), lds, stream, descs, geoms,
                     block_off, n_inst, n_dev);
  return hipGetLastError();
}

TileGeom kp_tile_geom(const SweepArgs &a, int U) {
  TileGeom g;
  g.U = U;
  g.M = a.pr.M;
  g.K = a.pr.K;
  g.aligned = a.pr.fmt == 0 && ((uintptr_t)a.pr.b & 15) == 0 && (((int64_t)U * g.M * g.K) & 3) == 0;
  return g;
}

size_t kp_coldesc_size() { return sizeof(ColDesc); }
void kp_coldesc_fill(void *dst, const double *partials, const double *lam, const double *B, double *out,
                     int nblk, int K, int col) {
  ColDesc d;
  d.partials = partials; d.lam = lam; d.B = B; d.out = out;
  d.nblk = nblk; d.K = K; d.col = col; d.pad = 0;
  memcpy(dst, &d, sizeof d);
}

// ---------------------------------------------------------------------------
// host-side launch helpers (called from the C ABI)
// ---------------------------------------------------------------------------
size_t kp_sweep_lds_bytes(int U, int M, int K, int L, bool scd, int fmt, bool hist = true) {
  auto r16 = [](size_t b) { return (b + 15) & ~(size_t)15; };
  const size_t R = (size_t)U * M, Q = (size_t)U * K;
  size_t s = r16(R * K * 4) + r16(R * 8) + r16(R) + r16((size_t)U * 8) * 2 + r16(Q * 8) +
             r16((size_t)U * 16) + r16((size_t)(K + 2) * 8);
  s += r16((size_t)K * 8);   // lambda
  s += r16(R * 4) + r16((R + 1) * 4) + r16(16);   // staged profits, row offsets, entry base
  if (scd) s += set_tree_bytes(L, M);
  if (scd) s += r16((size_t)U * 2);                // threshold elements
  if (scd) {
    // pairs left to look at and to walk (CSR: over the staged entries)
    const size_t q = 2 * r16(Q * 2) + r16(Q * 8), e = fmt == 1 ? (size_t)NT * ECH * 4 : 0;
    s += r16(16) + (fmt == 0 ? q : q > e ? r16(q - e) : 0);
  }
  if (scd && fmt == 1) s += r16(Q * 8);            // moving items of every (user, knapsack)
  if (fmt == 1) s += r16((size_t)NT * ECH * (scd ? 1 : 4)) + r16((size_t)NT * ECH * 4);  // staged CSR entries
  if (scd)
    s += r16((size_t)K * sizeof(KWalk)) + (hist ? r16((size_t)K * KP_NB * sizeof(XSum)) + r16((size_t)K * KP_NB * 4) : 0) +
         4 * r16((size_t)K * 4) + 2 * r16((size_t)K * 8) + r16(16) +
         r16(16) + r16((size_t)K * sizeof(XSum)) + r16((size_t)U * 16);   // widest window, corrections, per-user filter
  return s;
}

// Blocks of the batched sweep kernel that can be resident at once (0 if unknown).
int kp_sweep_batched_resident(size_t lds) {
  const void *fn = (const void *)k_sweep_batched;
  if (lds > 64 * 1024 && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return 0;
  int per_cu = 0, dev = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, NT, lds) != hipSuccess || per_cu < 1) return 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  return per_cu * cus;
}

// Blocks of the general sweep kernel that can be resident at once (0 if unknown).
int kp_sweep_resident_grid(int U, int M, int K, int L, bool scd, int fmt, bool hist = true) {
  const size_t lds = kp_sweep_lds_bytes(U, M, K, L, scd, fmt, hist);
  const void *fn = sweep_fn(fmt, scd, M, K);
  if (lds > 64 * 1024 && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return 0;
  int per_cu = 0, dev = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, NT, lds) != hipSuccess || per_cu < 1) return 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  return per_cu * cus;
}

hipError_t kp_launch_sweep(const SweepArgs &a, int U, int grid, bool scd, hipStream_t stream,
                           int *used) {
  TileGeom g;
  g.U = U;
  g.M = a.pr.M;
  g.K = a.pr.K;
  g.aligned = a.pr.fmt == 0 && ((uintptr_t)a.pr.b & 15) == 0 &&
              (((int64_t)U * g.M * g.K) & 3) == 0;
  const size_t lds = kp_sweep_lds_bytes(U, g.M, g.K, a.tree.L, scd, a.pr.fmt, !(scd && a.no_hist));
  const void *fn = sweep_fn(a.pr.fmt, scd, g.M, g.K);
  if (lds > 64 * 1024) {
    // shapes with many knapsacks need more than the default 64 KB of LDS
    // (gfx950 has 160 KB per workgroup)
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  // persistent launch: at most the blocks that can be resident at once
  int per_cu = 0, dev = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, NT, lds) == hipSuccess && per_cu > 0 &&
      hipGetDevice(&dev) == hipSuccess &&
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0) {
    if (grid > per_cu * cus) grid = per_cu * cus;
  }
  if (used) *used = grid;
  if (a.pr.fmt == 0 && g.M == 10 && g.K == 10) {
    if (scd) hipLaunchKernelGGL((k_sweep<0, true, 10, 10>), dim3(grid), dim3(NT), lds, stream, a, g);
    else hipLaunchKernelGGL((k_sweep<0, false, 10, 10>), dim3(grid), dim3(NT), lds, stream, a, g);
  } else if (a.pr.fmt == 0 && g.M == 20 && g.K == 50) {
    if (scd) hipLaunchKernelGGL((k_sweep<0, true, 20, 50>), dim3(grid), dim3(NT), lds, stream, a, g);
    else hipLaunchKernelGGL((k_sweep<0, false, 20, 50>), dim3(grid), dim3(NT), lds, stream, a, g);
  } else if (a.pr.fmt == 0) {
    if (scd) hipLaunchKernelGGL((k_sweep<0, true>), dim3(grid), dim3(NT), lds, stream, a, g);
    else hipLaunchKernelGGL((k_sweep<0, false>), dim3(grid), dim3(NT), lds, stream, a, g);
  } else {
    if (scd) hipLaunchKernelGGL((k_sweep<1, true>), dim3(grid), dim3(NT), lds, stream, a, g);
    else hipLaunchKernelGGL((k_sweep<1, false>), dim3(grid), dim3(NT), lds, stream, a, g);
  }
  return hipGetLastError();
}

hipError_t kp_launch_reduce_stats(const double *partials, int nblk, int K, const double *lam,
                                  const double *B, double *R, double *g, double *P,
                                  hipStream_t stream) {
  hipLaunchKernelGGL(k_reduce_stats, dim3(K + 2), dim3(256), 0, stream, partials, nblk, K, lam, B,
                     R, g, P);
  return hipGetLastError();
}

static unsigned gather_blocks(int64_t total) {
  int64_t b = (total + 255) / 256;
  return (unsigned)(b < 1 ? 1 : (b > 4096 ? 4096 : b));
}

hipError_t kp_launch_gather_dense(const float *p, const float *b, const int64_t *users, int64_t n, int M,
                                  int K, float *sp, float *sb, hipStream_t stream) {
  hipLaunchKernelGGL(k_gather_rows, dim3(gather_blocks(n * M)), dim3(256), 0, stream, p, sp, users, n,
                     (int64_t)M);
  if (b)
    hipLaunchKernelGGL(k_gather_rows, dim3(gather_blocks(n * M * K)), dim3(256), 0, stream, b, sb,
                       users, n, (int64_t)M * K);
  return hipGetLastError();
}

hipError_t kp_launch_gather_csr_ptr(const int64_t *rowptr, const int64_t *users, int64_t n, int M,
                                    int64_t *len, int64_t *subptr, hipStream_t stream) {
  hipLaunchKernelGGL(k_gather_len, dim3(gather_blocks(n * M)), dim3(256), 0, stream, rowptr, users, n,
                     M, len);
  hipLaunchKernelGGL(k_scan_i64, dim3(1), dim3(1024), 0, stream, len, subptr, n * M);
  return hipGetLastError();
}

hipError_t kp_launch_gather_csr(const int64_t *rowptr, const int32_t *col, const float *val,
                                const int64_t *users, int64_t n, int M, const int64_t *subptr,
                                int32_t *scol, float *sval, hipStream_t stream) {
  hipLaunchKernelGGL(k_gather_csr, dim3(gather_blocks(n * M)), dim3(256), 0, stream, rowptr, col, val,
                     users, n, M, subptr, scol, sval);
  return hipGetLastError();
}

hipError_t kp_launch_dd_update(int K, double alpha, const double *R, const double *B, double *lam,
                               hipStream_t stream) {
  hipLaunchKernelGGL(k_dd_update, dim3((K + 63) / 64), dim3(64), 0, stream, K, alpha, R, B, lam);
  return hipGetLastError();
}

hipError_t kp_launch_dual_backward(int K, const double *R, const double *B, const double *gout,
                                   double *glam, hipStream_t stream) {
  hipLaunchKernelGGL(k_dual_backward, dim3((K + 63) / 64), dim3(64), 0, stream, K, R, B, gout,
                     glam);
  return hipGetLastError();
}

hipError_t kp_launch_validate(const float *v, int64_t n, unsigned int *flags, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_validate, dim3((unsigned)blocks), dim3(256), 0, stream, v, n, flags);
  return hipGetLastError();
}

hipError_t kp_launch_validate_csr(const int64_t *rowptr, const int32_t *col, int64_t nrows, int K,
                                  unsigned int *flags, hipStream_t stream) {
  if (nrows <= 0) return hipSuccess;
  int64_t blocks = (nrows + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_validate_csr, dim3((unsigned)blocks), dim3(256), 0, stream, rowptr, col,
                     nrows, K, flags);
  return hipGetLastError();
}

__global__ void k_fill_f64(double *dst, int64_t n, double v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = v;
}

// A fill kernel rather than hipMemsetAsync, for paths a caller may capture in
// a HIP graph.
hipError_t kp_launch_fill_f64(double *dst, int64_t n, double v, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)blocks), dim3(256), 0, stream, dst, n, v);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Streaming-read probe: the achievable HBM read bandwidth for a buffer of
// the sweep's size (the ceiling its roofline fraction is also quoted
// against).  Every thread reads 16-byte words with four loads in flight,
// folds them with XOR (so no load is dead) and every block XORs its result
// into one word; XOR is order-free, so the word is deterministic.
// ---------------------------------------------------------------------------
#define SR_NT 256
typedef unsigned int sr_v4u __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(SR_NT) k_stream_read(const uint4 *src, int64_t n16, unsigned long long *out) {
  // eight nontemporal 16-byte loads per thread in flight (the sweep kernels'
  // staging uses the same cache policy)
  const sr_v4u *s = (const sr_v4u *)src;
  sr_v4u acc = {0u, 0u, 0u, 0u};
  const int64_t stride = (int64_t)gridDim.x * SR_NT;
  int64_t i = (int64_t)blockIdx.x * SR_NT + threadIdx.x;
  for (; i + 7 * stride < n16; i += 8 * stride) {
    sr_v4u v[8];
    #pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = __builtin_nontemporal_load(s + i + u * stride);
    #pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= v[u];
  }
  for (; i < n16; i += stride) acc ^= __builtin_nontemporal_load(s + i);
  unsigned long long v = ((unsigned long long)(acc.x ^ acc.z) << 32) | (unsigned long long)(acc.y ^ acc.w);
  for (int off = 32; off > 0; off >>= 1) v ^= __shfl_xor(v, off, 64);
  __shared__ unsigned long long part[SR_NT / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int w = 0; w < SR_NT / 64; ++w) t ^= part[w];
    atomicXor(out, t);
  }
}

// The resident blocks of the probe (at most `grid` when grid > 0).
hipError_t kp_launch_stream_read(const void *src, int64_t n16, unsigned long long *out, int grid,
                                 hipStream_t stream) {
  int per_cu = 0, dev = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_stream_read, SR_NT, 0) != hipSuccess ||
      per_cu < 1)
    per_cu = 8;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    cus = 256;
  int g = per_cu * cus;
  if (grid > 0 && grid < g) g = grid;
  hipLaunchKernelGGL(k_stream_read, dim3(g), dim3(SR_NT), 0, stream, (const uint4 *)src, n16, out);
  return hipGetLastError();
}
