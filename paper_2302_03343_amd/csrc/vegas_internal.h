// Pieces of the VEGAS path shared by the single-integral kernels
// (vegas.hip) and the batched persistent kernel (batch.hip): the grid map,
// the per-iteration record and its inverse-variance combination, Lepage's
// refinement of one dimension, and the context structure.
#pragma once

#include "common.h"
#include "integrands.h"
#include "ttbar.h"
#include "drellyan.h"
#include "singletop.h"
#include "ttbar_dyn.h"

#include <type_traits>

namespace vgx {

struct IterRecord {
  double mean, var, s1, s2;
  int64_t n;
  int32_t finite;
  int32_t pad;
};

struct Combined {
  double mean, sigma, chi2_dof;
  int32_t n_used;
  int32_t pad;
};

constexpr int MAX_RECORDS = 4096;

// Where a kernel leaves a completed record for the host: pinned host memory
// mirroring the records and the combination.  Null: the device copies only.
struct HostOut {
  IterRecord* rec;
  Combined* comb;
};

// Grid map (inverse transform through the piecewise-constant density of the
// bins): i = min(floor(u N), N-1), delta = u N - i,
// x = e_i + delta (e_{i+1} - e_i), J = prod_j N (e_{i+1} - e_i).
template <int D>
__device__ __forceinline__ double grid_map(const double (&u)[D], const double* se, int nb, double (&x)[D],
                                           int (&idx)[D]) {
  double jac = 1.0;
  const double dnb = (double)nb;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const double t = u[j] * dnb;
    int i = (int)t;
    i = i < nb - 1 ? i : nb - 1;
    i = i > 0 ? i : 0;  // points given by the caller may sit on or outside the cube's faces
    const double delta = t - (double)i;
    const double lo = se[j * (nb + 1) + i];
    const double w = se[j * (nb + 1) + i + 1] - lo;
    x[j] = fma(delta, w, lo);
    jac *= dnb * w;
    idx[j] = i;
  }
  return jac;
}

// The grid map of caller points from scaled coordinates t_j = u_j N: i =
// floor(t) clamped into [0, N-1] (points on or outside the cube's faces),
// delta = t - i, x = e_i + delta w_i (w_i = e_{i+1} - e_i), J = N^D prod_j w_i
// with the factor N^D given as nbD.  GLOBAL: the edge pairs come from global
// memory (one 16-byte load each, served by the L1: the grid is a few KB),
// else from LDS.
typedef double double2_a8 __attribute__((ext_vector_type(2), aligned(8)));
template <int D, bool GLOBAL>
__device__ __forceinline__ double grid_map_t(const double (&t)[D], const double* se, const double* __restrict__ ge,
                                             int nb, double nbD, double (&x)[D], int (&idx)[D]) {
  double jw = 1.0;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    int i = (int)t[j];
    i = i < nb - 1 ? i : nb - 1;
    i = i > 0 ? i : 0;
    const double delta = t[j] - (double)i;
    double lo, w;
    if constexpr (GLOBAL) {
      // a 32-bit byte offset from the uniform base (a scalar-base load)
      const uint32_t off = (uint32_t)(j * (nb + 1) + i) * 8u;
      const double2_a8 e = *(const double2_a8*)((const char*)ge + off);
      lo = e.x;
      w = e.y - lo;
    } else {
      lo = se[j * (nb + 1) + i];
      w = se[j * (nb + 1) + i + 1] - lo;
    }
    x[j] = fma(delta, w, lo);
    jw *= w;
    idx[j] = i;
  }
  return jw * nbD;
}

// The grid map of Philox words k_j, u_j = (k_j + 1/2) 2^-32: one 64-bit
// multiply-add k_j N + floor(N/2) has the bin in its upper word and the position
// in it, f_j 2^-32 (for odd N less half a step), in its lower, both exact.
// The bins' table holds (e_i, w_i 2^-32), so that x = e_i + f_j w_i is one FMA
// and the width needs no subtraction; x is bit for bit that of the map above.
// Per dimension two instructions find the bin and the position (the
// conversion to FP64, scaling, truncation and fraction were four) and one
// subtraction goes: with the leaner exponential 111 -> 97 VALU instructions
// per sample for the d = 4 Gaussian; 1e9 samples, 20 launches of each on one
// GPU: 3.45 -> 3.17 ms on average, 3.28 -> 2.95 the fastest.  ODD adds
// the half step, one FP64 addition per dimension, in kernels for odd counts (51
// bins, 2e8 samples: 604 -> 653 us; in the table instead, it rounds every edge
// once more, and as a branch per sample it cost even counts registers and moves).
// The table is read from global memory, one 16-byte load per dimension served
// by the L1 (a few KB): the LDS's load is the histogram's atomics and the
// integrand's tables.  J = nbDs prod_j w_j 2^-32, nbDs = (N 2^32)^D.
//
// A wave's load touches as many cache lines as the dimension's row has, 16
// bytes a bin: with many dimensions and bins that binds, and grid_map_edges
// reads the edges (8 bytes a bin) and takes two more instructions per dimension.
// Its x and J are the same bit for bit, for both parities.
__host__ __device__ inline double2 grid_bin(double lo, double hi) { return double2{lo, (hi - lo) * 0x1p-32}; }
template <int D, bool ODD>
__device__ __forceinline__ double grid_map_words(const uint32_t (&k)[D], const double2* __restrict__ bins, int nb,
                                                 double nbDs, double (&x)[D], int (&idx)[D]) {
  double jw = nbDs;  // first, so that no partial product leaves the FP64 range before J does
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const uint64_t p = (uint64_t)k[j] * (uint32_t)nb + (uint32_t)(nb >> 1);
    uint32_t i = (uint32_t)(p >> 32);
    asm("" : "+v"(i));  // keeps the shift below apart from the 64-bit one
    // a 32-bit byte offset from the uniform base (a scalar-base load)
    const double2 e = *(const double2*)((const char*)(bins + j * nb) + (i << 4));
    const double f = (double)(uint32_t)p;
    x[j] = fma(ODD ? f + 0.5 : f, e.y, e.x);
    jw *= e.y;
    idx[j] = (int)i;
  }
  return jw;
}

// hf: 2^-33 for odd N, else 0; nbD = N^D.
template <int D>
__device__ __forceinline__ double grid_map_edges(const uint32_t (&k)[D], const double* __restrict__ edges, int nb,
                                                 double hf, double nbD, double (&x)[D], int (&idx)[D]) {
  double jw = nbD;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const uint64_t p = (uint64_t)k[j] * (uint32_t)nb + (uint32_t)(nb >> 1);
    uint32_t i = (uint32_t)(p >> 32);
    asm("" : "+v"(i));
    const double2_a8 e = *(const double2_a8*)((const char*)(edges + j * (nb + 1)) + (i << 3));
    const double w = e.y - e.x;
    x[j] = fma(fma((double)(uint32_t)p, 0x1p-32, hf), w, e.x);
    jw *= w;
    idx[j] = (int)i;
  }
  return jw;
}

// The value of an integrand at a point the grid map made (inside the cube).
template <class F, class = void>
struct HasInside : std::false_type {};
template <class F>
struct HasInside<F, std::void_t<decltype(&F::eval_inside)>> : std::true_type {};
template <class F, int D>
__device__ __forceinline__ double eval_inside(const F& f, const double (&x)[D]) {
  if constexpr (HasInside<F>::value) return f.eval_inside(x);
  else return f.eval(x);
}

// Compensated sums of paired rows or halves of a wave, the lower one first.
template <int DIST>
__device__ __forceinline__ Comp pair_merge(Comp v) {
  Comp a, b;
  lane_pair<DIST>(v.s, a.s, b.s);
  lane_pair<DIST>(v.c, a.c, b.c);
  a.add(b.s);
  a.c += b.c;
  return a;
}

// Merge of compensated sums over the first `lanes` lanes of a wave (the
// others hold zeros) into lane 0, in a fixed order: pairs, quads, eights,
// sixteens by DPP, then across the rows of 16.  Levels beyond `lanes`
// (uniform) would add zeros and are skipped.
__device__ __forceinline__ Comp wave_merge(Comp a, int lanes) {
  auto level = [&](double os, double oc) {
    a.add(os);
    a.c += oc;
  };
  if (lanes > 1) level(dpp_get<kDppXor1>(a.s), dpp_get<kDppXor1>(a.c));
  if (lanes > 2) level(dpp_get<kDppXor2>(a.s), dpp_get<kDppXor2>(a.c));
  if (lanes > 4) level(dpp_get<kDppHalfMirror>(a.s), dpp_get<kDppHalfMirror>(a.c));
  if (lanes > 8) level(dpp_get<kDppMirror>(a.s), dpp_get<kDppMirror>(a.c));
  if (lanes > 16) a = pair_merge<16>(a);
  if (lanes > 32) a = pair_merge<32>(a);
  return a;
}

// Estimate of one iteration from its compensated sums, stored as record
// k_rec, then the inverse-variance combination of the finite records
// 0..k_rec with chi^2/dof:  E = S1/n, var(E) = max(S2/n - E^2, 0)/(n-1);
// E_bar = S^2 sum E_i/S_i^2, 1/S^2 = sum 1/S_i^2,
// chi^2/dof = sum (E_i - E_bar)^2/S_i^2/(M-1).  A zero variance makes that
// estimate exact (sigma 0).  Called by the 64 lanes of one wave, which split
// the records (lane l takes l, l+64, ...) so that the cost per iteration does
// not grow with the number of stored estimates; lane 0 writes the results,
// with host.rec set also to the host.
__device__ inline void finalize_record(double s1, double s2, int64_t n, IterRecord* rec, int k_rec, Combined* comb,
                                       const HostOut& host = {}) {
  // no contraction into FMAs, so that every kernel that inlines this gives the same bits
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63;
  // this lane's first stored record (k = lane), read before record k_rec is
  // written so that the read overlaps the caller's
  double mean0 = 0.0, var0 = 0.0;
  bool fin0 = false;
  if (lane < k_rec) {
    mean0 = rec[lane].mean;
    var0 = rec[lane].var;
    fin0 = rec[lane].finite;
  }
  IterRecord r;
  r.s1 = s1;
  r.s2 = s2;
  r.n = n;
  r.mean = s1 / (double)n;
  const double m2 = s2 / (double)n - r.mean * r.mean;
  r.var = n > 1 ? (m2 > 0.0 ? m2 : 0.0) / (double)(n - 1) : 0.0;
  r.finite = isfinite(r.mean) && isfinite(r.var);
  r.pad = 0;
  if (lane == 0) rec[k_rec] = r;
  // record k_rec is taken from registers: the other lanes must not read
  // the store lane 0 has just issued
  auto mean_var = [&](int k, double& mean, double& var) -> bool {
    if (k == k_rec) { mean = r.mean; var = r.var; return r.finite; }
    if (k == lane) { mean = mean0; var = var0; return fin0; }
    mean = rec[k].mean;
    var = rec[k].var;
    return rec[k].finite;
  };
  const int lanes = k_rec + 1 < 64 ? k_rec + 1 : 64;
  int used = 0, zero_var = MAX_RECORDS;
  Comp wsum, msum;
  for (int k0 = 0; k0 <= k_rec; k0 += 64) {
    const int k = k0 + lane;
    double mean = 0.0, var = 1.0;
    const bool ok = k <= k_rec && mean_var(k, mean, var);
    const unsigned long long zeros = __ballot(ok && var == 0.0);
    used += __popcll(__ballot(ok));
    if (zeros && zero_var == MAX_RECORDS) zero_var = k0 + __ffsll(zeros) - 1;
    if (ok && var != 0.0) {
      wsum.add(1.0 / var);
      msum.add(mean / var);
    }
  }
  Combined c{0.0, 0.0, 0.0, used, 0};
  if (zero_var < MAX_RECORDS) {
    double mean, var;
    mean_var(zero_var, mean, var);
    c.mean = mean;
  } else if (used > 0) {
    wsum = wave_merge(wsum, lanes);
    msum = wave_merge(msum, lanes);
    // lane 0's combination is the one written; every lane uses it
    c.mean = first_lane(msum.value() / wsum.value());
    c.sigma = sqrt(1.0 / first_lane(wsum.value()));
    if (used > 1) {
      Comp chi;
      for (int k = lane; k <= k_rec; k += 64) {
        double mean, var;
        if (!mean_var(k, mean, var)) continue;
        const double dd = mean - c.mean;
        chi.add(dd * dd / var);
      }
      chi = wave_merge(chi, lanes);
      c.chi2_dof = chi.value() / (double)(used - 1);
    }
  }
  if (lane == 0) {
    *comb = c;
    if (host.rec) {
      host.rec[k_rec] = r;
      *host.comb = c;
    }
  }
}

// Lepage's refinement of one dimension, by one 64-thread workgroup:
// 3-point smoothing of the accumulated (f J)^2 per bin, normalisation to
// p_i, damping r_i = ((1 - p_i)/ln(1/p_i))^alpha, re-binning to equal shares
// of sum r with r spread uniformly inside each old bin.  A dimension whose
// histogram is all zero, or not finite (an iteration with a non-finite
// weight, which the combination excludes too), is left unchanged.
//
// Bound by latency: one wave, a chain of dependent steps between two kernels
// of an iteration.  Lane l holds the bins [l C, l C + C), C = ceil(nb/64), in
// registers; sums and the cumulative r are wave scans (three serial loops
// of one thread over the bins took most of the 5.4 us that the kernel had for
// 50 bins).
__device__ inline void refine_dim(double* __restrict__ ej, double2* __restrict__ bj, const double* __restrict__ hj,
                                  int nb, double alpha) {
  __shared__ double d[VGX_MAX_BINS], r[VGX_MAX_BINS], cum[VGX_MAX_BINS + 1], e[VGX_MAX_BINS + 1];
  double* en = d;  // the new edges 1 .. nb - 1, once d has been read
  constexpr int CMAX = VGX_MAX_BINS / 64;
  const int lane = threadIdx.x & 63;
  const int C = (nb + 63) >> 6, i0 = lane * C;
  for (int i = lane; i < nb; i += 64) d[i] = hj[i];
  for (int i = lane; i <= nb; i += 64) e[i] = ej[i];
  __syncthreads();
  double sm[CMAX];
  double sd = 0.0, ss = 0.0;
#pragma unroll
  for (int c = 0; c < CMAX; ++c) {
    const int i = i0 + c;
    sm[c] = 0.0;
    if (c < C && i < nb) {
      const double di = d[i], dl = d[i > 0 ? i - 1 : 0], dr = d[i < nb - 1 ? i + 1 : nb - 1];
      sm[c] = i == 0 ? 0.5 * (di + dr) : i == nb - 1 ? 0.5 * (dl + di) : (dl + di + dr) / 3.0;
      sd += di;
      ss += sm[c];
    }
  }
  const double tot_d = last_lane(wave_scan(sd)), tot_sm = last_lane(wave_scan(ss));
  if (!(tot_d > 0.0) || !isfinite(tot_d)) return;  // uniform decision: every thread returns
  double run = 0.0;
  double rv[CMAX];
#pragma unroll
  for (int c = 0; c < CMAX; ++c) {
    rv[c] = 0.0;
    if (c < C && i0 + c < nb) {
      const double p = sm[c] / tot_sm;
      if (p > 0.0) {
        const double q = p >= 1.0 ? 1.0 : (1.0 - p) / -log(p);
        rv[c] = alpha == 1.5 ? q * sqrt(q) : pow(q, alpha);
      }
      run += rv[c];
    }
  }
  const double incl = wave_scan(run);
  double acc = __shfl_up(incl, 1, 64);  // the bins before this lane's
  if (lane == 0) acc = cum[0] = 0.0;
#pragma unroll
  for (int c = 0; c < CMAX; ++c)
    if (c < C && i0 + c < nb) {
      acc += rv[c];
      r[i0 + c] = rv[c];
      cum[i0 + c + 1] = c + 1 == C ? incl : acc;
    }
  __syncthreads();
  const double step = cum[nb] / (double)nb;
  for (int k = 1 + lane; k < nb; k += 64) {
    const double target = (double)k * step;
    // smallest i in [0, nb-1) with cum[i+1] >= target, else nb-1
    int lo = 0, hi = nb - 1;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (cum[mid + 1] >= target) hi = mid; else lo = mid + 1;
    }
    const int i = lo;
    double frac = 0.0;
    if (r[i] > 0.0) {
      frac = (target - cum[i]) / r[i];
      frac = frac < 0.0 ? 0.0 : (frac > 1.0 ? 1.0 : frac);
    }
    ej[k] = en[k] = e[i] + frac * (e[i + 1] - e[i]);
  }
  __syncthreads();
  for (int k = lane; k < nb; k += 64)
    bj[k] = grid_bin(k == 0 ? e[0] : en[k], k == nb - 1 ? e[nb] : en[k + 1]);
}

// The context's pinned memory; the grid (edges and bins) follows.
struct PinnedHost {
  IterRecord rec[MAX_RECORDS];
  Combined comb;
  double grid[1];
};

}  // namespace vgx

struct vgx_vegas {
  int device = 0;
  hipStream_t stream = nullptr;
  int kind = 0, dim = 0, nb = 0, prec = 0;
  double alpha = 1.5;
  uint64_t seed = 0;
  uint32_t stream_id = 0;
  vgx::IntegrandParams prm{};
  vgx::TTbarConst tt{};
  vgx::DYConst dy{};
  vgx::STConst st{};
  vgx::TTDynConst ttd{};  // TTBAR mode 2 (scale set per event)
  int tt_dyn = 0;
  int max_wg = 0;
  int pstride = 0;
  double* edges = nullptr;          // [dim][nb+1], then the bins
  double2* bins = nullptr;          // [dim][nb] grid_bin of the edges, in the same allocation
  double* hist = nullptr;           // [dim][nb]
  double* partials = nullptr;       // [max_wg][pstride]
  float* tables = nullptr;          // the integrand's LDS tables, staged once (hadronic kinds)
  int table_bytes = 0;
  vgx::IterRecord* rec = nullptr;   // [MAX_RECORDS]
  vgx::Combined* comb = nullptr;
  void* pinned = nullptr;           // host memory the device writes: PinnedHost
  int n_rec = 0;
  bool rec_host = true;             // the host mirror holds every record
  bool tail = false;                // work on the grid, histogram or records was enqueued since the stream was waited for
  bool comb_fresh = false;           // the host copy of the combination (in pinned) is current
  int pend_k = -1;                  // record holding only S1, S2 until the next refinement completes it (< 0: none)
  int64_t pend_n = 0;               // its sample count
  double judge_var = -1.0;          // n var(E) of the latest plain iteration read back (< 0: none)
  bool have_hist = false;
  // doubles of the edges (even, so that the bins are aligned) and of both
  size_t edge_doubles() const { return ((size_t)dim * (nb + 1) + 1) & ~(size_t)1; }
  size_t grid_doubles() const { return edge_doubles() + 2 * (size_t)dim * nb; }
  vgx::PinnedHost* host() const { return (vgx::PinnedHost*)pinned; }
  // kernel timing: event pairs recorded around the fused kernel, read back
  // (and summed) only when asked for, so timing does not synchronise
  static constexpr int kTimerPairs = 256;
  bool timing = false;
  int t_every = 1;                  // time one launch in t_every
  int64_t t_seen = 0;               // launches since timing was enabled
  hipEvent_t ev[2 * kTimerPairs] = {};
  int t_pending = 0;
  double t_ms = 0.0;
  int64_t t_launches = 0;
};

// Completes a record that vegas_iterate_async left pending (enqueued on the
// context's stream; nothing when none is pending).  Every path that reads
// the records or the combination, or adds a record, calls it first.
vgx_status vegas_flush_pending(vgx_vegas* v);
