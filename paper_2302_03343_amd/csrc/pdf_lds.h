// Log-bicubic interpolation with the grid in LDS, for batches of queries that
// fill the chip.
//
// Gathering each query's stencil from the L2 is bound by the texture
// addresser: 16-byte gathers of one query per lane from an L2-resident table
// take 49 to 122 clocks per wave instruction and CU, depending on the node
// stride (26 to 28 where neighbouring lanes share a node, as the gathering
// kernel arranges, with fewer queries per instruction), while random 16-byte
// reads of LDS take 13.4 (5.2 without bank conflicts; probe at 16 waves per CU).  All flavours of a grid do not fit in a CU's 160 KB, but
// 16 bytes of every node do (two FP64 or four FP32 flavours of 196 x 50
// nodes: 156.8 KB).  So a workgroup stages one group of flavours of the whole
// grid and evaluates that group for its queries; outputs stay
// structure-of-arrays and coalesced.  Two ways to cover the groups:
//   * one group per workgroup, for its lifetime: each group locates the
//     queries again, nothing is stored in between;
//   * all groups in turn (FP64, whose six groups locate most often): the
//     workgroup locates a tile of queries once and leaves cells and fractions
//     (16 bytes a query) where the first group's outputs will go; every
//     thread writes and reads only its own queries' words, the first group
//     comes last, and its outputs replace them.
// 1e8 queries: FP64 8.2 -> 5.3 ms (2.0 TB/s of the 104 bytes a query that
// have to move), FP32 5.9 -> 3.75 ms.  Counters of the FP64 kernel at 1e8: LDS
// busy 0.75 of the cycles (bank conflicts 0.49), VALU issue 0.52, and the
// records come back from beyond the L2 (21.8 GB read and written past it); of
// the FP32 kernel at 1e8: LDS 0.69 (0.45), VALU 0.74, at 1e6, copying the nodes
// in included, 0.49 and 0.52.
// Ordering each query's rows so that the lanes of an LDS cycle fall on
// different banks lowered the conflicts, not the time (1 %), and is not kept.
//
// Locating a query in one axis:
//   * cell: the top word of the FP64 value is a piecewise-linear logarithm;
//     shifted, it indexes a table of start cells, from which the exact
//     comparisons with the knots step forward (one step of two knots where
//     a bucket holds no more than two).  The cell is the binary search's.
//   * fraction: t = log(1 + d) / h_i, d = (v - v_i) / v_i, with 1/v_i and
//     1/h_i (from the knots in extended precision) tabled.  Every step keeps
//     its relative precision, where ln v - ln v_i loses the digits that the
//     two logarithms share: t is within 5e-16 (7e-17 rms) anywhere, ln v - ln v_i
//     within 2e-14 at x = 1e-9 and 5e-16 near x = 1 (emulated, 196 x 50 even
//     knots).  The values' error in the norm, measured against extended
//     precision per decade of x and in four ranges above 0.1, is 1.2e-16 to
//     1.5e-16 (gathering kernel 1.8e-16 to 3.2e-16).  t is exactly 0 on a
//     knot and 1 on the last one.
//     log(1 + d) = e ln 2 - ln c + log1p(r), r = (1 + d) 2^-e c - 1, for
//     1 + d = m 2^e, c = 1/(1 + k/32) with 1 + k/32 nearest to m (|r| <= 1/64,
//     c = 1 next to d = 0) and the Taylor series of log1p to eighth order
//     (remainder below 1e-17); only e and k come from the rounded 1 + d.
#pragma once

#include "pdf_internal.h"

#include <math.h>

namespace vgx {

constexpr int kLdsBlock = 1024;         // one workgroup per CU: four waves per SIMD
constexpr size_t kLdsCap = 160 * 1024;  // LDS of a CU
constexpr int kLogTab = 32;             // steps of the logarithm's table (one entry more)
constexpr int kMaxLdsKnots = 256;       // start cells are bytes

// The staged block: nodes [row][x] of 16 bytes | knots of x and of Q^2, each
// with its reciprocal (the last knot reads +inf, and one more follows) | 1/h
// of the cells of x and of Q^2 | the logarithm's table | start cells of x and
// of Q^2.

// Start cell, then the comparisons: the last k with knot[k] <= v (the knots
// of the subgrids are concatenated, a threshold appearing twice, so that the
// upper subgrid wins there); knot[n - 1] and knot[n] read +inf, so k <= n - 2.
__device__ __forceinline__ int lds_cell(const PdfLdsAxis& ax, const unsigned char* start, const double2* knot,
                                        double v) {
  int k = start[(__double2hiint(v) - ax.w0) >> ax.shift];
  while (true) {
    const double k1 = knot[k + 1].x, k2 = knot[k + 2].x;
    const bool far = v >= k2;
    k += (v >= k1 ? 1 : 0) + (far ? 1 : 0);
    if (!__any(far)) return k;
  }
}

// log(1 + d) for d >= 0 (see above).
constexpr double kLn2 = 0.6931471805599453;
__device__ __forceinline__ double lds_log1p(const double2* tab, double d) {
  const int hi = __double2hiint(1.0 + d), e = (hi >> 20) - 1023;
  const double2 c = tab[((hi & 0xFFFFF) + 0x4000) >> 15];
  const double ce = __builtin_amdgcn_ldexp(c.x, -e);
  const double r = fma(d, ce, ce - 1.0);
  double p = fma(r, -1.0 / 8, 1.0 / 7);
  p = fma(r, p, -1.0 / 6);
  p = fma(r, p, 1.0 / 5);
  p = fma(r, p, -1.0 / 4);
  p = fma(r, p, 1.0 / 3);
  p = fma(r, p, -1.0 / 2);
  p = fma(r * r, p, r);
  return fma((double)e, kLn2, c.y) + p;
}

// Weights of the nodes k-1 .. k+2 of the cubic Hermite with secant-average
// slopes at fraction t, r = (h_k/h_{k-1}, h_k/h_{k+1}).
__device__ __forceinline__ void lds_hermite(double t, double2 r, double (&c)[4]) {
  const double s = 1.0 - t, ts = 0.5 * t * s;
  const double a = ts * s, b = -ts * t;          // half the slope basis functions
  const double h01 = t * t * fma(-2.0, t, 3.0);
  c[0] = -a * r.x;
  c[3] = b * r.y;
  c[1] = (1.0 - h01) - (a + b) - c[0];
  c[2] = h01 + (a + b) - c[3];
}

// Linear weights (1 - t, t) on positions pos, pos + 1 of a four-node window.
__device__ __forceinline__ void lds_linear(double t, int pos, double (&c)[4]) {
  const double u = 1.0 - t;
  c[0] = pos == 0 ? u : 0.0;
  c[1] = pos == 1 ? u : (pos == 0 ? t : 0.0);
  c[2] = pos == 2 ? u : (pos == 1 ? t : 0.0);
  c[3] = pos == 2 ? t : 0.0;
}

// A located query: cells and fractions, or no value.
struct LdsQuery {
  int i, j;      // cells; i = kLdsNaN / kLdsSkip: no value, written as NaN / not written
  double ta, tb; // fractions in [0, 1]
};
constexpr int kLdsNaN = 0x1FF, kLdsSkip = 0x1FE;  // above any cell

// A cell and a fraction in 64 bits: t + 2^-6, whose exponent takes seven
// values, less the smallest of them fills the low 55, the cell the top 9.  t
// comes back as it was where the sum stays in t's binade (all but the last
// 2^-6 below a power of two, where it is rounded once), below 2^-6 to 2^-59.
constexpr double kPackShift = 0x1p-6;
constexpr unsigned kPackHi = 0x3F900000u;  // the top word of 2^-6
__device__ __forceinline__ double lds_pack(int cell, double t) {
  const double u = kPackShift + fmin(fmax(t, 0.0), 1.0);
  return __hiloint2double((int)(((unsigned)__double2hiint(u) - kPackHi) | ((unsigned)cell << 23)), __double2loint(u));
}
__device__ __forceinline__ int lds_cell_of(double w) { return (int)((unsigned)__double2hiint(w) >> 23); }
__device__ __forceinline__ double lds_fraction(double w) {
  return __hiloint2double((int)(((unsigned)__double2hiint(w) & 0x7FFFFFu) + kPackHi), __double2loint(w)) - kPackShift;
}

// MODE as in k_pdf_interp.  ratios: (h_k/h_{k-1}, h_k/h_{k+1}) per cell of
// both axes, first component negative where the four-knot stencil is
// incomplete: in global memory (the L1, whose path is idle) while the tables
// for locating fill the LDS, in their place where locating is done.
template <typename OutT, typename ValT, int MODE>
struct PdfLds {
  static constexpr int V = 16 / (int)sizeof(ValT);
  typedef ValT NodeV __attribute__((ext_vector_type(V)));

  const PdfLdsArgs& a;
  const unsigned char* nodes;  // LDS
  const unsigned char* tab;    // LDS
  const double2* ratios;
  unsigned long long* oor;
  bool count;                  // whether this workgroup counts the queries without a value

  __device__ __forceinline__ LdsQuery locate(double x, double q2) const {
    if constexpr (MODE == VGX_EXTRAP_FREEZE) {  // the nearest grid point
      if (x > 0.0 && q2 > 0.0 && isfinite(x) && isfinite(q2)) {
        x = fmin(fmax(x, a.x.lo), a.x.hi);
        q2 = fmin(fmax(q2, a.q.lo), a.q.hi);
      }
    }
    const bool inside = x >= a.x.lo && x <= a.x.hi && q2 >= a.q.lo && q2 <= a.q.hi;
    bool skip = false;
    if (!inside) {
      if constexpr (MODE == VGX_EXTRAP_CONTINUE)  // k_pdf_continue writes these
        skip = x > 0.0 && q2 > 0.0 && isfinite(x) && isfinite(q2) && x <= a.x.hi;
      if (!skip && count) atomicAdd(oor, 1ull);
      x = a.x.lo;  // any point of the grid
      q2 = a.q.lo;
    }
    const double2 *kx = (const double2*)(tab + a.o_kx), *kq = (const double2*)(tab + a.o_kq);
    const double *hx = (const double*)(tab + a.o_hx), *hq = (const double*)(tab + a.o_hq);
    const double2* lt = (const double2*)(tab + a.o_log);
    LdsQuery r;
    r.i = lds_cell(a.x, tab + a.o_bx, kx, x);
    r.j = lds_cell(a.q, tab + a.o_bq, kq, q2);
    const double2 ki = kx[r.i], kj = kq[r.j];
    const double ta = lds_log1p(lt, (x - ki.x) * ki.y) * hx[r.i];
    const double tb = lds_log1p(lt, (q2 - kj.x) * kj.y) * hq[r.j];
    r.ta = x == a.x.hi ? 1.0 : ta;
    r.tb = q2 == a.q.hi ? 1.0 : tb;
    if (!inside) r.i = skip ? kLdsSkip : kLdsNaN;
    return r;
  }

  // The group's flavours of a located query, stored at out (flavour stride n)
  __device__ __forceinline__ void evaluate(const LdsQuery& k, int nv, OutT* out, int64_t n) const {
    const bool inside = k.i < kLdsSkip;
    const int i = inside ? k.i : 0, j = k.j;
    const double2 rx = ratios[i], rq = ratios[a.x.n + j];
    double c[4], d[4];
    lds_hermite(k.ta, rx, c);
    lds_hermite(k.tb, rq, d);
    int i0 = i - 1, j0 = j - 1;
    const bool full = rx.x >= 0.0 && rq.x >= 0.0;
    if (!__all(full)) {  // bilinear cells, as a window with zero weights inside the grid
      if (!full) {
        i0 = i0 < 0 ? 0 : (i0 > a.x.n - 4 ? a.x.n - 4 : i0);
        j0 = j0 < 0 ? 0 : (j0 > a.q.n - 4 ? a.q.n - 4 : j0);
        lds_linear(k.ta, i - i0, c);
        lds_linear(k.tb, j - j0, d);
      }
    }
    const int row_bytes = a.x.n * 16;
    const unsigned char* p = nodes + j0 * row_bytes + i0 * 16;
    double acc[V];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const NodeV* node = (const NodeV*)(p + r * row_bytes);
      const NodeV v0 = node[0], v1 = node[1], v2 = node[2], v3 = node[3];
#pragma unroll
      for (int u = 0; u < V; ++u) {
        const double s = fma(c[0], (double)v0[u], fma(c[1], (double)v1[u], fma(c[2], (double)v2[u], c[3] * (double)v3[u])));
        acc[u] = r == 0 ? d[0] * s : fma(d[r], s, acc[u]);
      }
    }
    if (MODE != VGX_EXTRAP_CONTINUE || k.i != kLdsSkip) {
#pragma unroll
      for (int u = 0; u < V; ++u)
        if (u < nv) out[(int64_t)u * n] = inside ? (OutT)acc[u] : (OutT)NAN;
    }
  }

  // A located query as two words, in the place of a group's two outputs
  __device__ __forceinline__ void store(const LdsQuery& k, double* out, int64_t n) const {
    out[0] = lds_pack(k.i, k.ta);
    out[n] = lds_pack(k.j, k.tb);
  }
  __device__ __forceinline__ LdsQuery query(double wx, double wq) const {
    return {lds_cell_of(wx), lds_cell_of(wq), lds_fraction(wx), lds_fraction(wq)};
  }
};

// ALL: every group in turn per workgroup, else one group per workgroup.
template <typename OutT, typename ValT, int MODE, bool ALL>
__global__ __launch_bounds__(kLdsBlock) void k_pdf_interp_lds(PdfLdsArgs a, int64_t n, const double* __restrict__ qx,
                                                              const double* __restrict__ qq2,
                                                              const unsigned char* __restrict__ tables,
                                                              const unsigned char* __restrict__ nodes,
                                                              const double2* __restrict__ ratios, OutT* out,
                                                              unsigned long long* __restrict__ oor) {
  using P = PdfLds<OutT, ValT, MODE>;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  // this workgroup's group (all groups: the first) and its place among the group's workgroups
  const int last = ALL ? 0 : a.groups - 1;
  int g0 = blockIdx.x / a.wg_full;
  g0 = g0 < last ? g0 : last;
  const int first_wg = g0 * a.wg_full;
  const int wgs = g0 < last ? a.wg_full : (int)gridDim.x - first_wg;
  const int wg = blockIdx.x - first_wg;
  P p{a, lds_raw, lds_raw + a.node_bytes, ALL ? (const double2*)(lds_raw + a.node_bytes) : ratios,
      oor + blockIdx.x % kOorSlots * kOorStride, g0 == 0};
  if constexpr (!ALL) {
    copy16(lds_raw + a.node_bytes, tables, a.tab_bytes);
    copy16(lds_raw, nodes + (size_t)g0 * a.node_bytes, a.node_bytes);
    __syncthreads();
    OutT* o = out + (int64_t)g0 * P::V * n;
    const int nv = a.n_flav - g0 * P::V;
    const int64_t step = (int64_t)wgs * kLdsBlock;
    int64_t q = (int64_t)wg * kLdsBlock + threadIdx.x;
    double xn = 0.0, qn = 0.0;
    if (q < n) { xn = qx[q]; qn = qq2[q]; }
    for (; q < n; q += step) {
      const double x = xn, q2 = qn;
      if (q + step < n) { xn = qx[q + step]; qn = qq2[q + step]; }  // the next query, while this one is evaluated
      p.evaluate(p.locate(x, q2), nv, o + q, n);
    }
  } else {
    for (int64_t t0 = (int64_t)wg * a.tile; t0 < n; t0 += (int64_t)wgs * a.tile) {
      const int64_t t1 = t0 + a.tile < n ? t0 + a.tile : n;
      // the tables for locating, then (in their place) the ratios for evaluating
      __syncthreads();
      copy16(lds_raw + a.node_bytes, tables, a.tab_bytes);
      __syncthreads();
      for (int64_t q = t0 + threadIdx.x; q < t1; q += kLdsBlock) p.store(p.locate(qx[q], qq2[q]), out + q, n);
      for (int g = a.groups - 1; g >= 0; --g) {
        __syncthreads();  // the nodes of the previous group have been read
        copy16(lds_raw, nodes + (size_t)g * a.node_bytes, a.node_bytes);
        if (g == a.groups - 1) copy16(lds_raw + a.node_bytes, ratios, (a.x.n + a.q.n) * 16);
        __syncthreads();
        OutT* o = out + (int64_t)g * P::V * n;
        const int nv = a.n_flav - g * P::V;
        int64_t q = t0 + threadIdx.x;
        double xn = 0.0, qn = 0.0;
        if (q < t1) { xn = out[q]; qn = out[n + q]; }
        for (; q < t1; q += kLdsBlock) {
          const double wx = xn, wq = qn;
          if (q + kLdsBlock < t1) { xn = out[q + kLdsBlock]; qn = out[n + q + kLdsBlock]; }
          p.evaluate(p.query(wx, wq), nv, o + q, n);
        }
      }
    }
  }
}

// Nodes of one member in the layout that the workgroups stage: [group][node]
// of 16 bytes, flavours past the last zero.
template <typename ValT>
__global__ __launch_bounds__(256) void k_pdf_group(const ValT* __restrict__ vals, int n_nodes, int nf, int groups,
                                                   ValT* __restrict__ out) {
  constexpr int V = 16 / (int)sizeof(ValT);
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= groups * n_nodes * V) return;
  const int f = (k / (n_nodes * V)) * V + k % V, node = (k / V) % n_nodes;
  out[k] = f < nf ? vals[(size_t)node * nf + f] : (ValT)0;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
constexpr int kMinBuckets = 48;  // start cells an axis needs at least

inline int pdf_top_word(double v) {
  uint64_t b;
  memcpy(&b, &v, 8);
  return (int)(b >> 32);
}

// Last k <= n - 2 with knot[k] <= v.
inline int pdf_host_cell(const double* knot, int n, double v) {
  int k = 0;
  while (k < n - 2 && knot[k + 1] <= v) ++k;
  return k;
}

// Offsets of the staged block, or false for a grid that it cannot hold: the
// nodes, their tables and the start cells must fit in a CU's LDS (about 9850
// nodes), the windows need four knots per axis, start cells are bytes.
inline bool pdf_lds_plan(const vgx_pdf* p, PdfLdsArgs& a) {
  const int nx = p->n_x, nq = p->q_off[p->n_sub];
  const double tiny = 1e-150, huge = 1e150;  // 1/v is finite and normal, as is v/v_i in a cell however wide
  if (p->h_x[0] < tiny || p->h_x[nx - 1] > huge || p->h_q2[0] < tiny || p->h_q2[nq - 1] > huge) return false;
  if (nx < 4 || nq < 4 || nx > kMaxLdsKnots || nq > kMaxLdsKnots) return false;
  auto up16 = [](int b) { return (b + 15) & ~15; };
  int o = 0;
  auto place = [&](int bytes) { const int at = o; o += up16(bytes); return at; };
  a.node_bytes = nx * nq * 16;
  a.o_kx = place((nx + 1) * 16);
  a.o_kq = place((nq + 1) * 16);
  a.o_hx = place(nx * 8);
  a.o_hq = place(nq * 8);
  a.o_log = place((kLogTab + 1) * 16);
  const int left = ((int)kLdsCap - a.node_bytes - o) & ~15;
  if (left < 3 * kMinBuckets) return false;
  const int bx = ((left < 3072 ? left : 3072) * 2 / 3) & ~15, bq = (left < 3072 ? left : 3072) - bx;
  a.o_bx = place(bx);
  a.o_bq = place(bq);
  a.tab_bytes = o;
  auto axis = [](PdfLdsAxis& ax, const double* knot, int n, int buckets) {
    ax.n = n;
    ax.lo = knot[0];
    ax.hi = knot[n - 1];
    ax.w0 = pdf_top_word(ax.lo);
    ax.shift = 0;
    while (((pdf_top_word(ax.hi) - ax.w0) >> ax.shift) >= buckets) ++ax.shift;
  };
  axis(a.x, p->h_x, nx, bx);
  axis(a.q, p->h_q2, nq, bq);
  a.n_flav = p->n_flav;
  return true;
}

// The tables (tab_bytes) and the stencil ratios (16 bytes per cell, x then
// Q^2) of a planned grid, from its knots.
inline void pdf_lds_fill(const vgx_pdf* p, const PdfLdsArgs& a, unsigned char* tab, double* ratios) {
  memset(tab, 0, (size_t)a.tab_bytes);
  // spacings in the logarithm; zero for a threshold's two knots
  long double hx[kMaxLdsKnots], hq[kMaxLdsKnots];
  auto spacings = [](const double* knot, int n, long double* h) {
    for (int k = 0; k + 1 < n; ++k) h[k] = log1pl(((long double)knot[k + 1] - knot[k]) / knot[k]);
  };
  spacings(p->h_x, p->n_x, hx);
  spacings(p->h_q2, p->q_off[p->n_sub], hq);
  auto axis = [&](const PdfLdsAxis& ax, const double* knot, const long double* hl, int o_knot, int o_h, int o_start,
                  int o_end) {
    double* k2 = (double*)(tab + o_knot);
    double* h = (double*)(tab + o_h);
    for (int k = 0; k <= ax.n; ++k) {
      k2[2 * k] = k + 1 < ax.n ? knot[k] : INFINITY;
      k2[2 * k + 1] = k + 1 < ax.n ? 1.0 / knot[k] : 0.0;
      if (k < ax.n) h[k] = k + 1 < ax.n && hl[k] > 0.0L ? (double)(1.0L / hl[k]) : 0.0;
    }
    for (int b = 0; b < o_end - o_start; ++b) {
      // a bucket past the top word's range is never looked up
      const int64_t w = (int64_t)ax.w0 + ((int64_t)b << ax.shift);
      const uint64_t bits = (uint64_t)(w < 0x7FF00000 ? w : 0x7FEFFFFF) << 32;
      double v;
      memcpy(&v, &bits, 8);
      tab[o_start + b] = b == 0 ? 0 : (unsigned char)pdf_host_cell(knot, ax.n, v);
    }
  };
  axis(a.x, p->h_x, hx, a.o_kx, a.o_hx, a.o_bx, a.o_bq);
  axis(a.q, p->h_q2, hq, a.o_kq, a.o_hq, a.o_bq, a.tab_bytes);
  double* lt = (double*)(tab + a.o_log);
  for (int k = 0; k <= kLogTab; ++k) {  // exact at both ends: c = 1, and c = 1/2 with ln 2 as in lds_log1p
    const double c = 1.0 / (1.0 + (double)k / kLogTab);
    lt[2 * k] = c;
    lt[2 * k + 1] = k == 0 ? 0.0 : k == kLogTab ? kLn2 : (double)-logl((long double)c);
  }
  auto stencil = [](double* r, const long double* h, int n) {
    for (int k = 0; k < n; ++k) {
      const bool full = k >= 1 && k <= n - 3;
      r[2 * k] = full ? (double)(h[k] / h[k - 1]) : -1.0;
      r[2 * k + 1] = full ? (double)(h[k] / h[k + 1]) : 0.0;
    }
  };
  stencil(ratios, hx, p->n_x);
  for (int s = 0; s < p->n_sub; ++s) stencil(ratios + 2 * (p->n_x + p->q_off[s]), hq + p->q_off[s], p->nq[s]);
}

}  // namespace vgx
