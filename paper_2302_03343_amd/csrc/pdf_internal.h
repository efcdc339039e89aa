// Internal layout of a PDF grid on the device (shared by pdf.hip and the
// fused t tbar integrand).
#pragma once

#include "common.h"

#define VGX_MAX_SUB 8
#define VGX_MAX_FLAV 16

namespace vgx {

// Counters of the queries outside the grid, added up when they are asked for:
// one for most kernels, one per 128 bytes for workgroups that fill the chip
// and locate queries at the same time (1e6 queries, FP64, 1 % of them outside:
// 100 us per call at one address, now 65; 85 gathered).
constexpr int kOorSlots = 64, kOorStride = 16;

// One axis of a query located in LDS (pdf_lds.h): the start-cell bucket of a
// value whose FP64 top word is w is (w - w0) >> shift.
struct PdfLdsAxis {
  int n;  // knots (subgrids concatenated)
  int w0, shift;
  double lo, hi;
};

// The interpolation kernel with the grid in LDS: byte offsets of its tables
// (after the nodes), and the split of the workgroups over flavour groups.
struct PdfLdsArgs {
  PdfLdsAxis x, q;
  int n_flav, groups;
  int wg_full;                  // one group per workgroup: workgroups per full group (the last takes the rest)
  int tile;                     // all groups in turn: queries a workgroup locates at a time
  int node_bytes, tab_bytes;    // one group's nodes; the tables
  int o_kx, o_kq, o_hx, o_hq, o_log, o_bx, o_bq;
};

}  // namespace vgx

struct vgx_pdf {
  int device = 0;
  int n_x = 0, n_sub = 0, n_flav = 0;
  int n_members = 1;                  // members of a PDF set (shared knots), member-major values
  int fstride = 0;                    // node stride (= n_flav)
  int extrap = VGX_EXTRAP_ERROR;      // behaviour outside the grid (pdf_interp, pdf_alphas)
  int nq[VGX_MAX_SUB] = {0};
  int q_off[VGX_MAX_SUB + 1] = {0};   // knot offset of each subgrid
  // host copies (knots only; values stay on the device)
  double* h_x = nullptr;              // [n_x]
  double* h_q2 = nullptr;             // [q_off[n_sub]]
  // device arrays
  double* x = nullptr;                // [n_x]            x knots
  double* lx = nullptr;               // [n_x]            ln x knots
  double* q2 = nullptr;               // [total q]        Q^2 knots
  double* lq2 = nullptr;              // [total q]        ln Q^2 knots
  double* v64 = nullptr;              // [member][total q][n_x][fstride]  node values (FP64); member 0
                                      // is what pdf_interp and the fused integrands read
  float* v32 = nullptr;               // same, FP32 copy
  unsigned long long* oor = nullptr;  // out-of-range counters (kOorSlots)
  // tables of the interpolation with the grid in LDS (member 0), in one
  // block; null where a grid does not fit
  unsigned char* lds_block = nullptr;
  vgx::PdfLdsArgs lds_args{};
  size_t lds_o_ratios = 0, lds_o_n64 = 0, lds_o_n32 = 0;
  // alpha_s(Q) table (optional; pdf_set_alphas): knots on the Q^2 line split
  // into subgrids at duplicated knots
  int a_nsub = 0;
  int a_nq[VGX_MAX_SUB] = {0};
  int a_off[VGX_MAX_SUB + 1] = {0};
  double* h_aq2 = nullptr;            // host [total] knots
  double* h_aval = nullptr;           // host [total] values
  double* a_lq2 = nullptr;            // device [total] ln Q^2 knots
  double* a_val = nullptr;            // device [total] values
};
