// Batched VEGAS: many independent integrals of uneven dimension and sample
// count in one persistent launch per iteration, captured with the
// reductions and the refinements in one HIP graph.
//
// Each integral keeps its own grid, Philox stream and record list (its
// vgx_vegas context), so an integral computed in a batch draws exactly the
// samples it would draw alone (thesis VEGAS section for the per-integral
// algorithm; the batching is an implementation choice).
//
// MI355X design
//   * work is cut into tiles of T consecutive samples of one integral; the
//     tiles of all integrals form one index space, integral i owning the
//     range [tile0_i, tile0_i + ntiles_i);
//   * a persistent grid (as many workgroups as can be resident at once)
//     pops tile indices from an atomic counter, so integrals with 1e4 and
//     1e7 samples load-balance across the 256 CUs; the grid's bins are read
//     from global memory (L1), so nothing is staged per tile;
//   * the tile's histogram has up to 16 columns per bin in LDS (lane l adds
//     into column l mod columns), summed in a fixed order;
//   * every tile writes its own partial row (S1, S2 compensated, histogram),
//     so the reduction kernel sums each integral's rows in tile order: the
//     result does not depend on which workgroup took which tile;
//   * the dimension and family are switched per tile to fully unrolled
//     instantiations (D = 1..12);
//   * begin (counter reset, a kernel, not a memset), persistent kernel,
//     reduction and refinement are captured once in a graph; per-iteration
//     inputs (iteration number, record slots) are read from device memory,
//     which the host updates before each replay;
//   * the tile size T and block size are chosen by timing candidate
//     configurations once per batch (autotuner), unless given.
#include "common.h"
#include "integrands.h"
#include "vegas_internal.h"

#include <algorithm>
#include <math.h>
#include <stdlib.h>
#include <string.h>
#include <vector>

namespace vgx {

constexpr int BB_MAX = 256;  // launch bound of the persistent kernel
// A tile's histogram in LDS: [dim nb][columns] doubles, lane l adding into
// column l mod columns, up to 16 columns per integral, as many as fit in the
// workgroup's LDS.  LDS executes an FP64 atomic 16 lanes at a time,
// each group as often as its fullest bank pair has lanes: with random bins
// 27.5 clocks per wave instruction, with 8 columns 17.9, with 16 10.2.
// The registers allow two waves per SIMD, eight per CU, and the columns must
// not keep workgroups of them away: 160 KB over the workgroups, less the
// kernel's own LDS, and at most 40 KB.  16 integrals of 10 x 64 bins and 2e6
// samples: 64 threads (eight workgroups) 620 us with 40 KB, 401 now; 128 (four)
// 420 and 381; 256 (two) 351, and 362 with a few bytes less than 40 KB, which
// halves the columns here.
constexpr size_t kColsLds = 40 * 1024, kOwnLds = 256;
constexpr int kMaxColsLog2 = 4, kWavesPerCu = 8;
inline int hist_shift(int dim, int nb, int block) {
  const size_t fair = (size_t)160 * 1024 / (kWavesPerCu * 64 / block) - kOwnLds, room = fair < kColsLds ? fair : kColsLds;
  int s = 0;
  while (s < kMaxColsLog2 && (sizeof(double) * dim * nb) << (s + 1) <= room) ++s;
  return s;
}

struct BatchItem {
  int kind, prec, dim, nb;
  int shift;             // log2 of the LDS histogram's columns
  uint32_t sid, k0, k1;
  int pstride;           // 4 + dim * nb
  int64_t n;             // samples per iteration
  int64_t tile0;         // first tile of this integral
  int64_t ntiles;
  int64_t part_off;      // first double of this integral's tile partials
  double alpha;
  double* edges;         // context grid [dim][nb+1]
  double2* bins;         // and its bins [dim][nb]
  double* hist;          // context histogram [dim][nb]
  IterRecord* rec;       // context records
  Combined* comb;
  IntegrandParams prm;
};

// Per-iteration inputs, one host-to-device copy: the tile counter, the
// iteration number, then the record slot of every integral (int32[count]).
struct BatchState {
  unsigned long long tile_counter;
  int iteration;
  int pad;
};
__host__ __device__ inline int* batch_krec(BatchState* st) { return (int*)(st + 1); }

template <int D, bool ODD, class F>
__device__ __forceinline__ void run_tile_parity(const BatchItem& it, const F& f, double* sh, int64_t s0, int64_t s1,
                                         uint32_t iter, Comp& c1, Comp& c2) {
  double p1 = 0.0, p2 = 0.0;
  double nbDs = 1.0;
#pragma unroll
  for (int j = 0; j < D; ++j) nbDs *= (double)it.nb * 0x1p32;
  for (int64_t i = s0 + threadIdx.x; i < s1; i += blockDim.x) {
    double x[D];
    uint32_t k[D];
    int idx[D];
#pragma unroll
    for (int b = 0; b < (D + 3) / 4; ++b) {
      const u32x4 w4 = philox4x32_10((uint32_t)i, (uint32_t)((uint64_t)i >> 32), iter, (it.sid << 8) | (uint32_t)b,
                                     it.k0, it.k1);
      const uint32_t ww[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * b + e < D) k[4 * b + e < D ? 4 * b + e : 0] = ww[e];
    }
    const double jac = grid_map_words<D, ODD>(k, it.bins, it.nb, nbDs, x, idx);
    const double w = eval_inside(f, x) * jac;
    const double w2 = w * w;
    p1 += w;
    p2 += w2;
#pragma unroll
    for (int j = 0; j < D; ++j) atomicAdd(&sh[(j * it.nb + idx[j]) << it.shift], w2);
  }
  c1.add(p1);
  c2.add(p2);
}

template <int D, bool ODD, class F>
__device__ __forceinline__ void run_tile(const BatchItem& it, const F& f, double* sh, int64_t s0, int64_t s1,
                                         uint32_t iter, Comp& c1, Comp& c2) {
  if (ODD && (it.nb & 1)) run_tile_parity<D, true>(it, f, sh, s0, s1, iter, c1, c2);
  else run_tile_parity<D, false>(it, f, sh, s0, s1, iter, c1, c2);
}

template <int D, bool ODD>
__device__ __forceinline__ void run_tile_d(const BatchItem& it, double* sh, int64_t s0, int64_t s1, uint32_t iter,
                                           Comp& c1, Comp& c2) {
#define VGX_BT(T)                                                      \
  if (it.prec == VGX_F64) {                                            \
    T<D, double> f;                                                    \
    f.prm = it.prm;                                                    \
    run_tile<D, ODD>(it, f, sh, s0, s1, iter, c1, c2);             \
  } else {                                                             \
    T<D, float> f;                                                     \
    f.prm = it.prm;                                                    \
    run_tile<D, ODD>(it, f, sh, s0, s1, iter, c1, c2);             \
  }
  switch (it.kind) {
    case VGX_GAUSS: { VGX_BT(Gauss) break; }
    case VGX_GENZ_OSC: { VGX_BT(GenzOsc) break; }
    default: { VGX_BT(GenzPeak) break; }
  }
#undef VGX_BT
}

// Reset the tile counter at the start of an iteration (graph-safe: a kernel).
__global__ void k_batch_begin(BatchState* st) {
  if (threadIdx.x == 0 && blockIdx.x == 0) st->tile_counter = 0ull;
}

// ODD: some integral of the batch has an odd bin count, and the kernel holds
// the loops for both parities (64 integrals of even counts took 2077 us so, for
// three iterations, and take 2045 with the loops for even counts alone).
template <bool ODD>
__global__ __launch_bounds__(BB_MAX) void k_batch(const BatchItem* __restrict__ items, int count, int64_t total_tiles,
                                                 int tile, BatchState* __restrict__ st,
                                                 double* __restrict__ partials) {
  extern __shared__ double lds[];
  __shared__ int64_t s_tile;
  __shared__ int s_item;
  __shared__ double red[4][BB_MAX / 64];
  const uint32_t iter = (uint32_t)st->iteration;
  double* sh = lds;
  while (true) {
    if (threadIdx.x == 0) {
      const int64_t t = (int64_t)atomicAdd(&st->tile_counter, 1ull);
      s_tile = t;
      int lo = 0, hi = count - 1;  // integral owning tile t: last with tile0 <= t
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].tile0 <= t) lo = mid; else hi = mid - 1;
      }
      s_item = lo;
    }
    __syncthreads();
    const int64_t t = s_tile;
    if (t >= total_tiles) break;  // uniform: every wave leaves
    const int k = s_item;
    const BatchItem& it = items[k];
    const int cols = 1 << it.shift;
    for (int q = threadIdx.x; q < (it.dim * it.nb) << it.shift; q += blockDim.x) sh[q] = 0.0;
    __syncthreads();
    const int64_t lt = t - it.tile0;
    const int64_t s0 = lt * tile;
    const int64_t s1 = (s0 + tile < it.n) ? s0 + tile : it.n;
    Comp c1, c2;
    double* shl = sh + (threadIdx.x & (cols - 1));  // this lane's column
    switch (it.dim) {
      case 1: run_tile_d<1, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      case 2: run_tile_d<2, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      case 3: run_tile_d<3, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      case 4: run_tile_d<4, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      case 5: run_tile_d<5, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      case 6: run_tile_d<6, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      case 7: run_tile_d<7, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      case 8: run_tile_d<8, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      case 9: run_tile_d<9, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      case 10: run_tile_d<10, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      case 11: run_tile_d<11, ODD>(it, shl, s0, s1, iter, c1, c2); break;
      default: run_tile_d<12, ODD>(it, shl, s0, s1, iter, c1, c2); break;
    }
    const double v0 = wave_sum(c1.s), v1 = wave_sum(c1.c), v2 = wave_sum(c2.s), v3 = wave_sum(c2.c);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (lane == 0) { red[0][wv] = v0; red[1][wv] = v1; red[2][wv] = v2; red[3][wv] = v3; }
    __syncthreads();
    double* row = partials + it.part_off + lt * it.pstride;
    if (threadIdx.x < 4) {
      double s = 0.0;
      for (int q = 0; q < nw; ++q) s += red[threadIdx.x][q];
      row[threadIdx.x] = s;
    }
    for (int q = threadIdx.x; q < it.dim * it.nb; q += blockDim.x) {
      // from column q mod cols round: neighbouring q on different banks
      double h = 0.0;
      for (int c = 0; c < cols; ++c) h += sh[(q << it.shift) + ((c + q) & (cols - 1))];
      row[4 + q] = h;
    }
    __syncthreads();  // LDS histogram and s_tile are reused by the next tile
  }
}

// Per integral (blockIdx.y) and column block (blockIdx.x): sum the tile rows;
// block x = 0 finalises the record and the combination, and copies the record
// to out[blockIdx.y] (all integrals' records in one array: one read-back).
// Thread (g, c) of BR_GROUPS row groups sums rows g, g + BR_GROUPS, ... of column
// c, eight loads in flight (bound by their latency: four groups with one
// load at a time took 40 us for up to 610 rows per integral, this takes
// 11.6 us); the groups are merged in order.
constexpr int BR_GROUPS = 16, BR_COLS = 64;

__global__ __launch_bounds__(BR_GROUPS * BR_COLS) void k_batch_reduce(const BatchItem* __restrict__ items,
                                                                      const double* __restrict__ partials,
                                                                      BatchState* st, IterRecord* __restrict__ out) {
  const BatchItem& it = items[blockIdx.y];
  __shared__ double ss[BR_GROUPS][BR_COLS], sc[BR_GROUPS][BR_COLS];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int col = blockIdx.x * BR_COLS + lane;
  const int ncols = it.pstride;
  if (blockIdx.x * BR_COLS >= ncols) return;  // uniform per block
  Comp acc;
  if (col < ncols) {
    const double* p = partials + it.part_off + col;
    for (int64_t r = grp; r < it.ntiles; r += 8 * BR_GROUPS) {
      double v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int64_t k = r + q * BR_GROUPS;
        v[q] = k < it.ntiles ? p[k * it.pstride] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (r + q * BR_GROUPS < it.ntiles) acc.add(v[q]);
    }
  }
  ss[grp][lane] = acc.s;
  sc[grp][lane] = acc.c;
  __syncthreads();
  if (grp == 0) {
    Comp t;
    for (int g = 0; g < BR_GROUPS; ++g) { t.add(ss[g][lane]); t.c += sc[g][lane]; }
    ss[0][lane] = t.value();
    if (col >= 4 && col < ncols) it.hist[col - 4] = t.value();
  }
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    const int k_rec = batch_krec(st)[blockIdx.y];
    finalize_record(ss[0][0] + ss[0][1], ss[0][2] + ss[0][3], it.n, it.rec, k_rec, it.comb);
    if (threadIdx.x == 0) out[blockIdx.y] = it.rec[k_rec];  // the lane that stored it
  }
}

// Per integral (blockIdx.y) and dimension (blockIdx.x): Lepage refinement.
__global__ __launch_bounds__(64) void k_batch_refine(const BatchItem* __restrict__ items, BatchState* st) {
  const BatchItem& it = items[blockIdx.y];
  if ((int)blockIdx.x >= it.dim) return;  // uniform per block
  refine_dim(it.edges + (size_t)blockIdx.x * (it.nb + 1), it.bins + (size_t)blockIdx.x * it.nb,
             it.hist + (size_t)blockIdx.x * it.nb, it.nb, it.alpha);
}

}  // namespace vgx

using namespace vgx;

struct vgx_batch {
  int device = 0;
  hipStream_t stream = nullptr;      // replay stream (the first context's)
  hipStream_t cap = nullptr;         // private capture stream
  int count = 0;
  std::vector<vgx_vegas*> ctx;
  std::vector<int64_t> n;
  std::vector<BatchItem> items;      // host mirror
  BatchItem* d_items = nullptr;
  BatchState* d_state = nullptr;     // BatchState + int32 record slots [count]
  IterRecord* d_out = nullptr;       // this iteration's records [count]
  double* partials = nullptr;
  size_t part_cap = 0;               // doubles
  int tile = 0, block = 0, grid = 0;
  int64_t total_tiles = 0;
  size_t lds = 0;
  int max_cols = 0;
  bool odd = false;                  // an odd bin count among the integrals
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  IterRecord* pinned = nullptr;      // count records
  BatchState* pinned_state = nullptr;
};

namespace {

void layout(vgx_batch* b, int tile) {
  int64_t t0 = 0, off = 0;
  for (int k = 0; k < b->count; ++k) {
    BatchItem& it = b->items[k];
    it.tile0 = t0;
    it.ntiles = (b->n[k] + tile - 1) / tile;
    it.part_off = off;
    t0 += it.ntiles;
    off += it.ntiles * it.pstride;
  }
  b->total_tiles = t0;
  b->tile = tile;
}

size_t partial_doubles(const vgx_batch* b, int tile) {
  size_t off = 0;
  for (int k = 0; k < b->count; ++k) off += (size_t)((b->n[k] + tile - 1) / tile) * b->items[k].pstride;
  return off;
}

size_t state_bytes(int count) { return sizeof(BatchState) + sizeof(int) * (size_t)count; }

vgx_status upload_items(vgx_batch* b, hipStream_t st) {
  VGX_HIP(hipMemcpyAsync(b->d_items, b->items.data(), sizeof(BatchItem) * b->count, hipMemcpyHostToDevice, st));
  return VGX_OK;
}

vgx_status enqueue_iteration(vgx_batch* b, hipStream_t st, bool refine) {
  hipLaunchKernelGGL(k_batch_begin, dim3(1), dim3(64), 0, st, b->d_state);
  hipLaunchKernelGGL(b->odd ? k_batch<true> : k_batch<false>, dim3(b->grid), dim3(b->block), b->lds, st, b->d_items, b->count, b->total_tiles,
                     b->tile, b->d_state, b->partials);
  if (refine) {
    hipLaunchKernelGGL(k_batch_reduce, dim3((b->max_cols + BR_COLS - 1) / BR_COLS, b->count),
                       dim3(BR_GROUPS * BR_COLS), 0, st, b->d_items,
                       b->partials, b->d_state, b->d_out);
    hipLaunchKernelGGL(k_batch_refine, dim3(VGX_MAX_DIM, b->count), dim3(64), 0, st, b->d_items, b->d_state);
  }
  VGX_HIP(hipGetLastError());
  return VGX_OK;
}

// Block size of the persistent kernel, the columns of its LDS histograms, and
// a grid of as many workgroups as can be resident at once (the kernel's
// occupancy at that block size): more would only start once the tile queue is
// empty.
vgx_status set_block(vgx_batch* b, int block) {
  b->lds = 0;
  for (BatchItem& it : b->items) {
    it.shift = hist_shift(it.dim, it.nb, block);
    b->lds = std::max(b->lds, (sizeof(double) * it.dim * it.nb) << it.shift);
  }
  int per_cu = 0;
  const void* k = b->odd ? reinterpret_cast<const void*>(&k_batch<true>) : reinterpret_cast<const void*>(&k_batch<false>);
  VGX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, block, b->lds));
  b->block = block;
  b->grid = device_cus() * (per_cu > 0 ? per_cu : 1);
  return VGX_OK;
}

// Time the persistent kernel alone (grids untouched, records untouched) for
// candidate tile and block sizes; keep the fastest.
vgx_status autotune(vgx_batch* b, int fixed_tile, int fixed_block) {
  const int tiles[] = {2048, 4096, 8192, 16384, 32768};
  const int blocks[] = {128, 256};
  int best_t = fixed_tile > 0 ? fixed_tile : 8192, best_b = fixed_block > 0 ? fixed_block : 256;
  if (fixed_tile > 0 && fixed_block > 0) {
    layout(b, fixed_tile);
    return set_block(b, fixed_block);
  }
  hipEvent_t e0, e1;
  VGX_HIP(hipEventCreate(&e0));
  VGX_HIP(hipEventCreate(&e1));
  float best = 1e30f;
  for (int ti : tiles) {
    if (fixed_tile > 0 && ti != fixed_tile) continue;
    for (int bl : blocks) {
      if (fixed_block > 0 && bl != fixed_block) continue;
      layout(b, ti);
      VGX_TRY(set_block(b, bl));
      VGX_TRY(upload_items(b, b->stream));
      float ms_best = 1e30f;
      for (int rep = 0; rep < 3; ++rep) {
        VGX_HIP(hipEventRecord(e0, b->stream));
        VGX_TRY(enqueue_iteration(b, b->stream, false));
        VGX_HIP(hipEventRecord(e1, b->stream));
        VGX_HIP(hipEventSynchronize(e1));
        float ms = 0.f;
        VGX_HIP(hipEventElapsedTime(&ms, e0, e1));
        ms_best = ms < ms_best ? ms : ms_best;
      }
      if (ms_best < best) { best = ms_best; best_t = ti; best_b = bl; }
    }
  }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  layout(b, best_t);
  return set_block(b, best_b);
}

}  // namespace

// Waits for what a context's own stream still has to do on its grid,
// histogram and records, before the batch's stream touches them.
static vgx_status join_stream(const vgx_batch* b, vgx_vegas* c) {
  if (!c->tail || c->stream == b->stream) return VGX_OK;
  VGX_HIP(hipStreamSynchronize(c->stream));
  c->tail = false;
  return VGX_OK;
}

extern "C" vgx_status batch_create(vgx_vegas* const* ctxs, int32_t count, const int64_t* n_samples, int32_t tile,
                                   int32_t block, void* stream, vgx_batch** out) {
  VGX_CHECK(out && ctxs && n_samples, "batch_create: null argument");
  *out = nullptr;
  VGX_CHECK(count >= 1 && count <= 65535, "batch_create: count out of 1..65535");
  VGX_CHECK(tile == 0 || (tile >= 256 && tile <= (1 << 24)), "batch_create: tile out of 256..2^24 (0 = autotune)");
  VGX_CHECK(block == 0 || block == 64 || block == 128 || block == 256, "batch_create: block must be 64/128/256 (0 = autotune)");
  int dev = 0;
  hipGetDevice(&dev);
  for (int k = 0; k < count; ++k) {
    VGX_CHECK(ctxs[k], "batch_create: null context %d", k);
    VGX_CHECK(ctxs[k]->kind != VGX_TTBAR && ctxs[k]->kind != VGX_DRELLYAN && ctxs[k]->kind != VGX_SINGLETOP,
              "batch_create: context %d has a PDF integrand (not batchable)", k);
    VGX_CHECK(ctxs[k]->device == dev, "batch_create: context %d is on another device", k);
    VGX_CHECK(n_samples[k] >= 2, "batch_create: n_samples[%d] < 2", k);
    for (int q = 0; q < k; ++q) VGX_CHECK(ctxs[q] != ctxs[k], "batch_create: context %d listed twice", k);
  }
  vgx_batch* b = new vgx_batch();
  b->device = dev;
  b->stream = stream ? (hipStream_t)stream : ctxs[0]->stream;
  b->count = count;
  b->ctx.assign(ctxs, ctxs + count);
  b->n.assign(n_samples, n_samples + count);
  b->items.resize(count);
  for (int k = 0; k < count; ++k) {
    const vgx_vegas* c = ctxs[k];
    BatchItem it{};
    it.kind = c->kind;
    it.prec = c->prec;
    it.dim = c->dim;
    it.nb = c->nb;
    it.sid = c->stream_id;
    it.k0 = (uint32_t)c->seed;
    it.k1 = (uint32_t)(c->seed >> 32);
    it.pstride = 4 + c->dim * c->nb;
    it.n = n_samples[k];
    it.alpha = c->alpha;
    it.edges = c->edges;
    it.bins = c->bins;
    it.hist = c->hist;
    it.rec = c->rec;
    it.comb = c->comb;
    it.prm = c->prm;
    b->items[k] = it;
    b->odd |= (it.nb & 1) != 0;
    b->max_cols = it.pstride > b->max_cols ? it.pstride : b->max_cols;
  }
  vgx_status s = VGX_OK;
  do {
    b->part_cap = partial_doubles(b, tile > 0 ? tile : 2048);
    if ((s = dev_alloc((void**)&b->partials, sizeof(double) * b->part_cap)) != VGX_OK) break;
    if ((s = dev_alloc((void**)&b->d_items, sizeof(BatchItem) * count)) != VGX_OK) break;
    if ((s = dev_alloc((void**)&b->d_state, state_bytes(count))) != VGX_OK) break;
    if ((s = dev_alloc((void**)&b->d_out, sizeof(IterRecord) * count)) != VGX_OK) break;
    if ((s = host_alloc((void**)&b->pinned, sizeof(IterRecord) * count)) != VGX_OK) break;
    if ((s = host_alloc((void**)&b->pinned_state, state_bytes(count))) != VGX_OK) break;
  } while (0);
  if (s != VGX_OK) { batch_destroy(b); return s; }
  hipError_t e = hipMemsetAsync(b->d_state, 0, state_bytes(count), b->stream);
  if (e != hipSuccess) { s = hip_fail(e, "batch_create", __FILE__, __LINE__); batch_destroy(b); return s; }
  for (int k = 0; k < count && s == VGX_OK; ++k) s = join_stream(b, ctxs[k]);  // the tuning reads the grids
  if (s == VGX_OK) s = autotune(b, tile, block);
  if (s == VGX_OK) s = upload_items(b, b->stream);
  if (s == VGX_OK) {
    e = hipStreamSynchronize(b->stream);
    if (e != hipSuccess) s = hip_fail(e, "batch_create autotune", __FILE__, __LINE__);
  }
  // capture one iteration into a graph on a private stream
  if (s == VGX_OK) {
    e = hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      vgx_status cs = enqueue_iteration(b, b->cap, true);
      hipError_t e2 = hipStreamEndCapture(b->cap, &b->graph);
      if (cs != VGX_OK) s = cs;
      else if (e2 != hipSuccess) e = e2;
    }
    if (s == VGX_OK && e == hipSuccess) e = hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0);
    if (s == VGX_OK && e != hipSuccess) s = hip_fail(e, "batch_create graph capture", __FILE__, __LINE__);
  }
  if (s != VGX_OK) { batch_destroy(b); return s; }
  *out = b;
  return VGX_OK;
}

extern "C" vgx_status batch_iterate(vgx_batch* b, int32_t iteration, vgx_iter_result* out) {
  VGX_CHECK(b, "batch_iterate: null batch");
  // per-iteration inputs in one copy: the iteration number and each
  // integral's record slot (its context's count of stored records)
  int* krec = batch_krec(b->pinned_state);
  for (int k = 0; k < b->count; ++k) {
    if (b->ctx[k]->n_rec >= MAX_RECORDS) { set_error("batch_iterate: context %d has too many records", k); return VGX_ESTATE; }
    VGX_TRY(vegas_flush_pending(b->ctx[k]));
    VGX_TRY(join_stream(b, b->ctx[k]));
    krec[k] = b->ctx[k]->n_rec;
  }
  b->pinned_state->tile_counter = 0;
  b->pinned_state->iteration = iteration;
  b->pinned_state->pad = 0;
  VGX_HIP(hipMemcpyAsync(b->d_state, b->pinned_state, state_bytes(b->count), hipMemcpyHostToDevice, b->stream));
  VGX_HIP(hipGraphLaunch(b->exec, b->stream));
  VGX_HIP(hipMemcpyAsync(b->pinned, b->d_out, sizeof(IterRecord) * b->count, hipMemcpyDeviceToHost, b->stream));
  VGX_HIP(hipStreamSynchronize(b->stream));
  vgx_status s = VGX_OK;
  for (int k = 0; k < b->count; ++k) {
    b->ctx[k]->n_rec++;
    b->ctx[k]->comb_fresh = false;
    b->ctx[k]->rec_host = false;
    b->ctx[k]->have_hist = true;
    const IterRecord& r = b->pinned[k];
    if (out) {
      out[k].mean = r.mean;
      out[k].var = r.var;
      out[k].s1 = r.s1;
      out[k].s2 = r.s2;
      out[k].n = r.n;
    }
    if (!r.finite && s == VGX_OK) {
      set_error("batch_iterate: integral %d gave a non-finite estimate (excluded)", k);
      s = VGX_ENUMERIC;
    }
  }
  return s;
}

extern "C" vgx_status batch_config(vgx_batch* b, int32_t* tile, int32_t* block) {
  VGX_CHECK(b && tile && block, "batch_config: null argument");
  *tile = b->tile;
  *block = b->block;
  return VGX_OK;
}

extern "C" void batch_destroy(vgx_batch* b) {
  if (!b) return;
  if (b->stream) hipStreamSynchronize(b->stream);
  if (b->exec) hipGraphExecDestroy(b->exec);
  if (b->graph) hipGraphDestroy(b->graph);
  if (b->cap) hipStreamDestroy(b->cap);
  hipFree(b->partials);
  hipFree(b->d_items);
  hipFree(b->d_state);
  hipFree(b->d_out);
  if (b->pinned) hipHostFree(b->pinned);
  if (b->pinned_state) hipHostFree(b->pinned_state);
  delete b;
}
