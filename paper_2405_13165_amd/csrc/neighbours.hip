// Neighbourhoods S_i of Eq. (Nbd) by cell lists over Morton-ordered cells.
//
// Pipeline (one stream, one host read-back of sizes):
//   bbox/validate -> grid of each particle (model, support level) and its
//   cell key + per-cell counts (atomics) -> scan -> scatter into cell order
//   -> lists of units of cells and of search items -> finer Morton order inside
//   them and records in cell order -> search, count pass -> scan
//   -> fill pass -> per-row sort -> (several support levels: a second cell
//   pass over each model's finest grid, a model-wide Morton order) ->
//   grouping of particles by (model, neighbour-count band) for the batched
//   stencil kernels -> neighbour tiles.
// Each model has grids for up to four support levels (caps hmax, hmax/2,
// ...); a cell of a grid is a cube of edge slightly above its cap, and a row
// cell searches, in every grid of the requested models, the cells within
// (h_row + cap)/2 of its particles.
#include <algorithm>
#include <cstring>

#include "internal.h"

namespace {

constexpr int kBlock = 256;
constexpr int kMaxRow = 2048;

// -------------------------------------------------------------- reductions
// The butterfly steps move lanes without the LDS crossbar: DPP within rows of
// 16, then the swaps of rows and half waves, which give both values at once.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int64_t b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((int64_t)hi << 32) | (uint32_t)lo);
}
__device__ __forceinline__ double f64_of(unsigned lo, unsigned hi) {
  return __longlong_as_double(((int64_t)hi << 32) | lo);
}
template <bool MIN>
__device__ __forceinline__ double pick(double a, double b) { return MIN ? fmin(a, b) : fmax(a, b); }
// min / max of the first LANES (32 or 64) lanes, in each of them
template <bool MIN, int LANES>
__device__ __forceinline__ double lanes_pick(double v) {
  v = pick<MIN>(v, dpp_f64<0xB1>(v));   // quad_perm [1, 0, 3, 2]
  v = pick<MIN>(v, dpp_f64<0x4E>(v));   // quad_perm [2, 3, 0, 1]
  v = pick<MIN>(v, dpp_f64<0x141>(v));  // row_half_mirror
  v = pick<MIN>(v, dpp_f64<0x140>(v));  // row_mirror
  {
    const int64_t b = __double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    v = pick<MIN>(f64_of(l[0], h[0]), f64_of(l[1], h[1]));
  }
  if constexpr (LANES == 64) {
    const int64_t b = __double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    v = pick<MIN>(f64_of(l[0], h[0]), f64_of(l[1], h[1]));
  }
  return v;
}
__device__ inline int wave_sum_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// inclusive scans over the wave by lane moves within rows of 16 and row broadcasts
__device__ inline int wave_scan_add(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ inline int wave_scan_max(int v) {  // of values >= 0
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false));
  return v;
}

// orders the LDS traffic of the lanes of one wave
__device__ inline void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// per model: lo[3], hi[3], hmax, hmin (8 doubles) -> 16 doubles + invalid count
constexpr int kBoxVals = 16;
// value k of the box is reduced with min (else max)
__host__ __device__ inline bool box_is_min(int k) { return (k % 8) < 3 || (k % 8) == 7; }

constexpr int kBboxThreads = 1024;
__global__ void __launch_bounds__(kBboxThreads) k_bbox(const double *__restrict__ x, const double *__restrict__ y,
                                                 const double *__restrict__ z, const double *__restrict__ h,
                                                 const int8_t *__restrict__ model, int64_t n,
                                                 double *__restrict__ part, int *__restrict__ bad_part) {
  double v[kBoxVals];
  for (int m = 0; m < 2; ++m) {
    for (int d = 0; d < 3; ++d) { v[m * 8 + d] = INFINITY; v[m * 8 + 3 + d] = -INFINITY; }
    v[m * 8 + 6] = 0.0;
    v[m * 8 + 7] = INFINITY;
  }
  int bad = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    double p[3] = {x[i], y[i], z[i]};
    double hi = h[i];
    int m = model[i];
    bool ok = (m == 0 || m == 1) && isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]) && isfinite(hi) && hi > 0.0;
    if (!ok) { ++bad; continue; }
    for (int mm = 0; mm < 2; ++mm) {
      if (mm != m) continue;
      for (int d = 0; d < 3; ++d) {
        v[mm * 8 + d] = fmin(v[mm * 8 + d], p[d]);
        v[mm * 8 + 3 + d] = fmax(v[mm * 8 + 3 + d], p[d]);
      }
      v[mm * 8 + 6] = fmax(v[mm * 8 + 6], hi);
      v[mm * 8 + 7] = fmin(v[mm * 8 + 7], hi);
    }
  }
  __shared__ double sh[kBboxThreads / 64][kBoxVals];
  __shared__ int shb[kBboxThreads / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    if (__ballot(v[8 * m + 6] > 0.0)) {  // (most waves meet one model only)
#pragma unroll
      for (int k = 8 * m; k < 8 * m + 8; ++k) v[k] = box_is_min(k) ? lanes_pick<true, 64>(v[k]) : lanes_pick<false, 64>(v[k]);
    }
#pragma unroll
    for (int k = 8 * m; k < 8 * m + 8; ++k)
      if (lane == 0) sh[wid][k] = v[k];
  }
  int bs = wave_sum_i(bad);
  if (lane == 0) shb[wid] = bs;
  __syncthreads();
  if (threadIdx.x < kBoxVals) {
    int k = threadIdx.x;
    double r = sh[0][k];
    for (int w = 1; w < kBboxThreads / 64; ++w) r = box_is_min(k) ? fmin(r, sh[w][k]) : fmax(r, sh[w][k]);
    part[(int64_t)blockIdx.x * kBoxVals + k] = r;
  }
  if (threadIdx.x == 0) {
    int b = 0;
    for (int w = 0; w < kBboxThreads / 64; ++w) b += shb[w];
    bad_part[blockIdx.x] = b;
  }
}

// Sizes that the host needs are written by the device straight into the
// context's pinned host buffer: a copy of a few bytes would be a launch and a
// gap of its own.  host[k] = a[k] (k < na), host[na] = *last.
__global__ void k_publish(const int32_t *__restrict__ a, int na, const int64_t *__restrict__ last,
                          int64_t *__restrict__ host) {
  const int k = threadIdx.x;
  if (k < na) host[k] = a[k];
  if (k == na) host[na] = *last;
}

// one block: thread t combines value t % 16 of the block partials t / 16, t / 16 + 16, ...; out and
// bad_out lie in pinned host memory
constexpr int kBboxFin = 256;
constexpr int kBboxBlocks = 256;  // blocks of the first pass, at most
__global__ void __launch_bounds__(kBboxFin) k_bbox_final(const double *__restrict__ part,
                                                         const int *__restrict__ bad_part, int nblk,
                                                         double *__restrict__ out, int *__restrict__ bad_out) {
  constexpr int kParts = kBboxFin / kBoxVals;
  __shared__ double sh[kParts][kBoxVals];
  __shared__ int shb[kBboxFin / 64];
  const int k = threadIdx.x % kBoxVals, q = threadIdx.x / kBoxVals;
  const bool lo = box_is_min(k);
  double r = lo ? INFINITY : -INFINITY;
#pragma unroll 8
  for (int b = q; b < nblk; b += kParts) {
    const double t = part[(int64_t)b * kBoxVals + k];
    r = lo ? fmin(r, t) : fmax(r, t);
  }
  sh[q][k] = r;
  int sum = 0;
  for (int b = threadIdx.x; b < nblk; b += kBboxFin) sum += bad_part[b];
  sum = wave_sum_i(sum);
  if ((threadIdx.x & 63) == 0) shb[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (q == 0) {
    for (int w = 1; w < kParts; ++w) r = lo ? fmin(r, sh[w][k]) : fmax(r, sh[w][k]);
    out[k] = r;
  }
  if (threadIdx.x == 0) {
    int all = 0;
    for (int w = 0; w < kBboxFin / 64; ++w) all += shb[w];
    *bad_out = all;
  }
}

// -------------------------------------------------------------- grid
// One cell grid per (model, level): level l of model m holds the particles
// with hmax_m 2^-(l+1) < h <= hmax_m 2^-l (the last level takes the rest),
// so a cell's edge follows the supports of its own particles.  A row cell
// searches, in each target grid, the cells within (h_row + hcap_target)/2 of
// its particles: uneven supports and dense fine regions do not inflate the
// candidate sets of the others.
constexpr int kMaxLevels = 4;
constexpr int kMaxSlots = 2 * kMaxLevels;
constexpr int kMaxAxis = 1000000;  // cells per axis, at most: the last one also holds what lies beyond it
struct Grid {
  int nslots;
  int slot0[3];              // slots of model m: [slot0[m], slot0[m + 1])
  double lo[kMaxSlots][3];
  double edge[kMaxSlots], inv_edge[kMaxSlots];
  double hcap[kMaxSlots];    // every particle of the slot has h <= hcap (0: model absent)
  int dim[kMaxSlots][3];
  int bits[kMaxSlots][3];
  int64_t base[kMaxSlots];   // key offset of each slot's cells
  int64_t nkeys;
};

__host__ __device__ inline int slot_of(const Grid &g, int m, double h) {
  int s = g.slot0[m];
  while (s + 1 < g.slot0[m + 1] && h <= g.hcap[s + 1]) ++s;
  return s;
}

__device__ inline int cell_of(double v, double lo, double inv_edge, int dim) {
  double t = floor((v - lo) * inv_edge);
  int c = (t < 0.0) ? 0 : (t >= (double)dim ? dim - 1 : (int)t);
  return c;
}

// Morton interleave with possibly different bit counts per axis
__device__ inline int64_t morton(int cx, int cy, int cz, int bx, int by, int bz) {
  int64_t key = 0;
  int pos = 0;
  int mb = max(bx, max(by, bz));
  for (int b = 0; b < mb; ++b) {
    if (b < bx) key |= (int64_t)((cx >> b) & 1) << pos++;
    if (b < by) key |= (int64_t)((cy >> b) & 1) << pos++;
    if (b < bz) key |= (int64_t)((cz >> b) & 1) << pos++;
  }
  return key;
}


// the same for keys below 2^31
__device__ inline int32_t morton32(int cx, int cy, int cz, int bx, int by, int bz) {
  uint32_t key = 0;
  int pos = 0;
  const int mb = max(bx, max(by, bz));
  for (int b = 0; b < mb; ++b) {
    if (b < bx) key |= (((uint32_t)cx >> b) & 1u) << pos++;
    if (b < by) key |= (((uint32_t)cy >> b) & 1u) << pos++;
    if (b < bz) key |= (((uint32_t)cz >> b) & 1u) << pos++;
  }
  return (int32_t)key;
}

__global__ void __launch_bounds__(kBlock) k_fill_i32(int32_t *a, int64_t n, int32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    a[i] = v;
}

// counts[0 .. n) and small[0 .. 32) cleared
__global__ void __launch_bounds__(kBlock) k_clear(int32_t *__restrict__ counts, int64_t n, int32_t *__restrict__ small) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) counts[i] = 0;
  if (i < 32 && small) small[i] = 0;
}

// key[i]: cell of particle i; counts[k]: particles per cell
__global__ void __launch_bounds__(kBlock) k_keys(const double *__restrict__ x, const double *__restrict__ y,
                                                 const double *__restrict__ z, const double *__restrict__ h,
                                                 const int8_t *__restrict__ model, int64_t n, Grid g,
                                                 int32_t *__restrict__ key, int32_t *__restrict__ slot,
                                                 int32_t *__restrict__ counts) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63;
  int32_t k = -1;
  if (i < n) {
    const int s = slot_of(g, model[i], h[i]);
    const int cx = cell_of(x[i], g.lo[s][0], g.inv_edge[s], g.dim[s][0]);
    const int cy = cell_of(y[i], g.lo[s][1], g.inv_edge[s], g.dim[s][1]);
    const int cz = cell_of(z[i], g.lo[s][2], g.inv_edge[s], g.dim[s][2]);
    k = (int32_t)g.base[s] + morton32(cx, cy, cz, g.bits[s][0], g.bits[s][1], g.bits[s][2]);
    key[i] = k;
  }
  // Slot within the cell.  Particles numbered one after another often share a
  // cell, and atomics on one counter serialise, so a run of lanes with one key
  // shares one atomic: its first lane reserves the run's length.  (The order
  // within a cell is re-sorted later; only the set of slots 0..count-1 matters.
  // Runs, not all the lanes of a key: with particles in no order, as the jet's
  // film, a wave holds 64 keys and collecting each key's lanes took 64 rounds:
  // 126 -> 72 us on the jet, 27 -> 11 us on the mixed cloud.)
  const int32_t before = __shfl_up(k, 1, 64);
  const bool first = lane == 0 || k != before;
  const unsigned long long heads = __ballot(first);
  const int mine = 63 - __builtin_clzll(heads & (~0ull >> (63 - lane)));  // my run's first lane
  const unsigned long long after = lane == 63 ? 0ull : heads >> (lane + 1);
  int32_t base = 0;
  if (first && k >= 0) base = atomicAdd(&counts[k], after ? __builtin_ctzll(after) + 1 : 64 - lane);
  base = __shfl(base, mine, 64);
  if (i < n) slot[i] = base + lane - mine;
}

// Search items: the rows of one cell, or of an aligned Morton block of 2, 4 or
// 8 cells where the grid's cells hold few particles (film cells hold 9; the
// smallest such block with at least kItemFill particles by the grid's mean over
// its bounding box), in equal parts of at most `most` rows.  An item's rows are
// one range of the cell order (a multiple of four but for a unit's last, as the
// search takes rows in fours), and its candidates are read once for all of
// them.  items[k] = (first row, rows, grid); their order is left to the run (no
// result depends on it).  Also the units of the in-cell order, (first row, rows,
// grid, cells - 1): such a block, or each of its cells where it holds more than
// kCellSort particles; those of more than kUnitSmall rows in a list of their own as
// (first row, rows, grid, piece), a cell of more than kCellSort once for each piece
// of kUnitSmall rows.  And the number of particles of each grid.
constexpr int kUnitSmall = 256;
constexpr int kCellSort = 2048;
inline int64_t big_units(int64_t n) { return n / kUnitSmall + n / kCellSort + 1; }  // at most
constexpr int kItemFill = 20;
constexpr int kItemBits = 3;
struct CellLists {
  int4 *items, *units, *big;             // (items may be NULL: not wanted)
  int32_t *nitems, *nunits, *nbig;
  int32_t *slot_count;
};
// (a block's units and items take their places by one atomic each: a few
// addresses serve the whole grid)
constexpr int kItemsBlock = 1024;
__global__ void __launch_bounds__(kItemsBlock) k_items(const int32_t *__restrict__ cell_start, Grid g, int most,
                                                       CellLists out) {
  __shared__ int s_units[kItemsBlock / 64], s_items[kItemsBlock / 64], s_base[2];
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int a = 0, b = 0, s = 0, cells = 1;
  if (k < g.nkeys) {
    while (s + 1 < g.nslots && k >= g.base[s + 1]) ++s;
    const int64_t end = (s + 1 < g.nslots) ? g.base[s + 1] : g.nkeys;
    const int count = cell_start[end] - cell_start[g.base[s]];
    if (k == g.base[s]) out.slot_count[s] = count;
    const double mean = (double)count / ((double)g.dim[s][0] * g.dim[s][1] * g.dim[s][2]);
    int sh = 0;
    while (sh < kItemBits && mean * (double)(1 << sh) < (double)kItemFill && ((int64_t)2 << sh) <= end - g.base[s]) ++sh;
    if (((k - g.base[s]) & ((1 << sh) - 1)) == 0) {
      a = cell_start[k];
      b = cell_start[k + (1 << sh)];
      cells = 1 << sh;
    }
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, len = b - a;
  const bool small = len > 0 && len <= kUnitSmall;
  const int parts = out.items ? (len + most - 1) / most : 0;
  const uint64_t m = __ballot(small);
  const int inc = wave_scan_add(parts);
  if (lane == 63) {
    s_units[w] = (int)__popcll(m);
    s_items[w] = inc;
  }
  __syncthreads();
  int ub = 0, ib = 0, ut = 0, itot = 0;
  for (int q = 0; q < kItemsBlock / 64; ++q) {
    if (q < w) { ub += s_units[q]; ib += s_items[q]; }
    ut += s_units[q];
    itot += s_items[q];
  }
  if (threadIdx.x == 0) {
    s_base[0] = ut ? atomicAdd(out.nunits, ut) : 0;
    s_base[1] = itot ? atomicAdd(out.nitems, itot) : 0;
  }
  __syncthreads();
  if (small) {
    out.units[s_base[0] + ub + __popcll(m & ((1ull << lane) - 1ull))] = make_int4(a, len, s, cells - 1);
  } else if (len > 0 && len <= kCellSort) {
    out.big[atomicAdd(out.nbig, 1)] = make_int4(a, len, s, 0);
  } else if (len > 0) {
    for (int c = 0; c < cells; ++c) {
      const int ca = cell_start[k + c], cl = cell_start[k + c + 1] - ca;
      if (cl > kUnitSmall) {
        const int np = cl > kCellSort ? (cl + kUnitSmall - 1) / kUnitSmall : 1, at = atomicAdd(out.nbig, np);
        for (int q = 0; q < np; ++q) out.big[at + q] = make_int4(ca, cl, s, q);
      } else if (cl > 0) {
        out.units[atomicAdd(out.nunits, 1)] = make_int4(ca, cl, s, 0);
      }
    }
  }
  if (parts == 0) return;
  const int at = s_base[1] + ib + inc - parts;
  const int size = ((len + parts - 1) / parts + 3) & ~3;  // <= most
  for (int q = 0, f = a; f < b; ++q, f += size) out.items[at + q] = make_int4(f, min(size, b - f), s, 0);
}

__global__ void __launch_bounds__(kBlock) k_scatter(const int32_t *__restrict__ key, const int32_t *__restrict__ slot,
                                                    const int32_t *__restrict__ cell_start, int64_t n,
                                                    int32_t *__restrict__ order) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  order[cell_start[key[i]] + slot[i]] = (int32_t)i;
}

// Order the particles of each cell by a finer Morton key (kSubBits more bits
// per axis), ties by index, so that runs of the cell order stay spatially
// compact when a cell is much larger than a typical support (uneven h), and
// write the records (x, y, z, h / 2) of the cell order (sp may be NULL).  Units
// of up to kUnitSmall rows: a wave each, the rank of a particle counted over the
// unit's keys in LDS.  Inside a unit the fine keys differ only in the cell's
// place in the unit and the low kSubBits bits per axis, so those bits and the
// particle index, packed in 64 bits, order it exactly.  What bounds it: the
// gathers of the particles' data.  With the records written here (one more pass
// over the particles before) and a 12-bit sub key instead of the 63-bit one,
// sort and records of the mixed cloud take 16 us (55 before), of the 2.0M jet,
// whose film comes in no order, 126 us (447 before).
constexpr int kSubBits = 4;

// low kSubBits bits per axis of the fine Morton key, interleaved
__device__ inline uint32_t fine_sub(double x, double y, double z, const Grid &g, int s) {
  const double f = (double)(1 << kSubBits);
  const double v[3] = {x, y, z};
  uint32_t key = 0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double t = floor((v[d] - g.lo[s][d]) * g.inv_edge[s] * f);
    const double hi = (double)g.dim[s][d] * f - 1.0;
    const uint32_t c = (uint32_t)(int)(t < 0.0 ? 0.0 : (t > hi ? hi : t));
#pragma unroll
    for (int b = 0; b < kSubBits; ++b) key |= ((c >> b) & 1u) << (3 * b + d);
  }
  return key;
}

constexpr int kCellSortWaves = 4;
__global__ void __launch_bounds__(64 * kCellSortWaves) k_cell_sort_small(
    const int4 *__restrict__ units, const int32_t *__restrict__ nunits, const int32_t *__restrict__ key,
    const double *__restrict__ x, const double *__restrict__ y, const double *__restrict__ z,
    const double *__restrict__ h, Grid g, const int32_t *__restrict__ raw, int32_t *__restrict__ order,
    double4 *__restrict__ sp) {
  constexpr int NV = kUnitSmall / 64;
  __shared__ __attribute__((aligned(16))) uint64_t s_key[kCellSortWaves][kUnitSmall];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nu = *nunits, stride = gridDim.x * kCellSortWaves;
  for (int u = blockIdx.x * kCellSortWaves + w; u < nu; u += stride) {
    const int4 un = units[u];
    const int b = un.x, len = un.y, s = un.z;
    int32_t id[NV];
    double4 rec[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int t = lane + 64 * q;
      if (64 * q >= len) continue;
      id[q] = 0;
      uint64_t k = ~0ull;
      if (t < len) {
        const int32_t i = raw[b + t];
        id[q] = i;
        rec[q] = make_double4(x[i], y[i], z[i], 0.5 * h[i]);
        const uint32_t cell = (uint32_t)(key[i] - (int32_t)g.base[s]) & (uint32_t)un.w;
        const uint32_t sub = (cell << (3 * kSubBits)) | fine_sub(rec[q].x, rec[q].y, rec[q].z, g, s);
        k = ((uint64_t)sub << 32) | (uint32_t)i;
      }
      s_key[w][t] = k;
    }
    wave_fence();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int t = lane + 64 * q;
      if (64 * q >= len) continue;
      const uint64_t mine = s_key[w][t];
      int rank = 0;
      for (int c = 0; c < len; c += 2) {  // (an odd count's last pair ends in a pad, which is not smaller)
        const ulonglong2 kk = *reinterpret_cast<const ulonglong2 *>(&s_key[w][c]);
        rank += (kk.x < mine) + (kk.y < mine);
      }
      if (t < len) {
        order[b + rank] = id[q];
        if (sp) sp[b + rank] = rec[q];
      }
    }
    wave_fence();
  }
}

// Larger units, a block each, by a bitonic network in LDS over the whole fine
// key.  A cell of more than kCellSort particles takes a block per kUnitSmall of
// them, each of which counts how many of the cell's come before its own (2^12
// sub-keys, packed with the index as above): cells so full cost their pairs in the
// search too (8,000 particles in one cell: 115 us here, 360 there), and a launch
// that would merge sorted pieces takes 4 us in every build.  The neighbour sets do not depend on this order, but the tiles and so
// the order of the adjoints' sums do: it is the same for every build.
__device__ inline uint64_t fine_key(double x, double y, double z, const Grid &g, int s) {
  const double f = (double)(1 << kSubBits);
  int c[3];
  const double v[3] = {x, y, z};
  for (int d = 0; d < 3; ++d) {
    const double t = floor((v[d] - g.lo[s][d]) * g.inv_edge[s] * f);
    const double hi = (double)g.dim[s][d] * f - 1.0;
    c[d] = (int)(t < 0.0 ? 0.0 : (t > hi ? hi : t));
  }
  uint64_t key = 0;
  int pos = 0;
  for (int b = 0; b < 21; ++b)
    for (int d = 0; d < 3; ++d) key |= (uint64_t)((c[d] >> b) & 1) << pos++;
  return key;
}

static_assert(kBlock == kUnitSmall, "a thread per particle of a piece");
__global__ void __launch_bounds__(kBlock) k_cell_sort_big(const int4 *__restrict__ units, const int32_t *__restrict__ nunits,
                                                          const double *__restrict__ x, const double *__restrict__ y,
                                                          const double *__restrict__ z, const double *__restrict__ h,
                                                          Grid g, const int32_t *__restrict__ raw,
                                                          int32_t *__restrict__ order, double4 *__restrict__ sp) {
  __shared__ __attribute__((aligned(16))) uint64_t kk[kCellSort];
  __shared__ int32_t id[kCellSort];
  const int nu = *nunits;
  for (int u = blockIdx.x; u < nu; u += gridDim.x) {
    const int4 un = units[u];
    const int b = un.x, len = un.y, s = un.z;
    if (len > kCellSort) {
      const int t = un.w * kUnitSmall + (int)threadIdx.x;  // this thread's particle of the cell
      auto packed = [&](int32_t i) { return ((uint64_t)fine_sub(x[i], y[i], z[i], g, s) << 32) | (uint32_t)i; };
      const int32_t mine = t < len ? raw[b + t] : 0;
      const uint64_t key = packed(mine);
      int rank = 0;
      for (int c = 0; c < len; c += kCellSort) {
        const int m = min(kCellSort, len - c);
        for (int q = threadIdx.x; q < kCellSort; q += kBlock) kk[q] = q < m ? packed(raw[b + c + q]) : ~0ull;
        __syncthreads();
#pragma unroll 4
        for (int q = 0; q < m; q += 2) {  // (an odd count's last pair ends in a pad, which is not smaller)
          const ulonglong2 v = *reinterpret_cast<const ulonglong2 *>(&kk[q]);
          rank += (v.x < key) + (v.y < key);
        }
        __syncthreads();
      }
      if (t < len) {
        order[b + rank] = mine;
        if (sp) sp[b + rank] = make_double4(x[mine], y[mine], z[mine], 0.5 * h[mine]);
      }
      continue;
    }
    int P = 1;
    while (P < len) P <<= 1;
    for (int t = threadIdx.x; t < P; t += kBlock) {
      if (t < len) {
        const int32_t i = raw[b + t];
        kk[t] = fine_key(x[i], y[i], z[i], g, s);
        id[t] = i;
      } else {
        kk[t] = ~0ull;
        id[t] = 0x7fffffff;
      }
    }
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1) {
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int t = threadIdx.x; t < P; t += kBlock) {
          const int o = t ^ j;
          if (o > t) {
            const uint64_t a = kk[t], e = kk[o];
            const int32_t ia = id[t], ie = id[o];
            // ties (same sub-cell) by particle index: the order is deterministic
            const bool gt = (a > e) || (a == e && ia > ie);
            if (gt == ((t & k) == 0)) { kk[t] = e; kk[o] = a; id[t] = ie; id[o] = ia; }
          }
        }
        __syncthreads();
      }
    }
    for (int t = threadIdx.x; t < len; t += kBlock) {
      const int32_t i = id[t];
      order[b + t] = i;
      if (sp) sp[b + t] = make_double4(x[i], y[i], z[i], 0.5 * h[i]);
    }
    __syncthreads();
  }
}

// Eq. (Nbd) predicate, evaluated as written without contraction so that the
// decision is reproducible across implementations.  The records hold half
// supports: h_i / 2 + h_j / 2 is 0.5 (h_i + h_j) to the bit (halving is exact).
__device__ inline bool in_support(double4 a, double4 b) {
#pragma clang fp contract(off)
  double dx = b.x - a.x;
  double dy = b.y - a.y;
  double dz = b.z - a.z;
  double d2 = (dx * dx + dy * dy) + dz * dz;
  double r = a.w + b.w;
  return d2 <= r * r;
}

// Neighbour search, one wave per search item (up to kItemRows rows that follow
// one another in the cell order).
//  1. The bounding box and the largest support of the item's rows.
//  2. For each target grid (the row model's grids, or all grids for cross-model
//     sets) the cells within R = (max h of the rows + hcap of the grid)/2 of
//     the box are taken 64 at a time and their particles numbered through a
//     prefix sum of the cell ranges.  Each candidate is tested against the box
//     with its own support; those that may reach a row go to a ring in LDS.
//  3. Whenever the ring holds 64 candidates (and at the end), they are tested,
//     one per lane, against each row, the rows' records in scalar registers,
//     four rows at a time; a ballot gives a row's hits.
// MODE 0: count (cnt[i] = |S_i|, group histogram, max row); MODE 1: fill col
// (rows are sorted afterwards); MODE 2: count, and write each row's first sw
// hits to stage[i * sw ...] (sw, the stage width, 512 or 256 hits by the memory
// it takes), which saves the fill pass when no row is longer; with `stage` the
// fill pass writes only the longer rows.  Hits go out
// through buffer stores whose range is the row's room: the hardware drops the
// lanes without a hit (given an offset past any range) and the hits beyond it.
// Particles i >= n_rows (ghost particles) appear in the rows of others but
// their own row holds only i.
//
// What bounds it: VALU issue and the latency of a wave's serial chain.  A 3D
// row of the mixed cloud has ~730 candidates in its 27 cells, a row of the
// uneven jet ~2,700, of which ~100 and ~80 are hits; the box leaves ~450 and
// ~500.  A test of 64 candidates takes 11 FP64 instructions and 7 more for the
// output; VALU issue is 60-75% of the launch.  Against the predecessor (one wave
// per cell, every candidate against every row, ~40 instructions per 64 tests,
// most of them for the output): mixed cloud 512 -> 216 us, 2.0M jet 3.93 ->
// 1.68 ms, 25k-particle plate 334 -> 29 us (its few hundred cells left most of
// the chip idle), 916 particles 53 -> 16 us.  Rows per item at most 8 / 16 / 24
// / 32: mixed 266 / 231 / 216 / 238 us, jet 2.11 / 1.76 / 1.68 / 1.63 ms.
constexpr int kSearchBlock = 256;
constexpr int kSearchWaves = kSearchBlock / 64;
constexpr int kSearchBlocksPerCu = 8;
constexpr int kItemRows = 24;
constexpr int kRowPad = 4;              // entries of padding after the records and the order (rows are read in fours)
constexpr int kRing = 128;              // a batch adds at most 64 to at most 63 left over
constexpr int kStageWidths[2] = {512, 256};  // hits per row the count pass may stage, widest first
// Items are dealt to the XCDs in chunks: neighbouring items share candidates
// in one L2, and every XCD gets its share of bulk and film items.
constexpr int kItemChunk = 128;

// the value of v in lane r (r the same in every lane)
__device__ inline int64_t readlane64(int64_t v, int r) {
  return ((int64_t)__builtin_amdgcn_readlane((int)(v >> 32), r) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, r);
}

// a value known to be the same in every lane, moved to scalar registers
__device__ inline double uniform_f64(double v) {
  const int64_t b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((int64_t)hi << 32) | (uint32_t)lo);
}

// min / max over the first 32 lanes of the wave, uniform
static_assert(kItemRows <= 32, "an item's rows lie in the first 32 lanes");
__device__ inline double rows_min(double v) { return uniform_f64(lanes_pick<true, 32>(v)); }
__device__ inline double rows_max(double v) { return uniform_f64(lanes_pick<false, 32>(v)); }

template <int MODE>
__global__ void __launch_bounds__(kSearchBlock) k_search(const int32_t *__restrict__ order,
                                                         const double4 *__restrict__ sp,
                                                         const int32_t *__restrict__ cell_start,
                                                         const int4 *__restrict__ items,
                                                         const int32_t *__restrict__ nitems,
                                                         const int32_t *__restrict__ slot_count,
                                                         int64_t n_rows, Grid g, int cross,
                                                         int32_t *__restrict__ cnt, int32_t *__restrict__ hist,
                                                         int32_t *__restrict__ maxrow,  // [2] per model
                                                         const int64_t *__restrict__ row_ptr,
                                                         int32_t *__restrict__ col, int32_t *__restrict__ stage,
                                                         int sw) {
  __shared__ double2 s_xy[kSearchWaves][kRing], s_zh[kSearchWaves][kRing];  // the ring: positions, half supports,
  __shared__ int32_t s_id[kSearchWaves][kRing];                             // user indices
  __shared__ int32_t s_mark[kSearchWaves][64];
  __shared__ int32_t s_hist[2 * GF_NBAND + 2];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ni = *nitems;
  if (MODE != 1 && tid < 2 * GF_NBAND + 2) s_hist[tid] = 0;
  int hist_local = 0;  // lane b < 2*GF_NBAND: rows counted in bin b (MODE 0)
  int max_local[2] = {0, 0};
  const int nx = gridDim.x % 8 == 0 ? 8 : 1;
  const int xcd = blockIdx.x % nx, G = gridDim.x / nx * kSearchWaves;
  constexpr bool STORE = MODE != 0;
  for (int p = blockIdx.x / nx * kSearchWaves + w;; p += G) {
    const int chunk = p / kItemChunk;
    if ((int64_t)chunk * nx * kItemChunk >= ni) break;  // (every later p is past the end too)
    const int ii = (chunk * nx + xcd) * kItemChunk + p % kItemChunk;
    if (ii >= ni) continue;
    const int4 it = items[ii];
    const int r0 = it.x, nw = it.y;  // rows [r0, r0 + nw), nw <= kItemRows
    const int mrow = it.z < g.slot0[1] ? 0 : 1;
    const int t0 = cross ? 0 : g.slot0[mrow], t1 = cross ? g.nslots : g.slot0[mrow + 1];
    int32_t myi = -1;
    bool ghost = false;
    int64_t myoff = 0;
    int mylen = 0;  // MODE 1: entries of the row this pass writes
    double4 me = make_double4(0.0, 0.0, 0.0, 0.0);
    if (lane < nw) {
      myi = order[r0 + lane];
      me = sp[r0 + lane];
      ghost = myi >= n_rows;
      if (MODE == 1) {
        myoff = row_ptr[myi];
        mylen = (int)(row_ptr[myi + 1] - myoff);
        if (stage && mylen <= sw) mylen = 0;  // staged by the count pass: not written here
        if (ghost && mylen > 0) col[myoff] = myi;
      } else if (MODE == 2) {
        if (ghost) stage[(int64_t)myi * sw] = myi;
      }
    }
    const bool act = lane < nw && !ghost && (MODE != 1 || mylen > 0);
    const unsigned rows = (unsigned)__ballot(act);  // the rows searched
    int run = 0;  // lane r < nw: hits of row r0 + r so far
    if (rows) {
      const double b0[3] = {rows_min(act ? me.x : INFINITY), rows_min(act ? me.y : INFINITY),
                            rows_min(act ? me.z : INFINITY)};
      const double b1[3] = {rows_max(act ? me.x : -INFINITY), rows_max(act ? me.y : -INFINITY),
                            rows_max(act ? me.z : -INFINITY)};
      const double hrow = rows_max(act ? me.w : 0.0);  // half supports throughout
      double bc[3], be[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        bc[d] = uniform_f64(0.5 * (b0[d] + b1[d]));
        be[d] = uniform_f64(fmax(b1[d] - bc[d], bc[d] - b0[d]));
      }
      int head = 0, fill = 0;  // the ring: entries [head, head + fill) mod kRing
      // tests the ring's first min(fill, 64) candidates against the rows
      auto test = [&]() {
        wave_fence();
        const int at = (head + lane) & (kRing - 1);
        const double2 xy = s_xy[w][at], zh = s_zh[w][at];
        const int32_t j = s_id[w][at];
        // (a lane past the fill tests NaN, which no row reaches)
        const double4 q = make_double4(lane < fill ? xy.x : __builtin_nan(""), xy.y, zh.x, zh.y);
#pragma unroll 1
        for (int rq = 0; rq < nw; rq += 4) {
          // (the records and the order are padded: up to three rows past the item's are read, and masked)
          double4 pr[4];
          int32_t ir[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            pr[k] = sp[r0 + rq + k];
            ir[k] = order[r0 + rq + k];
          }
          bool hit[4];
          int pos[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) hit[k] = in_support(pr[k], q);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            uint64_t m = __ballot(hit[k]);
            if (!((rows >> (rq + k)) & 1u)) m = 0;
            const int run_r = __builtin_amdgcn_readlane(run, rq + k);
            pos[k] = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)run_r));
            if (lane == rq + k) run = run_r + __popcll(m);
          }
          if constexpr (STORE) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              int32_t *out;
              int lim;
              if (MODE == 1) {
                out = col + readlane64(myoff, rq + k);
                lim = __builtin_amdgcn_readlane(mylen, rq + k);
              } else {
                out = stage + (int64_t)ir[k] * sw;
                lim = sw;
              }
              const __amdgpu_buffer_rsrc_t rs =
                  __builtin_amdgcn_make_buffer_rsrc(out, 0, ((rows >> (rq + k)) & 1u) ? 4 * lim : 0, 0x00020000);
              __builtin_amdgcn_raw_buffer_store_b32(j, rs, hit[k] ? 4 * pos[k] : -4, 0, 0);
            }
          }
        }
        const int took = min(fill, 64);
        head = (head + took) & (kRing - 1);
        fill -= took;
        wave_fence();
      };
#pragma unroll 1
      for (int ts = t0; ts < t1; ++ts) {
        if (slot_count[ts] == 0) continue;  // an empty grid
        // cells within R of the rows (1e-6 margin against rounding of the cell coordinates)
        const double R = (hrow + 0.5 * g.hcap[ts]) * (1.0 + 1e-6);
        int a0[3], ext[3];
        bool none = false;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const double f0 = floor((b0[d] - R - g.lo[ts][d]) * g.inv_edge[ts]);
          const double f1 = floor((b1[d] + R - g.lo[ts][d]) * g.inv_edge[ts]);
          const double top = (double)(g.dim[ts][d] - 1);
          none = none || f1 < 0.0 || (f0 > top && g.dim[ts][d] < kMaxAxis);
          a0[d] = __builtin_amdgcn_readfirstlane((int)fmin(fmax(f0, 0.0), top));
          ext[d] = __builtin_amdgcn_readfirstlane((int)fmin(f1, top)) - a0[d] + 1;
        }
        if (none) continue;
        const unsigned nbox = (unsigned)ext[0] * ext[1] * ext[2];  // <= g.nkeys
        // (a particle lies in its cell's cube up to the rounding of its cell coordinate, below 1e-9 edges; the cubes are
        // taken from the grid's corner as that coordinate is, so this holds however far the corner is from the origin)
        const double edge = g.edge[ts], Rc = R + 1e-9 * edge;
#pragma unroll 1
        for (unsigned kb = 0; kb < nbox; kb += 64) {
          int len = 0, rb = 0;
          const unsigned kc = kb + lane;
          if (kc < nbox) {
            const unsigned q = kc / ext[0], qq = q / ext[1];
            const int cx = a0[0] + (int)(kc - q * ext[0]), cy = a0[1] + (int)(q - qq * ext[1]), cz = a0[2] + (int)qq;
            // distance of the cell's cube to the box; the last cell of an axis also holds what lies beyond it
            const int cc[3] = {cx, cy, cz};
            double u2 = 0.0;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
              const double lo = fma((double)cc[d], edge, g.lo[ts][d] - bc[d]);  // the cube's lower face, from the box's centre
              const double below = lo - be[d], above = cc[d] == g.dim[ts][d] - 1 ? 0.0 : -(lo + edge) - be[d];
              const double u = fmax(fmax(below, above), 0.0);
              u2 = fma(u, u, u2);
            }
            if (u2 <= Rc * Rc) {
              const int32_t key = (int32_t)g.base[ts] + morton32(cx, cy, cz, g.bits[ts][0], g.bits[ts][1], g.bits[ts][2]);
              rb = cell_start[key];
              len = cell_start[key + 1] - rb;
            }
          }
          const int pref = wave_scan_add(len) - len;  // candidates before this lane's cell
          const int C = __builtin_amdgcn_readlane(pref + len, 63);
          const int delta = rb - pref;                // sorted position of candidate c of this cell: c + delta
          int carry = 0;                              // 1 + the cell that the last candidate so far falls in
          // the sorted position of candidate cb + lane: each cell marks its first candidate, and the
          // largest mark up to a candidate is its cell
          auto cand = [&](int cb) -> int {
            s_mark[w][lane] = 0;
            wave_fence();
            if (len > 0 && pref >= cb && pref < cb + 64) s_mark[w][pref - cb] = lane + 1;
            wave_fence();
            const int mk = max(wave_scan_max(s_mark[w][lane]), carry);
            wave_fence();
            carry = __builtin_amdgcn_readlane(mk, 63);
            return cb + lane + __shfl(delta, mk - 1, 64);
          };
          // the next batch's candidates are requested while this batch is tested
          double4 qn = make_double4(0.0, 0.0, 0.0, 0.0);
          int32_t jn = 0;
          if (C > 0) {
            const int t = cand(0);
            if (lane < C) {
              qn = sp[t];
              jn = order[t];
            }
          }
#pragma unroll 1
          for (int cb = 0; cb < C; cb += 64) {
            const double4 q = qn;
            const int32_t j = jn;
            const bool cv = cb + lane < C;
            if (cb + 64 < C) {
              const int t = cand(cb + 64);
              if (cb + 64 + lane < C) {
                qn = sp[t];
                jn = order[t];
              }
            }
            const double dx = fmax(fabs(q.x - bc[0]) - be[0], 0.0);
            const double dy = fmax(fabs(q.y - bc[1]) - be[1], 0.0);
            const double dz = fmax(fabs(q.z - bc[2]) - be[2], 0.0);
            const double rr = (q.w + hrow) * (1.0 + 1e-6);  // (the differences above are rounded)
            const bool near = cv && dx * dx + dy * dy + dz * dz <= rr * rr;
            const uint64_t m = __ballot(near);
            if (near) {
              const int at = (head + fill + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))) &
                             (kRing - 1);
              s_xy[w][at] = make_double2(q.x, q.y);
              s_zh[w][at] = make_double2(q.z, q.w);
              s_id[w][at] = j;
            }
            fill += __popcll(m);
            if (fill >= 64) test();
          }
        }
      }
      if (fill > 0) test();
    }
    if (MODE != 1) {
      int bin = -1;
      if (lane < nw) {
        const int cc = ghost ? 1 : run;
        cnt[myi] = cc;
        int band = 0;
        while (band < GF_NBAND - 1 && cc > kBandHi[band]) ++band;
        bin = mrow * GF_NBAND + band;
        max_local[0] = max(max_local[0], mrow ? 0 : cc);
        max_local[1] = max(max_local[1], mrow ? cc : 0);
      }
      // per-wave histogram, all lanes active: lane b counts bin b
#pragma unroll
      for (int b = 0; b < 2 * GF_NBAND; ++b) {
        const int hb = __popcll(__ballot(bin == b));
        if (lane == b) hist_local += hb;
      }
    }
  }
  if (MODE != 1) {
    // one atomic per block and bin (a few addresses for the whole grid)
    __syncthreads();
    if (lane < 2 * GF_NBAND && hist_local) atomicAdd(&s_hist[lane], hist_local);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      int cm = max_local[m];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) cm = max(cm, __shfl_xor(cm, o, 64));
      if (lane == 0) atomicMax(&s_hist[2 * GF_NBAND + m], cm);
    }
    __syncthreads();
    if (tid < 2 * GF_NBAND && s_hist[tid]) atomicAdd(&hist[tid], s_hist[tid]);
    if (tid >= 2 * GF_NBAND && tid < 2 * GF_NBAND + 2 && s_hist[tid]) atomicMax(&maxrow[tid - 2 * GF_NBAND], s_hist[tid]);
  }
}

// Sort each row ascending.  One wave per chunk of rows (grid-stride over
// chunks), the chunk's row offsets one per lane.  A row is sorted in registers
// by a bitonic network of P = the next power of two >= its length: lane l holds
// positions l, l + 64, ...; exchanges at distance 64 and 128 stay in the lane,
// shorter ones take the partner's value by a lane move and keep the smaller or
// the larger of the two by a median of three.  Two neighbouring rows of at most
// 32 entries (film rows) are sorted side by side in the halves of the wave.
// The next rows' entries are loaded while the current ones are sorted.  Rows
// with more than 256 entries use a wave-private LDS buffer.
//
// What bounds it: VALU issue, 28 stages for a row of 65 to 128 entries.  A
// stage took a lane move (two and a select at distances 4 and 8, an LDS
// permute at 16 and 32), a minimum, a maximum and a select; now a lane move and
// the median.  Chunks shrink on small clouds, whose few long chunks left most of
// the chip idle.  Mixed cloud 225 -> 120 us, 2.0M jet 1.23 -> 0.65 ms, 25k-particle
// plate 99 -> 12 us, 916 particles 49 -> 4 us.
constexpr int kSortBlock = 256;
constexpr int kSortWaves = kSortBlock / 64;
constexpr int kSortChunk = 64;   // rows of a chunk, at most
constexpr int kNoEntry = 0x7fffffff;

// the median of three signed integers (one instruction)
__device__ __forceinline__ int32_t med3(int32_t a, int32_t b, int32_t c) { return max(min(a, b), min(max(a, b), c)); }

// One exchange at distance j (a power of two up to 32, a constant once the
// networks are unrolled) between lanes: the smaller of v and lane ^ j's value
// where bound is -1, the larger where it is kNoEntry (entries are >= 0).  The
// partner comes by a DPP quad permutation (1, 2), a half-row mirror and a quad
// mirror (4: 7 xor 3), a row rotation by half a row (8) or the swaps of rows
// and half waves (16, 32), which give both values of the pair at once.  Every
// lane of the wave is active here.
__device__ __forceinline__ int32_t exchange(int32_t v, int j, int32_t bound) {
  switch (j) {
    case 1: return med3(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true), bound);  // quad_perm [1, 0, 3, 2]
    case 2: return med3(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true), bound);  // quad_perm [2, 3, 0, 1]
    case 4: {
      const int32_t m = __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);             // row_half_mirror
      return med3(v, __builtin_amdgcn_mov_dpp(m, 0x1B, 0xF, 0xF, true), bound);         // quad_perm [3, 2, 1, 0]
    }
    case 8: return med3(v, __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true), bound);  // row_ror:8
    case 16: {
      const auto s = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
      return med3((int32_t)s[0], (int32_t)s[1], bound);
    }
    default: {
      const auto s = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
      return med3((int32_t)s[0], (int32_t)s[1], bound);
    }
  }
}

// The bitonic network for P (power of two) elements, position lane + 64 r in
// v[r] (P <= 64: v[0] alone; P <= 32: independently in every group of P lanes).
// low[b]: -1 in the lanes whose bit b is clear, else kNoEntry; the bounds of a
// descending sequence differ from an ascending one's in the top bit.
template <int P, int NV>
__device__ inline void sort_net(int32_t (&v)[NV], int lane, const int32_t (&low)[6]) {
  constexpr int R = P <= 64 ? 1 : P / 64;
  static_assert(R <= NV, "the network needs a register per 64 positions");
#pragma unroll
  for (int k = 2; k <= P; k <<= 1) {
    const int32_t flip = (k < 64 && k < P && (lane & k)) ? (int32_t)0x80000000 : 0;
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j >= 64) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int o = r ^ (j / 64);
          if (o < r) continue;
          const bool up = ((64 * r) & k) == 0;
          const int32_t a = min(v[r], v[o]), b = max(v[r], v[o]);
          v[r] = up ? a : b;
          v[o] = up ? b : a;
        }
      } else {
        const int bit = j == 1 ? 0 : j == 2 ? 1 : j == 4 ? 2 : j == 8 ? 3 : j == 16 ? 4 : 5;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const bool down = k >= 64 && k < P && ((64 * r) & k) != 0;
          v[r] = exchange(v[r], j, low[bit] ^ (down ? (int32_t)0x80000000 : flip));
        }
      }
    }
  }
}

// STAGED: a row of at most sw entries is read from stage[i * sw ...]
// (the count pass's copy) and written, sorted, to its CSR place; a longer row
// (filled by the fill pass), or every row without STAGED, is sorted in place.
// LONG: rows of more than 128 entries exist.
template <bool LONG, bool STAGED>
__global__ void __launch_bounds__(kSortBlock) k_row_sort(const int64_t *__restrict__ row_ptr, int32_t *col,
                                                         const int32_t *__restrict__ stage, int sw, int64_t n,
                                                         int chunk) {
  extern __shared__ int32_t sort_buf[];  // rows of more than 256 entries: kSortWaves x kMaxRow
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int32_t low[6];
#pragma unroll
  for (int b = 0; b < 6; ++b) low[b] = (lane >> b) & 1 ? kNoEntry : -1;
  const int64_t nchunks = (n + chunk - 1) / chunk;
  for (int64_t ch = (int64_t)blockIdx.x * kSortWaves + w; ch < nchunks; ch += (int64_t)gridDim.x * kSortWaves) {
    const int64_t i0 = ch * chunk;
    const int nr = (int)min((int64_t)chunk, n - i0);
    int64_t rb = 0;
    int rl = 0;
    if (lane < nr) {
      rb = row_ptr[i0 + lane];
      rl = (int)(row_ptr[i0 + lane + 1] - rb);
    }
    auto src = [&](int r) -> const int32_t * {
      if (STAGED && __builtin_amdgcn_readlane(rl, r) <= sw) return stage + (i0 + r) * (int64_t)sw;
      return col + readlane64(rb, r);
    };
    // rows of up to kRegRow entries are held in registers (NV per lane)
    constexpr int NV = LONG ? 4 : 2;
    constexpr int kRegRow = 64 * NV;
    // whether rows r and r + 1 are sorted side by side
    auto paired = [&](int r) {
      return r + 1 < nr && __builtin_amdgcn_readlane(rl, r) <= 32 && __builtin_amdgcn_readlane(rl, r + 1) <= 32;
    };
    auto fetch = [&](int r, int32_t (&a)[NV]) {
#pragma unroll
      for (int q = 0; q < NV; ++q) a[q] = kNoEntry;
      if (r >= nr) return;
      const int len = __builtin_amdgcn_readlane(rl, r);
      const int32_t *sr = src(r);
      if (paired(r)) {
        const int len1 = __builtin_amdgcn_readlane(rl, r + 1);
        const int32_t *s1 = src(r + 1);
        const int32_t *mine = lane < 32 ? sr + lane : s1 + (lane - 32);
        if ((lane & 31) < (lane < 32 ? len : len1)) a[0] = *mine;
      } else if (len <= kRegRow) {
#pragma unroll
        for (int q = 0; q < NV; ++q)
          if (lane + 64 * q < len) a[q] = sr[lane + 64 * q];
      }
    };
    int32_t v[NV];
    fetch(0, v);
    for (int r = 0; r < nr;) {
      const int64_t b = readlane64(rb, r);
      const int len = __builtin_amdgcn_readlane(rl, r);
      const bool two = paired(r);
      int32_t nx[NV];
      fetch(r + (two ? 2 : 1), nx);
      if (two) {
        const int64_t b1 = readlane64(rb, r + 1);
        const int len1 = __builtin_amdgcn_readlane(rl, r + 1);
        if (max(len, len1) <= 8) sort_net<8, NV>(v, lane, low);
        else if (max(len, len1) <= 16) sort_net<16, NV>(v, lane, low);
        else sort_net<32, NV>(v, lane, low);
        if ((lane & 31) < (lane < 32 ? len : len1)) col[(lane < 32 ? b : b1) + (lane & 31)] = v[0];
      } else if (len <= kRegRow) {
        if (len <= 16) sort_net<16, NV>(v, lane, low);
        else if (len <= 32) sort_net<32, NV>(v, lane, low);
        else if (len <= 64) sort_net<64, NV>(v, lane, low);
        else if (len <= 128) sort_net<128, NV>(v, lane, low);
        else if constexpr (LONG) sort_net<256, NV>(v, lane, low);
#pragma unroll
        for (int q = 0; q < NV; ++q)
          if (lane + 64 * q < len) col[b + lane + 64 * q] = v[q];
      } else if constexpr (LONG) {
        int32_t *bw = sort_buf + w * kMaxRow;
        const int32_t *sr = src(r);
        int P = 1;
        while (P < len) P <<= 1;
        for (int t = lane; t < P; t += 64) bw[t] = (t < len) ? sr[t] : kNoEntry;
        wave_fence();
        for (int k = 2; k <= P; k <<= 1) {
          for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = lane; t < P; t += 64) {
              const int u = t ^ j;
              if (u > t) {
                const int32_t a = bw[t], c = bw[u];
                if ((a > c) == ((t & k) == 0)) { bw[t] = c; bw[u] = a; }
              }
            }
            wave_fence();
          }
        }
        for (int t = lane; t < len; t += 64) col[b + t] = bw[t];
        wave_fence();
      }
#pragma unroll
      for (int q = 0; q < NV; ++q) v[q] = nx[q];
      r += two ? 2 : 1;
    }
  }
}

// Grouping.  The given order lists the particles of model 0, then those of
// model 1; each model's rows of more than kTileBandRow entries follow its tiled
// rows, the order kept in both parts.  pos: the long rows before each place.
__global__ void __launch_bounds__(kBlock) k_group_flag(const int32_t *__restrict__ order, const int32_t *__restrict__ cnt,
                                                       int64_t n, int32_t *__restrict__ flag) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s < n) flag[s] = cnt[order[s]] > kTileBandRow ? 1 : 0;
}

__global__ void __launch_bounds__(kBlock) k_group_scatter(const int32_t *__restrict__ order,
                                                          const int32_t *__restrict__ flag,
                                                          const int32_t *__restrict__ pos, int64_t n, int64_t n0,
                                                          int64_t long0, int64_t long1, int32_t *__restrict__ grouped) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  // first place, number of particles and of long rows of this place's model
  const int64_t m0 = s < n0 ? 0 : n0, mn = s < n0 ? n0 : n - n0, ml = s < n0 ? long0 : long1;
  const int64_t before = pos[s] - (s < n0 ? 0 : long0);
  grouped[flag[s] ? m0 + (mn - ml) + before : s - before] = order[s];
}

__global__ void __launch_bounds__(kBlock) k_copy_i32(const int32_t *__restrict__ a, int64_t n, int32_t *__restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = a[i];
}

// ---------------------------------------------------------------- tiles
// Tiled row ranges (one per model), as passed to the tile kernels: tiles
// [tile_start[q], tile_start[q+1]) cover rows [row_start[q], row_start[q] +
// nrows[q]) of the grouped order; gsel[q] is the model.
struct TileGroups {
  int nq = 0;
  int gsel[2];
  int64_t tile_start[3];
  int64_t row_start[2];
  int64_t nrows[2];
  int64_t uniq[2];       // first place of the range's tiles in the list of distinct indices,
  int entries[2];        // and places per tile: what its rows can hold
};
constexpr int kTileEntries = kTileRows * kTileBandRow;  // entries one tile can hold
constexpr int kTileThreads = 512;


__device__ inline int tile_group(const TileGroups &tg, int64_t t) {
  int q = 0;
  while (q + 1 < tg.nq && t >= tg.tile_start[q + 1]) ++q;
  return q;
}
// first place of tile t of range q
__device__ inline int64_t tile_uniq(const TileGroups &tg, int q, int64_t t) {
  return tg.uniq[q] + (t - tg.tile_start[q]) * tg.entries[q];
}

// One block per tile.  The tile's distinct indices go into an LDS hash set
// (open addressing, linear probing); the lane that inserts a key also takes a
// place for it in ulist (one counter update per wave).  The list is sorted in
// groups of 64 in registers, a key's rank is its place in its group plus the
// number of smaller keys of every other group (binary searches side by side),
// the sorted list is written to uniq[tile_uniq ...], and each entry's slot is
// the rank kept beside its key, read at the table position its insertion found;
// cnt[t] = number of distinct indices.  Each wave takes whole rows (w, w + 8,
// ...), a lane at most two entries of each (rows hold at most kTileBandRow = 128
// entries): its column indices are all requested at once, and all tried in the
// table at once, and stay in registers, with their table positions, until the
// slots are written.  The result does not depend on the order of the insertions.
//
// What bounds it: VALU issue and LDS latency.  A 3D tile of the mixed cloud
// has 460 distinct indices of 3,300; ranking each against all the others took
// two thirds of the kernel's instructions.  Mixed cloud 265 -> 193 us, 2.0M jet
// 835 -> 744 us (and the launch that counted each tile's entries, 20 and 28 us).
constexpr int kHashBits = 12;
constexpr int kHashSize = 1 << kHashBits;  // >= kTileEntries >= distinct keys: every probe ends
static_assert(kHashSize >= kTileEntries, "the hash set must hold every entry of a tile");

__device__ inline int hash_slot(int32_t j) { return (int)(((uint32_t)j * 2654435761u) >> (32 - kHashBits)); }

__global__ void __launch_bounds__(kTileThreads) k_tile_unique(TileGroups tg, const int64_t *__restrict__ row_ptr,
                                                              const int32_t *__restrict__ col,
                                                              const int32_t *__restrict__ grouped,
                                                              uint16_t *__restrict__ slot,
                                                              int32_t *__restrict__ uniq, int32_t *__restrict__ cnt,
                                                              int32_t *__restrict__ grp_max) {
  constexpr int NW = kTileThreads / 64;
  __shared__ int32_t hkey[kHashSize];
  __shared__ __attribute__((aligned(4))) uint16_t hrank[kHashSize];
  __shared__ int32_t ulist[kTileEntries];  // distinct indices, sorted in groups of 64
  // the list's length lies where the ranks go later: 40,960 bytes let four blocks share a CU
  int32_t &ucount = *reinterpret_cast<int32_t *>(hrank);
  const int64_t t = blockIdx.x;
  const int q = tile_group(tg, t);
  const int64_t r0 = (t - tg.tile_start[q]) * kTileRows;
  const int R = (int)min((int64_t)kTileRows, tg.nrows[q] - r0);
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  // 1. distinct indices; entry c of a lane: row wave + NW (c / 2), entry lane + 64 (c % 2)
  static_assert(kTileRows == 4 * NW && kTileBandRow == 128, "four rows per wave, two entries per lane and row");
  constexpr int kC = 8;
  int64_t base[kC / 2];
  int32_t jj[kC];
  int hh[kC];
#pragma unroll
  for (int c = 0; c < kC; c += 2) {
    const int r = wave + NW * (c >> 1);
    base[c / 2] = 0;
    int len = 0;
    if (r < R) {
      const int32_t i = grouped[tg.row_start[q] + r0 + r];
      base[c / 2] = row_ptr[i];
      len = (int)(row_ptr[i + 1] - base[c / 2]);  // <= kTileBandRow: tiled rows
    }
    jj[c] = lane < len ? col[base[c / 2] + lane] : -1;
    jj[c + 1] = lane + 64 < len ? col[base[c / 2] + lane + 64] : -1;
  }
  {
    const int4 none = make_int4(-1, -1, -1, -1);
    int4 *h4 = reinterpret_cast<int4 *>(hkey);
    for (int h = tid; h < kHashSize / 4; h += kTileThreads) h4[h] = none;
  }
  if (tid == 0) ucount = 0;
  __syncthreads();
  int32_t prev[kC];
#pragma unroll
  for (int c = 0; c < kC; ++c) {
    hh[c] = hash_slot(jj[c]);
    prev[c] = jj[c] >= 0 ? atomicCAS(&hkey[hh[c]], -1, jj[c]) : jj[c];
  }
  int fresh = 0;  // bit c: this lane inserted entry c's key
#pragma unroll
  for (int c = 0; c < kC; ++c) {
    while (prev[c] != -1 && prev[c] != jj[c]) {
      hh[c] = (hh[c] + 1) & (kHashSize - 1);
      prev[c] = atomicCAS(&hkey[hh[c]], -1, jj[c]);
    }
    if (prev[c] == -1 && jj[c] >= 0) fresh |= 1 << c;
  }
  {
    const int mine = __popc(fresh), inc = wave_scan_add(mine);
    int ub = 0;
    if (lane == 63 && inc) ub = atomicAdd(&ucount, inc);
    int s = __builtin_amdgcn_readlane(ub, 63) + inc - mine;
#pragma unroll
    for (int c = 0; c < kC; ++c)
      if ((fresh >> c) & 1) ulist[s++] = jj[c];
  }
  __syncthreads();
  const int U = ucount, NG = (U + 63) / 64;
  // 2. groups of 64 sorted in place (the last one padded with kNoEntry)
  int32_t low[6];
#pragma unroll
  for (int b = 0; b < 6; ++b) low[b] = (lane >> b) & 1 ? kNoEntry : -1;
  for (int gi = wave; gi < NG; gi += NW) {
    int32_t v[1] = {64 * gi + lane < U ? ulist[64 * gi + lane] : kNoEntry};
    sort_net<64, 1>(v, lane, low);
    ulist[64 * gi + lane] = v[0];
  }
  __syncthreads();
  // 3. ranks: to the sorted list, and beside the keys
  for (int gi = wave; gi < NG; gi += NW) {
    const int32_t v = ulist[64 * gi + lane];
    int rank = lane;
    for (int o = 0; o < NG; o += 4) {  // four groups' searches side by side
      int lo[4] = {0, 0, 0, 0};
      const int32_t *l[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) l[k] = ulist + 64 * min(o + k, NG - 1);
#pragma unroll
      for (int step = 32; step > 0; step >>= 1)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (l[k][lo[k] + step - 1] < v) lo[k] += step;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (o + k < NG && o + k != gi) rank += lo[k] + (l[k][lo[k]] < v ? 1 : 0);
    }
    if (v != kNoEntry) {
      uniq[tile_uniq(tg, q, t) + rank] = v;
      int h = hash_slot(v);
      while (hkey[h] != v) h = (h + 1) & (kHashSize - 1);
      hrank[h] = (uint16_t)rank;
    }
  }
  if (tid == 0) {
    cnt[t] = U;
    atomicMax(&grp_max[q], U);
  }
  __syncthreads();
  // 4. slots: the rank kept beside each entry's index
#pragma unroll
  for (int c = 0; c < kC; ++c)
    if (jj[c] >= 0) slot[base[c >> 1] + lane + 64 * (c & 1)] = hrank[hh[c]];
}

// uniq (at tile_uniq) -> tile_u (at the list offsets), a wave per tile
__global__ void __launch_bounds__(kBlock) k_tile_compact(TileGroups tg, const int64_t *__restrict__ u_off,
                                                         const int32_t *__restrict__ uniq, int64_t nt,
                                                         int32_t *__restrict__ tile_u) {
  const int64_t t = (int64_t)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (t >= nt) return;
  const int64_t a = tile_uniq(tg, tile_group(tg, t), t), b = u_off[t], m = u_off[t + 1] - b;
#pragma unroll 4
  for (int64_t s = threadIdx.x & 63; s < m; s += 64) tile_u[b + s] = uniq[a + s];
}

// reverse-edge map: rev[k] = position of (j, i) in row j for entry k = (i, j)
// (binary search in the sorted row j, -1 if i is not listed there); a team of
// kRevTeam lanes per row i, each lane running the searches of kRevU entries
// side by side, so that every step requests kRevU independent loads (a lone
// search waits for each of its ~log2 |S_j| steps in turn)
constexpr int kRevTeam = 8;
constexpr int kRevU = 4;
__global__ void __launch_bounds__(kBlock) k_rev(const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                                                int64_t n, int32_t *__restrict__ rev) {
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = gt / kRevTeam;
  if (i >= n) return;
  const int64_t b = row_ptr[i], e = row_ptr[i + 1];
  for (int64_t kb = b + gt % kRevTeam; kb < e; kb += kRevU * kRevTeam) {
    // entries past the row's end search for its last entry's twin and store nothing; a finished
    // search reads entry kb (in the row) so that no load is skipped
    int32_t jj[kRevU];
#pragma unroll
    for (int u = 0; u < kRevU; ++u) jj[u] = col[min(kb + u * kRevTeam, e - 1)];
    int64_t lo[kRevU], hi[kRevU], end[kRevU];
#pragma unroll
    for (int u = 0; u < kRevU; ++u) {
      lo[u] = row_ptr[jj[u]];
      hi[u] = end[u] = row_ptr[jj[u] + 1];
    }
    bool act = true;
    while (act) {
      int64_t mid[kRevU];
      int32_t v[kRevU];
#pragma unroll
      for (int u = 0; u < kRevU; ++u) {
        mid[u] = (lo[u] + hi[u]) >> 1;
        v[u] = col[lo[u] < hi[u] ? mid[u] : kb];
      }
      act = false;
#pragma unroll
      for (int u = 0; u < kRevU; ++u) {
        if (lo[u] < hi[u]) {
          if (v[u] < i) lo[u] = mid[u] + 1;
          else hi[u] = mid[u];
        }
        act |= lo[u] < hi[u];
      }
    }
    int32_t c[kRevU];
#pragma unroll
    for (int u = 0; u < kRevU; ++u) c[u] = col[lo[u] < end[u] ? lo[u] : kb];
#pragma unroll
    for (int u = 0; u < kRevU; ++u)
      if (kb + u * kRevTeam < e) rev[kb + u * kRevTeam] = (lo[u] < end[u] && c[u] == i) ? (int32_t)lo[u] : -1;
  }
}

int ceil_log2(int v) {
  int b = 0;
  while ((1 << b) < v) ++b;
  return b;
}

void free_nbr(gf_nbr *nb) {
  if (!nb) return;
  (void)hipSetDevice(nb->device);
  nbr_release(nb);
  delete nb;
}

template <class T>
bool take(gf_nbr *nb, T *&p, size_t count, bool kept = true) {
  p = static_cast<T *>(nbr_alloc(nb, sizeof(T) * std::max<size_t>(count, 1), kept));
  return p != nullptr;
}
// the same for an array of the maps built at first use, which a call that failed or was captured may have left
template <class T>
bool take_once(gf_nbr *nb, T *&p, size_t count, bool kept) {
  return p || take(nb, p, count, kept);
}

}  // namespace

extern "C" void gf_nbr_free(gf_nbr *nbr) { free_nbr(nbr); }

extern "C" gf_status gf_nbr_info(const gf_nbr *nbr, int64_t *n, int64_t *nnz, int32_t *max_row) {
  if (!nbr) return GF_EINVAL;
  if (n) *n = nbr->n;
  if (nnz) *nnz = nbr->nnz;
  if (max_row) *max_row = nbr->max_row;
  return GF_OK;
}

extern "C" gf_status gf_nbr_view(const gf_nbr *nbr, int64_t *nnz, const int64_t **row_ptr, const int32_t **col) {
  if (!nbr) return GF_EINVAL;
  if (nnz) *nnz = nbr->nnz;
  if (row_ptr) *row_ptr = nbr->row_ptr;
  if (col) *col = nbr->col;
  return GF_OK;
}

extern "C" gf_status gf_nbr_export(gf_ctx *ctx, const gf_nbr *nbr, int64_t *row_ptr, int32_t *col) {
  if (!ctx || !nbr) return GF_EINVAL;
  GF_HIP(ctx, hipSetDevice(ctx->device));
  if (row_ptr)
    GF_HIP(ctx, hipMemcpyAsync(row_ptr, nbr->row_ptr, sizeof(int64_t) * (nbr->n + 1), hipMemcpyDeviceToDevice, ctx->stream));
  if (col && nbr->nnz)
    GF_HIP(ctx, hipMemcpyAsync(col, nbr->col, sizeof(int32_t) * nbr->nnz, hipMemcpyDeviceToDevice, ctx->stream));
  return GF_OK;
}

gf_status ensure_rev(gf_ctx *ctx, gf_nbr *nbr) {
  if (nbr->built & gf_nbr::kRevMap) return GF_OK;
  if (nbr->nnz > (int64_t)0x7fffffff)
    return set_error(ctx, GF_ECAPACITY, "the reverse-edge map holds 32-bit positions; %lld entries exceed it",
                     (long long)nbr->nnz);
  const bool cap = capturing(ctx);
  if (!take_once(nbr, nbr->rev, nbr->nnz, !cap)) return set_error(ctx, GF_ENOMEM, "reverse-edge map allocation failed");
  hipLaunchKernelGGL(k_rev, dim3(grid_for(nbr->n * kRevTeam, kBlock)), dim3(kBlock), 0, ctx->stream, nbr->row_ptr, nbr->col,
                     nbr->n, nbr->rev);
  GF_LAUNCH_CHECK(ctx);
  if (!cap) nbr->built |= gf_nbr::kRevMap;
  return GF_OK;
}

namespace {
__global__ void __launch_bounds__(kBlock) k_grouped_len(const int32_t *__restrict__ grouped,
                                                        const int64_t *__restrict__ row_ptr, int64_t n,
                                                        int32_t *__restrict__ len, int32_t *__restrict__ gpos) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int32_t i = grouped[t];
  len[t] = (int32_t)(row_ptr[i + 1] - row_ptr[i]);
  gpos[i] = (int32_t)t;
}
// grev for the rows in grouped order, a team of kRevTeam lanes per row
__global__ void __launch_bounds__(kBlock) k_grouped_rev(const int32_t *__restrict__ grouped,
                                                        const int64_t *__restrict__ row_ptr,
                                                        const int32_t *__restrict__ col,
                                                        const int32_t *__restrict__ rev,
                                                        const int64_t *__restrict__ grow_ptr,
                                                        const int32_t *__restrict__ gpos, int64_t n,
                                                        int32_t *__restrict__ grev) {
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t t = gt / kRevTeam;
  const int lane = (int)(gt % kRevTeam);
  if (t >= n) return;
  const int32_t i = grouped[t];
  const int64_t b = row_ptr[i], len = row_ptr[i + 1] - b, ob = grow_ptr[t];
  for (int64_t o = lane; o < len; o += kRevTeam) {
    const int32_t j = col[b + o];
    const int32_t kr = rev[b + o];
    grev[ob + o] = (j == i || kr < 0) ? -1 : (int32_t)(grow_ptr[gpos[j]] + (kr - row_ptr[j]));
  }
}
}  // namespace

gf_status ensure_grouped_rows(gf_ctx *ctx, gf_nbr *nbr) {
  if (nbr->built & gf_nbr::kGroupedMaps) return GF_OK;
  gf_status st = ensure_rev(ctx, nbr);  // also checks that positions fit 32 bits
  if (st) return st;
  const int64_t n = nbr->n;
  const bool cap = capturing(ctx);
  if (!take_once(nbr, nbr->grow_ptr, n + 1, !cap) || !take_once(nbr, nbr->gpos, n, !cap) ||
      !take_once(nbr, nbr->grev, nbr->nnz, !cap))
    return set_error(ctx, GF_ENOMEM, "grouped row offsets allocation failed");
  Arena ar;
  if ((st = ensure_scratch(ctx, arena_bytes({sizeof(int32_t) * n, sizeof(int64_t) * scan_tmp_elems(n + 1)}), &ar)))
    return st;
  int32_t *len = ar.take<int32_t>(n);
  int64_t *tmp = ar.take<int64_t>(scan_tmp_elems(n + 1));
  hipLaunchKernelGGL(k_grouped_len, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, ctx->stream, nbr->grouped,
                     nbr->row_ptr, n, len, nbr->gpos);
  GF_LAUNCH_CHECK(ctx);
  if ((st = scan_i32_to_i64(ctx, len, nbr->grow_ptr, n, tmp))) return st;
  hipLaunchKernelGGL(k_grouped_rev, dim3(grid_for(n * kRevTeam, kBlock)), dim3(kBlock), 0, ctx->stream, nbr->grouped,
                     nbr->row_ptr, nbr->col, nbr->rev, nbr->grow_ptr, nbr->gpos, n, nbr->grev);
  GF_LAUNCH_CHECK(ctx);
  if (!cap) nbr->built |= gf_nbr::kGroupedMaps;
  return GF_OK;
}

namespace {
// Room for each transposed tile, in units of 64: the lengths, ceil(U / 64)
// groups of slots and at most kTileRows + entries / 64 steps (a group's length is
// at most the fewest entries of a slot of the group before, so that the padding
// of all groups together is less than the first group), rounded up to fours per
// group.
__global__ void __launch_bounds__(kBlock) k_tile_room(TileRows tr, const int64_t *__restrict__ row_ptr,
                                                      const int64_t *__restrict__ tile_off, int64_t nt,
                                                      int32_t *__restrict__ room) {
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t t = gt / kTileRows;
  if (t >= nt) return;  // (teams of kTileRows lanes leave together)
  const int32_t i = tile_row(tr, t, (int)(gt % kTileRows));
  int len = i >= 0 ? (int)(row_ptr[i + 1] - row_ptr[i]) : 0;
#pragma unroll
  for (int o = kTileRows / 2; o > 0; o >>= 1) len += __shfl_xor(len, o, kTileRows);
  if (gt % kTileRows == 0) room[t] = 1 + 4 * ((int)(tile_off[t + 1] - tile_off[t] + 63) / 64) + kTileRows + len / 64;
}

// A block per tile, a team of 8 lanes per row.  s_mask: the rows that list each
// slot, a bit each (a row lists a slot at most once), so an entry's place among
// its slot's is the number of lower bits: no pass waits for another row.  The
// slots' order among those of equal length is whichever comes first: it moves
// no sum's terms.  The block is put together in LDS and written in order.
__global__ void __launch_bounds__(kBlock) k_tile_transpose(TileRows tr, const int64_t *__restrict__ row_ptr,
                                                           const int32_t *__restrict__ col,
                                                           const uint16_t *__restrict__ slot,
                                                           const int64_t *__restrict__ tile_off,
                                                           const int64_t *__restrict__ tperm_off, int cap,
                                                           uint16_t *__restrict__ tperm, uint16_t *__restrict__ tself) {
  constexpr int T = kBlock / kTileRows, Q = kTileBandRow / T;
  extern __shared__ uint32_t s_mask[];                          // [cap]
  uint16_t *s_pos = reinterpret_cast<uint16_t *>(s_mask + cap);  // [cap] place in the order
  uint16_t *s_out = s_pos + ((cap + 1) & ~1);                    // the block
  __shared__ int s_off[kTileRows + 1];
  __shared__ int s_bin[kTileRows + 1];  // slots of each length, then the next place of each
  __shared__ int s_first[64];           // first step of each group
  const int64_t t = blockIdx.x;
  const int U = (int)(tile_off[t + 1] - tile_off[t]), G = (U + 63) / 64;
  const int team = threadIdx.x / T, lane = threadIdx.x % T;
  const int32_t i = tile_row(tr, t, team);
  const int64_t b = i >= 0 ? row_ptr[i] : 0;
  const int n = i >= 0 ? (int)(row_ptr[i + 1] - b) : 0;
  for (int s = threadIdx.x; s < U; s += kBlock) s_mask[s] = 0;
  if (threadIdx.x <= kTileRows) s_bin[threadIdx.x] = 0;
  if (threadIdx.x < 64) s_out[threadIdx.x] = 0;
  if (threadIdx.x == 0) s_off[0] = 0;
  if (lane == 0) s_off[team + 1] = n;
  __syncthreads();
  // (the row's slots stay in registers; past its end the last one, unused)
  uint16_t sl[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (n > q * T) sl[q] = slot[b + min(lane + q * T, n - 1)];
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (lane + q * T < n) atomicOr(&s_mask[sl[q]], 1u << team);
  if (threadIdx.x < 64) {
    int v = threadIdx.x < kTileRows ? s_off[threadIdx.x + 1] : 0;
    v = wave_scan_add(v);
    if (threadIdx.x < kTileRows) s_off[threadIdx.x + 1] = v;
  }
  __syncthreads();
  for (int s = threadIdx.x; s < U; s += kBlock) atomicAdd(&s_bin[__popc(s_mask[s])], 1);
  __syncthreads();
  if (threadIdx.x < 64) {  // lane l: length kTileRows - l
    const int v = threadIdx.x <= kTileRows ? s_bin[kTileRows - threadIdx.x] : 0;
    const int inc = wave_scan_add(v);
    if (threadIdx.x <= kTileRows) s_bin[kTileRows - threadIdx.x] = inc - v;
  }
  for (int s = U + threadIdx.x; s < 64 * G; s += kBlock) s_out[64 + s] = kSlotNone;
  __syncthreads();
  for (int s = threadIdx.x; s < U; s += kBlock) {
    const int len = __popc(s_mask[s]), p = atomicAdd(&s_bin[len], 1);
    s_pos[s] = (uint16_t)p;
    s_out[64 + p] = (uint16_t)s;
    if (p % 64 == 0) s_out[p / 64] = (uint16_t)len;
  }
  __syncthreads();
  const int E = s_off[kTileRows];
  uint16_t *steps = s_out + 64 * (1 + G);
  if (threadIdx.x < 64) {
    const int v = (s_out[threadIdx.x] + 3) & ~3, inc = wave_scan_add(v);
    s_first[threadIdx.x] = inc - v;
    if (threadIdx.x == 63) s_bin[0] = inc;
  }
  __syncthreads();
  const int S = s_bin[0];
  for (int k = threadIdx.x; k < 64 * S; k += kBlock) steps[k] = (uint16_t)E;
  __syncthreads();
  const int e0 = s_off[team];
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (lane + q * T < n) {
      const int s = sl[q], p = s_pos[s], lower = __popc(s_mask[s] & ((1u << team) - 1));
      steps[64 * (s_first[p / 64] + (lower & ~3)) + 4 * (p % 64) + (lower & 3)] = (uint16_t)(e0 + lane + q * T);
      if (col[b + lane + q * T] == i) tself[kTileRows * t + team] = (uint16_t)s;
    }
  __syncthreads();
  uint32_t *out = reinterpret_cast<uint32_t *>(tperm + 64 * tperm_off[t]);
  for (int k = threadIdx.x; k < 32 * (1 + G + S); k += kBlock) out[k] = reinterpret_cast<const uint32_t *>(s_out)[k];
}

// places of each particle, and the order in which they came (whatever it was).
// Ghost particles receive nothing, so their places are left out: a row's
// neighbours list it in turn and are at most kTileBandRow, but a ghost can be in
// the rows of any number of others.
__global__ void __launch_bounds__(kBlock) k_places_count(const int32_t *__restrict__ tile_u, int64_t total, int64_t n_rows,
                                                         int32_t *__restrict__ cnt, int32_t *__restrict__ rank) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < total && tile_u[k] < n_rows) rank[k] = atomicAdd(&cnt[tile_u[k]], 1);
}
__global__ void __launch_bounds__(kBlock) k_places_fill(const int32_t *__restrict__ tile_u, int64_t total, int64_t n_rows,
                                                        const int32_t *__restrict__ gptr,
                                                        const int32_t *__restrict__ rank, int32_t *__restrict__ raw) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < total && tile_u[k] < n_rows) raw[gptr[tile_u[k]] + rank[k]] = (int32_t)k;
}
// each particle's places ascending (a few tens): a place goes after the smaller ones
__global__ void __launch_bounds__(kBlock) k_places_sort(const int32_t *__restrict__ gptr, int64_t n,
                                                        const int32_t *__restrict__ raw, int32_t *__restrict__ gidx) {
  constexpr int T = 16;
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t j = gt / T;
  if (j >= n) return;
  const int32_t a = gptr[j], b = gptr[j + 1];
  for (int32_t k = a + (int)(gt % T); k < b; k += T) {
    const int32_t v = raw[k];
    int32_t r = a;
#pragma unroll 4
    for (int32_t q = a; q < b; ++q) r += raw[q] < v ? 1 : 0;
    gidx[r] = v;
  }
}
}  // namespace

gf_status ensure_tile_transpose(gf_ctx *ctx, gf_nbr *nb) {
  if (nb->built & gf_nbr::kTransposed) return GF_OK;
  if (nb->nnz > (int64_t)0x7fffffff)
    return set_error(ctx, GF_ECAPACITY, "the adjoints' maps hold 32-bit positions; %lld entries exceed them",
                     (long long)nb->nnz);
  const int64_t nt = nb->ntiles, n = nb->n, total = nb->tile_total;
  const bool cap = capturing(ctx);
  const int64_t room = nb->nnz / 64 + 4 * (total / 64 + nt) + nt * (kTileRows + 1) + 4;  // see k_tile_room
  if (!take_once(nb, nb->tperm_off, nt + 1, !cap) || !take_once(nb, nb->tperm, 64 * room, !cap) ||
      !take_once(nb, nb->tself, kTileRows * nt, !cap) || !take_once(nb, nb->gptr, n + 1, !cap) ||
      !take_once(nb, nb->gidx, total, !cap))
    return set_error(ctx, GF_ENOMEM, "transposed tile allocation failed");
  Arena ar;
  gf_status st;
  const int64_t nc = std::max(n, nt);
  if ((st = ensure_scratch(ctx, arena_bytes({sizeof(int32_t) * nc, sizeof(int64_t) * scan_tmp_elems(nc + 1),
                                             sizeof(int32_t) * total, sizeof(int32_t) * total}), &ar)))
    return st;
  int32_t *cnt = ar.take<int32_t>(nc);
  int64_t *tmp = ar.take<int64_t>(scan_tmp_elems(nc + 1));
  int32_t *rank = ar.take<int32_t>(total), *raw = ar.take<int32_t>(total);
  hipStream_t sm = ctx->stream;
  ProfScope prof(ctx, "tile_transpose");
  const TileRows tr = tile_rows(nb);
  hipLaunchKernelGGL(k_tile_room, dim3(grid_for(nt * kTileRows, kBlock)), dim3(kBlock), 0, sm, tr, nb->row_ptr,
                     nb->tile_off, nt, cnt);
  GF_LAUNCH_CHECK(ctx);
  if ((st = scan_i32_to_i64(ctx, cnt, nb->tperm_off, nt, tmp))) return st;
  const int most = std::max(nb->tile_max[0], nb->tile_max[1]);
  const size_t lds = sizeof(uint32_t) * most + sizeof(uint16_t) * ((most + 1) & ~1) +
                     sizeof(uint16_t) * 64 * (1 + 4 * ((most + 63) / 64) + kTileRows + kTileRows * (size_t)nb->max_row / 64);
  hipLaunchKernelGGL(k_tile_transpose, dim3((unsigned)nt), dim3(kBlock), lds, sm, tr, nb->row_ptr, nb->col, nb->slot,
                     nb->tile_off, nb->tperm_off, most, nb->tperm, nb->tself);
  hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, sm, cnt, n, 0);
  hipLaunchKernelGGL(k_places_count, dim3(grid_for(total, kBlock)), dim3(kBlock), 0, sm, nb->tile_u, total, nb->n_rows, cnt,
                     rank);
  GF_LAUNCH_CHECK(ctx);
  if ((st = scan_i32_to_i32(ctx, cnt, nb->gptr, n, (int32_t *)tmp))) return st;
  hipLaunchKernelGGL(k_places_fill, dim3(grid_for(total, kBlock)), dim3(kBlock), 0, sm, nb->tile_u, total, nb->n_rows,
                     nb->gptr, rank, raw);
  hipLaunchKernelGGL(k_places_sort, dim3(grid_for(n * 16, kBlock)), dim3(kBlock), 0, sm, nb->gptr, n, raw, nb->gidx);
  GF_LAUNCH_CHECK(ctx);
  if (!cap) nb->built |= gf_nbr::kTransposed;
  return GF_OK;
}

namespace {

// Cut the tiled groups into tiles and build slot[], tile_u[], tile_off[].
gf_status build_tiles(gf_ctx *ctx, gf_nbr *nb) {
  hipStream_t sm = ctx->stream;
  TileGroups tg;
  int64_t nt = 0, places = 0;
  for (int m = 0; m < 2; ++m) {
    nb->tile_start[m] = nt;
    const int64_t r0 = nb->group_start[m * GF_NBAND], r1 = nb->group_start[m * GF_NBAND + kTileBand + 1];
    if (r1 <= r0) continue;
    tg.gsel[tg.nq] = m;
    tg.tile_start[tg.nq] = nt;
    tg.row_start[tg.nq] = r0;
    tg.nrows[tg.nq] = r1 - r0;
    tg.uniq[tg.nq] = places;
    tg.entries[tg.nq] = kTileRows * std::min(nb->model_row[m], kTileBandRow);
    const int64_t k = (r1 - r0 + kTileRows - 1) / kTileRows;
    places += k * tg.entries[tg.nq];
    ++tg.nq;
    nt += k;
  }
  nb->tile_start[2] = nt;
  tg.tile_start[tg.nq] = nt;
  nb->ntiles = nt;
  if (nt == 0) return GF_OK;
  if (nt >= 0x7fffffff) return set_error(ctx, GF_ECAPACITY, "too many neighbour tiles");
  if (!take(nb, nb->slot, nb->nnz + kQuadPad) || !take(nb, nb->tile_off, nt + 1))
    return set_error(ctx, GF_ENOMEM, "neighbour tile allocation failed");
  Arena ar;
  std::vector<size_t> sz = {sizeof(int64_t) * scan_tmp_elems(nt + 1), sizeof(int32_t) * (size_t)places,
                            sizeof(int32_t) * nt, 64};
  gf_status st;
  if ((st = ensure_scratch(ctx, arena_bytes(sz), &ar))) return st;
  int64_t *tmp64 = ar.take<int64_t>(scan_tmp_elems(nt + 1));
  int32_t *uniq = ar.take<int32_t>((size_t)places);
  int32_t *cnt = ar.take<int32_t>(nt);
  int32_t *grp_max = ar.take<int32_t>(16);
  {
    ProfScope prof(ctx, "nbr_tile_unique");
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(kBlock), 0, sm, grp_max, (int64_t)16, 0);
    hipLaunchKernelGGL(k_tile_unique, dim3((unsigned)nt), dim3(kTileThreads), 0, sm, tg, nb->row_ptr, nb->col,
                       nb->grouped, nb->slot, uniq, cnt, grp_max);
    GF_LAUNCH_CHECK(ctx);
    if ((st = scan_i32_to_i64(ctx, cnt, nb->tile_off, nt, tmp64))) return st;
  }
  int64_t *hp = (int64_t *)ctx->host_pinned;
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, sm, grp_max, 2, nb->tile_off + nt, hp);
  GF_LAUNCH_CHECK(ctx);
  GF_HIP(ctx, hipStreamSynchronize(sm));
  for (int q = 0; q < tg.nq; ++q) nb->tile_max[tg.gsel[q]] = (int32_t)hp[q];  // per model
  const int64_t total = hp[2];
  nb->tile_total = total;
  if (!take(nb, nb->tile_u, total))
    return set_error(ctx, GF_ENOMEM, "neighbour tile list allocation failed");
  ProfScope prof(ctx, "nbr_tile_compact");
  hipLaunchKernelGGL(k_tile_compact, dim3(grid_for(nt, kBlock / 64)), dim3(kBlock), 0, sm, tg, nb->tile_off, uniq,
                     nt, nb->tile_u);
  GF_LAUNCH_CHECK(ctx);
  return GF_OK;
}

}  // namespace

extern "C" gf_status gf_build_neighbours(gf_ctx *ctx, const gf_particles *p, int cross_model, gf_nbr **out) {
  if (!ctx) return GF_EINVAL;
  if (!p) return set_error(ctx, GF_EINVAL, "particles are NULL");
  return gf_build_neighbours_rows(ctx, p, cross_model, p->n, out);
}

// the grid of each model's last (smallest-support) level alone: every
// particle of the model falls in its cells, which hold few particles each
static Grid finest_grid(const Grid &g) {
  Grid g1;
  memset(&g1, 0, sizeof(g1));
  int ns = 0;
  int64_t base = 0;
  for (int m = 0; m < 2; ++m) {
    g1.slot0[m] = ns;
    if (g.slot0[m + 1] > g.slot0[m]) {
      const int s = g.slot0[m + 1] - 1;
      for (int d = 0; d < 3; ++d) {
        g1.lo[ns][d] = g.lo[s][d];
        g1.dim[ns][d] = g.dim[s][d];
        g1.bits[ns][d] = g.bits[s][d];
      }
      g1.edge[ns] = g.edge[s];
      g1.inv_edge[ns] = g.inv_edge[s];
      g1.hcap[ns] = g.hcap[s];
      g1.base[ns] = base;
      base += (int64_t)1 << (g.bits[s][0] + g.bits[s][1] + g.bits[s][2]);
      ++ns;
    }
  }
  g1.slot0[2] = ns;
  g1.nslots = ns;
  g1.nkeys = base;
  return g1;
}

extern "C" gf_status gf_build_neighbours_rows(gf_ctx *ctx, const gf_particles *p, int cross_model, int64_t n_rows,
                                              gf_nbr **out) {
  if (!ctx) return GF_EINVAL;
  if (!out) return set_error(ctx, GF_EINVAL, "out is NULL");
  *out = nullptr;
  gf_status st = check_particles(ctx, p, false, false);
  if (st) return st;
  const int64_t n = p->n;
  if (n_rows < 0 || n_rows > n)
    return set_error(ctx, GF_EINVAL, "n_rows = %lld outside [0, %lld]", (long long)n_rows, (long long)n);
  hipStream_t sm = ctx->stream;

  // ---- bounding boxes and validation
  const int nblk = (int)std::min<int64_t>(kBboxBlocks, (n + kBboxThreads - 1) / kBboxThreads);
  Arena ar;
  std::vector<size_t> sz = {sizeof(double) * kBoxVals * nblk, sizeof(int) * nblk};
  if ((st = ensure_scratch(ctx, arena_bytes(sz), &ar))) return st;
  if ((st = ensure_host(ctx, 4096))) return st;
  double *part = ar.take<double>(kBoxVals * nblk);
  int *bad_part = ar.take<int>(nblk);
  double *hbox = (double *)ctx->host_pinned;
  int *hbad = (int *)((char *)ctx->host_pinned + 256);
  hipLaunchKernelGGL(k_bbox, dim3(nblk), dim3(kBboxThreads), 0, sm, p->x, p->y, p->z, p->h, p->model, n, part, bad_part);
  GF_LAUNCH_CHECK(ctx);
  hipLaunchKernelGGL(k_bbox_final, dim3(1), dim3(kBboxFin), 0, sm, part, bad_part, nblk, hbox, hbad);
  GF_LAUNCH_CHECK(ctx);
  GF_HIP(ctx, hipStreamSynchronize(sm));
  const int nbad = *hbad;
  if (nbad > 0)
    return set_error(ctx, GF_EINVAL, "%d particles have non-finite coordinates, h <= 0 or a model outside {0,1}", nbad);
  double bx[kBoxVals];
  memcpy(bx, hbox, sizeof(bx));

  // ---- grids: per model, levels with halving support caps (Grid); a grid's
  // edge is slightly above its cap so that rounding of the cell coordinate
  // never hides a neighbour
  Grid g;
  memset(&g, 0, sizeof(g));
  double lo[2][3], hi[2][3], hmx[2], hmn[2];
  for (int m = 0; m < 2; ++m) {
    for (int d = 0; d < 3; ++d) { lo[m][d] = bx[m * 8 + d]; hi[m][d] = bx[m * 8 + 3 + d]; }
    hmx[m] = bx[m * 8 + 6];
    hmn[m] = bx[m * 8 + 7];
  }
  const int64_t key_budget = std::max<int64_t>(4 * n, 1 << 16);  // per grid
  int64_t base = 0;
  int ns = 0;
  for (int m = 0; m < 2; ++m) {
    g.slot0[m] = ns;
    const bool empty = !(hmx[m] > 0.0);
    int L = 1;
    if (!empty)
      while (L < kMaxLevels && hmn[m] <= std::ldexp(hmx[m], -L)) ++L;
    for (int l = 0; l < L; ++l, ++ns) {
      g.hcap[ns] = empty ? 0.0 : std::ldexp(hmx[m], -l);
      double edge = empty ? 1.0 : g.hcap[ns] * (1.0 + 1e-9);
      for (int it = 0; it < 200; ++it) {
        int tb = 0;
        for (int d = 0; d < 3; ++d) {
          double span = empty ? 0.0 : hi[m][d] - lo[m][d];
          double dd = std::floor(span / edge) + 1.0;
          if (dd > kMaxAxis) dd = kMaxAxis;
          g.dim[ns][d] = (int)dd;
          g.bits[ns][d] = ceil_log2(g.dim[ns][d]);
          tb += g.bits[ns][d];
        }
        if (tb <= 30 && ((int64_t)1 << tb) <= key_budget) break;
        edge *= 1.5;
      }
      for (int d = 0; d < 3; ++d) g.lo[ns][d] = empty ? 0.0 : lo[m][d];
      g.edge[ns] = edge;
      g.inv_edge[ns] = 1.0 / edge;
      g.base[ns] = base;
      base += (int64_t)1 << (g.bits[ns][0] + g.bits[ns][1] + g.bits[ns][2]);
    }
  }
  g.slot0[2] = ns;
  g.nslots = ns;
  g.nkeys = base;
  if (g.nkeys >= (int64_t)0x7fffffff) return set_error(ctx, GF_ECAPACITY, "cell grid too large");

  // ---- sort particles into cells
  const int64_t K = g.nkeys;
  sz = {sizeof(int32_t) * n, sizeof(int32_t) * n, sizeof(int32_t) * (K + 1), sizeof(int32_t) * scan_tmp_elems(K + 1),
        sizeof(double4) * (n + kRowPad), sizeof(int32_t) * n, sizeof(int64_t) * scan_tmp_elems(n + 1),
        sizeof(int32_t) * 32, sizeof(int32_t) * n, sizeof(int32_t) * (n + 1), sizeof(int32_t) * scan_tmp_elems(n + 1),
        sizeof(int32_t) * n, sizeof(int4) * n, sizeof(int4) * n, sizeof(int4) * big_units(n),
        sizeof(int32_t) * (n + kRowPad)};
  // rows staged by the count pass (sw entries each, the widest that stays
  // under 8 GB); rows found longer are filled by a second search pass
  int sw = 0;
  for (int w : kStageWidths)
    if (sw == 0 && (double)n * w * sizeof(int32_t) <= 8e9) sw = w;
  const bool use_stage = sw > 0;
  if (use_stage) sz.push_back(sizeof(int32_t) * (size_t)n * sw);
  if ((st = ensure_scratch(ctx, arena_bytes(sz), &ar))) return st;
  int32_t *key = ar.take<int32_t>(n);
  int32_t *slot = ar.take<int32_t>(n);
  int32_t *cell_start = ar.take<int32_t>(K + 1);
  int32_t *tmp32 = ar.take<int32_t>(scan_tmp_elems(K + 1));
  double4 *sp = ar.take<double4>(n + kRowPad);
  int32_t *cnt = ar.take<int32_t>(n);
  int64_t *tmp64 = ar.take<int64_t>(scan_tmp_elems(n + 1));
  // hist[8], longest row per model [8], [9], search items, units and big units [10 .. 12], units and big units of the second order
  // [13], [14], particles per grid [16 .. 16 + kMaxSlots); zeroed before use
  int32_t *small = ar.take<int32_t>(32);
  int32_t *slot_count = small + 16;
  int32_t *gflag = ar.take<int32_t>(n);
  int32_t *gpos = ar.take<int32_t>(n + 1);
  int32_t *tmpg = ar.take<int32_t>(scan_tmp_elems(n + 1));
  int32_t *order1 = ar.take<int32_t>(n);  // model-wide cell order for the grouping (several levels)
  int4 *items = ar.take<int4>(n);
  int4 *units = ar.take<int4>(n);
  int4 *big = ar.take<int4>(big_units(n));
  int32_t *order = ar.take<int32_t>(n + kRowPad);  // particles in cell order
  int32_t *stage = use_stage ? ar.take<int32_t>((size_t)n * sw) : nullptr;

  gf_nbr *nb = new gf_nbr();
  nb->pool = ctx->pool;
  nb->device = ctx->device;
  nb->n = n;
  nb->n_rows = n_rows;
  nb->cross = cross_model ? 1 : 0;
  auto fail = [&](gf_status s2) { free_nbr(nb); return s2; };
  if (!device_alloc(*ctx->pool, &nb->waiter, 4096) || !take(nb, nb->row_ptr, n + 1) || !take(nb, nb->grouped, n))
    return fail(set_error(ctx, GF_ENOMEM, "neighbour handle allocation failed"));

  // The particles in the order of a grid's cells (fine Morton order inside them), the units and, with them, the
  // search items and the records of that order (sp).
  auto cell_order = [&](const Grid &gg, int32_t *ord, const CellLists &lists, double4 *recs, bool clear_small) {
    const int64_t KK = gg.nkeys;
    hipLaunchKernelGGL(k_clear, dim3(grid_for(KK + 1, kBlock)), dim3(kBlock), 0, sm, cell_start, KK + 1,
                       clear_small ? small : (int32_t *)nullptr);
    hipLaunchKernelGGL(k_keys, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, sm, p->x, p->y, p->z, p->h, p->model, n, gg,
                       key, slot, cell_start);
    gf_status s2 = scan_i32_to_i32(ctx, cell_start, cell_start, KK, tmp32);
    if (s2) return s2;
    hipLaunchKernelGGL(k_items, dim3(grid_for(KK, kItemsBlock)), dim3(kItemsBlock), 0, sm, cell_start, gg, kItemRows,
                       lists);
    int32_t *raw = gflag;  // (free until the grouping) the cells' particles in the order of their atomics
    hipLaunchKernelGGL(k_scatter, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, sm, key, slot, cell_start, n, raw);
    hipLaunchKernelGGL(k_cell_sort_small, dim3((unsigned)std::min<int64_t>(n / (8 * kCellSortWaves) + 1, 8 * ctx->num_cu)),
                       dim3(64 * kCellSortWaves), 0, sm, lists.units, lists.nunits, key, p->x, p->y, p->z, p->h, gg, raw,
                       ord, recs);
    hipLaunchKernelGGL(k_cell_sort_big, dim3((unsigned)std::min<int64_t>(n / kUnitSmall + 1, 4 * ctx->num_cu)),
                       dim3(kBlock), 0, sm, lists.big, lists.nbig, p->x, p->y, p->z, p->h, gg, raw, ord, recs);
    return hipGetLastError() == hipSuccess ? GF_OK : set_error(ctx, GF_EHIP, "cell order kernels failed");
  };
  {
  ProfScope prof_cells(ctx, "nbr_cells");
  const CellLists lists = {items, units, big, small + 10, small + 11, small + 12, slot_count};
  if ((st = cell_order(g, order, lists, sp, true))) return fail(st);
  }
  // as many blocks as fit at once (fewer on small clouds), a multiple of 8: dealt to the XCDs in turn
  const dim3 search_grid((unsigned)std::min<int64_t>((n / (2 * kSearchWaves) + 8) / 8 * 8,
                                                     (int64_t)ctx->num_cu * kSearchBlocksPerCu));
  {
  ProfScope prof_count(ctx, "nbr_count");
  hipLaunchKernelGGL(use_stage ? k_search<2> : k_search<0>, search_grid, dim3(kSearchBlock), 0, sm, order, sp,
                     cell_start, items, small + 10, slot_count, n_rows, g, cross_model ? 1 : 0, cnt, small, small + 8,
                     (const int64_t *)nullptr, (int32_t *)nullptr, stage, sw);
  }
  if (hipGetLastError() != hipSuccess) return fail(set_error(ctx, GF_EHIP, "count kernel launch failed"));
  if ((st = scan_i32_to_i64(ctx, cnt, nb->row_ptr, n, tmp64))) return fail(st);
  const int64_t *hs = (const int64_t *)ctx->host_pinned;  // histogram, longest rows, entries
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, sm, small, 10, nb->row_ptr + n, (int64_t *)ctx->host_pinned);
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(sm) != hipSuccess)
    return fail(set_error(ctx, GF_EHIP, "read-back of neighbour counts failed"));
  int64_t hist[2 * GF_NBAND];
  memcpy(hist, hs, sizeof(hist));
  // rows of the tiled bands are grouped together (under band kTileBand) so
  // that tiles stay spatially compact whatever the neighbour count
  for (int m = 0; m < 2; ++m)
    for (int band = 0; band < kTileBand; ++band) {
      hist[m * GF_NBAND + kTileBand] += hist[m * GF_NBAND + band];
      hist[m * GF_NBAND + band] = 0;
    }
  for (int m = 0; m < 2; ++m) nb->model_row[m] = (int32_t)hs[8 + m];
  nb->max_row = std::max(nb->model_row[0], nb->model_row[1]);
  nb->nnz = hs[10];
  if (nb->max_row > kMaxRow)
    return fail(set_error(ctx, GF_ECAPACITY, "a particle has %d neighbours; the limit is %d", nb->max_row, kMaxRow));
  if (nb->nnz >= (int64_t)1 << 40) return fail(set_error(ctx, GF_ECAPACITY, "too many neighbour pairs"));
  if (!take(nb, nb->col, nb->nnz))
    return fail(set_error(ctx, GF_ENOMEM, "neighbour list allocation (%lld entries) failed", (long long)nb->nnz));
  // staged rows need no fill pass; rows longer than sw (if any) are filled by one that
  // writes only those
  const bool staged = use_stage;
  if (!staged || nb->max_row > sw) {
    ProfScope prof_fill(ctx, "nbr_fill");
    hipLaunchKernelGGL(k_search<1>, search_grid, dim3(kSearchBlock), 0, sm, order, sp, cell_start, items,
                       small + 10, slot_count, n_rows, g, cross_model ? 1 : 0, (int32_t *)nullptr, (int32_t *)nullptr,
                       (int32_t *)nullptr, nb->row_ptr, nb->col, staged ? stage : (int32_t *)nullptr, sw);
  }
  {
    // staged rows: sorted on their way into the CSR; else sorted in place
    ProfScope prof_sort(ctx, "nbr_row_sort");
    // chunks of at most kSortChunk rows, fewer where the cloud would not give every SIMD eight waves
    int chunk = kSortChunk;
    while (chunk > 2 && n / chunk < (int64_t)ctx->num_cu * 32) chunk /= 2;
    const int64_t nchunks = (n + chunk - 1) / chunk;
    const dim3 sgrid((unsigned)std::max<int64_t>(1, std::min<int64_t>((nchunks + kSortWaves - 1) / kSortWaves, 4096)));
    const size_t lds = nb->max_row > 256 ? sizeof(int32_t) * kSortWaves * kMaxRow : 0;
    if (staged && nb->max_row > 128)
      hipLaunchKernelGGL((k_row_sort<true, true>), sgrid, dim3(kSortBlock), lds, sm, nb->row_ptr, nb->col, stage, sw, n,
                         chunk);
    else if (staged)
      hipLaunchKernelGGL((k_row_sort<false, true>), sgrid, dim3(kSortBlock), 0, sm, nb->row_ptr, nb->col, stage, sw, n,
                         chunk);
    else if (nb->max_row > 128)
      hipLaunchKernelGGL((k_row_sort<true, false>), sgrid, dim3(kSortBlock), lds, sm, nb->row_ptr, nb->col,
                         (const int32_t *)nullptr, 0, n, chunk);
    else
      hipLaunchKernelGGL((k_row_sort<false, false>), sgrid, dim3(kSortBlock), 0, sm, nb->row_ptr, nb->col,
                         (const int32_t *)nullptr, 0, n, chunk);
  }
  if (hipGetLastError() != hipSuccess) return fail(set_error(ctx, GF_EHIP, "fill/sort kernel launch failed"));

  // ---- groups by (model, band), Morton order kept inside each group.  The
  // cell order is level by level when a model has several support levels, so
  // a tile cut from it would gather particles of one level from a wide
  // region; the grouping then follows a model-wide order instead: the cells
  // of each model's smallest-support grid in Morton order, fine Morton key
  // inside each cell (the same kernels on a grid with one level per model).
  // The arrays of the first cell pass are free once the rows are written.
  const int32_t *gorder = order;
  if (g.slot0[1] - g.slot0[0] > 1 || g.slot0[2] - g.slot0[1] > 1) {
    ProfScope prof_o(ctx, "nbr_order");
    const Grid g1 = finest_grid(g);
    // (g1.nkeys <= K: its slots are slots of g)
    const CellLists lists = {nullptr, units, big, nullptr, small + 13, small + 14, slot_count};
    if ((st = cell_order(g1, order1, lists, nullptr, false))) return fail(st);
    gorder = order1;
  }
  int64_t off = 0;
  for (int gsel = 0; gsel < 2 * GF_NBAND; ++gsel) {
    nb->group_start[gsel] = off;
    off += hist[gsel];
  }
  nb->group_start[2 * GF_NBAND] = off;
  {
    ProfScope prof_group(ctx, "nbr_group");
    static_assert(kTileBand == 2 && GF_NBAND == 4 && kTileBandRow == 128, "one band of long rows per model");
    const dim3 gg(grid_for(n, kBlock)), gb(kBlock);
    if (nb->max_row <= kTileBandRow) {  // no long rows: the order is the grouping
      hipLaunchKernelGGL(k_copy_i32, gg, gb, 0, sm, gorder, n, nb->grouped);
    } else {
      hipLaunchKernelGGL(k_group_flag, gg, gb, 0, sm, gorder, cnt, n, gflag);
      if ((st = scan_i32_to_i32(ctx, gflag, gpos, n, tmpg))) return fail(st);
      hipLaunchKernelGGL(k_group_scatter, gg, gb, 0, sm, gorder, gflag, gpos, n, nb->group_start[GF_NBAND], hist[3],
                         hist[GF_NBAND + 3], nb->grouped);
    }
  }
  if (hipGetLastError() != hipSuccess) return fail(set_error(ctx, GF_EHIP, "grouping kernels failed"));
  if (off != n) return fail(set_error(ctx, GF_EHIP, "internal error: grouping covers %lld of %lld", (long long)off,
                                      (long long)n));
  if ((st = build_tiles(ctx, nb))) return fail(st);
  *out = nb;
  return GF_OK;
}
