// Implicit pressure-Poisson solve (projection scheme, Sec. 2.3) on the GFDM
// stencils: assembly of the matrix on the neighbour pattern, then
// right-preconditioned BiCGStab with the Jacobi preconditioner.
//
// The iteration runs as five fused kernels (direction update, SpMV + dot,
// intermediate update, SpMV + two dots, solution/residual update + two dots).
// Scalars (rho, alpha, omega, ...) stay on the device.  Every dot product is
// a deterministic two-level reduction: the kernels that produce it write one
// partial per block, and every block of the next vector update adds the
// partials up again, in block order, and derives the scalars itself (block 0
// keeps them for the kernels after it).  A one-block kernel per dot product
// took 4.7 us and a gap each, three times per iteration.  The kernel boundary
// makes the partials visible (no device-scope fences: on a chip whose XCDs have
// separate L2 caches each such fence writes back an L2).  The host reads the
// residual norm every few iterations, behind a one-block kernel of its own.
//
// The matrix of the tiled rows is kept packed (PackedTiles): the values in the
// order in which the waves of the SpMV read them.
//
// Mixed modes.  mixed = 1: one BiCGStab run whose SpMV reads FP32 matrix
// values (4 instead of 8 bytes per entry) while the Krylov vectors, dots and
// updates stay FP64; its recursive residual tracks b - A32 x, so whenever it
// has fallen by kReplace since the last replacement (and when it reaches the
// tolerance) it is replaced by the FP64 residual b - A64 x (residual
// replacement, a form of iterative refinement that keeps the Krylov space:
// no restart).  mixed = 2: iterative refinement with restarts: the residual
// r = b - A64 x in FP64, then an inner BiCGStab on FP32 values and FP32
// vectors (dots accumulated in FP64) solves A32 d = r from d = 0 to a
// relative reduction inner_rtol, and x += d.
#include <algorithm>
#include <chrono>
#include <cstring>

#include "stencil_common.h"

using namespace gfdm_dev;

namespace {
constexpr int kBlock = 256;
constexpr int kTeam = 8;
static_assert(kBlock / kTeam == kTileRows, "one team per row of a neighbour tile");

struct Scal {
  // rho, rho_old: of the last iteration whose scalars are final; rho_next: of the iteration under way
  double rho, rho_old, rho_next, alpha, omega, rv, ts, tt, rr, bb;
  // codes of a breakdown, zero if none: of the last finished iteration, and as found by the two updates
  // before its end.  A kernel never reads the one that it writes, so that all its threads decide alike.
  int breakdown, bd_p, bd_s;
  int half;  // the half step solved the system (t = A shat = 0)
};

// ---------------------------------------------------------------- reductions
__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
constexpr int kRedBlocks = 2048;   // blocks of the SpMV kernels, at most
constexpr int kVecBlocks = 512;    // blocks of the vector updates, at most: every one adds up all partials
constexpr double kReplace = 1e-2;  // mixed = 1: residual replacement after this reduction
constexpr int kFinThreads = 1024;  // threads of the finishing kernels

// sums over the block of BS threads, on every thread
template <int BS, int NV>
__device__ inline void block_sums(double v[NV]) {
  __shared__ double sh[NV][BS / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) sh[k][wid] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < BS / 64; ++w) r += sh[k][w];
    v[k] = r;
  }
}

// one partial per block and value: part[k * gridDim.x + blockIdx.x]
template <int BS, int NV>
__device__ inline void block_partials(double v[NV], double *part) {
  block_sums<BS, NV>(v);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) part[(int64_t)k * gridDim.x + blockIdx.x] = v[k];
  }
}

// sums of the partials of nblk blocks, on every thread (the same in every block of BS threads)
template <int BS, int NV>
__device__ inline void finish_partials(const double *part, int nblk, double res[NV]) {
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double acc = 0.0;
    for (int b = threadIdx.x; b < nblk; b += BS) acc += part[(int64_t)k * nblk + b];
    res[k] = acc;
  }
  block_sums<BS, NV>(res);
}

// ---------------------------------------------------------------- assembly
struct AsmArgs {
  const int64_t *row_ptr;
  const int32_t *col;
  const double *w;
  const int8_t *row_type;
  const double *h, *nx, *ny, *nz;
  double zeta, a;
  int max_type;
  double *dinv64;
  float *dinv32;
  int *bad;
};
struct RowKind {
  int rt;
  double nrm[3], zf;
};
__device__ inline RowKind row_kind(const AsmArgs &g, int64_t i) {
  RowKind r;
  r.rt = g.row_type[i];
  r.nrm[0] = r.nrm[1] = r.nrm[2] = 0.0;
  if (r.rt == GF_ROW_NEUMANN_COMBINED || r.rt == GF_ROW_NEUMANN) { r.nrm[0] = g.nx[i]; r.nrm[1] = g.ny[i]; r.nrm[2] = g.nz[i]; }
  r.zf = g.zeta / g.h[i];
  return r;
}
// the matrix value of an entry from its stencils (d/dx, d/dy), (d/dz, Laplacian)
__device__ inline double entry_value(const AsmArgs &g, const RowKind &r, const double2 &g01, const double2 &g23, bool self) {
  const double ngrad = r.nrm[0] * g01.x + r.nrm[1] * g01.y + r.nrm[2] * g23.x;
  switch (r.rt) {
    case GF_ROW_INTERIOR: return g23.y;
    case GF_ROW_DIRICHLET: return self ? 1.0 : 0.0;
    case GF_ROW_NEUMANN_COMBINED: return g23.y + r.zf * ngrad;
    case GF_ROW_IMPLICIT: return (self ? 1.0 : 0.0) - g.a * g23.y;
    default: return ngrad;
  }
}
// diag: the self value on the lane that holds it, zero on the others
__device__ inline void finish_assembled_row(const AsmArgs &g, int64_t i, int rt, double diag, int lane) {
  diag = team_sum(diag, kTeam);  // exactly the self value: the other lanes add zeros
  if (lane == 0) {
    if (rt < 0 || rt > g.max_type || diag == 0.0 || !isfinite(diag)) atomicAdd(g.bad, 1);
    if (g.dinv64) g.dinv64[i] = (diag != 0.0) ? 1.0 / diag : 0.0;
    if (g.dinv32) g.dinv32[i] = (diag != 0.0) ? (float)(1.0 / diag) : 0.0f;
  }
}

// One team of kTeam lanes per row (grid-stride) of the list `rows` (NULL: all
// rows): the row's values in CSR order, its diagonal (found by the lane holding
// the self entry) and the Jacobi inverse.
__global__ void __launch_bounds__(kBlock) k_assemble(AsmArgs g, const int32_t *__restrict__ rows, int64_t nrows,
                                                     double *__restrict__ val64, float *__restrict__ val32) {
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = (int)(gt % kTeam);
  const int64_t nteams = (int64_t)gridDim.x * blockDim.x / kTeam;
  for (int64_t q = gt / kTeam; q < nrows; q += nteams) {
    const int64_t i = rows ? rows[q] : q;
    const RowKind rk = row_kind(g, i);
    double diag = 0.0;  // nonzero only on the lane that holds the self entry
    for (int64_t k = g.row_ptr[i] + lane; k < g.row_ptr[i + 1]; k += kTeam) {
      const double2 *p = reinterpret_cast<const double2 *>(g.w) + 2 * k;
      const bool self = g.col[k] == i;
      const double v = entry_value(g, rk, p[0], p[1], self);
      if (val64) val64[k] = v;
      if (val32) val32[k] = (float)v;
      if (self) diag = v;
    }
    finish_assembled_row(g, i, rk.rt, diag, lane);
  }
}

// ---------------------------------------------------------------- packed tiles
// The matrix of the tiled rows, in the order in which the SpMV reads it.  A tile's
// 32 rows are taken in order of falling length (prow: the row of each of its 32
// teams, -1 none) in four groups of eight, one per wave of the SpMV's block.  A
// group's entries fill q = ceil(longest row / 8) units of 64 entries, from unit
// goff[group]: chunk c (two units) holds entries 16 c + 2 l and 16 c + 2 l + 1 of
// the row of lane 8 t + l at places 2 (8 t + l) and 2 (8 t + l) + 1, and the last
// unit of an odd q one entry per lane.  Places past a row's end hold value 0 and
// slot 0.  So every load of a wave covers 1,024 (values) or 256 (slots) bytes in
// one piece, where rows read at their CSR places took two loads of 16 bytes at a
// stride of 32 for lines that start anywhere.  As the rows are sorted, a tile's
// groups after the first are padded by less than the group before them holds, so
// that all groups fit in nnz + ntiles (8 longest + 4 x 56) entries.
struct PackedTiles {
  const int64_t *goff;
  const int32_t *prow;
  const uint16_t *slot;
};
constexpr int kGroups = kTileRows / 8;

// a wave per tile: rows by falling length (ties by place), group lengths
__global__ void __launch_bounds__(kBlock) k_pack_rows(TileRows tr, const int64_t *__restrict__ row_ptr,
                                                      int32_t *__restrict__ prow, int32_t *__restrict__ gq) {
  const int64_t t = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= tr.tile_start[2]) return;
  const int32_t i = lane < kTileRows ? tile_row(tr, t, lane) : -1;
  const int len = i >= 0 ? (int)(row_ptr[i + 1] - row_ptr[i]) : 0;
  int rank = 0;
#pragma unroll
  for (int o = 0; o < kTileRows; ++o) {
    const int lo = __builtin_amdgcn_readlane(len, o);
    rank += (lo > len || (lo == len && o < lane)) ? 1 : 0;
  }
  if (lane < kTileRows) {
    prow[kTileRows * t + rank] = i;
    if (rank % 8 == 0) gq[kGroups * t + rank / 8] = (len + 7) / 8;
  }
}

// a team per packed row (grid-stride): values and slots at their packed places
__global__ void __launch_bounds__(kBlock) k_assemble_packed(AsmArgs g, const int64_t *__restrict__ goff,
                                                            const int32_t *__restrict__ prow, int64_t nteamrows,
                                                            const uint16_t *__restrict__ slot,
                                                            double *__restrict__ val64, float *__restrict__ val32,
                                                            uint16_t *__restrict__ pslot) {
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = (int)(gt % kTeam);
  const int64_t nteams = (int64_t)gridDim.x * blockDim.x / kTeam;
  for (int64_t q = gt / kTeam; q < nteamrows; q += nteams) {
    const int32_t i = prow[q];
    const int64_t u0 = goff[q / 8], u1 = goff[q / 8 + 1];
    const int units = (int)(u1 - u0), l64 = (int)(q % 8) * 8 + lane;
    const int64_t b = i >= 0 ? g.row_ptr[i] : 0;
    const int len = i >= 0 ? (int)(g.row_ptr[i + 1] - b) : 0;
    RowKind rk;
    rk.rt = 0;
    if (i >= 0) rk = row_kind(g, i);
    double diag = 0.0;
    auto entry = [&](int e, double &v, uint16_t &s) {
      v = 0.0;
      s = 0;
      if (e < len) {
        const int64_t k = b + e;
        const double2 *p = reinterpret_cast<const double2 *>(g.w) + 2 * k;
        const bool self = g.col[k] == i;
        v = entry_value(g, rk, p[0], p[1], self);
        s = slot[k];
        if (self) diag = v;
      }
    };
    for (int c = 0; 2 * c + 1 < units; ++c) {
      double va, vb;
      uint16_t sa, sb;
      entry(16 * c + 2 * lane, va, sa);
      entry(16 * c + 2 * lane + 1, vb, sb);
      const int64_t at = 64 * u0 + 128 * c + 2 * l64;
      *reinterpret_cast<double2 *>(val64 + at) = make_double2(va, vb);
      if (val32) *reinterpret_cast<float2 *>(val32 + at) = make_float2((float)va, (float)vb);
      *reinterpret_cast<ushort2 *>(pslot + at) = make_ushort2(sa, sb);
    }
    if (units & 1) {
      double v;
      uint16_t sl;
      entry(8 * (units - 1) + lane, v, sl);
      const int64_t at = 64 * (u1 - 1) + l64;
      val64[at] = v;
      if (val32) val32[at] = (float)v;
      pslot[at] = sl;
    }
    if (i >= 0) finish_assembled_row(g, i, rk.rt, diag, lane);
  }
}

// ---------------------------------------------------------------- kernels
// Rows are taken by teams of kTeam lanes, grid-stride over the fixed grid.
#define GF_TEAM_ROWS(row)                                                              \
  const int64_t gt_ = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;                 \
  const int lane = (int)(gt_ % kTeam);                                                 \
  const int64_t nteams_ = (int64_t)gridDim.x * blockDim.x / kTeam;                     \
  for (int64_t row = gt_ / kTeam; row < n; row += nteams_)

// r = b - A x (FP64), optionally rhat = r; partials of (r,r) and (b,b)
__global__ void __launch_bounds__(kBlock) k_residual(const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                                                     const double *__restrict__ val, const double *__restrict__ b,
                                                     const double *__restrict__ x, int64_t n, double *__restrict__ r,
                                                     double *__restrict__ rhat, double *part) {
  double v[2] = {0.0, 0.0};
  GF_TEAM_ROWS(row) {
    double acc = 0.0;
    for (int64_t k = row_ptr[row] + lane; k < row_ptr[row + 1]; k += kTeam) acc += val[k] * x[col[k]];
    acc = team_sum(acc, kTeam);
    if (lane == 0) {
      const double ri = b[row] - acc;
      r[row] = ri;
      if (rhat) rhat[row] = ri;
      v[0] += ri * ri;
      v[1] += b[row] * b[row];
    }
  }
  block_partials<kBlock, 2>(v, part);
}

// residual replacement: r = b - A x with FP64 values; partials of (r, r) and
// (rhat, r), so that rho continues from the replaced residual
__global__ void __launch_bounds__(kBlock) k_residual_replace(const int64_t *__restrict__ row_ptr,
                                                             const int32_t *__restrict__ col,
                                                             const double *__restrict__ val, const double *__restrict__ b,
                                                             const double *__restrict__ x, const double *__restrict__ rhat,
                                                             int64_t n, double *__restrict__ r, double *part) {
  double v[2] = {0.0, 0.0};
  GF_TEAM_ROWS(row) {
    double acc = 0.0;
    for (int64_t k = row_ptr[row] + lane; k < row_ptr[row + 1]; k += kTeam) acc += val[k] * x[col[k]];
    acc = team_sum(acc, kTeam);
    if (lane == 0) {
      const double ri = b[row] - acc;
      r[row] = ri;
      v[0] += ri * ri;
      v[1] += rhat[row] * ri;
    }
  }
  block_partials<kBlock, 2>(v, part);
}

__global__ void __launch_bounds__(kFinThreads) k_fin_replace(const double *part, int nblk, Scal *S, Scal *host) {
  double res[2];
  finish_partials<kFinThreads, 2>(part, nblk, res);
  if (threadIdx.x != 0) return;
  S->rr = res[0];
  S->rho = res[1];  // rho_old keeps the value of the last iteration
  if (res[1] == 0.0 || !isfinite(res[1])) S->breakdown = 4;
  *host = *S;
}

// scalars after a residual: rr, bb; with reset, a fresh BiCGStab start (rhat = r)
__global__ void __launch_bounds__(kFinThreads) k_fin_residual(const double *part, int nblk, Scal *S, int reset, Scal *host) {
  double res[2];
  finish_partials<kFinThreads, 2>(part, nblk, res);
  if (threadIdx.x != 0) return;
  S->rr = res[0];
  S->bb = res[1];
  if (reset) {
    S->rho = res[0];
    S->rho_old = 1.0;
    S->alpha = 1.0;
    S->omega = 1.0;
    S->breakdown = S->bd_p = S->bd_s = 0;
    S->half = 0;
  }
  *host = *S;
}

// x32 = (float) r64; rhat32 = x32; p = v = 0; partial of (r,r)
template <typename XT>
__global__ void __launch_bounds__(kBlock) k_inner_init(const double *__restrict__ r64, int64_t n, XT *__restrict__ r,
                                                       XT *__restrict__ rhat, XT *__restrict__ p, XT *__restrict__ vv,
                                                       XT *__restrict__ x, double *part) {
  double v[1] = {0.0};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const XT ri = (XT)r64[i];
    r[i] = ri;
    rhat[i] = ri;
    p[i] = (XT)0;
    vv[i] = (XT)0;
    x[i] = (XT)0;
    v[0] += (double)ri * (double)ri;
  }
  block_partials<kBlock, 1>(v, part);
}

__global__ void __launch_bounds__(kFinThreads) k_fin_inner_init(const double *part, int nblk, Scal *S) {
  double res[1];
  finish_partials<kFinThreads, 1>(part, nblk, res);
  if (threadIdx.x != 0) return;
  S->rr = res[0];
  S->rho = res[0];
  S->rho_old = 1.0;
  S->alpha = 1.0;
  S->omega = 1.0;
  S->breakdown = S->bd_p = S->bd_s = 0;
  S->half = 0;
}

template <typename XT>
__global__ void __launch_bounds__(kBlock) k_zero_vecs(int64_t n, XT *a, XT *b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) { a[i] = (XT)0; b[i] = (XT)0; }
}

// The vector updates take the scalars that the dots before them give: nblk > 0
// partials in `part`, added up by every block (all get the same sums), or, with
// nblk = 0, the scalars as they stand in S.  Block 0 writes them down, in places
// that no thread of the same kernel reads.

// p = r + beta (p - omega v); phat = p * dinv.  part: (rhat, r), (r, r) of the iteration before.
template <int BS, typename XT>
__global__ void __launch_bounds__(BS) k_update_p(const XT *__restrict__ r, const XT *__restrict__ vv,
                                                 const XT *__restrict__ dinv, int64_t n, XT *__restrict__ p,
                                                 XT *__restrict__ phat, Scal *S, const double *part, int nblk) {
  const bool first = blockIdx.x == 0 && threadIdx.x == 0;
  int bd = S->breakdown;
  double rho = S->rho, rho_old = S->rho_old;
  const double alpha = S->alpha, omega = S->omega;
  const int half = S->half;
  if (!bd && nblk > 0) {
    double res[2];
    finish_partials<BS, 2>(part, nblk, res);
    rho_old = rho;
    rho = res[0];
    bd = half ? 5 : ((rho == 0.0 || !isfinite(rho)) ? 4 : 0);
    if (first) S->rr = res[1];
  }
  if (first) {
    S->rho_next = rho;
    S->bd_p = bd;
  }
  if (bd) return;
  const double beta = (rho / rho_old) * (alpha / omega);
  for (int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x; i < n; i += (int64_t)gridDim.x * BS) {
    const double pi = (double)r[i] + beta * ((double)p[i] - omega * (double)vv[i]);
    p[i] = (XT)pi;
    phat[i] = (XT)(pi * (double)dinv[i]);
  }
}

// y = A xin; partials of (other, y) and (y, y)
template <typename VT, typename XT>
__global__ void __launch_bounds__(kBlock) k_spmv_dot(const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                                                     const VT *__restrict__ val, const XT *__restrict__ xin, int64_t n,
                                                     XT *__restrict__ y, const XT *__restrict__ other, double *part,
                                                     const int *__restrict__ stop) {
  double v[2] = {0.0, 0.0};
  if (!*stop) {
    GF_TEAM_ROWS(row) {
      double acc = 0.0;
      for (int64_t k = row_ptr[row] + lane; k < row_ptr[row + 1]; k += kTeam) acc += (double)val[k] * (double)xin[col[k]];
      acc = team_sum(acc, kTeam);
      if (lane == 0) {
        const XT yi = (XT)acc;
        y[row] = yi;
        v[0] += (double)other[row] * (double)yi;
        v[1] += (double)yi * (double)yi;
      }
    }
  }
  block_partials<kBlock, 2>(v, part);
}

// two values in one load
template <typename T> struct Vec2;
template <> struct Vec2<double> { typedef double type __attribute__((ext_vector_type(2))); };
template <> struct Vec2<float> { typedef float type __attribute__((ext_vector_type(2))); };

// Neighbour tiles of the matrix pattern (the neighbour handle's tiles) and the
// packed matrix on them; rows with more than kTileBandRow entries are listed per
// model in grouped[b3_start[m] .. + b3_n[m]) and keep CSR values.
struct SpmvTiles {
  const int64_t *toff;
  const int32_t *tu;
  const int32_t *grouped;
  int64_t ntiles;
  int64_t b3_start[2], b3_n[2];
  int cap;  // LDS entries of the staged vector
  PackedTiles pk;
};

// What a SpMV does with y_i = (A xin)_i and which two dots it adds up:
//  kDots    y_i -> y;            (other, y), (y, y)
//  kResid   b_i - y_i -> y (and y2 if given);  (r, r), (b, b)        b = other
//  kReplace b_i - y_i -> y;      (r, r), (rhat, r)                   b = other, rhat = other2
enum { kDots = 0, kResid = 1, kReplaced = 2 };

// y = A xin over tiles.  The tiles are cut into eight contiguous slices,
// one per XCD (blocks are dealt to the XCDs in turn, so block b runs on
// XCD b mod 8 and neighbouring tiles, which share most of their lists,
// meet in one L2); the G = gridDim.x / 8 blocks of a slice walk it with
// stride G.  Each wave takes a group of eight packed rows (a team of kTeam lanes
// each), loads all its values and slots before it uses any, and reads the
// entries of xin from LDS through the slots; tiles whose list exceeds the LDS
// capacity gather through the tile list.  Then the untiled rows, a wave each.
//
// The walk is software-pipelined so that a tile costs about one memory
// latency instead of the chain tile offset -> tile list -> xin gather and
// group offset -> values: while the rows of tile t are summed from one LDS
// buffer, the loads for the following tiles are in flight: the xin entries
// of t+G (held in registers, written to the other buffer at the end of the
// step), the tile lists of t+2G, the tile offsets of t+3G, the group offsets and
// rows of t+G.  None of them depends on a load of the same step.  One barrier per
// tile separates the buffers.
// K = staged entries per thread (K * kBlock >= LDS capacity).
//
// What bounds it: HBM (10 bytes per entry in FP64, 6 with FP32 values).  A
// product of the 401,320-row cylinder (42.1M entries) takes 81 us, 5.2 TB/s of
// matrix (NT: non-temporal loads, see launch_spmv_tiles; 100 us without); 114 us
// with rows at their CSR places.  On a 25k-row plate 8 us against 19: its rows
// of more than 128 entries took 19 dependent gathers on eight lanes.
constexpr int kChunks = kTileBandRow / 16;  // chunks of a group, at most

template <typename VT, typename XT, int K, int EPI, bool NT>
__global__ void __launch_bounds__(kBlock) k_spmv_tiles(const int64_t *__restrict__ row_ptr,
                                                       const int32_t *__restrict__ col, const VT *__restrict__ val,
                                                       const VT *__restrict__ pval, const XT *__restrict__ xin,
                                                       XT *__restrict__ y, XT *__restrict__ y2,
                                                       const XT *__restrict__ other, const XT *__restrict__ other2,
                                                       double *part, const int *__restrict__ stop, SpmvTiles tl) {
  extern __shared__ unsigned char s_raw[];
  XT *sb = reinterpret_cast<XT *>(s_raw);  // two buffers of tl.cap entries
  double v[2] = {0.0, 0.0};
  const int lane64 = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  auto finish_row = [&](int32_t row, double acc) {
    if constexpr (EPI == kDots) {
      const XT yi = (XT)acc;
      y[row] = yi;
      v[0] += (double)other[row] * (double)yi;
      v[1] += (double)yi * (double)yi;
    } else {
      const double b = (double)other[row], r = b - acc;
      y[row] = (XT)r;
      if (EPI == kResid && y2) y2[row] = (XT)r;
      v[0] += r * r;
      v[1] += EPI == kResid ? b * b : (double)other2[row] * r;
    }
  };
  if (EPI != kDots || !*stop) {
    const int nslice = gridDim.x % 8 == 0 ? 8 : 1;
    const int slice = blockIdx.x % nslice;
    const int64_t G = gridDim.x / nslice;
    const int64_t nt = tl.ntiles * (slice + 1) / nslice;  // end of this block's slice
    const int cap = tl.cap;
    // list offset and length of tile t (length -1 past the last tile)
    auto extent = [&](int64_t t, int64_t &u0, int &cnt) {
      if (t < nt) {
        u0 = tl.toff[t];
        cnt = (int)(tl.toff[t + 1] - u0);
      } else {
        u0 = 0;
        cnt = -1;
      }
    };
    // this thread's share of a staged tile's list (-1: nothing)
    auto load_list = [&](int64_t u0, int cnt, int32_t idx[K]) {
      const bool staged = cnt >= 0 && cnt <= cap;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int s = threadIdx.x + j * kBlock;
        idx[j] = (staged && s < cnt) ? tl.tu[u0 + s] : -1;
      }
    };
    // this wave's group of tile t: its first unit, its units (0 past the slice), this team's row (-1: none)
    auto group = [&](int64_t t, int64_t &o, int &units, int32_t &row) {
      o = 0;
      units = 0;
      row = -1;
      if (t < nt) {
        o = tl.pk.goff[kGroups * t + w];
        units = (int)(tl.pk.goff[kGroups * t + w + 1] - o);
        row = tl.pk.prow[kTileRows * t + 8 * w + lane64 / kTeam];
      }
    };
    auto gather = [&](const int32_t idx[K], XT xv[K]) {
#pragma unroll
      for (int j = 0; j < K; ++j) xv[j] = idx[j] >= 0 ? xin[idx[j]] : (XT)0;
    };
    auto put = [&](XT *buf, const XT xv[K], int cnt) {
      if (cnt < 0 || cnt > cap) return;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int s = threadIdx.x + j * kBlock;
        if (s < cnt) buf[s] = xv[j];
      }
    };

    // prologue: tile t staged, the loads of t+G and t+2G issued
    int64_t t = tl.ntiles * slice / nslice + blockIdx.x / nslice;
    int64_t u0_0, u0_1, u0_2, o_c, o_n;
    int c0, c1, c2, q_c, q_n;
    int32_t row_c, row_n;
    extent(t, u0_0, c0);
    extent(t + G, u0_1, c1);
    extent(t + 2 * G, u0_2, c2);
    group(t, o_c, q_c, row_c);
    int32_t idx1[K];
    {
      int32_t idx0[K];
      XT x0[K];
      load_list(u0_0, c0, idx0);
      gather(idx0, x0);
      put(sb, x0, c0);
    }
    load_list(u0_1, c1, idx1);
    __syncthreads();
    int cur = 0;
    for (; t < nt; t += G) {
      // the group's values and slots, the first to be needed
      typename Vec2<VT>::type va[kChunks];
      ushort2 ss[kChunks];
      VT vt = (VT)0;
      uint16_t st = 0;
      const VT *pv = pval + 64 * o_c;
      const uint16_t *ps = tl.pk.slot + 64 * o_c;
#pragma unroll
      for (int c = 0; c < kChunks; ++c)
        if (2 * c + 1 < q_c) {
          const auto *a = reinterpret_cast<const typename Vec2<VT>::type *>(pv + 128 * c) + lane64;
          const uint32_t *b = reinterpret_cast<const uint32_t *>(ps + 128 * c) + lane64;
          if constexpr (NT) {
            va[c] = __builtin_nontemporal_load(a);
            ss[c] = __builtin_bit_cast(ushort2, __builtin_nontemporal_load(b));
          } else {
            va[c] = *a;
            ss[c] = __builtin_bit_cast(ushort2, *b);
          }
        }
      if (q_c & 1) {
        vt = pv[64 * (q_c - 1) + lane64];
        st = ps[64 * (q_c - 1) + lane64];
      }
      XT xn[K];
      gather(idx1, xn);  // entries of t+G
      int32_t idx2[K];
      load_list(u0_2, c2, idx2);  // list of t+2G
      int64_t u0_3;
      int c3;
      extent(t + 3 * G, u0_3, c3);
      group(t + G, o_n, q_n, row_n);
      double acc = 0.0;
      if (c0 <= cap) {
        const XT *buf = sb + cur * cap;
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
          if (2 * c + 1 < q_c) {
            acc = fma((double)va[c].x, (double)buf[ss[c].x], acc);
            acc = fma((double)va[c].y, (double)buf[ss[c].y], acc);
          }
        if (q_c & 1) acc = fma((double)vt, (double)buf[st], acc);
      } else {
        const int32_t *list = tl.tu + u0_0;
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
          if (2 * c + 1 < q_c) {
            acc = fma((double)va[c].x, (double)xin[list[ss[c].x]], acc);
            acc = fma((double)va[c].y, (double)xin[list[ss[c].y]], acc);
          }
        if (q_c & 1) acc = fma((double)vt, (double)xin[list[st]], acc);
      }
      acc = team_sum(acc, kTeam);
      if (lane64 % kTeam == 0 && row_c >= 0) finish_row(row_c, acc);
      put(sb + (cur ^ 1) * cap, xn, c1);
      __syncthreads();
      cur ^= 1;
      u0_0 = u0_1; c0 = c1;
      u0_1 = u0_2; c1 = c2;
      u0_2 = u0_3; c2 = c3;
#pragma unroll
      for (int j = 0; j < K; ++j) idx1[j] = idx2[j];
      o_c = o_n; q_c = q_n; row_c = row_n;
    }
    // untiled rows: waves grid-stride over each model's list, four entries per lane in flight
    const int64_t gw = (int64_t)blockIdx.x * (kBlock / 64) + w, nw = (int64_t)gridDim.x * (kBlock / 64);
    for (int m = 0; m < 2; ++m) {
      for (int64_t q = gw; q < tl.b3_n[m]; q += nw) {
        const int32_t row = tl.grouped[tl.b3_start[m] + q];
        const int64_t b = row_ptr[row], e = row_ptr[row + 1];
        double acc = 0.0;
        for (int64_t k = b + lane64; k < e; k += 4 * 64) {
          VT vv[4];
          XT xx[4];
          int32_t cc[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int64_t kk = min(k + 64 * u, e - 1);  // (past the end: the last entry, not added)
            cc[u] = col[kk];
            vv[u] = val[kk];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) xx[u] = xin[cc[u]];
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (k + 64 * u < e) acc = fma((double)vv[u], (double)xx[u], acc);
        }
        acc = wave_sum(acc);
        if (lane64 == 0) finish_row(row, acc);
      }
    }
  }
  block_partials<kBlock, 2>(v, part);
}

// s = r - alpha v; shat = s * dinv; alpha = rho / (rhat, v).  part: (rhat, v) first.
template <int BS, typename XT>
__global__ void __launch_bounds__(BS) k_update_s(const XT *__restrict__ r, const XT *__restrict__ vv,
                                                 const XT *__restrict__ dinv, int64_t n, XT *__restrict__ s,
                                                 XT *__restrict__ shat, Scal *S, const double *part, int nblk) {
  const bool first = blockIdx.x == 0 && threadIdx.x == 0;
  const int before = S->bd_p;
  if (before) {
    if (first) S->bd_s = before;
    return;
  }
  const double rho = S->rho_next;
  double res[1];
  finish_partials<BS, 1>(part, nblk, res);
  const double rv = res[0], alpha = rho / rv;
  const bool bad = rv == 0.0 || !isfinite(rv);
  if (first) {
    S->rv = rv;
    S->rho = rho;
    if (!bad) S->alpha = alpha;
    S->bd_s = bad ? 1 : 0;
  }
  if (bad) return;
  for (int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x; i < n; i += (int64_t)gridDim.x * BS) {
    const double si = (double)r[i] - alpha * (double)vv[i];
    s[i] = (XT)si;
    shat[i] = (XT)(si * (double)dinv[i]);
  }
}

// x += alpha phat + omega shat; r = s - omega t; omega = (t, s) / (t, t); partials of (rhat, r),
// (r, r) to `out`.  part: (t, s), (t, t).
template <int BS, typename XT>
__global__ void __launch_bounds__(BS) k_update_xr(const XT *__restrict__ phat, const XT *__restrict__ shat,
                                                  const XT *__restrict__ s, const XT *__restrict__ t,
                                                  const XT *__restrict__ rhat, int64_t n, XT *__restrict__ x,
                                                  XT *__restrict__ r, Scal *S, const double *part, int nblk,
                                                  double *out) {
  double v[2] = {0.0, 0.0};
  const bool first = blockIdx.x == 0 && threadIdx.x == 0;
  const int before = S->bd_s;
  if (before) {
    if (first) S->breakdown = before;
  } else {
    const double al = S->alpha;
    double res[2];
    finish_partials<BS, 2>(part, nblk, res);
    double om = 0.0;
    int bd = 0, half = 0;
    if (res[1] == 0.0) {
      // t = A shat = 0, so s = 0 for a nonsingular A: x + alpha phat already
      // solves the system.  Take that step (omega = 0) and restart from the
      // true residual afterwards (code 5).
      half = 1;
    } else if (!isfinite(res[1])) {
      bd = 2;
    } else {
      om = res[0] / res[1];
      if (om == 0.0) bd = 3;
    }
    if (first) {
      S->ts = res[0];
      S->tt = res[1];
      if (bd != 2) S->omega = om;
      if (half) S->half = 1;
      S->breakdown = bd;
    }
    if (bd == 0) {
      for (int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x; i < n; i += (int64_t)gridDim.x * BS) {
        x[i] = (XT)((double)x[i] + al * (double)phat[i] + om * (double)shat[i]);
        const double ri = (double)s[i] - om * (double)t[i];
        r[i] = (XT)ri;
        v[0] += (double)rhat[i] * (double)(XT)ri;
        v[1] += (double)(XT)ri * (double)(XT)ri;
      }
    }
  }
  block_partials<BS, 2>(v, out);
}

// the scalars after an iteration, for the host's check (the next direction update then takes them from S)
__global__ void __launch_bounds__(kFinThreads) k_fin_xr(const double *part, int nblk, Scal *S, Scal *host) {
  double res[2];
  finish_partials<kFinThreads, 2>(part, nblk, res);
  if (threadIdx.x != 0) return;
  if (!S->breakdown) {
    S->rho_old = S->rho;
    S->rho = res[0];
    S->rr = res[1];
    if (S->half) S->breakdown = 5;
    else if (res[0] == 0.0 || !isfinite(res[0])) S->breakdown = 4;
  }
  *host = *S;
}

template <typename XT>
__global__ void __launch_bounds__(kBlock) k_add_corr(double *__restrict__ x, const XT *__restrict__ d, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] += (double)d[i];
}

__global__ void k_reset_counter(unsigned *c) {
  if (threadIdx.x == 0) *c = 0u;
}

struct Solver {
  gf_ctx *ctx;
  const gf_nbr *nbr;
  int64_t n;
  double *part;   // [2 * kRedBlocks] partials of the SpMV kernels
  double *vpart;  // [2 * kVecBlocks] partials of the solution / residual update
  Scal *S;
  Scal *hS;
  unsigned grid_row;
  int vec_blocks;  // blocks of the vector updates
  bool vec_wide;   // of 1024 threads each (else kBlock)
  bool tiled;      // the SpMV runs on the neighbour tiles
  SpmvTiles tl;
  int tiles_grid[3][3] = {{0}};  // blocks of the tiled SpMV by types and epilogue, set at first use
  double *x_out = nullptr;  // the solution (refinement adds each inner correction here)
};

// staged-vector capacity of the tiled SpMV (entries)
constexpr int kSpmvCap = 2048;
static_assert(kSpmvCap <= 8 * kBlock, "the tiled SpMV stages at most 8 entries per thread");

// places that the packed matrix of the handle's tiles takes, at most (see PackedTiles; 0 without tiles)
int64_t packed_places(const gf_nbr *nb) {
  return nb->ntiles > 0 ? nb->nnz + nb->ntiles * (8 * (int64_t)((std::min(kTileBandRow, nb->max_row) + 7) / 8 * 8) + kGroups * 56) : 0;
}

void init_spmv_tiles(Solver &sv) {
  const gf_nbr *nb = sv.nbr;
  sv.tiled = nb->ntiles > 0 && nb->slot && nb->tile_u && nb->tile_off;
  SpmvTiles &t = sv.tl;
  t.toff = nb->tile_off; t.tu = nb->tile_u; t.grouped = nb->grouped;
  t.ntiles = nb->ntiles;
  int cap = 0;
  for (int m = 0; m < 2; ++m) {
    t.b3_start[m] = nb->group_start[m * GF_NBAND + kTileBand + 1];
    t.b3_n[m] = nb->group_start[(m + 1) * GF_NBAND] - t.b3_start[m];
    cap = std::max(cap, nb->tile_max[m]);
  }
  t.cap = std::min(cap, tile_capacity(sv.ctx, kSpmvCap));
  // Every block of a vector update adds up all partials of the kernel before it, so their grids are
  // small: blocks of 1024 threads on large systems, 256 (more CUs) where those give at most kVecBlocks.
  sv.vec_wide = sv.n > (int64_t)kVecBlocks * kBlock;
  const int64_t bs = sv.vec_wide ? kFinThreads : kBlock;
  sv.vec_blocks = (int)std::min<int64_t>(kVecBlocks, (sv.n + bs - 1) / bs);
}

// Blocks of the tiled SpMV: as many as are resident at once (a block walks
// its tiles to the end, so a block that waits for a slot would add its whole
// walk to the time), a multiple of 8, at most kRedBlocks, and no more than there
// are tiles (and long rows, four to a block): each writes a partial that every
// block of the next update reads.
template <typename VT, typename XT, int K, int EPI, bool NT>
int spmv_tiles_grid(const Solver &sv, size_t lds) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_spmv_tiles<VT, XT, K, EPI, NT>, kBlock, lds) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  const int64_t work = sv.tl.ntiles + (sv.tl.b3_n[0] + sv.tl.b3_n[1] + 3) / 4;
  const int64_t need = (work + 7) / 8 * 8;
  return (int)std::max<int64_t>(8, std::min<int64_t>(need, std::min(kRedBlocks, per_cu * sv.ctx->num_cu) / 8 * 8));
}

// a matrix: packed values of the tiled rows, CSR values of the others (or of all rows without tiles)
template <typename VT>
struct Matrix {
  const VT *csr, *packed;
};

// y = A xin with its epilogue (see k_spmv_tiles) over the tiles; returns the number of partials (blocks) written
template <typename VT, typename XT, int K, int EPI, bool NT>
int launch_spmv_nt(Solver &sv, const Matrix<VT> &m, const XT *xin, XT *y, XT *y2, const XT *other, const XT *other2,
                      const int *stop) {
  const size_t lds = 2 * sizeof(XT) * (size_t)sv.tl.cap;
  int &grid = sv.tiles_grid[sizeof(VT) == 8 ? 0 : (sizeof(XT) == 8 ? 1 : 2)][EPI];
  if (grid == 0) grid = spmv_tiles_grid<VT, XT, K, EPI, NT>(sv, lds);
  hipLaunchKernelGGL((k_spmv_tiles<VT, XT, K, EPI, NT>), dim3(grid), dim3(kBlock), lds, sv.ctx->stream, sv.nbr->row_ptr,
                     sv.nbr->col, m.csr, m.packed, xin, y, y2, other, other2, sv.part, stop, sv.tl);
  return grid;
}
// A matrix larger than the Infinity Cache (256 MB) comes from HBM at every product: non-temporal loads keep it from
// evicting the vectors and tile lists in L2.  A smaller one stays cached from one product to the next, which they would
// undo.  Iteration with and without them: 421 MB 204 / 229 us, 252 MB 151 / 158, 262 MB (FP64) 135 / 136, 157 MB
// 103 / 86, 94 MB 68 / 62, 20 MB 33 / 29.
constexpr double kStreamBytes = 240e6;
template <typename VT, typename XT, int K, int EPI>
int launch_spmv_tiles(Solver &sv, const Matrix<VT> &m, const XT *xin, XT *y, XT *y2, const XT *other, const XT *other2,
                      const int *stop) {
  const double bytes = (double)sv.nbr->nnz * (sizeof(VT) + sizeof(uint16_t));
  return bytes > kStreamBytes ? launch_spmv_nt<VT, XT, K, EPI, true>(sv, m, xin, y, y2, other, other2, stop)
                              : launch_spmv_nt<VT, XT, K, EPI, false>(sv, m, xin, y, y2, other, other2, stop);
}
template <typename VT, typename XT, int EPI>
int launch_spmv_k(Solver &sv, const Matrix<VT> &m, const XT *xin, XT *y, XT *y2, const XT *other, const XT *other2,
                  const int *stop) {
  const int k = (sv.tl.cap + kBlock - 1) / kBlock;
  if (k <= 1) return launch_spmv_tiles<VT, XT, 1, EPI>(sv, m, xin, y, y2, other, other2, stop);
  if (k <= 2) return launch_spmv_tiles<VT, XT, 2, EPI>(sv, m, xin, y, y2, other, other2, stop);
  if (k <= 3) return launch_spmv_tiles<VT, XT, 3, EPI>(sv, m, xin, y, y2, other, other2, stop);
  if (k <= 4) return launch_spmv_tiles<VT, XT, 4, EPI>(sv, m, xin, y, y2, other, other2, stop);
  return launch_spmv_tiles<VT, XT, 8, EPI>(sv, m, xin, y, y2, other, other2, stop);
}

// y = A xin; partials of (other, y), (y, y); returns their number.  Nothing is done where *stop.
template <typename VT, typename XT>
int launch_spmv(Solver &sv, const Matrix<VT> &m, const XT *xin, XT *y, const XT *other, const int *stop) {
  if (sv.tiled) return launch_spmv_k<VT, XT, kDots>(sv, m, xin, y, (XT *)nullptr, other, (const XT *)nullptr, stop);
  hipLaunchKernelGGL((k_spmv_dot<VT, XT>), dim3(kRedBlocks), dim3(kBlock), 0, sv.ctx->stream, sv.nbr->row_ptr,
                     sv.nbr->col, m.csr, xin, sv.n, y, other, sv.part, stop);
  return kRedBlocks;
}

// waits for the scalars that the last finishing kernel wrote down in pinned host memory (a copy of a few bytes would
// be a launch and a gap of its own)
gf_status read_scal(Solver &sv) {
  GF_HIP(sv.ctx, hipStreamSynchronize(sv.ctx->stream));
  return GF_OK;
}

template <typename VT, typename XT>
struct Vecs {
  Matrix<VT> A;
  const XT *dinv;
  XT *x, *r, *rhat, *p, *v, *phat, *s, *shat, *t;
};

// r = b - A x (and rhat = r with reset) followed by its scalar update
void launch_residual(Solver &sv, const Matrix<double> &A, const double *rhs, const double *x, double *r, double *rhat,
                     int reset) {
  hipStream_t sm = sv.ctx->stream;
  int nb = kRedBlocks;
  if (sv.tiled)
    nb = launch_spmv_k<double, double, kResid>(sv, A, x, r, rhat, rhs, (const double *)nullptr, (const int *)nullptr);
  else
    hipLaunchKernelGGL(k_residual, dim3(kRedBlocks), dim3(kBlock), 0, sm, sv.nbr->row_ptr, sv.nbr->col, A.csr, rhs, x,
                       sv.n, r, rhat, sv.part);
  hipLaunchKernelGGL(k_fin_residual, dim3(1), dim3(kFinThreads), 0, sm, sv.part, nb, sv.S, reset, sv.hS);
}

// residual replacement: r = b - A x, its norm and (rhat, r)
void launch_replace(Solver &sv, const Matrix<double> &A, const double *rhs, const double *x, const double *rhat,
                    double *r) {
  hipStream_t sm = sv.ctx->stream;
  int nb = kRedBlocks;
  if (sv.tiled)
    nb = launch_spmv_k<double, double, kReplaced>(sv, A, x, r, (double *)nullptr, rhs, rhat, (const int *)nullptr);
  else
    hipLaunchKernelGGL(k_residual_replace, dim3(kRedBlocks), dim3(kBlock), 0, sm, sv.nbr->row_ptr, sv.nbr->col, A.csr,
                       rhs, x, rhat, sv.n, r, sv.part);
  hipLaunchKernelGGL(k_fin_replace, dim3(1), dim3(kFinThreads), 0, sm, sv.part, nb, sv.S, sv.hS);
}

// One BiCGStab iteration (5 launches).  fresh: the scalars in S are final (a new start, or after the host's check);
// otherwise they follow from the partials of the iteration before.  check: the host looks next, so the scalars are
// finished by a launch of their own.
template <int BS, typename VT, typename XT>
gf_status bicgstab_iter_bs(Solver &sv, const Vecs<VT, XT> &V, bool fresh, bool check) {
  hipStream_t sm = sv.ctx->stream;
  const int64_t n = sv.n;
  const dim3 vg(sv.vec_blocks), vb(BS);
  ProfScope prof(sv.ctx, sizeof(VT) == 8 ? "bicgstab_iter_f64"
                        : (sizeof(XT) == 8 ? "bicgstab_iter_f32val" : "bicgstab_iter_f32"));
  hipLaunchKernelGGL((k_update_p<BS, XT>), vg, vb, 0, sm, V.r, V.v, V.dinv, n, V.p, V.phat, sv.S, sv.vpart,
                     fresh ? 0 : sv.vec_blocks);
  int nb = launch_spmv<VT, XT>(sv, V.A, V.phat, V.v, V.rhat, &sv.S->bd_p);
  hipLaunchKernelGGL((k_update_s<BS, XT>), vg, vb, 0, sm, V.r, V.v, V.dinv, n, V.s, V.shat, sv.S, sv.part, nb);
  nb = launch_spmv<VT, XT>(sv, V.A, V.shat, V.t, V.s, &sv.S->bd_s);
  hipLaunchKernelGGL((k_update_xr<BS, XT>), vg, vb, 0, sm, V.phat, V.shat, V.s, V.t, V.rhat, n, V.x, V.r, sv.S, sv.part,
                     nb, sv.vpart);
  if (check) hipLaunchKernelGGL(k_fin_xr, dim3(1), dim3(kFinThreads), 0, sm, sv.vpart, sv.vec_blocks, sv.S, sv.hS);
  GF_LAUNCH_CHECK(sv.ctx);
  return GF_OK;
}
template <typename VT, typename XT>
gf_status bicgstab_iter(Solver &sv, const Vecs<VT, XT> &V, bool fresh, bool check) {
  return sv.vec_wide ? bicgstab_iter_bs<kFinThreads, VT, XT>(sv, V, fresh, check)
                     : bicgstab_iter_bs<kBlock, VT, XT>(sv, V, fresh, check);
}

// One inner solve of the refinement: A32 d = r64 from d = 0 by Jacobi-BiCGStab
// on FP32 matrix values, until the recursive residual is below inner_target
// (or the iteration limits); then x += d.  `total` counts every iteration.
template <typename XT>
gf_status inner_solve(Solver &sv, const Vecs<float, XT> &V, const double *r64, double inner_target,
                      const gf_solve_params &prm, int &total, gf_solve_stats &sts) {
  gf_ctx *ctx = sv.ctx;
  hipStream_t sm = ctx->stream;
  hipLaunchKernelGGL(k_inner_init<XT>, dim3(kRedBlocks), dim3(kBlock), 0, sm, r64, sv.n, V.r, V.rhat, V.p, V.v, V.x,
                     sv.part);
  hipLaunchKernelGGL(k_fin_inner_init, dim3(1), dim3(kFinThreads), 0, sm, sv.part, kRedBlocks, sv.S);
  GF_LAUNCH_CHECK(ctx);
  gf_status st;
  int it = 0;
  bool fresh = true;
  while (it < prm.inner_maxit && total < prm.maxit) {
    const bool check = (it + 1) % prm.check_every == 0;
    if ((st = bicgstab_iter<float, XT>(sv, V, fresh, check))) return st;
    ++it;
    ++total;
    fresh = check;
    if (!check) continue;
    if ((st = read_scal(sv))) return st;
    if (sv.hS->breakdown) { ++sts.restarts; break; }
    if (std::sqrt(sv.hS->rr) <= inner_target) break;
  }
  hipLaunchKernelGGL(k_add_corr<XT>, dim3(sv.grid_row), dim3(kBlock), 0, sm, sv.x_out, V.x, sv.n);
  GF_LAUNCH_CHECK(ctx);
  return GF_OK;
}
}  // namespace

extern "C" void gf_solve_params_default(gf_solve_params *p) {
  if (!p) return;
  p->rtol = 1e-8;
  p->maxit = 20000;
  p->mixed = 0;
  p->inner_rtol = 1e-4;
  p->inner_maxit = 2000;
  p->zeta = 0.3;
  p->check_every = 4;
  p->implicit_a = 0.0;
}

// a: coefficient of GF_ROW_IMPLICIT rows; max_type: largest row type accepted
static AsmArgs asm_args(const gf_particles *p, const gf_nbr *nbr, const double *w64, const int8_t *row_type, double zeta,
                        double a, int max_type, double *dinv64, float *dinv32, int *bad) {
  AsmArgs g;
  g.row_ptr = nbr->row_ptr; g.col = nbr->col; g.w = w64; g.row_type = row_type;
  g.h = p->h; g.nx = p->nx; g.ny = p->ny; g.nz = p->nz;
  g.zeta = zeta; g.a = a; g.max_type = max_type;
  g.dinv64 = dinv64; g.dinv32 = dinv32; g.bad = bad;
  return g;
}

static gf_status check_solve_args(gf_ctx *ctx, const gf_particles *p, const gf_nbr *nbr, const double *w64,
                                  const int8_t *row_type) {
  gf_status st = check_particles(ctx, p, false, false);
  if (st) return st;
  if ((st = check_nbr(ctx, nbr, p->n))) return st;
  if (nbr->cross) return set_error(ctx, GF_EINVAL, "the pressure system lives on same-model neighbourhoods");
  if (!w64 || !row_type) return set_error(ctx, GF_EINVAL, "w64 and row_type are required");
  return GF_OK;
}

extern "C" gf_status gf_poisson_assemble(gf_ctx *ctx, const gf_particles *p, const gf_nbr *nbr, const double *w64,
                                         const int8_t *row_type, double zeta, double *val_out) {
  if (!ctx) return GF_EINVAL;
  gf_status st = check_solve_args(ctx, p, nbr, w64, row_type);
  if (st) return st;
  if (!val_out) return set_error(ctx, GF_EINVAL, "val_out is NULL");
  if (!p->nx || !p->ny || !p->nz) return set_error(ctx, GF_EINVAL, "normals are required for Neumann rows");
  Arena ar;
  if ((st = ensure_scratch(ctx, arena_bytes({64}), &ar))) return st;
  int *bad = ar.take<int>(16);
  hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(64), 0, ctx->stream, (unsigned *)bad);
  const AsmArgs g = asm_args(p, nbr, w64, row_type, zeta, 0.0, GF_ROW_NEUMANN, nullptr, nullptr, bad);
  hipLaunchKernelGGL(k_assemble, dim3(kRedBlocks), dim3(kBlock), 0, ctx->stream, g, (const int32_t *)nullptr, p->n, val_out,
                     (float *)nullptr);
  GF_LAUNCH_CHECK(ctx);
  return GF_OK;
}

extern "C" gf_status gf_poisson_solve(gf_ctx *ctx, const gf_particles *p, const gf_nbr *nbr, const double *w64,
                                      const int8_t *row_type, const double *rhs, double *p_inout,
                                      const gf_solve_params *params, gf_solve_stats *stats) {
  if (!ctx) return GF_EINVAL;
  gf_status st = check_solve_args(ctx, p, nbr, w64, row_type);
  if (st) return st;
  if (!rhs || !p_inout) return set_error(ctx, GF_EINVAL, "rhs and p_inout are required");
  if (!p->nx || !p->ny || !p->nz) return set_error(ctx, GF_EINVAL, "normals are required for Neumann rows");
  gf_solve_params prm;
  gf_solve_params_default(&prm);
  if (params) prm = *params;
  if (!(prm.rtol > 0.0) || prm.maxit <= 0 || prm.check_every <= 0 || prm.mixed < 0 || prm.mixed > 2 ||
      (prm.mixed && (!(prm.inner_rtol > 0.0) || prm.inner_maxit <= 0)))
    return set_error(ctx, GF_EINVAL, "invalid solver parameters");
  gf_solve_stats sts;
  memset(&sts, 0, sizeof(sts));
  const auto t_start = std::chrono::steady_clock::now();
  auto elapsed = [&]() { return std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count(); };
  const int64_t n = p->n, nnz = nbr->nnz;
  const bool mixed = prm.mixed != 0;
  const bool vec32 = prm.mixed == 2;  // FP32 Krylov vectors in the inner solve
  Arena ar;
  const int nblk_row = (int)grid_for(n, kBlock);
  // CSR values are only read where there are rows without a tile
  const int64_t n_long = nbr->group_start[GF_NBAND] - nbr->group_start[kTileBand + 1] +
                         nbr->group_start[2 * GF_NBAND] - nbr->group_start[GF_NBAND + kTileBand + 1];
  const int64_t csr = nbr->ntiles > 0 && n_long == 0 ? 1 : std::max<int64_t>(nnz, 1);
  const int64_t places = packed_places(nbr), ngroups = kGroups * nbr->ntiles;
  std::vector<size_t> sz = {sizeof(double) * csr, sizeof(double) * places, sizeof(uint16_t) * places,
                            sizeof(int64_t) * (ngroups + 1), sizeof(int32_t) * ngroups,
                            sizeof(int64_t) * scan_tmp_elems(ngroups + 1), sizeof(int32_t) * kTileRows * nbr->ntiles,
                            sizeof(double) * n, sizeof(double) * 2 * kRedBlocks, sizeof(double) * 2 * kVecBlocks,
                            sizeof(Scal), 64};
  for (int k = 0; k < 9; ++k) sz.push_back(sizeof(double) * n);
  if (mixed) {
    sz.push_back(sizeof(float) * csr);
    sz.push_back(sizeof(float) * places);
    sz.push_back(sizeof(float) * n);
    if (vec32)
      for (int k = 0; k < 9; ++k) sz.push_back(sizeof(float) * n);
  }
  if ((st = ensure_scratch(ctx, arena_bytes(sz), &ar))) return st;
  double *val64 = ar.take<double>(csr);
  double *pval64 = ar.take<double>(places);
  uint16_t *pslot = ar.take<uint16_t>(places);
  int64_t *goff = ar.take<int64_t>(ngroups + 1);
  int32_t *gq = ar.take<int32_t>(ngroups);
  int64_t *gtmp = ar.take<int64_t>(scan_tmp_elems(ngroups + 1));
  int32_t *prow = ar.take<int32_t>(kTileRows * nbr->ntiles);
  double *dinv64 = ar.take<double>(n);
  double *part = ar.take<double>(2 * kRedBlocks);
  double *vpart = ar.take<double>(2 * kVecBlocks);
  Scal *S = ar.take<Scal>(1);
  int *bad = ar.take<int>(16);
  double *vec64[9];
  for (int k = 0; k < 9; ++k) vec64[k] = ar.take<double>(n);
  float *val32 = nullptr, *pval32 = nullptr, *dinv32 = nullptr, *v32[9] = {nullptr};
  if (mixed) {
    val32 = ar.take<float>(csr);
    pval32 = ar.take<float>(places);
    dinv32 = ar.take<float>(n);
    if (vec32)
      for (int k = 0; k < 9; ++k) v32[k] = ar.take<float>(n);
  }
  if ((st = ensure_host(ctx, 4096))) return st;
  hipStream_t sm = ctx->stream;
  hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(64), 0, sm, (unsigned *)bad);
  Solver sv;
  sv.ctx = ctx; sv.nbr = nbr; sv.n = n; sv.part = part; sv.vpart = vpart; sv.S = S;
  sv.hS = (Scal *)ctx->host_pinned;
  sv.grid_row = (unsigned)nblk_row;
  sv.x_out = p_inout;
  init_spmv_tiles(sv);
  sv.tl.pk.goff = goff; sv.tl.pk.prow = prow; sv.tl.pk.slot = pslot;
  const AsmArgs ga = asm_args(p, nbr, w64, row_type, prm.zeta, prm.implicit_a, GF_ROW_IMPLICIT, dinv64, dinv32, bad);
  if (sv.tiled) {
    const TileRows tr = tile_rows(nbr);
    hipLaunchKernelGGL(k_pack_rows, dim3(grid_for(nbr->ntiles, kBlock / 64)), dim3(kBlock), 0, sm, tr, nbr->row_ptr, prow, gq);
    GF_LAUNCH_CHECK(ctx);
    if ((st = scan_i32_to_i64(ctx, gq, goff, ngroups, gtmp))) return st;
    hipLaunchKernelGGL(k_assemble_packed, dim3(kRedBlocks), dim3(kBlock), 0, sm, ga, goff, prow,
                       (int64_t)kTileRows * nbr->ntiles, nbr->slot, pval64, pval32, pslot);
    for (int m = 0; m < 2; ++m)
      if (sv.tl.b3_n[m] > 0)
        hipLaunchKernelGGL(k_assemble, dim3(kRedBlocks), dim3(kBlock), 0, sm, ga, nbr->grouped + sv.tl.b3_start[m],
                           sv.tl.b3_n[m], val64, val32);
  } else {
    hipLaunchKernelGGL(k_assemble, dim3(kRedBlocks), dim3(kBlock), 0, sm, ga, (const int32_t *)nullptr, n, val64, val32);
  }
  GF_LAUNCH_CHECK(ctx);
  const Matrix<double> A64 = {val64, pval64};
  const Matrix<float> A32 = {val32, pval32};
  int *hbad = (int *)((char *)ctx->host_pinned + 1024);
  GF_HIP(ctx, hipMemcpyAsync(hbad, bad, sizeof(int), hipMemcpyDeviceToHost, sm));
  // FP64 work vectors: x is the caller's array
  Vecs<double, double> V64;
  V64.A = A64; V64.dinv = dinv64; V64.x = p_inout;
  V64.r = vec64[0]; V64.rhat = vec64[1]; V64.p = vec64[2]; V64.v = vec64[3]; V64.phat = vec64[4];
  V64.s = vec64[5]; V64.shat = vec64[6]; V64.t = vec64[7];
  // initial residual
  launch_residual(sv, A64, rhs, p_inout, V64.r, V64.rhat, 1);
  hipLaunchKernelGGL(k_zero_vecs<double>, dim3(sv.grid_row), dim3(kBlock), 0, sm, n, V64.p, V64.v);
  GF_LAUNCH_CHECK(ctx);
  if ((st = read_scal(sv))) return st;
  if (*hbad > 0) return set_error(ctx, GF_EINVAL, "%d rows have an unknown row type or a zero/non-finite diagonal", *hbad);
  const double bnorm = std::sqrt(sv.hS->bb);
  double rnorm = std::sqrt(sv.hS->rr);
  if (bnorm == 0.0) {
    // the solution of A p = 0 is p = 0
    hipLaunchKernelGGL(k_zero_vecs<double>, dim3(sv.grid_row), dim3(kBlock), 0, sm, n, p_inout, V64.r);
    GF_LAUNCH_CHECK(ctx);
    sts.converged = 1;
    sts.seconds = elapsed();
    if (stats) *stats = sts;
    return GF_OK;
  }
  const double target = prm.rtol * bnorm;
  int total = 0;
  if (!mixed) {
    sts.outer_its = 1;
    // true residual at the last restart; restarts that no longer reduce it
    // mean the tolerance is below the attainable accuracy
    double restart_rnorm = rnorm;
    int stagnant = 0;
    bool fresh = true;
    while (rnorm > target && total < prm.maxit) {
      const bool check = (total + 1) % prm.check_every == 0 || total + 1 >= prm.maxit;
      if ((st = bicgstab_iter<double, double>(sv, V64, fresh, check))) return st;
      ++total;
      fresh = check;
      if (!check) continue;
      if ((st = read_scal(sv))) return st;
      if (sv.hS->breakdown) {
        if (++sts.restarts > 50) {
          sts.inner_its_total = total;
          sts.seconds = elapsed();
    if (stats) *stats = sts;
          return set_error(ctx, GF_EBREAKDOWN, "BiCGStab broke down repeatedly (code %d)", sv.hS->breakdown);
        }
        launch_residual(sv, A64, rhs, p_inout, V64.r, V64.rhat, 1);
        hipLaunchKernelGGL(k_zero_vecs<double>, dim3(sv.grid_row), dim3(kBlock), 0, sm, n, V64.p, V64.v);
        if ((st = read_scal(sv))) return st;
        rnorm = std::sqrt(sv.hS->rr);
        stagnant = rnorm < 0.9 * restart_rnorm ? 0 : stagnant + 1;
        restart_rnorm = std::min(restart_rnorm, rnorm);
        if (stagnant >= 3) break;
        continue;
      }
      rnorm = std::sqrt(sv.hS->rr);
      if (rnorm <= target) {
        // replace the recursive residual by the true one
        launch_residual(sv, A64, rhs, p_inout, V64.r, nullptr, 0);
        if ((st = read_scal(sv))) return st;
        rnorm = std::sqrt(sv.hS->rr);
      }
    }
  } else if (!vec32) {
    // FP32 matrix values, FP64 vectors, residual replacement with the FP64 matrix
    Vecs<float, double> V1 = {A32, dinv64, p_inout, V64.r, V64.rhat, V64.p, V64.v, V64.phat, V64.s, V64.shat, V64.t};
    sts.outer_its = 1;
    double last_true = rnorm;  // true residual at the last replacement (or restart)
    int stagnant = 0;
    bool fresh = true;
    while (rnorm > target && total < prm.maxit) {
      const bool check = (total + 1) % prm.check_every == 0 || total + 1 >= prm.maxit;
      if ((st = bicgstab_iter<float, double>(sv, V1, fresh, check))) return st;
      ++total;
      fresh = check;
      if (!check) continue;
      if ((st = read_scal(sv))) return st;
      if (sv.hS->breakdown) {
        if (++sts.restarts > 50) {
          sts.inner_its_total = total;
          sts.seconds = elapsed();
          if (stats) *stats = sts;
          return set_error(ctx, GF_EBREAKDOWN, "BiCGStab broke down repeatedly (code %d)", sv.hS->breakdown);
        }
        launch_residual(sv, A64, rhs, p_inout, V64.r, V64.rhat, 1);
        hipLaunchKernelGGL(k_zero_vecs<double>, dim3(sv.grid_row), dim3(kBlock), 0, sm, n, V64.p, V64.v);
        if ((st = read_scal(sv))) return st;
        rnorm = std::sqrt(sv.hS->rr);
        stagnant = rnorm < 0.9 * last_true ? 0 : stagnant + 1;
        last_true = std::min(last_true, rnorm);
        if (stagnant >= 3) break;
        continue;
      }
      const double rrec = std::sqrt(sv.hS->rr);
      if (rrec > std::max(target, kReplace * last_true)) {
        rnorm = rrec;
        continue;
      }
      // replace the recursive residual by the FP64 one
      launch_replace(sv, A64, rhs, p_inout, V64.rhat, V64.r);
      GF_LAUNCH_CHECK(ctx);
      if ((st = read_scal(sv))) return st;
      rnorm = std::sqrt(sv.hS->rr);
      ++sts.outer_its;
      // replacements that no longer cut the true residual: the tolerance is below what the FP32 matrix allows
      stagnant = rnorm < 0.9 * last_true ? 0 : stagnant + 1;
      last_true = rnorm;
      if (stagnant >= 3) break;
    }
  } else {
    // iterative refinement with restarts, FP32 inner vectors
    Vecs<float, float> Vf;
    Vf.A = A32; Vf.dinv = dinv32; Vf.x = v32[8];
    Vf.r = v32[0]; Vf.rhat = v32[1]; Vf.p = v32[2]; Vf.v = v32[3]; Vf.phat = v32[4];
    Vf.s = v32[5]; Vf.shat = v32[6]; Vf.t = v32[7];
    while (rnorm > target && total < prm.maxit) {
      ++sts.outer_its;
      // inner solve of A32 d = r64 from d = 0; the last one need not go below half the overall target
      const double inner_target = std::max(prm.inner_rtol * rnorm, 0.5 * target);
      if ((st = inner_solve<float>(sv, Vf, V64.r, inner_target, prm, total, sts))) return st;
      launch_residual(sv, A64, rhs, p_inout, V64.r, nullptr, 0);
      GF_LAUNCH_CHECK(ctx);
      if ((st = read_scal(sv))) return st;
      const double prev = rnorm;
      rnorm = std::sqrt(sv.hS->rr);
      if (sts.restarts > 50) break;
      if (!(rnorm < prev) && sts.outer_its > 3) break;  // refinement stagnated
    }
  }
  sts.inner_its_total = total;
  sts.final_rel_res = rnorm / bnorm;
  sts.converged = rnorm <= target;
  sts.seconds = elapsed();
  if (stats) *stats = sts;
  if (!sts.converged)
    return set_error(ctx, GF_ENOTCONV, "not converged: relative residual %.3e after %d iterations", sts.final_rel_res, total);
  return GF_OK;
}
