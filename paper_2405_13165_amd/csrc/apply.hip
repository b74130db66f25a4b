// Stencil application (Eq. GFDM_Definition, differenced form) and its
// transpose.  Rows are taken in the grouped Morton order of the neighbour
// handle; a team of T lanes strides over a row's entries so one wave
// instruction reads T consecutive 16-byte (FP32) or 32-byte (FP64) weight
// records; partial sums are combined by a butterfly over the team and
// accumulated in FP64.
#include <algorithm>

#include "stencil_common.h"

using namespace gfdm_dev;

namespace {
constexpr int kBlock = 256;

template <typename WT>
struct W4;
template <>
struct W4<float> {
  static __device__ inline void load(const void *w, int64_t k, double c[4]) {
    const float4 v = reinterpret_cast<const float4 *>(w)[k];
    c[0] = v.x; c[1] = v.y; c[2] = v.z; c[3] = v.w;
  }
};
template <>
struct W4<double> {
  static __device__ inline void load(const void *w, int64_t k, double c[4]) {
    const double2 *p = reinterpret_cast<const double2 *>(w) + 2 * k;
    const double2 a = p[0], b = p[1];
    c[0] = a.x; c[1] = a.y; c[2] = b.x; c[3] = b.y;
  }
};

template <int T, typename WT, typename IOT>
__global__ void __launch_bounds__(kBlock) k_apply(const int32_t *__restrict__ sched, int64_t nrows,
                                                  const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                                                  const void *__restrict__ w, unsigned mask,
                                                  const IOT *__restrict__ u, IOT *__restrict__ out, int64_t n) {
  const int64_t gt = (int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
  const int64_t team = gt / T;
  const int lane = (int)(gt % T);
  if (team >= nrows) return;
  const int32_t i = sched[team];
  const int64_t b = row_ptr[i], e = row_ptr[i + 1];
  const double ui = (double)u[i];
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t k = b + lane; k < e; k += T) {
    const int32_t j = col[k];
    double c[4];
    W4<WT>::load(w, k, c);
    const double du = (j != i) ? (double)u[j] - ui : 0.0;
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[s] += c[s] * du;
  }
  if constexpr (T > 1) {
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[s] = team_sum(acc[s], T);
  }
  if (lane == 0) {
    int q = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (mask & (1u << s)) out[(int64_t)(q++) * n + i] = (IOT)acc[s];
  }
}

// A stencil record (four operators of one entry) as loaded, converted to
// FP64 only where it is used: a conversion right after the load would wait
// for it there.
// NT: read past the caches (each line by one instruction only).
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
template <typename WT>
struct WRec;
template <>
struct WRec<float> {
  f32x4 v;
  template <bool NT = false>
  __device__ inline void load(const void *w, int64_t k) {
    const f32x4 *p = reinterpret_cast<const f32x4 *>(w) + k;
    if constexpr (NT) v = __builtin_nontemporal_load(p);
    else v = *p;
  }
  __device__ inline double get(int s) const { return s == 0 ? v.x : s == 1 ? v.y : s == 2 ? v.z : v.w; }
};
template <>
struct WRec<double> {
  f64x2 a, b;
  template <bool NT = false>
  __device__ inline void load(const void *w, int64_t k) {
    const f64x2 *p = reinterpret_cast<const f64x2 *>(w) + 2 * k;
    a = p[0];
    b = p[1];
  }
  __device__ inline double get(int s) const { return s == 0 ? a.x : s == 1 ? a.y : s == 2 ? b.x : b.y; }
};

// Tiled application (rows of the tiled bands): one block per neighbour tile;
// the field values of the tile's distinct neighbours are staged in LDS and
// each entry reads its value through slot[] (2 bytes) instead of col[]
// (4 bytes) plus a gather.  The diagonal entry contributes u_i - u_i = 0.
// A lane's first kApplyAhead stencil records and slots are requested before the
// tile is staged, and each next group while the last one is used: the wait for
// the chain tile offset -> list -> field values -> barrier then covers them too.
// One launch takes the tiles of both models where their team sizes agree.
//
// A team starts at the aligned block of T entries at or below its row, so that
// each step of 8 lanes reads whole 128-byte lines of FP32 records, once: rows
// start anywhere, and lines read half by one step and half by the next do not
// survive in L2 between the two when every CU keeps hundreds of rows in flight.
//
// What bounds it: HBM (18 bytes per entry with FP32 stencils).  Mixed cloud
// (534 MB of stencils, four operators) 158 -> 147.6 us over repeated calls; in one
// trial after another (141 us then) with four or seven records ahead 154 and 180 us,
// without the aligned start 168 us, without NT (stencils beyond the Infinity Cache,
// FP32) 150 us; at an eighth of the size 23.6 -> 19.1 us.  NT takes 55 against 43 us
// at 200 MB, which stay cached between calls; FP64 records, whose lines two
// instructions share, lose by it (270 against 250 us).
struct ApplyTiles {
  const int32_t *grouped;
  int nranges;
  int64_t tile0[2], ntiles[2];   // tiles of the ranges
  int64_t row0[2], nrows[2];     // their rows of grouped[]
  int cap;
};
constexpr int kApplyAhead = 2;
constexpr double kApplyStream = 240e6;  // bytes of stencils above which they are streamed

template <int T, typename WT, typename IOT, bool NT>
__global__ void __launch_bounds__(kTileRows * T) k_apply_tile(ApplyTiles at, const int64_t *__restrict__ row_ptr,
                                                              const int32_t *__restrict__ col,
                                                              const uint16_t *__restrict__ slot,
                                                              const int64_t *__restrict__ toff,
                                                              const int32_t *__restrict__ tu,
                                                              const void *__restrict__ w, unsigned mask,
                                                              const IOT *__restrict__ u, IOT *__restrict__ out,
                                                              int64_t n) {
  extern __shared__ double s_u[];
  constexpr int A = kApplyAhead;
  // each range is cut into slices for the XCDs by itself (a 3D tile costs four film tiles); the first
  // takes a multiple of eight blocks, so that the second starts at XCD 0 again
  const unsigned n0 = ((unsigned)at.ntiles[0] + 7u) & ~7u;
  const int m = blockIdx.x >= n0 ? 1 : 0;
  const int64_t tm = m ? xcd_block(blockIdx.x - n0, gridDim.x - n0) : xcd_block(blockIdx.x, at.nranges == 2 ? n0 : gridDim.x);
  if (tm >= at.ntiles[m]) return;  // (the whole block)
  const int64_t tl = at.tile0[m] + tm;
  const int team = threadIdx.x / T, lane = threadIdx.x % T;
  const int64_t r = tm * kTileRows + team;
  // row prologue first: its loads overlap the staging below
  const bool live = r < at.nrows[m];
  const int32_t i = live ? at.grouped[at.row0[m] + r] : 0;
  const int64_t b = live ? row_ptr[i] : 0, e = live ? row_ptr[i + 1] : 0;
  const double ui = (double)u[i];
  WRec<WT> ra[A], rb[A];
  uint16_t sa[A], sb[A];
  auto fetch = [&](int64_t k, WRec<WT> (&rec)[A], uint16_t (&sl)[A]) {
#pragma unroll
    for (int q = 0; q < A; ++q)
      if (k + q * T >= b && k + q * T < e) {
        rec[q].template load<NT>(w, k + q * T);
        sl[q] = slot[k + q * T];
      }
  };
  const int64_t kb = (b & ~(int64_t)(T - 1)) + lane;
  fetch(kb, ra, sa);
  const int64_t u0 = toff[tl];
  const int cnt = (int)(toff[tl + 1] - u0);
  const bool staged = cnt <= at.cap;
  if (staged)
    for (int s = threadIdx.x; s < cnt; s += blockDim.x) s_u[s] = (double)u[tu[u0 + s]];
  __syncthreads();
  if (!live) return;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (staged) {
    auto use = [&](int64_t k, const WRec<WT> (&rec)[A], const uint16_t (&sl)[A]) {
#pragma unroll
      for (int q = 0; q < A; ++q)
        if (k + q * T >= b && k + q * T < e) {
          const double du = s_u[sl[q]] - ui;
#pragma unroll
          for (int s = 0; s < 4; ++s) acc[s] += rec[q].get(s) * du;
        }
    };
#pragma unroll 1
    for (int64_t k = kb; k < e; k += 2 * A * T) {
      fetch(k + A * T, rb, sb);
      use(k, ra, sa);
      fetch(k + 2 * A * T, ra, sa);
      use(k + A * T, rb, sb);
    }
  } else {
    for (int64_t k = b + lane; k < e; k += T) {
      double c[4];
      W4<WT>::load(w, k, c);
      const double du = (double)u[col[k]] - ui;
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[s] += c[s] * du;
    }
  }
  if constexpr (T > 1) {
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[s] = team_sum(acc[s], T);
  }
  if (lane == 0) {
    int q = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (mask & (1u << s)) out[(int64_t)(q++) * n + i] = (IOT)acc[s];
  }
}

// field values a tiled apply block may stage
constexpr int kApplyCap = 2048;

// ubar_j = sum_{i : j in S_i, i != j} c_ij ybar_i - ybar_j sum_{k in S_j, k != j} c_jk,
// the first sum gathered through the reverse-edge map (entry (i,j) sits at
// rev[k] for the entry k = (j,i) of row j); an entry of row j without a twin
// (towards a ghost particle, which has no row) adds only its own term.
// Taken where some row has more than kTileBandRow entries (on the mixed cloud,
// which has none, 463 us against 206 + 37 over transposed tiles).
// One team of adj_team lanes per row j (the lanes stride over the row), K the
// number of selected operators.  Each lane takes adj_unroll entries per step: their
// columns and twin positions, then their two stencil records (c_ij of row i,
// c_ji of row j) and seeds ybar_i are all requested before the first is used,
// in one straight block (so that no load is moved down to its use); entries
// past the row's end read its last entry and an entry without a twin reads
// the stencil record 0 (both valid, added as zero), so no load is skipped.
// Team width and entries per step, as measured on the mixed cloud (FP32
// stencils: 8 x 4 took 572 / 631 us for one / four operators, 8 x 8 461 / 626,
// 16 x 4 495 / 569); FP64 records are twice as large and keep 8 x 4.
template <typename WT>
__host__ __device__ constexpr int adj_team(int K) { return (sizeof(WT) == 4 && K >= 3) ? 16 : 8; }
template <typename WT>
__host__ __device__ constexpr int adj_unroll(int K) { return (sizeof(WT) == 4 && K <= 2) ? 8 : 4; }
template <typename WT, int K>
__global__ void __launch_bounds__(kBlock) k_apply_adjoint(const int64_t *__restrict__ row_ptr,
                                                          const int32_t *__restrict__ col,
                                                          const int32_t *__restrict__ rev, const void *__restrict__ w,
                                                          unsigned mask, const double *__restrict__ ybar, int64_t n,
                                                          double *__restrict__ ubar) {
  constexpr int kAdjTeam = adj_team<WT>(K), kAU = adj_unroll<WT>(K);
  const int64_t gt = (int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
  const int64_t j = gt / kAdjTeam;
  const int lane = (int)(gt % kAdjTeam);
  if (j >= n) return;
  int sel[K];  // the selected operators in ascending order
  unsigned m = mask;
#pragma unroll
  for (int q = 0; q < K; ++q) {
    sel[q] = K == 4 ? q : __builtin_ctz(m);
    m &= m - 1;
  }
  double yj[K];
#pragma unroll
  for (int q = 0; q < K; ++q) yj[q] = ybar[(int64_t)q * n + j];
  double acc = 0.0;
  const int64_t b = row_ptr[j], e = row_ptr[j + 1], kl = e - 1;
#pragma unroll 1
  for (int64_t kb = b + lane; kb < e; kb += kAU * kAdjTeam) {
    int32_t ci[kAU], kr[kAU];
#pragma unroll
    for (int u = 0; u < kAU; ++u) {
      const int64_t kk = min(kb + u * kAdjTeam, kl);
      ci[u] = col[kk];
      kr[u] = rev[kk];
    }
    WRec<WT> win[kAU], wout[kAU];
    double y[kAU][K];
#pragma unroll
    for (int u = 0; u < kAU; ++u) {
      win[u].load(w, kr[u] >= 0 ? kr[u] : 0);
      wout[u].load(w, min(kb + u * kAdjTeam, kl));
#pragma unroll
      for (int q = 0; q < K; ++q) y[u][q] = ybar[(int64_t)q * n + ci[u]];
    }
#pragma unroll
    for (int u = 0; u < kAU; ++u) {
      const bool on = kb + u * kAdjTeam < e && ci[u] != j;
#pragma unroll
      for (int q = 0; q < K; ++q) {
        const double t = (kr[u] >= 0 ? win[u].get(sel[q]) * y[u][q] : 0.0) - wout[u].get(sel[q]) * yj[q];
        acc += on ? t : 0.0;
      }
    }
  }
  acc = team_sum(acc, kAdjTeam);
  if (lane == 0) ubar[j] = acc;
}

// The same where every row is tiled.  Entry (i, j) gives t = sum_s c_ij^s
// ybar_i^s to ubar_j and takes it from ubar_i: one pass over the stencils, read
// once and in order, instead of two reads of each, one of them scattered.  A
// block takes a tile: its rows' terms go to LDS, and each distinct neighbour's
// are added up in row order through the transposed tile; part holds a tile's
// sums at the places of its list, and k_places_sum adds up each particle's.  No
// atomics: the result is deterministic.  Ghost particles (j >= n_rows) list
// nobody, so they receive nothing.
//
// What bounds it: HBM (20 bytes per entry with FP32 stencils), at 1.15 GB on
// 80^3 particles 4.1 TB/s: 278 + 39 us (k_places_sum) where two reads of each
// stencil, one of them scattered, took 511.  A lane per slot in the tile's own
// order took 389 us, the general path's map of twin entries 1.7 ms to build once
// per neighbourhood (the transposed tiles 0.4).
template <typename WT, int K, bool NT>
__global__ void __launch_bounds__(kBlock) k_apply_adjoint_tile(TileRows tr, const int64_t *__restrict__ row_ptr,
                                                               const int64_t *__restrict__ tile_off,
                                                               const int64_t *__restrict__ tperm_off,
                                                               const uint16_t *__restrict__ tperm,
                                                               const uint16_t *__restrict__ tself,
                                                               const uint16_t *__restrict__ slot,
                                                               const void *__restrict__ w, unsigned mask,
                                                               const double *__restrict__ ybar, int64_t n,
                                                               double *__restrict__ part, double *__restrict__ ubar) {
  constexpr int T = kBlock / kTileRows, A = 4;
  extern __shared__ double s_t[];  // the tile's terms, in tile order
  __shared__ int32_t s_len[kTileRows], s_off[kTileRows];
  const int64_t t = xcd_block(blockIdx.x, gridDim.x);
  const int team = threadIdx.x / T, lane = threadIdx.x % T;
  const int32_t i = tile_row(tr, t, team);
  const int64_t b = i >= 0 ? row_ptr[i] : 0, e = i >= 0 ? row_ptr[i + 1] : 0;
  WRec<WT> rec[A];
  uint16_t sj[A];
  const int64_t kb = (b & ~(int64_t)(T - 1)) + lane;  // aligned blocks, as in k_apply_tile
  auto fetch = [&](int64_t k) {
#pragma unroll
    for (int q = 0; q < A; ++q)
      if (k + q * T >= b && k + q * T < e) {
        rec[q].template load<NT>(w, k + q * T);
        sj[q] = slot[k + q * T];
      }
  };
  fetch(kb);
  const int64_t u0 = tile_off[t], p0 = tperm_off[t];
  const int U = (int)(tile_off[t + 1] - u0);
  const uint16_t *block = tperm + 64 * p0;
  const int self = i >= 0 ? tself[kTileRows * t + team] : -1;
  const uint32_t line = TileSum<kBlock>::warm(block, tperm_off[t + 1] - p0);
  int sel[K];  // the selected operators in ascending order
  unsigned m = mask;
#pragma unroll
  for (int q = 0; q < K; ++q) {
    sel[q] = K == 4 ? q : __builtin_ctz(m);
    m &= m - 1;
  }
  double y[K];
#pragma unroll
  for (int q = 0; q < K; ++q) y[q] = i >= 0 ? ybar[(int64_t)q * n + i] : 0.0;
  if (lane == 0) s_len[team] = (int)(e - b);
  __syncthreads();
  // entries of the tile before each row
  if (threadIdx.x < 64) {
    const int len = threadIdx.x < kTileRows ? s_len[threadIdx.x] : 0;
    int inc = len;
#pragma unroll
    for (int o = 1; o < kTileRows; o <<= 1) {
      const int v = __shfl_up(inc, o, 64);
      if ((int)threadIdx.x >= o) inc += v;
    }
    if (threadIdx.x < kTileRows) s_off[threadIdx.x] = inc - len;
    if (threadIdx.x == kTileRows - 1) s_t[inc] = 0.0;  // the term of the padding
  }
  __syncthreads();
  double own = 0.0;
  double *mine = s_t + s_off[team];
#pragma unroll 1
  for (int64_t k = kb; k < e; k += A * T) {
#pragma unroll
    for (int q = 0; q < A; ++q)
      if (k + q * T >= b && k + q * T < e) {
        double v = 0.0;
#pragma unroll
        for (int s = 0; s < K; ++s) v += rec[q].get(sel[s]) * y[s];
        if (sj[q] == self) v = 0.0;  // the diagonal entry multiplies u_i - u_i
        mine[k + q * T - b] = v;
        own += v;
      }
    fetch(k + A * T);
  }
  asm volatile("" : : "v"(line));
  TileSum<kBlock> ts;
  ts.begin(block, U);
  own = team_sum(own, T);
  if (lane == 0 && i >= 0) ubar[i] = 0.0 - own;
  __syncthreads();
  ts.template sum<1>(s_t, part + u0);
}

template <typename WT, typename IOT>
gf_status launch_apply(gf_ctx *ctx, const gf_nbr *nbr, const void *w, unsigned mask, const void *u, void *out,
                       int only_unit = -1, int team_override = 0) {
  LaunchUnit units[2 * GF_NBAND];
  const int nu = launch_units(nbr, units);
  const IOT *uu = (const IOT *)u;
  IOT *oo = (IOT *)out;
  unsigned done = 0;  // units that went with an earlier launch
  for (int q = 0; q < nu; ++q) {
    if ((only_unit >= 0 && q != only_unit) || ((done >> q) & 1u)) continue;
    const LaunchUnit &lu = units[q];
    const int T = team_override > 0 ? team_override : ctx->ateam[lu.model][lu.band];
    const int32_t *sched = nbr->grouped + lu.row0;
    const int64_t nrows = lu.nrows;
    ProfScope prof(ctx, lu.model == 0 ? "apply_3d" : "apply_film");
    if (lu.tiled) {
      ApplyTiles at;
      at.grouped = nbr->grouped;
      at.nranges = 1;
      at.tile0[0] = lu.tile0;
      at.ntiles[0] = lu.ntiles;
      at.row0[0] = lu.row0;
      at.nrows[0] = lu.nrows;
      at.tile0[1] = at.ntiles[1] = at.row0[1] = at.nrows[1] = 0;
      int64_t blocks = lu.ntiles;
      int tmax = lu.tile_max;
      // one launch for both models' tiles
      for (int q2 = q + 1; q2 < nu && only_unit < 0; ++q2) {
        const LaunchUnit &l2 = units[q2];
        if (!l2.tiled || ctx->ateam[l2.model][l2.band] != T) continue;
        at.nranges = 2;
        at.tile0[1] = l2.tile0;
        at.ntiles[1] = l2.ntiles;
        at.row0[1] = l2.row0;
        at.nrows[1] = l2.nrows;
        blocks = (lu.ntiles + 7) / 8 * 8 + l2.ntiles;
        tmax = std::max(tmax, l2.tile_max);
        done |= 1u << q2;
      }
      at.cap = std::min(tmax, tile_capacity(ctx, kApplyCap));
      const dim3 tgrid(grid_for(blocks, 1)), tblock(kTileRows * std::min(T, 32));
      const size_t lds = sizeof(double) * at.cap;
      const bool nt = sizeof(WT) == 4 && (double)nbr->nnz * 4 * sizeof(WT) > kApplyStream;
#define GF_APPLY_TILE_NT(TT, NT)                                                                                       \
  hipLaunchKernelGGL((k_apply_tile<TT, WT, IOT, NT>), tgrid, tblock, lds, ctx->stream, at, nbr->row_ptr, nbr->col,  \
                     nbr->slot, nbr->tile_off, nbr->tile_u, w, mask, uu, oo, nbr->n)
#define GF_APPLY_TILE(TT)                                                                                              \
  if (nt && TT >= 8) GF_APPLY_TILE_NT(TT, (sizeof(WT) == 4 && TT >= 8));                                               \
  else GF_APPLY_TILE_NT(TT, false)
      switch (std::min(T, 32)) {
        case 4: GF_APPLY_TILE(4); break;
        case 8: GF_APPLY_TILE(8); break;
        case 16: GF_APPLY_TILE(16); break;
        default: GF_APPLY_TILE(32); break;
      }
#undef GF_APPLY_TILE
#undef GF_APPLY_TILE_NT
      GF_LAUNCH_CHECK(ctx);
      continue;
    }
    const dim3 grid(grid_for(nrows * T, kBlock)), block(kBlock);
    switch (T) {
      case 4: hipLaunchKernelGGL((k_apply<4, WT, IOT>), grid, block, 0, ctx->stream, sched, nrows, nbr->row_ptr, nbr->col, w, mask, uu, oo, nbr->n); break;
      case 8: hipLaunchKernelGGL((k_apply<8, WT, IOT>), grid, block, 0, ctx->stream, sched, nrows, nbr->row_ptr, nbr->col, w, mask, uu, oo, nbr->n); break;
      case 16: hipLaunchKernelGGL((k_apply<16, WT, IOT>), grid, block, 0, ctx->stream, sched, nrows, nbr->row_ptr, nbr->col, w, mask, uu, oo, nbr->n); break;
      case 32: hipLaunchKernelGGL((k_apply<32, WT, IOT>), grid, block, 0, ctx->stream, sched, nrows, nbr->row_ptr, nbr->col, w, mask, uu, oo, nbr->n); break;
      default: hipLaunchKernelGGL((k_apply<64, WT, IOT>), grid, block, 0, ctx->stream, sched, nrows, nbr->row_ptr, nbr->col, w, mask, uu, oo, nbr->n); break;
    }
    GF_LAUNCH_CHECK(ctx);
  }
  return GF_OK;
}
}  // namespace

// Team-size search for the application kernel (FP64 field), per launch unit.
gf_status tune_apply(gf_ctx *ctx, const gf_nbr *nbr, const void *w, gf_dtype wtype) {
  double *u = nullptr, *out = nullptr;
  if (!device_alloc(*ctx->pool, (void **)&u, sizeof(double) * nbr->n)) return set_error(ctx, GF_ENOMEM, "tuning buffer");
  if (!device_alloc(*ctx->pool, (void **)&out, sizeof(double) * 4 * nbr->n)) {
    (void)hipFree(u);
    return set_error(ctx, GF_ENOMEM, "tuning buffer");
  }
  (void)hipMemsetAsync(u, 0, sizeof(double) * nbr->n, ctx->stream);
  hipEvent_t e0, e1;
  (void)hipEventCreate(&e0);
  (void)hipEventCreate(&e1);
  const int sizes[5] = {4, 8, 16, 32, 64};
  gf_status st = GF_OK;
  LaunchUnit units[2 * GF_NBAND];
  const int nu = launch_units(nbr, units);
  for (int q = 0; q < nu && !st; ++q) {
    float best = INFINITY;
    int bestT = ctx->ateam[units[q].model][units[q].band];
    // tiled blocks hold kTileRows teams: at most 32 lanes each
    const int nsizes = units[q].tiled ? 4 : 5;
    for (int t = 0; t < nsizes && !st; ++t) {
      float times[3];
      for (int rep = -1; rep < 3 && !st; ++rep) {
        if (rep >= 0) (void)hipEventRecord(e0, ctx->stream);
        st = (wtype == GF_F32) ? launch_apply<float, double>(ctx, nbr, w, 0xF, u, out, q, sizes[t])
                               : launch_apply<double, double>(ctx, nbr, w, 0xF, u, out, q, sizes[t]);
        if (rep >= 0) {
          (void)hipEventRecord(e1, ctx->stream);
          (void)hipEventSynchronize(e1);
          (void)hipEventElapsedTime(&times[rep], e0, e1);
        }
      }
      if (st) break;
      std::sort(times, times + 3);
      if (times[1] < best) { best = times[1]; bestT = sizes[t]; }
    }
    ctx->ateam[units[q].model][units[q].band] = bestT;
  }
  (void)hipStreamSynchronize(ctx->stream);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)hipFree(u);
  (void)hipFree(out);
  return st;
}

extern "C" gf_status gf_apply_stencil(gf_ctx *ctx, const gf_nbr *nbr, gf_dtype wtype, const void *w, unsigned op_mask,
                                      gf_dtype io, const void *u, void *out) {
  if (!ctx) return GF_EINVAL;
  if (!nbr) return set_error(ctx, GF_EINVAL, "neighbour handle is NULL");
  gf_status st = check_nbr(ctx, nbr, nbr->n);
  if (st) return st;
  if (nbr->cross) return set_error(ctx, GF_EINVAL, "stencils live on same-model neighbourhoods");
  if (!w || !u || !out) return set_error(ctx, GF_EINVAL, "w, u and out are required");
  if (reinterpret_cast<uintptr_t>(w) & 15) return set_error(ctx, GF_EINVAL, "w must be 16-byte aligned");
  if ((op_mask & 0xF) == 0 || (op_mask & ~0xFu)) return set_error(ctx, GF_EINVAL, "op_mask must select 1..4 operators");
  if ((wtype != GF_F32 && wtype != GF_F64) || (io != GF_F32 && io != GF_F64))
    return set_error(ctx, GF_EINVAL, "unknown dtype");
  GF_HIP(ctx, hipSetDevice(ctx->device));
  if (wtype == GF_F32) {
    return io == GF_F64 ? launch_apply<float, double>(ctx, nbr, w, op_mask, u, out)
                        : launch_apply<float, float>(ctx, nbr, w, op_mask, u, out);
  }
  return io == GF_F64 ? launch_apply<double, double>(ctx, nbr, w, op_mask, u, out)
                      : launch_apply<double, float>(ctx, nbr, w, op_mask, u, out);
}

extern "C" gf_status gf_apply_stencil_adjoint(gf_ctx *ctx, const gf_nbr *nbr, gf_dtype wtype, const void *w,
                                              unsigned op_mask, const double *ybar, double *ubar) {
  if (!ctx) return GF_EINVAL;
  if (!nbr) return set_error(ctx, GF_EINVAL, "neighbour handle is NULL");
  gf_status st = check_nbr(ctx, nbr, nbr->n);
  if (st) return st;
  if (nbr->cross) return set_error(ctx, GF_EINVAL, "stencils live on same-model neighbourhoods");
  if (!w || !ybar || !ubar) return set_error(ctx, GF_EINVAL, "w, ybar and ubar are required");
  if (reinterpret_cast<uintptr_t>(w) & 15) return set_error(ctx, GF_EINVAL, "w must be 16-byte aligned");
  if ((op_mask & 0xF) == 0 || (op_mask & ~0xFu)) return set_error(ctx, GF_EINVAL, "op_mask must select 1..4 operators");
  if (wtype != GF_F32 && wtype != GF_F64) return set_error(ctx, GF_EINVAL, "unknown dtype");
  GF_HIP(ctx, hipSetDevice(ctx->device));
  if (all_tiled(nbr)) {
    if ((st = ensure_tile_transpose(ctx, const_cast<gf_nbr *>(nbr)))) return st;
    Arena ar;
    if ((st = ensure_scratch(ctx, arena_bytes({sizeof(double) * (size_t)nbr->tile_total}), &ar))) return st;
    double *part = ar.take<double>(nbr->tile_total);
    const TileRows tr = tile_rows(nbr);
    const size_t lds = sizeof(double) * (kTileRows * (size_t)nbr->max_row + 1);
    const bool nt = wtype == GF_F32 && (double)nbr->nnz * 16 > kApplyStream;
    ProfScope prof(ctx, "apply_adjoint");
#define GF_ADJ_T(WT, K, NT)                                                                                        \
  hipLaunchKernelGGL((k_apply_adjoint_tile<WT, K, NT>), dim3((unsigned)nbr->ntiles), dim3(kBlock), lds, ctx->stream, tr, \
                     nbr->row_ptr, nbr->tile_off, nbr->tperm_off, nbr->tperm, nbr->tself, nbr->slot, w, op_mask, ybar, nbr->n, \
                     part, ubar)
#define GF_ADJ_TK(WT, NT)                  \
  switch (__builtin_popcount(op_mask)) {   \
    case 1: GF_ADJ_T(WT, 1, NT); break;    \
    case 2: GF_ADJ_T(WT, 2, NT); break;    \
    case 3: GF_ADJ_T(WT, 3, NT); break;    \
    default: GF_ADJ_T(WT, 4, NT); break;   \
  }
    if (nt) {
      GF_ADJ_TK(float, true)
    } else if (wtype == GF_F32) {
      GF_ADJ_TK(float, false)
    } else {
      GF_ADJ_TK(double, false)
    }
#undef GF_ADJ_TK
#undef GF_ADJ_T
    GF_LAUNCH_CHECK(ctx);
    launch_places_sum<1>(ctx->stream, nbr, part, ubar);
    GF_LAUNCH_CHECK(ctx);
    return GF_OK;
  }
  if ((st = ensure_rev(ctx, const_cast<gf_nbr *>(nbr)))) return st;
  const dim3 block(kBlock);
  ProfScope prof(ctx, "apply_adjoint");
#define GF_ADJ(WT, K)                                                                                            \
  hipLaunchKernelGGL((k_apply_adjoint<WT, K>), dim3(grid_for(nbr->n * adj_team<WT>(K), kBlock)), block, 0,         \
                     ctx->stream, nbr->row_ptr, nbr->col, nbr->rev, w, op_mask, ybar, nbr->n, ubar)
#define GF_ADJ_K(WT)                       \
  switch (__builtin_popcount(op_mask)) {   \
    case 1: GF_ADJ(WT, 1); break;          \
    case 2: GF_ADJ(WT, 2); break;          \
    case 3: GF_ADJ(WT, 3); break;          \
    default: GF_ADJ(WT, 4); break;         \
  }
  if (wtype == GF_F32) {
    GF_ADJ_K(float)
  } else {
    GF_ADJ_K(double)
  }
#undef GF_ADJ_K
#undef GF_ADJ
  GF_LAUNCH_CHECK(ctx);
  return GF_OK;
}
