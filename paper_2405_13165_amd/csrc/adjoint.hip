// Gradient of L(out), out_i^s = sum_{j != i} c_ij^s (u_j - u_i), with respect
// to particle positions through the stencil weights.
//
// For particle i, with G = sum_j w_j phi_j phi_j^T, L_i = sum_s ybar_i^s L(out)_s
// is sum_j w_j (phi_j . Lambda) du_j with du_j = u_j - u_i and Lambda =
// G^{-1} sum_s ybar_i^s d_s: the selected operators enter only through Lambda
// (on a film ybar_x, ybar_y, ybar_z first give the tangential ones).  With
// mu = G^{-1} sum_j w_j du_j phi_j, r_j = du_j - mu . phi_j (the residual of the
// fit of u) and a_j = phi_j . Lambda, the chain rule gives
//   dbar_j = w_j (r_j (d phi / d d)^T Lambda - a_j (d phi / d d)^T mu) + r_j a_j dw/dd
// for the offset d = x_j - x_i; x_j gains dbar_j, x_i loses it.  The stencils
// are recomputed (nothing is stored but the neighbour lists).
//
// Where every row is tiled, a tile's entries are added up per neighbour in LDS
// through the transposed tile and then per particle; otherwise (a row of more
// than kTileBandRow neighbours, or tiles too wide for LDS) per-entry
// contributions go to scratch with the rows laid out in grouped (Morton) order
// and are gathered per particle, in the same order, through the reverse-edge
// map: the twin entry (j, i) of (i, j) lies in a Morton-near row, so the gather
// stays in L2.  No atomics: the result is deterministic, and as the tiles follow
// the cell order, which is fixed, the same for every handle of a cloud.
// Rows whose forward stencils are zero (status 2 or 3 of the stencil call,
// when the caller passes those statuses) contribute nothing, and so do rows
// whose Gram matrix is not positive definite.
#include "stencil_common.h"

using namespace gfdm_dev;

namespace {
constexpr int kBlock = 256;
constexpr int kT = 8;
constexpr size_t kTilePart = 40;          // bytes staged per distinct neighbour of a tile
constexpr size_t kAdjTileLds = 48 * 1024;  // with the teams' 10 KB two tiles still fit a CU, wider ones take the general path

struct AArgs {
  const double *x, *y, *z, *h, *nx, *ny, *nz;
  const double4 *pos;  // (x, y, z, h) packed per particle
  const int64_t *row_ptr;
  const int32_t *col;
  const int32_t *sched;
  int64_t nrows, n;
  WeightFn wf;
  unsigned mask;
  const double *u, *ybar;
  const int8_t *status;  // forward stencil statuses (may be NULL)
  double *dbar;  // [nnz][3], rows in grouped order
  double *xbar;  // [n][3]: each row subtracts its own entries' sum here
  const int64_t *gbase;  // per team: offset of its row in dbar (grouped row offsets)
};

// A team of kT lanes per particle, in the form of the batched stencil kernel:
// pass 1 adds up the weighted moments of the offsets and sum_j w_j du_j phi_j
// (one walk: neither needs the other), the team inverts G (Gauss-Jordan, lane
// owns rows lane + q kT) and shares Lambda and mu through its LDS area, pass 2
// forms the entries.  Everything is written in the unscaled offsets d (physical
// targets); the weights leave out their normalising factor 1 / (1 - e^{-a}): a
// common factor of the weights cancels from the stencils and from every term
// above (G and sum w du phi scale with it, Lambda with its inverse).
template <int M>
constexpr int adj_lds_doubles() {  // per team: moments / pivot row / Lambda and mu
  return (cmax(cmax(nmom<M>() + M, red_lanes(kT) * red_lanes(kT)), cmax(M + 1, 2 * M)) + 1) & ~1;
}

// Visit the entries k = lane, lane + T, ... of a row of n >= 1 entries at CSR
// entry b, calling body(k, j, position of j, field value of j); the
// column two steps ahead and the position and field value one step ahead
// are in flight during the arithmetic.  Loads past the row's end read its
// last entry (valid, never used), so every load is unconditional.
template <int T, class Body>
__device__ inline void adj_walk(const AArgs &a, int64_t b, int n, int lane, Body &&body) {
  const int kmax = n - 1;
  int32_t jc = a.col[b + min(lane, kmax)];
  int32_t jn = a.col[b + min(lane + T, kmax)];
  double4 pc = a.pos[jc];
  double uc = a.u[jc];
#pragma unroll 1
  for (int k = lane; k < n; k += T) {
    const int32_t j = jc;
    const double4 pj = pc;
    const double uj = uc;
    jc = jn;
    pc = a.pos[jn];
    uc = a.u[jn];
    jn = a.col[b + min(k + 2 * T, kmax)];
    body(k, j, pj, uj);
  }
}

// unnormalised weight e^{-a q^2} - e^{-a}, q^2 = |d|^2 / r^2, r = (h_i + h_j) / 2;
// e = e^{-a q^2} and ir2 = 1 / r^2 give dw/dd = -2 a e ir2 d.  Equal
// supports take the row's 1 / h_i^2; others 1 / r^2 from the reciprocal
// estimate and two Newton steps
template <bool UNI = false>  // UNI: all supports are known to be equal
__device__ inline double adj_weight(const WeightFn &wf, double hi, double ir2_row, double hj, double d2, double &e,
                                    double &ir2) {
  ir2 = ir2_row;
  if (!UNI && hj != hi) {
    const double r = 0.5 * (hi + hj), rr = r * r;
    double q = __builtin_amdgcn_rcp(rr);
    q = fma(q, fma(-rr, q, 1.0), q);
    ir2 = fma(q, fma(-rr, q, 1.0), q);
  }
  e = exp2_raw(d2 * (ir2 * wf.nl2a));
  return e - wf.ea;
}

// V += w du phi
template <int M>
__device__ inline void adj_add_fit(double *V, double cw, double X, double Y, double Z) {
  V[0] += cw;
  if constexpr (M == 10) {
    const double cx = cw * X, cy = cw * Y, cz = cw * Z;
    V[1] += cx; V[2] += cy; V[3] += cz;
    V[4] = fma(cx, X, V[4]); V[5] = fma(cy, Y, V[5]); V[6] = fma(cz, Z, V[6]);
    V[7] = fma(cx, Y, V[7]); V[8] = fma(cx, Z, V[8]); V[9] = fma(cy, Z, V[9]);
  } else {
    const double cx = cw * X, cy = cw * Y;
    V[1] += cx; V[2] += cy;
    V[3] = fma(cx, X, V[3]); V[4] = fma(cy, Y, V[4]); V[5] = fma(cx, Y, V[5]);
  }
}

// dbar of the entry at offset (dx, dy, dz)
template <int M>
__device__ inline void adj_entry(const RowGeom &g, const double *lam, const double *mu, double dx, double dy, double dz,
                                 double w, double du, double de, double out[3]) {
  double X, Y, Z, lx, ly, lz, mx, my, mz;
  local_raw<M>(g, dx, dy, dz, X, Y, Z);
  const double al = poly_grad<M>(lam, X, Y, Z, lx, ly, lz);
  const double r = du - poly_grad<M>(mu, X, Y, Z, mx, my, mz);
  const double wr = w * r, wa = w * al, f = (r * al) * de;
  const double gx = fma(wr, lx, -(wa * mx)), gy = fma(wr, ly, -(wa * my));
  if constexpr (M == 10) {
    out[0] = fma(f, dx, gx);
    out[1] = fma(f, dy, gy);
    out[2] = fma(f, dz, fma(wr, lz, -(wa * mz)));
  } else {
    out[0] = fma(f, dx, fma(gy, g.t2[0], gx * g.t1[0]));
    out[1] = fma(f, dy, fma(gy, g.t2[1], gx * g.t1[1]));
    out[2] = fma(f, dz, fma(gy, g.t2[2], gx * g.t1[2]));
  }
}

// G from the moments, G^{-1}, Lambda and mu (squares' terms doubled, see
// poly_grad) at sm[0 .. M) and sm[M .. 2M); false if G is not positive definite
// (the same on every lane of the team)
template <int M>
__device__ inline bool adj_solve(const RowGeom &g, double (&mv)[nmom<M>() + M], double (&yb)[4],
                                 int lane, double *sm) {
  constexpr int T = kT, NR = (M + T - 1) / T;
  team_vector_sum<nmom<M>() + M, T>(mv, lane, sm);
  double row[NR][M], V[M];
#pragma unroll
  for (int r = 0; r < M; ++r) V[r] = sm[nmom<M>() + r];
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int r = lane + q * T;
    const bool own = r < M;
#pragma unroll
    for (int c = 0; c < M; ++c) {
      const int mi = own ? (M == 10 ? kGram3.v[r][c] : kGram2.v[r][c]) : 0;
      row[q][c] = own ? sm[mi] : 0.0;
    }
  }
  wave_sync();  // the pivot rows overwrite the moments
  if (!team_gauss_jordan<M, T>(row, lane, sm)) return false;
  // sum_s ybar_s t_s: t_s the target of stencil s (on a film the tangential ones, s = 0, 1)
  if constexpr (M == 6) {
    const double y1 = g.t1[0] * yb[0] + g.t1[1] * yb[1] + g.t1[2] * yb[2];
    const double y2 = g.t2[0] * yb[0] + g.t2[1] * yb[1] + g.t2[2] * yb[2];
    yb[0] = y1; yb[1] = y2; yb[2] = 0.0;
  }
  double tc[M];
#pragma unroll
  for (int c = 0; c < M; ++c) {
    tc[c] = 0.0;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (target_coef<M>(s, c) != 0.0) tc[c] += target_coef<M>(s, c) * yb[s];
  }
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int r = lane + q * T;
    if (r < M) {
      double l = 0.0, m = 0.0;
#pragma unroll
      for (int c = 0; c < M; ++c) {
        if (c >= 1 && c <= (M == 10 ? 6 : 4)) l = fma(row[q][c], tc[c], l);
        m = fma(row[q][c], V[c], m);
      }
      const double f = (M == 10 ? r >= 4 && r <= 6 : r == 3 || r == 4) ? 2.0 : 1.0;
      sm[r] = f * l;
      sm[M + r] = f * m;
    }
  }
  wave_sync();
  return true;
}

// ybar of row i, per stencil s (zero if not selected)
__device__ inline void adj_ybar(const AArgs &a, int32_t i, double (&yb)[4]) {
  int q = 0;
#pragma unroll
  for (int s = 0; s < 4; ++s) yb[s] = (a.mask & (1u << s)) ? a.ybar[(int64_t)(q++) * a.n + i] : 0.0;
}

template <int M>
__device__ inline void adj_geom(const AArgs &a, int32_t i, RowGeom &g) {
  g.xi = a.x[i]; g.yi = a.y[i]; g.zi = a.z[i]; g.hi = a.h[i]; g.inv_h = 1.0;  // unscaled monomials
  if constexpr (M == 6) tangent_frame(a.nx[i], a.ny[i], a.nz[i], g.t1, g.t2);
}

template <int M>
__device__ void adjoint_row(const AArgs &a, int32_t i, int64_t ob, int lane, double *sm) {
  constexpr int T = kT;
  const int64_t b = a.row_ptr[i];
  const int n = (int)(a.row_ptr[i + 1] - b);
  RowGeom g;
  adj_geom<M>(a, i, g);
  auto zero_out = [&]() {
    for (int k = lane; k < n; k += T) {
      double *d = a.dbar + 3 * (ob + k);
      d[0] = 0.0; d[1] = 0.0; d[2] = 0.0;
    }
  };
  // n < M (status 3) and rank-deficient rows (status 2) have constant zero stencils
  if (n < M || (a.status && a.status[i] >= 2)) {
    zero_out();
    return;
  }
  const double ir2_row = 1.0 / (g.hi * g.hi), ui = a.u[i];
  double yb[4];
  adj_ybar(a, i, yb);
  double mv[nmom<M>() + M];  // moments, then sum w du phi
#pragma unroll
  for (int p = 0; p < nmom<M>() + M; ++p) mv[p] = 0.0;
  adj_walk<T>(a, b, n, lane, [&](int, int32_t j, const double4 &pj, double uj) {
    const double dx = pj.x - g.xi, dy = pj.y - g.yi, dz = pj.z - g.zi;
    double e, ir2, X, Y, Z;
    const double w = adj_weight(a.wf, g.hi, ir2_row, pj.w, fma(dz, dz, fma(dy, dy, dx * dx)), e, ir2);
    local_raw<M>(g, dx, dy, dz, X, Y, Z);
    moments_add_raw<M>(mv, w, X, Y, Z);
    adj_add_fit<M>(mv + nmom<M>(), j != i ? w * (uj - ui) : 0.0, X, Y, Z);
  });
  if (!adj_solve<M>(g, mv, yb, lane, sm)) {
    zero_out();
    return;
  }
  double lam[M], mu[M];
#pragma unroll
  for (int r = 0; r < M; ++r) {
    lam[r] = sm[r];
    mu[r] = sm[M + r];
  }
  double own[3] = {0.0, 0.0, 0.0};  // this lane's share of sum_j dbar(i, j)
  // each entry's dbar is stored one step late, at the start of the next
  // step: a load and a store in flight count against one counter, and the
  // wait for the next entry's column would otherwise wait for the store
  double po[3] = {0.0, 0.0, 0.0};
  int kp = -1;
  auto flush_prev = [&]() {
    if (kp >= 0) {
      double *out = a.dbar + 3 * (ob + kp);
      out[0] = po[0]; out[1] = po[1]; out[2] = po[2];
    }
  };
  adj_walk<T>(a, b, n, lane, [&](int k, int32_t j, const double4 &pj, double uj) {
    flush_prev();
    kp = k;
    if (j == i) {
      po[0] = 0.0; po[1] = 0.0; po[2] = 0.0;
      return;
    }
    const double dx = pj.x - g.xi, dy = pj.y - g.yi, dz = pj.z - g.zi;
    double e, ir2;
    const double w = adj_weight(a.wf, g.hi, ir2_row, pj.w, fma(dz, dz, fma(dy, dy, dx * dx)), e, ir2);
    adj_entry<M>(g, lam, mu, dx, dy, dz, w, uj - ui, -2.0 * a.wf.alpha * e * ir2, po);
    own[0] += po[0];
    own[1] += po[1];
    own[2] += po[2];
  });
  flush_prev();
  // x_i loses every dbar(i, j), whether or not (j, i) is listed
#pragma unroll
  for (int c = 0; c < 3; ++c) own[c] = team_sum(own[c], T);
  if (lane == 0) {
#pragma unroll
    for (int c = 0; c < 3; ++c) a.xbar[3 * (int64_t)i + c] -= own[c];
  }
}

template <int M>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(M == 6 ? 4 : 3))) k_adjoint_x(AArgs a) {
  __shared__ double smem[(kBlock / kT) * adj_lds_doubles<M>()];
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t team = gt / kT;
  const int lane = (int)(gt % kT);
  if (team >= a.nrows) return;
  adjoint_row<M>(a, a.sched[team], a.gbase[team], lane, smem + (threadIdx.x / kT) * adj_lds_doubles<M>());
}

// A block per tile, a team of kT lanes per row.  The tile's positions and field
// values are staged in LDS; each lane keeps the dbar of its entries (at most
// Q) in registers, and one component at a time they go to LDS,
// over the staged positions, in tile order, where each distinct neighbour's are
// added up in row order through the transposed tile.  part: see k_places_sum.
//
// What bounds it: FP64 issue (4500 vector instructions per wave and tile, 470 us
// of it on 80^3 particles) at two waves per SIMD, which the 96 registers of
// dbar allow: 1035 us + 64 us (k_places_sum).  Writing every entry's dbar to
// memory and gathering its twin took 1061 + 531 us; three waves per SIMD spill
// (1800 us).
struct ATile {
  TileRows tr;
  int64_t t0;  // the model's first tile
  const int64_t *tile_off, *tperm_off;
  const int32_t *tile_u;
  const uint16_t *slot, *tperm, *tself;
  double *part;
};
// Entries per lane.  Film rows of at most 64 entries, by the film's own longest
// row, leave registers for a third wave per SIMD: 159 us on 500^2 film rows of 28
// entries against 220 (the row kernel of before took 168 to 246 by the operators,
// and about 50 for its gather); 3D rows at three waves spill.
constexpr int kShortQ = 8, kLongQ = kTileBandRow / kT;

struct AdjTile {
  const double2 *sxy, *szu;
  const double *sh;
  const uint16_t *sl;  // the row's slots
};
// The row of a team: its dbar entries (lane + q kT) to dd, their sum from xbar.
// Both passes take their entries two at a time without branches (an entry past
// the row's end is its last one with weight zero), so that the loads and the
// long chain of one weight overlap another's.  Returns false where the row
// contributes nothing (dd is not set).
template <int M, int Q, bool UNI>
__device__ inline bool adj_tile_row(const AArgs &a, const AdjTile &tl, const RowGeom &g, int32_t i, int n, int lane,
                                    double ui, int self, bool on, double (&yb)[4], const double (&xb)[3], double *sm,
                                    double (&dd)[Q][3]) {
  constexpr int T = kT;
  const double ir2_row = 1.0 / (g.hi * g.hi);
  uint32_t ss[Q / 2];
  if (on) {
    double mv[nmom<M>() + M];  // moments, then sum w du phi
#pragma unroll
    for (int p = 0; p < nmom<M>() + M; ++p) mv[p] = 0.0;
    // slots two steps ahead (past the row's end its last entry)
    int s[2], sn[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      s[u] = tl.sl[min(lane + u * T, n - 1)];
      sn[u] = tl.sl[min(lane + (2 + u) * T, n - 1)];
    }
#pragma unroll 1
    for (int k = lane; k - lane < n; k += 2 * T) {  // (the team's lanes leave together)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const double2 pxy = tl.sxy[s[u]], pzu = tl.szu[s[u]];
        const double hj = UNI ? g.hi : tl.sh[s[u]];
        const double dx = pxy.x - g.xi, dy = pxy.y - g.yi, dz = pzu.x - g.zi, du = pzu.y - ui;
        double e, ir2, X, Y, Z;
        double w = adj_weight<UNI>(a.wf, g.hi, ir2_row, hj, fma(dz, dz, fma(dy, dy, dx * dx)), e, ir2);
        if (k + u * T >= n) w = 0.0;
        local_raw<M>(g, dx, dy, dz, X, Y, Z);
        moments_add_raw<M>(mv, w, X, Y, Z);
        adj_add_fit<M>(mv + nmom<M>(), s[u] != self ? w * du : 0.0, X, Y, Z);
        s[u] = sn[u];
        sn[u] = tl.sl[min(k + (4 + u) * T, n - 1)];
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint32_t v = tl.sl[min(lane + q * T, n - 1)];
      ss[q / 2] = q & 1 ? ss[q / 2] | v << 16 : v;
    }
    on = adj_solve<M>(g, mv, yb, lane, sm);
  }
  if (!on) return false;
  double lam[M], mu[M], own[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int r = 0; r < M; ++r) {
    lam[r] = sm[r];
    mu[r] = sm[M + r];
  }
#pragma unroll
  for (int q2 = 0; q2 < Q; q2 += 2) {
    if (q2 * T < n) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int q = q2 + u, s = u ? ss[q / 2] >> 16 : ss[q / 2] & 0xffff;
        const double2 pxy = tl.sxy[s], pzu = tl.szu[s];
        const double hj = UNI ? g.hi : tl.sh[s];
        const double dx = pxy.x - g.xi, dy = pxy.y - g.yi, dz = pzu.x - g.zi;
        double e, ir2, d[3];
        const double w = adj_weight<UNI>(a.wf, g.hi, ir2_row, hj, fma(dz, dz, fma(dy, dy, dx * dx)), e, ir2);
        adj_entry<M>(g, lam, mu, dx, dy, dz, w, pzu.y - ui, -2.0 * a.wf.alpha * e * ir2, d);
        const bool in = lane + q * T < n && s != self;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          dd[q][c] = in ? d[c] : 0.0;
          own[c] += dd[q][c];
        }
      }
    }
  }
  // x_i loses every dbar(i, j), whether or not (j, i) is listed
#pragma unroll
  for (int c = 0; c < 3; ++c) own[c] = team_sum(own[c], T);
  if (lane == 0) {
#pragma unroll
    for (int c = 0; c < 3; ++c) a.xbar[3 * (int64_t)i + c] = xb[c] - own[c];
  }
  return true;
}

template <int M, int Q>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(Q > kShortQ ? 2 : 3)))
k_adjoint_tile(AArgs a, ATile at, int cap) {
  constexpr int T = kT;
  static_assert(kBlock == kTileRows * kT, "a team per row of the tile");
  extern __shared__ double s_tile[];  // cap x (x, y), cap x (z, u), cap x h; then the terms of one component
  __shared__ double smem[kTileRows * adj_lds_doubles<M>()];
  __shared__ int32_t s_len[kTileRows], s_off[kTileRows + 1];
  const int64_t t = at.t0 + xcd_block(blockIdx.x, gridDim.x);
  const int team = threadIdx.x / T, lane = threadIdx.x % T;
  const int32_t i = tile_row(at.tr, t, team);
  const int64_t b = i >= 0 ? a.row_ptr[i] : 0;
  int n = i >= 0 ? (int)(a.row_ptr[i + 1] - b) : 0;
  const int64_t u0 = at.tile_off[t];
  const int U = (int)(at.tile_off[t + 1] - u0);
  // what the row needs besides the tile, requested before the staging so that
  // one latency covers both (past the model's last row: the tile's first row)
  const int32_t ir = i >= 0 ? i : tile_row(at.tr, t, 0);
  RowGeom g;
  g.xi = a.x[ir]; g.yi = a.y[ir]; g.zi = a.z[ir]; g.hi = a.h[ir]; g.inv_h = 1.0;
  double nrm[3] = {0.0, 0.0, 0.0};
  if constexpr (M == 6) { nrm[0] = a.nx[ir]; nrm[1] = a.ny[ir]; nrm[2] = a.nz[ir]; }
  const double ui = a.u[ir];
  double yb[4], xb[3];
  adj_ybar(a, ir, yb);
#pragma unroll
  for (int c = 0; c < 3; ++c) xb[c] = a.xbar[3 * (int64_t)ir + c];
  const int8_t status = a.status ? a.status[ir] : 0;
  const int self = at.tself[kTileRows * t + team];
  double2 *sxy = reinterpret_cast<double2 *>(s_tile), *szu = sxy + cap;
  double *sh = reinterpret_cast<double *>(szu + cap);
  const uint16_t *block = at.tperm + 64 * at.tperm_off[t];
  const uint32_t line = TileSum<kBlock>::warm(block, at.tperm_off[t + 1] - at.tperm_off[t]);
  const double h0 = a.h[at.tile_u[u0]];  // (a tile lists at least its own rows)
  bool same = true;
  double v[kStage][5];
  stage_tile<kBlock>(
      at.tile_u + u0, U,
      [&](int q, int32_t j) {
        v[q][0] = a.x[j]; v[q][1] = a.y[j]; v[q][2] = a.z[j]; v[q][3] = a.u[j]; v[q][4] = a.h[j];
      },
      [&](int q, int s) {
        sxy[s] = make_double2(v[q][0], v[q][1]);
        szu[s] = make_double2(v[q][2], v[q][3]);
        sh[s] = v[q][4];
        same = same && v[q][4] == h0;
      });
  if (lane == 0) s_len[team] = n;
  if constexpr (M == 6) tangent_frame(nrm[0], nrm[1], nrm[2], g.t1, g.t2);
  bool on = n >= M && status < 2;  // the same on every lane of the team
  asm volatile("" : : "v"(line));
  const bool uni = __syncthreads_and(same);
  if (threadIdx.x < 64) {  // entries of the tile before each row
    const int len = threadIdx.x < kTileRows ? s_len[threadIdx.x] : 0;
    int inc = len;
#pragma unroll
    for (int o = 1; o < kTileRows; o <<= 1) {
      const int v = __shfl_up(inc, o, 64);
      if ((int)threadIdx.x >= o) inc += v;
    }
    if (threadIdx.x < kTileRows) {
      s_off[threadIdx.x] = inc - len;
      if (threadIdx.x == kTileRows - 1) s_off[kTileRows] = inc;
    }
  }
  double *sm = smem + team * adj_lds_doubles<M>();
  double dd[Q][3];
  const AdjTile tile{sxy, szu, sh, at.slot + b};
  if (uni)
    on = adj_tile_row<M, Q, true>(a, tile, g, i, n, lane, ui, self, on, yb, xb, sm, dd);
  else
    on = adj_tile_row<M, Q, false>(a, tile, g, i, n, lane, ui, self, on, yb, xb, sm, dd);
  if (!on) {
#pragma unroll
    for (int q = 0; q < Q; ++q) dd[q][0] = dd[q][1] = dd[q][2] = 0.0;
  }
  TileSum<kBlock> ts;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    __syncthreads();
    double *mine = s_tile + s_off[team] + lane;
    asm volatile("" : "+v"(n));
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (lane + q * T < n) mine[q * T] = dd[q][c];
    if (threadIdx.x == 0) s_tile[s_off[kTileRows]] = 0.0;  // the term of the padding
    ts.begin(block, U);
    __syncthreads();
    ts.template sum<3>(s_tile, at.part + 3 * u0 + c);
  }
}

// xbar_j += sum over entries (j, i) of row j, i != j, of dbar(i, j) (x_j gains
// what row i differentiated with respect to it; the row's own entries were
// subtracted by the row kernel); rows in grouped order, a team of kGT lanes
// per row; the twin dbar(i, j) sits at grev[g] (a Morton-near row).  An entry
// (j, i) without a twin (i a ghost particle whose row holds only itself)
// adds nothing.
constexpr int kGT = 8;  // lanes per row of the gather
// entries per lane and step of the gather (lanes x entries on the mixed cloud:
// 8 x 8 481 us, 8 x 4 497, 16 x 4 488, 4 x 8 526)
constexpr int kGU = 8;
__global__ void __launch_bounds__(kBlock) k_adjoint_gather(const int32_t *__restrict__ grouped,
                                                           const int64_t *__restrict__ grow_ptr,
                                                           const int32_t *__restrict__ grev,
                                                           const double *__restrict__ dbar, int64_t n,
                                                           double *__restrict__ xbar) {
  const int64_t gt = (int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
  const int64_t t = gt / kGT;
  const int lane = (int)(gt % kGT);
  if (t >= n) return;
  const int32_t j = grouped[t];
  const int64_t g0 = grow_ptr[t], g1 = grow_ptr[t + 1];
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
  // kGU entries per lane and step: every twin position of the step, then
  // every dbar record, is requested before the first is used (a straight
  // block, so none of the loads is moved down to its use); reads past the
  // row's end take its last entry, an entry without a twin reads record 0
  // (both valid, neither added)
  const int64_t gl = g1 - 1;  // a step starts only at gk < g1: gl is in the row
#pragma unroll 1
  for (int64_t gk = g0 + lane; gk < g1; gk += kGU * kGT) {
    int32_t tw[kGU];
#pragma unroll
    for (int u = 0; u < kGU; ++u) tw[u] = grev[min(gk + u * kGT, gl)];
    double da[kGU], db[kGU], dc[kGU];
#pragma unroll
    for (int u = 0; u < kGU; ++u) {
      const int64_t q = 3 * (int64_t)(tw[u] >= 0 ? tw[u] : 0);
      da[u] = dbar[q];
      db[u] = dbar[q + 1];
      dc[u] = dbar[q + 2];
    }
#pragma unroll
    for (int u = 0; u < kGU; ++u) {  // in entry order
      const bool on = tw[u] >= 0 && gk + u * kGT < g1;
      s0 += on ? da[u] : 0.0;
      s1 += on ? db[u] : 0.0;
      s2 += on ? dc[u] : 0.0;
    }
  }
  s0 = team_sum(s0, kGT);
  s1 = team_sum(s1, kGT);
  s2 = team_sum(s2, kGT);
  if (lane == 0) {
    xbar[3 * j] += s0;
    xbar[3 * j + 1] += s1;
    xbar[3 * j + 2] += s2;
  }
}
}  // namespace

extern "C" gf_status gf_gfdm_weights_adjoint(gf_ctx *ctx, const gf_particles *p, const gf_nbr *nbr,
                                             const gf_ls_params *params, unsigned op_mask, const double *u,
                                             const double *ybar, const int8_t *status_n, double *xbar_3n) {
  if (!ctx) return GF_EINVAL;
  gf_status st = check_particles(ctx, p, false, false);
  if (st) return st;
  if ((st = check_nbr(ctx, nbr, p->n))) return st;
  if (nbr->cross) return set_error(ctx, GF_EINVAL, "stencils need same-model neighbourhoods");
  if (!u || !ybar || !xbar_3n) return set_error(ctx, GF_EINVAL, "u, ybar and xbar are required");
  if ((op_mask & 0xF) == 0 || (op_mask & ~0xFu)) return set_error(ctx, GF_EINVAL, "op_mask must select 1..4 operators");
  const bool has_film = nbr->group_start[2 * GF_NBAND] > nbr->group_start[GF_NBAND];
  if (has_film && (!p->nx || !p->ny || !p->nz)) return set_error(ctx, GF_EINVAL, "film particles need normals");
  gf_ls_params prm;
  gf_ls_params_default(&prm);
  if (params) prm = *params;
  AArgs a;
  a.x = p->x; a.y = p->y; a.z = p->z; a.h = p->h; a.nx = p->nx; a.ny = p->ny; a.nz = p->nz;
  a.row_ptr = nbr->row_ptr; a.col = nbr->col; a.n = p->n;
  a.wf = make_weight_fn(prm.alpha_w);
  a.mask = op_mask; a.u = u; a.ybar = ybar; a.status = status_n;
  a.xbar = xbar_3n;
  Arena ar;
  auto lds = [&](int m) { return std::max(kTilePart * (size_t)nbr->tile_max[m], sizeof(double) * (kTileRows * (size_t)nbr->model_row[m] + 1)); };
  if (all_tiled(nbr) && std::max(lds(0), lds(1)) <= kAdjTileLds) {
    if ((st = ensure_tile_transpose(ctx, const_cast<gf_nbr *>(nbr)))) return st;
    if ((st = ensure_scratch(ctx, arena_bytes({sizeof(double) * 3 * (size_t)nbr->tile_total}), &ar))) return st;
    ATile at;
    at.tr = tile_rows(nbr);
    at.tile_off = nbr->tile_off; at.tperm_off = nbr->tperm_off; at.tile_u = nbr->tile_u;
    at.slot = nbr->slot; at.tperm = nbr->tperm; at.tself = nbr->tself;
    at.part = ar.take<double>(3 * (size_t)nbr->tile_total);
    for (int m = 0; m < 2; ++m) {
      at.t0 = nbr->tile_start[m];
      const int64_t nt = nbr->tile_start[m + 1] - at.t0;
      if (nt <= 0) continue;
      ProfScope prof(ctx, m == 0 ? "weights_adjoint_3d" : "weights_adjoint_film");
      if (m == 0)
        hipLaunchKernelGGL((k_adjoint_tile<10, kLongQ>), dim3((unsigned)nt), dim3(kBlock), lds(m), ctx->stream, a, at, nbr->tile_max[m]);
      else if (nbr->model_row[1] <= kShortQ * kT)
        hipLaunchKernelGGL((k_adjoint_tile<6, kShortQ>), dim3((unsigned)nt), dim3(kBlock), lds(m), ctx->stream, a, at, nbr->tile_max[m]);
      else
        hipLaunchKernelGGL((k_adjoint_tile<6, kLongQ>), dim3((unsigned)nt), dim3(kBlock), lds(m), ctx->stream, a, at, nbr->tile_max[m]);
      GF_LAUNCH_CHECK(ctx);
    }
    ProfScope prof(ctx, "weights_adjoint_gather");
    launch_places_sum<3>(ctx->stream, nbr, at.part, xbar_3n);
    GF_LAUNCH_CHECK(ctx);
    return GF_OK;
  }
  if ((st = ensure_grouped_rows(ctx, const_cast<gf_nbr *>(nbr)))) return st;
  if ((st = ensure_scratch(ctx, arena_bytes({sizeof(double) * 3 * (size_t)std::max<int64_t>(nbr->nnz, 1),
                                             sizeof(double4) * (size_t)p->n}), &ar)))
    return st;
  a.dbar = ar.take<double>(3 * (size_t)std::max<int64_t>(nbr->nnz, 1));
  double4 *pos = ar.take<double4>(p->n);
  {
    ProfScope prof(ctx, "pack_positions");
    hipLaunchKernelGGL(k_pack_pos, dim3(grid_for(p->n, 256)), dim3(256), 0, ctx->stream, p->x, p->y, p->z, p->h, p->n,
                       pos);
    GF_LAUNCH_CHECK(ctx);
  }
  a.pos = pos;
  for (int m = 0; m < 2; ++m) {
    const int64_t s0 = nbr->group_start[m * GF_NBAND], s1 = nbr->group_start[(m + 1) * GF_NBAND];
    if (s1 <= s0) continue;
    a.sched = nbr->grouped + s0;
    a.gbase = nbr->grow_ptr + s0;
    a.nrows = s1 - s0;
    const dim3 grid(grid_for(a.nrows * kT, kBlock)), block(kBlock);
    ProfScope prof(ctx, m == 0 ? "weights_adjoint_3d" : "weights_adjoint_film");
    if (m == 0) hipLaunchKernelGGL(k_adjoint_x<10>, grid, block, 0, ctx->stream, a);
    else hipLaunchKernelGGL(k_adjoint_x<6>, grid, block, 0, ctx->stream, a);
    GF_LAUNCH_CHECK(ctx);
  }
  {
    ProfScope prof(ctx, "weights_adjoint_gather");
    hipLaunchKernelGGL(k_adjoint_gather, dim3(grid_for(p->n * kGT, kBlock)), dim3(kBlock), 0, ctx->stream,
                       nbr->grouped, nbr->grow_ptr, nbr->grev, a.dbar, p->n, xbar_3n);
    GF_LAUNCH_CHECK(ctx);
  }
  return GF_OK;
}
