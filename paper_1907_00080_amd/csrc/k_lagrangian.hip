// k_lagrangian.hip - Lagrangian side of the LB-IB step (gfx950), float64.
//
// Per time step n (the order is the one used throughout the library):
//   k_body_chunks first one workgroup per lattice instance:
//                   - bond kinetics: rupture pass, then formation pass in
//                     ascending ligand order (Sec. 2.2 Wall-Particle Interaction),
//                     with Philox4x32-10 uniforms keyed by (step, ligand).
//                 then one wave per vertex chunk of every body (a particle's
//                 chunk has a second one for the fluid at its vertices):
//                   - membrane strain, bending and area forces (Eqs. strainFor,
//                     bendFor, areaFor), adhesion springs (Eq. adhFor);
//                   - particles: probe pressure/viscous loads (Eqs. hydroForP,
//                     hydroForNu) from the pre-forcing fluid state, soft Verlet
//                     position update (Eqs. newtonSoft, verletPos) or rigid BDF2
//                     (Eqs. linearVelRig, angularVelRig), weak-coupling force.
//   (the fused lattice kernel runs here)
//   k_advance     two waves per chunk: red cells by the kinematic IB
//                 (Eq. kinematicPos), particles adopt their new positions;
//                 the stencil of the new position (centre node floor(X + 1/2)
//                 and the 3+3 weights of the Roma 3-point kernel) is stored
//                 and the marker joins the bins of every lattice tile that
//                 stencil overlaps, for the next step's fused kernel.
//
// No multiply-add contraction in this file: the same quantity is computed by
// several kernels and instantiations (a stencil by the advance and by the
// stencil pass, each transfer form), and all of them must round alike.  The
// fused operations are explicit (__fma_rn).
#pragma clang fp contract(off)
#include "lbib_dev.h"
#include "mls.h"

namespace lbib {

// ------------------------------------------------------------------ helpers
// Populations at a node after streaming, before forcing (walls: bounce-back),
// from a state of streaming scheme sch.
// The slots are those of streamed_slot, addressed as the fused kernel
// addresses them: the node's neighbour columns and row offsets once, then a
// uniform plane offset plus a 32-bit in-plane offset per direction (a plane
// holds at most 2^31 nodes).
template <typename T>
__device__ __forceinline__ void pull_node(const T* A, int sch, long long N, int nx, int ny, int pitch, bool pery,
                                 int x, int y, T hv[kQ]) {
  const unsigned o0 = (unsigned)y * (unsigned)pitch + (unsigned)x;
  if (sch == 2) {   // node-local layout: slot i of the node itself
#pragma unroll
    for (int i = 0; i < kQ; ++i) hv[i] = A[i * N + o0];
    return;
  }
  const bool lo = !pery && y == 0, hi = !pery && y == ny - 1;   // first / last row of a walled lattice
  const unsigned cm = x == 0 ? nx - 1 : x - 1, cp = x == nx - 1 ? 0 : x + 1;
  const unsigned rm = (unsigned)(y == 0 ? (pery ? ny - 1 : y) : y - 1) * (unsigned)pitch;
  const unsigned rp = (unsigned)(y == ny - 1 ? (pery ? 0 : y) : y + 1) * (unsigned)pitch;
  const unsigned r0 = (unsigned)y * (unsigned)pitch;
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    const unsigned c = ex(i) > 0 ? cm : (ex(i) < 0 ? cp : (unsigned)x);
    const unsigned r = ey(i) > 0 ? rm : (ey(i) < 0 ? rp : r0);
    // bounce-back: h*_opp(i) of the node itself
    const bool bounce = (ey(i) > 0 && lo) || (ey(i) < 0 && hi);
    const int pl = bounce ? (sch == 1 ? i : opp(i)) : (sch == 1 ? opp(i) : i);
    hv[i] = A[pl * N + (bounce ? o0 : r + c)];
  }
}

// Velocity walls: a wall node of the pre-forcing state takes the drive as its
// force (the step's IB forces are not known yet).
template <typename T>
__device__ __forceinline__ void wall_fill_drive(const LatDev& L, int y, T hv[kQ]) {
  const T lo = T(L.u_wall_lo), hi = T(L.u_wall_hi);   // values, not places, to choose from
  if (L.wall_mode == 1 && !L.periodic_y && (y == 0 || y == L.ny - 1))
    zou_he_fill(hv, y == 0, y == 0 ? lo : hi, T(L.gx), T(L.gy));
}

// rho* - 1 and u* = (sum f e + g/2) / rho* of a node of the pre-forcing
// state from its pulled moments, each rounded to the storage type T: the
// values the particles' LDS cache holds, so that a probe evaluated from the
// cache and one evaluated straight from the populations agree to the bit.
// The deviation rho* - 1 is what is stored, not rho* (in float32, rho*
// itself, about 1 + 1e-4, would keep only the leading digits of the
// deviation that the probe pressure cs^2 (rho* - 1) is made of).
template <typename T>
__device__ __forceinline__ void star_values(const LatDev& L, double drho, double jx, double jy, T& d,
                                            T& ux, T& uy) {
  const double r = 1.0 + drho;
  d = T(drho);
  ux = T((jx + 0.5 * L.gx) / r);
  uy = T((jy + 0.5 * L.gy) / r);
}

// MLS interpolant of rho*, u* at a point and (GRAD) its gradient (the MLS
// shape functions and their derivatives), from the node values fetch(a, b,
// x, row, rho, ux, uy) of stencil node (a, b) (x unwrapped; row unwrapped on
// a periodic lattice, else clamped: a row beyond a wall has weight zero, so
// it reads the wall row, inside the lattice and any cache of the point's
// nodes).
template <bool GRAD, typename Fetch>
__device__ __forceinline__ void interp_mls(const LatDev& L, double X, double Y, Fetch fetch,
                                           double& rho, double& ux, double& uy, double g[4]) {
  double ph[9], px[9], py[9];
  mls_shape<GRAD>(L, X, Y, ph, px, py);
  const double cxr = floor(X + 0.5), cyr = floor(Y + 0.5);
  rho = 0; ux = 0; uy = 0;
  g[0] = g[1] = g[2] = g[3] = 0;
  const bool pery = L.periodic_y != 0;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    int row = (int)(cyr + (b - 1));
    row = pery ? row : min(max(row, 0), L.ny - 1);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double r, u, v;
      fetch(a, b, (int)(cxr + (a - 1)), row, r, u, v);
      const double w = ph[3 * b + a];
      rho += r * w;
      ux += u * w;
      uy += v * w;
      if (GRAD) {
        g[0] += u * px[3 * b + a];
        g[1] += u * py[3 * b + a];
        g[2] += v * px[3 * b + a];
        g[3] += v * py[3 * b + a];
      }
    }
  }
}

// The star field (4 values per node: rho* - 1, u*x, u*y, unused) that the
// advance and stencil passes leave over every particle's node box, at the
// 3 x 3 nodes of a point: loaded first (nine 4-wide loads), summed by
// star_sum, so that a caller can have the loads of several points in flight
// together.  Rows beyond a wall read the wall row (weight zero).
template <typename T>
struct Star9 {
  T r[9], u[9], v[9];
};

template <typename T>
__device__ __forceinline__ void star_load(const T* S, const LatDev& L, double X, double Y, Star9<T>& n) {
  // one division for the centre column (X is unwrapped), then neighbours; node
  // numbers fit 32 bits (a plane holds at most 2^31 nodes)
  const int cx = wrap_i((int)floor(X + 0.5), L.nx), cy = (int)floor(Y + 0.5);
  const bool pery = L.periodic_y != 0;
  const int ry = pery ? wrap_i(cy, L.ny) : cy;
  unsigned col[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) col[a] = wrap_near(cx + a - 1, L.nx);
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const int row = pery ? wrap_near(ry + b - 1, L.ny) : min(max(ry + b - 1, 0), L.ny - 1);
    const unsigned r0 = (unsigned)row * (unsigned)L.pitch;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const T* q = S + 4ull * (r0 + col[a]);
      n.r[3 * b + a] = q[0];
      n.u[3 * b + a] = q[1];
      n.v[3 * b + a] = q[2];
    }
  }
}

// Kernel (or, with MLS compiled in and selected, MLS) interpolant of rho*, u*
// (and with GRAD its gradient) from the node values star_load gave.  MLS =
// false compiles the kernel weights only: the latency-bound kernels of runs
// without the MLS transfer carry none of its code.
template <bool MLS, bool GRAD, typename T>
__device__ __forceinline__ void star_sum(const LatDev& L, double X, double Y, const Star9<T>& n,
                                         double& rho, double& ux, double& uy, double g[4]) {
  constexpr bool grad = GRAD;
  const double cxr = floor(X + 0.5), cyr = floor(Y + 0.5);
  const bool pery = L.periodic_y != 0;
  if (MLS && use_mls(L)) {
    auto fetch = [&](int a, int b, int, int, double& r, double& u, double& v) {
      r = 1.0 + double(n.r[3 * b + a]);
      u = double(n.u[3 * b + a]);
      v = double(n.v[3 * b + a]);
    };
    interp_mls<GRAD>(L, X, Y, fetch, rho, ux, uy, g);
    return;
  }
  rho = 0; ux = 0; uy = 0;
  g[0] = g[1] = g[2] = g[3] = 0;
  double wxa[3], dwxa[3], wya[3], dwya[3];
  roma_weights3<true>(cxr - X, wxa, dwxa);
  roma_weights3<true>(cyr - Y, wya, dwya);
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const int ry = (int)(cyr + (b - 1));
    const bool ok = pery || (ry >= 0 && ry < L.ny);
    const double wy = ok ? wya[b] : 0.0;
    const double dwy = ok ? dwya[b] : 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double wx = wxa[a], dwx = dwxa[a];
      const double r = 1.0 + double(n.r[3 * b + a]), u = double(n.u[3 * b + a]), v = double(n.v[3 * b + a]);
      rho += r * wx * wy;
      ux += u * wx * wy;
      uy += v * wx * wy;
      if (grad) {
        g[0] -= u * dwx * wy;
        g[1] -= u * wx * dwy;
        g[2] -= v * dwx * wy;
        g[3] -= v * wx * dwy;
      }
    }
  }
}

__device__ __forceinline__ double wrap_x(double cx, int nx) { return cx - nx * floor(cx / nx); }

__device__ __forceinline__ double min_image(double xr, double cxw, int nx) {
  double d = xr - cxw;
  if (d > 0.5 * nx) d -= nx;
  else if (d < -0.5 * nx) d += nx;
  return d;
}

// Bond length between element centroid c and receptor (xr, wall).
__device__ __forceinline__ double bond_len(double cx, double cy, double xr, int wall, const LatDev& L) {
#pragma clang fp contract(off)
  const double dx = min_image(xr, wrap_x(cx, L.nx), L.nx);
  const double yw = wall == 0 ? L.y_wall_lo : L.y_wall_hi;
  const double dy = cy - yw;
  return sqrt(dx * dx + dy * dy);
}

// ---------------------------------------------------------------- marker bins
// Register a marker (one per lane, centre node cx, cy inside the lattice along
// periodic axes) in every tile its 3x3 stencil overlaps.  Three consecutive
// columns (rows) touch at most three tiles (a ragged last tile can be one
// column wide), so a marker joins at most nine bins; more than two columns or
// rows of tiles is rare.  A full bin drops the registration and counts it in
// *overflow (the fused kernel then poisons that tile's force so the watchdog
// reports it).  Slots come from wave-aggregated atomics: a run of adjacent
// lanes that hit the same tile (neighbours along a membrane) shares one; an
// atomic per lane queues at the counters (advance on 2000x200 9.6 us against
// 6.7).  In two halves: bins_reserve issues the reservations, bins_commit waits
// for them and stores the marker ids, so that a caller can do other work while
// they are in flight.
struct BinSlots {
  int key[9];           // tile of slot 3 * row + column, -1: none
  int leader[9], rank[9], base[9];
  unsigned used;        // slots some lane of the wave uses (wave-uniform)
};

// The distinct non-negative values of (a, b, c), in order, else -1.
__device__ __forceinline__ void distinct3(int a, int b, int c, int d[3]) {
  const bool nb = b >= 0 && b != a, nc = c >= 0 && c != a && c != b;
  const int x = a >= 0 ? a : (nb ? b : c);                       // the first
  const int y = a >= 0 ? (nb ? b : (nc ? c : -1)) : (nb && nc ? c : -1);
  d[0] = x;
  d[1] = y;
  d[2] = a >= 0 && nb && nc ? c : -1;
}

template <int TX, int TY>
__device__ __forceinline__ void bins_reserve(int* cnt, const LatDev& L, int cx, int cy, bool active,
                                             BinSlots& S) {
  const bool pery = L.periodic_y != 0;
  int tc[3], tr[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    tc[a] = active ? (int)((unsigned)wrap_near(cx + a - 1, L.nx) / TX) : -1;
    const int r = cy + a - 1, rw = pery ? wrap_near(r, L.ny) : r;
    tr[a] = rw >= 0 && rw < L.ny ? (int)((unsigned)rw / TY) : -1;
  }
  int dc[3], dr[3];
  distinct3(tc[0], tc[1], tc[2], dc);
  distinct3(tr[0], tr[1], tr[2], dr);
  const int lane = threadIdx.x & 63;
  const unsigned long long lt = (1ull << lane) - 1ull, le = lt | (1ull << lane);
  // 1. group the lanes of every slot by tile, no memory traffic
  int count[9];
  unsigned used = 0;
  const bool wide = __ballot(dc[2] >= 0 || dr[2] >= 0) != 0ull;
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const int i = q / 3, j = q % 3;
    S.key[q] = -1;
    S.leader[q] = lane;
    S.rank[q] = 0;
    count[q] = 0;
    if ((i == 2 || j == 2) && !wide) continue;
    const bool has = dr[i] >= 0 && dc[j] >= 0;
    const unsigned long long hasm = __ballot(has);
    if (hasm == 0ull) continue;
    used |= 1u << q;
    const int k = has ? L.tile_base + dr[i] * L.ntx + dc[j] : -1;
    S.key[q] = k;
    const int kprev = dpp_i<kDppWaveShr1>(k);   // lane 0: its own (not used)
    const unsigned long long heads = __ballot(has && (lane == 0 || kprev != k));
    const unsigned long long mine = heads & le;
    const int ld = mine ? 63 - __clzll((long long)mine) : lane;
    S.leader[q] = ld;
    S.rank[q] = lane - ld;
    const unsigned long long brk = (heads | ~hasm) & ~le;   // lanes after this one that end the run
    const int next = brk ? __ffsll((long long)brk) - 1 : 64;
    count[q] = has && lane == ld ? next - lane : 0;
  }
  // 2. every group leader reserves its slots, all in flight together
#pragma unroll
  for (int q = 0; q < 9; ++q)
    S.base[q] = (used >> q & 1u) && count[q] > 0 ? atomicAdd(&cnt[S.key[q]], count[q]) : 0;
  S.used = used;
}

// 3. positions first, then the stores (a store issued between two of the
// shuffles would be waited for by the next one)
__device__ __forceinline__ void bins_commit(int* bin, int cap, int* overflow, int gm, const BinSlots& S) {
  int pos[9], dropped = 0;
#pragma unroll
  for (int q = 0; q < 9; ++q) pos[q] = S.used >> q & 1u ? __shfl(S.base[q], S.leader[q]) + S.rank[q] : 0;
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    if (!(S.used >> q & 1u) || S.key[q] < 0) continue;
    if (pos[q] < cap) bin[(long long)S.key[q] * cap + pos[q]] = gm;
    else ++dropped;
  }
  if (dropped) atomicAdd(overflow, dropped);
}

// ---------------------------------------------------------------- stencils
// Stencil of a marker at (X, Y): centre node floor(X + 1/2) (column wrapped,
// row wrapped on a periodic lattice, else kept raw so rows beyond the walls
// can be recognised) and the weights of its 3x3 nodes: the Roma kernel
// along each axis (zero for rows beyond the walls), or the MLS shape
// functions.
// Stencil centre node of a marker at (X, Y), as marker_stencil stores it.
__device__ __forceinline__ void stencil_centre(const LatDev& L, double X, double Y, int& ocx, int& ocy) {
  const bool pery = L.periodic_y != 0;
  const double cxr = floor(X + 0.5), cyr = floor(Y + 0.5);
  ocx = wrap_i((int)cxr, L.nx);
  ocy = pery ? wrap_i((int)cyr, L.ny) : (int)fmin(fmax(cyr, -4.0), (double)(L.ny + 3));
}

template <bool MLS = true, typename T>
__device__ __forceinline__ void marker_stencil(const Ptrs<T>& p, const LatDev& L, int gm, double X, double Y,
                                      int& ocx, int& ocy) {
  const int nm = p.nm_total;
  const bool pery = L.periodic_y != 0;
  const double cxr = floor(X + 0.5), cyr = floor(Y + 0.5);
  if (MLS && use_mls(L)) {
    double ph[9];
    mls_shape<false>(L, X, Y, ph, nullptr, nullptr);
#pragma unroll
    for (int k = 0; k < 9; ++k) p.wx[k * nm + gm] = ph[k];
  } else {
    double w3x[3], w3y[3], d3[3];
    roma_weights3<false>(cxr - X, w3x, d3);
    roma_weights3<false>(cyr - Y, w3y, d3);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      p.wx[a * nm + gm] = w3x[a];
      const double ry = cyr + (a - 1);
      const bool valid = pery || (ry >= 0.0 && ry < (double)L.ny);
      p.wy[a * nm + gm] = valid ? w3y[a] : 0.0;
    }
  }
  ocx = wrap_i((int)cxr, L.nx);
  ocy = pery ? wrap_i((int)cyr, L.ny) : (int)fmin(fmax(cyr, -4.0), (double)(L.ny + 3));
  p.cx[gm] = ocx;
  p.cy[gm] = ocy;
}

// ---------------------------------------------------------------- advance
// Kinematic IB update of a red-cell vertex (Eq. kinematicPos): the velocity
// of the step, interpolated at X^n with the stencil stored for X^n, then
// BDF2 (forward Euler on the first step).
// Split in two so that a lane handling several vertices issues every load
// of all of them before it waits: first the stencil and X^{n-1} (needed by
// BDF2 only, loaded unconditionally), then the velocity gather.
// MLS = false: the Roma kernel's per-axis weights (the layout the kernels
// without MLS keep: a wider one costs them register spills); MLS = true: nine
// slots, the Roma weights in 0..5 (wx then wy) or the nine MLS weights.
template <bool MLS> struct RbcAdv;
template <> struct RbcAdv<false> {
  int cx, cy;
  double wx[3], wy[3];
  double xm, ym;
};
template <> struct RbcAdv<true> {
  int cx, cy;
  double ph[9];
  double xm, ym;
};

template <bool MLS, typename T>
__device__ __forceinline__ void rbc_adv_load(const Ptrs<T>& p, const LatDev& L, int gm, RbcAdv<MLS>& a) {
  const int nm = p.nm_total;
  a.cx = p.cx[gm];
  a.cy = p.cy[gm];
  if constexpr (MLS) {
    // one load per slot from the array the transfer uses (fixed slots, no
    // branch around the writes, so the struct stays in registers)
    const bool mls = use_mls(L);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const double* src = (mls || k < 3) ? p.wx + k * nm : p.wy + (k - 3) * nm;
      a.ph[k] = src[gm];
    }
#pragma unroll
    for (int k = 6; k < 9; ++k) a.ph[k] = mls ? p.wx[k * nm + gm] : 0.0;
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      a.wx[k] = p.wx[k * nm + gm];
      a.wy[k] = p.wy[k * nm + gm];
    }
  }
  a.xm = p.xm[gm];
  a.ym = p.ym[gm];
}

template <bool MLS, typename T>
__device__ __forceinline__ void rbc_adv_finish(const Ptrs<T>& p, const LatDev& L, const RbcAdv<MLS>& in, double X,
                                      double Y, bool first, double& xn, double& yn) {
  const T* U = p.U + 2 * L.node_base;
  const T* V = U + L.plane;
  const int cx = in.cx, cy = in.cy;   // inside the lattice along periodic axes
  double ux = 0.0, uy = 0.0;
  // a row beyond a wall has weight exactly zero: it reads a clamped row and
  // adds zeros, so the loads are independent of control flow.  Away from the
  // seam a row's three nodes are consecutive: one wide load each.
  const bool seam = __ballot(cx < 1 || cx + 1 >= L.nx) != 0ull;
  T u[9], v[9];
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    int row = cy + b - 1;
    if (L.periodic_y) row = wrap_near(row, L.ny);
    else row = min(max(row, 0), L.ny - 1);
    const unsigned r0 = (unsigned)row * (unsigned)L.pitch;
    if (seam) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const unsigned node = r0 + (unsigned)wrap_near(cx + a - 1, L.nx);
        u[3 * b + a] = U[node];
        v[3 * b + a] = V[node];
      }
    } else {
      const T *ur = U + (r0 + cx - 1u), *vr = V + (r0 + cx - 1u);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        u[3 * b + a] = ur[a];
        v[3 * b + a] = vr[a];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    double w;
    if constexpr (MLS) w = use_mls(L) ? in.ph[k] : in.ph[k % 3] * in.ph[3 + k / 3];
    else w = in.wx[k % 3] * in.wy[k / 3];
    ux += double(u[k]) * w;
    uy += double(v[k]) * w;
  }
  if (first) {
    xn = X + ux;
    yn = Y + uy;
  } else {
    xn = (2.0 / 3.0) * (2.0 * X - 0.5 * in.xm + ux);
    yn = (2.0 / 3.0) * (2.0 * Y - 0.5 * in.ym + uy);
  }
}

template <bool MLS, typename T>
__device__ __forceinline__ void advance_rbc(const Ptrs<T>& p, const LatDev& L, int gm, double X, double Y,
                                   bool first, double& xn, double& yn) {
  RbcAdv<MLS> a;
  rbc_adv_load<MLS>(p, L, gm, a);
  rbc_adv_finish<MLS>(p, L, a, X, Y, first, xn, yn);
}

// ---------------------------------------------------------------- k_bonds
// First of the strictly increasing xs[0, n) (in [0, nx)) not left of x.  The
// place that even spacing gives is tried first: one trip to memory instead of
// one per halving.
__device__ __forceinline__ int first_not_left(const double* xs, int n, double x, int nx) {
  const int g = min(max((int)(x * n / nx), 0), n - 1);
  const double before = xs[max(g - 1, 0)], at = xs[g], after = xs[min(g + 1, n - 1)];
  if (at >= x && (g == 0 || before < x)) return g;
  if (at < x && (g + 1 == n || after >= x)) return g + 1;
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (xs[mid] < x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

constexpr int kBodyThreads = 64 * kBodyWaves;
// the wave's number in its workgroup, in a scalar register
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

constexpr int kLigRanks = 2;   // ligands per lane and pass of the bond kinetics

// What the bond workgroup holds in LDS: the eligible ligands per wave and
// rank (two sets, used by alternate passes), and the first 64 eligible ones.
struct BondLds {
  int cnt[2][kLigRanks][kBodyWaves];
  int code[64];                  // ligand << 1 | wall
  double cx[64], cy[64], sig[64];
};

// The step waits for this chain (the particles near a wall need its bonds), so
// it is kept short: all loads of a pass in flight together, one barrier per
// pass, and the first 64 eligible ligands handed to the formation through LDS.
// (Six boxes with a particle at the wall: the flag goes up after 4.2 us, 5.9
// with three barriers per pass and the ligands read back from memory; the
// kernel takes 9.3 us, 11.2 before.)
template <typename T>
__device__ __forceinline__ void bonds_kinetics(const Ptrs<T>& p, const LatDev& L, int inst, long long n,
                                               int nx, int ny, BondLds& S) {
  constexpr int R = kLigRanks, nt = kBodyThreads, nw = kBodyWaves;
  const int tid = threadIdx.x;
  // bond kinetics (Sec. 2.2): rupture then formation (a frozen topology
  // skips both); then every bond's spring coefficient sigma (y_l - y_eq)
  // at X^n for the particles' spring forces (Eq. adhFor)
  if (L.n_lig == 0) return;
  const bool kinetics = !L.freeze;
  const double y_cr = L.y_cr;
  unsigned long long ties = 0;
  // (a) rupture (independent per bond) and formation eligibility; R
  // ligands per lane and pass (l0 + r nt + tid), their loads in flight
  // together
  const int lane = tid & 63, w = wave_id();
  const unsigned long long lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  int ne = 0;        // eligible ligands of the passes so far
  bool odd = false;
  for (int l0 = 0; l0 < L.n_lig; l0 += R * nt, odd = !odd) {
    int gl[R], va[R], vb[R], rr[R], flag[R];
    double sigma[R], x0[R], x1[R], y0[R], y1[R], xr[R];
    // ranks that hold a ligand (the same for every lane)
    auto held = [&](int r) { return l0 + r * nt < L.n_lig; };
    auto on = [&](int r) { return l0 + r * nt + tid < L.n_lig; };
#pragma unroll
    for (int r = 0; r < R; ++r) {
      flag[r] = 0;
      if (!held(r)) continue;
      gl[r] = L.lig_base + (on(r) ? l0 + r * nt + tid : 0);
      va[r] = p.lig_va[gl[r]];
      vb[r] = p.lig_vb[gl[r]];
      rr[r] = p.l2r[gl[r]];
      sigma[r] = p.lig_sigma[gl[r]];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (!held(r)) continue;
      // particle positions X^n: xn (equal to x once a step has ended)
      x0[r] = p.xn[va[r]];
      x1[r] = p.xn[vb[r]];
      y0[r] = p.yn[va[r]];
      y1[r] = p.yn[vb[r]];
      xr[r] = p.rec_x[rr[r] >= 0 ? L.rec_base + rr[r] : 0];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (!on(r)) continue;
      const int l = l0 + r * nt + tid;
      x0[r] = 0.5 * (x0[r] + x1[r]);   // the element's centroid
      y0[r] = 0.5 * (y0[r] + y1[r]);
      const double cx = x0[r], cy = y0[r];
      const int rc = rr[r];
      if (rc >= 0) {
        const int wall = rc < L.n_rec0 ? 0 : 1;
        const double yl = bond_len(cx, cy, xr[r], wall, L);
        const double sig = sigma[r], sts = L.sigma_ts_frac * sig;
        const double dy = yl - L.y_eq;
        bool broken = false;
        if (kinetics) {
          const double kr = L.kr0_dt * exp((sig - sts) * dy * dy / (2.0 * L.kbt));
          const double P = 1.0 - exp(-kr);
          const double u = philox_uniform(L.seed, n, l, 1, L.instance);
          ties += fabs(u - P) < 1e-12;
          broken = u < P;
        }
        if (broken) {
          // atomic: body waves read the table while this runs
          __hip_atomic_store(&p.l2r[gl[r]], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          p.r2l[L.rec_base + rc] = -1;
        } else {
          p.lig_sp[gl[r]] = sig * dy;
        }
      } else if (kinetics) {
        const double d0 = cy - L.y_wall_lo, d1 = L.y_wall_hi - cy;
        const int wall = d0 <= d1 ? 0 : 1;
        const double d = wall == 0 ? d0 : d1;
        if (d < y_cr) flag[r] = 1 + wall;
      }
    }
    if (!kinetics) continue;
    // ordered compaction of the eligible ligands (ascending ligand id):
    // per-wave counts by ballot, then every lane's place from the counts of
    // the earlier ligand ranges and waves.  The next pass writes the other
    // set of counts: a set is written again only after the barrier that
    // follows its last reading.
    int(*cnt)[kBodyWaves] = S.cnt[odd];
    unsigned long long bal[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      bal[r] = __ballot(flag[r] != 0);
      if (lane == 0) cnt[r][w] = __popcll(bal[r]);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      int before = 0, tot = 0;
#pragma unroll
      for (int k = 0; k < nw; ++k) {
        const int c = cnt[r][k];
        before += k < w ? c : 0;
        tot += c;
      }
      if (flag[r]) {
        const int pos = ne + before + __popcll(bal[r] & lt);
        const int code = ((l0 + r * nt + tid) << 1) | (flag[r] - 1);
        if (pos < 64) {
          S.code[pos] = code;
          S.cx[pos] = x0[r];
          S.cy[pos] = y0[r];
          S.sig[pos] = sigma[r];
        } else {
          p.lig_flag[L.lig_base + pos] = code;
        }
      }
      ne += tot;
    }
  }
  // (b) formation, in ascending ligand order.  A ligand's choice (the nearest
  // free receptor of its wall) and draw depend on the earlier ones only
  // through the receptors they take, so the lanes of one wave choose and draw
  // for 64 eligible ligands together; then the bonds form in order, and only a
  // ligand whose receptor has just gone chooses again.  (One lane taking the
  // ligands one after the other cost about 3 us each.)
  if (ne == 0) {
    if (ties) atomicAdd(&p.ties[inst], ties);
    return;
  }
  __syncthreads();   // the eligible ligands, and the receptors that rupture freed
  if (tid < 64) {
    for (int q0 = 0; q0 < ne; q0 += 64) {
      const bool on = q0 + lane < ne;
      int code = 0;
      double cx = 0.0, cy = 0.0, sig = 0.0;
      if (q0 == 0) {
        if (on) {
          code = S.code[lane];
          cx = S.cx[lane];
          cy = S.cy[lane];
          sig = S.sig[lane];
        }
      } else {
        code = on ? p.lig_flag[L.lig_base + q0 + lane] : 0;
        const int g = L.lig_base + (code >> 1);
        const int va = p.lig_va[g], vb = p.lig_vb[g];
        cx = 0.5 * (p.xn[va] + p.xn[vb]);
        cy = 0.5 * (p.yn[va] + p.yn[vb]);
        sig = p.lig_sigma[g];
      }
      const int l = code >> 1, wall = code & 1;
      const int gl = L.lig_base + l;
      const int nr = wall == 0 ? L.n_rec0 : L.n_rec1;
      const int roff = wall == 0 ? 0 : L.n_rec0;
      const double* xs = p.rec_x + L.rec_base + roff;
      const int* taken = p.r2l + L.rec_base + roff;
      const double cxw = wrap_x(cx, nx);
      const bool can = on && nr > 0;
      const double sts = L.sigma_ts_frac * sig;
      const int lo = can ? first_not_left(xs, nr, cxw, nx) : 0;
      const double u = philox_uniform(L.seed, n, l, 0, L.instance);
      int best = -1;
      double dy = 0.0;
      bool forms = false, tie = false;
      auto choose = [&] {
        // merge the rightward and leftward sequences by their own distances;
        // each receptor is met first at its minimum-image distance
        int ir = lo == nr ? 0 : lo, il = lo == 0 ? nr - 1 : lo - 1;
        best = -1;
        double xb = 0.0;
        for (int it = 0; it < 2 * nr && best < 0; ++it) {
          const double xr = xs[ir], xl = xs[il];
          const int tr = taken[ir], tl = taken[il];
          double dr = xr - cxw;
          if (dr < 0) dr += nx;
          double dl = cxw - xl;
          if (dl < 0) dl += nx;
          // oracle's minimum image: equal to the smaller of the two one-sided
          // distances; ties between the two sides go to the lower index
          const bool take_r = dr < dl || (dr == dl && ir <= il);
          xb = take_r ? xr : xl;
          if ((take_r ? tr : tl) < 0) best = take_r ? ir : il;
          else if (take_r) ir = ir + 1 == nr ? 0 : ir + 1;
          else il = il == 0 ? nr - 1 : il - 1;
        }
        forms = tie = false;
        if (best < 0) return;
        const double yl = bond_len(cx, cy, xb, wall, L);
        dy = yl - L.y_eq;
        const double kf = L.kf0_dt * exp(-sts * dy * dy / (2.0 * L.kbt));
        const double P = 1.0 - exp(-kf);
        tie = fabs(u - P) < 1e-12;
        forms = u < P;
      };
      if (can) choose();
      unsigned long long todo = __ballot(forms);
      while (todo) {
        const int q = __ffsll((long long)todo) - 1;
        const int rec = roff + best;
        const int gone = __shfl(rec, q);
        if (lane == q) {
          __hip_atomic_store(&p.l2r[gl], rec, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          p.r2l[L.rec_base + rec] = gl;
          p.lig_sp[gl] = sig * dy;
        }
        __threadfence_block();   // the receptor is taken for the lanes that choose again
        if (lane > q && best >= 0 && rec == gone) choose();
        todo = __ballot(lane > q && forms);
      }
      ties += tie;
    }
  }
  if (ties) atomicAdd(&p.ties[inst], ties);
}

// Step bookkeeping and bond kinetics of one lattice instance (the first
// workgroups of the body kernel).  Raises the instance's flag that particle
// workgroups wait for before they read the bond table.
template <typename T>
__device__ __forceinline__ void bonds_impl(const Ptrs<T>& p, int inst, BondLds& S) {
  const LatDev L = load_uniform(p.lat + inst);
  const long long n = load_uniform(p.step_next + inst);
  const int tid = threadIdx.x;
  bonds_kinetics(p, L, inst, n, L.nx, L.ny, S);
  // publish: the barrier orders every lane's writes before thread 0's
  // release store of the flag (one write-back of the cache, not one per lane)
  __syncthreads();
  if (tid == 0) {
    p.step_cur[inst] = n;
    p.step_next[inst] = n + 1;
    __hip_atomic_store(&p.bond_flag[inst], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (inst == 0) {
    // the other slot was last used by the previous step, whose kernels have
    // all finished: clear it for the next step
    for (int i = tid; i < p.ninst; i += kBodyThreads) {
      p.fmax_next[i] = 0ull;
      p.bond_flag_next[i] = 0;
    }
  }
}

// ---------------------------------------------------------------- star field
// Node box of a set of positions: floor of the smallest and ceiling of the
// largest x and y (wave-wide; lanes with on = false do not count).
struct IBox {
  int x0, x1, y0, y1;
};
__device__ __forceinline__ IBox wave_box(double x, double y, bool on) {
  const auto mn = [](int a, int b) { return min(a, b); };
  const auto mx = [](int a, int b) { return max(a, b); };
  return IBox{wave_reduce_i(on ? (int)floor(x) : 0x7fffffff, mn), wave_reduce_i(on ? (int)ceil(x) : -0x7fffffff, mx),
              wave_reduce_i(on ? (int)floor(y) : 0x7fffffff, mn), wave_reduce_i(on ? (int)ceil(y) : -0x7fffffff, mx)};
}

__device__ __forceinline__ void put_box(int* pbox, int chunk, const IBox& q) {
  pbox[4 * chunk] = q.x0;
  pbox[4 * chunk + 1] = q.x1;
  pbox[4 * chunk + 2] = q.y0;
  pbox[4 * chunk + 3] = q.y1;
}

// rho* - 1 and u* (star_values) of the pre-forcing state at every node of
// one particle's box: the box of its vertices (the union of its chunk
// boxes) widened by 4 nodes (probe 1.2 along the normal, stencil reach 1.5,
// a node of margin), rows clamped to the lattice unless it is periodic.
// Entry w of the star work list names the particle, this workgroup's rank
// and the particle's workgroup count; src holds the populations the next
// step streams from, in streaming scheme sch.  Nodes of overlapping boxes
// are written twice with the same values.
// The kernels below copy their instance's lattice record into registers
// before their first store: read through a reference, its fields are
// reloaded (and waited for) after every store, which may alias them.
template <typename T>
__device__ __forceinline__ void star_pass(const Ptrs<T>& p, const T* src, int sch, int w) {
  const int b = p.star_wg[3 * w], rank = p.star_wg[3 * w + 1], K = p.star_wg[3 * w + 2];
  const BodyDev B = load_uniform(p.body + b);
  const LatDev L = load_uniform(p.lat + B.inst);
  const int nch = chunks_of(B.nv);
  int x0 = 0x7fffffff, x1 = -0x7fffffff, y0 = 0x7fffffff, y1 = -0x7fffffff;
  for (int k0 = 0; k0 < nch; k0 += 4) {   // four chunk boxes in flight together
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int4 q = load_uniform((const int4*)p.pbox + B.chunk0 + min(k0 + k, nch - 1));
      x0 = min(x0, q.x);
      x1 = max(x1, q.y);
      y0 = min(y0, q.z);
      y1 = max(y1, q.w);
    }
  }
  x0 -= 4; x1 += 4; y0 -= 4; y1 += 4;
  const bool pery = L.periodic_y != 0;
  if (!pery) {
    y0 = max(y0, 0);
    y1 = min(y1, L.ny - 1);
  }
  const int bw = x1 - x0 + 1, bh = y1 - y0 + 1;
  if (bw <= 0 || bh <= 0) return;
  const int nbox = bw * bh;
  const T* A = src + 9 * L.node_base;
  T* S = p.star + 4 * L.node_base;
  // one node per lane and pass (four before): the wave's chain of instructions
  // bounds this pass, and the chip has room for the workgroups
  for (int k = rank * kStarNodes + threadIdx.x; k < nbox; k += K * kStarNodes) {
    const unsigned dr = (unsigned)k / (unsigned)bw, dc = (unsigned)k - dr * (unsigned)bw;
    const int col = wrap_i(x0 + (int)dc, L.nx);
    int row = y0 + (int)dr;
    if (pery) row = wrap_i(row, L.ny);
    T hv[kQ];
    pull_node(A, sch, L.plane, L.nx, L.ny, L.pitch, pery, col, row, hv);
    wall_fill_drive(L, row, hv);
    double drho = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      const double h = double(hv[i]);
      drho += h;
      jx += ex(i) * h;
      jy += ey(i) * h;
    }
    T* o = S + 4ull * ((unsigned)row * (unsigned)L.pitch + (unsigned)col);
    star_values(L, drho, jx, jy, o[0], o[1], o[2]);
  }
}

// ---------------------------------------------------------------- body kernel
constexpr int kSpinMax = 1 << 22;   // bounded wait for the bond flag (~0.2 s)

// max that propagates NaN (fmax drops it)
__device__ __forceinline__ double fmax_nan(double a, double b) { return (a > b || a != a) ? a : b; }

// Particles read the bond table (and rigid ones the step counter) that this
// instance's bond workgroup writes during the same launch: each wave waits
// for its flag (bounded spin; the bond workgroups have the lowest ids, so
// they are always dispatched).  The polls are relaxed and one acquire fence
// follows them: an acquire load invalidates the cache on every poll.
template <typename T>
__device__ __forceinline__ void wait_bonds(const Ptrs<T>& p, int inst) {
  if ((threadIdx.x & 63) == 0) {
    int it = 0;
    while (__hip_atomic_load(&p.bond_flag[inst], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0 &&
           it < kSpinMax) {
      __builtin_amdgcn_s_sleep(2);
      ++it;
    }
    if (it == kSpinMax) atomicAdd(p.spin_timeouts, 1);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// ---- membrane and particle arithmetic

// Element from (x0, y0) to (x1, y1): length and unit tangent.  The outward
// normal of the counter-clockwise contour is (ty, -tx).
__device__ __forceinline__ void edge_of(double x0, double y0, double x1, double y1, double& len,
                                        double& tx, double& ty) {
  const double dx = x1 - x0, dy = y1 - y0;
  len = sqrt(dx * dx + dy * dy);
  tx = dx / len;
  ty = dy / len;
}

// Vertex normal normalize(n_L + n_R) from the unit tangents of the left and
// right elements (reading R14).
__device__ __forceinline__ void vertex_normal(double txl, double tyl, double txr, double tyr,
                                              double& bnx, double& bny) {
  const double nsx = tyl + tyr, nsy = -txl - txr;
  const double nn = sqrt(nsx * nsx + nsy * nsy);
  bnx = nsx / nn;
  bny = nsy / nn;
}

// k_b (theta - theta_0), theta the signed turning angle from the left to the
// right tangent (Eq. bendFor, reading R13).
__device__ __forceinline__ double bend_coeff(double txl, double tyl, double txr, double tyr, double kb,
                                             double th0) {
  const double cr = txl * tyr - tyl * txr;
  const double dt = txl * txr + tyl * tyr;
  return kb * (atan2(cr, dt) - th0);
}

// Probe point 1.2 dx along the outward normal from the element centroid,
// kept inside the fluid (Sec. 2.2 Hydrodynamics Stresses; reading R24).
__device__ __forceinline__ void probe_point(const LatDev& L, double cx, double cy, double nxl,
                                            double nyl, double& qx, double& qy) {
  qx = cx + 1.2 * nxl;
  qy = cy + 1.2 * nyl;
  if (!L.periodic_y) qy = fmin(fmax(qy, 0.5), L.ny - 1.5);
}

// Pressure and viscous load of an element (Eqs. hydroForP, hydroForNu) from
// the probe's rho* and velocity gradient g = (du/dx, du/dy, dv/dx, dv/dy).
__device__ __forceinline__ void probe_load(double rho, const double g[4], double nu, double nxl,
                                           double nyl, double len, double& fx, double& fy) {
  const double pr = (rho - 1.0) * (1.0 / 3.0);
  const double txx = 2.0 * nu * g[0], tyy = 2.0 * nu * g[3], txy = nu * (g[1] + g[2]);
  fx = (-pr * nxl + txx * nxl + txy * nyl) * len;
  fy = (-pr * nyl + txy * nxl + tyy * nyl) * len;
}

// Load of one element: area penalty (Eq. areaFor, coefficient ca), adhesion
// spring (Eq. adhFor, sp = sigma (y_l - y_eq)) along the outward normal, and
// the probe load, summed in this order.
__device__ __forceinline__ void element_load(bool area_on, double ca, bool spring_on, double sp,
                                             bool probe_on, double pfx, double pfy, double nxl,
                                             double nyl, double& fex, double& fey) {
  fex = 0.0;
  fey = 0.0;
  if (area_on) {
    fex += ca * nxl;
    fey += ca * nyl;
  }
  if (spring_on) {
    fex += sp * nxl;
    fey += sp * nyl;
  }
  if (probe_on) {
    fex += pfx;
    fey += pfy;
  }
}

// What the force on vertex v needs from its neighbourhood: elements v-2 ..
// v+1 and vertices v-1 .. v+1.
struct VertexNbr {
  double len_mm, len_m, len, len_p;          // lengths of elements v-2, v-1, v, v+1
  double nx_m, ny_m, nx, ny;                 // outward normals of elements v-1, v
  double bc_m, bc, bc_p;                     // k_b (theta - theta_0) at v-1, v, v+1
  double bnx_m, bny_m, bnx, bny, bnx_p, bny_p;   // vertex normals at v-1, v, v+1
  double fex_m, fey_m, fex, fey;             // loads of elements v-1, v
};

// Force on vertex v: strain of its two elements (Eq. strainFor), bending at
// v-1, v and v+1 (Eq. bendFor with the lever-rule weights of reading R13b: a
// neighbour's share is the length of the edge on the far side of the bent
// vertex over the two lengths, so the three forces exert no net moment),
// half of each adjacent element's load, then the repulsion magnitude sv
// (Eq. repFor) along the inward vertex normal.
__device__ __forceinline__ void membrane_force(const VertexNbr& q, double ks, double l0v, double l0m,
                                               bool bend, bool rep, double sv, double& fx, double& fy) {
  const double sr = ks * (q.len - l0v);
  const double sl = ks * (q.len_m - l0m);
  // tangents from normals: t = (-n_y, n_x)
  fx = sr * (-q.ny) - sl * (-q.ny_m);
  fy = sr * q.nx - sl * q.nx_m;
  if (bend) {
    const double fr = q.len_mm / (q.len_mm + q.len_m);
    fx += q.bc_m * fr * q.bnx_m;
    fy += q.bc_m * fr * q.bny_m;
    fx -= q.bc * q.bnx;
    fy -= q.bc * q.bny;
    const double fl = q.len_p / (q.len + q.len_p);
    fx += q.bc_p * fl * q.bnx_p;
    fy += q.bc_p * fl * q.bny_p;
  }
  fx += 0.5 * q.fex + 0.5 * q.fex_m;
  fy += 0.5 * q.fey + 0.5 * q.fey_m;
  if (rep) {
    fx -= sv * q.bnx;
    fy -= sv * q.bny;
  }
}

// Soft-particle vertex (Eqs. newtonSoft, verletPos): new position from the
// fluid velocity u* at the vertex and half the force over the vertex mass.
// The weak coupling drives the fluid towards the vertex displacement of the
// step (readings R26, R26': the second-order velocity of Eq. verletVel turns
// the coupling into a feedback that grows next to walls), spread with the
// weight ds.
__device__ __forceinline__ void soft_vertex(double X, double Y, double ux, double uy, double fx,
                                            double fy, double mv, double ds, double& xn, double& yn,
                                            double& ffx, double& ffy) {
  xn = X + ux + 0.5 * fx / mv;
  yn = Y + uy + 0.5 * fy / mv;
  const double Ux = xn - X, Uy = yn - Y;
  ffx = (2.0 * (Ux - ux)) * ds;
  ffy = (2.0 * (Uy - uy)) * ds;
}

// One vertex's terms of a rigid particle's sums: the load of element l at
// its centroid (cx, cy) relative to the reference point, and the repulsion
// (frx, fry) at the vertex (lever lx, ly).
__device__ __forceinline__ void rigid_terms(double fex, double fey, double cx, double cy, bool rep,
                                            double frx, double fry, double lx, double ly,
                                            double t[3]) {
  t[0] = fex;
  t[1] = fey;
  t[2] = cx * fey - cy * fex;
  if (rep) {
    t[0] += frx;
    t[1] += fry;
    t[2] += lx * fry - ly * frx;
  }
}

// Rigid particle (Eqs. linearVelRig, angularVelRig; readings R28, R29): BDF2
// for U and Omega from the summed force and torque (forward Euler on the
// first step), then the reference point and the angle move by them.
// st = (U_x, U_y, Omega, x_c, y_c, theta) after the step.
__device__ __forceinline__ void rigid_step(const BodyDev* Bp, bool first, const double r3[3],
                                           double st[6]) {
  double U[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const double a = r3[k] / Bp->mass;
    U[k] = first ? Bp->U[k] + a : (2.0 / 3.0) * (2.0 * Bp->U[k] - 0.5 * Bp->Um[k] + a);
  }
  const double al = r3[2] / Bp->inertia;
  const double Om = first ? Bp->Om + al : (2.0 / 3.0) * (2.0 * Bp->Om - 0.5 * Bp->Omm + al);
  st[0] = U[0];
  st[1] = U[1];
  st[2] = Om;
  st[3] = Bp->xc + U[0];
  st[4] = Bp->yc + U[1];
  st[5] = Bp->theta + Om;
}

__device__ __forceinline__ void rigid_commit(BodyDev* Bp, const double st[6]) {
  Bp->stepped = 1;
  Bp->Um[0] = Bp->U[0];
  Bp->Um[1] = Bp->U[1];
  Bp->U[0] = st[0];
  Bp->U[1] = st[1];
  Bp->Omm = Bp->Om;
  Bp->Om = st[2];
  Bp->xc = st[3];
  Bp->yc = st[4];
  Bp->theta = st[5];
}

// Rigid-particle vertex: its position from the reference shape (rx, ry)
// rotated by theta (cos cs, sin sn), and the weak-coupling force towards the
// rigid-body velocity U + Omega x r there (reading R26).
__device__ __forceinline__ void rigid_vertex(double rx, double ry, const double st[6], double cs,
                                             double sn, double ux, double uy, double ds, double& xn,
                                             double& yn, double& fx, double& fy) {
  xn = st[3] + (rx * cs + ry * (-sn));
  yn = st[4] + (rx * sn + ry * cs);
  const double relx = xn - st[3], rely = yn - st[4];
  const double ukx = st[0] + st[2] * (-rely), uky = st[1] + st[2] * relx;
  fx = (2.0 * (ukx - ux)) * ds;
  fy = (2.0 * (uky - uy)) * ds;
}

// ---------------------------------------------------------------- chunked body kernel
// One wave per vertex chunk (lane i holds vertex first + i - 2 of the body;
// the chunk's own vertices are lanes 2 .. 2 + cnt - 1).  Neighbour data come
// from the neighbouring lanes, the body's area from the chunk records of
// X^n that the advance (or stencil) pass left, so a red cell's or a soft
// particle's chunk needs nothing from any other wave.  A rigid particle's
// force and torque need all its chunks: up to kGroupChunks of them meet in the
// LDS of their workgroup; in a larger body each chunk stores its partial sums
// and the fluid velocity at its vertices, and the chunk that arrives last
// (a counter per body) takes the rigid step and moves every vertex.
//
// Bound by the chain of instructions of one wave (a lone wave issues one every
// 4 to 10 cycles).  A particle's chunk needs the fluid at two points per vertex,
// the probe of its element and the vertex itself: a second wave takes the
// vertices and hands u* over in LDS, while the first takes the probes.  (Body
// kernel of a 1237x149 run with moving least squares 8.7 us, 11.5 with one wave
// for both; of a 2000x200 capillary 6.9, 7.2; of 96 lattices with 1150 particle
// chunks 14.2, 16.3.)
struct BodyLds {
  double rp[3][kGroupChunks];       // a rigid body's sums, per chunk
  double uv[2][kGroupChunks][64];   // u* at the vertices of each chunk's lanes
  unsigned long long fmax;          // largest |F| of the waves that have ended, as bits
  int ended;
};

// Largest |F| a wave hands to the fluid (m: each lane's), folded into its
// instance's maximum (non-negative doubles order like their bit patterns; NaN
// and Inf sort above every finite value, so a broken force shows up as a
// non-finite maximum).  Atomics on one instance's maximum are taken one after
// the other, so where a workgroup holds n > 0 red-cell chunks of one instance its
// last wave sends one for all (body kernel of 16 lattices with 990 chunks 8.5 us,
// 10.5 with one per chunk; 6667x667 with 372 chunks 8.3, 9.5).  No wave waits for
// another, as it would at a barrier: ended waves make room (96 lattices with 12
// particles and 16 red-cell chunks each: 14.2 us, 17.5 with a barrier).
__device__ __forceinline__ void record_fmax(unsigned long long* slot, double m, int n, BodyLds& S) {
  m = wave_reduce_d(m, [](double a, double b) { return fmax_nan(a, b); });
  if ((threadIdx.x & 63) != 0) return;
  unsigned long long f = (unsigned long long)__double_as_longlong(m);
  if (n > 0) {
    __hip_atomic_fetch_max(&S.fmax, f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (__hip_atomic_fetch_add(&S.ended, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) != n - 1) return;
    f = __hip_atomic_load(&S.fmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  if (f != 0) atomicMax(slot, f);
}

// u* at the vertices of a chunk, for wave w of the workgroup.
template <typename T, bool MLS>
__device__ __forceinline__ void sample_vertices(const Ptrs<T>& p, const ChunkSlot& sl, int w, BodyLds& S) {
  const int lane = threadIdx.x & 63;
  const int gm = sl.v0 + chunk_vertex(lane, sl.first, sl.nv);
  const double X = p.x[gm], Y = p.y[gm];
  const LatDev L = load_uniform(p.lat + (sl.kind_inst >> 2));
  Star9<T> n;
  star_load(p.star + 4 * L.node_base, L, X, Y, n);
  double rho, ux, uy, g[4];
  star_sum<MLS, false>(L, X, Y, n, rho, ux, uy, g);
  S.uv[0][w][lane] = ux;
  S.uv[1][w][lane] = uy;
}

template <typename T, bool MLS>
__device__ __forceinline__ double chunk_impl(const Ptrs<T>& p, const ChunkSlot& sl, BodyLds& lds) {
  const int lane = threadIdx.x & 63;
  // the slot alone gives the wave its vertices; the body record (in registers,
  // read before any store: the rigid step writes it back through Bp) is in
  // flight with them
  const int chunk = sl.chunk, b = sl.body;
  const int kind = sl.kind_inst & 3, inst = sl.kind_inst >> 2, nv = sl.nv, v0 = sl.v0, ch0 = sl.chunk0;
  BodyDev* Bp = p.body + b;
  const BodyDev B = *Bp;
  const int nch = chunks_of(nv);
  const int first_v = sl.first, cnt = min(kChunk, nv - first_v);
  const int v = chunk_vertex(lane, first_v, nv), gm = v0 + v;
  const bool inner = lane >= 2 && lane < 2 + cnt;     // the chunk's own vertices
  const bool has_elem = lane >= 1 && lane < 2 + cnt;  // elements v -> v+1 they touch
  const LatDev L = load_uniform(p.lat + inst);
  const T* S = p.star + 4 * L.node_base;   // rho*, u* over the particles' boxes
  const bool rigid = kind == kRigid, particle = kind != kRBC;
  const bool rep = L.rep_coeff > 0.0;
  const double X = p.x[gm], Y = p.y[gm];
  // a rigid vertex's reference offset, for its move after the rigid step
  const double r0xv = rigid && inner ? p.r0x[gm] : 0.0, r0yv = rigid && inner ? p.r0y[gm] : 0.0;
  const double l0v = rigid ? 0.0 : p.l0[gm];
  const double th0v = rigid ? 0.0 : p.th0[gm];
  const double sv = rep && inner ? p.frep[gm] : 0.0;
  // the ligand of element v and its bond table entry as this wave finds it:
  // the bond workgroup rewrites the table while the wave runs (see below)
  const int ls = particle ? B.lig_stride : 0;
  int vq = 0, vr = 1;   // v / ls and its remainder (usually every or every other element)
  if (ls > 0) {
    vq = (ls & (ls - 1)) == 0 ? v >> __builtin_ctz(ls) : v / ls;
    vr = v - vq * ls;
  }
  const bool lig = has_elem && vr == 0;
  const int gl = lig ? B.lig_base + vq : 0;
  const int r_seen = lig ? __hip_atomic_load(&p.l2r[gl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : -1;
  const double area_t = rigid ? 0.0 : area_term(p.area_part, p.nchunk_total, ch0, nch, lane);

  // element v -> v+1 and the bending at v
  const double Xp = lane_next(X), Yp = lane_next(Y);
  double len, tx, ty;
  edge_of(X, Y, Xp, Yp, len, tx, ty);
  const double enx = ty, eny = -tx;
  const double txl = lane_prev(tx), tyl = lane_prev(ty);
  double bnx = 0.0, bny = 0.0, bc = 0.0;
  const bool bend = !rigid && B.kb != 0.0;   // the capillary's red cells have none
  if (bend || rep) vertex_normal(txl, tyl, tx, ty, bnx, bny);
  if (bend) bc = bend_coeff(txl, tyl, tx, ty, B.kb, th0v);

  // particles: probe load of the element, from the star field of the
  // particle's box
  const double cx = 0.5 * (X + Xp), cy = 0.5 * (Y + Yp);
  double pfx = 0.0, pfy = 0.0, uvx = 0.0, uvy = 0.0;
  const bool grouped = rigid_grouped(kind, nv);
  if (particle) {
    const double nu = (L.tau - 0.5) / 3.0;
    // lanes without an element probe at the vertex: always a point of the box
    double qx = X, qy = Y;
    if (has_elem) probe_point(L, cx, cy, enx, eny, qx, qy);
    Star9<T> nq;
    star_load(S, L, qx, qy, nq);
    double rho, ux, uy, g[4];
    star_sum<MLS, true>(L, qx, qy, nq, rho, ux, uy, g);
    if (has_elem) probe_load(rho, g, nu, enx, eny, len, pfx, pfy);
  }
  // u* at the vertices, from the sampling wave; a grouped rigid body takes it
  // over at the barrier of its sums
  auto take_samples = [&] {
    if (inner) {
      uvx = lds.uv[0][wave_id()][lane];
      uvy = lds.uv[1][wave_id()][lane];
    }
  };
  if (particle && !grouped) {
    __syncthreads();
    take_samples();
  }
  // adhesion springs on bonded ligand elements (after this step's bond
  // update).  A ligand element whose centroid lies farther than y_cr from
  // both wall lines cannot form a bond in this step, and a bond broken in
  // this step is not re-formed in it: if the entry the wave read is free,
  // whether it was the entry before the update or after it, the element
  // holds no bond after the update.  A chunk whose ligands are all such
  // needs nothing from the bond workgroup and does not wait for it.
  bool spring_on = false;
  double sp = 0.0;
  if (particle) {
    const double dw = fmin(cy - L.y_wall_lo, L.y_wall_hi - cy);
    const bool maybe = lig && (r_seen >= 0 || dw < L.y_cr + 0.25);
    if (__ballot(maybe) != 0ull) {
      wait_bonds(p, inst);
      if (lig) {
        const int r = p.l2r[gl];
        sp = p.lig_sp[gl];   // sigma (y_l - y_eq), from the bond workgroup
        spring_on = r >= 0;
      }
    }
  }
  const bool first = rigid && B.stepped == 0;
  double ca = 0.0;
  if (!rigid) {
    const double area = body_area2(p.area_part, p.nchunk_total, ch0, nch, area_t) * 0.5;
    ca = B.ka * (1.0 - area / B.A0) * B.p_ref * len;
  }
  double fex, fey;
  element_load(!rigid, ca, spring_on, sp, particle, pfx, pfy, enx, eny, fex, fey);
  const double len_m = lane_prev(len);
  const double ds = 0.5 * (len_m + len);   // spreading weight of the vertex

  double fm = 0.0;
  if (rigid) {
    const double xc0 = B.xc, yc0 = B.yc;
    double t3[3] = {0.0, 0.0, 0.0};
    if (inner) {
      rigid_terms(fex, fey, cx - xc0, cy - yc0, rep, -sv * bnx, -sv * bny, X - xc0, Y - yc0, t3);
      if (rep) p.frep[gm] = 0.0;   // applied: the next step's repulsion kernel rewrites it
    }
    double s3[3] = {t3[0], t3[1], t3[2]};
    wave_sum3(s3);
    double st[6], xn = 0.0, yn = 0.0, fx, fy;
    if (grouped) {
      // the body's chunks are on neighbouring waves of this workgroup, the
      // first on wave w0
      const int w0 = wave_id() - (chunk - ch0);
      if (lane < 3) lds.rp[lane][wave_id()] = lane == 0 ? s3[0] : (lane == 1 ? s3[1] : s3[2]);
      __syncthreads();
      double r3[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {   // in chunk order, as chunk_total
        double q[kGroupChunks], s = 0.0;
#pragma unroll
        for (int c = 0; c < kGroupChunks; ++c) q[c] = lds.rp[k][min(w0 + c, kGroupChunks - 1)];
#pragma unroll
        for (int c = 0; c < kGroupChunks; ++c) s = c < nch ? s + q[c] : s;
        r3[k] = s;
      }
      take_samples();
      rigid_step(&B, first, r3, st);
      __syncthreads();   // every wave has read the rigid state
      if (lane == 0 && chunk == ch0) rigid_commit(Bp, st);
      double sn, cs;
      sincos(st[5], &sn, &cs);
      if (inner) {
        rigid_vertex(r0xv, r0yv, st, cs, sn, uvx, uvy, ds, xn, yn, fx, fy);
        p.xn[gm] = xn;
        p.yn[gm] = yn;
        p.fx[gm] = fx;
        p.fy[gm] = fy;
        fm = fmax_nan(fabs(fx), fabs(fy));
      }
      const IBox q = wave_box(xn, yn, inner);
      if (lane == 0) put_box(p.pbox, chunk, q);
    } else {
      // a larger rigid body: its chunks' partial sums meet in memory, and
      // the chunk that arrives last takes the rigid step for all vertices
      const int nct = p.nchunk_total;
      if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) p.rig_part[k * nct + chunk] = s3[k];
      }
      if (inner) {
        p.s_fex[gm] = uvx;
        p.s_fey[gm] = uvy;
        p.s_len[gm] = ds;
      }
      __threadfence();
      int done = 0;
      if (lane == 0)
        done = __hip_atomic_fetch_add(&p.body_cnt[b], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
      done = __builtin_amdgcn_readfirstlane(done);   // lane 0's count
      if (done != nch - 1) return 0.0;   // a later chunk finishes the body
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      if (lane == 0) p.body_cnt[b] = 0;
      double r3[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) r3[k] = chunk_total(p.rig_part + k * nct + ch0, nch);
      rigid_step(&B, first, r3, st);
      if (lane == 0) rigid_commit(Bp, st);
      double sn, cs;
      sincos(st[5], &sn, &cs);
      IBox q{0x7fffffff, -0x7fffffff, 0x7fffffff, -0x7fffffff};
      // four vertices per lane and pass, their loads issued before any store
      for (int w0 = 0; w0 < nv; w0 += 4 * 64) {
        double rx[4], ry[4], ux[4], uy[4], dv[4];
        int g2[4];
        bool on[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int w = w0 + j * 64 + lane;
          on[j] = w < nv;
          g2[j] = v0 + (on[j] ? w : 0);
          rx[j] = p.r0x[g2[j]];
          ry[j] = p.r0y[g2[j]];
          ux[j] = p.s_fex[g2[j]];
          uy[j] = p.s_fey[g2[j]];
          dv[j] = p.s_len[g2[j]];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (!on[j]) continue;
          rigid_vertex(rx[j], ry[j], st, cs, sn, ux[j], uy[j], dv[j], xn, yn, fx, fy);
          p.xn[g2[j]] = xn;
          p.yn[g2[j]] = yn;
          p.fx[g2[j]] = fx;
          p.fy[g2[j]] = fy;
          fm = fmax_nan(fm, fmax_nan(fabs(fx), fabs(fy)));
          q.x0 = min(q.x0, (int)floor(xn)); q.x1 = max(q.x1, (int)ceil(xn));
          q.y0 = min(q.y0, (int)floor(yn)); q.y1 = max(q.y1, (int)ceil(yn));
        }
      }
      const auto mn = [](int a, int b) { return min(a, b); };
      const auto mx = [](int a, int b) { return max(a, b); };
      q = IBox{wave_reduce_i(q.x0, mn), wave_reduce_i(q.x1, mx), wave_reduce_i(q.y0, mn),
               wave_reduce_i(q.y1, mx)};
      for (int k = lane; k < nch; k += 64) put_box(p.pbox, ch0 + k, q);
    }
    return fm;
  }

  // red cells and soft particles: vertex forces
  VertexNbr q;
  // (two lanes back: lane 1 gets lane 0's value, which only the halo uses)
  q.len_mm = lane_prev(len_m);
  q.len_m = len_m;
  q.len = len;
  q.len_p = lane_next(len);
  q.nx_m = lane_prev(enx);
  q.ny_m = lane_prev(eny);
  q.nx = enx;
  q.ny = eny;
  q.bc_m = lane_prev(bc);
  q.bc = bc;
  q.bc_p = lane_next(bc);
  q.bnx_m = lane_prev(bnx);
  q.bny_m = lane_prev(bny);
  q.bnx = bnx;
  q.bny = bny;
  q.bnx_p = lane_next(bnx);
  q.bny_p = lane_next(bny);
  q.fex_m = lane_prev(fex);
  q.fey_m = lane_prev(fey);
  q.fex = fex;
  q.fey = fey;
  const double l0m = lane_prev(l0v);
  double sxn = 0.0, syn = 0.0, ffx, ffy;   // a soft particle's new position
  if (inner) {
    double fx, fy;
    membrane_force(q, B.ks, l0v, l0m, bend, rep, sv, fx, fy);
    if (rep) p.frep[gm] = 0.0;   // applied: the next step's repulsion kernel rewrites it
    if (kind == kRBC) {
      p.fx[gm] = fx;
      p.fy[gm] = fy;
      fm = fmax_nan(fabs(fx), fabs(fy));
    } else {
      soft_vertex(X, Y, uvx, uvy, fx, fy, B.mv, ds, sxn, syn, ffx, ffy);
      p.xn[gm] = sxn;
      p.yn[gm] = syn;
      p.fx[gm] = ffx;
      p.fy[gm] = ffy;
      fm = fmax_nan(fabs(ffx), fabs(ffy));
    }
  }
  if (kind == kSoft) {
    const IBox q = wave_box(sxn, syn, inner);
    if (lane == 0) put_box(p.pbox, chunk, q);
  }
  return fm;
}

// The other bin set (last read two steps ago) starts its next use empty.
// Called after a wave's own work: no load of it then waits behind these stores.
template <typename T>
__device__ __forceinline__ void clear_bins(const Ptrs<T>& p) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < p.ntile_total; t += gridDim.x * blockDim.x)
    p.cnt_next[t] = 0;
}

// Workgroups [0, ninst) run the bond kinetics of each instance; then the waves
// of the slot list.
template <typename T, bool MLS>
__global__ __launch_bounds__(kBodyThreads) void k_body_chunks(Ptrs<T>) {
  const Ptrs<T>& p = launch_args<T>();
  __shared__ union {
    BondLds bond;
    BodyLds body;
  } lds;
  if ((int)blockIdx.x < p.ninst) {
    bonds_impl(p, blockIdx.x, lds.bond);
    clear_bins(p);
    return;
  }
  const int slot = (blockIdx.x - p.ninst) * kBodyWaves + wave_id();
  if (slot < p.nslot) {   // nslot holds whole workgroups
    const ChunkSlot sl = load_uniform(p.slot_chunk + slot);
    const int barriers = sl.role & 3, w = ((sl.role >> 2) & 15) - 1, n = sl.role >> 8;
    if (n > 0) {
      if (threadIdx.x == 0) {
        lds.body.fmax = 0ull;
        lds.body.ended = 0;
      }
      __syncthreads();
    }
    if (sl.chunk == -1 || w >= 0) {
      // no chunk of its own: the barriers of the waves that have one
      if (w >= 0) sample_vertices<T, MLS>(p, sl, w, lds.body);
      for (int k = 0; k < barriers; ++k) __syncthreads();
    } else {
      const double fm = chunk_impl<T, MLS>(p, sl, lds.body);
      record_fmax(p.fmax_bits + (sl.kind_inst >> 2), fm, n, lds.body);
    }
  }
  clear_bins(p);
}

// ---------------------------------------------------------------- advance and stencil passes
constexpr int kAdvWaves = 4;   // waves per workgroup
// chunks per workgroup: an advancing chunk has two waves
template <bool ADVANCE>
__host__ __device__ constexpr int adv_chunks() { return ADVANCE ? kAdvWaves / 2 : kAdvWaves; }
// Bound by the chain of one wave: its records, its vertices, the velocities
// the lattice kernel left on other XCDs, then about 600 instructions at the
// 4 to 10 cycles each that a wave alone on its SIMD issues at.  Measured (us,
// before -> after the compacted bin slots, row loads of the velocity and one
// star node per lane): 2000x200 7.6 -> 6.7, 6667x667 9.2 -> 7.6, 16-lattice
// sweep 9.7 -> 9.1.  When advancing, a chunk has two waves: the first moves the
// vertices and registers them in the bins, the second takes the new positions
// from LDS and does the stencils and the area record meanwhile: 2000x200 7.3 ->
// 6.3, 6667x667 7.7 -> 7.0, sweep 9.2 -> 8.9, 1237x149 with moving least squares
// 8.1 -> 6.1, 48 lattices of 14 cells 26.9 -> 26.3.
// A chunk's own vertices are on lanes 2 .. 2 + cnt - 1 (the halo lanes idle:
// their vertices belong to waves that move them in place).
// ADVANCE: every vertex moves to X^{n+1} (red cells by the kinematic update,
// particles adopt the positions of their dynamics); otherwise X stays (the
// stencil pass after set-up or after the positions were set).  Each vertex
// stores its stencil and joins the bins (cnt, bin) of the next fused
// kernel.  The chunk's area record of the new positions (its interior-edge
// shoelace sum, its first and last vertex) is what the next body kernel
// adds up into the body's area.
template <typename T, int TX, int TY, bool MLS, bool ADVANCE>
__device__ __forceinline__ void advance_chunk(const Ptrs<T>& p, int* cnt, int* bin) {
  constexpr int kChunks = adv_chunks<ADVANCE>();
  __shared__ double s_xy[kChunks][2][64];   // new positions, from a chunk's first wave to its second
  const int lane = threadIdx.x & 63;
  const int w = wave_id() % kChunks;
  const bool second = wave_id() >= kChunks;
  const int chunk = blockIdx.x * kChunks + w;
  const bool held = chunk < p.nchunk_total;   // the same for the whole wave
  // one load gives the wave its vertices (the body record is not needed)
  const int4 ci = load_uniform(p.chunk_info + (held ? chunk : 0));
  const int kind = ci.w & 3, inst = ci.w >> 2, cnt_v = ci.z;
  const bool inner = held && lane >= 2 && lane < 2 + cnt_v;
  const int gm = inner ? ci.y + lane : 0;
  const LatDev L = load_uniform(p.lat + inst);
  double X = 0.0, Y = 0.0, xn = 0.0, yn = 0.0;
  int ncx = 0, ncy = 0;
  if (inner && !second) {
    X = p.x[gm];
    Y = p.y[gm];
    xn = X;
    yn = Y;
    if (ADVANCE) {
      if (kind == kRBC) {
        advance_rbc<MLS>(p, L, gm, X, Y, p.step_cur[inst] == 0, xn, yn);
      } else {
        xn = p.xn[gm];
        yn = p.yn[gm];
      }
    }
    stencil_centre(L, xn, yn, ncx, ncy);
  }
  if constexpr (ADVANCE) {
    if (!second) {
      s_xy[w][0][lane] = xn;
      s_xy[w][1][lane] = yn;
    }
    __syncthreads();
    if (second) {
      xn = s_xy[w][0][lane];
      yn = s_xy[w][1][lane];
    }
  }
  if (!held) return;
  // bin slots for the new stencil: the reservations (atomics) go out first
  // and the stores below are issued while they are in flight
  BinSlots S;
  if (!second) {
    bins_reserve<TX, TY>(cnt, L, ncx, ncy, inner, S);
    if (ADVANCE && inner) {
      p.xm[gm] = X;
      p.ym[gm] = Y;
      p.x[gm] = xn;
      p.y[gm] = yn;
    }
  }
  if (!ADVANCE || second) {
    // stencil of the new position, used by the next step's spreading and
    // interpolation (the first wave has finished reading the old one: the
    // position it handed over depends on all of it)
    if (inner) marker_stencil<MLS>(p, L, gm, xn, yn, ncx, ncy);
    const double xr = lane_next(xn), yr = lane_next(yn);
    const double part = wave_sum(lane >= 2 && lane < 1 + cnt_v ? shoelace_term(xn, yn, xr, yr) : 0.0);
    const int nct = p.nchunk_total;
    if (lane == 0) p.area_part[chunk] = part;
    if (lane == 2) {
      p.area_part[nct + chunk] = xn;
      p.area_part[2 * nct + chunk] = yn;
    }
    if (lane == 1 + cnt_v) {
      p.area_part[3 * nct + chunk] = xn;
      p.area_part[4 * nct + chunk] = yn;
    }
    if (!ADVANCE && kind != kRBC) {
      // the stencil pass boxes the particles for the star pass that follows
      // it (when advancing, the body kernel has boxed their new positions)
      const IBox q = wave_box(xn, yn, inner);
      if (lane == 0) put_box(p.pbox, chunk, q);
    }
  }
  if (!second) bins_commit(bin, p.bin_cap, p.overflow, gm, S);
}

template <bool ADVANCE>
inline __host__ __device__ int chunk_blocks(int nchunk) {
  return (nchunk + adv_chunks<ADVANCE>() - 1) / adv_chunks<ADVANCE>();
}

// Marker advance, new stencils, bins and area records (kernel weights only,
// or with the MLS transfer compiled in, launched when an instance uses it);
// the workgroups after the chunks' fill the star field of the particles'
// boxes from the populations this step's fused kernel wrote.
template <typename T, int TX, int TY>
__global__ __launch_bounds__(256) void k_advance(Ptrs<T>) {
  const Ptrs<T>& p = launch_args<T>();
  const int cb = chunk_blocks<true>(p.nchunk_total);
  if ((int)blockIdx.x >= cb) {
    star_pass(p, p.B, p.sch_next, blockIdx.x - cb);
    return;
  }
  advance_chunk<T, TX, TY, false, true>(p, p.cnt_next, p.bin_next);
}

template <typename T, int TX, int TY>
__global__ __launch_bounds__(256) void k_advance_mls(Ptrs<T>) {
  const Ptrs<T>& p = launch_args<T>();
  const int cb = chunk_blocks<true>(p.nchunk_total);
  if ((int)blockIdx.x >= cb) {
    star_pass(p, p.B, p.sch_next, blockIdx.x - cb);
    return;
  }
  advance_chunk<T, TX, TY, true, true>(p, p.cnt_next, p.bin_next);
}

// Star field of the particles' boxes from the current populations (after
// the stencil pass).
template <typename T>
__global__ __launch_bounds__(256) void k_star(Ptrs<T>) {
  const Ptrs<T>& p = launch_args<T>();
  star_pass(p, p.A, p.sch, blockIdx.x);
}

// Stencils, bins and area partials of all markers from their current
// positions (after set-up or after positions were overwritten from the host).
template <typename T, int TX, int TY>
__global__ __launch_bounds__(256) void k_stencil(Ptrs<T>) {
  const Ptrs<T>& p = launch_args<T>();
  advance_chunk<T, TX, TY, true, false>(p, p.cnt_cur, p.bin_cur);
}

// ------------------------------------------------------------------ launchers
#define LBIB_TILE_DISPATCH(a, KERNEL, ...)                                                   \
  do {                                                                                     \
    if ((a).tile_x == 64 && (a).tile_y == 4) hipLaunchKernelGGL((KERNEL<T, 64, 4>), __VA_ARGS__);          \
    else if ((a).tile_x == 128 && (a).tile_y == 2) hipLaunchKernelGGL((KERNEL<T, 128, 2>), __VA_ARGS__);   \
    else if ((a).tile_x == 32 && (a).tile_y == 8) hipLaunchKernelGGL((KERNEL<T, 32, 8>), __VA_ARGS__);     \
    else hipLaunchKernelGGL((KERNEL<T, 256, 1>), __VA_ARGS__);                             \
  } while (0)

template <typename T>
void launch_stencil(const Ptrs<T>& p, const StepArgs& a, hipStream_t s) {
  if (p.nchunk_total == 0) return;
  LBIB_TILE_DISPATCH(a, k_stencil, dim3(chunk_blocks<false>(p.nchunk_total)), dim3(256), 0, s, p);
  if (p.nstar_wg > 0) hipLaunchKernelGGL((k_star<T>), dim3(p.nstar_wg), dim3(256), 0, s, p);
}

template <typename T>
void launch_lagrangian(const Ptrs<T>& p, const StepArgs& a, hipStream_t s) {
  const dim3 grid(p.ninst + (unsigned)(p.nslot / kBodyWaves)), block(kBodyThreads);
  if (a.any_mls) hipLaunchKernelGGL((k_body_chunks<T, true>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((k_body_chunks<T, false>), grid, block, 0, s, p);
}

template <typename T>
void launch_advance(const Ptrs<T>& p, const StepArgs& a, hipStream_t s) {
  if (p.nchunk_total == 0) return;
  const dim3 grid((unsigned)(chunk_blocks<true>(p.nchunk_total) + p.nstar_wg)), block(64 * kAdvWaves);
  if (a.any_mls) LBIB_TILE_DISPATCH(a, k_advance_mls, grid, block, 0, s, p);
  else LBIB_TILE_DISPATCH(a, k_advance, grid, block, 0, s, p);
}
#undef LBIB_TILE_DISPATCH

template void launch_lagrangian<float>(const Ptrs<float>&, const StepArgs&, hipStream_t);
template void launch_lagrangian<double>(const Ptrs<double>&, const StepArgs&, hipStream_t);
template void launch_advance<float>(const Ptrs<float>&, const StepArgs&, hipStream_t);
template void launch_advance<double>(const Ptrs<double>&, const StepArgs&, hipStream_t);
template void launch_stencil<float>(const Ptrs<float>&, const StepArgs&, hipStream_t);
template void launch_stencil<double>(const Ptrs<double>&, const StepArgs&, hipStream_t);

}  // namespace lbib
