// k_repulsion.hip - repulsion between vertices of different bodies (gfx950),
// Sec. 2.2 "Particle-Particle Interaction", Eq. (repFor).
//
// A vertex at distance d < r_c from a vertex of another body is pushed along
// its own inward normal with magnitude c sqrt(1 / d^5) (lattice units); the
// magnitudes of all such neighbours add.  This kernel computes the summed
// magnitude S_v of every vertex at X^n; the body kernel applies -S_v n_v with
// the vertex normal it computes anyway (red cells and soft particles add it to
// the vertex force, rigid particles to their force and torque) and clears S_v
// after use.
//
// One workgroup per chunk of kRepChunk consecutive vertices of a body (the
// host lists the chunks), so that a large body is spread over many
// workgroups and each looks at a small neighbourhood.  The marker bins of the
// step (every marker is registered in the tiles its 3x3 stencil overlaps)
// serve as the cell list:
//   1. the chunk's bounding box gives the tile columns and rows that can hold
//      the stencil centre of a vertex within r_c of it;
//   2. the bins of those tiles are read with all loads of a round in flight
//      together; a marker is taken from the bin of the tile that holds its
//      stencil centre only (so once), if it belongs to another body and lies
//      within r_c of the box;
//   3. the accepted candidates are ranked in LDS by (x, marker id), a total
//      order independent of the order the bins were filled in, so every sum
//      below is taken in a fixed order (deterministic results);
//   4. each vertex binary-searches the x window [x - r_c, x + r_c]; 16 lanes
//      evaluate its candidates and add the terms in rank order.
// Bound by its chain of dependent steps (record, vertices, bin counts, bin
// entries, candidates), so nothing in it is left to one lane: every wave finds
// the box and the tiles in its own registers, the offsets of the bins are
// running scalar sums, candidates are placed by one LDS counter, and a vertex's
// terms (a root, a quotient and the image quotients each) are taken side by
// side.  1555x187 with 14 cells and 9 particles: 7.6 us, 9.5 with the tiles
// listed by one lane, block-wide scans and the terms one after the other.
// Distances use the minimum image along x, and along y on a periodic lattice.
// Candidate lists that exceed their fixed capacity are truncated and counted
// in *overflow, which the host reports.
#include "lbib_dev.h"

namespace lbib {

constexpr int kRepThreads = 256;
constexpr int kRepCand = 512;      // candidate vertices of other bodies per chunk
constexpr int kRepTiles = 256;     // neighbour tiles per chunk
constexpr int kRepAxis = 64;       // tile columns / rows per chunk
constexpr int kRepPerLane = 4;     // bin entries per lane and round
static_assert(kRepThreads == 16 * kRepChunk, "16 lanes per vertex");

// Minimum image of d; a distance well inside half the lattice is its own image
// (the quotient then rounds to 0).
__device__ __forceinline__ double min_image_n(double d, int n) {
  return fabs(d) < 0.49 * n ? d : d - n * rint(d / n);
}
// i modulo n, without the division where i lies within a lattice of [0, n).
__device__ __forceinline__ int wrap_near_or(int i, int n) {
  return i >= -n && i < 2 * n ? wrap_near(i, n) : wrap_i(i, n);
}

// Tiles along one axis whose nodes meet [n0, n1] (unwrapped node indices):
// first, first + 1, ... (after the axis' last tile its first again), count of
// them; wrapped on a periodic axis, clamped to [0, n) otherwise.
struct TileRange {
  int first, count, all;
  __device__ __forceinline__ int at(int k) const { return first + k < all ? first + k : first + k - all; }
};
__device__ __forceinline__ TileRange axis_tiles(int n0, int n1, int n, int tw, bool periodic) {
  TileRange r;
  r.all = (n + tw - 1) / tw;
  if (!periodic) {
    const int lo = max(n0, 0), hi = min(n1, n - 1);
    r.first = lo / tw;
    r.count = lo <= hi ? hi / tw - r.first + 1 : 0;
  } else if (n1 - n0 + 1 >= n) {
    r.first = 0;
    r.count = r.all;
  } else {
    const int w0 = wrap_i(n0, n), w1 = wrap_i(n1, n);
    r.first = w0 / tw;
    // across the seam: on to the last tile, then from the first (the tile it
    // began in may be met again)
    r.count = w0 <= w1 ? w1 / tw - r.first + 1 : min(r.all - r.first + w1 / tw + 1, r.all);
  }
  return r;
}

template <typename T, int TX, int TY>
__global__ __launch_bounds__(kRepThreads) void k_repulsion(Ptrs<T>, const int4* chunks) {
  const Ptrs<T>& p = launch_args<T>();
  __shared__ int s_n;                                 // candidates accepted
  __shared__ double s_x[kRepCand], s_y[kRepCand];     // candidates as accepted
  __shared__ int s_id[kRepCand];
  __shared__ double s_sx[kRepCand], s_sy[kRepCand];   // ranked by (x, id)

  // chunk record: body, first global vertex, vertex count, lattice instance
  const int4 ck = load_uniform(chunks + blockIdx.x);
  const int b = ck.x, gv0 = ck.y, nvc = ck.z;
  const LatDev L = load_uniform(p.lat + ck.w);
  const int t = threadIdx.x, lane = t & 63;
  if (!(L.rep_coeff > 0.0)) return;   // the body kernel then reads the cleared zeros
  if (t == 0) s_n = 0;
  const double coeff = L.rep_coeff, rc = L.rep_cutoff;
  const int nx = L.nx, ny = L.ny, ntx = L.ntx;
  const bool pery = L.periodic_y != 0;

  // ---- 1. the chunk's box, in every 16-lane row of every wave; vertex v of
  // the chunk belongs to lanes 16 v .. 16 v + 15 of the workgroup
  const int v = t >> 4;
  const int ga = gv0 + min(lane & 15, nvc - 1), gv = gv0 + min(v, nvc - 1);
  const double xa = p.x[ga], ya = p.y[ga], xv = p.x[gv], yv = p.y[gv];
  double box[4] = {xa, -xa, ya, -ya};   // the smallest of each
#pragma unroll
  for (int k = 0; k < 4; ++k) box[k] = fmin(box[k], dpp_d<kDppRowRor8>(box[k]));
#pragma unroll
  for (int k = 0; k < 4; ++k) box[k] = fmin(box[k], dpp_d<kDppRowRor4>(box[k]));
#pragma unroll
  for (int k = 0; k < 4; ++k) box[k] = fmin(box[k], dpp_d<kDppRowRor2>(box[k]));
#pragma unroll
  for (int k = 0; k < 4; ++k) box[k] = fmin(box[k], dpp_d<kDppRowRor1>(box[k]));
  const double bx0 = box[0], bx1 = -box[1], by0 = box[2], by1 = -box[3];
  const double xm = 0.5 * (bx0 + bx1), hw = 0.5 * (bx1 - bx0);
  const double ym = 0.5 * (by0 + by1), hh = 0.5 * (by1 - by0);

  // ---- 2. tiles that can hold the stencil centre (the nearest node) of
  // a vertex within rc of the box: one node of margin beyond rc
  const auto uniform = [](double x) { return __builtin_amdgcn_readfirstlane((int)x); };
  const TileRange cols = axis_tiles(uniform(floor(bx0 - rc)) - 1, uniform(ceil(bx1 + rc)) + 1, nx, TX, true);
  const TileRange rows = axis_tiles(uniform(floor(by0 - rc)) - 1, uniform(ceil(by1 + rc)) + 1, ny, TY, pery);
  const int ncol = min(cols.count, kRepAxis);
  int nrow = min(rows.count, kRepAxis);
  if (cols.count > kRepAxis || rows.count > kRepAxis || ncol * nrow > kRepTiles) {
    if (t == 0) atomicAdd(p.overflow, 1);
    nrow = min(nrow, kRepTiles / max(ncol, 1));
  }
  const int ntl = ncol * nrow;
  __syncthreads();   // the count of candidates is cleared

  const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  for (int tb = 0; tb < ntl; tb += 64) {   // 64 tiles, one per lane of every wave
    const int nt = min(ntl - tb, 64);
    int tile = 0, cnt = 0;
    if (lane < nt) {
      const int r = (tb + lane) / ncol;
      tile = L.tile_base + rows.at(r) * ntx + cols.at(tb + lane - r * ncol);
      cnt = min(p.cnt_cur[tile], p.bin_cap);
    }
    int E = cnt;   // entries of these tiles
    E = wave_reduce_i(E, [](int a, int c) { return a + c; });
    // kRepPerLane entries per lane per round, loads issued together
    for (int e0 = 0; e0 < E; e0 += kRepPerLane * kRepThreads) {
      int m2[kRepPerLane], tl[kRepPerLane], at[kRepPerLane], bd2[kRepPerLane];
      double x2[kRepPerLane], y2[kRepPerLane];
      auto held = [&](int q) { return e0 + q * kRepThreads < E; };   // the same for every lane
      for (int i = 0, off = 0; i < nt; ++i) {   // the last tile that starts at or before the entry
        const int tt = __builtin_amdgcn_readlane(tile, i);
#pragma unroll
        for (int q = 0; q < kRepPerLane; ++q) {
          if (!held(q)) continue;
          const int e = e0 + q * kRepThreads + t;
          if (i == 0 || e >= off) {
            tl[q] = tt;
            at[q] = e - off;
          }
        }
        off += __builtin_amdgcn_readlane(cnt, i);
      }
#pragma unroll
      for (int q = 0; q < kRepPerLane; ++q) {
        m2[q] = -1;
        if (held(q) && e0 + q * kRepThreads + t < E) m2[q] = p.bin_cur[(long long)tl[q] * p.bin_cap + at[q]];
      }
#pragma unroll
      for (int q = 0; q < kRepPerLane; ++q) {
        if (!held(q)) continue;
        const int m = m2[q] >= 0 ? m2[q] : 0;
        bd2[q] = p.mbody[m];
        x2[q] = p.x[m];
        y2[q] = p.y[m];
      }
#pragma unroll
      for (int q = 0; q < kRepPerLane; ++q) {
        if (!held(q)) continue;
        // home tile: the one holding the marker's stencil centre, the nearest
        // node (as the stencil takes it), a centre beyond a wall in the edge row
        const int cx2 = wrap_near_or((int)floor(x2[q] + 0.5), nx);
        const double fy = floor(y2[q] + 0.5);
        const int cy2 = pery ? wrap_near_or((int)fy, ny) : (int)fmin(fmax(fy, 0.0), (double)(ny - 1));
        const int home = L.tile_base + (cy2 / TY) * ntx + cx2 / TX;
        bool keep = m2[q] >= 0 && home == tl[q] && bd2[q] != b;
        const double dx = min_image_n(x2[q] - xm, nx);
        const double dyr = y2[q] - ym;
        keep = keep && fabs(dx) - hw < rc && fabs(pery ? min_image_n(dyr, ny) : dyr) - hh < rc;
        const unsigned long long bal = __ballot(keep);
        if (bal == 0) continue;
        int base = 0;
        if (lane == 0) base = atomicAdd(&s_n, __popcll(bal));
        const int pos = __builtin_amdgcn_readfirstlane(base) + __popcll(bal & below);
        if (keep && pos < kRepCand) {
          s_x[pos] = xm + dx;   // unwrapped next to the box
          s_y[pos] = y2[q];
          s_id[pos] = m2[q];
        }
      }
    }
  }
  __syncthreads();
  int ncand = s_n;
  if (ncand > kRepCand) {
    if (t == 0) atomicAdd(p.overflow, 1);
    ncand = kRepCand;
  }

  // ---- 3. rank by (x, id): a fixed order for the sums (four lanes per
  // candidate)
  for (int i0 = 0; i0 < ncand; i0 += kRepThreads / 4) {
    const int i = min(i0 + (t >> 2), ncand - 1);
    const double xi = s_x[i];
    const int ii = s_id[i];
    int r = 0;
    for (int j = t & 3; j < ncand; j += 4) {
      const double xj = s_x[j];
      r += (xj < xi || (xj == xi && s_id[j] < ii)) ? 1 : 0;
    }
    r += __shfl_xor(r, 1);
    r += __shfl_xor(r, 2);
    if ((t & 3) == 0 && i0 + (t >> 2) < ncand) {
      s_sx[r] = xi;
      s_sy[r] = s_y[i];
    }
  }
  __syncthreads();

  // ---- 4. per vertex: the close candidates of the x window, in rank order.
  // A box wider than about half the lattice could see a candidate through
  // both images; the vertex then scans all candidates with the minimum
  // image per pair.
  const bool window = 2.0 * (hw + rc) + 2.0 < 0.5 * nx;
  const double xvr = xm + min_image_n(xv - xm, nx);
  int j0 = 0, j1 = ncand;
  if (window) {
    // first candidate with x >= xv - rc, and first with x > xv + rc
    int lo = 0, hi = ncand, lo1 = 0, hi1 = ncand;
    while (lo < hi || lo1 < hi1) {
      const int mid = (lo + hi) >> 1, mid1 = (lo1 + hi1) >> 1;
      const double a = s_sx[min(mid, kRepCand - 1)], c = s_sx[min(mid1, kRepCand - 1)];
      if (lo < hi) {
        if (a < xvr - rc) lo = mid + 1; else hi = mid;
      }
      if (lo1 < hi1) {
        if (c <= xvr + rc) lo1 = mid1 + 1; else hi1 = mid1;
      }
    }
    j0 = lo;
    j1 = lo1;
  }
  double S = 0.0;
  while (__ballot(j0 < j1) != 0ull) {   // 16 candidates of each of the wave's vertices
    const int j = j0 + (lane & 15);
    double term = 0.0;
    if (j < j1) {
      const double dx = min_image_n(s_sx[j] - xvr, nx);
      const double dyr = s_sy[j] - yv;
      const double dy = pery ? min_image_n(dyr, ny) : dyr;
      const double d = sqrt(dx * dx + dy * dy);
      if (d < rc) {
        const double d2 = d * d;
        term = sqrt(1.0 / (d2 * d2 * d));
      }
    }
    // the terms of the vertex in rank order (those that are zero add nothing)
    unsigned on = (unsigned)(__ballot(term != 0.0) >> (lane & 48)) & 0xffffu;
    while (__ballot(on != 0u) != 0ull) {
      const double a = __shfl(term, (lane & 48) | (on != 0u ? __ffs((int)on) - 1 : 0));
      if (on != 0u) S += coeff * a;
      on &= on - 1;
    }
    j0 += 16;
  }
  if ((lane & 15) == 0 && v < nvc) p.frep[gv] = S;
}

template <typename T>
void launch_repulsion(const Ptrs<T>& p, const StepArgs& a, const int* chunks, int nchunk,
                      hipStream_t s) {
  if (nchunk == 0) return;
  const dim3 grid(nchunk), block(kRepThreads);
  if (a.tile_x == 64 && a.tile_y == 4)
    hipLaunchKernelGGL((k_repulsion<T, 64, 4>), grid, block, 0, s, p, (const int4*)chunks);
  else if (a.tile_x == 128 && a.tile_y == 2)
    hipLaunchKernelGGL((k_repulsion<T, 128, 2>), grid, block, 0, s, p, (const int4*)chunks);
  else if (a.tile_x == 32 && a.tile_y == 8)
    hipLaunchKernelGGL((k_repulsion<T, 32, 8>), grid, block, 0, s, p, (const int4*)chunks);
  else
    hipLaunchKernelGGL((k_repulsion<T, 256, 1>), grid, block, 0, s, p, (const int4*)chunks);
}

template void launch_repulsion<float>(const Ptrs<float>&, const StepArgs&, const int*, int, hipStream_t);
template void launch_repulsion<double>(const Ptrs<double>&, const StepArgs&, const int*, int,
                                       hipStream_t);

}  // namespace lbib
