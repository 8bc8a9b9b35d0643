// One sweep for everything of an iteration of Algorithm 2 outside the Poisson
// solve: z-step, q-step, both multiplier steps and (between iterations without
// a residual check) the next right-hand side, from phi and the old (q, alpha,
// beta). The separate sweeps (kernels_update.hpp) hand the weighted w
// components from the z-step to the q-step through 4D + 1 planes and read q
// and beta again for the beta step; here z stays in registers between the
// steps, and only the iterate itself moves.
//
// Dependences of one node x: q_d(x) needs w at x and x + e_d (cells t - 1 and
// t), beta(x) and the right-hand side need q_d at x - e_d and x. A workgroup
// owns a box of spatial nodes (FuseGeo::a, one node per lane) and a run of
// time nodes; the cells next to the box on each side of each axis are further
// lanes ("halo"), which repeat the projection of their cell (and, on the
// lower sides, the one q_d that the box needs). The lanes march through time
// together; per slice w goes to the lower neighbour and q to the upper one
// through LDS. Halo lanes read old values that their owner is updating, so
// alpha and beta alternate between two places like q does (iteration parity).
//
// Bound by memory: 2D moves 34 planes of 8 bytes per iteration (FP64) instead
// of 58. 2D 64x256^2: 278 us FP64 and 190 us mixed (the separate sweeps took 490
// and 290), for 1154 and 696 MB if every element is moved once, 4.2 and 3.7 TB/s;
// with the halo's reads the counters give 1.30 GB in FP64, 4.7 TB/s, where a 1 GiB
// copy reaches 4.8. Nontemporal stores made it slower (389 -> 425 us per
// iteration: the planes no longer wait in the last-level cache), two slices of
// loads in flight changed nothing.
#pragma once
#include "geometry.hpp"
#include "kernels_update.hpp"

namespace dot {

// Lanes of a workgroup of the one-sweep iteration (at most).
constexpr int fuse_max_lanes() { return 512; }

struct FuseGeo {
  int32_t a[kMaxAxes];   // nodes of the box along the spatial axes 1..D
  int32_t nt[kMaxAxes];  // boxes along each spatial axis
  int32_t ni;            // a[1] * ... * a[D]
  int32_t lanes;         // ni and the halo lanes, 2 ni / a[d] per axis
  int32_t tc;            // time nodes per workgroup
  uint32_t ntile;        // boxes
  uint32_t nblk;         // workgroups: ntile * ceil(N0 / tc)
};

// What a lane loads for the cell of one time slice c (one slice ahead): its
// beta, its q0, q_d of node c + 1 and phi of node c + 1.
template <typename T, int D>
struct FuseCell {
  T bt[4 * D + 2];
  T q0;
  T fb[kMaxAxes][2];
  double ph1;
};
// What it loads for the node c, at the start of the slice and used after the
// z-step.
template <int D>
struct FuseNode {
  double a0;
  double ad[kMaxAxes];
};

// Position of a lane: its node, its part in the box or the halo, and the lanes
// it exchanges with.
struct FuseLane {
  uint32_t xs;
  int x[kMaxAxes];
  bool live;           // the node exists
  bool inner;          // in the box (live)
  bool qr[kMaxAxes];   // computes q_d
  uint32_t up[kMaxAxes], dn[kMaxAxes];  // elements to x + e_d and x - e_d (0 outside the grid)
  int plus[kMaxAxes];  // lane of x + e_d
  int minus[kMaxAxes]; // lane of x - e_d
};

// Lane order: the rows of the box along the last axis, each with its two halo
// nodes at the ends (a row's lanes read consecutive addresses), then the halo
// rows on the lower and upper side of each other axis.
template <int D>
__device__ __forceinline__ FuseLane fuse_lane(const Geo& g, const FuseGeo& f, uint32_t tile) {
  FuseLane s;
  int lo[kMaxAxes];  // first node of the box per axis
#pragma unroll
  for (int d = D; d >= 1; --d) {
    const uint32_t q = tile / (uint32_t)f.nt[d];
    lo[d] = (int)(tile - q * (uint32_t)f.nt[d]) * f.a[d];
    tile = q;
  }
  const int tid = threadIdx.x, row = f.a[D] + 2, body = f.ni / f.a[D] * row;
  int l[kMaxAxes] = {0, 0, 0, 0};
  int hd = 0, side = 0;  // halo lanes: axis and side (1: upper)
  bool used = tid < body;
  int p;
  if (used) {
    p = tid / row;
    l[D] = tid - p * row - 1;
    side = l[D] == f.a[D] ? 1 : 0;
    hd = l[D] < 0 || side ? D : 0;
  } else {
    p = tid - body;
#pragma unroll
    for (int d = 1; d < D; ++d) {
      const int gsz = f.ni / f.a[d];
      if (!used && p < 2 * gsz) {
        used = true;
        hd = d;
        side = p >= gsz ? 1 : 0;
        p -= side * gsz;
      } else if (!used) {
        p -= 2 * gsz;
      }
    }
    const int q = p / f.a[D];
    l[D] = p - q * f.a[D];
    p = q;
  }
#pragma unroll
  for (int d = D - 1; d >= 1; --d) {
    if (d == hd) {
      l[d] = side ? f.a[d] : -1;
    } else {
      const int q = p / f.a[d];
      l[d] = p - q * f.a[d];
      p = q;
    }
  }
  s.live = used;
  s.xs = 0;
#pragma unroll
  for (int d = 1; d <= D; ++d) {
    s.x[d] = lo[d] + l[d];
    s.live = s.live && s.x[d] >= 0 && s.x[d] < g.N[d];
    s.xs += (uint32_t)s.x[d] * (uint32_t)g.stride[d];
  }
  s.inner = s.live && hd == 0;
  if (!s.live) s.xs = 0;  // reads node 0 and keeps nothing
  // lane strides of the rows, and the first halo lane of each axis before the last
  int ls[kMaxAxes];
  ls[D] = 1;
  if (D > 1) ls[D > 1 ? D - 1 : 1] = D > 1 ? row : 1;
#pragma unroll
  for (int d = D - 1; d > 1; --d) ls[d - 1] = ls[d] * f.a[d];
  int hb = body;
#pragma unroll
  for (int d = 1; d <= D; ++d) {
    const int gsz = f.ni / f.a[d];
    int pos = 0, flat = 1;  // position among the other axes; lane of l with l[d] = 0
#pragma unroll
    for (int e = 1; e <= D; ++e) {
      if (e == d) continue;
      pos = pos * f.a[e] + l[e];
      flat += l[e] * ls[e];
    }
    s.qr[d] = (s.inner || (s.live && hd == d && side == 0)) && s.x[d] < g.n[d];
    if (d == D) {
      s.plus[d] = tid + 1;
      s.minus[d] = tid - 1;
    } else {
      s.plus[d] = l[d] < 0 ? flat : (l[d] + 1 < f.a[d] ? tid + ls[d] : hb + gsz + pos);
      s.minus[d] = l[d] > 0 ? tid - ls[d] : hb + pos;
      hb += 2 * gsz;
    }
    if (!s.inner) s.minus[d] = 0;
    if (!s.qr[d]) s.plus[d] = 0;
    s.up[d] = s.live && s.x[d] < g.n[d] ? (uint32_t)g.stride[d] : 0u;
    s.dn[d] = s.live && s.x[d] >= 1 ? (uint32_t)g.stride[d] : 0u;
  }
  return s;
}

// Element at byte offset `off` of a plane: a uniform base and a 32-bit lane
// offset (a plane holds at most 2^31 bytes), so that no lane computes 64-bit
// addresses.
template <typename T>
__device__ __forceinline__ T ld(gp<const T> base, uint32_t off) {
  return *(gp<const T>)((gp<const char>)base + off);
}
template <typename T>
__device__ __forceinline__ void st(gp<T> base, uint32_t off, T v) {
  *(gp<T>)((gp<char>)base + off) = v;
}

// Loads are not predicated: a neighbour outside the grid reads the node itself
// and a lane without a node reads node 0; those values are not used.
template <typename T, int D>
__device__ __forceinline__ void fuse_load_cell(const Geo& g, const FuseLane& L, int c, gp<const double> phi,
                                               gp<const T> q, const BetaPlanes<T>& beta, FuseCell<T, D>& s) {
  constexpr int K = 4 * D + 2;
  const uint32_t nb = (uint32_t)g.nb, nx = (uint32_t)g.nx, w = sizeof(T);
  const uint32_t i = (uint32_t)min(c, g.n[0] - 1) * nx + L.xs;  // the last node has no cell
  const uint32_t o = i * w, o1 = (i + nx) * w;
#pragma unroll
  for (int k = 0; k < K; ++k) s.bt[k] = ld<T>(beta_plane<T, D>(beta, k, nb), o);
  s.q0 = ld<T>(q, o);
#pragma unroll
  for (int d = 1; d <= D; ++d) {
    gp<const T> qd = q + (size_t)d * nb;
    s.fb[d][0] = ld<T>(qd, o1 - L.dn[d] * w);
    s.fb[d][1] = ld<T>(qd, o1);
  }
  s.ph1 = ld<double>(phi, (i + nx) * 8u);
}

template <int D>
__device__ __forceinline__ void fuse_load_node(const Geo& g, const FuseLane& L, int c, gp<const double> alpha,
                                               FuseNode<D>& s) {
  const uint32_t nb = (uint32_t)g.nb, nx = (uint32_t)g.nx;
  const uint32_t p = ((uint32_t)c * nx + L.xs) * 8u;
  s.a0 = ld<double>(alpha, p);
#pragma unroll
  for (int d = 1; d <= D; ++d) s.ad[d] = ld<double>(alpha + (size_t)d * nb, p);
}

// A wave-uniform value into scalar registers.
__device__ __forceinline__ double uniform(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}

// RHS: also the right-hand side of the next iteration (its defect against phi
// with DEFECT) into `out`; SSQ (checks): |z - B F q_new - d|^2 of each cell
// into `ssq`.
template <typename T, int D, bool DEFECT, bool RHS, bool SSQ>
__device__ __forceinline__ void fuse_body(const Geo& g, const FuseGeo& f, const double* __restrict__ phi_,
                                          const T* __restrict__ q_, T* __restrict__ qn_,
                                          const BetaPlanes<T>& beta, const BetaPlanes<T>& beta_out,
                                          const double* __restrict__ alpha_, double* __restrict__ alpha_out_,
                                          const double* __restrict__ sw_sp, const double* __restrict__ om_sp,
                                          const double* __restrict__ c_lo, const double* __restrict__ c_hi,
                                          T* __restrict__ out_, double* __restrict__ ssq_, Ctl* __restrict__ ctl,
                                          uint32_t blk) {
  constexpr int K = 4 * D + 2;
  constexpr int NT = fuse_max_lanes();
  // exchange of one slice: weighted w_{d,1} of the cell c and w_{d,3} of the
  // cell c - 1 (read by the lane of x - e_d), new q_d and q_d - alpha_d / sigma
  // (read by the lane of x + e_d), phi of the node c
  __shared__ double shp[NT];
  __shared__ T sh1[D][NT], sh3[D][NT], shq[D][NT];
  __shared__ double shy[RHS ? D : 1][RHS ? NT : 1];
  const uint32_t chunk = blk / f.ntile;
  const FuseLane L = fuse_lane<D>(g, f, blk - chunk * f.ntile);
  const int tid = threadIdx.x;
  const int n0 = g.n[0];
  const int t0 = (int)chunk * f.tc, t1 = min(t0 + f.tc, g.N[0]);
  const int cs = max(t0 - 1, 0), ce = min(t1, n0);
  gp<const double> phi = glob(phi_);
  gp<const T> q = glob(q_);
  gp<T> qn = glob(qn_);
  gp<const double> alpha = glob(alpha_);
  gp<double> alpha_out = glob(alpha_out_);
  const uint32_t nb = (uint32_t)g.nb, nx = (uint32_t)g.nx, w = sizeof(T);
  const double sigma = glob(ctl)->sigma;
  const double ts = uniform(glob(ctl)->tau * sigma), inv_sigma = uniform(1.0 / sigma);
  const double sw = glob(sw_sp)[L.xs];
  double omsum[kMaxAxes];
  double ph, phm = 0.0;
  T fa[kMaxAxes][2];  // old q_d at node c
  {
    const uint32_t i = (uint32_t)cs * nx + L.xs;
    ph = phi[i];
#pragma unroll
    for (int d = 1; d <= D; ++d) {
      gp<const T> qd = q + (size_t)d * nb;
      const T lo = qd[i - L.dn[d]], hi = qd[i];
      fa[d][0] = L.x[d] >= 1 ? lo : T(0);
      fa[d][1] = L.x[d] < g.n[d] ? hi : T(0);
      omsum[d] = glob(om_sp)[L.xs] + glob(om_sp)[L.xs + L.up[d]];
    }
  }
  // carried to the next slice: z and beta of the components (d, 3), (d, 4) of
  // the cell (and its sum of squares so far), weighted w_{d,3} and w_{d,4},
  // q0 - alpha0 / sigma
  double z34[kMaxAxes][2], ssq = 0.0, y0m = 0.0;
  T b34[kMaxAxes][2], w3p[kMaxAxes], w4p[kMaxAxes];
#pragma unroll
  for (int d = 1; d <= D; ++d) {
    w3p[d] = w4p[d] = b34[d][0] = b34[d][1] = T(0);
    z34[d][0] = z34[d][1] = 0.0;
  }
  FuseCell<T, D> cur, nxt;
  fuse_load_cell<T, D>(g, L, cs, phi, q, beta, cur);
  for (int c = cs; c <= ce; ++c) {
    FuseNode<D> nd;
    fuse_load_node<D>(g, L, c, alpha, nd);
    fuse_load_cell<T, D>(g, L, c + 1, phi, q, beta, nxt);  // in flight while slice c is computed
    const uint32_t i = (uint32_t)c * nx + L.xs;
    const bool now = c < n0, prev = c >= 1, own = c >= t0 && c < t1;
    // z-step of the cell c
    double u[K], p[K];
    T fb[kMaxAxes][2], w2[kMaxAxes], w3[kMaxAxes], w4[kMaxAxes];
#pragma unroll
    for (int d = 1; d <= D; ++d) {
      // q_d outside its set: zero
      fb[d][0] = L.x[d] >= 1 ? cur.fb[d][0] : T(0);
      fb[d][1] = L.x[d] < g.n[d] ? cur.fb[d][1] : T(0);
    }
    cone_arg<T, D>(cur.bt, (double)cur.q0, fa, fb, sw, inv_sigma, u, p);
    soc_project_select<K>(u);
#pragma unroll
    for (int d = 1; d <= D; ++d) {
      const int k = 1 + 4 * (d - 1);
      sh1[d - 1][tid] = cone_w<T>(u[k + 0], p[k + 0], sw);
      sh3[d - 1][tid] = w3p[d];
      w2[d] = cone_w<T>(u[k + 1], p[k + 1], sw);
      w3[d] = cone_w<T>(u[k + 2], p[k + 2], sw);
      w4[d] = cone_w<T>(u[k + 3], p[k + 3], sw);
      fa[d][0] = fb[d][0];
      fa[d][1] = fb[d][1];
    }
    const double wsum = cone_dw<K>(u, p);
    shp[tid] = ph;
    __syncthreads();
    // q-step and alpha at node c (nodes t0..t1; t1 only for the beta step of
    // the last cell) and, per cell, q0 and alpha0
    T gn[kMaxAxes][2];  // new q_d at node c
    double yd[kMaxAxes], phs[kMaxAxes][2];  // phi at x - e_d and x + e_d
#pragma unroll
    for (int d = 1; d <= D; ++d) {
      phs[d][1] = shp[L.plus[d]];
      phs[d][0] = DEFECT && RHS ? shp[L.minus[d]] : 0.0;
      double acc = 0.0;
      if (now) acc += (double)sh1[d - 1][L.plus[d]] + (double)w2[d];
      if (prev) acc += (double)sh3[d - 1][L.plus[d]] + (double)w4p[d];
      const double ct = (double)now + (double)prev;
      const double diag = fma(0.5 * ct, omsum[d], 1.0);
      const double dphi = phs[d][1] - ph;
      const double qdn = qd_new<D>(dphi, g.inv_h[d], nd.ad[d], inv_sigma, acc, diag);
      const double an = alpha_new(nd.ad[d], ts, dphi, g.inv_h[d], qdn);
      const T qt = (T)qdn;
      gn[d][1] = L.x[d] < g.n[d] ? qt : T(0);
      yd[d] = fma(-inv_sigma, an, (double)qt);
      shq[d - 1][tid] = qt;
      if (RHS) shy[RHS ? d - 1 : 0][RHS ? tid : 0] = yd[d];
      if (own && L.inner && L.x[d] < g.n[d]) {
        st<T>(qn + (size_t)d * nb, i * w, qt);
        st<double>(alpha_out + (size_t)d * nb, i * 8u, an);
      }
    }
    double q0n, y0;
    {
      const double dphi = cur.ph1 - ph;
      const double v = q0_new(dphi, g.inv_h[0], nd.a0, inv_sigma, wsum);
      const double an = alpha_new(nd.a0, ts, dphi, g.inv_h[0], v);
      q0n = (double)(T)v;
      y0 = fma(-inv_sigma, an, q0n);
      if (own && now && L.inner) {
        st<T>(qn, i * w, (T)v);
        st<double>(alpha_out, i * 8u, an);
      }
    }
    __syncthreads();
    double yl[kMaxAxes];
#pragma unroll
    for (int d = 1; d <= D; ++d) {
      const T ql = shq[d - 1][L.minus[d]];
      gn[d][0] = L.x[d] >= 1 ? ql : T(0);
      yl[d] = RHS ? shy[RHS ? d - 1 : 0][RHS ? L.minus[d] : 0] : 0.0;
    }
    if (c > t0) {
      // beta step of the cell c - 1, components that meet q at node c
      T bn[kMaxAxes][2];
      ssq = beta_second<T, D>(z34, b34, gn, sw, ts, ssq, bn);
      if (L.inner) {
#pragma unroll
        for (int d = 1; d <= D; ++d) {
#pragma unroll
          for (int v = 0; v < 2; ++v)
            st<T>(beta_plane<T, D>(beta_out, 4 * (d - 1) + 3 + v, nb), (i - nx) * w, bn[d][v]);
        }
        if (SSQ) st<double>(glob(ssq_), (i - nx) * 8u, ssq);
      }
    }
    if (own && now) {
      // beta step of the cell c, components that meet q at node c
      T bn[K];
      ssq = beta_first<T, D>(u, cur.bt, q0n, gn, sw, ts, bn);
      if (L.inner) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
          if (k == 0 || k == K - 1 || (k - 1) % 4 < 2) st<T>(beta_plane<T, D>(beta_out, k, nb), i * w, bn[k]);
        }
      }
    }
    if (RHS && own) {
      double b = 0.0;
      if (prev) b = fma(y0m, g.inv_h[0], b);
      if (now) b = fma(-g.inv_h[0], y0, b);
#pragma unroll
      for (int d = 1; d <= D; ++d) {
        const double bl = fma(yl[d], g.inv_h[d], b);
        b = L.x[d] >= 1 ? bl : b;
        const double bh = fma(-g.inv_h[d], yd[d], b);
        b = L.x[d] < g.n[d] ? bh : b;
      }
      if (c == 0) b = fma(-inv_sigma, glob(c_lo)[L.xs], b);
      if (c == n0) b = fma(-inv_sigma, glob(c_hi)[L.xs], b);
      if (DEFECT) b -= neg_laplacian<D>(g, c, L.x, ph, phm, cur.ph1, phs);
      if (L.inner) st<T>(glob(out_), i * w, (T)b);
    }
    phm = ph;
    ph = cur.ph1;
    y0m = y0;
#pragma unroll
    for (int d = 1; d <= D; ++d) {
      w3p[d] = w3[d];
      w4p[d] = w4[d];
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        z34[d][v] = u[4 * (d - 1) + 3 + v];
        b34[d][v] = cur.bt[4 * (d - 1) + 3 + v];
      }
    }
    cur = nxt;
  }
  if (blk == 0 && tid == 0) glob(ctl)->iter += 1;
}

}  // namespace dot
