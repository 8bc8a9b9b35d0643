// Descriptor-driven launches: every kernel of an iteration is one launch over
// all instances of a batch (a single solve is a batch of one). Workgroup b of
// a launch takes the logical index L = xcd_remap(b) and serves instance
// map[L]; its block index inside that instance is L minus the instance's
// first block in that launch's grid. Instances may
// have different grids; each carries its own geometry, state pointers,
// constant tables and control block (sigma, stop flag), so each converges and
// stops on its own.
#pragma once
#include "geometry.hpp"
#include "kernels_dct.hpp"
#include "kernels_fused.hpp"
#include "kernels_plane.hpp"
#include "kernels_update.hpp"

namespace dot {

// Every workgroup starts by reading its descriptor: what the sweeps and the
// passes read stands together, in whole 64-byte lines.
template <typename T>
struct alignas(64) Inst {
  Geo g;
  double* phi;      // FP64 potential
  T* work;          // transform work plane: phi itself (FP64) or the FP32 scratch
  T* q[2];          // q and q_new, swapped every iteration (parity argument)
  double* alpha;    // multipliers alpha (FP64 in both modes: they accumulate updates)
  T* beta;
  T* W;             // 4D weighted w planes of the z-step
  double* dw;       // w_{K-1} - w_0 of the z-step (FP64)
  Ctl* ctl;         // nullptr for step-level calls (sigma from the argument)
  double* partials;
  const double* sw;
  const double* om;
  const double* c_lo;
  const double* c_hi;
  const T* lam_other;
  const T* lam_last;
  uint32_t blk0;             // first block in the per-node grid
  uint32_t tile0[kMaxAxes];  // first tile in each axis-pass grid
  int32_t tri;               // last axis solved by tridiagonal elimination (else transform, 1/Lambda, transform)
  AxisTab<T> tab[kMaxAxes];
  FinArgs fa;
  // one-sweep iteration: the second place of beta and alpha (the first is beta
  // and alpha above), the plane of its right-hand side and, at checks, of each
  // cell's |z - B F q_new - d|^2, and its workgroups
  BetaPlanes<T> beta2;
  double* alpha2;
  T* rhs2;
  double* ssq;
  double* ckpt;              // c' checkpoints of the one-lane elimination (W plane 0 without it)
  const double* piv;         // pivots of the last axis's lines (plans with few long lines)
  FuseGeo fg;
  uint32_t fblk0;            // first block in the fused grid
  uint32_t plane0;           // first block in the plane-solve grid
  uint32_t line0;            // first block in the long-line grid
};

// Instance of logical block L: map[L], or 0 without a map (an executor of
// one instance launches without one, saving the map load at every entry).
__device__ __forceinline__ uint32_t inst_of_block(const uint16_t* __restrict__ map, uint32_t L) {
  return map ? glob(map)[L] : 0u;
}

template <typename T>
__device__ __forceinline__ bool stopped(const Inst<T>& s) {
  return s.ctl && glob(s.ctl)->stop;
}

// z-step of iteration par's parity: cone gather and projection from q[par]
// and beta into the W planes.
template <typename T, int D>
__global__ void __launch_bounds__(256)
kb_cone(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int par) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  cone_body<T, D>(s.g, s.q[par], s.beta, s.sw, s.W, s.dw, s.ctl, L - s.blk0);
}

// q-step and alpha update: q[par ^ 1] from phi, alpha and the W planes.
template <typename T, int D>
__global__ void __launch_bounds__(256)
kb_q(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int par) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  q_body<T, D>(s.g, s.phi, s.alpha, s.om, s.q[par ^ 1], s.W, s.dw, s.ctl, L - s.blk0);
}

template <typename T, int D>
__global__ void __launch_bounds__(256)
kb_beta(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int par, int check) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  beta_body<T, D>(s.g, s.q[par], s.q[par ^ 1], s.beta, s.sw, s.ctl, s.partials, check, L - s.blk0);
}

// beta update of iteration it (no residual check) and the right-hand side of
// iteration it + 1 in one launch: both are sweeps over the same workgroups
// and neither reads what the other writes (rhs reads the new q and alpha, and
// phi for the defect; beta reads q, q_new and beta). sigma does not change
// between them (no check).
template <typename T, int D, bool DEFECT>
__global__ void __launch_bounds__(256)
kb_beta_rhs(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int par) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  const double inv_sigma = 1.0 / glob(s.ctl)->sigma;
  beta_body<T, D>(s.g, s.q[par], s.q[par ^ 1], s.beta, s.sw, s.ctl, s.partials, 0, L - s.blk0);
  rhs_body<T, D, DEFECT>(s.g, s.q[par ^ 1], s.alpha, s.phi, s.c_lo, s.c_hi, s.work, inv_sigma, L - s.blk0);
}

// beta update of iteration it (parity par, no residual check) and the z-step
// of iteration it + 1 (parity par ^ 1) in one sweep.
template <typename T, int D>
__global__ void __launch_bounds__(256)
kb_beta_cone(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int par) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  beta_cone_body<T, D>(s.g, s.q[par], s.q[par ^ 1], s.beta, s.sw, s.W, s.dw, s.ctl, L - s.blk0);
}

// kb_beta_cone and the right-hand side of iteration it + 1 in one launch (the
// right-hand side reads the new q, alpha and phi, none of which the other
// two steps write).
template <typename T, int D, bool DEFECT>
__global__ void __launch_bounds__(256)
kb_beta_cone_rhs(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int par) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  const double inv_sigma = 1.0 / glob(s.ctl)->sigma;
  beta_cone_body<T, D>(s.g, s.q[par], s.q[par ^ 1], s.beta, s.sw, s.W, s.dw, s.ctl, L - s.blk0);
  rhs_body<T, D, DEFECT>(s.g, s.q[par ^ 1], s.alpha, s.phi, s.c_lo, s.c_hi, s.work, inv_sigma, L - s.blk0);
}

// z-step and right-hand side of one iteration in one launch, where neither
// can join the previous beta update (after a residual check, whose sigma
// decision they must see, and at the start of a run): both read q[par] and
// write disjoint planes (W and dw; the transform work plane), and neither
// reads what the other writes.
template <typename T, int D, bool DEFECT>
__global__ void __launch_bounds__(256)
kb_cone_rhs(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int par) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  const double inv_sigma = 1.0 / glob(s.ctl)->sigma;
  cone_body<T, D>(s.g, s.q[par], s.beta, s.sw, s.W, s.dw, s.ctl, L - s.blk0);
  rhs_body<T, D, DEFECT>(s.g, s.q[par], s.alpha, s.phi, s.c_lo, s.c_hi, s.work, inv_sigma, L - s.blk0);
}

// The whole iteration outside the Poisson solve in one sweep (kernels_fused.hpp):
// alpha and beta from their place `par` (0: alpha, beta; 1: alpha2, beta2) into
// the other one, q[par] into q[par ^ 1].
template <typename T, int D, bool DEFECT, bool RHS, bool SSQ>
__global__ void __launch_bounds__(fuse_max_lanes(), 2)
kb_fuse(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int par) {
  const uint32_t L = xcd_remap32(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  const BetaPlanes<T> home{s.beta, s.beta + (size_t)(4 * D) * (size_t)s.g.nb};
  fuse_body<T, D, DEFECT, RHS, SSQ>(s.g, s.fg, s.phi, s.q[par], s.q[par ^ 1], par ? s.beta2 : home,
                                    par ? home : s.beta2, par ? s.alpha2 : s.alpha, par ? s.alpha : s.alpha2, s.sw,
                                    s.om, s.c_lo, s.c_hi, s.rhs2, s.ssq, s.ctl, L - s.fblk0);
}

// Right-hand side (or its defect against phi) of the Poisson solve into the
// transform work plane, from (q[par], alpha); place: where alpha is.
template <typename T, int D, bool DEFECT>
__global__ void __launch_bounds__(256)
kb_rhs(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int par, double sigma_arg, int place) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  const double inv_sigma = 1.0 / (s.ctl ? glob(s.ctl)->sigma : sigma_arg);
  rhs_body<T, D, DEFECT>(s.g, s.q[par], place ? s.alpha2 : s.alpha, s.phi, s.c_lo, s.c_hi, s.work, inv_sigma,
                         L - s.blk0);
}

// Residual partials at the iterate held in q[par] (the newest q). SSQ: slot 11
// (|z - B F q - d|^2) from the cells' plane that the one-sweep iteration wrote,
// with alpha and beta at `place`; otherwise kb_beta has filled it.
template <typename T, int D, bool SSQ>
__global__ void __launch_bounds__(256)
kb_resid(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int par, int place) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  const BetaPlanes<T> home{s.beta, s.beta + (size_t)(4 * D) * (size_t)s.g.nb};
  const bool alt = SSQ && place;
  resid_body<T, D, SSQ>(s.g, s.phi, s.q[par], alt ? s.alpha2 : s.alpha, alt ? s.beta2 : home, s.om, s.sw, s.c_lo,
                        s.c_hi, s.ssq, s.partials, L - s.blk0);
}

// First stage of the residual reduction: kFinChunks blocks per instance
// (block b: instance b / kFinChunks, chunk b % kFinChunks); instances below
// kFinStageMinRows rows return at once.
template <typename T>
__global__ void __launch_bounds__(256)
kb_fin_stage(const Inst<T>* __restrict__ I) {
  const Inst<T>& s = I[blockIdx.x / kFinChunks];
  if (!s.fa.staged || stopped(s)) return;
  fin_stage_body(s.fa, s.partials, (int)(blockIdx.x % kFinChunks));
}

// One block of 256 threads per instance.
template <typename T>
__global__ void __launch_bounds__(256)
kb_finalize(const Inst<T>* __restrict__ I, int update_ctl) {
  const Inst<T>& s = I[blockIdx.x];
  finalize_body(s.fa, s.partials, s.ctl, update_ctl);  // returns before the update if the instance stopped
}

template <typename T, int D, int KIND, int SRC, int DST, int CW>
__global__ void __launch_bounds__(kMaxWaves * 64)
kb_axis_pass(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int axis) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  if (KIND == kFwdScaleInv && s.tri) return;  // this instance's last axis takes kb_tri_pass
  PassArgs pa;
  pa.inner = s.g.stride[axis];
  pa.ncols = s.g.nb / s.g.N[axis];
  axis_pass_body<T, D, KIND, SRC, DST, CW>(s.g, pa, s.tab[axis], SRC == kSrcAlt ? s.rhs2 : nullptr, s.work, s.phi,
                                           s.lam_other, s.lam_last, (int64_t)(L - s.tile0[axis]));
}

// One plane of the last two axes per workgroup (kernels_plane.hpp).
template <typename T, int D, int SRC, int DST, int KS>
__global__ void __launch_bounds__(kPlaneThreads)
kb_plane(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  plane_body<T, D, SRC, DST, KS>(s.g, s.tab[D - 1], s.tab[D], SRC == kSrcAlt ? s.rhs2 : nullptr, s.work, s.phi,
                                 s.lam_other, s.lam_last, L - s.plane0);
}

// Last-axis tridiagonal solve over the tiles of the last-axis grid (CW lines
// each); the c' checkpoints go to W plane 0 where the separate sweeps run (an
// executor with such an instance runs the cone step after the phi-step, not
// beside it), to a buffer of their own where W holds the second place of beta.
template <typename T, int D, int CW>
__global__ void __launch_bounds__(kTriThreads)
kb_tri_pass(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s) || !s.tri || s.g.N[D] <= kTriPartMaxNodes) return;  // shorter lines: kb_tri_part
  tri_pass_body<T, CW>(s.g, s.work, s.ckpt, s.lam_other, (int64_t)(L - s.tile0[D]));
}

// The same where the launch has few long lines (tri_line_body), cw lines per
// workgroup of a grid of its own, and the pivots that it reads.
template <typename T, int D>
__global__ void __launch_bounds__(kTriThreads)
kb_tri_line(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int cw) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s)) return;
  tri_line_body<T>(s.g, s.work, s.piv, s.lam_other, (int64_t)(L - s.line0), cw);
}
template <typename T>
__global__ void __launch_bounds__(64)
kb_tri_pivots(Geo g, const T* __restrict__ lam_other, double* __restrict__ piv) {
  const int64_t line = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (line < g.nb / g.N[g.D]) tri_pivots<T>(g, lam_other, piv, line);
}

// Partitioned last-axis solve (lines of up to kTriPartMaxNodes nodes) over the
// same tile grid: tile t of an instance holds its lines [t cw, (t + 1) cw).
template <typename T, int D>
__global__ void __launch_bounds__(kTriThreads, 2)
kb_tri_part(const Inst<T>* __restrict__ I, const uint16_t* __restrict__ map, int cw) {
  const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
  const Inst<T>& s = I[inst_of_block(map, L)];
  if (stopped(s) || !s.tri || s.g.N[D] > kTriPartMaxNodes) return;
  tri_part_body<T>(s.g, s.work, s.lam_other, (int64_t)(L - s.tile0[D]), cw);
}

// ---- step-level kernels (single instance, caller pointers) ----------------

// Zero n 32-bit words.
__global__ void __launch_bounds__(256) kb_clear_words(uint32_t* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

template <typename T, int D>
__global__ void __launch_bounds__(256)
kb_cone_out(const Inst<T>* __restrict__ I, double inv_sigma, T* __restrict__ z) {
  const Inst<T>& s = I[0];
  cone_out_body<T, D>(s.g, s.q[0], s.beta, s.sw, inv_sigma, z, blockIdx.x);
}

template <typename T, int D>
__global__ void __launch_bounds__(256)
kb_zres(const Inst<T>* __restrict__ I, const T* __restrict__ z) {
  const Inst<T>& s = I[0];
  zres_body<T, D>(s.g, z, s.q[0], s.sw, s.partials, xcd_remap(blockIdx.x, gridDim.x));
}

template <typename T, int D>
__global__ void __launch_bounds__(256)
kb_divergence(const Inst<T>* __restrict__ I, double inv_sigma, double* __restrict__ b) {
  const Inst<T>& s = I[0];
  const Geo& g = s.g;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.nb) return;
  const int t = (int)(i / g.stride[0]);
  const uint32_t xs = (uint32_t)(i % g.stride[0]);
  int x[kMaxAxes];
  spatial_coords<D>(g, xs, x);
  b[i] = divergence_at<T, D>(g, s.q[0], s.alpha, s.c_lo, s.c_hi, inv_sigma, t, xs, x);
}

}  // namespace dot
