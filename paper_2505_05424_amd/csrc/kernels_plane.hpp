// Poisson solve along the last two axes of one plane in one workgroup: forward
// transforms along both, 1/Lambda, inverse transforms along both, with the
// plane in LDS from one load to one store. It replaces three passes
// (kernels_dct.hpp) and computes the same products in the same order.
//
// It is bound by latency, not by memory or the matrix cores: a launch takes
// 7.6 us at 1D 16x32 in FP64 and 11.9 us at 2D 32x63^2 in mixed precision, and
// an iteration 17.3 us instead of 23.7 and 38.2 instead of 43.7. So every wave
// of the workgroup has its share of a transform from the start: it keeps one
// 16-row block of a half matrix in registers (requested a transform ahead, one
// coalesced load per k-step) and runs it over one block of 16 lines (two on
// axes of more than 64 points); the folds of the first axis join the load and
// the store. Reading the fragments from the passes' chunked tables instead
// cost 0.7 us a launch at 1D 16x32.
#pragma once
#include "kernels_dct.hpp"

namespace dot {

// KS = 8 k-steps hold a half matrix of an axis of up to 64 points (at most two
// row blocks a parity, so 16 waves take four line blocks at once); KS = 9 of
// up to 72, with two line blocks per wave.
constexpr int kPlaneAxis = 72, kPlaneThreads = 1024, kPlaneWaves = kPlaneThreads / 64;
constexpr int plane_items(int KS) { return KS == 8 ? 1 : 2; }
constexpr int plane_rows(int L) { return ((L - L / 2) + 15) / 16 + (L / 2 + 15) / 16; }  // row blocks of both halves
// Line blocks of one wave of a transform along L points over `lines` lines.
constexpr int plane_blocks(int L, int lines) {
  return ((lines + 15) / 16 + kPlaneWaves / plane_rows(L) - 1) / (kPlaneWaves / plane_rows(L));
}
// LDS row of n points of T: lanes that read 16 rows at one column fall on
// different banks (FP64: odd; FP32: 2 mod 4, two columns at a time).
template <typename T>
__host__ __device__ constexpr int plane_stride(int n) {
  return sizeof(T) == 8 ? (n | 1) : n + (2 - n % 4 + 4) % 4;
}

// The half matrices again, lane-major, follow the chunked tables of an axis
// that the plane solve may take (fe, fo, ie, io, then these four in the same
// order): element (row block m, k-step s, lane) at (m * steps + s) * 64 + lane,
// steps = the k-steps that hold inputs, so a k-step is one coalesced load.
// Offset of the one asked for from fe.
template <typename T>
__host__ __device__ inline uint32_t plane_tab(const AxisTab<T>& a, bool inv, bool odd) {
  const uint32_t ce = (uint32_t)a.rb_e * (a.ks_e / kU + 1) * 64 * kU, co = (uint32_t)a.rb_o * (a.ks_o / kU + 1) * 64 * kU;
  const uint32_t le = (uint32_t)a.rb_e * ((a.ne + 3) / 4) * 64, lo = (uint32_t)a.rb_o * ((a.no + 3) / 4) * 64;
  return 2 * (ce + co) + (inv ? le + lo : 0u) + (odd ? le : 0u);
}

// Fragments of the row block of this wave (wave w of a transform: row block
// w % R of its R, line blocks w / R, w / R + 16 / R, ...).
template <typename T, int KS>
__device__ __forceinline__ void plane_coef(const AxisTab<T>& a, bool inv, T (&cf)[KS]) {
  const int R = a.rb_e + a.rb_o;
  const int rb = wave_id() % R;
  const bool odd = rb >= a.rb_e;
  const int m = odd ? rb - a.rb_e : rb;
  const int kr = ((odd ? a.no : a.ne) + 3) >> 2;
  gp<const T> t = glob(a.fe) + plane_tab(a, inv, odd) + (uint32_t)(m * kr) * 64 + (threadIdx.x & 63);
#pragma unroll
  for (int s = 0; s < KS; ++s) cf[s] = s < kr ? t[s * 64] : T(0);
}

// Both half-size products of one direction over the lines of the plane:
// element k of line c at k * sk + c * sc. scale(slot, line) multiplies the
// result of a forward transform before it is stored.
template <typename T, int KS, typename Scale>
__device__ __forceinline__ void plane_mfma(T* tile, const AxisTab<T>& a, bool inv, int sk, int sc, int lines,
                                           const T (&cf)[KS], Scale&& scale) {
  typedef typename MfmaOps<T>::acc_t acc_t;
  const int lane = threadIdx.x & 63, w = wave_id();
  const int R = a.rb_e + a.rb_o;
  const int rb = w % R, lb0 = w / R, gr = kPlaneWaves / R;
  const bool odd = rb >= a.rb_e;
  const int m = odd ? rb - a.rb_e : rb;
  const int nin = odd ? a.no : a.ne;
  const int kr = (nin + 3) >> 2;
  // slots of input k: first + step k
  const int step = inv ? 2 : (odd ? -1 : 1);
  const int first = inv ? (odd ? 1 : 0) : (odd ? a.L - 1 : 0);
  acc_t acc[plane_items(KS)];
#pragma unroll
  for (int b = 0; b < plane_items(KS); ++b) {
    acc[b] = acc_t{0, 0, 0, 0};
    const int c = (lb0 + b * gr) * 16 + (lane & 15);
    if (lb0 >= gr || (lb0 + b * gr) * 16 >= lines) continue;
    const int at = first * sk + min(c, lines - 1) * sc;  // lines past the last: repeated, not stored
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s < kr) {
        const int k = min(4 * s + (lane >> 4), nin - 1);  // padded inputs: zero coefficient
        acc[b] = MfmaOps<T>::mma(cf[s], tile[at + k * step * sk], acc[b]);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < plane_items(KS); ++b) {
    const int c = (lb0 + b * gr) * 16 + (lane & 15);
    if (lb0 >= gr || c >= lines) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = m * 16 + MfmaOps<T>::out_row(lane, v);
      if (r < nin) {  // a half matrix is square
        const int sl = out_slot(inv, odd, a.L, r);
        tile[sl * sk + c * sc] = acc[b][v] * scale(sl, c);
      }
    }
  }
  __syncthreads();
}

// Plane `o` (N1 x N2 points, contiguous) of the work plane, in place; 1D: the
// whole box, from the source and to the destination of the first and last pass.
template <typename T, int D, int SRC, int DST, int KS>
__device__ __forceinline__ void plane_body(const Geo& g, const AxisTab<T>& t1, const AxisTab<T>& t2,
                                           const T* __restrict__ src, T* __restrict__ plane,
                                           double* __restrict__ phi, const T* __restrict__ lam_other,
                                           const T* __restrict__ lam_last, uint32_t o) {
  extern __shared__ unsigned char smem_raw[];
  T* tile = reinterpret_cast<T*>(smem_raw);
  const int N1 = g.N[D - 1], N2 = g.N[D];
  const int S = plane_stride<T>(N2);
  T* lam_c = tile + N1 * S;
  T* lam_r = lam_c + N1;
  const uint32_t base = o * (uint32_t)(N1 * N2);
  gp<T> pl = glob(plane);
  gp<double> ph = glob(phi);
  T c0[KS], c1[KS];
  plane_coef<T, KS>(t1, false, c0);
  plane_coef<T, KS>(t2, false, c1);
  for (int e = threadIdx.x; e < N1 + N2; e += kPlaneThreads) {
    if (e < N1)
      lam_c[e] = glob(lam_other)[o * (uint32_t)N1 + e];
    else
      lam_r[e - N1] = glob(lam_last)[e - N1];
  }
  auto read = [&](uint32_t i) -> T {
    return SRC == kSrcPlaneF64 ? (T)ph[i] : (SRC == kSrcAlt ? glob(src)[i] : pl[i]);
  };
  // load with the fold of the first axis: rows j and N1 - 1 - j together (the
  // middle row of an odd count stays as it is)
  const int pairs = (N1 - N1 / 2) * N2;
  for (int e0 = threadIdx.x; e0 < pairs; e0 += 4 * kPlaneThreads) {
    T lo[4], hi[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int e = e0 + r * kPlaneThreads;
      const int j = e / N2, c = e - j * N2;
      lo[r] = e < pairs ? read(base + (uint32_t)e) : T(0);
      hi[r] = e < pairs ? read(base + (uint32_t)((N1 - 1 - j) * N2 + c)) : T(0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int e = e0 + r * kPlaneThreads;
      if (e >= pairs) continue;
      const int j = e / N2, c = e - j * N2;
      const bool mid = 2 * j == N1 - 1;
      tile[j * S + c] = mid ? lo[r] : lo[r] + hi[r];
      if (!mid) tile[(N1 - 1 - j) * S + c] = lo[r] - hi[r];
    }
  }
  __syncthreads();
  auto one = [](int, int) { return T(1); };
  const int M2 = N2 / 2;
  plane_mfma<T, KS>(tile, t1, false, S, 1, N2, c0, one);
  plane_coef<T, KS>(t2, true, c0);
  for (int e = threadIdx.x; e < M2 * N1; e += kPlaneThreads) {
    const int c = e / M2, j = e - c * M2;
    const T x0 = tile[c * S + j], x1 = tile[c * S + N2 - 1 - j];
    tile[c * S + j] = x0 + x1;
    tile[c * S + N2 - 1 - j] = x0 - x1;
  }
  __syncthreads();
  plane_mfma<T, KS>(tile, t2, false, 1, S, N1, c1, [&](int k, int c) {
    const T lam = lam_c[c] + lam_r[k];
    return lam > T(0) ? T(1) / lam : T(0);  // mode (0,...,0): phi in rge A^*
  });
  plane_coef<T, KS>(t1, true, c1);
  plane_mfma<T, KS>(tile, t2, true, 1, S, N1, c0, one);
  for (int e = threadIdx.x; e < M2 * N1; e += kPlaneThreads) {
    const int c = e / M2, j = e - c * M2;
    const T x0 = tile[c * S + j], x1 = tile[c * S + N2 - 1 - j];
    tile[c * S + j] = x0 + x1;
    tile[c * S + N2 - 1 - j] = x0 - x1;
  }
  __syncthreads();
  plane_mfma<T, KS>(tile, t1, true, S, 1, N2, c1, one);
  auto put = [&](uint32_t i, T v) {
    if (DST == kDstPhiAdd)
      ph[i] += (double)v;
    else if (DST == kDstPhiSet)
      ph[i] = (double)v;
    else
      pl[i] = v;
  };
  for (int e = threadIdx.x; e < pairs; e += kPlaneThreads) {
    const int j = e / N2, c = e - j * N2;
    const T x0 = tile[j * S + c];
    if (2 * j == N1 - 1) {
      put(base + (uint32_t)e, x0);
    } else {
      const T x1 = tile[(N1 - 1 - j) * S + c];
      put(base + (uint32_t)e, x0 + x1);
      put(base + (uint32_t)((N1 - 1 - j) * N2 + c), x0 - x1);
    }
  }
}

}  // namespace dot
