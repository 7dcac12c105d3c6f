// Pieces the per-iteration launches and the persistent iteration kernel have
// in common: block sizes, launch modes and the terms of one contact pair.
#pragma once

#include "sweep_common.h"

namespace pncg {

// Threads per block of the vertex-centric sweep: it is latency bound and
// gains from more resident waves per compute unit than the 256-thread blocks
// of the other kernels give (the grid, and so the number of partials, stays
// the same).  Measured on the 110k-tet pile: float 448 (seven waves, about
// 115 VGPRs, so two blocks hold 14 waves of a compute unit: 24.2 us against
// 25.4 us at 384; 512 needs 131 VGPRs and drops to three waves per SIMD).
// Double 448 too (122 VGPRs, no spill; 512 with a four-wave cap spilled
// 16 B per lane): the 30,000-tet bar's forward step 13.6 -> 13.1 ms; except
// the corotated model (below).
template <typename R, int M>
struct GradBlock {
  static constexpr int value = 448, min_waves = 1;
};
// The float64 corotated sweep needs 134-156 VGPRs: at 448 threads one block
// fills a compute unit; 512 threads capped at four waves per SIMD keep two.
template <>
struct GradBlock<double, kModelCorot> {
  static constexpr int value = 512, min_waves = 4;
};

// Threads per block of the direction kernel.  With more than kSBlock, the
// first kSBlock threads take the tets while the waves beyond them take the
// vertices, so that the two passes' memory round trips overlap instead of
// adding up (pile: 12.6 -> 12.3 us float, 14.7 -> 14.3 us float64).  The
// float64 corotated instantiation keeps kSBlock threads doing both passes:
// with the split it measured 17.4 against 10.9 us on the 30,000-tet bar.
template <typename R, int M>
struct DirBlock {
  static constexpr int value = (sizeof(R) == sizeof(double) && M == kModelCorot) ? kSBlock : 384;
};

enum FirstMode { kModeNormal = 0, kModeFinish = 1, kModeResume = 2, kModeContinue = 3 };

// ----------------------------------------------------------- pair terms
// One candidate pair at positions from `pos`: closest points (Sec. 3.2),
// returns false if inactive.  Penetration raises the error bit.
template <typename R, typename Pos>
__device__ __forceinline__ bool pair_closest(const Args<R>& A, int q, const Pos& pos, int (&iv)[4], Closest& c,
                                             long long npt) {
  V3<double> X[4];
  if (A.pv) {
    // the pair index holds the corner vertices: one load fewer on the way
    // to the positions
    const int4 w = A.pv[q];
    iv[0] = w.x; iv[1] = w.y; iv[2] = w.z; iv[3] = w.w >= 0 ? w.w : ~w.w;
#pragma unroll
    for (int i = 0; i < 4; ++i) X[i] = pos(iv[i]);
    c = w.w >= 0 ? closest_pt(X[0], X[1], X[2], X[3]) : closest_ee(X[0], X[1], X[2], X[3]);
    if (!(c.d > 0.0)) {
      raise_err(A.status, kErrPenetration);
      return false;
    }
    return c.d < A.dhat;
  }
  int2 pr = A.cand[q];
  // kind: by position in a sorted list (npt >= 0), or in the pair itself
  // (npt < 0: edge-edge pairs are stored as (e1, ~e2))
  if (npt >= 0 ? q < npt : pr.y >= 0) {
    iv[0] = pr.x;
    iv[1] = A.tris[3 * pr.y]; iv[2] = A.tris[3 * pr.y + 1]; iv[3] = A.tris[3 * pr.y + 2];
#pragma unroll
    for (int i = 0; i < 4; ++i) X[i] = pos(iv[i]);
    c = closest_pt(X[0], X[1], X[2], X[3]);
  } else {
    const int e2 = pr.y >= 0 ? pr.y : ~pr.y;
    iv[0] = A.edges[2 * pr.x]; iv[1] = A.edges[2 * pr.x + 1];
    iv[2] = A.edges[2 * e2]; iv[3] = A.edges[2 * e2 + 1];
#pragma unroll
    for (int i = 0; i < 4; ++i) X[i] = pos(iv[i]);
    c = closest_ee(X[0], X[1], X[2], X[3]);
  }
  if (!(c.d > 0.0)) {
    raise_err(A.status, kErrPenetration);
    return false;
  }
  return c.d < A.dhat;
}

// coefficient of (J t)(J t)^T and of J J^T in kappa * d2b/dx2 (eq9, or its
// PSD projection (b''/d^2)(J t)(J t)^T when not BARRIER_FULL)
template <typename R>
__device__ __forceinline__ void pair_hess_coefs(const Args<R>& A, double d, double& ca, double& cb) {
  const double b1 = barrier_db(d, A.dhat), b2 = barrier_d2b(d, A.dhat);
  if (A.flags & 1u) {
    ca = A.kappa * (b2 / (d * d) - b1 / (d * d * d));
    cb = A.kappa * b1 / d;
  } else {
    ca = A.kappa * b2 / (d * d);
    cb = 0.0;
  }
}

// a[i] of four values by selects: a register array indexed by a runtime value
// would be kept in scratch memory.
template <typename T>
__device__ __forceinline__ T pick4(const T (&a)[4], int i) {
  const T lo = i == 0 ? a[0] : a[1], hi = i == 2 ? a[2] : a[3];
  return i < 2 ? lo : hi;
}

// Barrier gradient and diagonal at corner i of an active pair (eq8, eq10,
// eq11): val = {g xyz, diag xyz}.
template <typename R>
__device__ __forceinline__ void pair_grad_diag_corner(const Args<R>& A, const Closest& c, int i, double (&val)[6]) {
  const double d = c.d;
  const double cg = A.kappa * barrier_db(d, A.dhat) / d;
  double ca, cb;
  pair_hess_coefs(A, d, ca, cb);
  const double ci = pick4(c.c, i);
  const double tx = ci * c.t.x, ty = ci * c.t.y, tz = ci * c.t.z;
  const double dj = cb * ci * ci;
  val[0] = cg * tx; val[1] = cg * ty; val[2] = cg * tz;
  val[3] = fma(ca * tx, tx, dj); val[4] = fma(ca * ty, ty, dj); val[5] = fma(ca * tz, tz, dj);
}

// p^T H p of an active pair from sp = sum_i c_i p_i and t (eq12, eq13)
__device__ __forceinline__ double pair_pHp(double ca, double cb, V3<double> sp, V3<double> t) {
  const double st = dot(sp, t);
  return fma(cb, dot(sp, sp), ca * st * st);
}

// ---------------------------------------------------------- vertex terms
// One component of g and of diag(H) without planes and pairs, from the sums
// sg, sd of the element terms: h^2 times those and the inertia.
__device__ __forceinline__ double vertex_g(double h2, double sg, double m, double x, double xt) {
  return fma(h2, sg, m * (x - xt));
}
__device__ __forceinline__ double vertex_diag(double h2, double sd, double m) { return fma(h2, sd, m); }
// a plane's part, component n of its normal: b1, b2 = kappa b', kappa b''
__device__ __forceinline__ void add_plane(double b1, double b2, double n, double& g, double& d) {
  g = fma(b1, n, g);
  d = fma(b2 * n, n, d);
}
// The products for beta, one component: g, P g, the previous g, p, and 1 / diag
__device__ __forceinline__ void add_beta_dots(double g, double pg, double g_prev, double p, double P, double* dots) {
  const double y = g - g_prev;
  dots[0] = fma(g, g, dots[0]);
  dots[1] = fma(g, pg, dots[1]);
  dots[2] = fma(g * P, y, dots[2]);
  dots[3] = fma(y, p, dots[3]);
  dots[4] = fma(y * P, y, dots[4]);
  dots[5] = fma(p, g, dots[5]);
}

// ------------------------------------------------------- iteration scalars
// d^T g of the direction -P g + beta p
__device__ __forceinline__ double direction_gTp(double beta, double pg, double gPg) { return fma(beta, pg, -gPg); }
// predicted decrease (Sec. 4.4)
__device__ __forceinline__ double predicted_dE(double alpha, double gTp, double pHp) {
  return fma(-(0.5 * alpha * alpha), pHp, -(alpha * gTp));
}

}  // namespace pncg
