// hydro_device.hpp -- device-side arithmetic shared by the forward and the
// adjoint kernels of libhydro: ghost-cell maps, conserved->primitive recovery,
// flux splitting, the WENO7 reconstruction, jet helpers.
#pragma once

#include <hip/hip_runtime.h>

#include "hydro_internal.hpp"

namespace hydro {

// ---------------------------------------------------------------------------
// Ghost-cell index map: outflow = copy of the edge cell, periodic = wrap.
__device__ __forceinline__ int map_idx(int p, int n, int bc) {
  if (bc) {
    int r = p % n;
    return r < 0 ? r + n : r;
  }
  return min(max(p, 0), n - 1);
}

template <class R>
__device__ __forceinline__ void load5(const R* __restrict__ W, long long nc, long long cell, R u[5]) {
#pragma unroll
  for (int c = 0; c < 5; ++c) u[c] = W[c * nc + cell];
}

// ---------------------------------------------------------------------------
// Reciprocal for FP64: hardware estimate, two Newton steps (quadratic
// convergence from the estimate's ~23 bits to full precision).
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  return r;
}

// num / den from one reciprocal plus a residual correction: the estimate
// (~23 bits) after one Newton step (~46 bits) gives q = num r to ~2^-46, and
// q + (num - den q) r squares that error away (below the rounding of q).
__device__ __forceinline__ double div_nr(double num, double den) {
  double r = __builtin_amdgcn_rcp(den);
  r = fma(fma(-den, r, 1.0), r, r);
  const double q = num * r;
  return fma(fma(-den, q, num), r, q);
}

// sqrt(x) for normal x > 0: from the reciprocal square root estimate (~23
// bits) one Newton step for sqrt(x) (~45 bits) and one residual correction,
// whose factor 1/(2 sqrt(x)) need not be better than the estimate.
__device__ __forceinline__ double sqrt_nr(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y;
  const double h = 0.5 * y;
  g = fma(g, fma(-g, h, 0.5), g);
  return fma(fma(-g, g, x), h, g);
}

// Conserved -> primitive for p = e/3 (FP64): e = 3(E^2 - M^2)/(E + sqrt(4E^2
// - 3M^2)), v = M/(E + e/3).  Non-admissible cells are fixed up for the
// primitive calculation only (E <= 1e-12: vacuum at rest; |M| >= (1-1e-10) E:
// M rescaled to that speed) and counted.
struct PrimV {
  double e;
  double v[3];
};

__device__ __forceinline__ PrimV c2p(double E, double Mx, double My, double Mz, unsigned& fix) {
  PrimV r;
  if (E <= kEFloor) {
    ++fix;
    r.e = kEFloor;
    r.v[0] = r.v[1] = r.v[2] = 0.0;
    return r;
  }
  const double E2 = E * E;
  double M2 = fma(Mz, Mz, fma(My, My, Mx * Mx));
  if (M2 >= kVCap * kVCap * E2) {
    ++fix;
    const double sc = kVCap * E / sqrt(M2);
    Mx = Mx * sc;
    My = My * sc;
    Mz = Mz * sc;
    M2 = fma(Mz, Mz, fma(My, My, Mx * Mx));
  }
  const double n = 3.0 * (E2 - M2);  // 4E^2 - 3M^2 = E^2 + n
  const double e = div_nr(n, E + sqrt_nr(E2 + n));
  const double iW = rcp_nr(fma(e, 1.0 / 3.0, E));
  r.e = e;
  r.v[0] = Mx * iW;
  r.v[1] = My * iW;
  r.v[2] = Mz * iW;
  return r;
}

template <class R>
__device__ __forceinline__ PrimV c2p(const R u[5], unsigned& fix) {
  return c2p((double)u[0], (double)u[1], (double)u[2], (double)u[3], fix);
}

// Physical flux along axis AX and twice its Lax-Friedrichs split (alpha = 1),
// f + u and f - u (FP64: products in fmas, one rounding fewer each):
// f = (M_AX, M_x v_AX + p d_{x,AX}, M_y v_AX + p d_{y,AX}, M_z v_AX + p d_{z,AX}, N v_AX).
template <class R, int AX>
__device__ __forceinline__ void split_flux(const R u[5], const PrimV& p, R Fp[5], R Fm[5]) {
  const R vd = (R)p.v[AX];
  const R pr = (R)(p.e * (1.0 / 3.0));
  Fp[0] = u[1 + AX] + u[0];
  Fm[0] = u[1 + AX] - u[0];
#pragma unroll
  for (int c = 1; c < 5; ++c) {
    if (sizeof(R) == 8 && c != 1 + AX) {
      Fp[c] = fma(u[c], vd, u[c]);
      Fm[c] = fma(u[c], vd, -u[c]);
    } else {
      const R f = sizeof(R) == 8 ? fma(u[c], vd, pr) : (c == 1 + AX ? u[c] * vd + pr : u[c] * vd);
      Fp[c] = f + u[c];
      Fm[c] = f - u[c];
    }
  }
}

// ---------------------------------------------------------------------------
// WENO7 value at x_{i+1/2} from the left, a0..a6 = a_{i-3}..a_{i+3}, from
// nested differences e (first), f (second) and g (third) of the values, each
// formed once per point and shared by every face of a line.
//
// Stencil k's cubic enters through three numbers: its slope
// s_k (with a 24th of the third derivative), curvature c_k and third derivative
// g_k at the centre of cell i, in cell widths:
//   s0 = e2 + f1/2 + g0/3, s1 = e2 + f2/2 - g1/6, s2 = e2 + f2/2 - g2/6,
//   s3 = e3 - f3/2 + g3/3,  c0 = f1 + g0, c1 = c2 = f2, c3 = f3 - g3.
// Its value at the face is q_k = a_i + s_k/2 + c_k/12 (p(1/2) = p(0) + s/2 +
// c/8 and p(0) = a_i - c/24), so a candidate costs one fma beside its
// indicator b_k = s_k^2 + 13/12 c_k^2 + 781/720 g_k^2 + eps (Jiang-Shu: the
// integral over the cell of the squared derivatives), and it holds values of
// its own stencil only: a stencil across a jump, whose weight vanishes, leaves
// no rounding of the jump behind.  f is kept scaled by sqrt(13/12), so c_k^2
// needs no factor; G = 781/780 g^2 + eps is shared.  Indicators vanish exactly
// on flat stencils.  WENO-Z (p = 2): w_k = 1 + (tau/b_k)^2, tau = |b0 - b3 +
// 3(b1 - b2)|; Jiang-Shu: w_k = 1/b_k^2; the result is sum w_k d_k q_k /
// sum w_k d_k, 35 d = (1, 12, 18, 4).
//
// Bound by VALU issue.
template <class R>
__device__ __forceinline__ R rcp_approx(R x);
template <>
__device__ __forceinline__ float rcp_approx<float>(float x) {
  return __builtin_amdgcn_rcpf(x);
}
template <>
__device__ __forceinline__ double rcp_approx<double>(double x) {
  return 1.0 / x;
}

// num / den: with the estimate r = (1 - d) / den, d = 1 - den r (~2^-23),
// num r (1 + d + d^2) leaves d^3, below the rounding.
__device__ __forceinline__ double quot(double num, double den) {
  const double r = __builtin_amdgcn_rcp(den);
  const double d = fma(-den, r, 1.0);
  const double q = num * r;
  return fma(q, fma(d, d, d), q);
}
__device__ __forceinline__ float quot(float num, float den) { return num * __builtin_amdgcn_rcpf(den); }

constexpr double kCurv = 1.0408329997330663;  // sqrt(13/12)

// One WENO7 face from its differences: ai = a_i, e2, e3; f1, f2, f3; g, G =
// four third differences and their indicator terms.
template <class R, int S>
__device__ __forceinline__ R weno7_face(R ai, R e2, R e3, R f1, R f2, R f3, const R* g, const R* G) {
  const R sm = fma(R(0.5 / kCurv), f2, e2);
  const R s0 = fma(R(1.0 / (3.0 * kCurv)), g[0], fma(R(0.5 / kCurv), f1, e2));
  const R s1 = fma(R(-1.0 / (6.0 * kCurv)), g[1], sm);
  const R s2 = fma(R(-1.0 / (6.0 * kCurv)), g[2], sm);
  const R s3 = fma(R(1.0 / (3.0 * kCurv)), g[3], fma(R(-0.5 / kCurv), f3, e3));
  const R c0 = f1 + g[0], c3 = f3 - g[3];
  // candidates as 12 sqrt(13/12) (q_k - a_i)
  const R r0 = fma(R(6.0 * kCurv), s0, c0), r1 = fma(R(6.0 * kCurv), s1, f2), r2 = fma(R(6.0 * kCurv), s2, f2),
          r3 = fma(R(6.0 * kCurv), s3, c3);
  if (S == kWenoLinear)
    return fma(R(1.0 / (35.0 * 12.0 * kCurv)), fma(R(4), r3, fma(R(18), r2, fma(R(12), r1, r0))), ai);
  const R b0 = fma(s0, s0, fma(c0, c0, G[0]));
  const R b1 = fma(s1, s1, fma(f2, f2, G[1]));
  const R b2 = fma(s2, s2, fma(f2, f2, G[2]));
  const R b3 = fma(s3, s3, fma(c3, c3, G[3]));
  const R tau = fma(R(3), b1 - b2, b0 - b3);  // enters squared
  R num, den;
  if (sizeof(R) == 8) {
    // Weights over a common denominator: with B_k = b_k^2 the WENO-Z weight
    // 1 + tau^2/B_k is proportional to (B_k + tau^2) prod_{j!=k} B_j, the
    // Jiang-Shu weight 1/B_k to prod_{j!=k} B_j; w0 and w1 share the factor
    // B_2 B_3, w2 and w3 the factor B_0 B_1.  One division.
    // (WENO-Z: (B_0 + tau^2) B_1 = B_0 B_1 + tau^2 B_1, and so on, one fma each.)
    const R B0 = b0 * b0, B1 = b1 * b1, B2 = b2 * b2, B3 = b3 * b3;
    const R P01 = B0 * B1, P23 = B2 * B3;
    R a0, a1, a2, a3;
    if (S == kWenoZ) {
      const R t2 = tau * tau;
      a0 = fma(t2, B1, P01);
      a1 = fma(t2, B0, P01);
      a2 = fma(t2, B3, P23);
      a3 = fma(t2, B2, P23);
    } else {
      a0 = B1;
      a1 = B0;
      a2 = B3;
      a3 = B2;
    }
    const R P = R(4) * P01;  // 18 and 4 as 4 times 4.5 and 1
    num = fma(P23, fma(R(12), a1 * r1, a0 * r0), P * fma(R(4.5), a2 * r2, a3 * r3));
    den = fma(P23, fma(R(12), a1, a0), P * fma(R(4.5), a2, a3));
  } else {
    const R i0 = rcp_approx<R>(b0), i1 = rcp_approx<R>(b1), i2 = rcp_approx<R>(b2), i3 = rcp_approx<R>(b3);
    R w0, w1, w2, w3;
    if (S == kWenoZ) {
      const R z0 = tau * i0, z1 = tau * i1, z2 = tau * i2, z3 = tau * i3;
      w0 = fma(z0, z0, R(1));
      w1 = fma(z1, z1, R(1));
      w2 = fma(z2, z2, R(1));
      w3 = fma(z3, z3, R(1));
    } else {
      w0 = i0 * i0;
      w1 = i1 * i1;
      w2 = i2 * i2;
      w3 = i3 * i3;
    }
    num = fma(R(4), w3 * r3, fma(R(18), w2 * r2, fma(R(12), w1 * r1, w0 * r0)));
    den = fma(R(4), w3, fma(R(18), w2, fma(R(12), w1, w0)));
  }
  return fma(R(1.0 / (12.0 * kCurv)), quot(num, den), ai);
}

// One WENO5 face (quadratics through three cells) in the same form: s0 = e1 +
// f0/2, s1 = e1 + f1/2, s2 = e2 - f2/2, c_k = f_k, q_k = a_i + s_k/2 + f_k/12,
// b_k = s_k^2 + F_k with F = 13/12 f^2 + eps, 10 d = (1, 6, 3), WENO-Z tau =
// |b0 - b2|.  e1, e2: the differences left and right of cell i.
template <class R, int S>
__device__ __forceinline__ R weno5_face(R ai, R e1, R e2, const R* f, const R* F) {
  const R s0 = fma(R(0.5), f[0], e1), s1 = fma(R(0.5), f[1], e1), s2 = fma(R(-0.5), f[2], e2);
  const R r0 = fma(R(6), s0, f[0]), r1 = fma(R(6), s1, f[1]), r2 = fma(R(6), s2, f[2]);  // 12 (q_k - a_i)
  if (S == kWeno5Linear) return fma(R(1.0 / 120.0), fma(R(3), r2, fma(R(6), r1, r0)), ai);
  const R b0 = fma(s0, s0, F[0]), b1 = fma(s1, s1, F[1]), b2 = fma(s2, s2, F[2]);
  const R tau = b0 - b2;  // enters squared
  R num, den;
  if (sizeof(R) == 8) {
    // common denominator, as in weno7_face
    const R B0 = b0 * b0, B1 = b1 * b1, B2 = b2 * b2;
    const R P01 = B0 * B1;
    R a0, a1, a2;
    if (S == kWeno5Z) {
      const R t2 = tau * tau;
      a0 = fma(t2, B1, P01);
      a1 = fma(t2, B0, P01);
      a2 = (B2 + t2) * P01;
    } else {
      a0 = B1;
      a1 = B0;
      a2 = P01;
    }
    num = fma(B2, fma(R(6), a1 * r1, a0 * r0), R(3) * (a2 * r2));
    den = fma(B2, fma(R(6), a1, a0), R(3) * a2);
  } else {
    const R i0 = rcp_approx<R>(b0), i1 = rcp_approx<R>(b1), i2 = rcp_approx<R>(b2);
    R w0, w1, w2;
    if (S == kWeno5Z) {
      const R z0 = tau * i0, z1 = tau * i1, z2 = tau * i2;
      w0 = fma(z0, z0, R(1));
      w1 = fma(z1, z1, R(1));
      w2 = fma(z2, z2, R(1));
    } else {
      w0 = i0 * i0;
      w1 = i1 * i1;
      w2 = i2 * i2;
    }
    num = fma(R(3), w2 * r2, fma(R(6), w1 * r1, w0 * r0));
    den = fma(R(3), w2, fma(R(6), w1, w0));
  }
  return fma(R(1.0 / 12.0), quot(num, den), ai);
}

// Both face values of a cell from one window (MUSTA-FORCE): `right` at i + 1/2
// as above, `left` at i - 1/2, p_k(-1/2) = a_i - s_k/2 + c_k/12 with the linear
// weights mirrored.  Differences, indicators and nonlinear weights serve both.
// s_1 and s_2 take the slope (e2 + e3)/2, so that a mirrored window gives the
// mirrored values bit for bit.
template <class R>
__device__ __forceinline__ void weno7_sides(R ai, R e2, R e3, R f1, R f2, R f3, const R* g, const R* G, R& right,
                                            R& left) {
  const R sm = R(0.5) * (e2 + e3);
  const R s0 = fma(R(1.0 / (3.0 * kCurv)), g[0], fma(R(0.5 / kCurv), f1, e2));
  const R s1 = fma(R(-1.0 / (6.0 * kCurv)), g[1], sm);
  const R s2 = fma(R(-1.0 / (6.0 * kCurv)), g[2], sm);
  const R s3 = fma(R(1.0 / (3.0 * kCurv)), g[3], fma(R(-0.5 / kCurv), f3, e3));
  const R c0 = f1 + g[0], c3 = f3 - g[3];
  const R b0 = fma(s0, s0, fma(c0, c0, G[0]));
  const R b1 = fma(s1, s1, fma(f2, f2, G[1]));
  const R b2 = fma(s2, s2, fma(f2, f2, G[2]));
  const R b3 = fma(s3, s3, fma(c3, c3, G[3]));
  const R tau = fma(R(3), b1 - b2, b0 - b3);  // enters squared
  const R kR = R(6.0 * kCurv), kL = R(-6.0 * kCurv);
  const R r0 = fma(kR, s0, c0), r1 = fma(kR, s1, f2), r2 = fma(kR, s2, f2), r3 = fma(kR, s3, c3);
  const R l0 = fma(kL, s0, c0), l1 = fma(kL, s1, f2), l2 = fma(kL, s2, f2), l3 = fma(kL, s3, c3);
  R numr, denr, numl, denl;
  if (sizeof(R) == 8) {
    const R B0 = b0 * b0, B1 = b1 * b1, B2 = b2 * b2, B3 = b3 * b3;
    const R P01 = B0 * B1, P23 = B2 * B3;
    const R t2 = tau * tau;
    const R a0 = fma(t2, B1, P01), a1 = fma(t2, B0, P01), a2 = fma(t2, B3, P23), a3 = fma(t2, B2, P23);
    const R P = R(4) * P01, Q = R(4) * P23;
    numr = fma(P23, fma(R(12), a1 * r1, a0 * r0), P * fma(R(4.5), a2 * r2, a3 * r3));
    denr = fma(P23, fma(R(12), a1, a0), P * fma(R(4.5), a2, a3));
    numl = fma(P01, fma(R(12), a2 * l2, a3 * l3), Q * fma(R(4.5), a1 * l1, a0 * l0));
    denl = fma(P01, fma(R(12), a2, a3), Q * fma(R(4.5), a1, a0));
  } else {
    const R z0 = tau * rcp_approx<R>(b0), z1 = tau * rcp_approx<R>(b1), z2 = tau * rcp_approx<R>(b2),
            z3 = tau * rcp_approx<R>(b3);
    const R w0 = fma(z0, z0, R(1)), w1 = fma(z1, z1, R(1)), w2 = fma(z2, z2, R(1)), w3 = fma(z3, z3, R(1));
    numr = fma(R(4), w3 * r3, fma(R(18), w2 * r2, fma(R(12), w1 * r1, w0 * r0)));
    denr = fma(R(4), w3, fma(R(18), w2, fma(R(12), w1, w0)));
    numl = fma(R(4), w0 * l0, fma(R(18), w1 * l1, fma(R(12), w2 * l2, w3 * l3)));
    denl = fma(R(4), w0, fma(R(18), w1, fma(R(12), w2, w3)));
  }
  right = fma(R(1.0 / (12.0 * kCurv)), quot(numr, denr), ai);
  left = fma(R(1.0 / (12.0 * kCurv)), quot(numl, denl), ai);
}

template <class R>
__device__ __forceinline__ void weno5_sides(R ai, R e1, R e2, const R* f, const R* F, R& right, R& left) {
  const R s0 = fma(R(0.5), f[0], e1), s1 = R(0.5) * (e1 + e2), s2 = fma(R(-0.5), f[2], e2);
  const R r0 = fma(R(6), s0, f[0]), r1 = fma(R(6), s1, f[1]), r2 = fma(R(6), s2, f[2]);
  const R l0 = fma(R(-6), s0, f[0]), l1 = fma(R(-6), s1, f[1]), l2 = fma(R(-6), s2, f[2]);
  const R b0 = fma(s0, s0, F[0]), b1 = fma(s1, s1, F[1]), b2 = fma(s2, s2, F[2]);
  const R tau = b0 - b2;  // enters squared
  R w0, w1, w2;
  if (sizeof(R) == 8) {  // over the common denominator, in a form that mirrors
    const R B0 = b0 * b0, B1 = b1 * b1, B2 = b2 * b2;
    const R t2 = tau * tau;
    w0 = (B0 + t2) * (B1 * B2);
    w1 = (B1 + t2) * (B0 * B2);
    w2 = (B2 + t2) * (B0 * B1);
  } else {
    const R z0 = tau * rcp_approx<R>(b0), z1 = tau * rcp_approx<R>(b1), z2 = tau * rcp_approx<R>(b2);
    w0 = fma(z0, z0, R(1));
    w1 = fma(z1, z1, R(1));
    w2 = fma(z2, z2, R(1));
  }
  right = fma(R(1.0 / 12.0), quot(fma(R(3), w2 * r2, fma(R(6), w1 * r1, w0 * r0)), fma(R(3), w2, fma(R(6), w1, w0))),
              ai);
  left = fma(R(1.0 / 12.0), quot(fma(R(3), w0 * l0, fma(R(6), w1 * l1, w2 * l2)), fma(R(3), w0, fma(R(6), w1, w2))),
             ai);
}

// L neighbouring faces of one line: put(k, R(a_k..a_{k+6})), k = 0..L-1, from
// the values get(0..L+5), taken in this order, value k + 6 before face k;
// schemes kWeno5* use the middle five of each window.
// Differences are formed as the faces reach them and every face by the same
// operations whatever L is, so that all splits of a line give the same bits.
// The scheduling barriers keep the live set at one face.  SIDES: put(k, right,
// left) with both face values of the windows' middle cells (WENO-Z).
template <class R, int S, int L, bool SIDES = false, class Get, class Put>
__device__ __forceinline__ void weno_line(Get get, R eps, Put put) {
  if constexpr (S >= kWeno5Z) {
    R a[L + 6], e[L + 4], f[L + 3], F[L + 3];  // a[0] and a[k + 6] are read, not used
#pragma unroll
    for (int k = 0; k < L; ++k) {
#pragma unroll
      for (int m = (k == 0 ? 0 : k + 6); m <= k + 6; ++m) {
        a[m] = get(m);
        if (m >= 3) e[m - 2] = a[m - 1] - a[m - 2];
        if (m >= 4) {
          f[m - 3] = e[m - 2] - e[m - 3];
          F[m - 3] = fma(R(13.0 / 12.0) * f[m - 3], f[m - 3], eps);
        }
      }
      if constexpr (SIDES) {
        R r, l;
        weno5_sides<R>(a[k + 3], e[k + 2], e[k + 3], f + k + 1, F + k + 1, r, l);
        put(k, r, l);
      } else {
        put(k, weno5_face<R, S>(a[k + 3], e[k + 2], e[k + 3], f + k + 1, F + k + 1));
      }
      if (L > 1) __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    R a[L + 6], e[L + 5], f[L + 4], g[L + 3], G[L + 3];
#pragma unroll
    for (int k = 0; k < L; ++k) {
#pragma unroll
      for (int m = (k == 0 ? 0 : k + 6); m <= k + 6; ++m) {
        a[m] = get(m);
        if (m >= 1) e[m - 1] = a[m] - a[m - 1];
        if (m >= 2) f[m - 2] = R(kCurv) * (e[m - 1] - e[m - 2]);
        if (m >= 3) {
          g[m - 3] = f[m - 2] - f[m - 3];
          G[m - 3] = fma(R(781.0 / 780.0) * g[m - 3], g[m - 3], eps);
        }
      }
      if constexpr (SIDES) {
        R r, l;
        weno7_sides<R>(a[k + 3], e[k + 2], e[k + 3], f[k + 1], f[k + 2], f[k + 3], g + k, G + k, r, l);
        put(k, r, l);
      } else {
        put(k, weno7_face<R, S>(a[k + 3], e[k + 2], e[k + 3], f[k + 1], f[k + 2], f[k + 3], g + k, G + k));
      }
      if (L > 1) __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <class R, int S>
__device__ __forceinline__ R weno7(R a0, R a1, R a2, R a3, R a4, R a5, R a6, R eps) {
  const R v[7] = {a0, a1, a2, a3, a4, a5, a6};
  R r;
  weno_line<R, S, 1>([&](int m) { return v[m]; }, eps, [&](int, R x) { r = x; });
  return r;
}

// Face flux from the 8-point window Fp/Fm[m] = split fluxes at i-3+m:
// F(i+1/2) = R_L(F+_{i-3..i+3}) + R_L(F-_{i+4..i-2}).
template <class R, int S>
__device__ __forceinline__ R face_flux(const R* fp, const R* fm, R eps) {
  return weno7<R, S>(fp[0], fp[1], fp[2], fp[3], fp[4], fp[5], fp[6], eps) +
         weno7<R, S>(fm[7], fm[6], fm[5], fm[4], fm[3], fm[2], fm[1], eps);
}

// ---------------------------------------------------------------------------
// MUSTA-FORCE flux (Toro's multi-stage centred flux), the alternative solver:
// kernels take it as the flag kMusta on the scheme template argument and then
// keep the conserved values (not the split fluxes) in their LDS tiles.  The
// face states uL, uR come from the WENO reconstruction of those values; on a
// local two-cell mesh with dt/dx = 0.9 (S_max = 1) each stage forms the FORCE
// flux, the mean of the Lax-Friedrichs flux (fL + fR)/2 - (uR - uL)/(2 * 0.9)
// and the flux of the Richtmyer state (uL + uR)/2 - 0.45 (fR - fL); the last
// stage's FORCE flux is the face flux, the stages before it move the local
// states: uL -= 0.9 (F - fL), uR -= 0.9 (fR - F).  Recovery in FP64 as
// everywhere; fixed-up recoveries are counted.
template <class R, int AX>
__device__ __forceinline__ void phys_flux(const R u[5], R f[5], unsigned& fix) {
  const PrimV p = c2p(u, fix);
  const R vd = (R)p.v[AX];
  const R pr = (R)(p.e * (1.0 / 3.0));
  f[0] = u[1 + AX];
  f[1] = (AX == 0) ? u[1] * vd + pr : u[1] * vd;
  f[2] = (AX == 1) ? u[2] * vd + pr : u[2] * vd;
  f[3] = (AX == 2) ? u[3] * vd + pr : u[3] * vd;
  f[4] = u[4] * vd;
}

template <class R, int AX>
__device__ __forceinline__ void musta_force(R uL[5], R uR[5], int k, R F[5], unsigned& fix) {
  for (int l = 1;; ++l) {
    R fL[5], fR[5], uM[5], fM[5];
    phys_flux<R, AX>(uL, fL, fix);
    phys_flux<R, AX>(uR, fR, fix);
#pragma unroll
    for (int c = 0; c < 5; ++c) uM[c] = R(0.5) * (uL[c] + uR[c]) - R(0.45) * (fR[c] - fL[c]);
    phys_flux<R, AX>(uM, fM, fix);
#pragma unroll
    for (int c = 0; c < 5; ++c) F[c] = R(0.5) * ((R(0.5) * (fL[c] + fR[c]) - R(0.5 / 0.9) * (uR[c] - uL[c])) + fM[c]);
    if (l >= k) return;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      uL[c] = uL[c] - R(0.9) * (F[c] - fL[c]);
      uR[c] = uR[c] - R(0.9) * (fR[c] - F[c]);
    }
  }
}

// One face with the MUSTA-FORCE flux: at(c, m) is component c of the
// conserved value at window point m = 0..7 (points i-3..i+4 for face i+1/2);
// uL the right value of the cell with window 0..6, uR the left value of the
// next one (WENO5: the middle five of each).
template <class R, int SC, int AX, class At>
__device__ __forceinline__ void musta_face(At at, R eps, int k, R F[5], unsigned& fix) {
  R uL[5], uR[5];
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    weno_line<R, SC, 1, true>([&](int m) { return at(c, m); }, eps, [&](int, R r, R) { uL[c] = r; });
    weno_line<R, SC, 1, true>([&](int m) { return at(c, m + 1); }, eps, [&](int, R, R l) { uR[c] = l; });
  }
  musta_force<R, AX>(uL, uR, k, F, fix);
}

// ---------------------------------------------------------------------------
// Positivity-preserving flux limiter (after Zhang and Shu).  Kernels take it
// as the flag kPP on the scheme template argument.
//
// A forward-Euler update u_i - sum_d (dt/dx_d)(F_{d,i+1/2} - F_{d,i-1/2}) is
// the mean over the axes, with weights (dt/dx_d) / sum(dt/dx), of the two
// half states of each axis
//   R = u_i - mu (F_{i+1/2} - f_i/2),   L = u_i + mu (F_{i-1/2} - f_i/2),
// mu = 2 dt sum_d 1/dx_d.  For the first-order flux F+(u_i) + F-(u_{i+1})
// they are (1 - mu/2) u_i + mu/2 (u_{i+1} - f_{i+1}) and (1 - mu/2) u_i +
// mu/2 (u_{i-1} + f_{i-1}): admissible for mu/2 <= 1, since u +- f(u) is for
// alpha = 1.  Each face flux F becomes theta F + (1 - theta) F_LF with the
// largest theta of the chord rule (below) that keeps E - |M| >= kPPEps and
// N >= kPPEps in the half state on each side of the face.  The split fluxes
// of the two cells give u = F+ - F-, f = F+ + F- and F_LF = F+_i + F-_{i+1}.
// FP64 in every form; a face that needs no limiting keeps its flux bit for bit.
// All of it is in the doubled units of split_flux (face values, half states
// and the bound: exact powers of two).
constexpr double kPPEps = 2.0 * 1e-13;

// Largest theta in [0, 1] with h(theta) >= 0 for h concave: 1 if h(1) >= 0,
// 0 if h(0) <= 0, else the root of the chord from (0, h0) to (1, h1), below
// which h stays above the chord and so non-negative.
__device__ __forceinline__ double pp_chord(double h0, double h1) {
  if (h1 >= 0.0) return 1.0;
  if (h0 <= 0.0) return 0.0;
  return h0 / (h0 - h1);
}

// E - |M| >= eps and N >= eps for E, |M|^2, N, without the square root.
__device__ __forceinline__ bool pp_inside(double E, double m2, double N) {
  const double a = E - kPPEps;
  return a >= 0.0 && a * a >= m2 && N >= kPPEps;
}

// E, |M|^2 and N of a half state next to a face (side 0: the low cell's
// u - mu (F - f/2), side 1: the high cell's u + mu (F - f/2)) for the face flux
// F_c = H_c, or (lf) the first-order flux F+_low + F-_high.
struct PPHalf {
  double e, m2, n;
};

template <class R, class Get>
__device__ __forceinline__ PPHalf pp_half(const R H[5], Get get, double mu, int side, bool lf) {
  PPHalf r = {0.0, 0.0, 0.0};
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    const double p = (double)get(c, 2 * side), m = (double)get(c, 2 * side + 1);
    const double F = lf ? (double)get(c, 0) + (double)get(c, 3) : (double)H[c];
    const double hs = side ? fma(mu, fma(-0.5, p + m, F), p - m) : fma(-mu, fma(-0.5, p + m, F), p - m);
    if (c == 0) r.e = hs;
    else if (c == 4) r.n = hs;
    else r.m2 = fma(hs, hs, r.m2);
  }
  return r;
}

// theta of one side from its half states with the first-order flux (s0) and
// with H (s1).
__device__ __forceinline__ double pp_side(const PPHalf& s0, const PPHalf& s1) {
  const double tq = pp_chord(s0.e - sqrt(s0.m2) - kPPEps, s1.e - sqrt(s1.m2) - kPPEps);
  const double tn = pp_chord(s0.n - kPPEps, s1.n - kPPEps);
  return fmin(tq, tn);
}

// H: the face's five fluxes (in/out).  get(c, k) returns component c of the
// split fluxes of the two cells next to the face: k = 0 F+ and 1 F- of the
// cell on the low side, 2 F+ and 3 F- of the cell on the high side.  Half
// states are folded into E, |M|^2 and N component by component and one side
// at a time, so that few values stay live.
template <class R, class Get>
__device__ __forceinline__ void pp_limit(R H[5], Get get, double mu) {
  bool inside;
  __asm__ __volatile__("" ::: "memory");
  {
    const PPHalf a1 = pp_half<R>(H, get, mu, 0, false);
    inside = pp_inside(a1.e, a1.m2, a1.n);
  }
  __asm__ __volatile__("" ::: "memory");
  if (inside) {
    const PPHalf b1 = pp_half<R>(H, get, mu, 1, false);
    inside = pp_inside(b1.e, b1.m2, b1.n);
  }
  if (inside) return;
  // rarely taken: each side again, with the first-order flux beside it.  The
  // empty asm with a memory clobber makes the compiler read the split fluxes
  // again here instead of keeping them in registers across the common path.
  __asm__ __volatile__("" ::: "memory");
  const double ta = pp_side(pp_half<R>(H, get, mu, 0, true), pp_half<R>(H, get, mu, 0, false));
  __asm__ __volatile__("" ::: "memory");
  const double tb = pp_side(pp_half<R>(H, get, mu, 1, true), pp_half<R>(H, get, mu, 1, false));
  const double th = fmin(ta, tb);
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    const double fl = (double)get(c, 0) + (double)get(c, 3);
    H[c] = (R)fma(th, (double)H[c], (1.0 - th) * fl);
  }
}

__device__ __forceinline__ void add_fixups(unsigned long long* ctr, unsigned fix) {
  if (fix) atomicAdd(ctr, (unsigned long long)fix);
}

// ---------------------------------------------------------------------------
// Jet helpers (Eq. 3, nearest grid point, cell centres, T(e)).
__device__ __forceinline__ int ngp_index(double x, int n, double dx) {
  const double x_lo = -0.5 * n * dx;
  const double u = (x - x_lo) / dx + 1e-9;
  const double f = floor(u);
  if (f < 0.0 || f >= (double)n) return -1;
  return (int)f;
}

__device__ __forceinline__ double temperature(double e, double g, double hc) {
  return sqrt(sqrt(30.0 * e * (hc * hc * hc) / (g * 3.14159265358979323846 * 3.14159265358979323846)));
}

__device__ __forceinline__ double energy_loss(const JetDev& jt, double T, double ell, double hc) {
  return jt.kappa_coll * jt.crcf * T * T / hc + jt.kappa_rad * jt.crcf * T * T * T * ell / (hc * hc);
}

__device__ __forceinline__ double cell_centre(int i, int n, double dx) { return (i - 0.5 * (n - 1)) * dx; }

}  // namespace hydro
