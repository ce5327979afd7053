// hydro_adjoint.hip -- reverse mode (vector-Jacobian products) of one SSP-RK3
// stage, of the jet source, of the anisotropy observable eps2 and of the
// primitive->conserved map of the initial state.
//
// For a stage  Y = a U^n + b (W + dt L(W)),  L = D + S, the reverse sweep
// needs G = (dL/dW)^T lambda_Y.  D's part goes face by face:
//   phi(face i+1/2) = (lambda_{i+1} - lambda_i)/dx       (face adjoint)
//   -> reverse of F(i+1/2) = R_L(F+_{i-3..i+3}) + R_L(F-_{i+4..i-2})
//   -> adjoints of the split fluxes at each point
//   -> (F+- = (f +- W)/2, f through the FP64 conserved->primitive recovery)
//   -> adjoint of W at the point; ghost points pass theirs to the cell they copy.
// A workgroup owns whole lines along the axis, so every face that touches a
// cell of a line is handled in the same workgroup: each lane reverses a run of
// neighbouring faces, and the runs' contributions to a point are added in a
// fixed order (deterministic, no atomics).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "hydro_device.hpp"
#include "hydro_internal.hpp"

namespace hydro {

// ---------------------------------------------------------------------------
// Conserved -> primitive with its derivatives (FP64).  Without fix-up:
// s = sqrt(4E^2 - 3M^2), e = s - E (evaluated as 3(E^2 - M^2)/(E + s)),
// de/dE = 4E/s - 1, de/dM_j = -3 M_j/s, v = M/(E + e/3).
struct PrimJ {
  double E;
  double e, v[3], iW;  // values; iW = 1/(E + p) = 1/(E + e/3)
  double eE, eM[3];    // de/dE, de/dM_j (at the possibly rescaled M)
  double Mc[3];        // M used in the recovery (rescaled when capped)
  double Mh[3];        // M/|M| (cap)
  double capf;         // (1 - 1e-10) E / |M| (cap)
  bool vac, cap;
};

__device__ __forceinline__ PrimJ c2p_jac(double E, double Mx, double My, double Mz) {
  PrimJ J;
  J.E = E;
  J.vac = false;
  J.cap = false;
  J.capf = 1.0;
  double M[3] = {Mx, My, Mz};
  if (E <= kEFloor) {
    J.vac = true;
    J.e = kEFloor;
    J.iW = 1.0 / (kEFloor + kEFloor / 3.0);
    for (int k = 0; k < 3; ++k) {
      J.v[k] = 0.0;
      J.eM[k] = 0.0;
      J.Mc[k] = 0.0;
      J.Mh[k] = 0.0;
    }
    J.eE = 0.0;
    return J;
  }
  double M2 = M[0] * M[0] + M[1] * M[1] + M[2] * M[2];
  if (M2 >= kVCap * kVCap * E * E) {
    J.cap = true;
    const double inrm = 1.0 / sqrt(M2);
    const double sc = kVCap * E * inrm;
    J.capf = sc;
    for (int k = 0; k < 3; ++k) {
      J.Mh[k] = M[k] * inrm;
      M[k] = M[k] * sc;
    }
    M2 = M[0] * M[0] + M[1] * M[1] + M[2] * M[2];
  }
  const double s = sqrt(4.0 * E * E - 3.0 * M2);
  const double is = 1.0 / s;
  const double e = 3.0 * (E * E - M2) / (E + s);
  J.e = e;
  J.iW = 1.0 / (E + e * (1.0 / 3.0));
  for (int k = 0; k < 3; ++k) {
    J.Mc[k] = M[k];
    J.v[k] = M[k] * J.iW;
    J.eM[k] = -3.0 * M[k] * is;
  }
  J.eE = 4.0 * E * is - 1.0;
  return J;
}

// Given adjoints eb of e and vb of v, the adjoints of (E, M):
// with Q = (vb . v)/(E + p) and kappa = eb - Q/3:
//   Eb = kappa de/dE - Q,  Mb_k = kappa de/dM_k + vb_k/(E + p),
// then through the velocity cap M' = c M, c = (1 - 1e-10) E/|M|.
__device__ __forceinline__ void c2p_vjp(const PrimJ& J, double eb, const double vb[3], double& Eb, double Mb[3]) {
  if (J.vac) {
    Eb = 0.0;
    Mb[0] = Mb[1] = Mb[2] = 0.0;
    return;
  }
  const double Q = (vb[0] * J.v[0] + vb[1] * J.v[1] + vb[2] * J.v[2]) * J.iW;
  const double kap = eb - Q * (1.0 / 3.0);
  double Ebp = kap * J.eE - Q;
  double Mbp[3];
  for (int k = 0; k < 3; ++k) Mbp[k] = kap * J.eM[k] + vb[k] * J.iW;
  if (!J.cap) {
    Eb = Ebp;
    for (int k = 0; k < 3; ++k) Mb[k] = Mbp[k];
    return;
  }
  const double dM = Mbp[0] * J.Mc[0] + Mbp[1] * J.Mc[1] + Mbp[2] * J.Mc[2];
  const double dh = Mbp[0] * J.Mh[0] + Mbp[1] * J.Mh[1] + Mbp[2] * J.Mh[2];
  Eb = Ebp + dM / J.E;
  for (int k = 0; k < 3; ++k) Mb[k] = J.capf * (Mbp[k] - J.Mh[k] * dh);
}

// Adjoint of the split fluxes at one point (axis AX): ap, am are the adjoints
// of F+ and F-; returns the adjoint of the conserved W of that point.
template <class R, int AX>
__device__ __forceinline__ void split_flux_vjp(const R u[5], const PrimJ& J, const double ap[5], const double am[5],
                                               double ub[5]) {
  double fb[5];
  for (int c = 0; c < 5; ++c) {
    fb[c] = 0.5 * (ap[c] + am[c]);
    ub[c] = 0.5 * (ap[c] - am[c]);
  }
  const double vd = (double)(R)J.v[AX];
  ub[1 + AX] += fb[0];
  double vbd = 0.0;
  for (int j = 0; j < 3; ++j) {
    ub[1 + j] += fb[1 + j] * vd;
    vbd += fb[1 + j] * (double)u[1 + j];
  }
  ub[4] += fb[4] * vd;
  vbd += fb[4] * (double)u[4];
  const double pb = fb[1 + AX];
  double vb[3] = {0.0, 0.0, 0.0};
  vb[AX] = vbd;
  double Eb, Mb[3];
  c2p_vjp(J, pb * (1.0 / 3.0), vb, Eb, Mb);
  ub[0] += Eb;
  for (int k = 0; k < 3; ++k) ub[1 + k] += Mb[k];
}

// The same for an admissible cell (no fix-up) whose e is known from the
// recovery: sqrt(4E^2 - 3M^2) = E + e, one division, and only v_AX has an
// adjoint, so few values stay live.
template <class R, int AX>
__device__ __forceinline__ void split_flux_vjp_known(const R u[5], double e, const double ap[5], const double am[5],
                                                     double ub[5]) {
  const double E = (double)u[0];
  const double s = E + e, W = E + e * (1.0 / 3.0);
  const double inv = rcp_nr(s * W);
  const double is = W * inv, iW = s * inv;
  const double v = (double)u[1 + AX] * iW, vd = (double)(R)v;
  double vbd = 0.5 * (ap[4] + am[4]) * (double)u[4];
  ub[4] = fma(0.5 * (ap[4] + am[4]), vd, 0.5 * (ap[4] - am[4]));
#pragma unroll
  for (int j = 1; j < 4; ++j) {
    const double fb = 0.5 * (ap[j] + am[j]);
    vbd = fma(fb, (double)u[j], vbd);
    ub[j] = fma(fb, vd, 0.5 * (ap[j] - am[j]));
  }
  const double Q = vbd * v * iW;
  const double kap = (0.5 * (ap[1 + AX] + am[1 + AX]) - Q) * (1.0 / 3.0);
  ub[0] = 0.5 * (ap[0] - am[0]) + (kap * (4.0 * E * is - 1.0) - Q);
  ub[1 + AX] = ub[1 + AX] + fma(vbd, iW, 0.5 * (ap[0] + am[0]));
  const double km = -3.0 * kap * is;
#pragma unroll
  for (int j = 1; j < 4; ++j) ub[j] = fma(km, (double)u[j], ub[j]);
}

// ---------------------------------------------------------------------------
// Reverse mode of weno7_face: adds phi dR/d(e, f, g) of one face to the
// adjoints ea2, ea3 of the first, fa1..fa3 of the (scaled) second and ga of
// the third differences (the a_i term, phi itself, is the caller's).  Forward
// arithmetic as there, weights by reciprocals: w_k = 1 + z_k^2, z_k = tau/b_k
// (Jiang-Shu: 1/b_k^2), R = a_i + num / (12 sqrt(13/12) den), num = sum d_k w_k
// r_k, den = sum d_k w_k.  ea3, fa3 and ga[3] are first touched by this face.
template <class R, int S>
__device__ __forceinline__ void weno7_face_vjp(R phi, R e2, R e3, R f1, R f2, R f3, const R* g, const R* G, R& ea2,
                                               R& ea3, R& fa1, R& fa2, R& fa3, R* ga) {
  const R sm = fma(R(0.5 / kCurv), f2, e2);
  const R s0 = fma(R(1.0 / (3.0 * kCurv)), g[0], fma(R(0.5 / kCurv), f1, e2));
  const R s1 = fma(R(-1.0 / (6.0 * kCurv)), g[1], sm);
  const R s2 = fma(R(-1.0 / (6.0 * kCurv)), g[2], sm);
  const R s3 = fma(R(1.0 / (3.0 * kCurv)), g[3], fma(R(-0.5 / kCurv), f3, e3));
  const R c0 = f1 + g[0], c3 = f3 - g[3];
  R rb0, rb1, rb2, rb3;                             // adjoints of the candidates r_k
  R bb0 = R(0), bb1 = R(0), bb2 = R(0), bb3 = R(0);  // twice those of the indicators
  if (S == kWenoLinear) {
    const R pin = R(1.0 / (35.0 * 12.0 * kCurv)) * phi;
    rb0 = pin;
    rb1 = R(12) * pin;
    rb2 = R(18) * pin;
    rb3 = R(4) * pin;
  } else {
    const R r0 = fma(R(6.0 * kCurv), s0, c0), r1 = fma(R(6.0 * kCurv), s1, f2), r2 = fma(R(6.0 * kCurv), s2, f2),
            r3 = fma(R(6.0 * kCurv), s3, c3);
    const R b0 = fma(s0, s0, fma(c0, c0, G[0]));
    const R b1 = fma(s1, s1, fma(f2, f2, G[1]));
    const R b2 = fma(s2, s2, fma(f2, f2, G[2]));
    const R b3 = fma(s3, s3, fma(c3, c3, G[3]));
    R i0, i1, i2, i3;
    if (sizeof(R) == 8) {
      const R p01 = b0 * b1, p23 = b2 * b3;
      const R inv = (R)rcp_nr((double)(p01 * p23));
      const R u23 = inv * p23, u01 = inv * p01;
      i0 = u23 * b1;
      i1 = u23 * b0;
      i2 = u01 * b3;
      i3 = u01 * b2;
    } else {
      i0 = rcp_approx<R>(b0);
      i1 = rcp_approx<R>(b1);
      i2 = rcp_approx<R>(b2);
      i3 = rcp_approx<R>(b3);
    }
    const R tau = fma(R(3), b1 - b2, b0 - b3);
    const R z0 = tau * i0, z1 = tau * i1, z2 = tau * i2, z3 = tau * i3;
    const R w0 = S == kWenoZ ? fma(z0, z0, R(1)) : i0 * i0;
    const R w1 = R(12) * (S == kWenoZ ? fma(z1, z1, R(1)) : i1 * i1);
    const R w2 = R(18) * (S == kWenoZ ? fma(z2, z2, R(1)) : i2 * i2);
    const R w3 = R(4) * (S == kWenoZ ? fma(z3, z3, R(1)) : i3 * i3);
    const R den = (w0 + w1) + (w2 + w3);
    const R num = fma(w3, r3, fma(w2, r2, fma(w1, r1, w0 * r0)));
    const R invd = sizeof(R) == 8 ? (R)rcp_nr((double)den) : rcp_approx<R>(den);
    const R corr = num * invd;
    const R pin = R(1.0 / (12.0 * kCurv)) * (phi * invd);
    rb0 = pin * w0;
    rb1 = pin * w1;
    rb2 = pin * w2;
    rb3 = pin * w3;
    // 4 times the adjoints of w_k (without their d_k in w1..w3 above)
    const R v0 = (R(4) * pin) * (r0 - corr), v1 = (R(48) * pin) * (r1 - corr), v2 = (R(72) * pin) * (r2 - corr),
            v3 = (R(16) * pin) * (r3 - corr);
    if (S == kWenoZ) {
      const R t0 = v0 * (z0 * i0), t1 = v1 * (z1 * i1), t2 = v2 * (z2 * i2), t3 = v3 * (z3 * i3);
      const R t = (t0 + t1) + (t2 + t3);  // twice the adjoint of tau
      bb0 = fma(-t0, z0, t);
      bb1 = fma(-t1, z1, R(3) * t);
      bb2 = fma(-t2, z2, R(-3) * t);
      bb3 = fma(-t3, z3, -t);
    } else {
      bb0 = -v0 * ((i0 * i0) * i0);
      bb1 = -v1 * ((i1 * i1) * i1);
      bb2 = -v2 * ((i2 * i2) * i2);
      bb3 = -v3 * ((i3 * i3) * i3);
    }
  }
  const R sb0 = fma(s0, bb0, R(6.0 * kCurv) * rb0), sb1 = fma(s1, bb1, R(6.0 * kCurv) * rb1),
          sb2 = fma(s2, bb2, R(6.0 * kCurv) * rb2), sb3 = fma(s3, bb3, R(6.0 * kCurv) * rb3);
  const R cb0 = fma(c0, bb0, rb0), cb3 = fma(c3, bb3, rb3);
  const R cbm = fma(f2, bb1 + bb2, rb1 + rb2), sbm = sb1 + sb2;
  constexpr double kG = 781.0 / 780.0;
  ga[0] = fma(R(1.0 / (3.0 * kCurv)), sb0, fma(R(kG) * g[0], bb0, ga[0] + cb0));
  ga[1] = fma(R(-1.0 / (6.0 * kCurv)), sb1, fma(R(kG) * g[1], bb1, ga[1]));
  ga[2] = fma(R(-1.0 / (6.0 * kCurv)), sb2, fma(R(kG) * g[2], bb2, ga[2]));
  ga[3] = fma(R(1.0 / (3.0 * kCurv)), sb3, fma(R(kG) * g[3], bb3, -cb3));
  fa1 = fma(R(0.5 / kCurv), sb0, fa1 + cb0);
  fa2 = fma(R(0.5 / kCurv), sbm, fa2 + cbm);
  fa3 = fma(R(-0.5 / kCurv), sb3, cb3);
  ea2 = ea2 + (sb0 + sbm);
  ea3 = sb3;
}

// L neighbouring faces of one line in reverse: get(m), m = 0..L+5 in order
// (value k + 6 before face k), phi(k) the adjoint of face k, put(j, adjoint of
// value j by these faces), j = 0..L+5 in order.  A difference's adjoint is
// complete once the last face that uses it is done, and passes on to the two
// differences (values) it was formed from: seven operations a point in the
// place of a face's seven partials.
template <class R, int S, int L, class Get, class Phi, class Put>
__device__ __forceinline__ void weno_line_vjp(Get get, Phi phi, R eps, Put put) {
  R a[L + 6], e[L + 5], f[L + 4], g[L + 3], G[L + 3];
  R aa[L + 6], ea[L + 5], fa[L + 4], ga[L + 3];
#pragma unroll
  for (int m = 0; m < L + 6; ++m) aa[m] = R(0);
#pragma unroll
  for (int m = 0; m < L + 5; ++m) ea[m] = R(0);
#pragma unroll
  for (int m = 0; m < L + 4; ++m) fa[m] = R(0);
#pragma unroll
  for (int m = 0; m < L + 3; ++m) ga[m] = R(0);
  auto pass = [&](int j) {  // values and differences j are complete
    if (j < L + 3) {
      fa[j + 1] = fa[j + 1] + ga[j];
      fa[j] = fa[j] - ga[j];
    }
    if (j < L + 4) {
      const R p = R(kCurv) * fa[j];
      ea[j + 1] = ea[j + 1] + p;
      ea[j] = ea[j] - p;
    }
    if (j < L + 5) {
      aa[j + 1] = aa[j + 1] + ea[j];
      aa[j] = aa[j] - ea[j];
    }
    put(j, aa[j]);
  };
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
    const R ph = phi(k);
    weno7_face_vjp<R, S>(ph, e[k + 2], e[k + 3], f[k + 1], f[k + 2], f[k + 3], g + k, G + k, ea[k + 2], ea[k + 3],
                         fa[k + 1], fa[k + 2], fa[k + 3], ga + k);
    aa[k + 3] = aa[k + 3] + ph;
    pass(k);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int j = L; j < L + 6; ++j) pass(j);
}

// ---------------------------------------------------------------------------
// Line adjoint along axis AX: G (first: =, else +=) receives (dD_AX/dW)^T mu
// of whole lines (faces -1/2..n-3/2; periodic: face -1/2 is also the right face
// of cell n-1; outflow: also face n-1/2).  A workgroup owns NL neighbouring
// lines, so that the loads of y and z lines fetch runs of consecutive x.
//   (1) The cells' split fluxes go to LDS (area 2 field + split, [slot][line];
//       F- in reverse slot order), and so do the faces' adjoints phi.
//   (2) Each wave takes whole areas: it copies the ghost slots and marches; its
//       lanes are the lines by 64 / NL runs of L faces, turn after turn along
//       the line.  The adjoint of a run's value takes the value's place, L - 7
//       faces late (the run before it reads value L + j at face L + j - 7), and
//       the six values beyond the run are added to those of the run that starts
//       there, for a turn's last run in the next turn.  The ghosts' adjoints
//       are added to their cells'.  Lanes execute their LDS operations in
//       order, and no other wave uses the area.
//   (3) Each cell reverses the splits through its recovery (recomputed) and
//       finishes G or, on the last axis, the reverse RK combine.
//
// Bound by VALU issue (FP64) and by its serial chains at five waves a SIMD
// (FP32).  One lane per face, its seven partials of a split gathered through
// LDS (two barriers a field, one or two lines a workgroup, face n-1/2 in a
// launch of its own), took 194 operations a reconstruction, this 150.  us an
// axis (x, y, z) before and after, those launches included: 60x52x66 FP64 41,
// 39, 53 / 27, 23, 29; 128^3 FP32 119, 113, 117 / 121, 102, 99.
__device__ __forceinline__ long long line_base(int AX, long long L, const Grid& g, long long& stride) {
  const int nx = g.n[0], ny = g.n[1];
  if (AX == 0) {
    stride = 1;
    return L * nx;
  }
  if (AX == 1) {
    stride = nx;
    const long long x = L % nx, z = L / nx;
    return z * (long long)nx * ny + x;
  }
  stride = (long long)nx * ny;
  const long long x = L % nx, y = L / nx;
  return y * nx + x;
}

// Block order: consecutive groups of lines (neighbours in memory for the y/z
// axes) go to the same XCD (blocks are dealt round-robin over the 8 XCDs).
__device__ __forceinline__ long long xcd_group(long long groups) {
  const long long per = (groups + 7) / 8;
  return (long long)(blockIdx.x % 8) * per + blockIdx.x / 8;
}

// SEG: a workgroup owns a segment of its lines, cells c0..c1-1, and reverses
// the faces c0-3..c1+3 (face f lies between cells f-1 and f) that touch them,
// from the points seven cells further out on each side.
template <class R, int S, int AX, int L, int NL, bool SEG>
__global__ void __launch_bounds__(line_adj_block((int)sizeof(R)), sizeof(R) == 8 ? 4 : 5) k_line_adj(AdjArgs<R> a) {
  constexpr int kBlock = line_adj_block((int)sizeof(R));
  extern __shared__ __align__(16) unsigned char smem_raw[];
  R* s = reinterpret_cast<R*>(smem_raw);
  constexpr int nl = NL, rpt = 64 / NL;  // lines, runs of a wave's turn
  constexpr int pitch = line_adj_pitch(AX, NL);
  const int n = a.g.n[AX];
  const int bc = a.g.bc[AX];
  const long long nc = a.g.nc;
  const long long nlines = AX == 0 ? (long long)a.g.n[1] * a.g.n[2]
                                   : (AX == 1 ? (long long)a.g.n[0] * a.g.n[2] : (long long)a.g.n[0] * a.g.n[1]);
  const int segs = SEG ? (n + a.seglen - 1) / a.seglen : 1;
  const long long item = xcd_group((nlines + nl - 1) / nl * segs);
  const long long grp = SEG ? item / segs : item;
  const long long line0 = grp * nl;
  if (line0 >= nlines) return;  // whole workgroup
  // own cells c0..c1-1; faces f0..f0+nf-1; slot j holds position f0 - 4 + j
  const int c0 = SEG ? (int)(item - grp * segs) * a.seglen : 0, c1 = SEG ? min(n, c0 + a.seglen) : n;
  const int f0 = SEG ? (bc ? c0 - 3 : max(0, c0 - 3)) : 0;
  const int nf = SEG ? (bc ? c1 + 3 : min(n, c1 + 3)) - f0 + 1 : n + (bc ? 0 : 1);
  // cells that the points f0 - 4..f0 + nf + 2 are, those beyond outflow ends not
  const int x0 = SEG ? (bc ? f0 - 4 : max(0, f0 - 4)) : 0, x1 = SEG ? (bc ? f0 + nf + 3 : min(n, f0 + nf + 3)) : n;
  auto wrap = [&](int x) { return SEG && bc ? (x < 0 ? x + n : (x >= n ? x - n : x)) : x; };
  const int area = line_adj_slots(nf, L) * pitch;
  const int fields = a.skip_n ? 4 : 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q = threadIdx.x & 63;
  unsigned fix = 0;

  // Line, first point and step of a lane in the point phases: y and z: lines
  // fastest; x: 64 neighbouring cells of a row a wave, the waves dealt over the rows.
  constexpr int kWaves = kBlock / 64, kRows = kWaves < nl ? kWaves : nl;  // x: rows under way at once
  const int l0 = AX == 0 ? w % kRows : (int)threadIdx.x & (nl - 1), lstep = AX == 0 ? kRows : nl;
  const int p0 = AX == 0 ? w / kRows * 64 + q : (int)threadIdx.x / nl;
  constexpr int pstep = AX == 0 ? kWaves / kRows * 64 : kBlock / nl;
  R* const hold = s + 2 * fields * area;            // [area][6][line], the last run of a turn's values beyond it
  R* const phi = hold + 2 * fields * 6 * nl;        // [field][face + pad][pitch], zeros beyond the faces
  const int pad = (nf + L - 1) / L * L - nf, prows = line_adj_phi_rows(nf, L);
  const int parea = prows * pitch;
  // slot j holds padded position j - 4; F- slot j at nf + 6 - j (slot nf + 7
  // belongs to no face)
#pragma unroll 1
  for (int l = l0; l < nl && line0 + l < nlines; l += lstep) {
    long long stride;
    const long long base = line_base(AX, line0 + l, a.g, stride);
#pragma unroll 1
    for (int x = x0 + p0; x < x1; x += pstep) {
      long long cell = base + wrap(x) * stride;
      __asm__ __volatile__("" : "+v"(cell));  // as in (3)
      R u[5], Fp[5], Fm[5];
      load5(a.W, nc, cell, u);
      const PrimV pv = c2p(u, fix);
      split_flux<R, AX>(u, pv, Fp, Fm);
      R* sp = s + (x - f0 + 4) * pitch + l;
      R* sm = s + area + (nf + 2 - x + f0) * pitch + l;
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        if (c < fields) {
          sp[2 * c * area] = Fp[c];
          sm[2 * c * area] = Fm[c];
        }
      }
    }
    // the last run's values past the line: any finite ones (phi is 0 there)
    for (int j = nf + 7 + p0; j < line_adj_slots(nf, L); j += pstep)
      for (int ar = 0; ar < 2 * fields; ++ar) s[ar * area + j * pitch + l] = R(0);
    // face f = 0.. is f - 1/2: phi = (mu(f) - mu(f - 1)) / dx, outflow: nothing
    // beyond the ends
#pragma unroll 1
    for (int k = p0; k < prows; k += pstep) {
      const bool face = k >= pad && k - pad < nf;
      const int f = SEG ? wrap(f0 + k - pad) : k - pad;
      const int fl = f == 0 ? (bc ? n - 1 : -1) : f - 1;
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        if (c < fields) {
          const R* mu = a.mu + c * nc + base;
          const R left = face && fl >= 0 ? mu[fl * stride] : R(0);
          const R right = face && f < n ? mu[f * stride] : R(0);
          phi[c * parea + k * pitch + l] = (right - left) * a.inv_d;
        }
      }
    }
  }
  __syncthreads();

  {
    const int runs = (nf + L - 1) / L;
    for (int ar = w; ar < 2 * fields; ar += kBlock / 64) {
      // the empty asm keeps the lane's addresses from being formed ahead of
      // the loops and held in registers through the march
      int qa = q;
      __asm__ __volatile__("" : "+v"(qa));
      const int l = qa & (nl - 1);
      const bool in = line0 + l < nlines;
      R* const hd = hold + ar * 6 * nl + l;
      R* const line = s + ar * area + l;
      auto at = [&](int slot) { return ((ar & 1) ? nf + 6 - slot : slot) * pitch; };
      // ghost slots: copies of their cells
      const int h = qa / nl;
      if constexpr (SEG) {  // points beyond outflow ends
        const int left = bc ? 0 : max(0, 4 - f0), end = n - f0 + 4, right = bc ? 0 : max(0, nf + 7 - end);
        if (h < left) line[at(h)] = line[at(left)];
        if (h >= 4 && h - 4 < right) line[at(end + h - 4)] = line[at(end - 1)];
      } else {
        const int gj = h < 4 ? h : n + h;
        if (h < 8 && gj <= nf + 6) line[at(gj)] = line[at(map_idx(gj - 4, n, bc) + 4)];
      }
      __asm__ __volatile__("" ::: "memory");
      for (int r0 = 0; r0 < runs; r0 += rpt) {
        int qr = qa;
        __asm__ __volatile__("" : "+v"(qr));
        const int r = r0 + qr / nl;
        const bool act = in && r < runs;
        R* const t = s + ar * area + r * L * pitch + l;
        R beyond[6];
        if (act) {
          // faces r L.. of the area's order: F- runs from face nf - 1 down
          const int fr = (ar & 1) ? nf - 1 - r * L : r * L;
          const R* ph = phi + (ar >> 1) * parea + (fr + pad) * pitch + l;
          const int pstep1 = (ar & 1) ? -pitch : pitch;
          R next = t[0];
          R late[L + 6];
          weno_line_vjp<R, S, L>(
              [&](int m) {
                const R v = next;
                if (m + 1 < L + 6) next = t[(m + 1) * pitch];
                __asm__ __volatile__("" ::: "memory");
                return v;
              },
              [&](int k) {
                return ph[k * pstep1];
              },
              a.eps,
              [&](int j, R v) {
                constexpr int kLate = L > 7 ? L - 7 : 0;
                late[j] = v;
                if (j >= L) beyond[j - L] = v;
                if (j >= kLate && j - kLate < L) t[(j - kLate) * pitch] = late[j - kLate];
                __asm__ __volatile__("" ::: "memory");
              });
        }
        __builtin_amdgcn_wave_barrier();
        __asm__ __volatile__("" ::: "memory");
        if (act) {
          const bool group0 = r0 > 0 && r == r0, end = r == runs - 1, last = r == r0 + rpt - 1 && !end;
#pragma unroll
          for (int m = 0; m < 6; ++m) {
            if (group0) t[m * pitch] = t[m * pitch] + hd[m * nl];
          }
          __asm__ __volatile__("" ::: "memory");
#pragma unroll
          for (int m = 0; m < 6; ++m) {
            R* d = t + (L + m) * pitch;
            if (last) hd[m * nl] = beyond[m];
            else *d = end ? beyond[m] : *d + beyond[m];  // past the last run no run starts
          }
        }
        __builtin_amdgcn_wave_barrier();
        __asm__ __volatile__("" ::: "memory");
      }
      // ghosts' adjoints onto the cells they copy, in slot order (slot nf + 6
      // in the area's order belongs to no face); several onto one cell unless
      // the axis is periodic with at least 8 cells
      int qg = q;
      __asm__ __volatile__("" : "+v"(qg));
      R* const gl = s + ar * area + (qg & (nl - 1));
      const int gh = qg / nl, gs = gh < 4 ? gh : n + gh;
      if (gh == 0) gl[(nf + 6) * pitch] = R(0);
      __asm__ __volatile__("" ::: "memory");
      if constexpr (SEG) {
        if (!bc && gh < 2) {
          const int left = max(0, 4 - f0), end = n - f0 + 4, right = max(0, nf + 7 - end);
          const int j0 = gh == 0 ? 0 : end, count = gh == 0 ? left : right;
          R* d = gl + at(gh == 0 ? left : end - 1);
          for (int k = 0; k < count; ++k) *d = *d + gl[at(j0 + k)];
        }
      } else if (bc && n >= 8) {
        if (gh < 8 && gs <= nf + 6) {
          R* d = gl + at(map_idx(gs - 4, n, bc) + 4);
          *d = *d + gl[at(gs)];
        }
      } else if (!bc && n >= 2) {
        if (gh < 2) {
          R* d = gl + at(gh == 0 ? 4 : n + 3);
          const int j0 = gh == 0 ? 0 : n + 4;
          *d = (((*d + gl[at(j0)]) + gl[at(j0 + 1)]) + gl[at(j0 + 2)]) + gl[at(j0 + 3)];
        }
      } else if (gh == 0) {
        for (int k = 0; k < 8; ++k) {
          const int j = k < 4 ? k : n + k;
          if (j <= nf + 6) {
            R* d = gl + at(map_idx(j - 4, n, bc) + 4);
            *d = *d + gl[at(j)];
          }
        }
      }
    }
  }
  __syncthreads();

  // (3) cells without a fix-up, then those with one: the general Jacobian's
  // registers stay out of the first loop
  bool any = false;
  auto cells = [&](auto slow) {
    constexpr bool SLOW = decltype(slow)::value;
#pragma unroll 1
    for (int l = l0; l < nl && line0 + l < nlines; l += lstep) {
      long long stride;
      const long long base = line_base(AX, line0 + l, a.g, stride);
#pragma unroll 1
      for (int x = c0 + p0; x < c1; x += pstep) {
        long long cell = base + x * stride;
        // opaque: the loop keeps one index, not a pointer per array and field
        __asm__ __volatile__("" : "+v"(cell));
        R u[5];
        load5(a.W, nc, cell, u);
        // split-flux adjoint -> adjoint of W at the cell
        unsigned f1 = 0;
        const PrimV pv = c2p(u, f1);
        any = any || f1 != 0;
        if (SLOW != (f1 != 0)) continue;
        const R* sp = s + (x - f0 + 4) * pitch + l;
        const R* sm = s + area + (nf + 2 - x + f0) * pitch + l;
        double dp[5], dm[5], ub[5];
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          dp[c] = c < fields ? (double)sp[2 * c * area] : 0.0;
          dm[c] = c < fields ? (double)sm[2 * c * area] : 0.0;
        }
        if constexpr (SLOW)
          split_flux_vjp<R, AX>(u, c2p_jac((double)u[0], (double)u[1], (double)u[2], (double)u[3]), dp, dm, ub);
        else
          split_flux_vjp_known<R, AX>(u, pv.e, dp, dm, ub);
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          __asm__ __volatile__("" ::: "memory");  // one field's loads at a time: fewer registers
          const long long k = c * nc + cell;
          const R gv = a.first ? (R)ub[c] : a.G[k] + (R)ub[c];
          if (a.stage == 0) {
            a.G[k] = gv;
          } else {
            const R my = (c == 4 && a.skip_n) ? R(0) : a.mu[k];
            const R t = fma(a.dt, gv, my);
            if (a.stage == 3) {
              a.lW[k] = R(2.0 / 3.0) * t;
              a.acc[k] = R(1.0 / 3.0) * my;
            } else if (a.stage == 2) {
              a.lW[k] = R(0.25) * t;
              a.acc[k] = fma(R(0.75), my, a.acc[k]);
            } else {
              a.lW[k] = a.acc[k] + t;
            }
          }
        }
      }
    }
  };
  cells(std::false_type{});
  if (any) cells(std::true_type{});
  add_fixups(a.fixups, fix);
}

// ---------------------------------------------------------------------------
// Jet source adjoint: G += (dS/dW)^T mu at the deposit cells, and
// grad[j] += bdt * (dS/dtheta)^T mu for theta = (kappa_rad, kappa_coll, x0, y0, z0).
template <class R>
__global__ void __launch_bounds__(512) k_jet_adj(JetAdjArgs a) {
  const R* W = static_cast<const R*>(a.W);
  const R* mu = static_cast<const R*>(a.mu);
  R* G = static_cast<R*>(a.G);
  const long long nc = a.g.nc;
  const double dV = a.g.dx[0] * a.g.dx[1] * a.g.dx[2];
  const double hc = a.hbarc;
  __shared__ double red[8][12];  // per-wave sums
  __shared__ double tot[12];     // the workgroup's sums
  __shared__ double wraw[3][7], wax[3][7], dwax[3][7];
  __shared__ int ctr_s[3];
  __shared__ int inside_s;
  const int t = threadIdx.x;
  for (int j = 0; j < a.njet; ++j) {
    const JetDev jt = a.s->jets[j];
    const bool chi = a.Ehist[j] > 0.0;
    const double ell = a.t - jt.t_start;
    // footprint weights: lane t < 21 takes axis t / 7, offset t % 7 (the
    // sums over the seven offsets in offset order, as one lane would)
    const int wd = t / 7, wm = t % 7;
    // the lane's axis by selects (an index by wd would put the structs in
    // scratch memory)
    auto pick = [wd](double v0, double v1, double v2) { return wd == 0 ? v0 : (wd == 1 ? v1 : v2); };
    const int wn = wd == 0 ? a.g.n[0] : (wd == 1 ? a.g.n[1] : a.g.n[2]);
    const double wdx = pick(a.g.dx[0], a.g.dx[1], a.g.dx[2]);
    double wx = 0.0, wdel = 0.0, wsig2 = 1.0;
    if (t < 21) {
      wx = pick(jt.x0[0], jt.x0[1], jt.x0[2]) + pick(jt.dir[0], jt.dir[1], jt.dir[2]) * ell;
      const int c = ngp_index(wx, wn, wdx);
      if (wm == 0) ctr_s[wd] = c;
      wsig2 = wdx * wdx;
      wdel = cell_centre(c - 3 + wm, wn, wdx) - wx;
      if (a.deposit == 1) wraw[wd][wm] = exp(-(wdel * wdel) / (2.0 * wsig2));
    }
    __syncthreads();
    if (t == 0) inside_s = (chi && ell >= 0.0 && ctr_s[0] >= 0 && ctr_s[1] >= 0 && ctr_s[2] >= 0) ? 1 : 0;
    if (a.deposit == 1) {
      if (t < 21) {
        double sum = 0.0;
        for (int m = 0; m < 7; ++m) sum = sum + wraw[wd][m];
        wax[wd][wm] = wraw[wd][wm] / sum;
      }
      __syncthreads();
      if (t < 21) {
        double dsum = 0.0;
        for (int m = 0; m < 7; ++m) {
          const double del = cell_centre(ctr_s[wd] - 3 + m, wn, wdx) - wx;
          dsum += wax[wd][m] * del / wsig2;
        }
        dwax[wd][wm] = wax[wd][wm] * (wdel / wsig2 - dsum);  // d w_m / d x
      }
    }
    __syncthreads();
    if (inside_s) {
      if (a.deposit == 0) {
        if (t == 0) {
          const long long cell = ((long long)ctr_s[2] * a.g.n[1] + ctr_s[1]) * a.g.n[0] + ctr_s[0];
          R gv[4];  // the cell's G, read with its state
          for (int k = 0; k < 4; ++k) gv[k] = G[k * nc + cell];
          const PrimJ J = c2p_jac((double)W[cell], (double)W[nc + cell], (double)W[2 * nc + cell],
                                  (double)W[3 * nc + cell]);
          const double T = temperature(J.e, a.eos_dof, hc);
          const double sig = ((double)mu[cell] + jt.dir[0] * (double)mu[nc + cell] +
                              jt.dir[1] * (double)mu[2 * nc + cell] + jt.dir[2] * (double)mu[3 * nc + cell]) / dV;
          const double dPdT = 2.0 * jt.kappa_coll * jt.crcf * T / hc + 3.0 * jt.kappa_rad * jt.crcf * T * T * ell / (hc * hc);
          const double eb = sig * dPdT * T / (4.0 * J.e);
          const double vb[3] = {0.0, 0.0, 0.0};
          double Eb, Mb[3];
          c2p_vjp(J, eb, vb, Eb, Mb);
          G[cell] = gv[0] + (R)Eb;
          for (int k = 0; k < 3; ++k) G[(1 + k) * nc + cell] = gv[1 + k] + (R)Mb[k];
          double* gr = a.grad + 5 * j;
          gr[0] += a.bdt * sig * jt.crcf * T * T * T * ell / (hc * hc);
          gr[1] += a.bdt * sig * jt.crcf * T * T / hc;
        }
      } else {
        // 7^3 footprint, thread t < 343
        double w = 0.0, T = 0.0, sig = 0.0, dw[3] = {0.0, 0.0, 0.0};
        long long cell = -1;
        PrimJ J;
        R gv[4];  // the cell's G, read with its state
        if (t < 343) {
          const int mi = t % 7, mj = (t / 7) % 7, mk = t / 49;
          const int i = ctr_s[0] - 3 + mi, jj = ctr_s[1] - 3 + mj, k = ctr_s[2] - 3 + mk;
          if (i >= 0 && i < a.g.n[0] && jj >= 0 && jj < a.g.n[1] && k >= 0 && k < a.g.n[2]) {
            cell = ((long long)k * a.g.n[1] + jj) * a.g.n[0] + i;
            w = wax[0][mi] * wax[1][mj] * wax[2][mk];
            dw[0] = dwax[0][mi] * wax[1][mj] * wax[2][mk];
            dw[1] = wax[0][mi] * dwax[1][mj] * wax[2][mk];
            dw[2] = wax[0][mi] * wax[1][mj] * dwax[2][mk];
            for (int q = 0; q < 4; ++q) gv[q] = G[q * nc + cell];
            J = c2p_jac((double)W[cell], (double)W[nc + cell], (double)W[2 * nc + cell], (double)W[3 * nc + cell]);
            T = temperature(J.e, a.eos_dof, hc);
            sig = ((double)mu[cell] + jt.dir[0] * (double)mu[nc + cell] + jt.dir[1] * (double)mu[2 * nc + cell] +
                   jt.dir[2] * (double)mu[3 * nc + cell]) / dV;
          }
        }
        // reductions: 0 wsum, 1 sum wT, 2 sum sig w, 3-5 sum sig dw, 6-8 sum dw T, 9-11 sum dw;
        // butterfly within each wave, then lane r < 12 adds the eight waves in order
#pragma unroll
        for (int r = 0; r < 12; ++r) {
          double v = r == 0 ? w : r == 1 ? w * T : r == 2 ? sig * w : r < 6 ? sig * dw[r - 3] : r < 9 ? dw[r - 6] * T : dw[r - 9];
#pragma unroll
          for (int off = 32; off > 0; off >>= 1) v = v + __shfl_xor(v, off, 64);
          if ((t & 63) == 0) red[t >> 6][r] = v;
        }
        __syncthreads();
        if (t < 12) {
          double v = red[0][t];
          for (int wv = 1; wv < 8; ++wv) v = v + red[wv][t];
          tot[t] = v;
        }
        __syncthreads();
        const double wsum = tot[0];
        const double Tj = tot[1] / wsum;
        const double Pj = energy_loss(jt, Tj, ell, hc);
        const double dJdP = tot[2];
        const double dPdT = 2.0 * jt.kappa_coll * jt.crcf * Tj / hc + 3.0 * jt.kappa_rad * jt.crcf * Tj * Tj * ell / (hc * hc);
        const double dJdT = dJdP * dPdT;
        if (cell >= 0) {
          const double eb = dJdT * (w / wsum) * T / (4.0 * J.e);
          const double vb[3] = {0.0, 0.0, 0.0};
          double Eb, Mb[3];
          c2p_vjp(J, eb, vb, Eb, Mb);
          G[cell] = gv[0] + (R)Eb;
          for (int k = 0; k < 3; ++k) G[(1 + k) * nc + cell] = gv[1 + k] + (R)Mb[k];
        }
        if (t == 0) {
          double* gr = a.grad + 5 * j;
          gr[0] += a.bdt * dJdP * jt.crcf * Tj * Tj * Tj * ell / (hc * hc);
          gr[1] += a.bdt * dJdP * jt.crcf * Tj * Tj / hc;
          for (int d = 0; d < 3; ++d) {
            const double dTj = (tot[6 + d] - Tj * tot[9 + d]) / wsum;
            gr[2 + d] += a.bdt * (Pj * tot[3 + d] + dJdT * dTj);
          }
        }
      }
    }
    __syncthreads();
  }
}

template <class R>
__global__ void __launch_bounds__(256) k_copy(const R* __restrict__ src, R* __restrict__ dst, long long n) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) dst[q] = src[q];
}

__global__ void k_copy_f64(const double* __restrict__ src, double* __restrict__ dst, int n) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) dst[q] = src[q];
}

template <class R>
__global__ void __launch_bounds__(256) k_fill(R* dst, long long n, R v) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) dst[q] = v;
}

// ---------------------------------------------------------------------------
// eps2 = sum (y^2 - x^2) e / sum (y^2 + x^2) e on the z = 0 plane (mean of
// the two middle planes for even nz).  Partial sums per block, then one block;
// the seed kernel writes d eps2 / dU on those planes (other cells: 0).
__device__ __forceinline__ void z0_planes(int nz, int& k0, int& k1) {
  if (nz % 2 == 0) {
    k0 = nz / 2 - 1;
    k1 = nz / 2;
  } else {
    k0 = k1 = (nz - 1) / 2;
  }
}

template <class R>
__global__ void __launch_bounds__(256) k_eps2_partial(const R* __restrict__ U, Grid g, double* part) {
  const int nx = g.n[0], ny = g.n[1];
  int k0, k1;
  z0_planes(g.n[2], k0, k1);
  const long long nc = g.nc;
  double num = 0.0, den = 0.0;
  unsigned fix = 0;
  for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < (long long)nx * ny;
       q += (long long)gridDim.x * blockDim.x) {
    const int i = (int)(q % nx), j = (int)(q / nx);
    const double x = cell_centre(i, nx, g.dx[0]), y = cell_centre(j, ny, g.dx[1]);
    const long long ca = ((long long)k0 * ny + j) * nx + i, cb = ((long long)k1 * ny + j) * nx + i;
    const PrimV pa = c2p((double)U[ca], (double)U[nc + ca], (double)U[2 * nc + ca], (double)U[3 * nc + ca], fix);
    const PrimV pb = c2p((double)U[cb], (double)U[nc + cb], (double)U[2 * nc + cb], (double)U[3 * nc + cb], fix);
    const double e = 0.5 * (pa.e + pb.e);
    num += (y * y - x * x) * e;
    den += (y * y + x * x) * e;
  }
  __shared__ double rn[256], rd[256];
  rn[threadIdx.x] = num;
  rd[threadIdx.x] = den;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      rn[threadIdx.x] += rn[threadIdx.x + h];
      rd[threadIdx.x] += rd[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = rn[0];
    part[2 * blockIdx.x + 1] = rd[0];
  }
}

__global__ void __launch_bounds__(256) k_eps2_final(const double* part, int nb, double* out3) {
  __shared__ double rn[256], rd[256];
  double num = 0.0, den = 0.0;
  for (int b = threadIdx.x; b < nb; b += blockDim.x) {
    num += part[2 * b];
    den += part[2 * b + 1];
  }
  rn[threadIdx.x] = num;
  rd[threadIdx.x] = den;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      rn[threadIdx.x] += rn[threadIdx.x + h];
      rd[threadIdx.x] += rd[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out3[0] = rn[0] / rd[0];
    out3[1] = rn[0];
    out3[2] = rd[0];
  }
}

template <class R>
__global__ void __launch_bounds__(256) k_eps2_seed(const R* __restrict__ U, Grid g, const double* eps3, R* lam,
                                                   double scale) {
  const int nx = g.n[0], ny = g.n[1];
  int k0, k1;
  z0_planes(g.n[2], k0, k1);
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (long long)nx * ny) return;
  const long long nc = g.nc;
  const int i = (int)(q % nx), j = (int)(q / nx);
  const double x = cell_centre(i, nx, g.dx[0]), y = cell_centre(j, ny, g.dx[1]);
  const double eps2 = eps3[0], den = eps3[2];
  const double de = scale * 0.5 * ((y * y - x * x) - eps2 * (y * y + x * x)) / den;  // d eps2 / d e_plane
  const int planes[2] = {k0, k1};
  for (int p = 0; p < 2; ++p) {
    const long long cell = ((long long)planes[p] * ny + j) * nx + i;
    const PrimJ J = c2p_jac((double)U[cell], (double)U[nc + cell], (double)U[2 * nc + cell], (double)U[3 * nc + cell]);
    const double vb[3] = {0.0, 0.0, 0.0};
    double Eb, Mb[3];
    c2p_vjp(J, de, vb, Eb, Mb);
    if (k0 == k1 && p == 1) break;  // odd nz: the single plane takes both halves
    const double f = (k0 == k1) ? 2.0 : 1.0;
    lam[cell] = lam[cell] + (R)(f * Eb);
    for (int k = 0; k < 3; ++k) lam[(1 + k) * nc + cell] = lam[(1 + k) * nc + cell] + (R)(f * Mb[k]);
  }
}

// Adjoint of primitive (e, v, n) -> conserved (FP64 out [5][nc]):
// E = (4/3 g2 - 1/3) e, M = 4/3 e g2 v, N = n g, g2 = 1/(1 - v^2).
template <class R>
__global__ void __launch_bounds__(256) k_prim_vjp(const double* __restrict__ prim, const R* __restrict__ lam,
                                                  double* __restrict__ out, long long nc) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nc) return;
  const double e = prim[q], n = prim[4 * nc + q];
  const double v[3] = {prim[nc + q], prim[2 * nc + q], prim[3 * nc + q]};
  const double v2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
  const double g2 = 1.0 / (1.0 - v2);
  const double gm = sqrt(g2);
  const double lE = (double)lam[q], lN = (double)lam[4 * nc + q];
  const double lM[3] = {(double)lam[nc + q], (double)lam[2 * nc + q], (double)lam[3 * nc + q]};
  const double lMv = lM[0] * v[0] + lM[1] * v[1] + lM[2] * v[2];
  out[q] = lE * (4.0 * g2 - 1.0) / 3.0 + 4.0 / 3.0 * g2 * lMv;
  for (int k = 0; k < 3; ++k) {
    // d g2 / d v_k = 2 v_k g2^2
    const double dg2 = 2.0 * v[k] * g2 * g2;
    out[(1 + k) * nc + q] = lE * 4.0 / 3.0 * e * dg2 + 4.0 / 3.0 * e * (g2 * lM[k] + dg2 * lMv) + lN * n * v[k] * g2 * gm;
  }
  out[4 * nc + q] = lN * gm;
}

// ---------------------------------------------------------------------------
// Host-side launchers.
// Lines of a workgroup (8, 4, 2 or 1) and faces of a run (6, 8, 9 or 13) of a
// line adjoint, by an estimate of the time.  Many lines fill the waves' lanes
// where a line has few runs; few lines leave LDS for a second workgroup on the
// CU and give the chip enough workgroups when there are few or long lines.  Its
// unit is a wave's step over one face; a workgroup takes its chain of steps at
// 2.5 (FP32: 3) units each, or its share of the CU's four SIMDs if they are
// busier than that, and y and z loads of under 32 neighbouring bytes cost more.
// Against the fastest of the four for 216 sets of lines (8 to 600 cells, 256 to
// 16384 lines, four and five fields) it loses 1 % (FP64) and 2 % on average.
// us an axis, as many lines as LDS holds / this / a lane per face: FP32 x, 500
// cells, 8192 lines 484 / 184 / 233, 256 lines 51 / 17 / 17; y, 16 cells, 16384
// lines 63 / 36 / 44; FP64 x, 64 cells, 16384 lines 182 / 129 / 126, 300 cells,
// 256 lines 29 / 15 / 18.
// The run length depends on type and face count alone, so that every number of
// lines adds in the same order (same bits).
constexpr size_t kOnePerCU = 160 * 1024;

inline double line_adj_cost(int AX, int n, int nf, long long nlines, int L, int nl, int fields, int elem) {
  const size_t lds = line_adj_lds_bytes(AX, nf, L, nl, fields, elem);
  if (lds > kOnePerCU) return 1e300;
  const int waves = line_adj_block(elem) / 64;
  const int fit = std::min((int)(kOnePerCU / lds), (elem == 8 ? 16 : 20) / waves);  // workgroups on a CU (VGPRs)
  const int steps = ((nf + L - 1) / L * nl + 63) / 64 * (L + 1);  // of an area: turns of runs, about one more to finish each
  const double chain = (2 * fields + waves - 1) / waves * steps + (n * nl + 64 * waves - 1) / (64 * waves);
  const double load = AX == 0 ? 1.0 : 1.0 + (elem == 8 ? 2.0 : 3.0) * std::max(0.0, 32.0 / (nl * elem) - 1.0);
  const double issue = 0.25 * (2 * fields * steps + (n * nl + 63) / 64 * load) + (elem == 8 ? 2.0 : 0.0);
  const double per_cu = (double)((nlines + nl - 1) / nl) / 256.0, wait = (elem == 8 ? 2.5 : 3.0) * chain;
  if (per_cu <= fit) return std::max(wait, std::max(per_cu, 1.0) * issue);
  return per_cu / fit * std::max(wait, fit * issue);
}

template <class R, int S, int AX, int L, int NL>
void launch_line_adj_n(const AdjArgs<R>& a, long long nlines, hipStream_t st) {
  const int nf = a.g.n[AX] + (a.g.bc[AX] ? 0 : 1);
  const size_t lds = line_adj_lds_bytes(AX, nf, L, NL, a.skip_n ? 4 : 5, (int)sizeof(R));
  const long long ng = (nlines + NL - 1) / NL;
  hipLaunchKernelGGL((k_line_adj<R, S, AX, L, NL, false>), dim3((unsigned)(((ng + 7) / 8) * 8)),
                     dim3(line_adj_block((int)sizeof(R))), lds, st, a);
}

// Segments of at most seglen cells of long y and z lines, four lines a workgroup.
// Of the face counts that take as many runs as seglen + 7, the most LDS: phi has
// a row more for every face fewer.
constexpr int seg_faces(int seglen, int L) { return (seglen + 6) / L * L + 1; }

template <class R, int S, int AX, int L>
void launch_line_adj_seg(AdjArgs<R> a, int seglen, hipStream_t st) {
  const int segs = (a.g.n[AX] + seglen - 1) / seglen;
  const long long nlines = (long long)a.g.n[0] * a.g.n[AX == 1 ? 2 : 1];
  const size_t lds = line_adj_lds_bytes(AX, seg_faces(seglen, L), L, 4, a.skip_n ? 4 : 5, (int)sizeof(R));
  const long long ng = (nlines + 3) / 4 * segs;
  a.seglen = seglen;
  hipLaunchKernelGGL((k_line_adj<R, S, AX, L, 4, true>), dim3((unsigned)(((ng + 7) / 8) * 8)),
                     dim3(line_adj_block((int)sizeof(R))), lds, st, a);
}

template <class R, int S, int AX, int L>
void launch_line_adj_l(const AdjArgs<R>& a, hipStream_t st) {
  const int n = a.g.n[AX], nf = n + (a.g.bc[AX] ? 0 : 1);
  const long long nlines = AX == 0 ? (long long)a.g.n[1] * a.g.n[2]
                                   : (AX == 1 ? (long long)a.g.n[0] * a.g.n[2] : (long long)a.g.n[0] * a.g.n[1]);
  // the fastest, and the fastest within the caller's limit if that is as fast; of
  // equals the fewer lines where the chip is full (FP32 x at 96^3: 89 -> 58 us),
  // the more where it is not (FP64 at 24^3: 22 -> 17 us)
  auto fewer = [&](int lines) { return (nlines + lines - 1) / lines > 256; };
  double best = 1e301, within = 1e301;
  int nl = 1, nw = 1;
  for (int c : {8, 4, 2, 1}) {
    const double t = line_adj_cost(AX, n, nf, nlines, L, c, a.skip_n ? 4 : 5, (int)sizeof(R));
    if (t < best || (t == best && fewer(nl))) {
      best = t;
      nl = c;
    }
    if (c <= a.lines && (t < within || (t == within && fewer(nw)))) {
      within = t;
      nw = c;
    }
  }
  if (a.lines > 0 && within <= 1.05 * best) nl = nw;
  if (nl == 8) launch_line_adj_n<R, S, AX, L, 8>(a, nlines, st);
  else if (nl == 4) launch_line_adj_n<R, S, AX, L, 4>(a, nlines, st);
  else if (nl == 2) launch_line_adj_n<R, S, AX, L, 2>(a, nlines, st);
  else launch_line_adj_n<R, S, AX, L, 1>(a, nlines, st);
}

// Run length, and segments of long y and z lines where they are cheaper by the
// same estimate (of 4096 lines with five fields, whatever the call's are, so that
// the form and with it every bit depend on the line's length alone). A whole line
// of 256 FP64 cells fills the LDS with one workgroup; its segments leave room for
// two, for 13 cells computed twice at each cut. Whole lines -> segments, us:
// y 64x256x256 525 -> 441 (FP64, four fields), 607 -> 539 (five); y 64x300x216 604
// -> 487; z 64x256x256 727 -> 545, FP32 547 -> 426; y 64x500x128 FP32 384 -> 230.
// Dearer where few lines leave the chip idle either way: y 16x400x16 FP32 23.7 -> 26.4.
template <class R, int S, int AX>
void launch_line_adj(const AdjArgs<R>& a, hipStream_t st) {
  const int n = a.g.n[AX], nf = n + (a.g.bc[AX] ? 0 : 1);
  int L = 8, seglen = n;
  double best = 1e301;
  for (int c : {8, 6, 9, 13}) {
    for (int nl : {8, 4, 2, 1}) {
      const double t = line_adj_cost(1, n, nf, 4096, c, nl, 5, (int)sizeof(R));
      if (t < best) {
        best = t;
        L = c;
      }
    }
  }
  if constexpr (AX != 0) {
    for (int k = 2; n / k >= 64; ++k) {
      const int m = (n + k - 1) / k;
      for (int c : {8, 6, 9, 13}) {
        const double t = line_adj_cost(1, m + 13, seg_faces(m, c), 4096LL * k, c, 4, 5, (int)sizeof(R));
        if (t < best) {
          best = t;
          L = c;
          seglen = m;
        }
      }
    }
    if (seglen < n) {
      if (L == 6) launch_line_adj_seg<R, S, AX, 6>(a, seglen, st);
      else if (L == 9) launch_line_adj_seg<R, S, AX, 9>(a, seglen, st);
      else if (L == 13) launch_line_adj_seg<R, S, AX, 13>(a, seglen, st);
      else launch_line_adj_seg<R, S, AX, 8>(a, seglen, st);
      return;
    }
  }
  if (L == 6) launch_line_adj_l<R, S, AX, 6>(a, st);
  else if (L == 9) launch_line_adj_l<R, S, AX, 9>(a, st);
  else if (L == 13) launch_line_adj_l<R, S, AX, 13>(a, st);
  else launch_line_adj_l<R, S, AX, 8>(a, st);
}

template <class R, int S>
void launch_adj_axis_t(int AX, const AdjArgs<R>& a0, hipStream_t st) {
  AdjArgs<R> a = a0;
  a.inv_d = R(1.0 / a.g.dx[AX]);
  a.eps = R(4) * a.eps;  // indicators of the doubled split fluxes; the partials dR/da do not change
  if (AX == 0) launch_line_adj<R, S, 0>(a, st);
  if (AX == 1) launch_line_adj<R, S, 1>(a, st);
  if (AX == 2) launch_line_adj<R, S, 2>(a, st);
}

template <class R>
hipError_t launch_adj_axis(int AX, const AdjArgs<R>& a, int scheme, hipStream_t st) {
  if (scheme == kWenoJS)
    launch_adj_axis_t<R, kWenoJS>(AX, a, st);
  else if (scheme == kWenoLinear)
    launch_adj_axis_t<R, kWenoLinear>(AX, a, st);
  else
    launch_adj_axis_t<R, kWenoZ>(AX, a, st);
  return hipGetLastError();
}

template <class R>
hipError_t launch_jet_adj(const JetAdjArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((k_jet_adj<R>), dim3(1), dim3(512), 0, st, a);
  return hipGetLastError();
}

template <class R>
hipError_t launch_copy(const R* src, R* dst, long long n, hipStream_t st) {
  hipLaunchKernelGGL((k_copy<R>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, dst, n);
  return hipGetLastError();
}

hipError_t launch_copy_f64(const double* src, double* dst, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_copy_f64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, dst, n);
  return hipGetLastError();
}

template <class R>
hipError_t launch_fill(R* dst, long long n, R v, hipStream_t st) {
  hipLaunchKernelGGL((k_fill<R>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, dst, n, v);
  return hipGetLastError();
}

template <class R>
hipError_t launch_eps2(const R* U, const Grid& g, double* part, double* out3, hipStream_t st) {
  hipLaunchKernelGGL((k_eps2_partial<R>), dim3(256), dim3(256), 0, st, U, g, part);
  hipLaunchKernelGGL(k_eps2_final, dim3(1), dim3(256), 0, st, part, 256, out3);
  return hipGetLastError();
}

template <class R>
hipError_t launch_eps2_seed(const R* U, const Grid& g, const double* out3, R* lam, double scale, hipStream_t st) {
  const long long np = (long long)g.n[0] * g.n[1];
  hipLaunchKernelGGL((k_eps2_seed<R>), dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, U, g, out3, lam, scale);
  return hipGetLastError();
}

template <class R>
hipError_t launch_prim_vjp(const double* prim, const R* lam, double* out, long long nc, hipStream_t st) {
  hipLaunchKernelGGL((k_prim_vjp<R>), dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, st, prim, lam, out, nc);
  return hipGetLastError();
}

#define HYDRO_ADJ_INSTANTIATE(R)                                                                               \
  template hipError_t launch_adj_axis<R>(int, const AdjArgs<R>&, int, hipStream_t);                           \
  template hipError_t launch_jet_adj<R>(const JetAdjArgs&, hipStream_t);                                     \
  template hipError_t launch_copy<R>(const R*, R*, long long, hipStream_t);                                   \
  template hipError_t launch_fill<R>(R*, long long, R, hipStream_t);                                          \
  template hipError_t launch_eps2<R>(const R*, const Grid&, double*, double*, hipStream_t);                    \
  template hipError_t launch_eps2_seed<R>(const R*, const Grid&, const double*, R*, double, hipStream_t);       \
  template hipError_t launch_prim_vjp<R>(const double*, const R*, double*, long long, hipStream_t);

HYDRO_ADJ_INSTANTIATE(double)
HYDRO_ADJ_INSTANTIATE(float)

}  // namespace hydro
