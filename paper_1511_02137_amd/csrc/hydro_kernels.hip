// hydro_kernels.hip -- HIP kernels of one SSP-RK3 stage for gfx950.
//
// The stage computes L(W) = D(W) + S(W) and the Runge-Kutta combine:
//   D: flux divergence of 7th-order WENO reconstructions of the
//      Lax-Friedrichs split fluxes F+- = (f +- W)/2 (alpha = 1), one axis at
//      a time, component by component (Eq. 1 with the paper's WENO7);
//   S: jet source, Eq. (2) and Eq. (3);
//   combine: Shu-Osher SSP-RK3.
//
// Work split (all kernels of a stage run on one stream):
//   k_line    x, y or z faces from LDS tiles of 16 lines: one lane per point
//             recovers it, lanes then march over runs of faces.  x assigns its
//             divergence to D, y adds, z adds its own, does the RK combine and
//             writes the stage output.
//   k_march   lanes along x (coalesced), each lane marches along y or z over
//             a segment, keeping the split fluxes of the 8-point stencil in
//             registers: one new cell and one face per step, no halo recompute.
//   k_jet     the source at the jet cells (between the y and z faces).
// All recovery of primitives is FP64; the flux and WENO arithmetic is in the
// field type R (double or float).  FP contraction is off: every fma is
// explicit, so every face is computed by the same sequence of roundings.

#include <hip/hip_runtime.h>

#include "hydro_device.hpp"
#include "hydro_internal.hpp"

namespace hydro {

// What the face kernels keep per point: twice the Lax-Friedrichs split fluxes
// (F+, F-; face_scale sets what that changes), or with MUSTA-FORCE the
// conserved values themselves (in the F+ slots; no recovery needed).
template <class R, int S, int AX>
__device__ __forceinline__ void point_values(const R u[5], R Fp[5], R Fm[5], unsigned& fix) {
  if constexpr ((S & kMusta) != 0) {
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      Fp[c] = u[c];
      Fm[c] = R(0);
    }
  } else {
    const PrimV pv = c2p(u, fix);
    split_flux<R, AX>(u, pv, Fp, Fm);
  }
}

// Weights' epsilon and 1/dx for the point values above: with doubled split
// fluxes the indicators are four times as large and the face fluxes twice
// (powers of two: every value scales exactly).
template <class R, int S>
__host__ __device__ __forceinline__ void face_scale(StageArgs<R>& a, double inv_d) {
  constexpr bool twice = (S & kMusta) == 0;
  a.inv_d = (R)((twice ? 0.5 : 1.0) * inv_d);
  if (twice) a.eps = R(4) * a.eps;
}

// SSP-RK3 combine of the last face kernel of a stage (z).  With L = Dxy + Dz
// (Dxy: the x and y divergences and the source, already in D; Dz: the z
// divergence), the stage value w + dt L enters as p = w + dt Dxy, then
// p + dt Dz (two fmas), so that a kernel can fold w into p before its
// reconstructions and keep one value per field instead of two.  Stage 0
// returns L itself.
template <class R>
__device__ __forceinline__ R rk_pre(int stage, R w, R dxy, R dt) {
  return stage == 0 ? dxy : fma(dt, dxy, w);
}
template <class R>
__device__ __forceinline__ R rk_out(int stage, R p, R dz, R dt, const R* Un, long long i) {
  if (stage == 0) return p + dz;
  const R v = fma(dt, dz, p);
  if (stage == 1) return v;
  if (stage == 2) return R(0.75) * Un[i] + R(0.25) * v;
  return R(1.0 / 3.0) * Un[i] + R(2.0 / 3.0) * v;
}
// the same with U^n already read (un; used in stages 2 and 3 only)
template <class R>
__device__ __forceinline__ R rk_out_v(int stage, R p, R dz, R dt, R un) {
  if (stage == 0) return p + dz;
  const R v = fma(dt, dz, p);
  if (stage == 1) return v;
  if (stage == 2) return R(0.75) * un + R(0.25) * v;
  return R(1.0 / 3.0) * un + R(2.0 / 3.0) * v;
}

// ---------------------------------------------------------------------------
// March along axis AX (1 = y, 2 = z).  blockDim = (64, BY): lanes along x,
// threadIdx.y over the other transverse axis; blockIdx.z = segment of `seg`
// cells along AX.  LAST: z-march, which finishes L and does the RK combine.
// The limiter on the march's window: the face between window points 3 and 4.
template <class R>
__device__ __forceinline__ void march_limit(R H[5], const R (&fp)[5][8], const R (&fm)[5][8], double mu) {
  pp_limit<R>(H, [&](int c, int k) { return (k & 1) ? fm[c][3 + (k >> 1)] : fp[c][3 + (k >> 1)]; }, mu);
}

template <class R, int S, int AX, bool LAST>
__global__ void __launch_bounds__(256) k_march(StageArgs<R> a) {
  const int nx = a.g.n[0], ny = a.g.n[1], nz = a.g.n[2];
  const int x = blockIdx.x * 64 + threadIdx.x;
  const int o = blockIdx.y * blockDim.y + threadIdx.y;
  const int n = (AX == 1) ? ny : nz;
  const int no = (AX == 1) ? nz : ny;
  if (x >= nx || o >= no) return;
  const long long nc = a.g.nc;
  const long long stride = (AX == 1) ? (long long)nx : (long long)nx * ny;
  const long long base = (AX == 1) ? (long long)o * nx * ny + x : (long long)o * nx + x;
  const int bc = a.g.bc[AX];
  const int i0 = blockIdx.z * a.seg;
  const int i1 = min(i0 + a.seg, n);
  unsigned fix = 0;

  R fp[5][8], fm[5][8];  // split fluxes at points i-3..i+4 for face i+1/2
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    R u[5];
    load5(a.W, nc, base + (long long)map_idx(i0 - 4 + m, n, bc) * stride, u);
    R Fp[5], Fm[5];
    point_values<R, S, AX>(u, Fp, Fm, fix);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      fp[c][m] = Fp[c];
      fm[c][m] = Fm[c];
    }
  }
  auto face = [&](R fh[5]) {
    if constexpr ((S & kMusta) != 0) {
      musta_face<R, (S & 7), AX>([&](int c, int m) { return fp[c][m]; }, a.eps, a.musta_k, fh, fix);
    } else {
#pragma unroll
      for (int c = 0; c < 5; ++c) fh[c] = face_flux<R, (S & 7)>(fp[c], fm[c], a.eps);
      if constexpr ((S & kPP) != 0) march_limit<R>(fh, fp, fm, a.pp_mu);
    }
  };
  R prev[5];
  face(prev);

  for (int i = i0; i < i1; ++i) {
#pragma unroll
    for (int c = 0; c < 5; ++c) {
#pragma unroll
      for (int m = 0; m < 7; ++m) {
        fp[c][m] = fp[c][m + 1];
        fm[c][m] = fm[c][m + 1];
      }
    }
    {
      R u[5];
      load5(a.W, nc, base + (long long)map_idx(i + 4, n, bc) * stride, u);
      R Fp[5], Fm[5];
      point_values<R, S, AX>(u, Fp, Fm, fix);
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        fp[c][7] = Fp[c];
        fm[c][7] = Fm[c];
      }
    }
    const long long cell = base + (long long)i * stride;
    R fh[5];
    face(fh);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      const R div = (prev[c] - fh[c]) * a.inv_d;
      prev[c] = fh[c];
      R* d = a.D + c * nc + cell;
      if (!LAST) {
        *d = *d + div;
      } else {
        const R p = rk_pre(a.stage, a.W[c * nc + cell], *d, a.dt);
        a.out[c * nc + cell] = rk_out(a.stage, p, div, a.dt, a.Un, c * nc + cell);
      }
    }
  }
  add_fixups(a.fixups, fix);
}

// ---------------------------------------------------------------------------
// Faces taken along lines (plain WENO fluxes; MUSTA-FORCE and the limiter have
// their own sharing out, in line_body).  A lane marches over neighbouring faces of one split of
// one field of its line, so that the differences and their indicator terms of
// a point serve every face of the run (weno_line).  A workgroup has eight
// waves, which the hardware deals evenly over the four SIMDs; the ten (field,
// split) areas are shared out so that all have the same work: wave w marches
// over area w, and the eight waves take the N field's two areas in short runs,
// whose results stay in registers until a barrier.  (One wave per area: 24.0
// ms for three steps at 256^3 FP64, two SIMDs with three waves and two with
// two; four (field, split, half) units for some waves and six for others: 18.9
// ms.)  F- is stored in reverse slot order, so that both splits march upwards.
//
// A run reads its values one ahead and stores each result, one face late, in
// the place of its first value: the lanes of a wave execute their LDS
// operations in order, and result j of a run follows the read of value j + 8
// (its last value, if that comes first), after which no run before it needs
// anything more from that place.
template <class R, int S, int L, class Idx>
__device__ __forceinline__ void line_faces(R* area, Idx idx, R eps) {
  R next = area[idx(0)], last = R(0);
  weno_line<R, S, L>(
      [&](int m) {
        const R v = next;
        if (m + 1 < L + 6) next = area[idx(m + 1)];
        __asm__ __volatile__("" ::: "memory");
        return v;
      },
      eps,
      [&](int k, R x) {
        if (k > 0) area[idx(k - 1)] = last;
        last = x;
        __asm__ __volatile__("" ::: "memory");
      });
  area[idx(L - 1)] = last;
}

// Line tiles: a workgroup owns A = 31 or 32 cells (A = 15, in half a workgroup,
// where the axis has no more) along AX by 16 lines (y and z: 16 cells along x at
// one value of the remaining axis; x: 16 rows in memory order, whatever their y
// and z: x at 256x1x256 31 -> 9 us).  One lane per own cell, and 128 lanes for the 4 ghost slots on each
// side, recover the points and store their split AX-fluxes in LDS; four lane
// groups of a wave march over the line_rows(A) face rows in runs of a quarter of
// them, and with A = 32 lanes 0..159 take the 33rd row, one face each; each own
// cell's lane forms its divergence.  D is loaded before the march (LAST: folded
// into the combine's p = w + dt D, rk_pre), to hide its latency; x is the first
// axis and assigns D.  x tiles load along x (coalesced) and keep a pitch of 17
// words, so that their stores do not meet in a bank.
template <class R, int S, int AX, bool LAST, int A>
__device__ __forceinline__ void line_body(const StageArgs<R>& a, int bx, int by, int bz, R* s) {
  constexpr bool kM = (S & kMusta) != 0, kL = (S & kPP) != 0;
  constexpr int kP = A + 8;  // points of a line
  constexpr int kRows = line_rows(A), kWaves = kRows / 4, kHalves = kRows / 16;
  constexpr int kRow = AX == 0 ? kLineX + 1 : kLineX;
  constexpr int kArea = kP * kRow;  // one (field, split): area 2 field + split
  const int nx = a.g.n[0], ny = a.g.n[1];
  const int n = a.g.n[AX];
  const unsigned no = AX == 0 ? (unsigned)ny * (unsigned)a.g.n[2] : (unsigned)nx;  // lines that bx counts
  const int bc = a.g.bc[AX];
  const long long nc = a.g.nc;
  const int stride = AX == 0 ? 1 : (AX == 1 ? nx : nx * ny);
  const int t = threadIdx.x;
  const int w = t >> 6;
  const int a0 = by * A;
  const int len = min(A, n - a0);
  const unsigned line0 = (unsigned)bx * kLineX;
  const long long base = AX == 0 ? (long long)line0 * nx
                                 : (AX == 1 ? (long long)bz * nx * ny + line0 : (long long)bz * nx + line0);
  const int lstep = AX == 0 ? nx : 1;  // cells between lines
  unsigned fix = 0;

  // own cell of the lane: line tx, cell ta of the tile (lanes run along x in memory)
  const int tx = AX == 0 ? (unsigned)t / kRows : t & (kLineX - 1);
  const int ta = AX == 0 ? t & (kRows - 1) : t >> 4;
  const bool own = line0 + tx < no && ta < len;
  const long long cell = base + tx * lstep + (long long)(a0 + ta) * stride;
  R dpre[5];
  auto point = [&](int line, int slot, const R u[5]) {
    R Fp[5], Fm[5];
    point_values<R, S, AX>(u, Fp, Fm, fix);
    R* sp = s + slot * kRow + line;
    R* sm = s + kArea + (kP - 1 - slot) * kRow + line;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      sp[2 * c * kArea] = Fp[c];
      if (!kM) sm[2 * c * kArea] = Fm[c];
    }
  };
  // the last two waves also take ghost slots 0..3 and len + 4..len + 7; their
  // loads go first, so that their latency overlaps the own cells' recovery
  const int gq = t - (kWaves - 2) * 64;
  const int gl = AX == 0 ? gq >> 3 : gq & (kLineX - 1);
  const int gh = AX == 0 ? gq & 7 : gq >> 4;
  const int gslot = gh < 4 ? gh : gh + len;
  const bool ghost = w >= kWaves - 2 && line0 + gl < no;
  R ug[5];
  if (ghost) {
    int p = a0 - 4 + gslot;
    if ((unsigned)p >= (unsigned)n) p = map_idx(p, n, bc);
    load5(a.W, nc, base + gl * lstep + (long long)p * stride, ug);
  }
  if (own) {
    R u[5];
    load5(a.W, nc, cell, u);
    if (AX != 0) {
#pragma unroll
      for (int c = 0; c < 5; ++c) dpre[c] = a.D[c * nc + cell];
    }
    point(tx, ta + 4, u);
    if (LAST) {
#pragma unroll
      for (int c = 0; c < 5; ++c) dpre[c] = rk_pre(a.stage, u[c], dpre[c], a.dt);
    }
  }
  if (ghost) point(gl, gslot, ug);
  __syncthreads();
  const int xl = t & (kLineX - 1), grp = (t >> 4) & 3;
  if constexpr (kM) {
    // MUSTA-FORCE: points in area 2 field; window q (slots q..q+6, cell slot
    // q + 3) gives uL of face row q (right value) and uR of face row q - 1
    // (left value).  Waves 2c and 2c + 1 march over rows 0..15 and 16..31 of
    // field c = 0..3 (A = 15: wave c over its 16 rows), every lane takes one
    // window of N, and lanes of the first waves the windows from kRows on; the results wait in registers until all
    // points are read, then uL goes to area 2 field and uR to the next.
    // One window per cell and field instead of two per face, and then one lane
    // per face with its 3 k recoveries, which bound the kernel: ~112 registers,
    // so 4 waves a SIMD (6 would spill).  At 128^3 in double precision, k = 2:
    // 106 to 114 us a launch, a step 1170 -> 895 us.
    const int c4 = w / kHalves, q4 = (w % kHalves) * 16 + grp * 4, qn = t >> 4;
    const R* v4 = s + 2 * c4 * kArea + q4 * kRow + xl;
    R ur[4], ul[4], nr, nl, xr = R(0), xm = R(0);
    weno_line<R, (S & 7), 4, true>([&](int m) { return v4[m * kRow]; }, a.eps, [&](int k, R r, R l) {
      ur[k] = r;
      ul[k] = l;
    });
    const R* vn = s + 8 * kArea + qn * kRow + xl;
    weno_line<R, (S & 7), 1, true>([&](int m) { return vn[m * kRow]; }, a.eps, [&](int, R r, R l) {
      nr = r;
      nl = l;
    });
    // windows kRows .. A + 1
    const int xc = (t >> 4) % 5, xq = kRows + (t >> 4) / 5;
    const bool extra = xq <= A + 1;
    const R* vx = s + 2 * xc * kArea + xq * kRow + xl;
    if (extra) {
      weno_line<R, (S & 7), 1, true>([&](int m) { return vx[m * kRow]; }, a.eps, [&](int, R r, R l) {
        xr = r;
        xm = l;
      });
    }
    __syncthreads();
    auto store = [&](int c, int q, R r, R l) {
      R* d = s + 2 * c * kArea + q * kRow + xl;
      if (q <= A) d[0] = r;
      if (q > 0) d[kArea - kRow] = l;
    };
#pragma unroll
    for (int k = 0; k < 4; ++k) store(c4, q4 + k, ur[k], ul[k]);
    store(4, qn, nr, nl);
    if (extra) store(xc, xq, xr, xm);
    __syncthreads();
    // one lane per face: row t / 16, and row 32 by the first 16 lanes
    auto flux = [&](int row) {
      R* d = s + row * kRow + xl;
      R uL[5], uR[5], F[5];
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        uL[c] = d[2 * c * kArea];
        uR[c] = d[(2 * c + 1) * kArea];
      }
      musta_force<R, AX>(uL, uR, a.musta_k, F, fix);
#pragma unroll
      for (int c = 0; c < 5; ++c) d[2 * c * kArea] = F[c];
    };
    const bool line_in = line0 + xl < no;
    if (line_in && qn <= len) flux(qn);
    if (A == 32 && t < kLineX && line_in && len == 32) flux(32);
    __syncthreads();
  } else if constexpr (kL) {
    // Limiter: it reads the split fluxes of the two cells next to a face, so
    // the points stay and the face fluxes get rows of their own.  Waves 2c and
    // 2c + 1 (A = 15: wave c) march over the rows of field c = 0..3, F+ and then F-
    // (its run starts at the last face); every lane takes one face of N, and
    // the first lanes row 32.  The rows of their own bring the tile to 72 KB in
    // FP64, two workgroups a CU, which its registers (82) allow as well: 4 waves
    // a SIMD still issue at the peak rate.  Against tiles of whole faces per
    // lane, us a step without jets: FP64 128^3 989 -> 815, 31^3 99 -> 85; FP32
    // 128^3 623 -> 515; batches of 16 x 64^3 2542 -> 1732 (FP64), 1644 -> 1017.
    const int c4 = w / kHalves, q4 = (w % kHalves) * 16 + grp * 4, qn = t >> 4;
    auto rowp = [&](int c, int q) { return s + 2 * c * kArea + q * kRow + xl; };
    auto rowm = [&](int c, int q) { return s + (2 * c + 1) * kArea + (A - q) * kRow + xl; };
    auto flux = [&](int c, int q) { return s + 10 * kArea + (c * (A + 1) + q) * kRow + xl; };
    R fr[4];
    const R* vp = rowp(c4, q4);
    weno_line<R, (S & 7), 4>([&](int m) { return vp[m * kRow]; }, a.eps, [&](int k, R v) { fr[k] = v; });
    const R* vm = rowm(c4, q4 + 3);
    weno_line<R, (S & 7), 4>([&](int m) { return vm[m * kRow]; }, a.eps, [&](int k, R v) { fr[3 - k] = fr[3 - k] + v; });
    R* d = flux(c4, q4);
#pragma unroll
    for (int k = 0; k < 4; ++k) d[k * kRow] = fr[k];
    auto one = [&](int c, int q) {
      R f = R(0);
      const R* p = rowp(c, q);
      weno_line<R, (S & 7), 1>([&](int m) { return p[m * kRow]; }, a.eps, [&](int, R v) { f = v; });
      const R* m0 = rowm(c, q);
      weno_line<R, (S & 7), 1>([&](int m) { return m0[m * kRow]; }, a.eps, [&](int, R v) { f = f + v; });
      *flux(c, q) = f;
    };
    one(4, qn);
    if (A == 32 && t < 80) one(t >> 4, 32);
    __syncthreads();
    // one lane per face, as above
    auto limit = [&](int q) {
      R H[5];
#pragma unroll
      for (int c = 0; c < 5; ++c) H[c] = *flux(c, q);
      const R* p = rowp(0, q + 3);
      const R* m = rowm(0, q - 4);
      pp_limit<R>(
          H, [&](int c, int k) { return (k & 1) ? m[2 * c * kArea - (k >> 1) * kRow] : p[2 * c * kArea + (k >> 1) * kRow]; },
          a.pp_mu);
#pragma unroll
      for (int c = 0; c < 5; ++c) *flux(c, q) = H[c];
    };
    const bool line_in = line0 + xl < no;
    if (line_in && qn <= len) limit(qn);
    if (A == 32 && t < kLineX && line_in && len == 32) limit(32);
    __syncthreads();
  } else {
    // face row f: face (a0 - 1 + f) + 1/2; F+ at slots f..f+6, its result in
    // row f; F- at slots f+7..f+1, stored from row A - f on, its result there
    constexpr int kRun = kRows / 4;
    // 8 face rows or fewer: runs of two (F-: in the upper half of the area)
    const bool few = A == 15 && len < 8;
    const int up = few && (w & 1) ? 8 : 0;
    R* area = s + w * kArea + (up + grp * (few ? 2 : kRun)) * kRow + xl;
#pragma unroll 1
    for (int c = 0; c < 8; c += kWaves, area += kWaves * kArea) {
      if (few) line_faces<R, S, 2>(area, [](int m) { return m * kRow; }, a.eps);
      else line_faces<R, S, kRun>(area, [](int m) { return m * kRow; }, a.eps);
    }
    // N: split w & 1, rows 2q and 2q + 1, q = 4 (w >> 1) + grp
    R* const nrow = s + (8 + (w & 1)) * kArea + (up + (w >> 1) * 8 + grp * 2) * kRow + xl;
    R nf[2] = {R(0), R(0)};
    if (!few || w < 2)
      weno_line<R, S, 2>([&](int m) { return nrow[m * kRow]; }, a.eps, [&](int k, R v) { nf[k] = v; });
    R ex = R(0);
    const bool extra = A == 32 && t < 160;  // row 32 of area t / 16
    R* const xrow = s + (t >> 4) * kArea + 32 * kRow + xl;
    if (extra) {
      weno_line<R, S, 1>([&](int m) { return xrow[m * kRow]; }, a.eps, [&](int, R v) { ex = v; });
    }
    __syncthreads();  // the points of N and of row 32 are no longer read
    if (!few || w < 2) {
      nrow[0] = nf[0];
      nrow[kRow] = nf[1];
    }
    if (extra) *xrow = ex;
    __syncthreads();
  }
  // the own cell once more, in FP64 from a lane index that the compiler cannot
  // match with the first one: kept across the faces, the cell's offset takes two
  // registers too many for three workgroups a CU and is spilled (0.15 GB of
  // scratch a launch at 256^3; three steps 18.08 -> 17.69 ms)
  int t2 = threadIdx.x;
  if (sizeof(R) == 8) __asm__ __volatile__("" : "+v"(t2));
  const int tx2 = AX == 0 ? (unsigned)t2 / kRows : t2 & (kLineX - 1);
  const int ta2 = AX == 0 ? t2 & (kRows - 1) : t2 >> 4;
  if (line0 + tx2 < no && ta2 < len) {
    const long long cell2 = base + tx2 * lstep + (long long)(a0 + ta2) * stride;
    // LAST, stages 2 and 3: the five U^n values are read before any output
    // is stored (out may be U^n itself, so the compiler would otherwise keep
    // each read behind the previous field's store: five round trips)
    R unv[5];
    if (LAST && a.stage >= 2) {
#pragma unroll
      for (int c = 0; c < 5; ++c) unv[c] = a.Un[c * nc + cell2];
    }
    const R* sp = s + (kL ? 10 * kArea : 0) + ta2 * kRow + tx2;
    const R* sm = s + kArea + (A - 1 - ta2) * kRow + tx2;  // F- of the right face; the left face's follows
    constexpr int kStep = kL ? (A + 1) * kRow : 2 * kArea;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      const R fl = kM || kL ? sp[c * kStep] : sp[c * kStep] + sm[c * kStep + kRow];
      const R fr = kM || kL ? sp[c * kStep + kRow] : sp[c * kStep + kRow] + sm[c * kStep];
      const R div = (fl - fr) * a.inv_d;
      if (AX == 0) {
        a.D[c * nc + cell2] = div;
      } else if (!LAST) {
        a.D[c * nc + cell2] = dpre[c] + div;
      } else {
        a.out[c * nc + cell2] = rk_out_v(a.stage, dpre[c], div, a.dt, unv[c]);
      }
    }
  }
  add_fixups(a.fixups, fix);
}

template <class R, int S, int AX, bool LAST, int A>
__global__ void __launch_bounds__(kLineX * line_rows(A), (S & (kMusta | kPP)) ? 4 : 6) k_line(StageArgs<R> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  R* const s = reinterpret_cast<R*>(smem_raw);
  if constexpr (AX == 0) {
    line_body<R, S, AX, LAST, A>(a, blockIdx.x + gridDim.x * blockIdx.z, blockIdx.y, 0, s);
  } else {
    // blockIdx.x: 16 lines; tile along AX and transverse index in either order
    unsigned b0 = blockIdx.x, b1 = blockIdx.y;
    if (a.seg != 0) {  // a.seg = ceil(2^32 / gridDim.x): neighbours on one XCD
      const unsigned id = b0 + gridDim.x * b1, per = (gridDim.x * gridDim.y) >> 3;
      if (id < 8 * per) {
        const unsigned to = (id & 7) * per + (id >> 3);
        b1 = __umulhi(to, (unsigned)a.seg);
        b0 = to - b1 * gridDim.x;
      }
    }
    const int by = a.order ? blockIdx.z : b1;
    const int bz = a.order ? b1 : blockIdx.z;
    line_body<R, S, AX, LAST, A>(a, b0, by, bz, s);
  }
}

// ---------------------------------------------------------------------------
// Jet source (Eq. 2 and 3).  One workgroup of 512 threads.  The kernel is a
// chain of memory latencies and of serial FP64 arithmetic (a microsecond each),
// not work, so every lane finds the jet's cell itself and all that needs no
// other result is under way at once.  NGP: lane j of the first wave takes jet
// j; jets in one cell add in jet order, each lane of that cell forming the same
// sum (ensemble with up to three jets an event: 6.4 us a launch, 12.5
// one jet after the other).
// Gaussian: jets in order, 343 lanes for the 7^3 footprint, its weights by 21
// lanes, the sums by wave shuffles (5.1 us a launch; 9.9 with the weights by
// one lane and two trees of nine barriers).
template <class R>
__device__ __forceinline__ void jet_body(const JetArgs& a) {
  const R* W = static_cast<const R*>(a.W);
  R* D = static_cast<R*>(a.D);
  const long long nc = a.g.nc;
  const double dV = a.g.dx[0] * a.g.dx[1] * a.g.dx[2];
  const int t = threadIdx.x;
  unsigned fix = 0;
  // deposits of a step, added to the ledger in jet order
  auto deposit_of = [&](int j, double P) {
    return a.dt * ((1.0 / 6.0) * a.s->P[0][j] + (1.0 / 6.0) * a.s->P[1][j] + (2.0 / 3.0) * P);
  };
  if (a.deposit == 0) {
    if (t >= 64) return;
    const bool mine = t < a.njet;
    const JetDev jt = a.s->jets[mine ? t : 0];
    const double E = a.s->E_jet[mine ? t : 0];
    const bool chi = mine && E > 0.0;
    const double ell = a.t - jt.t_start;
    int c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) c[d] = ngp_index(jt.x0[d] + jt.dir[d] * ell, a.g.n[d], a.g.dx[d]);
    const bool in = chi && ell >= 0.0 && c[0] >= 0 && c[1] >= 0 && c[2] >= 0;
    long long cell = -1 - t;  // distinct
    double P = 0.0;
    R dv[4] = {R(0), R(0), R(0), R(0)}, sv[4] = {R(0), R(0), R(0), R(0)};
    if (in) {
      cell = ((long long)c[2] * a.g.n[1] + c[1]) * a.g.n[0] + c[0];
      R u[5];
      load5(W, nc, cell, u);
#pragma unroll
      for (int d = 0; d < 4; ++d) dv[d] = D[d * nc + cell];
      const PrimV pv = c2p(u, fix);
      P = energy_loss(jt, temperature(pv.e, a.eos_dof, a.hbarc), ell, a.hbarc);
      const double s0 = P / dV;
      sv[0] = (R)s0;
#pragma unroll
      for (int d = 0; d < 3; ++d) sv[1 + d] = (R)(jt.dir[d] * s0);
    }
    for (int j = 0; j < a.njet; ++j) {
      const bool same = __shfl(cell, j, 64) == cell;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const R v = __shfl(sv[d], j, 64);
        if (same) dv[d] = dv[d] + v;
      }
    }
    if (in) {
#pragma unroll
      for (int d = 0; d < 4; ++d) D[d * nc + cell] = dv[d];
    }
    if (a.stage == 3) {
      const double dep = chi ? deposit_of(t, P) : 0.0;
      double ledger = a.s->ledger;
      for (int j = 0; j < a.njet; ++j) {
        const double v = __shfl(dep, j, 64);
        if (__shfl(chi ? 1 : 0, j, 64)) ledger = ledger + v;
      }
      if (t == 0) a.s->ledger = ledger;
      if (chi) a.s->E_jet[t] = E - dep > 0.0 ? E - dep : 0.0;
    }
    if (mine && a.stage > 0) a.s->P[a.stage - 1][t] = P;
    add_fixups(&a.s->fixups, fix);
    return;
  }
  __shared__ double red[8][2];
  __shared__ double raw[3][7];
  const int wd = t / 7, wm = t % 7;
  for (int j = 0; j < a.njet; ++j) {
    const JetDev jt = a.s->jets[j];
    const double E = a.s->E_jet[j];
    const bool chi = E > 0.0;
    const double ell = a.t - jt.t_start;
    double x[3];
    int c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      x[d] = jt.x0[d] + jt.dir[d] * ell;
      c[d] = ngp_index(x[d], a.g.n[d], a.g.dx[d]);
    }
    const bool in = chi && ell >= 0.0 && c[0] >= 0 && c[1] >= 0 && c[2] >= 0;  // uniform
    double P = 0.0;
    if (in) {
      // 7^3 footprint, thread t < 343 owns cell (mi, mj, mk)
      const int mi = t % 7, mj = (t / 7) % 7, mk = t / 49;
      long long cell = -1;
      R u[5], dv[4];
      if (t < 343) {
        const int i = c[0] - 3 + mi, jj = c[1] - 3 + mj, k = c[2] - 3 + mk;
        if (i >= 0 && i < a.g.n[0] && jj >= 0 && jj < a.g.n[1] && k >= 0 && k < a.g.n[2]) {
          cell = ((long long)k * a.g.n[1] + jj) * a.g.n[0] + i;
          load5(W, nc, cell, u);
#pragma unroll
          for (int d = 0; d < 4; ++d) dv[d] = D[d * nc + cell];
        }
      }
      if (t < 21) {  // the lane's axis by selects (an index would put the structs in scratch memory)
        const double xd = wd == 0 ? x[0] : (wd == 1 ? x[1] : x[2]);
        const double dx = wd == 0 ? a.g.dx[0] : (wd == 1 ? a.g.dx[1] : a.g.dx[2]);
        const int cd = wd == 0 ? c[0] : (wd == 1 ? c[1] : c[2]);
        const int nd = wd == 0 ? a.g.n[0] : (wd == 1 ? a.g.n[1] : a.g.n[2]);
        const double del = cell_centre(cd - 3 + wm, nd, dx) - xd;
        raw[wd][wm] = exp(-(del * del) / (2.0 * dx * dx));
      }
      __syncthreads();
      double w = 0.0, wT = 0.0;
      if (cell >= 0) {
        double sum[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          sum[d] = 0.0;
#pragma unroll
          for (int m = 0; m < 7; ++m) sum[d] = sum[d] + raw[d][m];
        }
        w = (raw[0][mi] / sum[0]) * (raw[1][mj] / sum[1]) * (raw[2][mk] / sum[2]);
        const PrimV pv = c2p(u, fix);
        wT = w * temperature(pv.e, a.eos_dof, a.hbarc);
      }
      double ws = w, wts = wT;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        ws = ws + __shfl_xor(ws, off, 64);
        wts = wts + __shfl_xor(wts, off, 64);
      }
      if ((t & 63) == 0) {
        red[t >> 6][0] = ws;
        red[t >> 6][1] = wts;
      }
      __syncthreads();
      double wsum = red[0][0], T = red[0][1];
#pragma unroll
      for (int k = 1; k < 8; ++k) {
        wsum = wsum + red[k][0];
        T = T + red[k][1];
      }
      T = T / wsum;
      const double Pj = energy_loss(jt, T, ell, a.hbarc);
      P = Pj * wsum;
      if (cell >= 0) {
        const double s0 = Pj * w / dV;
        D[cell] = dv[0] + (R)s0;
        for (int d = 0; d < 3; ++d) D[(1 + d) * nc + cell] = dv[1 + d] + (R)(jt.dir[d] * s0);
      }
    }
    if (t == 0 && a.stage > 0) {
      if (a.stage == 3 && chi) {
        const double dep = deposit_of(j, P);
        a.s->ledger = a.s->ledger + dep;
        a.s->E_jet[j] = E - dep > 0.0 ? E - dep : 0.0;
      }
      a.s->P[a.stage - 1][j] = P;
    }
    __syncthreads();  // D and raw, red before the next jet
  }
  add_fixups(&a.s->fixups, fix);
}

template <class R>
__global__ void __launch_bounds__(512) k_jet(JetArgs a) {
  jet_body<R>(a);
}

// ---------------------------------------------------------------------------
// FP64 sums of the five fields, fixed order: per-block partials, then one block.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

template <class R>
__device__ __forceinline__ void sums_partial_body(const R* __restrict__ U, long long nc, double* part, int b, int nb) {
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (long long i = (long long)b * blockDim.x + threadIdx.x; i < nc; i += (long long)nb * blockDim.x) {
#pragma unroll
    for (int c = 0; c < 5; ++c) acc[c] += (double)U[c * nc + i];
  }
  __shared__ double red[5][4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    const double v = wave_sum(acc[c]);
    if (lane == 0) red[c][wv] = v;
  }
  __syncthreads();
  if (threadIdx.x < 5) {
    const int c = threadIdx.x;
    part[(long long)b * 5 + c] = (red[c][0] + red[c][1]) + (red[c][2] + red[c][3]);
  }
}

template <class R>
__global__ void __launch_bounds__(256) k_sums_partial(const R* __restrict__ U, long long nc, double* part) {
  sums_partial_body<R>(U, nc, part, blockIdx.x, gridDim.x);
}

__device__ __forceinline__ void sums_final_body(const double* part, int nblocks, double dV, double* sums) {
  __shared__ double red[5][4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int c = 0; c < 5; ++c) {
    double acc = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) acc += part[(long long)b * 5 + c];
    const double v = wave_sum(acc);
    if (lane == 0) red[c][wv] = v;
  }
  __syncthreads();
  if (threadIdx.x < 5) {
    const int c = threadIdx.x;
    sums[c] = ((red[c][0] + red[c][1]) + (red[c][2] + red[c][3])) * dV;
  }
}

__global__ void __launch_bounds__(256) k_sums_final(const double* part, int nblocks, double dV, double* sums) {
  sums_final_body(part, nblocks, dV, sums);
}

// ---------------------------------------------------------------------------
// Primitive (e, vx, vy, vz, n; FP64) -> conserved: E = (e+p) g^2 - p,
// M = (e+p) g^2 v, N = n g, p = e/3.
template <class R>
__global__ void __launch_bounds__(256) k_prim_to_cons(const double* __restrict__ prim, R* __restrict__ U, long long nc) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nc) return;
  const double e = prim[q], v0 = prim[nc + q], v1 = prim[2 * nc + q], v2 = prim[3 * nc + q], n = prim[4 * nc + q];
  const double v2s = v0 * v0 + v1 * v1 + v2 * v2;
  const double g2 = 1.0 / (1.0 - v2s);
  const double p = e / 3.0;
  const double w = (e + p) * g2;
  U[q] = (R)(w - p);
  U[nc + q] = (R)(w * v0);
  U[2 * nc + q] = (R)(w * v1);
  U[3 * nc + q] = (R)(w * v2);
  U[4 * nc + q] = (R)(n * sqrt(g2));
}

// Conserved -> (e, vx, vy, vz, n, T) in the field type.
template <class R>
__global__ void __launch_bounds__(256) k_primitives(const R* __restrict__ U, R* __restrict__ prim, long long nc,
                                                    double g, double hc, unsigned long long* fixups) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  unsigned fix = 0;
  if (q < nc) {
    R u[5];
    load5(U, nc, q, u);
    const PrimV pv = c2p(u, fix);
    const double v2 = pv.v[0] * pv.v[0] + pv.v[1] * pv.v[1] + pv.v[2] * pv.v[2];
    prim[q] = (R)pv.e;
    prim[nc + q] = (R)pv.v[0];
    prim[2 * nc + q] = (R)pv.v[1];
    prim[3 * nc + q] = (R)pv.v[2];
    prim[4 * nc + q] = (R)((double)u[4] * sqrt(1.0 - v2));
    prim[5 * nc + q] = (R)temperature(pv.e, g, hc);
  }
  add_fixups(fixups, fix);
}

// ---------------------------------------------------------------------------
// Batched stage kernels.  Each workgroup walks the work items blockIdx.x,
// blockIdx.x + gridDim.x, ... (persistent when the grid is smaller than the
// item count); an item is one tile of one event and runs the same body as the
// single-event kernel, so every face has the same arithmetic.
__device__ __forceinline__ int batch_event_of(const long long* off, int n, long long item) {
  int lo = 0, hi = n;  // off[lo] <= item < off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= item) lo = mid;
    else hi = mid;
  }
  return lo;
}

template <class R, int S>
__device__ __forceinline__ StageArgs<R> batch_stage_args(const BatchEvent& ev, int stage, R eps, int AX) {
  StageArgs<R> a;
  R* U = static_cast<R*>(ev.U);
  R* U1 = static_cast<R*>(ev.U1);
  R* U2 = static_cast<R*>(ev.U2);
  a.W = (stage <= 1) ? U : (stage == 2 ? U1 : U2);
  a.Un = U;
  a.out = (stage <= 1) ? U1 : (stage == 2 ? U2 : U);
  a.D = static_cast<R*>(ev.D);
  a.g = ev.g;
  a.order = 0;
  a.dt = (R)ev.dt;
  a.eps = eps;
  face_scale<R, S>(a, ev.inv_d[AX]);
  a.stage = stage;
  a.seg = 0;
  a.fixups = &ev.dev->fixups;
  a.pp_mu = ev.pp_mu;
  a.musta_k = ev.musta_k;
  return a;
}

__device__ __forceinline__ double batch_stage_time(const BatchEvent& ev, long long step, int stage) {
  const double tn = ev.t0 + (double)step * ev.dt;
  const double c = stage == 2 ? 1.0 : (stage == 3 ? 0.5 : 0.0);
  return tn + c * ev.dt;
}

// Line tiles of every event (line_body; tile length 31 or 32 by event).  PERSIST:
// workgroups walk items blockIdx.x, blockIdx.x + gridDim.x, ...; otherwise one
// item per workgroup (the loop's live state costs ~20 VGPRs, a workgroup per CU).
template <class R, int S, int AX, int A>
__device__ __forceinline__ void bline_item(const BatchArgs<R>& b, const BatchEvent& ev, long long local, R* s) {
  const StageArgs<R> a = batch_stage_args<R, S>(ev, b.stage, b.eps, AX);
  const int T = (ev.g.n[AX] + A - 1) / A;
  const int gx = AX == 0 ? ev.xside : (ev.g.n[0] + kLineX - 1) / kLineX;
  const int bx = (int)(local % gx), by = (int)((local / gx) % T), bz = (int)(local / ((long long)gx * T));
  line_body<R, S, AX, AX == 2, A>(a, AX == 0 ? bx + gx * bz : bx, by, bz, s);
}

// A: the tile length of every event along the axis, 0 where they differ.
template <class R, int S, int AX, int A, bool PERSIST>
__global__ void __launch_bounds__(kLineBlock) k_bline(BatchArgs<R> b) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  R* s = reinterpret_cast<R*>(smem_raw);
  auto item = [&](long long it) {
    if (sizeof(R) == 4) {  // contiguous parts to the XCDs, as in launch_line_t
      const long long per = b.items >> 3;
      if (it < 8 * per) it = (it & 7) * per + (it >> 3);
    }
    const int e = batch_event_of(b.off, b.n_events, it);
    const BatchEvent& ev = b.ev[e];
    const long long local = it - b.off[e];
    if constexpr (A != 0) {
      bline_item<R, S, AX, A>(b, ev, local, s);
    } else {
      if (tile_len(ev.g.n[AX]) == 31) bline_item<R, S, AX, 31>(b, ev, local, s);
      else bline_item<R, S, AX, 32>(b, ev, local, s);
    }
  };
  if constexpr (PERSIST) {
    for (long long it = blockIdx.x; it < b.items; it += gridDim.x) {
      item(it);
      __syncthreads();  // the next item overwrites the LDS tile
    }
  } else {
    if ((long long)blockIdx.x < b.items) item(blockIdx.x);  // uniform
  }
}

template <class R>
__global__ void __launch_bounds__(512) k_bjet(BatchArgs<R> b) {
  const BatchEvent& ev = b.ev[blockIdx.x];
  if (ev.njet == 0) return;  // whole workgroup
  const int stage = b.stage;
  JetArgs j;
  j.W = (stage <= 1) ? ev.U : (stage == 2 ? ev.U1 : ev.U2);
  j.D = ev.D;
  j.s = ev.dev;
  j.g = ev.g;
  j.njet = ev.njet;
  j.stage = stage;
  j.deposit = ev.deposit;
  j.t = batch_stage_time(ev, *b.step, stage);
  j.dt = ev.dt;
  j.eos_dof = ev.eos_dof;
  j.hbarc = ev.hbarc;
  jet_body<R>(j);
}

// FP64 conservation sums of every event (grid kSumBlocks x n_events, then n_events).
template <class R>
__global__ void __launch_bounds__(256) k_bsums_partial(BatchArgs<R> b) {
  const BatchEvent& ev = b.ev[blockIdx.y];
  sums_partial_body<R>(static_cast<const R*>(ev.U), ev.g.nc, ev.part, blockIdx.x, gridDim.x);
}

template <class R>
__global__ void __launch_bounds__(256) k_bsums_final(BatchArgs<R> b) {
  const BatchEvent& ev = b.ev[blockIdx.x];
  sums_final_body(ev.part, kSumBlocks, ev.dV, ev.dev->sums);
}

__global__ void k_bstep(long long* step) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *step = *step + 1;
}

// ---------------------------------------------------------------------------
// Host-side launchers (called from hydro_api.hip).
// Line tiles along AX.
template <class R, int S, int AX>
void launch_line_t(const StageArgs<R>& base, hipStream_t st) {
  StageArgs<R> a = base;
  face_scale<R, S>(a, 1.0 / a.g.dx[AX]);
  const int n = a.g.n[AX];
  // Up to 15 cells, tiles of 15: marching 32 face rows for a few of them took,
  // us a launch in FP64, z at 256x256x1 52 (30 with a lane per face), x at
  // 1x256x256 59 (27); tiles of 15 take 22 and 24.
  const int A = n <= 15 ? 15 : tile_len(n);
  a.order = AX == 0 ? 0 : (base.order >> (AX - 1)) & 1;
  const LineGroups lg = line_groups(AX, a.g);
  dim3 grid(lg.x, (n + A - 1) / A, lg.z);
  if (a.order) grid = dim3(grid.x, grid.z, grid.y);
  // FP32: 16 cells are half a cache line, so the workgroups that share lines,
  // dealt round-robin over the eight XCDs as they are, fetch them into several
  // L2s; a plane's workgroups go to the XCDs in contiguous parts instead (z at
  // 256^3: 467 -> 417 us; y and x, whose neighbours run side by side anyway,
  // 1 % slower; FP64 z 709 -> 726)
  const bool xcd = sizeof(R) == 4 && AX == 2 && grid.x > 1 && (unsigned long long)grid.x * grid.x * grid.y < 0xffffffffULL;
  a.seg = xcd ? (int)((0x100000000ULL + grid.x - 1) / grid.x) : 0;
  const size_t lds = line_lds_bytes(AX, A, S, (int)sizeof(R));
  if (A == 15) hipLaunchKernelGGL((k_line<R, S, AX, AX == 2, 15>), grid, dim3(kLineBlock / 2), lds, st, a);
  else if (A == 31) hipLaunchKernelGGL((k_line<R, S, AX, AX == 2, 31>), grid, dim3(kLineBlock), lds, st, a);
  else hipLaunchKernelGGL((k_line<R, S, AX, AX == 2, 32>), grid, dim3(kLineBlock), lds, st, a);
}

template <class R, int S, int AX>
void launch_march_t(const StageArgs<R>& base, int seg, hipStream_t st) {
  StageArgs<R> a = base;
  const int nx = a.g.n[0], ny = a.g.n[1], nz = a.g.n[2];
  a.seg = seg;
  face_scale<R, S>(a, 1.0 / a.g.dx[AX]);
  const int n = (AX == 1) ? ny : nz;
  const int no = (AX == 1) ? nz : ny;
  dim3 grid((nx + 63) / 64, (no + 3) / 4, (n + seg - 1) / seg);
  hipLaunchKernelGGL((k_march<R, S, AX, AX == 2>), grid, dim3(64, 4), 0, st, a);
}

// kernel: 0 x faces, 1 y, 2 z (+ combine), 3 y-march, 4 z-march (+ combine)
template <class R>
hipError_t launch_face_kernel(int kernel, const StageArgs<R>& a, int scheme, int seg, hipStream_t st) {
#define HYDRO_DISPATCH(S)                                  \
  switch (kernel) {                                        \
    case 0: launch_line_t<R, S, 0>(a, st); break;          \
    case 1: launch_line_t<R, S, 1>(a, st); break;          \
    case 2: launch_line_t<R, S, 2>(a, st); break;          \
    case 3: launch_march_t<R, S, 1>(a, seg, st); break;    \
    default: launch_march_t<R, S, 2>(a, seg, st); break;   \
  }
  switch (scheme) {
    case kWenoJS: HYDRO_DISPATCH(kWenoJS) break;
    case kWenoLinear: HYDRO_DISPATCH(kWenoLinear) break;
    case kWeno5Z: HYDRO_DISPATCH(kWeno5Z) break;
    case kWeno5JS: HYDRO_DISPATCH(kWeno5JS) break;
    case kWeno5Linear: HYDRO_DISPATCH(kWeno5Linear) break;
    case kWenoZ | kPP: HYDRO_DISPATCH(kWenoZ | kPP) break;
    case kWenoJS | kPP: HYDRO_DISPATCH(kWenoJS | kPP) break;
    case kWenoLinear | kPP: HYDRO_DISPATCH(kWenoLinear | kPP) break;
    case kWeno5Z | kPP: HYDRO_DISPATCH(kWeno5Z | kPP) break;
    case kWeno5JS | kPP: HYDRO_DISPATCH(kWeno5JS | kPP) break;
    case kWeno5Linear | kPP: HYDRO_DISPATCH(kWeno5Linear | kPP) break;
    case kWenoZ | kMusta: HYDRO_DISPATCH(kWenoZ | kMusta) break;
    case kWeno5Z | kMusta: HYDRO_DISPATCH(kWeno5Z | kMusta) break;
    default: HYDRO_DISPATCH(kWenoZ) break;
  }
#undef HYDRO_DISPATCH
  return hipGetLastError();
}

template <class R>
hipError_t launch_jet(const JetArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((k_jet<R>), dim3(1), dim3(512), 0, st, a);
  return hipGetLastError();
}

template <class R>
hipError_t launch_sums(const R* U, long long nc, double dV, double* part, double* sums, hipStream_t st) {
  hipLaunchKernelGGL((k_sums_partial<R>), dim3(kSumBlocks), dim3(256), 0, st, U, nc, part);
  hipLaunchKernelGGL(k_sums_final, dim3(1), dim3(256), 0, st, part, kSumBlocks, dV, sums);
  return hipGetLastError();
}

template <class R>
hipError_t launch_prim_to_cons(const double* prim, R* U, long long nc, hipStream_t st) {
  const unsigned nb = (unsigned)((nc + 255) / 256);
  hipLaunchKernelGGL((k_prim_to_cons<R>), dim3(nb), dim3(256), 0, st, prim, U, nc);
  return hipGetLastError();
}

template <class R>
hipError_t launch_primitives(const R* U, R* prim, long long nc, double g, double hc, unsigned long long* fixups,
                             hipStream_t st) {
  const unsigned nb = (unsigned)((nc + 255) / 256);
  hipLaunchKernelGGL((k_primitives<R>), dim3(nb), dim3(256), 0, st, U, prim, nc, g, hc, fixups);
  return hipGetLastError();
}

// Work items of one event for the batched launches: the tiles of an axis.
long long batch_items(int AX, const Grid& g) {
  const int A = tile_len(g.n[AX]);
  const LineGroups lg = line_groups(AX, g);
  return (long long)((g.n[AX] + A - 1) / A) * lg.x * lg.z;
}

template <class R, int S, int AX>
void launch_bline_ax(bool persist, dim3 grid, const BatchArgs<R>& b, hipStream_t st) {
  const dim3 tb(kLineBlock);
  const size_t lds = line_lds_bytes(AX, b.tile_a == 31 ? 31 : 32, S, (int)sizeof(R));
  if (b.tile_a == 31) {
    if (persist) hipLaunchKernelGGL((k_bline<R, S, AX, 31, true>), grid, tb, lds, st, b);
    else hipLaunchKernelGGL((k_bline<R, S, AX, 31, false>), grid, tb, lds, st, b);
  } else if (b.tile_a == 32) {
    if (persist) hipLaunchKernelGGL((k_bline<R, S, AX, 32, true>), grid, tb, lds, st, b);
    else hipLaunchKernelGGL((k_bline<R, S, AX, 32, false>), grid, tb, lds, st, b);
  } else {
    hipLaunchKernelGGL((k_bline<R, S, AX, 0, true>), grid, tb, lds, st, b);
  }
}

template <class R, int S>
void launch_bline(int AX, bool persist, dim3 grid, const BatchArgs<R>& b, hipStream_t st) {
  if (AX == 0) launch_bline_ax<R, S, 0>(persist, grid, b, st);
  if (AX == 1) launch_bline_ax<R, S, 1>(persist, grid, b, st);
  if (AX == 2) launch_bline_ax<R, S, 2>(persist, grid, b, st);
}

// blocks: workgroups of the launch (0: one per item).
template <class R>
hipError_t launch_batch_axis(int AX, const BatchArgs<R>& b, int scheme, long long blocks, hipStream_t st) {
  const long long nb = batch_grid(b.items, blocks);
  if (nb <= 0) return hipSuccess;
  const dim3 grid((unsigned)nb);
  const bool persist = nb < b.items;
  switch (scheme) {
    case kWenoJS: launch_bline<R, kWenoJS>(AX, persist, grid, b, st); break;
    case kWenoLinear: launch_bline<R, kWenoLinear>(AX, persist, grid, b, st); break;
    case kWeno5Z: launch_bline<R, kWeno5Z>(AX, persist, grid, b, st); break;
    case kWeno5JS: launch_bline<R, kWeno5JS>(AX, persist, grid, b, st); break;
    case kWeno5Linear: launch_bline<R, kWeno5Linear>(AX, persist, grid, b, st); break;
    case kWenoZ | kPP: launch_bline<R, (kWenoZ | kPP)>(AX, persist, grid, b, st); break;
    case kWenoJS | kPP: launch_bline<R, (kWenoJS | kPP)>(AX, persist, grid, b, st); break;
    case kWenoLinear | kPP: launch_bline<R, (kWenoLinear | kPP)>(AX, persist, grid, b, st); break;
    case kWeno5Z | kPP: launch_bline<R, (kWeno5Z | kPP)>(AX, persist, grid, b, st); break;
    case kWeno5JS | kPP: launch_bline<R, (kWeno5JS | kPP)>(AX, persist, grid, b, st); break;
    case kWeno5Linear | kPP: launch_bline<R, (kWeno5Linear | kPP)>(AX, persist, grid, b, st); break;
    case kWenoZ | kMusta: launch_bline<R, (kWenoZ | kMusta)>(AX, persist, grid, b, st); break;
    case kWeno5Z | kMusta: launch_bline<R, (kWeno5Z | kMusta)>(AX, persist, grid, b, st); break;
    default: launch_bline<R, kWenoZ>(AX, persist, grid, b, st); break;
  }
  return hipGetLastError();
}

template <class R>
hipError_t launch_batch_jet(const BatchArgs<R>& b, hipStream_t st) {
  hipLaunchKernelGGL((k_bjet<R>), dim3(b.n_events), dim3(512), 0, st, b);
  return hipGetLastError();
}

template <class R>
hipError_t launch_batch_sums(const BatchArgs<R>& b, long long* step, hipStream_t st) {
  hipLaunchKernelGGL((k_bsums_partial<R>), dim3(kSumBlocks, b.n_events), dim3(256), 0, st, b);
  hipLaunchKernelGGL((k_bsums_final<R>), dim3(b.n_events), dim3(256), 0, st, b);
  if (step) hipLaunchKernelGGL(k_bstep, dim3(1), dim3(64), 0, st, step);
  return hipGetLastError();
}

#define HYDRO_INSTANTIATE(R)                                                                          \
  template hipError_t launch_batch_axis<R>(int, const BatchArgs<R>&, int, long long, hipStream_t);      \
  template hipError_t launch_batch_jet<R>(const BatchArgs<R>&, hipStream_t);                          \
  template hipError_t launch_batch_sums<R>(const BatchArgs<R>&, long long*, hipStream_t);              \
  template hipError_t launch_face_kernel<R>(int, const StageArgs<R>&, int, int, hipStream_t);          \
  template hipError_t launch_jet<R>(const JetArgs&, hipStream_t);                                     \
  template hipError_t launch_sums<R>(const R*, long long, double, double*, double*, hipStream_t);     \
  template hipError_t launch_prim_to_cons<R>(const double*, R*, long long, hipStream_t);              \
  template hipError_t launch_primitives<R>(const R*, R*, long long, double, double, unsigned long long*, hipStream_t);

HYDRO_INSTANTIATE(double)
HYDRO_INSTANTIATE(float)

}  // namespace hydro
