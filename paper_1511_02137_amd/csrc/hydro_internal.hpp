// hydro_internal.hpp -- structures shared by the host part of libhydro and
// its HIP kernels.  Not part of the public ABI (see include/hydro.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hydro {

constexpr int kMaxJets = 64;       // jets per context
constexpr double kEFloor = 1e-12;  // E at or below: vacuum fix-up
constexpr double kVCap = 1.0 - 1e-10;  // |v| cap of the fix-up
constexpr int kSumBlocks = 1024;   // fixed number of reduction blocks (fixed order)

// WENO7 with Z, Jiang-Shu or linear weights; 3..5: the same for WENO5.
enum Scheme { kWenoZ = 0, kWenoJS = 1, kWenoLinear = 2, kWeno5Z = 3, kWeno5JS = 4, kWeno5Linear = 5 };
// Flag on the face kernels' scheme template argument: positivity-preserving
// flux limiter on.
constexpr int kPP = 8;
// Flag on the same argument: MUSTA-FORCE face fluxes of WENO-reconstructed
// conserved states instead of WENO of the Lax-Friedrichs split fluxes.
constexpr int kMusta = 16;

// Grid of one event.
struct Grid {
  int n[3];        // nx, ny, nz
  int bc[3];       // 0 outflow, 1 periodic
  double dx[3];    // cell widths
  long long nc;    // nx*ny*nz
};

// Static description of a jet on the device (FP64).
struct JetDev {
  double x0[3];
  double dir[3];
  double t_start;
  double kappa_rad, kappa_coll, crcf;
};

// Per-context device scalars (library-owned, a few KB).
struct DevScalars {
  JetDev jets[kMaxJets];
  double E_jet[kMaxJets];     // remaining energy
  double P[3][kMaxJets];      // deposited rate of each stage of the current step
  double ledger;              // deposited energy so far
  double sums[5];             // conservation sums (x dV) of the last hydro_sums call
  double step_sums[5];        // conservation sums (x dV) taken by the last RK3 step
  unsigned long long fixups;  // conserved->primitive fix-ups
  unsigned long long fixups_save;  // fixups on entry to an adjoint sweep (restored on exit)
};

// Arguments of the stage kernels (device pointers).
template <class R>
struct StageArgs {
  const R* W;   // stage input [5][nc]
  const R* Un;  // U^n (stages 2 and 3)
  R* out;       // stage output (may alias Un in stage 3)
  R* D;         // flux divergence accumulator [5][nc]
  Grid g;
  R inv_d;      // 1/dx of the kernel's axis
  R dt;
  R eps;        // epsilon of the WENO weights
  int stage;    // 1, 2, 3 (RK stage); 0: write L = D + S instead of combining
  int seg;      // march segment length (y/z kernels)
  int order;    // LDS tiles: bit AX-1 set = blockIdx.y runs over the transverse axis, blockIdx.z over the tiles
  unsigned long long* fixups;
  double pp_mu;  // 2 dt sum_d 1/dx_d, the half-state factor of the positivity limiter
  int musta_k;   // MUSTA-FORCE stages
};

// Arguments of the jet kernel.
struct JetArgs {
  const void* W;   // stage input
  void* D;         // divergence accumulator (source is added)
  DevScalars* s;
  Grid g;
  int njet;
  int stage;       // 1, 2, 3 (stage 3 also advances E_jet and the ledger); 0: RHS only
  int deposit;     // 0 NGP, 1 Gauss
  double t;        // stage time
  double dt;
  double eos_dof, hbarc;
};

// Cells per LDS tile along the reconstructed axis: 31 (32 face rows, four runs of
// eight) unless 32-cell tiles (33 face rows, the last one by lanes beside the
// runs) are fewer by more than they cost: 3 to 8 % a tile, MUSTA-FORCE 13 %
// (FP64, z at 128 x 128 x n, us with 31 and with 32: n = 62 37.1 and 37.8, n = 64
// 48.1 and 38.4; MUSTA-FORCE 42.5 and 46.1, 55.1 and 47.9).
__host__ __device__ constexpr int tile_len(int n) {
  return (n + 30) / 31 * 100 > 109 * ((n + 31) / 32) ? 32 : 31;
}

// Line tiles: 16 lines of A + 8 points for each (field, split), and with the
// limiter A + 1 face fluxes for each field.
constexpr int kLineX = 16;
// Face rows that a tile marches over, a lane each in a workgroup of 16 of them.
__host__ __device__ constexpr int line_rows(int A) { return A == 32 ? 32 : A + 1; }
// Groups of 16 lines of a grid: x in groups of rows, whatever their y and z, up
// to 16 groups side by side (a tile of the same rows follows soon after, while
// their cache lines last) as evenly dealt as they go; y and z along x at each
// value of the remaining axis.
struct LineGroups {
  int x, z;
};
inline LineGroups line_groups(int AX, const Grid& g) {
  if (AX != 0) return {(g.n[0] + kLineX - 1) / kLineX, g.n[AX == 1 ? 2 : 1]};
  const long long groups = ((long long)g.n[1] * g.n[2] + kLineX - 1) / kLineX;
  const long long side = groups <= 16LL * 65535 ? 16 : (groups + 65534) / 65535;
  const long long z = (groups + side - 1) / side;
  return {(int)((groups + z - 1) / z), (int)z};
}
__host__ __device__ constexpr size_t line_lds_bytes(int AX, int A, int scheme, int elem) {
  return (size_t)(10 * (A + 8) + ((scheme & kPP) ? 5 * (A + 1) : 0)) * (AX == 0 ? kLineX + 1 : kLineX) * elem;
}

// Lanes of a line-tile workgroup, and workgroups of a batched axis launch: one
// per item (blocks 0), or `blocks` that walk the items.  A launch holds fewer
// than 2^32 lanes, 8388607 workgroups; thin events (an item of one cell) have
// more items than that long before memory ends, and a grid of that many walks.
constexpr int kLineBlock = 512;
__host__ __device__ constexpr long long batch_grid(long long items, long long blocks) {
  const long long nb = (blocks <= 0 || blocks > items) ? items : blocks, most = 0xffffffffLL / kLineBlock;
  return nb < most ? nb : most;
}

// One event of a batch (device table, see hydro_batch.hip).
struct BatchEvent {
  Grid g;
  void* U;            // caller's state [5][nc]
  void* U1;           // stage states and divergence (workspace)
  void* U2;
  void* D;
  double* part;       // reduction partials [kSumBlocks][5]
  DevScalars* dev;    // jets, E_jet, ledger, sums, fix-ups
  double t0, dt;
  double inv_d[3];    // 1/dx per axis
  double dV;
  double eos_dof, hbarc;
  double pp_mu;       // 2 dt sum_d 1/dx_d (positivity limiter)
  int musta_k;        // MUSTA-FORCE stages
  int xside;          // line_groups(0, g).x
  int njet;
  int deposit;
};

// Arguments of the batched kernels: the work items of one axis are the tiles
// of every event in event order; off[e] is the first item of event e.
template <class R>
struct BatchArgs {
  const BatchEvent* ev;
  const long long* off;   // [n_events + 1] for the launched axis
  long long items;        // off[n_events]
  const long long* step;  // device step counter (stage times)
  int n_events;
  int stage;              // 1..3; 0: L written to U1 (no state change)
  R eps;
  int tile_a;             // 31 or 32: every event's tile length along the launched axis (0: they differ)
};

// Arguments of the line adjoint kernels (device pointers).
template <class R>
struct AdjArgs {
  const R* W;   // stage input
  const R* mu;  // adjoint of the stage output (lambda_Y)
  R* G;         // (dL/dW)^T mu accumulator [5][nc]
  Grid g;
  R inv_d;      // 1/dx of the kernel's axis (set by the launcher)
  R eps;        // epsilon of the WENO weights
  int first;    // 1: G = contribution, 0: G += contribution
  unsigned long long* fixups;
  // RK combine in reverse, fused into the last axis (stage 0: none, G is
  // stored).  With b_k the stage weight of W and a_k that of U^n:
  //   lW = b_k (mu + dt G), acc (adjoint of U^n) += a_k mu; stage 1: lW = acc + mu + dt G.
  int stage;
  R dt;
  R* acc;
  R* lW;
  // 1: the N component of mu is taken as zero; N's reverse reconstructions are
  // skipped and its outputs (G, lW, acc) are zero.  N enters no other field's
  // flux and no source, so with a zero N adjoint on entry this is exact.
  int skip_n;
  // most lines per workgroup asked for by the caller (0: no limit; 1, 2 or 4):
  // kept where that costs no time, else the launcher takes what is fastest
  int lines;
  int seglen;  // cells of a line's segments (set by the launcher for the SEG form)
};

// Bound on the adjoint's axis lengths (hydro_workspace_bytes): elements of the
// field type that must fit 64 KiB.
constexpr long long line_adj_lds_elems(int n) { return 10LL * (n + 8) + 14LL * (n + 16); }
// Line adjoint: LDS slots of a line of nf faces in runs of L (the last run's
// values included), words between slots (x with eight lines: one more, so that a
// wave's cells of a row fall in different banks, 25.7 -> 24.6 us at 60x52x66 in
// FP64; two and four lines lose nothing without it and more workgroups share a CU:
// with five fields 256x64x256 FP64 738 -> 556 us, 128x128x128 FP64 380 -> 267, FP32
// 166 -> 140), bytes of the two areas of each field, of the
// six values a line that pass from a turn to the next, and of phi.
// Workgroups: with 128 VGPRs in FP64 two of eight waves share a CU (four lines
// in four waves, with half the LDS and loads half as wide, were 1.2x slower at
// 60x52x66); FP32 takes four waves, five workgroups a CU (eight waves of eight
// lines: 112 against 107 us an axis at 128^3).
__host__ __device__ constexpr int line_adj_block(int elem) { return elem == 8 ? 512 : 256; }
__host__ __device__ constexpr int line_adj_slots(int nf, int L) { return (nf + L - 1) / L * L + 7; }
__host__ __device__ constexpr int line_adj_pitch(int AX, int lines) { return AX == 0 && lines > 4 ? lines + 1 : lines; }
// phi rows: the faces and zeros up to a run's length less one on each side
__host__ __device__ constexpr int line_adj_phi_rows(int nf, int L) { return 2 * ((nf + L - 1) / L * L) - nf; }
__host__ __device__ constexpr size_t line_adj_lds_bytes(int AX, int nf, int L, int lines, int fields, int elem) {
  return (size_t)fields * ((2 * line_adj_slots(nf, L) + line_adj_phi_rows(nf, L)) * line_adj_pitch(AX, lines) +
                           12 * lines) * elem;
}

// Arguments of the jet-source adjoint kernel.
struct JetAdjArgs {
  const void* W;        // stage input
  const void* mu;       // adjoint of the stage output
  void* G;              // accumulator
  DevScalars* s;
  const double* Ehist;  // jet energies at the start of the step [kMaxJets]
  double* grad;         // parameter gradients [njet][5] (+=)
  Grid g;
  int njet;
  int deposit;
  double t;             // stage time
  double bdt;           // b_k * dt of the stage
  double eos_dof, hbarc;
};

// Freeze-out spectra (hydro_freezeout): limits and arguments.
constexpr int kFoThreads = 256;           // lanes per workgroup
constexpr int kFoMaxOut = 1024;           // (1 + n_pt) * n_phi outputs
constexpr int kFoOutPerLane = kFoMaxOut / kFoThreads;
constexpr int kFoMaxPt = 15;              // p_T values of the differential rows
constexpr int kFoMaxHarm = 32;            // harmonics n = 1..n_harm
constexpr int kFoBlocks = 1024;           // workgroups of the partial-sum pass (fixed order)

template <class R>
struct FreezeArgs {
  const R* U;
  long long nc;
  int n_phi;             // azimuths phi_k = 2 pi k / n_phi
  int rows;              // 1 + n_pt
  int n_out;             // rows * n_phi
  int groups;            // lane groups sharing one set of outputs (n_out <= kFoThreads / groups)
  double pt[kFoMaxPt];   // p_T of rows 1..
  double smax[kFoMaxPt]; // 2^30 / p_T (set by the launcher)
  double T_min;          // cells with T < T_min are left out
  double pref_dV;        // g dV / (2 pi hbar c)^3
  double eos_dof, hbarc; // T(e) of the fluid
  double* part;          // [kFoBlocks][n_out] partial sums
  unsigned long long* fixups;
};

}  // namespace hydro
