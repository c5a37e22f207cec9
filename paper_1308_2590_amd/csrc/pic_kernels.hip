// HIP kernels (gfx950) of the implicit 2D3V PIC particle stage.
//
// Field solve (FP64, one thread per node / cell):
//   k_solve_e   Eq. (4) per node: E_new = (I + S)^{-1}[(I - S)E + dt(curl H - dj)] with curl H
//               from the 2x2 neighbouring cells (Sec. 3.3 Step 5); on an absorbing x axis the
//               thread of the inner node next to a boundary node also applies the first-order
//               Mur condition to E - E_inc there (Steps 3, 4, 6).  Moments are read, then
//               cleared for the next deposit, only where the deposit flags say so.
//   k_update_h  Eq. (5) at cell centres with curl E from the 4 corner nodes (Steps 8-9), and
//               clears the deposit flags.
// Particles (one block per tile of cells; a wavefront takes groups of 64 consecutive slots of the
// tile's rows, or a row of the tile where cells hold few particles and in mixed precision):
//   k_particles gather E-bar (bilinear from the 4 corner nodes) and B (the particle's cell),
//               implicit push (Eq. (2a) solved for the time-centred momentum), position
//               advance, move code, then deposit of S-hat, delta-j and density (Step 1,
//               Eq. (3)) at the new position into LDS accumulators covering the tile plus a
//               halo, folded once per tile into the FP64 moment planes with global atomics.
//               It also counts the particles leaving each cell per move code and arriving in
//               each cell.  Grouped or direct form, FP64 and mixed (FP32 particles); mixed runs alone
//               take the direct form or
//   k_particles_runs  lane runs (pic_runs.h).
// Sort (stable by cell, removed particles dropped):
//   k_scan      exclusive scan of the arrival counts -> next cell start offsets, and flags of
//               the tiles holding particles in the next order;
//   k_tile_flags / k_tile_compact  the same flags and the ordered tile list from cell starts
//               (after loads);
//   k_rank / k_rank_cells  stable destination of every particle: cell start + particles arriving from
//               source cells with a smaller key + rank within (source cell, move code),
//               written as the next cycle's slot -> location permutation; one extra block
//               makes the next order's tile list.
// Positions never move more than one cell per cycle because dt <= min(dx, dz) and |v| < c,
// which is what keeps the sort a 3x3 neighbourhood redistribution.
//
// The file is compiled with -ffp-contract=off: fused multiply-adds appear only where written.
// The FP64 mover evaluates the same expressions as a plain implementation of the method up to
// rounding (vector form of the response, Newton-refined reciprocals), so FP64 results agree
// with the oracle to about 1e-15 relative per cycle.

#include <algorithm>
#include <type_traits>

#include "pic_device.h"
#include "pic_internal.h"
#include "pic_runs.h"

namespace pic {
namespace {

// ------------------------------------------------------------------------------------------
// Field solve
// ------------------------------------------------------------------------------------------

// The incident E_y at (t, x, z) is source_s(t - x) exp(-sz^2 / 2) source_e(t - x): Step 4 needs it at
// two times and two columns, the same for every node but for the factor of z.
__device__ __forceinline__ double source_s(const LaserArgs &L, double tau) { return L.a0 * sin(L.omega * tau); }
__device__ __forceinline__ double source_e(const LaserArgs &L, double tau) {
  const double st = (tau - L.t_center) / L.fwhm_t;
  return exp(-2.0 * 0.6931471805599453 * st * st);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Whether the moment planes of node n can hold a deposit: the flag of its run of kFlagNodes
// nodes.  Elsewhere the planes are zero.
__device__ __forceinline__ bool node_deposited(const FieldArgs &a, int64_t n) {
  return !a.mflag || a.mflag[n / kFlagNodes] != 0;
}

// Zero every moment plane of node n once its values have been read, so the next deposit
// starts from zero.  Each node is read and cleared by one thread.
__device__ __forceinline__ void clear_node_moments(const FieldArgs &a, int64_t n) {
  for (int p = 0; p < a.g.n_planes; ++p) a.M[p * a.g.nnodes + n] = 0.0;
}

// Inputs of Eq. (4) at the node (i, k), i an interior column: curl H from the 2x2 cells
// around the node, E^n, and S-hat and delta-j where a deposit can have reached the node (zero
// elsewhere).  Loads only: a thread gathers the inputs of all its nodes before its first
// store (the compiler cannot tell the planes apart, so a load after a store waits for it).
struct NodeIn {
  double curl[3], e[3], S[9], J[3];
  int64_t n;
  bool dep;
};

__device__ __forceinline__ void node_load(const FieldArgs &a, int i, int k, NodeIn &in) {
  const GridArgs &g = a.g;
  const int nx = g.nx, nz = g.nz;
  const int64_t nn = g.nnodes, nc = g.ncells;
  int iR = wrap1(i, nx), iL = wrap1(i - 1, nx);
  int kU = wrap1(k, nz), kD = wrap1(k - 1, nz);
  int64_t cUR = (int64_t)kU * nx + iR, cUL = (int64_t)kU * nx + iL;
  int64_t cDR = (int64_t)kD * nx + iR, cDL = (int64_t)kD * nx + iL;
  const double *Hx = a.H, *Hy = a.H + nc, *Hz = a.H + 2 * nc;
  double dHx_dz = ((Hx[cUR] + Hx[cUL]) - (Hx[cDR] + Hx[cDL])) * a.r2dz;
  double dHy_dz = ((Hy[cUR] + Hy[cUL]) - (Hy[cDR] + Hy[cDL])) * a.r2dz;
  double dHy_dx = ((Hy[cUR] + Hy[cDR]) - (Hy[cUL] + Hy[cDL])) * a.r2dx;
  double dHz_dx = ((Hz[cUR] + Hz[cDR]) - (Hz[cUL] + Hz[cDL])) * a.r2dx;
  in.curl[0] = -dHy_dz;
  in.curl[1] = dHx_dz - dHz_dx;
  in.curl[2] = dHy_dx;
  const int64_t n = (int64_t)k * g.nxn + i;
  in.n = n;
#pragma unroll
  for (int r = 0; r < 3; ++r) in.e[r] = a.E[r * nn + n];
  in.dep = node_deposited(a, n);
  if (in.dep) {
#pragma unroll
    for (int r = 0; r < 9; ++r) in.S[r] = a.M[r * nn + n];
#pragma unroll
    for (int r = 0; r < 3; ++r) in.J[r] = a.M[(9 + r) * nn + n];
  } else {
#pragma unroll
    for (int r = 0; r < 9; ++r) in.S[r] = 0.0;
#pragma unroll
    for (int r = 0; r < 3; ++r) in.J[r] = 0.0;
  }
}

// Eq. (4): E^{n+1} = (I + S)^{-1} [(I - S) E^n + dt (curl H - delta-j)].
__device__ __forceinline__ void node_solve(const FieldArgs &a, const NodeIn &in, double out[3]) {
  const double dt = a.g.dt;
  const double *S = in.S, *e = in.e;
  double rhs[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    double se = S[3 * r] * e[0] + S[3 * r + 1] * e[1] + S[3 * r + 2] * e[2];
    rhs[r] = (e[r] - se) + dt * (in.curl[r] - in.J[r]);
  }
  double A[9];
#pragma unroll
  for (int r = 0; r < 9; ++r) A[r] = S[r] + ((r % 4 == 0) ? 1.0 : 0.0);
  // Cramer's rule; I + S has a positive-definite symmetric part, so det > 0.
  double c00 = A[4] * A[8] - A[5] * A[7];
  double c01 = A[5] * A[6] - A[3] * A[8];
  double c02 = A[3] * A[7] - A[4] * A[6];
  double det = A[0] * c00 + A[1] * c01 + A[2] * c02;
  double c10 = A[2] * A[7] - A[1] * A[8];
  double c11 = A[0] * A[8] - A[2] * A[6];
  double c12 = A[1] * A[6] - A[0] * A[7];
  double c20 = A[1] * A[5] - A[2] * A[4];
  double c21 = A[2] * A[3] - A[0] * A[5];
  double c22 = A[0] * A[4] - A[1] * A[3];
  const double rdet = 1.0 / det;
  out[0] = (c00 * rhs[0] + c10 * rhs[1] + c20 * rhs[2]) * rdet;
  out[1] = (c01 * rhs[0] + c11 * rhs[1] + c21 * rhs[2]) * rdet;
  out[2] = (c02 * rhs[0] + c12 * rhs[1] + c22 * rhs[2]) * rdet;
}

// E^{n+1} of node n.  (The particle kernel forms E-bar = (E^n + E^{n+1}) / 2 where it reads
// the fields.)
__device__ __forceinline__ void write_e(const FieldArgs &a, int64_t n, const double en[3]) {
  const int64_t nn = a.g.nnodes;
#pragma unroll
  for (int r = 0; r < 3; ++r) a.E_new[r * nn + n] = en[r];
}

// E^n of a boundary column's node and whether a deposit can have reached it.
struct MurIn {
  double e[3];
  bool dep;
};
__device__ __forceinline__ void mur_load(const FieldArgs &a, int64_t nb, MurIn &in) {
#pragma unroll
  for (int r = 0; r < 3; ++r) in.e[r] = a.E[r * a.g.nnodes + nb];
  in.dep = node_deposited(a, nb);
}

// Mur boundary (Step 3) at node nb of the column i = 0 or i = nx of an absorbing axis, from E^n
// (eo_in) and the new E (ein) of the inner column next to it; the x = 0 column takes the source of
// Step 4 on E_y, inc: the incident E_y at (t, 0), (t + dt, 0), (t, dx), (t + dt, dx).
__device__ __forceinline__ void mur_node(const FieldArgs &a, bool left, int64_t nb, const MurIn &b,
                                         const double eo_in[3], const double ein[3],
                                         const double inc[4]) {
  const GridArgs &g = a.g;
  const double kappa = (g.dt - g.dx) / (g.dt + g.dx);
  double en[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const bool src = left && r == 1;
    const double i00 = src ? inc[0] : 0.0, i10 = src ? inc[1] : 0.0;
    const double i01 = src ? inc[2] : 0.0, i11 = src ? inc[3] : 0.0;
    if (left)
      en[r] = i10 + (eo_in[r] - i01) + kappa * ((ein[r] - i11) - (b.e[r] - i00));
    else
      en[r] = eo_in[r] + kappa * (ein[r] - b.e[r]);
  }
  write_e(a, nb, en);
  // the boundary node takes deposits too; its planes are not used by the solve
  if (b.dep) clear_node_moments(a, nb);
}

// Nodes n0, n0 + stride, ... of the E solve (kSolveNodes per thread, their inputs loaded
// together).  On an absorbing axis the thread of the inner column next to a boundary column
// also writes that column, so every node's moments are read and cleared by a single thread (an
// absorbing axis has nx >= 2).  What the boundary needs is loaded before the first store (a load
// after stores waits for them), and the source's four times are evaluated by four lanes at once:
// one lane evaluating them in turn at the end, a sine and two exponentials each, took 5 of the 18
// us of a small slab's field solve.  They come first, where their registers are free again before
// the nodes' loads (beside them they cost a wavefront per SIMD).
__device__ __forceinline__ void solve_e_body(const FieldArgs &a, double tE, int64_t n0,
                                             int64_t stride) {
  const GridArgs &g = a.g;
  const bool absorbing = g.bc_x == PIC_BC_ABSORBING;
  NodeIn in[kSolveNodes];
  bool live[kSolveNodes];
  int ii[kSolveNodes], kk[kSolveNodes];
#pragma unroll
  for (int q = 0; q < kSolveNodes; ++q) {
    const int64_t n = n0 + q * stride;
    kk[q] = (int)(n / g.nxn);
    ii[q] = (int)(n - (int64_t)kk[q] * g.nxn);
    live[q] = n < g.nnodes && !(absorbing && (ii[q] == 0 || ii[q] == g.nx));
  }
  bool left[kSolveNodes], any_left = false;
#pragma unroll
  for (int q = 0; q < kSolveNodes; ++q) {
    left[q] = absorbing && live[q] && ii[q] == 1;
    any_left = any_left || left[q];
  }
  const bool source = a.laser.a0 != 0.0 && __any(any_left);
  double ss[4] = {0.0, 0.0, 0.0, 0.0}, se[4] = {0.0, 0.0, 0.0, 0.0};
  if (source) {
    const int j = threadIdx.x & 3;
    const double tau = (j & 1 ? tE + g.dt : tE) - (j & 2 ? g.dx : 0.0);
    const double s = source_s(a.laser, tau), e = source_e(a.laser, tau);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      ss[t] = lane_value(s, t);
      se[t] = lane_value(e, t);
    }
  }
#pragma unroll
  for (int q = 0; q < kSolveNodes; ++q)
    if (live[q]) node_load(a, ii[q], kk[q], in[q]);
  double en[kSolveNodes][3];
#pragma unroll
  for (int q = 0; q < kSolveNodes; ++q)
    if (live[q]) node_solve(a, in[q], en[q]);
  MurIn mur[kSolveNodes];
  double ez[kSolveNodes];
#pragma unroll
  for (int q = 0; q < kSolveNodes; ++q) {
    ez[q] = 0.0;
    if (absorbing && live[q] && (left[q] || ii[q] == g.nx - 1)) {
      mur_load(a, in[q].n + (left[q] ? -1 : 1), mur[q]);
      if (source && left[q]) {
        const double sz = ((double)kk[q] * g.dz - a.laser.z_center) / a.laser.sigma_z;
        ez[q] = exp(-0.5 * sz * sz);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kSolveNodes; ++q) {
    if (!live[q]) continue;
    if (in[q].dep) clear_node_moments(a, in[q].n);
    write_e(a, in[q].n, en[q]);
    if (absorbing) {
      const double inc[4] = {ss[0] * ez[q] * se[0], ss[1] * ez[q] * se[1], ss[2] * ez[q] * se[2],
                             ss[3] * ez[q] * se[3]};
      if (left[q]) mur_node(a, true, in[q].n - 1, mur[q], in[q].e, en[q], inc);
      if (ii[q] == g.nx - 1) {
        if (left[q]) mur_load(a, in[q].n + 1, mur[q]);  // (two columns of cells: both boundaries)
        mur_node(a, false, in[q].n + 1, mur[q], in[q].e, en[q], inc);
      }
    }
  }
}

// Block b of a grid of 8 * per blocks runs on XCD b % 8 (round-robin dispatch); give the
// blocks of one XCD a contiguous band of the grid, so the neighbouring rows a stencil reads
// are mostly in the same L2.  Returns -1 for the padding blocks.
__device__ __forceinline__ int64_t xcd_band_block(int64_t nblocks) {
  const int64_t per = (nblocks + 7) >> 3;
  const int64_t b = blockIdx.x;
  const int64_t idx = (b & 7) * per + (b >> 3);
  return idx < nblocks ? idx : -1;
}

__global__ __launch_bounds__(kBlock) void k_solve_e(const FieldArgs a, int64_t nblocks) {
  const int64_t blk = xcd_band_block(nblocks);
  if (blk < 0) return;
  solve_e_body(a, a.t, blk * (kSolveNodes * kBlock) + threadIdx.x, kBlock);
}

// Cells c0, c0 + stride, ... of the H update (kHCells per thread, all loads before the
// stores).
__device__ __forceinline__ void update_h_body(const FieldArgs &a, int64_t c0, int64_t stride) {
  const GridArgs &g = a.g;
  const int nx = g.nx, nz = g.nz, nxn = g.nxn;
  const int64_t nn = g.nnodes, nc = g.ncells;
  const double *Ex = a.E_new, *Ey = a.E_new + nn, *Ez = a.E_new + 2 * nn;
  double hn[kHCells][3];
  bool live[kHCells];
#pragma unroll
  for (int q = 0; q < kHCells; ++q) {
    const int64_t c = c0 + q * stride;
    live[q] = c < nc;
    if (!live[q]) continue;
    int k = (int)(c / nx), i = (int)(c - (int64_t)k * nx);
    int i1 = (g.bc_x == PIC_BC_PERIODIC) ? wrap1(i + 1, nx) : i + 1;
    int k1 = wrap1(k + 1, nz);
    int64_t na = (int64_t)k * nxn + i, nb = (int64_t)k * nxn + i1;
    int64_t ncn = (int64_t)k1 * nxn + i, nd = (int64_t)k1 * nxn + i1;
    double dEx_dz = ((Ex[ncn] + Ex[nd]) - (Ex[na] + Ex[nb])) * a.r2dz;
    double dEy_dz = ((Ey[ncn] + Ey[nd]) - (Ey[na] + Ey[nb])) * a.r2dz;
    double dEy_dx = ((Ey[nb] + Ey[nd]) - (Ey[na] + Ey[ncn])) * a.r2dx;
    double dEz_dx = ((Ez[nb] + Ez[nd]) - (Ez[na] + Ez[ncn])) * a.r2dx;
    hn[q][0] = a.H[c] - g.dt * (-dEy_dz);
    hn[q][1] = a.H[nc + c] - g.dt * (dEx_dz - dEz_dx);
    hn[q][2] = a.H[2 * nc + c] - g.dt * dEy_dx;
  }
#pragma unroll
  for (int q = 0; q < kHCells; ++q) {
    if (!live[q]) continue;
    const int64_t c = c0 + q * stride;
    a.H_new[c] = hn[q][0];
    a.H_new[nc + c] = hn[q][1];
    a.H_new[2 * nc + c] = hn[q][2];
    // The E solve has read the deposit flags: clear them for the next deposit (there are
    // fewer flags than cells: nodes <= 2 cells).
    if (a.mflag && c < (nn + kFlagNodes - 1) / kFlagNodes) a.mflag[c] = 0;
    // the next order's tile flags, set again by the sort's scan (batched cycle; there are no
    // more tiles than cells)
    if (a.tact_next && c < (int64_t)a.ntiles_next) a.tact_next[c] = 0;
  }
}

__global__ __launch_bounds__(kBlock) void k_update_h(const FieldArgs a, int64_t nblocks) {
  const int64_t blk = xcd_band_block(nblocks);
  if (blk < 0) return;
  update_h_body(a, blk * (kHCells * kBlock) + threadIdx.x, kBlock);
}

// ------------------------------------------------------------------------------------------
// Particles
// ------------------------------------------------------------------------------------------

// Stores of the particle kernel as raw buffer stores: a lane without a value passes an offset
// past the buffer's range, which the hardware drops, so the store needs no branch.  Every array
// gets the same range, 2^31 bytes (a species holds fewer than 2^28 particles).
constexpr int kStoreDrop = (int)0xFFFFFF00u;
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t store_rsrc(void *p) {
  return __builtin_amdgcn_make_buffer_rsrc(p, (short)0, (int)0x80000000u, 0x00020000);
}
__device__ __forceinline__ void store_or_drop(double *p, int i, bool on, double v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), store_rsrc(p), on ? i * 8 : kStoreDrop, 0, 0);
}
__device__ __forceinline__ void store_or_drop(float *p, int i, bool on, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), store_rsrc(p), on ? i * 4 : kStoreDrop, 0, 0);
}
__device__ __forceinline__ void store_or_drop(int32_t *p, int i, bool on, int32_t v) {
  __builtin_amdgcn_raw_buffer_store_b32((uint32_t)v, store_rsrc(p), on ? i * 4 : kStoreDrop, 0, 0);
}
__device__ __forceinline__ void store_or_drop(uint8_t *p, int i, bool on, uint8_t v) {
  __builtin_amdgcn_raw_buffer_store_b8(v, store_rsrc(p), on ? i : kStoreDrop, 0, 0);
}
__device__ __forceinline__ void store_or_drop(uint32_t *p, int i, bool on, uint32_t v) {
  __builtin_amdgcn_raw_buffer_store_b32(v, store_rsrc(p), on ? i * 4 : kStoreDrop, 0, 0);
}

// One particle's compact moments added to the LDS accumulators of its cell (lower-left
// accumulator node o, ring cell rc), corner by corner.  Lanes of odd index take the corners in
// the order (i,k+1), (i+1,k+1), (i,k), (i+1,k): neighbouring lanes often hold particles of one
// cell, and same-address atomics of one instruction are serialised (different rows cost less).
template <typename T>
__device__ __forceinline__ void deposit_one(const AccLds &acc, int o, int rc, T fx, T fz,
                                            const Compact<T> &m, T w, int dplane) {
  // odd lanes take the upper row of corners first (corners 2, 3, 0, 1)
  const bool odd = threadIdx.x & 1;
  const T gx[2] = {T(1) - fx, fx};
  const T gz[2] = {odd ? fz : T(1) - fz, odd ? T(1) - fz : fz};
  const int orow[2] = {o + (odd ? acc.LW : 0), o + (odd ? 0 : acc.LW)};
  const int crow[2] = {odd ? 2 : 0, odd ? 0 : 2};
#pragma unroll
  for (int c0 = 0; c0 < 4; ++c0) {
    const int cx = c0 & 1, row = c0 >> 1;
    const T W = gx[cx] * gz[row];
    corner_add(acc, orow[row] + cx, rc, crow[row] + cx, W * m.a0, W * m.a1, W * m.a2, W * m.j0,
               W * m.j1, W * m.j2, W * w, dplane);
  }
}

// Direct form: a particle whose new cell (gi, gk) lies outside the tile adds its moments to
// the global moment planes at once, at the cell's 4 corner nodes: the same products as an LDS
// deposit, with S-hat expanded with that cell's B as the fold expands the per-cell sums.  At
// a few particles per cell about one in three hundred leaves its tile in a cycle, and the
// tile's LDS then holds the nodes and cells of the tile alone.
template <typename T>
__device__ void deposit_global(const StepArgs &a, int gi, int gk, T fx, T fz, const Compact<T> &m,
                               T w, T B0t, T B1t, T B2t, int dplane) {
  const GridArgs &g = a.g;
  const int64_t nn = g.nnodes;
  const int gi1 = (g.bc_x == PIC_BC_PERIODIC && gi + 1 == g.nx) ? 0 : gi + 1;
  const int gk1 = gk + 1 == g.nz ? 0 : gk + 1;
#pragma unroll 1
  for (int c = 0; c < 4; ++c) {
    const int cx = c & 1, cz = c >> 1;
    const T W = (cx ? fx : T(1) - fx) * (cz ? fz : T(1) - fz);
    const double A0 = (double)(W * m.a0), A1 = (double)(W * m.a1), A2 = (double)(W * m.a2);
    const double B0 = (double)B0t, B1 = (double)B1t, B2 = (double)B2t;
    double *M = a.M + ((int64_t)(cz ? gk1 : gk) * g.nxn + (cx ? gi1 : gi));
    unsafeAtomicAdd(M, fma(A2, B0 * B0, A0));
    unsafeAtomicAdd(M + nn, fma(A2, B0 * B1, A1 * B2));
    unsafeAtomicAdd(M + 2 * nn, fma(A2, B0 * B2, -A1 * B1));
    unsafeAtomicAdd(M + 3 * nn, fma(A2, B1 * B0, -A1 * B2));
    unsafeAtomicAdd(M + 4 * nn, fma(A2, B1 * B1, A0));
    unsafeAtomicAdd(M + 5 * nn, fma(A2, B1 * B2, A1 * B0));
    unsafeAtomicAdd(M + 6 * nn, fma(A2, B2 * B0, A1 * B1));
    unsafeAtomicAdd(M + 7 * nn, fma(A2, B2 * B1, -A1 * B0));
    unsafeAtomicAdd(M + 8 * nn, fma(A2, B2 * B2, A0));
    unsafeAtomicAdd(M + 9 * nn, (double)(W * m.j0));
    unsafeAtomicAdd(M + 10 * nn, (double)(W * m.j1));
    unsafeAtomicAdd(M + 11 * nn, (double)(W * m.j2));
    unsafeAtomicAdd(M + (9 + dplane) * nn, (double)(W * w));
    if (a.mflag) a.mflag[((int64_t)(cz ? gk1 : gk) * g.nxn + (cx ? gi1 : gi)) / kFlagNodes] = 1;
  }
}

// Grouped form: deposit of a group of 64 particles, one per lane, through the matrix cores.
// S-hat and delta-j of a cell's particles are the contraction over the particles of 4 corner
// weights and 7 compact moments.  v_mfma_f64_4x4x4_4b contracts 4 blocks of 4 particles at a
// time: lane 16 k + 4 b + i holds A[i][k] and B[k][i] of block b and receives D[i][j] in lane
// 16 i + 4 b + j.  Block b takes the 16 particles of lanes 16 b .. 16 b + 15 in four rounds, so
// eight instructions sum the 28 products of 64 particles, without the 56 registers of per-lane
// sums and with two LDS atomic instructions for the result.  The particles go from one per lane
// to the operands' layout through LDS: kStagePlanes planes (f_x, f_z, delta-j x, y, z, density,
// a0, a1, a2), particle P at P + P / 16, planes kStagePitch doubles apart: the 16 lanes of one
// LDS pass then read doubles 4 i + b (mod 16), which differ, and write consecutive ones.
constexpr int kStagePlanes = 9;
constexpr int kStagePitch = 68;
// bytes of a wavefront's staging area: the planes, 64 cells, 64 movers, 64 pass numbers (see Stage)
constexpr int kStageBytes = kStagePlanes * kStagePitch * 8 + 128 * 4 + 64;

// LDS layout of the particle kernel (byte offsets): the moment accumulators (delta-j and
// density per node, S-hat scalars per cell corner), the fields the tile's particles read (E-bar
// on the tile's nodes, H^{n+1/2} on its cells, H^{n+3/2} on its cells plus the one-cell ring a
// particle can move into), the per-wave deposit staging, per species the int move counters of
// the tile's cells and the arrival counts of the tile's cells and their ring, and the first and
// end slot of every tile row of every species slot.  Two layouts: the grouped form (waves > 0)
// has accumulators over the tile and its ring and a staging area per wavefront; the direct form
// (waves = 0) covers the tile's own nodes and cells, particles leaving the tile deposit to the
// global planes, and the arrivals take the place of the staged fields, which brings a 32 x 4 tile
// of two species to 40 KB: four blocks per CU.  Accumulators and staging
// are FP64; fields use the kernel's arithmetic type.
struct TileLds {
  int LW, LH, plane;          // accumulator node grid (tx + 3) x (tz + 3), or (tx + 1) x (tz + 1)
  int EW, EPL;                // E-bar node grid (tx + 1) x (tz + 1)
  int HPL;                    // H^{n+1/2} cells tx x tz
  int NW, NPL;                // H^{n+3/2} cells (tx + 2) x (tz + 2)
  int CPL;                    // pitch of the S-hat corner planes: NPL, or HPL padded
  int n_node;                 // node accumulator planes: 3 + species
  size_t acc, accc, eb, ho, hn, stage, cnt, arr, rows;  // byte offsets
  size_t bytes;
  __host__ __device__ TileLds(int n_planes, int tx, int tz, int tsize, int waves) {
    const int ring = waves ? 1 : 0;
    LW = tx + 1 + 2 * ring;
    LH = tz + 1 + 2 * ring;
    plane = LW * LH;
    // grouped form: the 16 results of a cell (4 corners x 4 planes, and 4 corners x 3 scalars) go
    // to LDS in one instruction; these pitches spread them over the banks
    if (ring) plane += (5 - plane % 16 + 16) % 16;
    EW = tx + 1;
    EPL = EW * (tz + 1);
    HPL = tx * tz;
    NW = tx + 2;
    NPL = NW * (tz + 2);
    // without the ring the corner-plane pitch is padded to 4 (mod 8) doubles: the two lanes of
    // one cell, whose corners are two planes apart, then use complementary LDS banks
    CPL = ring ? NPL | 1 : HPL + ((4 - HPL % 8) + 8) % 8;
    n_node = 3 + (n_planes - 12);
    acc = 0;
    accc = acc + (size_t)n_node * plane * sizeof(double);
    stage = accc + (size_t)12 * CPL * sizeof(double);
    eb = stage + (size_t)waves * kStageBytes;
    ho = eb + 3 * (size_t)EPL * tsize;
    hn = ho + 3 * (size_t)HPL * tsize;
    cnt = (hn + 3 * (size_t)NPL * tsize + 7) & ~(size_t)7;
    arr = cnt + (size_t)(n_node - 3) * tx * tz * kMoveCodes * sizeof(int);
    const size_t arr_bytes = (size_t)(n_node - 3) * (tx + 2) * (tz + 2) * sizeof(int);
    rows = arr + arr_bytes;
    // the direct form counts arrivals where E-bar and H^{n+1/2} were, if they fit
    if (!ring && arr_bytes <= hn - eb) {
      rows = arr;
      arr = eb;
    }
    bytes = rows + (size_t)(n_node - 3) * tz * 2 * sizeof(int);
  }
};

// Location and move code of slot j as the rankers read them, (location << 4) | code: stored so by
// the direct form; the other kernels write a particle to the location of its slot and store a byte
// per slot, its code.
__device__ __forceinline__ uint32_t slot_code(const StepArgs &a, const SpeciesArgs &sp, int j) {
  return a.slot_codes ? ((uint32_t)j << 4) | reinterpret_cast<const uint8_t *>(sp.locode)[j] : sp.locode[j];
}

// The staging area of a wavefront: the planes, then per block the cell of every pass of the
// deposit, the list of the movers (cell, and place in the planes in the high 8 bits) and per
// particle its pass.
struct Stage {
  double *v;       // [kStagePlanes][kStagePitch]
  int *key;        // [4 blocks][16 passes]
  int *mover;      // [64]
  uint8_t *pass;   // [64]: particle 16 b + 4 t + k at 16 b + 4 k + t
  __device__ __forceinline__ explicit Stage(char *p)
      : v(reinterpret_cast<double *>(p)),
        key(reinterpret_cast<int *>(p + kStagePlanes * kStagePitch * sizeof(double))),
        mover(key + 64),
        pass(reinterpret_cast<uint8_t *>(key + 128)) {}
};

// The moments of a group's particles, one per lane, from the wavefront's staging area into the
// LDS accumulators.  act: lanes with a slot; alive: with a particle to deposit; src, dst: its old
// and new cell (ring cell in the low 16 bits, accumulator row above).
//
// The particles that stay in their cell: a pass takes one cell per block of 16 lanes, in their
// (sorted) order; the other particles' weights are masked to zero (their staged values are
// finite: only particles with finite moments are staged, and the area starts at zero).  At 64 particles per
// cell a group takes one or two passes, at 11 about three.
//
// The movers go one by one, four at a time: 16 lanes compute a mover's 28 products (corner i,
// moments j and 4 + j) and add them with two LDS atomic instructions.  A group has two movers in
// a 1 keV plasma, ten or more in a laser-heated one, and as passes of their own (or a pass per
// destination) they cost more than the particles that stay.
__device__ __forceinline__ void deposit_group(const AccLds &acc, const Stage &st, bool act,
                                              bool alive, int src, int dst, int own, int lane,
                                              int dplane) {
  const int mi = lane & 3, mb = (lane >> 2) & 3, mk4 = lane >> 4;  // i or j, block, k
  const int ob = lane >> 4, ol = lane & 15;                        // block and place of the lane's own particle
  const bool mover = alive && src != dst;
  const int before = lane_before(src);  // (all lanes active)
  const bool head = act && (ol == 0 || before != src);
  const uint64_t heads = __ballot(head), movers = __ballot(mover);
  auto in_block = [](uint64_t m, int b) { return (uint32_t)(m >> (16 * b)) & 0xffffu; };
  {
    const int seg = __popc(in_block(heads, ob) & ((2u << ol) - 1u)) - 1;
    if (head) st.key[ob * 16 + seg] = src;
    if (mover) st.mover[__popcll(movers & ((1ull << lane) - 1ull))] = dst | (own << 24);
    st.pass[ob * 16 + (ol & 3) * 4 + (ol >> 2)] = (uint8_t)(alive && !mover ? seg : 255);
  }
  int n_pass = 0;  // of the block with most passes
#pragma unroll
  for (int b = 0; b < 4; ++b) n_pass = max(n_pass, __popc(in_block(heads, b)));
  const int n_mine = __popc(in_block(heads, mb)), n_movers = __popcll(movers);
  wave_sync();
  // corner weights, moments and passes of the block's four particles of each round
  const int at = mb * 17 + mk4;
  double A[4], B0[4], B1[4];
  const int p0 = (2 + mi) * kStagePitch, p1 = (6 + min(mi, 2)) * kStagePitch;  // the planes of moments j, 4 + j
  const uint32_t pass4 = *reinterpret_cast<const uint32_t *>(st.pass + 16 * mb + 4 * mk4);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const double fx = st.v[at + 4 * t], fz = st.v[kStagePitch + at + 4 * t];
    const double gx = (mi & 1) ? fx : 1.0 - fx, gz = (mi & 2) ? fz : 1.0 - fz;
    A[t] = gx * gz;
    B0[t] = st.v[p0 + at + 4 * t];
    B1[t] = st.v[p1 + at + 4 * t];
  }
  // the accumulators of corner c, moments j and 4 + j
  auto node_of = [&](int c) { return acc.node + (mi < 3 ? mi : dplane) * acc.plane + (c & 1) + (c >> 1) * acc.LW; };
  auto cell_of = [&](int c) { return acc.cell + (min(mi, 2) * 4 + c) * acc.npl; };
  {
    // result lane 16 i + 4 b + j: corner i (of the cell), moment j
    double *const node = node_of(mk4), *const cell = cell_of(mk4);
    for (int p = 0; p < n_pass; ++p) {
      const int k = st.key[mb * 16 + p];
      double d0 = 0.0, d1 = 0.0;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const double w = ((pass4 >> (8 * t)) & 255u) == (uint32_t)p ? A[t] : 0.0;
        d0 = __builtin_amdgcn_mfma_f64_4x4x4f64(w, B0[t], d0, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f64_4x4x4f64(w, B1[t], d1, 0, 0, 0);
      }
      if (p < n_mine) {
        const int rc = k & 0xffff;               // ring cell; its lower-left node is rc + row
        atomicAdd(&node[rc + (k >> 16)], d0);
        if (mi < 3) atomicAdd(&cell[rc], d1);
      }
    }
  }
  if (n_movers) {
    // lane 16 g + 4 i + j: mover g of the step, corner i, moments j and 4 + j
    double *const node = node_of(mb), *const cell = cell_of(mb);
    for (int m = mk4; m < n_movers; m += 4) {
      const int k = st.mover[m], q = k >> 24, rc = k & 0xffff;
      const double fx = st.v[q], fz = st.v[kStagePitch + q];
      const double w = ((mb & 1) ? fx : 1.0 - fx) * ((mb & 2) ? fz : 1.0 - fz);
      atomicAdd(&node[rc + ((k >> 16) & 0xff)], w * st.v[p0 + q]);
      if (mi < 3) atomicAdd(&cell[rc], w * st.v[p1 + q]);
    }
  }
}

// One block per tile of cells (tile rows are cell rows).  MIXED selects the mixed-precision
// form: FP32 state, gather and push, added into FP64 LDS accumulators and the FP64 moment
// planes.  IDS adds the copy of particle ids (tests only).  PW selects per-particle densities:
// each particle's moments are those of unit density times its own density, which is read with
// the state and written with the pushed state (a species with one density reads it from a
// one-element array with stride 0).
//
// Two forms.  The grouped form (DIRECT = false) takes the particles of a tile row (a contiguous
// range of the cell-sorted order) in groups of 64 consecutive slots, one per lane, the groups of
// the tile dealt to the block's wavefronts in turn.  A particle's pushed state goes to the
// location of its slot, so stores are coalesced, and next cycle's reads through the permutation
// too: most particles keep their cell, so 64 consecutive slots read a few runs of consecutive
// locations.  The group's moments are summed per cell by deposit_group, movers like the others,
// into accumulators that cover the tile and its ring.
//
// The direct form (few particles per cell: a lane holds one to five particles per row) splits the
// row into 64 contiguous runs, one per lane, whose lengths differ by at most one, loads two
// particles of a lane at a time, adds each particle's moments to LDS at once, keeps accumulators
// for the tile's own nodes and cells only and sends the moments of a particle that leaves the
// tile to the global planes: about 120 VGPRs (FP64) and 40 KB of LDS at 32 x 4, four blocks per
// CU.  The pushed state of the particle at iteration `it` of lane `l` is written to location
// row_start + 64 it + l.
template <bool PUSH, bool MIXED, bool IDS, bool PW, bool DIRECT = false>
__device__ __forceinline__ void particles_body(const StepArgs &a, int tile) {
  using T = typename std::conditional<MIXED, float, double>::type;
  static_assert(PUSH || !DIRECT, "the deposit of a loaded state uses the grouped form");
  const GridArgs &g = a.g;
  const TileArgs &t = a.t;
  const int tzi = tile / t.ntx, txi = tile - tzi * t.ntx;
  const int i0 = txi * t.tx, k0 = tzi * t.tz;
  const int i1 = min(i0 + t.tx, g.nx), k1 = min(k0 + t.tz, g.nz);
  const int ntc = t.tx * t.tz;
  const int64_t nn = g.nnodes, nc = g.ncells;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;

  extern __shared__ double lds[];
  char *ldsb = reinterpret_cast<char *>(lds);
  const TileLds Lo(g.n_planes, t.tx, t.tz, (int)sizeof(T), DIRECT ? 0 : nwaves);
  const AccLds acc{reinterpret_cast<double *>(ldsb + Lo.acc),
                   reinterpret_cast<double *>(ldsb + Lo.accc), Lo.plane, Lo.CPL, Lo.LW, Lo.NW};
  T *Eb = reinterpret_cast<T *>(ldsb + Lo.eb);
  T *Ho = reinterpret_cast<T *>(ldsb + Lo.ho);
  T *Hn = reinterpret_cast<T *>(ldsb + Lo.hn);
  int *cntL = reinterpret_cast<int *>(ldsb + Lo.cnt);  // [species][9 codes][cells of the tile]
  int *arrL = reinterpret_cast<int *>(ldsb + Lo.arr);  // [species][tile and ring]
  const int LW = Lo.LW, plane = Lo.plane;  // plane: pitch of the node planes, LW * LH nodes
  // node planes, cell-corner planes and (grouped) the staging areas, which follow them
  const int n_zero = Lo.n_node * plane + 12 * Lo.CPL + (DIRECT ? 0 : nwaves * (kStageBytes / 8));

  for (int e = 2 * threadIdx.x; e < n_zero; e += 2 * blockDim.x) {
    if (e + 1 < n_zero)
      *reinterpret_cast<double2 *>(acc.node + e) = make_double2(0.0, 0.0);
    else
      acc.node[e] = 0.0;
  }
  constexpr bool kTileOnly = DIRECT;  // accumulators over the tile's own nodes and cells (no ring)
  const int AW = t.tx + 2, AH = t.tz + 2;  // arrival counts: the tile's cells and their ring
  if (PUSH) {
    const int nsl = Lo.n_node - 3;
    // the counters of the particles that stay (code 4) start at the cell's particles (below)
    for (int s = 0; s < nsl; ++s)
      for (int e = threadIdx.x; e < (kMoveCodes - 1) * ntc; e += blockDim.x)
        cntL[s * ntc * kMoveCodes + e + (e >= 4 * ntc ? ntc : 0)] = 0;
    if constexpr (!DIRECT)
      for (int e = threadIdx.x; e < nsl * AW * AH; e += blockDim.x) arrL[e] = 0;
  }
  const int cw = i1 - i0, chh = k1 - k0;  // the tile's cells inside the grid
  // a tile and its two-cell ring fit in the grid along an axis: wraps need one compare there
  const bool nearx = g.nx >= t.tx + 3, nearz = g.nz >= t.tz + 3;
  // Stage the fields of the tile, the particles of every cell and the slot range of every tile
  // row of every species.  The elements of the three field arrays (H^{n+3/2} on the cells and
  // their ring, E-bar on the nodes, H^{n+1/2} on the cells, which also brings the cell's slots)
  // are numbered one after the other and dealt to the threads, so a thread computes the address
  // of one element (direct form, with half the threads: two, loaded before it stores either) and
  // the block waits for one memory round trip.  (Every thread computing an element of each array
  // took 550 instructions, 3 us of a tile's time with four wavefronts per SIMD.)
  constexpr int kEl = DIRECT ? 2 : 1;
  const int nrows_t = k1 - k0;
  int *rowsL = reinterpret_cast<int *>(ldsb + Lo.rows);  // [species][row]: first, end slot
  const int v_e = PUSH ? Lo.NPL : 0, v_h = v_e + (PUSH ? Lo.EPL : 0), v_n = v_h + Lo.HPL;
  // (the pointers are kept in registers: a choice between two members of the kernel's arguments
  // would be made by their address, and the arguments copied to scratch memory for it)
  const double *p_ho = a.Hold, *p_eo = a.Eold, *p_hn = a.Hnew;
  asm("" : "+v"(p_ho), "+v"(p_eo), "+v"(p_hn));
  for (int v0 = threadIdx.x; v0 < v_n; v0 += kEl * blockDim.x) {
    double fa[kEl][3], fb[kEl][3];
    int cb[kEl][kMaxSpecies], ce[kEl][kMaxSpecies], el[kEl], row[kEl];
    bool is_e[kEl], is_h[kEl], in[kEl], first[kEl], last[kEl];
#pragma unroll
    for (int u = 0; u < kEl; ++u) {
      const int v = min(v0 + u * (int)blockDim.x, v_n - 1);  // (past the end: the last one again)
      is_h[u] = v >= v_h;
      is_e[u] = v >= v_e && !is_h[u];
      el[u] = v - (is_h[u] ? v_h : is_e[u] ? v_e : 0);
      const int off = is_h[u] || is_e[u] ? 0 : -1;  // the ring starts one cell before the tile
      const int W = is_h[u] ? t.tx : is_e[u] ? Lo.EW : Lo.NW;
      const int ez = SmallDiv(W).q(el[u]), ex = el[u] - ez * W;
      const int xmax = is_e[u] ? g.nxn - 1 : g.nx - 1;
      int gi = i0 + off + ex, gk = k0 + off + ez;
      row[u] = ez;
      if (is_h[u]) {
        in[u] = gi < g.nx && gk < g.nz;
        gk = min(gk, g.nz - 1);
      } else {
        gk = wrap_t(gk, g.nz, nearz);
        if (g.bc_x == PIC_BC_PERIODIC) gi = wrap_t(gi, g.nx, nearx);
        in[u] = gi >= 0 && gi <= xmax;
      }
      first[u] = in[u] && ex == 0;
      last[u] = in[u] && ex == cw - 1;
      const int64_t n = (int64_t)gk * (is_e[u] ? g.nxn : g.nx) + min(max(gi, 0), xmax);
      const double *f = (is_h[u] ? p_ho : is_e[u] ? p_eo : p_hn) + n;
      const int64_t pitch = is_e[u] ? nn : nc;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        fa[u][q] = f[q * pitch];
        fb[u][q] = 0.0;
      }
      if (is_e[u]) {
#pragma unroll
        for (int q = 0; q < 3; ++q) fb[u][q] = a.Enew[q * nn + n];
      }
#pragma unroll
      for (int q = 0; q < kMaxSpecies; ++q) {
        cb[u][q] = 0;
        ce[u][q] = 0;
        if (is_h[u] && q < a.nsp && a.sp[q].active) {
          cb[u][q] = a.sp[q].cs[n];
          ce[u][q] = a.sp[q].cs[n + 1];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kEl; ++u) {
      T *d = (is_h[u] ? Ho : is_e[u] ? Eb : Hn) + el[u];
      const int pitch = is_h[u] ? Lo.HPL : is_e[u] ? Lo.EPL : Lo.NPL;
#pragma unroll
      for (int q = 0; q < 3; ++q)
        d[q * pitch] = in[u] ? (T)(is_e[u] ? 0.5 * (fa[u][q] + fb[u][q]) : fa[u][q]) : T(0);
      if (is_h[u]) {
#pragma unroll
        for (int q = 0; q < kMaxSpecies; ++q) {
          if (q < a.nsp) {
            if (PUSH) cntL[(q * kMoveCodes + 4) * ntc + el[u]] = in[u] ? ce[u][q] - cb[u][q] : 0;
            if (first[u]) rowsL[2 * (q * nrows_t + row[u])] = cb[u][q];
            if (last[u]) rowsL[2 * (q * nrows_t + row[u]) + 1] = ce[u][q];
          }
        }
      }
    }
  }
  __syncthreads();

  // the tile touches the grid's border: its particles may wrap or leave
  const bool edge = i0 == 0 || i1 == g.nx || k0 == 0 || k1 == g.nz;

  int gr = wave;  // grouped form: the wavefront's next group
  for (int s = 0; s < a.nsp; ++s) {
    const SpeciesArgs &sp = a.sp[s];
    if (!sp.active) continue;
    int *const cntS = cntL + s * ntc * kMoveCodes;  // the species' move counters
    // (a species with one density keeps its own constants, also in a kernel with densities per
    // particle: its moments are then the same bits in both)
    const bool own_w = PW && sp.w_stride != 0;
    const SpConst<T> K{(T)sp.beta, (T)(own_w ? sp.cS1 : sp.cS), (T)(own_w ? sp.kJ1 : sp.kJ), (T)sp.w};
    const typename Pstate<MIXED>::Src src(sp);
    // per-particle densities: index p * wstride (stride 0 reads a species' single density)
    const T *wsrc = nullptr;
    T *wdst = nullptr;
    if constexpr (MIXED) {
      wsrc = sp.msrc_w;
      wdst = sp.mdst_w;
    } else {
      wsrc = sp.src_w;
      wdst = sp.dst_w;
    }
    const int wstride = sp.w_stride;
    const int32_t *perm = sp.perm;
    const int dplane = 3 + s;  // density plane of the species in the node accumulators
    const int nrows = k1 - k0;
    const uint32_t loc_max = (uint32_t)(sp.cap - 1);
    // A particle outside the cell its slot says: raise the flag and drop it.  (Never in a
    // consistent state; the counts keep the slot, so the next order stays in bounds.)
    auto drop_slot = [&](int j, uint32_t loc) {
      atomicOr(a.flags, kFlagOrder);
      if (!PUSH) return;
      if constexpr (DIRECT)
        sp.locode[j] = (loc << 4) | kAbsorbed;
      else
        reinterpret_cast<uint8_t *>(sp.locode)[j] = kAbsorbed;
    };
    if constexpr (!DIRECT) {
      const Stage stage(ldsb + Lo.stage + wave * kStageBytes);
      double *const st = stage.v;
      const int own = lane + (lane >> 4);  // this lane's particle in a staging plane
      // (a density beyond 32 bits goes with its particles, alone)
      if constexpr (!PW) st[5 * kStagePitch + own] = MIXED && !isfinite(K.w) ? 0.0 : (double)K.w;
      // The tile's groups, row by row, are dealt to the wavefronts (a power of two) in turn, on
      // from where the last species ended: group gr of row r holds slots jg .. jg + ngr - 1
      // (ngr = 0: no group left).
      gr &= nwaves - 1;
      int r = k0, rb = 0, re = 0, jg = 0, ngr = 0;
      auto take_row = [&]() {
        rb = __builtin_amdgcn_readfirstlane(rowsL[2 * (s * nrows_t + (r - k0))]);
        re = __builtin_amdgcn_readfirstlane(rowsL[2 * (s * nrows_t + (r - k0)) + 1]);
      };
      auto settle = [&]() {  // the group at or after (r, gr)
        while (r < k1) {
          jg = rb + 64 * gr;
          ngr = min(64, re - jg);
          if (ngr > 0) return;
          gr -= (re - rb + 63) >> 6;
          if (++r < k1) take_row();
        }
        jg = ngr = 0;
      };
      take_row();
      settle();
      // Pipeline: while a group's moments are deposited, the state of the next group and the
      // permutation of the one after it are on their way.  The loads of a group go out between
      // the push and the stores of the group before it: stores share the vector-memory counter
      // with loads, in order, so waiting for a load issued after stores would wait for the stores.
      auto load_perm = [&]() { return (int)min((uint32_t)at(perm, jg + min(lane, max(ngr - 1, 0))), loc_max); };
      int rc_ = r, jc = jg, nc_ = ngr;  // the current group
      Pstate<MIXED> ps{};
      T wp = K.w;
      int pc = load_perm();
      gr += nwaves;
      settle();
      int rn = r, jn = jg, nn_ = ngr;  // the next group
      int pn = load_perm();
      ps.load(src, pc);
      if constexpr (PW) wp = at(wsrc, pc * wstride);
      // wait for the first loads here: a load pending on entry only would make the compiler wait
      // at the head of every iteration for everything issued before it
      asm volatile("" ::"v"(pn), "v"(ps.x), "v"(ps.z), "v"(ps.u0), "v"(ps.u1), "v"(ps.u2), "v"(wp));
      while (nc_ > 0) {
        {
          const int r = rc_, j = jc + lane, p = pc;
          const bool act = lane < nc_;
          const int lk = r - k0;
          int i, k;
          T fx, fz;
          if constexpr (MIXED) {
            k = r;
            i = ps.cell - r * g.nx;
            fx = ps.x;
            fz = ps.z;
          } else {
            const double xf = floor(ps.x), zf = floor(ps.z);
            i = (int)xf;
            k = (int)zf;
            fx = ps.x - xf;
            fz = ps.z - zf;
          }
          const bool ok = act && k == r && i >= i0 && i < i1;
          if (act && !ok) drop_slot(j, (uint32_t)j);
          // Lanes without a valid particle run the arithmetic on the tile's first cell and
          // discard the results.
          const int li = ok ? i - i0 : 0;
          const int hc = lk * t.tx + li;
          T fB[3];
#pragma unroll
          for (int qq = 0; qq < 3; ++qq) fB[qq] = Ho[qq * Lo.HPL + hc];
          Compact<T> m;
          T dfx = fx, dfz = fz;
          const T wcur = wp;
          auto next_loads = [&]() {
            pc = pn;
            ps.load(src, pc);
            if constexpr (PW) wp = at(wsrc, pc * wstride);
            gr += nwaves;
            settle();
            pn = load_perm();
          };
          int ring = (lk + 1) * Lo.NW + li + 1;  // ring cell of the deposit
          const int key_src = ((lk + 1) << 16) | ring;
          int key = key_src;
          bool alive = ok;
          if constexpr (!PUSH) {
            const T ginv = rsqT(fmaT(ps.u2, ps.u2, fmaT(ps.u1, ps.u1, fmaT(ps.u0, ps.u0, T(1)))));
            m = compact_moments(K, ginv, ps.u0, ps.u1, ps.u2, fB[0], fB[1], fB[2]);
            next_loads();
          } else {
            T fE[12];
            const int e00 = lk * Lo.EW + li;
#pragma unroll
            for (int qq = 0; qq < 3; ++qq) {
              const T *f = Eb + qq * Lo.EPL + e00;
              fE[4 * qq] = f[0];
              fE[4 * qq + 1] = f[1];
              fE[4 * qq + 2] = f[Lo.EW];
              fE[4 * qq + 3] = f[Lo.EW + 1];
            }
            Pushed<T> o;
            push_one<MIXED>(g, K, ps, i, k, fx, fz, fE, fB, edge, ok, o);
            if (ok && !o.finite) atomicOr(a.flags, kFlagNonFinite);
            if (o.jump) atomicOr(a.flags, kFlagJump);
            alive = o.alive;
            const uint32_t code = alive ? (uint32_t)((o.dk + 1) * 3 + (o.di + 1)) : kAbsorbed;
            // moments M^{n+3/2} at x^{n+3/2} with u^{n+1}, 1/gamma(u^{n+1}) and H^{n+3/2}
            // of the new cell
            ring += __mul24(o.dk, Lo.NW) + o.di;
            key = ((lk + 1 + o.dk) << 16) | ring;
            m = compact_moments(K, o.rg1, o.n0, o.n1, o.n2, Hn[ring], Hn[Lo.NPL + ring], Hn[2 * Lo.NPL + ring]);
            dfx = o.fx;
            dfz = o.fz;
            next_loads();
            if constexpr (MIXED) {
              store_or_drop(sp.mdst_cell, j, ok, o.k2 * g.nx + o.i2);
              store_or_drop(sp.mdst[0], j, ok, o.xn);
              store_or_drop(sp.mdst[1], j, ok, o.zn);
              store_or_drop(sp.mdst[2], j, ok, o.n0);
              store_or_drop(sp.mdst[3], j, ok, o.n1);
              store_or_drop(sp.mdst[4], j, ok, o.n2);
            } else {
              store_or_drop(sp.dst[0], j, ok, o.xn);
              store_or_drop(sp.dst[1], j, ok, o.zn);
              store_or_drop(sp.dst[2], j, ok, o.n0);
              store_or_drop(sp.dst[3], j, ok, o.n1);
              store_or_drop(sp.dst[4], j, ok, o.n2);
            }
            if constexpr (PW) store_or_drop(wdst, j, ok && wstride != 0, wcur);
            store_or_drop(reinterpret_cast<uint8_t *>(sp.locode), j, ok, (uint8_t)code);
            // particle ids (tests only)
            if (IDS && ok && sp.dst_id) sp.dst_id[j] = sp.src_id[p];
            if (ok && code != 4u) {
              atomicSub(&cntS[4 * ntc + hc], 1);
              if (alive) atomicAdd(&cntS[__mul24((int)code, ntc) + hc], 1);
            }
          }
          if constexpr (PW) scale_compact(m, own_w ? wcur : T(1));
          // A particle with a moment that is not finite (a momentum or a B too large to square, in
          // 32 bits with a0 = 0 beside it, or a density times a charge) goes alone: in the group's
          // sums it would reach its neighbours' cells, as zero times it.
          const T all = m.a0 + m.a1 + m.a2 + m.j0 + m.j1 + m.j2;
          if (alive && !(isfinite(all) && (!MIXED || isfinite(wcur)))) {
            deposit_one(acc, (key & 0xffff) + (key >> 16), key & 0xffff, dfx, dfz, m, wcur, dplane);
            alive = false;
          }
          if (alive) {
            st[own] = (double)dfx;
            st[kStagePitch + own] = (double)dfz;
            st[2 * kStagePitch + own] = (double)m.j0;
            st[3 * kStagePitch + own] = (double)m.j1;
            st[4 * kStagePitch + own] = (double)m.j2;
            if constexpr (PW) st[5 * kStagePitch + own] = (double)wcur;
            st[6 * kStagePitch + own] = (double)m.a0;
            st[7 * kStagePitch + own] = (double)m.a1;
            st[8 * kStagePitch + own] = (double)m.a2;
          }
          wave_sync();
          deposit_group(acc, stage, act, alive, key_src, key, own, lane, dplane);
          wave_sync();
        }
        rc_ = rn;
        jc = jn;
        nc_ = nn_;
        rn = r;
        jn = jg;
        nn_ = ngr;
      }
    } else {
      // A tile with fewer rows than wavefronts splits each row's particles into wpr contiguous
      // parts, one per wavefront, so short tiles keep every wavefront busy.
      const int wpr = nrows < nwaves ? nwaves / nrows : 1;  // a power of two (up to eight wavefronts)
      const int wsh = wpr == 8 ? 3 : wpr == 4 ? 2 : wpr == 2 ? 1 : 0;
      const int part = wave % wpr;
      for (int r = k0 + wave / wpr; r < k1; r += nwaves / wpr) {
        const int rb = rowsL[2 * (s * nrows_t + (r - k0))], re = rowsL[2 * (s * nrows_t + (r - k0)) + 1];
        const int jb = rb + (int)(((uint32_t)(re - rb) * (uint32_t)part) >> wsh);
        const int je = rb + (int)(((uint32_t)(re - rb) * (uint32_t)(part + 1)) >> wsh);
        const int L = je - jb;
        if (L == 0) continue;
        const int q = L >> 6, rr = L & 63;
        const int my_n = q + (lane < rr ? 1 : 0);
        const int start = jb + lane * q + min(lane, rr);
        const int iters = q + (rr > 0 ? 1 : 0);
        const int lk = r - k0;
        // The run is processed two particles at a time: their state loads are issued together
        // (with the next two permutation entries), then they are pushed from registers in an
        // unrolled sequence.  Global stores share the vector-memory counter with loads, so a load
        // whose value is still in flight across a loop iteration makes the compiler wait for all
        // earlier stores too; keeping every loaded value inside one iteration lets it wait for
        // the loads alone.  Loads are issued unconditionally (slots past a lane's run read a
        // location inside the state arrays, and their values go unused): a load under a divergent
        // branch also forces a full wait.
        constexpr int kChunk = 2;
        Pstate<MIXED> cb[kChunk];
        int cp_[kChunk], np_[kChunk];
        T cw_[kChunk];
        // A chunk's permutation entries come in one 8-byte load per lane (the array is padded
        // so the load stays inside it); entries past the lane's run are clamped to a location
        // inside the state arrays and their particles go unused.
        static_assert(kPermPad >= 2 * kChunk, "one int2 of entries per chunk");
        auto perm2 = [&](int first, int out[kChunk]) {
          int2 v;
          __builtin_memcpy(&v, perm + first, sizeof(v));
          out[0] = (int)min((uint32_t)v.x, loc_max);
          out[1] = (int)min((uint32_t)v.y, loc_max);
        };
        perm2(start, np_);
        for (int c0 = 0; c0 < iters; c0 += kChunk) {
#pragma unroll
          for (int kk = 0; kk < kChunk; ++kk) {
            cp_[kk] = np_[kk];
            cb[kk].load(src, cp_[kk]);
            if constexpr (PW) cw_[kk] = wsrc[cp_[kk] * wstride];
          }
          perm2(start + c0 + kChunk, np_);
#pragma unroll
          for (int kk = 0; kk < kChunk; ++kk) {
            const int it = c0 + kk;
            if (it >= iters) break;
            const bool act = it < my_n;
            const int j = start + it;
            const int p = cp_[kk];
            const Pstate<MIXED> &ps = cb[kk];
            int i, k;
            T fx, fz;
            if constexpr (MIXED) {
              k = r;
              i = ps.cell - r * g.nx;
              fx = ps.x;
              fz = ps.z;
            } else {
              const double xf = floor(ps.x), zf = floor(ps.z);
              i = (int)xf;
              k = (int)zf;
              fx = ps.x - xf;
              fz = ps.z - zf;
            }
            const T wp = PW ? cw_[kk] : K.w;  // the particle's density
            const bool ok = act && k == r && i >= i0 && i < i1;
            const int loc = jb + it * 64 + lane;
            if (act && !ok) drop_slot(j, (uint32_t)loc);
            // Lanes without a valid particle run the arithmetic on the tile's first cell and
            // discard the results, so the main path has no branches around it.
            const int li = ok ? i - i0 : 0;
            const int hc = lk * t.tx + li;
            // The fields are read from LDS for every particle (a lane holds a few per row,
            // and fields kept across particles would hold about 30 registers).
            T fB[3], fE[12];
#pragma unroll
            for (int qq = 0; qq < 3; ++qq) fB[qq] = Ho[qq * Lo.HPL + hc];
            const int e00 = lk * Lo.EW + li;
#pragma unroll
            for (int qq = 0; qq < 3; ++qq) {
              const T *f = Eb + qq * Lo.EPL + e00;
              fE[4 * qq] = f[0];
              fE[4 * qq + 1] = f[1];
              fE[4 * qq + 2] = f[Lo.EW];
              fE[4 * qq + 3] = f[Lo.EW + 1];
            }
            Pushed<T> o;
            push_one<MIXED>(g, K, ps, i, k, fx, fz, fE, fB, edge, ok, o);
            if (ok && !o.finite) atomicOr(a.flags, kFlagNonFinite);
            if (o.jump) atomicOr(a.flags, kFlagJump);
            const bool alive = o.alive;
            const uint32_t code = alive ? (uint32_t)((o.dk + 1) * 3 + (o.di + 1)) : kAbsorbed;
            // moments M^{n+3/2} at x^{n+3/2} with u^{n+1}, 1/gamma(u^{n+1}) and H^{n+3/2}
            // of the new cell (read before any LDS atomic of this particle is issued)
            const int hn = (lk + o.dk + 1) * Lo.NW + (li + o.di + 1);
            Compact<T> m = compact_moments(K, o.rg1, o.n0, o.n1, o.n2, Hn[hn], Hn[Lo.NPL + hn], Hn[2 * Lo.NPL + hn]);
            // the new cell, tile-local (a dead particle stays, unused)
            const int ldx = li + o.di, ldz = lk + o.dk;
            const bool inside = ldx >= 0 && ldx < cw && ldz >= 0 && ldz < chh;
            if constexpr (PW) scale_compact(m, own_w ? wp : T(1));
            if constexpr (MIXED) {
              if (ok) {
                sp.mdst_cell[loc] = o.k2 * g.nx + o.i2;
                sp.mdst[0][loc] = o.xn;
                sp.mdst[1][loc] = o.zn;
                sp.mdst[2][loc] = o.n0;
                sp.mdst[3][loc] = o.n1;
                sp.mdst[4][loc] = o.n2;
                if (PW && wstride) wdst[loc] = wp;
                sp.locode[j] = ((uint32_t)loc << 4) | code;
              }
            } else {
              // FP64: every lane issues the stores, without a branch (a lane without a
              // particle passes an offset the hardware drops), so the compiler knows how many
              // stores each particle issues and waits for the next particle's loads alone.
              // (The mixed form measured no gain from this and keeps plain stores.)
              store_or_drop(sp.dst[0], loc, ok, o.xn);
              store_or_drop(sp.dst[1], loc, ok, o.zn);
              store_or_drop(sp.dst[2], loc, ok, o.n0);
              store_or_drop(sp.dst[3], loc, ok, o.n1);
              store_or_drop(sp.dst[4], loc, ok, o.n2);
              if constexpr (PW) store_or_drop(wdst, loc, ok && wstride != 0, wp);
              store_or_drop(sp.locode, j, ok, ((uint32_t)loc << 4) | code);
            }
            if (IDS && ok && sp.dst_id) sp.dst_id[loc] = sp.src_id[p];
            if (ok && code != 4u) {
              atomicSub(&cntS[4 * ntc + hc], 1);
              if (alive) atomicAdd(&cntS[__mul24((int)code, ntc) + hc], 1);
            }
            // every particle goes to the LDS accumulators at once, or to the global planes if
            // it leaves the tile
            if (alive && inside)
              deposit_one(acc, ldz * LW + ldx, ldz * t.tx + ldx, o.fx, o.fz, m, wp, dplane);
            if (alive && !inside)
              deposit_global(a, o.i2, o.k2, o.fx, o.fz, m, wp, Hn[hn], Hn[Lo.NPL + hn],
                             Hn[2 * Lo.NPL + hn], dplane);
          }
        }
      }
    }
  }
  __syncthreads();
  // Move counts of the tile's cells, for the ranking.  The counts of every species are kept
  // until here, so the species need no barriers between them.  With code masks only the nonzero
  // counts are written (most cells send all their particles with one code).  The grouped form's
  // blocks have more threads than cells: one thread per (code, cell) pair (2.4 -> 1.2 us of a
  // 32 x 2 tile's time against one per cell, which the direct form keeps, the species dealt to the
  // wavefronts).
  if constexpr (PUSH && !DIRECT) {
    const SmallDiv div_ntc(ntc), div_tx(t.tx);
    for (int s = 0; s < a.nsp; ++s) {
      const SpeciesArgs &sp = a.sp[s];
      if (!sp.active) continue;
      const int *cntS = cntL + s * ntc * kMoveCodes;
      int *arrS = arrL + s * AW * AH;
      for (int e = threadIdx.x; e < kMoveCodes * ntc; e += blockDim.x) {
        const int d = div_ntc.q(e), c = e - d * ntc;
        const int lkk = div_tx.q(c), li = c - lkk * t.tx;
        const int v = cntS[e];
        if (li >= cw || lkk >= chh) continue;
        if (!a.count_masks || v) sp.cnt[(int64_t)d * nc + (int64_t)(k0 + lkk) * g.nx + (i0 + li)] = v;
        const int dz = d >= 6 ? 2 : d >= 3 ? 1 : 0;
        if (v) atomicAdd(&arrS[(lkk + dz) * AW + (li + d - 3 * dz)], v);
      }
      if (!a.count_masks) continue;
      for (int c = threadIdx.x; c < ntc; c += blockDim.x) {
        const int lkk = div_tx.q(c), li = c - lkk * t.tx;
        uint32_t mask = 0;
#pragma unroll
        for (int d = 0; d < kMoveCodes; ++d) mask |= cntS[d * ntc + c] ? 1u << d : 0u;
        if (li < cw && lkk < chh) sp.cmask[(int64_t)(k0 + lkk) * g.nx + (i0 + li)] = (uint16_t)mask;
      }
    }
  }
  if constexpr (DIRECT) {
    for (int e = threadIdx.x; e < a.nsp * AW * AH; e += blockDim.x) arrL[e] = 0;
    __syncthreads();
    const int n_part = (ntc + 63) >> 6;
    const SmallDiv div_part(n_part), div_tx(t.tx);
    for (int u = wave; u < a.nsp * n_part; u += nwaves) {
      const int s = __builtin_amdgcn_readfirstlane(div_part.q(u));
      const SpeciesArgs &sp = a.sp[s];
      if (!sp.active) continue;
      const int *cntS = cntL + s * ntc * kMoveCodes;
      int *arrS = arrL + s * AW * AH;
      const int c = (u - s * n_part) * 64 + lane;
      const int lkk = div_tx.q(c), li = c - lkk * t.tx;
      if (c >= ntc || li >= cw || lkk >= chh) continue;
      const int64_t cg = (int64_t)(k0 + lkk) * g.nx + (i0 + li);
      uint32_t mask = 0;
#pragma unroll
      for (int d = 0; d < kMoveCodes; ++d) {
        const int v = cntS[d * ntc + c];
        if (!a.count_masks || v) sp.cnt[(int64_t)d * nc + cg] = v;
        if (v) {
          mask |= 1u << d;
          atomicAdd(&arrS[(lkk + d / 3) * AW + (li + d % 3)], v);
        }
      }
      if (a.count_masks) sp.cmask[cg] = (uint16_t)mask;
    }
  }
  fold_tile<PUSH, kTileOnly>(a, Lo, acc, Ho, Hn, i0, k0, nearx, nearz);
  if constexpr (PUSH) {
    __syncthreads();  // (the count pass sums the arrivals in LDS)
    add_arrivals<true>(a, arrL, i0, k0);
  }
}

// Four waves per SIMD in every form (at most 128 VGPRs).
template <bool PUSH, bool MIXED, bool IDS, bool PW, bool DIRECT = false>
__global__ __launch_bounds__(kMaxWaves * 64) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_particles(const StepArgs a) {
  // clear the next order's tile flags (set by the scan of this cycle's sort); the grid has a
  // block for every tile index
  if (threadIdx.x == 0 && (int)blockIdx.x < a.t.ntiles) a.tile_active_next[blockIdx.x] = 0;
  // (said to be uniform: after a branch on the thread the compiler takes the tile, and with it
  // the loop over the tile's groups, to differ between lanes, and keeps both in vector registers)
  const int tile = __builtin_amdgcn_readfirstlane(block_tile(a.t, a.tile_list));
  if (tile < 0) return;
  particles_body<PUSH, MIXED, IDS, PW, DIRECT>(a, tile);
}

// The lane-run form of the mixed kernel (about 150 VGPRs: three waves per SIMD).
template <bool PUSH, bool IDS, bool PW>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3, 3)))
void k_particles_runs(const StepArgs a) {
  if (threadIdx.x == 0 && (int)blockIdx.x < a.t.ntiles) a.tile_active_next[blockIdx.x] = 0;
  const int tile = block_tile(a.t, a.tile_list);
  if (tile < 0) return;
  runs_body<PUSH, IDS, PW>(a, tile);
}

// ------------------------------------------------------------------------------------------
// Sort
// ------------------------------------------------------------------------------------------

__device__ __forceinline__ int wave_incl_scan(int v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int y = __shfl_up(v, o, 64);
    if (lane >= o) v += y;
  }
  return v;
}

// Block-wide exclusive scan of one value per thread; returns the block total too.
__device__ int block_excl_scan(int v, int *sh, int *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int inc = wave_incl_scan(v, lane);
  if (lane == 63) sh[wave] = inc;
  __syncthreads();
  int off = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    if (w < wave) off += sh[w];
    tot += sh[w];
  }
  __syncthreads();
  *total = tot;
  return off + inc - v;
}

// Stable destinations of one tile's particles.  The destination base of every (cell, move code) of
// the tile is computed once into LDS; then the wavefronts take the tile's cells, LPC lanes per cell
// (64, or 16 where cells hold fewer particles), and walk each cell's slots LPC at a time, the codes
// of the next four chunks on their way.  The
// particles that stay (most) get consecutive slots from one ballot and a running base in a
// register; the others consecutive ranks per code from ballots of the code's bits, their bases
// counted on in the LDS table.  (The walk along tile rows in groups of 64 slots searched every
// lane's cell and ranked all codes alike: about 150 instructions per group, 101 us on 21M particles
// at 128 per cell, about 80 now.)
template <int LPC>
__device__ __forceinline__ void rank_body(const StepArgs &a, int tile, int species) {
  const GridArgs &g = a.g;
  const TileArgs &t = a.t;
  const SpeciesArgs &sp = a.sp[species];
  if (!sp.active) return;
  const int tzi = tile / t.ntx, txi = tile - tzi * t.ntx;
  const int i0 = txi * t.tx, k0 = tzi * t.tz;
  const int i1 = min(i0 + t.tx, g.nx), k1 = min(k0 + t.tz, g.nz);
  const int cw = i1 - i0, ch = k1 - k0, ncell = cw * ch;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
  extern __shared__ int ldsi[];
  const int RW = t.tx + 4, RH = t.tz + 4;  // ring of two cells: destinations +-1, their sources +-1
  int *btab = ldsi;                        // [cells][9]
  int *cst = btab + t.tx * t.tz * kMoveCodes;  // [cells]: first slot
  int *cen = cst + t.tx * t.tz;                // [cells]: end slot
  int *rcnt = cen + t.tx * t.tz;               // [9][ring]
  int *rcsn = rcnt + kMoveCodes * RW * RH;     // [ring]
  int *rkey = rcsn + RW * RH;                  // [ring]
  const int total = sp.cs_new[g.ncells];
  // counts of the tile and its ring (sources of the destinations reached from the tile),
  // next-order starts of the same region, and the slots of the tile's cells, staged in LDS; a
  // tile and its ring fit in the grid along an axis: wraps need one compare there
  const bool nearx = g.nx >= t.tx + 4, nearz = g.nz >= t.tz + 4;
  const SmallDiv div_rw(RW), div_tx(t.tx), div_tz(t.tz), div_cw(cw);
  for (int e = threadIdx.x; e < RW * RH; e += blockDim.x) {
    const int rz = div_rw.q(e), rx = e - rz * RW;
    int gi = i0 - 2 + rx;
    const int gk = wrap_t(k0 - 2 + rz, g.nz, nearz);
    bool in = true;
    if (g.bc_x == PIC_BC_PERIODIC) gi = wrap_t(gi, g.nx, nearx); else in = gi >= 0 && gi < g.nx;
    // The counts are valid only in tiles that held particles (the tile flag); they are
    // loaded together with the flag (from a cell inside the grid) and kept or dropped after.
    const int gic = min(max(gi, 0), g.nx - 1);
    const int64_t c = (int64_t)gk * g.nx + gic;
    const bool act = in && a.tile_active[div_tz.q(gk) * t.ntx + div_tx.q(gic)] != 0;
    int v[kMoveCodes];
#pragma unroll
    for (int d = 0; d < kMoveCodes; ++d) v[d] = sp.cnt[(int64_t)d * g.ncells + c];
    const int csn_c = sp.cs_new[c], csb = sp.cs[c], cse = sp.cs[c + 1];
#pragma unroll
    for (int d = 0; d < kMoveCodes; ++d) rcnt[d * RW * RH + e] = act ? v[d] : 0;
    rcsn[e] = in ? csn_c : 0;
    rkey[e] = in ? (int)c : -1;  // sort key of the cell; -1 outside an absorbing axis
    if (rx >= 2 && rx < cw + 2 && rz >= 2 && rz < ch + 2) {
      cst[(rz - 2) * cw + rx - 2] = csb;
      cen[(rz - 2) * cw + rx - 2] = cse;
    }
  }
  __syncthreads();
  // one (code, cell) pair per thread, consecutive threads on consecutive cells of one code
  // (so their LDS reads of the staged counts fall in different banks)
  const SmallDiv div_cells(ncell);
  for (int e = threadIdx.x; e < ncell * kMoveCodes; e += blockDim.x) {
    const int d = div_cells.q(e), cell = e - d * ncell;
    const int lk = div_cw.q(cell), li = cell - lk * cw;
    // First slot, in the next order, of the particles moving from this cell with code d:
    // the start of the destination cell plus the particles arriving there from source
    // cells earlier in the current (cell-sorted) order.  Destination and sources lie in
    // the ring, so they are found by ring offsets; the order uses the cells' sort keys.
    const int rc = (lk + 2) * RW + (li + 2);
    int b = 0;
    if (rcnt[d * RW * RH + rc] > 0) {
      const int rd = rc + (d / 3 - 1) * RW + (d % 3 - 1);  // destination
      if (rkey[rd] >= 0) {
        const int key_c = rkey[rc];
        b = rcsn[rd];
#pragma unroll
        for (int d2 = 0; d2 < kMoveCodes; ++d2) {
          const int rs = rd - (d2 / 3 - 1) * RW - (d2 % 3 - 1);  // source sending d2 to rd
          const int ks = rkey[rs];
          if (ks >= 0 && ks < key_c) b += rcnt[d2 * RW * RH + rs];
        }
      }
    }
    btab[cell * kMoveCodes + d] = b;
  }
  __syncthreads();
  // The walk: sub-wavefront `sub` of LPC lanes takes cells first, first + stride, ...
  constexpr int kSub = 64 / LPC;
  const int sub = lane / LPC, sl = lane & (LPC - 1), stride = nwaves * kSub;
  const uint64_t sub_mask = (LPC == 64 ? ~0ull : ((1ull << LPC) - 1ull) << (sub * LPC));
  const uint64_t lt_mask = ((1ull << lane) - 1ull) & sub_mask;
  int cell = wave * kSub + sub - stride, pos = 0, end = 0, base4 = 0;
  constexpr int kAhead = LPC == 64 ? 4 : 2;  // chunks of LPC slots whose codes are loaded together
  auto next_part = [&](int &c, int &p, int &e) {  // the part after (c, p, e); c >= ncell: none
    p += kAhead * LPC;
    while (p >= e) {
      c += stride;
      if (c >= ncell) break;
      p = cst[c];
      e = cen[c];
    }
  };
  auto load_codes = [&](int c, int p, int e, uint32_t out[kAhead]) {
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int j = p + q * LPC + sl;
      out[q] = c < ncell && j < e ? slot_code(a, sp, j) : (uint32_t)kAbsorbed;
    }
  };
  uint32_t lc[kAhead], lcn[kAhead];
  next_part(cell, pos, end);
  load_codes(cell, pos, end, lc);
  if (cell < ncell) base4 = btab[cell * kMoveCodes + 4];
  while (__any(cell < ncell)) {
    int ncl = cell, npos = pos, nend = end;
    if (cell < ncell) next_part(ncl, npos, nend);
    load_codes(ncl, npos, nend, lcn);
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int d = (int)(lc[q] & 15u), loc = (int)(lc[q] >> 4);
      const uint64_t stay = __ballot(d == 4) & sub_mask, move = __ballot(d != 4 && d < kMoveCodes);
      if (!__any(d < kMoveCodes)) continue;  // past the end of every cell
      int slot = base4 + __popcll(stay & lt_mask);
      if (move) {
        const bool m = d != 4 && d < kMoveCodes;
        // the lanes of the same cell with the same move code: one ballot per bit of the code
        uint64_t same = move & sub_mask;
#pragma unroll
        for (int bit = 0; bit < 4; ++bit) {
          const bool on = (d >> bit) & 1;
          const uint64_t w = __ballot(m && on);
          same &= on ? w : ~w;
        }
        if (m) {
          int *bt = btab + cell * kMoveCodes + d;
          slot = *bt + __popcll(same & lt_mask);
          // the last lane of each code carries the count to the cell's next chunk
          if ((same >> lane) == 1ull) *bt = slot + 1;
        }
        wave_sync();
      }
      if (d < kMoveCodes) {
        if (slot >= 0 && slot < total)
          sp.perm_new[slot] = loc;
        else
          atomicOr(a.flags, kFlagSlot);
      }
      base4 += __popcll(stay);
    }
    if (ncl != cell && ncl < ncell) base4 = btab[ncl * kMoveCodes + 4];
    cell = ncl;
    pos = npos;
    end = nend;
#pragma unroll
    for (int q = 0; q < kAhead; ++q) lc[q] = lcn[q];
  }
}

// Stable destinations with one thread per cell of an active tile (one species per block,
// wavefronts over runs of 64 cells).  A cell's particles that move with code d go, in the
// next order, to the start of the destination cell, plus the particles arriving there from
// source cells with a smaller key, plus their rank among the cell's earlier slots with code d.
// The thread computes that first slot for each code its cell uses, from the destination's
// next-order start and the counts of the destination's sources (read only for a source that
// holds particles in the current order: the counts of a cell without particles may be left
// from an earlier cycle), then walks its cell's slots in order.  Move codes are canonical
// after the wrap (one code per source and destination pair), so on grids one or two cells
// wide a source listed under two codes has a zero count under the other.  No LDS and no
// cross-lane work: for few particles per cell the per-tile staging of the other ranker costs more.
// MASKS: the particle kernel wrote each cell's mask of used codes and only the nonzero counts
// (most cells send every particle with one code), so a cell's own codes come from its mask
// and a source's count is read only where the source's mask has the code.
template <bool MASKS>
__device__ __forceinline__ void rank_cells_body(const StepArgs &a, int tile, int species) {
  const GridArgs &g = a.g;
  const TileArgs &t = a.t;
  const SpeciesArgs &sp = a.sp[species];
  if (!sp.active) return;
  const int tzi = tile / t.ntx, txi = tile - tzi * t.ntx;
  const int i0 = txi * t.tx, k0 = tzi * t.tz;
  const int cw = min(i0 + t.tx, g.nx) - i0, ch = min(k0 + t.tz, g.nz) - k0;
  const int ncell = cw * ch;
  const int total = sp.cs_new[g.ncells];
  const bool periodic_x = g.bc_x == PIC_BC_PERIODIC;
  const SmallDiv div_cw(cw);
  // the count a source cell sent with code d2, valid only if the source holds particles now
  // (with masks, read only where its mask has the code: the other counts are not written)
  auto source_count = [&](int sc, int d2) -> int {
    const int sb = sp.cs[sc], se = sp.cs[sc + 1];
    if constexpr (MASKS) {
      const uint32_t m = sp.cmask[sc];
      return (se > sb && ((m >> d2) & 1u)) ? sp.cnt[(int64_t)d2 * g.ncells + sc] : 0;
    } else {
      const int v = sp.cnt[(int64_t)d2 * g.ncells + sc];
      return se > sb ? v : 0;
    }
  };
  for (int e = threadIdx.x; e < ncell; e += blockDim.x) {
    const int lk = div_cw.q(e), li = e - lk * cw;
    const int ci = i0 + li, ck = k0 + lk;
    const int c = ck * g.nx + ci;
    // Issued together: the cell's slot range and used codes, its own next-order start, and
    // what the sources that precede it among the sources of its own cell as a destination
    // (code 4, the particles that stay) sent it: in key order these are the row below and the
    // left neighbour (codes 5 to 8); codes 0 to 3 come before it only through a wrap.
    const int cb = sp.cs[c], ce = sp.cs[c + 1];
    int cur[kMoveCodes];
    if constexpr (MASKS) {
      const uint32_t mc = sp.cmask[c];
#pragma unroll
      for (int d = 0; d < kMoveCodes; ++d) cur[d] = (int)((mc >> d) & 1u);
    } else {
#pragma unroll
      for (int d = 0; d < kMoveCodes; ++d) cur[d] = sp.cnt[(int64_t)d * g.ncells + c];
    }
    int stay = sp.cs_new[c];
    int pv[4], pb[4], pe[4];
    uint32_t pmk[4];
    bool pm[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int d2 = 5 + q;
      int si = ci - (d2 % 3 - 1), sk = ck - (d2 / 3 - 1);
      bool in = true;
      if (periodic_x) {
        if (si < 0) si += g.nx;
        if (si >= g.nx) si -= g.nx;
      } else {
        in = si >= 0 && si < g.nx;
      }
      if (sk < 0) sk += g.nz;
      const int sc = in ? sk * g.nx + si : c;
      pm[q] = in && sc < c;
      pb[q] = sp.cs[sc];
      pe[q] = sp.cs[sc + 1];
      if constexpr (MASKS) {
        pmk[q] = sp.cmask[sc];
        pv[q] = sc;
      } else {
        pmk[q] = ~0u;
        pv[q] = sp.cnt[(int64_t)d2 * g.ncells + sc];
      }
    }
    if (cb >= ce) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (pm[q] && pe[q] > pb[q] && ((pmk[q] >> (5 + q)) & 1u)) {
        if constexpr (MASKS)
          stay += sp.cnt[(int64_t)(5 + q) * g.ncells + pv[q]];
        else
          stay += pv[q];
      }
    }
    if (ck == g.nz - 1 || (periodic_x && ci == g.nx - 1)) {
#pragma unroll 1
      for (int d2 = 0; d2 < 4; ++d2) {
        int si = ci - (d2 % 3 - 1), sk = ck - (d2 / 3 - 1);
        bool in = true;
        if (periodic_x) {
          if (si < 0) si += g.nx;
          if (si >= g.nx) si -= g.nx;
        } else {
          in = si >= 0 && si < g.nx;
        }
        if (sk >= g.nz) sk -= g.nz;
        const int sc = sk * g.nx + si;
        if (in && sc < c) stay += source_count(sc, d2);
      }
    }
    // The other codes a cell uses (particles that change cell: few per cycle).  Away from the
    // grid's border the sources before this one among a destination's are those with the larger
    // codes: no wrap and no comparison needed (sort of 2048 x 2048 cells 240 -> 227 us).
    const bool inner = ci >= 2 && ci < g.nx - 2 && ck >= 2 && ck < g.nz - 2;
#pragma unroll
    for (int d = 0; d < kMoveCodes; ++d) {
      if (d == 4) {
        cur[d] = stay;
        continue;
      }
      if (cur[d] <= 0) continue;
      if (inner) {
        const int dc = c + (d / 3 - 1) * g.nx + (d % 3 - 1);
        int b = sp.cs_new[dc];
#pragma unroll
        for (int d2 = d + 1; d2 < kMoveCodes; ++d2)
          b += source_count(dc - (d2 / 3 - 1) * g.nx - (d2 % 3 - 1), d2);
        cur[d] = b;
        continue;
      }
      // destination (inside the grid: an absorbed particle has its own code)
      int di = ci + (d % 3 - 1), dk = ck + (d / 3 - 1);
      if (di < 0) di += g.nx;
      if (di >= g.nx) di -= g.nx;
      if (dk < 0) dk += g.nz;
      if (dk >= g.nz) dk -= g.nz;
      const int dc = dk * g.nx + di;
      int b = sp.cs_new[dc];
#pragma unroll 1
      for (int d2 = 0; d2 < kMoveCodes; ++d2) {
        // the source that sends code d2 to the destination
        int si = di - (d2 % 3 - 1), sk = dk - (d2 / 3 - 1);
        bool in = true;
        if (periodic_x) {
          if (si < 0) si += g.nx;
          if (si >= g.nx) si -= g.nx;
        } else {
          in = si >= 0 && si < g.nx;
        }
        if (sk < 0) sk += g.nz;
        if (sk >= g.nz) sk -= g.nz;
        const int sc = sk * g.nx + si;
        if (in && sc < c) b += source_count(sc, d2);
      }
      cur[d] = b;
    }
    // the cell's slots in order, four move codes loaded at a time
    for (int j = cb; j < ce; j += 4) {
      uint32_t lc[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) lc[q] = slot_code(a, sp, min(j + q, ce - 1));
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (j + q >= ce) break;
        const int d = (int)(lc[q] & 15u);
        int slot = -1;
#pragma unroll
        for (int dd = 0; dd < kMoveCodes; ++dd) {
          if (d == dd) {
            slot = cur[dd];
            cur[dd] = slot + 1;
          }
        }
        if (d < kMoveCodes) {
          if (slot >= 0 && slot < total) {
            sp.perm_new[slot] = (int)(lc[q] >> 4);
          } else {
            atomicOr(a.flags, kFlagSlot);
          }
        }
      }
    }
  }
}

// Flag per tile: does it hold particles of any species in the order given by the cell starts
// (the current order, or the next one when from_next is set).  One thread per tile.
__device__ __forceinline__ void tile_flags_body(const StepArgs &a, int tile, int from_next) {
  const GridArgs &g = a.g;
  const TileArgs &t = a.t;
  if (tile >= t.ntiles) return;
  const int tzi = tile / t.ntx, txi = tile - tzi * t.ntx;
  const int i0 = txi * t.tx, k0 = tzi * t.tz;
  const int i1 = min(i0 + t.tx, g.nx), k1 = min(k0 + t.tz, g.nz);
  int act = 0;
  for (int s = 0; s < a.nsp; ++s) {
    const SpeciesArgs &sp = a.sp[s];
    if (!sp.active) continue;
    const int32_t *cs = from_next ? sp.cs_new : sp.cs;
    for (int r = k0; r < k1; ++r) act |= cs[(int64_t)r * g.nx + i1] > cs[(int64_t)r * g.nx + i0];
  }
  a.tile_active_next[tile] = (uint8_t)act;
}

__global__ __launch_bounds__(kBlock) void k_tile_flags(const StepArgs a, int from_next) {
  tile_flags_body(a, blockIdx.x * blockDim.x + threadIdx.x, from_next);
}

// Ordered list of the flagged tiles, count at [ntiles].  One block; each thread takes a run of
// kPer consecutive flags (loaded together), one block-wide scan per pass places the runs.  The
// list order decides which block takes which tile: in tile order, the blocks of one XCD take
// neighbouring tiles.
__device__ __forceinline__ void tile_compact_body(const StepArgs &a) {
  __shared__ int sh[1024 / 64];
  // A pass takes 16 flags per thread (a 16-byte word; tb is a multiple of 16), counts them with
  // popcounts (flags are 0 or 1), places them with one block scan and writes the active tiles in
  // order.  (More flags per thread would raise the registers of the rank kernels, which run this
  // in one block beside their own.)
  constexpr int kPer = 16;
  const int ntiles = a.t.ntiles;
  const uint8_t *flags = a.tile_active_next;
  int carry = 0;
  for (int pbase = 0; pbase < ntiles; pbase += (int)blockDim.x * kPer) {
    const int tb = pbase + (int)threadIdx.x * kPer;
    uint32_t w[kPer / 4];
#pragma unroll
    for (int h = 0; h < kPer / 16; ++h) {
      const int w0 = tb + 16 * h;
      if (w0 + 16 <= ntiles) {
        const uint4 v = *reinterpret_cast<const uint4 *>(flags + w0);
        w[4 * h] = v.x;
        w[4 * h + 1] = v.y;
        w[4 * h + 2] = v.z;
        w[4 * h + 3] = v.w;
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t x = 0u;
          for (int b = 0; b < 4; ++b) {
            const int t = w0 + 4 * q + b;
            if (t < ntiles) x |= (uint32_t)flags[t] << (8 * b);
          }
          w[4 * h + q] = x;
        }
      }
    }
    int n = 0;
#pragma unroll
    for (int q = 0; q < kPer / 4; ++q) n += __popc(w[q]);
    int total;
    int pos = carry + block_excl_scan(n, sh, &total);
#pragma unroll
    for (int q = 0; q < kPer / 4; ++q) {
      uint32_t x = w[q];
      while (x) {
        const int bit = __ffs(x) - 1;  // the set bit is bit 0 of byte bit / 8
        a.tile_list_next[pos++] = tb + 4 * q + (bit >> 3);
        x &= x - 1u;
      }
    }
    carry += total;
  }
  if (threadIdx.x == 0) a.tile_list_next[ntiles] = carry;
}

__global__ __launch_bounds__(1024) void k_tile_compact(const StepArgs a) { tile_compact_body(a); }

// ---- scan of a cycle's sort -----------------------------------------------------------------
// Block bx of species s: the arrivals before its kScanBlock cells from the block sums, which the
// particle kernel makes beside the arrival counts, then the exclusive scan of its own counts
// (cleared for the next cycle) into the next order's cell starts, and the next order's tile flags
// (a tile is active when particles arrive in one of its cells; the particle kernel of the cycle
// cleared the flags).  One pass over the counts, without waiting for other blocks: a second
// kernel that added the block totals took 4 to 6 us a cycle on small grids and 32 us on 2048 x
// 2048 cells (the list of tiles was made there too).
__device__ __forceinline__ void scan_body(const StepArgs &a, int bx, int s) {
  __shared__ int sh[2 * kBlock / 64];
  const SpeciesArgs &sp = a.sp[s];
  if (!sp.active) return;
  const GridArgs &g = a.g;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t c0 = (int64_t)bx * kScanBlock + (int64_t)threadIdx.x * kScanItems;
  const bool whole = c0 + kScanItems <= g.ncells;
  static_assert(kScanItems == 4, "one int4 per thread");
  int in[kScanItems] = {0, 0, 0, 0};
  if (whole) {
    const int4 v = *reinterpret_cast<const int4 *>(sp.arr + c0);
    in[0] = v.x;
    in[1] = v.y;
    in[2] = v.z;
    in[3] = v.w;
  } else {
#pragma unroll
    for (int q = 0; q < kScanItems; ++q)
      if (c0 + q < g.ncells) in[q] = sp.arr[c0 + q];
  }
  // the sums of the blocks before this one (up to 16 per thread on a 2048 x 2048 grid): unrolled
  // so that a thread's loads are issued together
  int part = 0;
#pragma unroll 8
  for (int b = threadIdx.x; b < bx; b += kBlock) part += sp.bsum[b];
  const int sum = in[0] + in[1] + in[2] + in[3];
  const int inc = wave_incl_scan(sum, lane);
  part = wave_sums(part);
  if (lane == 63) {
    sh[wave] = inc;
    sh[kBlock / 64 + wave] = part;
  }
  if (sum) {
    if (whole) {
      *reinterpret_cast<int4 *>(sp.arr + c0) = make_int4(0, 0, 0, 0);
    } else {
#pragma unroll
      for (int q = 0; q < kScanItems; ++q)
        if (in[q]) sp.arr[c0 + q] = 0;
    }
    int k = (int)(c0 / g.nx), i = (int)(c0 - (int64_t)k * g.nx);
    const SmallDiv div_tx(a.t.tx), div_tz(a.t.tz);
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
      if (in[q] && k < g.nz) a.tile_active_next[div_tz.q(k) * a.t.ntx + div_tx.q(i)] = 1;
      if (++i == g.nx) {
        i = 0;
        ++k;
      }
    }
  }
  __syncthreads();
  int run = inc - sum, total = 0;
#pragma unroll
  for (int w = 0; w < kBlock / 64; ++w) {
    run += sh[kBlock / 64 + w] + (w < wave ? sh[w] : 0);
    total += sh[kBlock / 64 + w] + sh[w];
  }
  if (whole) {
    int4 v;
    v.x = run;
    v.y = v.x + in[0];
    v.z = v.y + in[1];
    v.w = v.z + in[2];
    *reinterpret_cast<int4 *>(sp.cs_new + c0) = v;
  } else {
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
      if (c0 + q < g.ncells) sp.cs_new[c0 + q] = run;
      run += in[q];
    }
  }
  if (bx == a.n_scan_blocks - 1 && threadIdx.x == 0) sp.cs_new[g.ncells] = total;
}

__global__ __launch_bounds__(kBlock) void k_scan(const StepArgs a) {
  scan_body(a, blockIdx.x, blockIdx.y);
}

// The block sums from the arrival counts, after a particle kernel that does not make them.
__global__ __launch_bounds__(kBlock) void k_block_sums(const StepArgs a) {
  __shared__ int sh[kBlock / 64];
  const SpeciesArgs &sp = a.sp[blockIdx.y];
  if (!sp.active) return;
  const int64_t c0 = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
  int v = 0;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q)
    if (c0 + q * kBlock < a.g.ncells) v += sp.arr[c0 + q * kBlock];
  v = wave_sums(v);
  if ((threadIdx.x & 63) == 63) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) sp.bsum[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

// What one extra block of the rank kernels does: the next order's tile list, and the block sums
// cleared for the next cycle.
__device__ __forceinline__ void sort_end_body(const StepArgs &a) {
  tile_compact_body(a);
  for (int s = 0; s < a.nsp; ++s)
    if (a.sp[s].active)
      for (int b = threadIdx.x; b < a.n_scan_blocks; b += blockDim.x) a.sp[s].bsum[b] = 0;
}

// (the extra block is the last of the first species: it starts before the other species' blocks)
__global__ __launch_bounds__(kBlock) void k_rank_cells(const StepArgs a) {
  if (blockIdx.x == gridDim.x - 1) {
    if (blockIdx.y == 0) sort_end_body(a);
    return;
  }
  const int tile = block_tile(a.t, a.tile_list);
  if (tile < 0) return;
  if (a.count_masks)
    rank_cells_body<true>(a, tile, blockIdx.y);
  else
    rank_cells_body<false>(a, tile, blockIdx.y);
}

template <int LPC>
__global__ __launch_bounds__(kBlock) void k_rank(const StepArgs a) {
  if (blockIdx.x == gridDim.x - 1) {
    if (blockIdx.y == 0) sort_end_body(a);
    return;
  }
  const int tile = block_tile(a.t, a.tile_list);
  if (tile < 0) return;
  rank_body<LPC>(a, tile, blockIdx.y);
}

// ------------------------------------------------------------------------------------------
// Batched cycle: every kernel launched once for all runs of a batch, one block per work item
// of all runs (a run's items are numbered after the previous runs'); the run of an item is
// found in the exclusive prefix of item counts.
// ------------------------------------------------------------------------------------------

// The run owning work item w: the last r with pre[r] <= w (pre is the exclusive prefix of the
// runs' item counts, non-decreasing, pre[0] = 0; a run without items is skipped).  The 64
// lanes of the wavefront each load one pivot, spaced evenly over the range left, and a ballot
// keeps the interval of the last pivot <= w: one memory round trip per factor 64 of runs
// (the item index is uniform across the wavefront, which must be whole).
__device__ __forceinline__ int find_run(const int32_t *pre, int nruns, int w) {
  const int lane = threadIdx.x & 63;
  int lo = 0, n = nruns;
  while (n > 1) {
    const int step = (n + 63) >> 6;
    const int idx = lo + lane * step;
    const bool le = idx < lo + n && pre[idx] <= w;
    const uint64_t m = __ballot(le);
    const int last = 63 - __clzll((long long)m);  // lane 0 holds pre[lo] <= w
    const int nlo = lo + last * step;
    n = min(step, lo + n - nlo);
    lo = nlo;
  }
  return lo;
}

// The argument tables are read through the constant address space: they do not change during
// a launch, so their fields can be loaded into scalar registers like kernel arguments.
__device__ __forceinline__ const StepArgs &run_step(const BatchArgs &b, int r, const int32_t *par) {
  const int p = par[r];
  const StepArgs __attribute__((address_space(4))) *t =
      (const StepArgs __attribute__((address_space(4))) *)(b.step);
  return *(const StepArgs *)(t + 2 * r + p);
}
__device__ __forceinline__ const FieldArgs &run_field(const BatchArgs &b, int r) {
  const int p = b.par[r];
  const FieldArgs __attribute__((address_space(4))) *t =
      (const FieldArgs __attribute__((address_space(4))) *)(b.field);
  return *(const FieldArgs *)(t + 2 * r + p);
}

// The field kernels' items (node and cell blocks of every run) do not change between
// rebuilds of the batch, so these launch one block per item, with the items of each XCD a
// contiguous band (as in a single run) instead of a persistent loop.
__global__ __launch_bounds__(kBlock) void kb_solve_e(const BatchArgs b, int total) {
  const int w = (int)xcd_band_block(total);
  if (w < 0) return;
  const int r = find_run(b.pre_nodes, b.nruns, w);
  const FieldArgs &fa = run_field(b, r);
  const double tE = (double)b.step_ctr[r] * fa.g.dt;
  solve_e_body(fa, tE, (int64_t)(w - b.pre_nodes[r]) * (kSolveNodes * kBlock) + threadIdx.x, kBlock);
}

// Work prefixes of the active tiles of every run's current order, and the parities' copy for the
// rank kernel (one block of the H update).
__device__ __forceinline__ void batch_prefix_body(const BatchArgs &b) {
  __shared__ int sh[kBlock / 64];
  int carry_t = 0, carry_r = 0;
  for (int base = 0; base < b.nruns; base += blockDim.x) {
    const int r = base + threadIdx.x;
    int nt = 0, nr = 0;
    if (r < b.nruns) {
      const StepArgs &sa = run_step(b, r, b.par);
      nt = sa.tile_list[sa.t.ntiles];
      nr = nt * sa.nsp;
      b.par_rank[r] = b.par[r];
    }
    int tot_t, tot_r;
    const int off_t = block_excl_scan(nt, sh, &tot_t);
    const int off_r = block_excl_scan(nr, sh, &tot_r);
    if (r < b.nruns) {
      b.pre_tiles[r] = carry_t + off_t;
      b.pre_rank[r] = carry_r + off_r;
    }
    carry_t += tot_t;
    carry_r += tot_r;
  }
  if (threadIdx.x == 0) {
    b.pre_tiles[b.nruns] = carry_t;
    b.pre_rank[b.nruns] = carry_r;
  }
}

__global__ __launch_bounds__(kBlock) void kb_update_h(const BatchArgs b, int total) {
  if (blockIdx.x == gridDim.x - 1) {
    batch_prefix_body(b);
    return;
  }
  const int w = (int)xcd_band_block(total);
  if (w < 0) return;
  const int r = find_run(b.pre_cells, b.nruns, w);
  update_h_body(run_field(b, r), (int64_t)(w - b.pre_cells[r]) * (kHCells * kBlock) + threadIdx.x, kBlock);
}

// The particle and rank kernels' items (active tiles, and tiles x species) change every cycle;
// they launch one block per item any run could have, and the blocks past the cycle's items
// return at once, so the hardware hands the items, of very unequal cost, to the CUs as they
// free up.  Block b takes item b: consecutive items (the tiles of one run) go to different
// XCDs.  (Contiguous bands of items per XCD, as in a single run, were measured slower: runs
// differ in cost, so the bands load the XCDs unequally.)
__device__ __forceinline__ int batch_item(int w, int total) { return w < total ? w : -1; }

// DIRECT: some member takes the direct form (a pass of 32 runs without one, 20 cycles: 9675 us, with
// the branch 9782).
template <bool MIXED, bool IDS, bool PW, bool DIRECT>
__global__ __launch_bounds__(kMaxWaves * 64) __attribute__((amdgpu_waves_per_eu(4, 4)))
void kb_particles(const BatchArgs b) {
  const int w = batch_item((int)blockIdx.x, b.pre_tiles[b.nruns]);
  if (w < 0) return;
  const int r = find_run(b.pre_tiles, b.nruns, w);
  const StepArgs &sa = run_step(b, r, b.par);
  const int tile = sa.tile_list[w - b.pre_tiles[r]];
  if (DIRECT && sa.direct)
    particles_body<true, MIXED, IDS, PW, true>(sa, tile);
  else
    particles_body<true, MIXED, IDS, PW>(sa, tile);
}

// The scan of every run's sort, over (run, species, block of cells) items, which are fixed between
// rebuilds: a block per item.  The next order's tile flags were cleared by the H update of the
// cycle.
__global__ __launch_bounds__(kBlock) void kb_scan(const BatchArgs b, int total) {
  const int w = (int)blockIdx.x;
  if (w >= total) return;
  const int r = find_run(b.pre_scan, b.nruns, w);
  const StepArgs &sa = run_step(b, r, b.par);
  const int li = w - b.pre_scan[r];
  const int s = li / sa.n_scan_blocks;
  scan_body(sa, li - s * sa.n_scan_blocks, s);
}

// The ranks, after one block per run for the end of its sort and of its cycle: buffer parity
// flipped and cycle counted (the kernel's other blocks read the parities' copy).
__global__ __launch_bounds__(kBlock) void kb_rank(const BatchArgs b) {
  if ((int)blockIdx.x < b.nruns) {
    const int r = (int)blockIdx.x;
    sort_end_body(run_step(b, r, b.par_rank));
    if (threadIdx.x == 0) {
      b.par[r] = b.par_rank[r] ^ 1;
      b.step_ctr[r] += 1;
    }
    return;
  }
  const int w = batch_item((int)blockIdx.x - b.nruns, b.pre_rank[b.nruns]);
  if (w < 0) return;
  const int r = find_run(b.pre_rank, b.nruns, w);
  const StepArgs &sa = run_step(b, r, b.par_rank);
  const int li = w - b.pre_rank[r];
  const int idx = li / sa.nsp;
  if (sa.rank_cells && sa.count_masks)
    rank_cells_body<true>(sa, sa.tile_list[idx], li - idx * sa.nsp);
  else if (sa.rank_cells)
    rank_cells_body<false>(sa, sa.tile_list[idx], li - idx * sa.nsp);
  else
    rank_body<16>(sa, sa.tile_list[idx], li - idx * sa.nsp);
}

__global__ void k_iota(int32_t *p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (int32_t)i;
}

}  // namespace

size_t particle_lds_bytes(const GridArgs &g, const TileArgs &t, bool mixed, int waves) {
  return TileLds(g.n_planes, t.tx, t.tz, mixed ? (int)sizeof(float) : (int)sizeof(double), waves).bytes;
}

size_t runs_lds_bytes(const GridArgs &g, const TileArgs &t, bool pw) {
  return RunsLds(g.n_planes, t.tx, t.tz, pw).bytes;
}

size_t rank_lds_bytes(const TileArgs &t) {
  const size_t ring = (size_t)(t.tx + 4) * (t.tz + 4);
  return ((size_t)t.tx * t.tz * (kMoveCodes + 2) + ring * (kMoveCodes + 2)) * sizeof(int);
}

hipError_t launch_field_solve(const FieldArgs &a, hipStream_t s) {
  const int64_t nb_nodes = (a.g.nnodes + kSolveNodes * kBlock - 1) / (kSolveNodes * kBlock);
  const int64_t nb_cells = (a.g.ncells + kHCells * kBlock - 1) / (kHCells * kBlock);
  hipLaunchKernelGGL(k_solve_e, dim3(8u * (unsigned)((nb_nodes + 7) / 8)), dim3(kBlock), 0, s, a, nb_nodes);
  hipLaunchKernelGGL(k_update_h, dim3(8u * (unsigned)((nb_cells + 7) / 8)), dim3(kBlock), 0, s, a, nb_cells);
  return hipGetLastError();
}

// The kernel instantiation of the direct and grouped forms for a cycle (push) or a deposit of the
// current state: precision, particle-id copy (push only) and per-particle densities.  A mixed run alone
// pushes in the direct form or in lane runs.
template <bool IDS, bool PW>
static void launch_tiles(const StepArgs &a, bool push, size_t lds, hipStream_t s) {
  const dim3 grid(8u * (unsigned)a.t.per_xcd), blk(64u * (unsigned)a.waves);
  if (a.mixed && push)
    hipLaunchKernelGGL((k_particles<true, true, IDS, PW, true>), grid, blk, lds, s, a);
  else if (a.mixed)
    hipLaunchKernelGGL((k_particles<false, true, false, PW>), grid, blk, lds, s, a);
  else if (!push)
    hipLaunchKernelGGL((k_particles<false, false, false, PW>), grid, blk, lds, s, a);
  else if (a.direct)
    hipLaunchKernelGGL((k_particles<true, false, IDS, PW, true>), grid, blk, lds, s, a);
  else
    hipLaunchKernelGGL((k_particles<true, false, IDS, PW>), grid, blk, lds, s, a);
}

static void launch_runs(const StepArgs &a, bool push, bool ids, bool pw, hipStream_t s) {
  const size_t lds = runs_lds_bytes(a.g, a.t, pw);
  const dim3 grid(8u * (unsigned)a.t.per_xcd), blk(kBlock);
  if (push && ids && pw)
    hipLaunchKernelGGL((k_particles_runs<true, true, true>), grid, blk, lds, s, a);
  else if (push && ids)
    hipLaunchKernelGGL((k_particles_runs<true, true, false>), grid, blk, lds, s, a);
  else if (push && pw)
    hipLaunchKernelGGL((k_particles_runs<true, false, true>), grid, blk, lds, s, a);
  else if (push)
    hipLaunchKernelGGL((k_particles_runs<true, false, false>), grid, blk, lds, s, a);
  else if (pw)
    hipLaunchKernelGGL((k_particles_runs<false, false, true>), grid, blk, lds, s, a);
  else
    hipLaunchKernelGGL((k_particles_runs<false, false, false>), grid, blk, lds, s, a);
}

hipError_t launch_particles(const StepArgs &a, bool push, hipStream_t s) {
  bool ids = false, pw = false;
  for (int q = 0; q < a.nsp; ++q) {
    ids = ids || a.sp[q].dst_id != nullptr;
    pw = pw || (a.sp[q].active && a.sp[q].w_stride != 0);
  }
  if (a.runs) {
    launch_runs(a, push, ids, pw, s);
    return hipGetLastError();
  }
  // the direct form has no staging
  const size_t lds = particle_lds_bytes(a.g, a.t, a.mixed != 0, push && a.direct ? 0 : a.waves);
  if (ids && pw)
    launch_tiles<true, true>(a, push, lds, s);
  else if (ids)
    launch_tiles<true, false>(a, push, lds, s);
  else if (pw)
    launch_tiles<false, true>(a, push, lds, s);
  else
    launch_tiles<false, false>(a, push, lds, s);
  return hipGetLastError();
}

hipError_t launch_sort(const StepArgs &a, hipStream_t s) {
  const dim3 scan((unsigned)a.n_scan_blocks, (unsigned)a.nsp);
  if (!a.block_sums) hipLaunchKernelGGL(k_block_sums, scan, dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_scan, scan, dim3(kBlock), 0, s, a);
  const dim3 grid(8u * (unsigned)a.t.per_xcd + 1u, (unsigned)a.nsp);
  if (a.rank_cells) {
    // one thread per cell of a tile, at most a full block
    const int cells = a.t.tx * a.t.tz;
    const int rounded = (cells + 63) / 64 * 64;
    const unsigned threads = (unsigned)(rounded < kBlock ? rounded : kBlock);
    hipLaunchKernelGGL(k_rank_cells, grid, dim3(threads), 0, s, a);
  } else {
    if (a.dense)
      hipLaunchKernelGGL(k_rank<64>, grid, dim3(kBlock), rank_lds_bytes(a.t), s, a);
    else
      hipLaunchKernelGGL(k_rank<16>, grid, dim3(kBlock), rank_lds_bytes(a.t), s, a);
  }
  return hipGetLastError();
}

hipError_t launch_tile_list(const StepArgs &a, bool from_next_order, hipStream_t s) {
  const unsigned ntb = (unsigned)((a.t.ntiles + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(k_tile_flags, dim3(ntb), dim3(kBlock), 0, s, a, from_next_order ? 1 : 0);
  hipLaunchKernelGGL(k_tile_compact, dim3(1), dim3(1024), 0, s, a);
  return hipGetLastError();
}

typedef void (*BatchParticlesKernel)(BatchArgs);

// The batched particle kernel instantiation: precision, particle-id copy, per-particle densities and
// whether some member takes the direct form.
template <bool MIXED, bool IDS, bool PW>
static BatchParticlesKernel batch_particles_kernel(bool direct) {
  return direct ? kb_particles<MIXED, IDS, PW, true> : kb_particles<MIXED, IDS, PW, false>;
}
template <bool MIXED>
static BatchParticlesKernel batch_particles_kernel(const BatchLaunch &l) {
  if (l.ids) return l.pw ? batch_particles_kernel<MIXED, true, true>(l.direct) : batch_particles_kernel<MIXED, true, false>(l.direct);
  return l.pw ? batch_particles_kernel<MIXED, false, true>(l.direct) : batch_particles_kernel<MIXED, false, false>(l.direct);
}

hipError_t launch_batch_cycle(const BatchArgs &b, const BatchLaunch &l, hipStream_t s) {
  const dim3 blk(kBlock);
  hipLaunchKernelGGL(kb_solve_e, dim3(8u * (unsigned)std::max(1, (l.items_nodes + 7) / 8)), blk, 0,
                     s, b, l.items_nodes);
  hipLaunchKernelGGL(kb_update_h, dim3(8u * (unsigned)std::max(1, (l.items_cells + 7) / 8) + 1u), blk, 0,
                     s, b, l.items_cells);
  const dim3 gp((unsigned)l.grid_particles);
  hipLaunchKernelGGL(l.mixed ? batch_particles_kernel<true>(l) : batch_particles_kernel<false>(l), gp, dim3(64u * (unsigned)l.waves),
                     l.lds_particles, s, b);
  hipLaunchKernelGGL(kb_scan, dim3((unsigned)std::max(1, l.items_scan)), blk, 0, s, b, l.items_scan);
  hipLaunchKernelGGL(kb_rank, dim3((unsigned)(b.nruns + l.grid_rank)), blk, l.lds_rank, s, b);
  return hipGetLastError();
}

hipError_t launch_iota(int32_t *p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_iota, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace pic
