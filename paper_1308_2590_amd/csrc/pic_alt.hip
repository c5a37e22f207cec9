// HIP kernels (gfx950) for the mover options and the energy diagnostic.
//
//   k_particles_alt  the particle stage of a cycle with a mover option (FP64): one thread per
//                    sorted slot; gather E-bar (bilinear from the 4 corner nodes), B at the
//                    particle (its cell's H, or bilinear from the 4 surrounding cell centres),
//                    gamma-bar (gamma(u^n), or gamma(u^n + beta E^n) with E^n interpolated at
//                    the particle), the implicit push of Eq. (2), position advance and move
//                    code, then the deposit of S-hat, delta-j and density (Step 1, Eq. (3)) at
//                    the new position with the same options, into the global moment planes with
//                    FP64 atomics, each value first summed over a block's particles per cell
//                    (matrix cores, then LDS) and over the cells around a node, or, for few
//                    particles per cell, over a wavefront's runs of one cell (shuffles).  It
//                    writes the move codes, counts and arrivals the cycle's sort reads, exactly as
//                    the tile kernel does.  Without push it deposits the current state.
//   k_energy         field energy (1/2)(sum |E|^2 over nodes + sum |H|^2 over cells) dx dz and
//                    kinetic energy sum w m (gamma - 1) dx dz per species.
//
// The options are two readings of what the paper leaves open (the Lorentz factor inside the
// linearised mover and B at a particle when H is cell-centred).  Per-particle B makes S-hat
// differ from particle to particle, so these kernels deposit each particle's expanded moments
// instead of per-cell sums; they trade speed for the choice.

#include <algorithm>
#include <mutex>

#include "pic_device.h"
#include "pic_internal.h"

namespace pic {
namespace {

// The four corner nodes of cell (i, k) (order (i,k), (i+1,k), (i,k+1), (i+1,k+1)) and the
// linear weights of offsets (fx, fz).
__device__ __forceinline__ void corners(const GridArgs &g, int i, int k, double fx, double fz,
                                        int64_t node[4], double W[4]) {
  const int i1 = g.bc_x == PIC_BC_PERIODIC ? wrap1(i + 1, g.nx) : i + 1;
  const int k1 = wrap1(k + 1, g.nz);
  node[0] = (int64_t)k * g.nxn + i;
  node[1] = (int64_t)k * g.nxn + i1;
  node[2] = (int64_t)k1 * g.nxn + i;
  node[3] = (int64_t)k1 * g.nxn + i1;
  W[0] = (1.0 - fx) * (1.0 - fz);
  W[1] = fx * (1.0 - fz);
  W[2] = (1.0 - fx) * fz;
  W[3] = fx * fz;
}

__device__ __forceinline__ double at_nodes(const double *f, const int64_t node[4], const double W[4]) {
  return W[0] * f[node[0]] + W[1] * f[node[1]] + W[2] * f[node[2]] + W[3] * f[node[3]];
}

// B at position (x, z) in cell (i, k) from the cell-centred planes H.
__device__ void b_at(const GridArgs &g, const double *H, int mover, double x, double z, int i,
                     int k, double B[3]) {
  const int64_t nc = g.ncells;
  if (!(mover & PIC_MOVER_B_BILINEAR)) {
    const int64_t c = (int64_t)k * g.nx + i;
    for (int r = 0; r < 3; ++r) B[r] = H[r * nc + c];
    return;
  }
  const double sx = x - 0.5, sz = z - 0.5;
  const int ic = (int)floor(sx), kc = (int)floor(sz);
  const double gx = sx - (double)ic, gz = sz - (double)kc;
  int ci[2], ck[2];
  for (int t = 0; t < 2; ++t) {
    const int ii = ic + t;
    ci[t] = g.bc_x == PIC_BC_PERIODIC ? wrap1(ii, g.nx) : min(max(ii, 0), g.nx - 1);
    ck[t] = wrap1(kc + t, g.nz);
  }
  const double Wc[4] = {(1.0 - gx) * (1.0 - gz), gx * (1.0 - gz), (1.0 - gx) * gz, gx * gz};
  const int64_t c4[4] = {(int64_t)ck[0] * g.nx + ci[0], (int64_t)ck[0] * g.nx + ci[1],
                         (int64_t)ck[1] * g.nx + ci[0], (int64_t)ck[1] * g.nx + ci[1]};
  for (int r = 0; r < 3; ++r)
    B[r] = Wc[0] * H[r * nc + c4[0]] + Wc[1] * H[r * nc + c4[1]] + Wc[2] * H[r * nc + c4[2]] +
           Wc[3] * H[r * nc + c4[3]];
}

// gamma-bar for momentum u at a particle with corner nodes/weights: gamma(u), or with the
// predictor gamma(u + beta E) for E interpolated from the planes En.
__device__ double gamma_bar(const GridArgs &g, const double *En, int mover, double beta,
                            const double u[3], const int64_t node[4], const double W[4]) {
  if (!(mover & PIC_MOVER_GAMMA_PREDICT)) return sqrt(1.0 + u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
  double um[3];
  for (int r = 0; r < 3; ++r) um[r] = u[r] + beta * at_nodes(En + r * g.nnodes, node, W);
  return sqrt(1.0 + um[0] * um[0] + um[1] * um[1] + um[2] * um[2]);
}

// One particle's S-hat (9), delta-j (3) and density: with s = beta / gamma-bar and
// D = 1 + s^2 B.B, S-hat = (w q^2 dt^2 / (4 m gamma-bar D)) (I + s [B]x + s^2 B B^T) and
// delta-j = (w q / (gamma-bar D)) (u + s u x B + s^2 (B.u) B), w the particle's density (wp
// when the species carries one per particle).
__device__ void moments13(const SpeciesArgs &sp, double gam, const double u[3], const double B[3],
                          double wp, double v[13]) {
  const double sg = sp.beta / gam;
  const double inv = 1.0 / (1.0 + sg * sg * (B[0] * B[0] + B[1] * B[1] + B[2] * B[2]));
  const double cS = sp.w_stride ? sp.cS1 * wp : sp.cS;
  const double kJ = sp.w_stride ? sp.kJ1 * wp : sp.kJ;
  const double a0 = cS / gam * inv, a1 = a0 * sg, a2 = a1 * sg;
  const double kk = kJ / gam * inv;
  const double bu = B[0] * u[0] + B[1] * u[1] + B[2] * u[2];
  v[0] = a2 * B[0] * B[0] + a0;
  v[1] = a2 * B[0] * B[1] + a1 * B[2];
  v[2] = a2 * B[0] * B[2] - a1 * B[1];
  v[3] = a2 * B[1] * B[0] - a1 * B[2];
  v[4] = a2 * B[1] * B[1] + a0;
  v[5] = a2 * B[1] * B[2] + a1 * B[0];
  v[6] = a2 * B[2] * B[0] + a1 * B[1];
  v[7] = a2 * B[2] * B[1] - a1 * B[0];
  v[8] = a2 * B[2] * B[2] + a0;
  v[9] = kk * (u[0] + sg * (u[1] * B[2] - u[2] * B[1]) + sg * sg * bu * B[0]);
  v[10] = kk * (u[1] + sg * (u[2] * B[0] - u[0] * B[2]) + sg * sg * bu * B[1]);
  v[11] = kk * (u[2] + sg * (u[0] * B[1] - u[1] * B[0]) + sg * sg * bu * B[2]);
  v[12] = sp.w_stride ? wp : sp.w;
}

// The threads of a wavefront follow the cell-sorted order, so lanes that add to the same
// addresses (one cell's nodes, counter or arrival count) are neighbours, and their contributions
// are summed before one global atomic per value: same-address atomics from the lanes of one cell
// would be serialised.  The moments, 4 corner weights times 13 values per particle, are contracted
// over the particles of a cell with v_mfma_f64_4x4x4_4b (lane 16 k + 4 b + i holds A[i][k] and
// B[k][i] of block b and receives D[i][j] in lane 16 i + 4 b + j), four instructions per round of
// four particles of each block of 16 lanes.  (Segmented sums by lane shuffles, 52 values times up
// to six steps of two 32-bit LDS permutes each, were bound by the LDS: 91 us for 524,288
// particles at 16 per cell, 52 us now with the accumulators below.)
constexpr int kAltPlanes = 15;  // f_x, f_z, the 13 values
constexpr int kAltPitch = 68;   // particle P at P + P / 16: the 16 lanes of an LDS pass hit 16 banks
constexpr int kAltWaveBytes = kAltPlanes * kAltPitch * 8 + 2 * 64 * 4 * 4 + 2 * 64 + 2 * 64 * 4;
// A block's particles lie in consecutive cells; the sums of the first kAltCells go to LDS
// accumulators per (cell, corner, value) first and from there to the nodes, each value once
// per block: the global atomics, executed at the memory side, were half of the kernel's time
// (16 particles per cell: 96 us with one set per wavefront block and cell, 44 without any).  (400 x
// 400 cells at 10 per cell, where a block fills 26 or 27: 522 us without accumulators for any of
// them, 327 so; 26 accumulators leave two blocks per CU instead of three, 16 per cell 430 -> 508.)
constexpr int kAltCells = 24;
constexpr int kAltVals = 13;

struct AltStage {
  double *v;        // [kAltPlanes][kAltPitch]
  uint32_t *seg;    // [64][4]: corner nodes of the cell of pass p of block b at 16 b + p
  uint32_t *mov;    // [64][4]: corner nodes of mover m
  int *segc, *movc; // [64]: the cells
  uint8_t *movq;    // [64]: the mover's place in the planes
  uint8_t *pass;    // [64]: pass of particle 16 b + 4 t + k at 16 b + 4 k + t (255: none)
  __device__ __forceinline__ explicit AltStage(char *p)
      : v(reinterpret_cast<double *>(p)),
        seg(reinterpret_cast<uint32_t *>(p + kAltPlanes * kAltPitch * 8)),
        mov(seg + 256),
        segc(reinterpret_cast<int *>(mov + 256)),
        movc(segc + 64),
        movq(reinterpret_cast<uint8_t *>(movc + 64)),
        pass(movq + 64) {}
};

// Deposit of a wavefront's particles, one per lane: val = f_x, f_z and the 13 values (dep lanes).
// act: lanes with a slot; stay: the particle deposits in the cell its slot is in (node_src: its
// corner nodes), otherwise, if dep, in another (node_dst).  head_b: first lane of its cell in its
// block of 16.  A pass takes one cell per block, the other particles' weights masked to zero;
// movers go one by one, four at a time (16 lanes: corner, value).  acc: the block's accumulators,
// for the cells c0 .. c0 + span - 1 (span 0: none), everything else goes to the planes M.
__device__ __forceinline__ void alt_deposit(const AltStage &st, bool act, bool dep, bool stay, bool head_b,
                                            int src, int dst, const uint32_t node_src[4],
                                            const uint32_t node_dst[4], const double val[kAltPlanes],
                                            double *M, int64_t nn, int splane, double *acc, int c0,
                                            int span) {
  const int lane = threadIdx.x & 63;
  const int mi = lane & 3, mb = (lane >> 2) & 3, mk4 = lane >> 4;
  const int ob = lane >> 4, ol = lane & 15, own = lane + (lane >> 4);
  const bool mover = dep && !stay;
  const uint64_t heads = __ballot(act && head_b), movers = __ballot(mover);
  auto in_block = [](uint64_t m, int b) { return (uint32_t)(m >> (16 * b)) & 0xffffu; };
  const int seg = __popc(in_block(heads, ob) & ((2u << ol) - 1u)) - 1;
  const int mseq = __popcll(movers & ((1ull << lane) - 1ull));
  if (act && head_b) {
#pragma unroll
    for (int c = 0; c < 4; ++c) st.seg[(ob * 16 + seg) * 4 + c] = node_src[c];
    st.segc[ob * 16 + seg] = src;
  }
  if (mover) {
#pragma unroll
    for (int c = 0; c < 4; ++c) st.mov[mseq * 4 + c] = node_dst[c];
    st.movq[mseq] = (uint8_t)own;
    st.movc[mseq] = dst;
  }
  st.pass[ob * 16 + (ol & 3) * 4 + (ol >> 2)] = (uint8_t)(dep && stay ? seg : 255);
#pragma unroll
  for (int q = 0; q < kAltPlanes; ++q) st.v[q * kAltPitch + own] = dep ? val[q] : 0.0;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  int n_pass = 0;
#pragma unroll
  for (int b = 0; b < 4; ++b) n_pass = max(n_pass, __popc(in_block(heads, b)));
  const int n_mine = __popc(in_block(heads, mb)), n_movers = __popcll(movers);
  // value 4 q + j of this lane's column j (the fourth set holds the density alone), its plane
  int pl[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) pl[q] = (2 + min(4 * q + mi, 12)) * kAltPitch;
  // value 4 q + j at corner c of cell `cell` (node n): to the block's accumulators or the planes
  auto add = [&](int q, int c, int cell, uint32_t n, double v) {
    if (q == 3 && mi != 0) return;
    const uint32_t l = (uint32_t)(cell - c0);
    if (l < (uint32_t)span)
      atomicAdd(&acc[(l * 4 + c) * kAltVals + 4 * q + mi], v);
    else
      unsafeAtomicAdd(M + (int64_t)(q < 3 ? 4 * q + mi : splane) * nn + n, v);
  };
  {
    const int at = mb * 17 + mk4;
    const uint32_t pass4 = *reinterpret_cast<const uint32_t *>(st.pass + 16 * mb + 4 * mk4);
    double A[4], B[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const double fx = st.v[at + 4 * t], fz = st.v[kAltPitch + at + 4 * t];
      A[t] = ((mi & 1) ? fx : 1.0 - fx) * ((mi & 2) ? fz : 1.0 - fz);
#pragma unroll
      for (int q = 0; q < 4; ++q) B[q][t] = st.v[pl[q] + at + 4 * t];
    }
    for (int p = 0; p < n_pass; ++p) {
      const int ps = mb * 16 + min(p, max(n_mine - 1, 0));
      const uint32_t n = st.seg[ps * 4 + mk4];
      const int cell = st.segc[ps];
      double d[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const double w = ((pass4 >> (8 * t)) & 255u) == (uint32_t)p ? A[t] : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) d[q] = __builtin_amdgcn_mfma_f64_4x4x4f64(w, B[q][t], d[q], 0, 0, 0);
      }
      if (p < n_mine) {
#pragma unroll
        for (int q = 0; q < 4; ++q) add(q, mk4, cell, n, d[q]);
      }
    }
  }
  for (int m = mk4; m < n_movers; m += 4) {
    const int q0 = st.movq[m];
    const uint32_t n = st.mov[m * 4 + mb];
    const int cell = st.movc[m];
    const double fx = st.v[q0], fz = st.v[kAltPitch + q0];
    const double w = ((mb & 1) ? fx : 1.0 - fx) * ((mb & 2) ? fz : 1.0 - fz);
#pragma unroll
    for (int q = 0; q < 4; ++q) add(q, mb, cell, n, w * st.v[pl[q] + q0]);
  }
}

// Few particles per cell: a block's 256 particles fill many more cells than the accumulators hold, and
// the matrix cores take a pass per cell of a few particles.  There the values are summed over each
// run of lanes with one cell by shuffles towards its first lane, few steps for short runs, which
// issues one global atomic per value.  All 64 lanes take part; a lane without a value has a key of
// its own (negative).
struct Seg {
  int lane, seg_end, steps;
  bool head;
};

__device__ __forceinline__ Seg seg_of(int key) {
  const int lane = threadIdx.x & 63;
  const int prev = __shfl_up(key, 1, 64);
  const bool head = lane == 0 || prev != key;
  const uint64_t heads = __ballot(head);
  const uint64_t above = heads & ~((2ull << lane) - 1ull);
  Seg sg{lane, above ? __ffsll((unsigned long long)above) - 1 : 64, 0, head};
  while (sg.steps < 6 && __any(lane + (1 << sg.steps) < sg.seg_end)) ++sg.steps;
  return sg;
}

__device__ __forceinline__ double seg_sum(const Seg &sg, double v) {
  for (int q = 0; q < sg.steps; ++q) {
    const int d = 1 << q;
    const double t = __shfl_down(v, d, 64);
    if (sg.lane + d < sg.seg_end) v += t;
  }
  return v;
}

// SPARSE: the deposit by shuffles (see Seg), without LDS.
template <bool PUSH, bool SPARSE>
__global__ __launch_bounds__(kBlock) void k_particles_alt(const StepArgs a, int mover) {
  const GridArgs &g = a.g;
  // the next order's tile flags are set by the sort's scan; every node may hold deposits
  if (blockIdx.y == 0) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (PUSH)
      for (int64_t t = t0; t < a.t.ntiles; t += stride) a.tile_active_next[t] = 0;
    if (a.mflag)
      for (int64_t f = t0; f < (a.g.nnodes + kFlagNodes - 1) / kFlagNodes; f += stride) a.mflag[f] = 1;
  }
  const int s = blockIdx.y;
  const SpeciesArgs &sp = a.sp[s];
  if (!sp.active) return;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = sp.cs[g.ncells];
  if ((int)(blockIdx.x * blockDim.x) >= n) return;  // the whole block past the particles
  __shared__ __align__(16) char lds[SPARSE ? 16 : (kBlock / 64) * kAltWaveBytes];
  __shared__ double acc[SPARSE ? 1 : kAltCells * 4 * kAltVals];
  __shared__ int range[2];  // first and last cell of the block
  if constexpr (!SPARSE)
    for (int e = threadIdx.x; e < kAltCells * 4 * kAltVals; e += blockDim.x) acc[e] = 0.0;
  const int lane = threadIdx.x & 63;
  // the particle's old cell (act), whether it deposits (dep) and where: its old cell (stay) or not
  bool act = false, dep = false, stay = false;
  int src = -1, dst = -1;
  uint32_t code = 4u;
  uint32_t node_src[4] = {0u, 0u, 0u, 0u}, node_dst[4] = {0u, 0u, 0u, 0u};
  double val[kAltPlanes];
#pragma unroll
  for (int r = 0; r < kAltPlanes; ++r) val[r] = 0.0;
  if (j < n) {
    const int p = sp.perm[j];
    const double x = sp.src[0][p], z = sp.src[1][p];
    const double u[3] = {sp.src[2][p], sp.src[3][p], sp.src[4][p]};
    const double wp = sp.w_stride ? sp.src_w[p] : sp.w;
    const int i = (int)floor(x), k = (int)floor(z);
    if (i < 0 || i >= g.nx || k < 0 || k >= g.nz) {
      atomicOr(a.flags, kFlagOrder);
      if (PUSH) reinterpret_cast<uint8_t *>(sp.locode)[j] = kAbsorbed;
    } else {
      int64_t node[4];
      double W[4], v[13];
      corners(g, i, k, x - (double)i, z - (double)k, node, W);
#pragma unroll
      for (int c = 0; c < 4; ++c) node_src[c] = (uint32_t)node[c];
      act = true;
      src = dst = k * g.nx + i;
      double B[3];
      b_at(g, a.Hold, mover, x, z, i, k, B);
      const double gam = gamma_bar(g, a.Eold, mover, sp.beta, u, node, W);
      if (!PUSH) {
        moments13(sp, gam, u, B, wp, v);
        dep = stay = true;
        val[0] = x - (double)i;
        val[1] = z - (double)k;
#pragma unroll
        for (int r = 0; r < 13; ++r) val[2 + r] = v[r];
      } else {
        // E-bar at the particle and the implicit push: a = u + beta E-bar, b = beta B / gamma-bar,
        // u-bar = (a + a x b + (a.b) b) / (1 + b.b), u' = 2 u-bar - u
        const int64_t nn = g.nnodes;
        double Eb[3];
        for (int r = 0; r < 3; ++r) {
          const double *eo = a.Eold + r * nn, *en = a.Enew + r * nn;
          double acc = 0.0;
          for (int c = 0; c < 4; ++c) acc += W[c] * (0.5 * (eo[node[c]] + en[node[c]]));
          Eb[r] = acc;
        }
        const double bx = sp.beta / gam * B[0], by = sp.beta / gam * B[1], bz = sp.beta / gam * B[2];
        const double a0 = u[0] + sp.beta * Eb[0], a1 = u[1] + sp.beta * Eb[1], a2 = u[2] + sp.beta * Eb[2];
        const double inv = 1.0 / (1.0 + bx * bx + by * by + bz * bz);
        const double ab = a0 * bx + a1 * by + a2 * bz;
        double un[3];
        un[0] = 2.0 * ((a0 + (a1 * bz - a2 * by) + ab * bx) * inv) - u[0];
        un[1] = 2.0 * ((a1 + (a2 * bx - a0 * bz) + ab * by) * inv) - u[1];
        un[2] = 2.0 * ((a2 + (a0 * by - a1 * bx) + ab * bz) * inv) - u[2];
        const double g1 = sqrt(1.0 + un[0] * un[0] + un[1] * un[1] + un[2] * un[2]);
        double xn = x + g.cx * (un[0] / g1), zn = z + g.cz * (un[2] / g1);
        bool alive = true;
        if (g.bc_x == PIC_BC_PERIODIC) {
          if (xn < 0.0) xn += (double)g.nx;
          if (xn >= (double)g.nx) xn -= (double)g.nx;
        } else if (xn < 0.0 || xn >= (double)g.nx) {
          alive = false;
        }
        if (zn < 0.0) zn += (double)g.nz;
        if (zn >= (double)g.nz) zn -= (double)g.nz;
        const bool finite = isfinite(g1) && isfinite(xn) && isfinite(zn);
        if (!finite) atomicOr(a.flags, kFlagNonFinite);
        alive = alive && finite;
        const int i2 = finite ? (int)floor(xn) : i, k2 = finite ? (int)floor(zn) : k;
        int di = i2 - i, dk = k2 - k;
        if (di > 1) di -= g.nx;
        if (di < -1) di += g.nx;
        if (dk > 1) dk -= g.nz;
        if (dk < -1) dk += g.nz;
        const bool jump = di < -1 || di > 1 || dk < -1 || dk > 1;
        if (alive && jump) atomicOr(a.flags, kFlagJump);
        alive = alive && !jump;
        code = alive ? (uint32_t)((dk + 1) * 3 + (di + 1)) : kAbsorbed;
        // the pushed state goes to location j of the other buffer; the sort reads the codes
        sp.dst[0][j] = xn;
        sp.dst[1][j] = zn;
        sp.dst[2][j] = un[0];
        sp.dst[3][j] = un[1];
        sp.dst[4][j] = un[2];
        if (sp.dst_id) sp.dst_id[j] = sp.src_id[p];
        if (sp.w_stride) sp.dst_w[j] = wp;
        reinterpret_cast<uint8_t *>(sp.locode)[j] = (uint8_t)code;
        if (alive) {
          // the moments at x^{n+3/2} with u^{n+1}, B = H^{n+3/2} at the new position and
          // E^{n+1}
          corners(g, i2, k2, xn - (double)i2, zn - (double)k2, node, W);
          double B2[3];
          b_at(g, a.Hnew, mover, xn, zn, i2, k2, B2);
          const double gam2 = gamma_bar(g, a.Enew, mover, sp.beta, un, node, W);
          moments13(sp, gam2, un, B2, wp, v);
          dep = true;
          dst = k2 * g.nx + i2;
          stay = dst == src;
          val[0] = xn - (double)i2;
          val[1] = zn - (double)k2;
#pragma unroll
          for (int r = 0; r < 13; ++r) val[2 + r] = v[r];
#pragma unroll
          for (int c = 0; c < 4; ++c) node_dst[c] = (uint32_t)node[c];
        }
      }
    }
  }
  const int before = lane_before(src);  // (all lanes active)
  const bool head = act && (lane == 0 || before != src);
  if (PUSH) {
    // move counts and arrivals: the particles of a run that keep their cell together, the others
    // one by one
    const uint64_t stays = __ballot(dep && stay && code == 4u), heads = __ballot(head);
    const uint64_t above = heads & ~((2ull << lane) - 1ull);
    const uint64_t run = (above ? (above & -above) - 1ull : ~0ull) & ~((1ull << lane) - 1ull);
    const int n_stay = head ? __popcll(stays & run) : 0;
    if (n_stay > 0) {
      atomicAdd(&sp.cnt[4 * g.ncells + src], n_stay);
      atomicAdd(&sp.arr[src], n_stay);
    }
    if (dep && !(stay && code == 4u)) {
      atomicAdd(&sp.cnt[(int64_t)code * g.ncells + src], 1);
      atomicAdd(&sp.arr[dst], 1);
    }
  }
  if constexpr (SPARSE) {
    const Seg sd = seg_of(dep ? dst : -1 - lane);
    for (int c = 0; c < 4; ++c) {
      const double w = ((c & 1) ? val[0] : 1.0 - val[0]) * ((c & 2) ? val[1] : 1.0 - val[1]);
      const uint32_t node = stay ? node_src[c] : node_dst[c];
      for (int q = 0; q < kAltVals; ++q) {
        const double t = seg_sum(sd, w * val[2 + q]);
        if (dep && sd.head) unsafeAtomicAdd(a.M + (int64_t)(q < 12 ? q : 12 + s) * g.nnodes + node, t);
      }
    }
    return;
  }
  if (threadIdx.x == 0) range[0] = src;
  if (threadIdx.x == min((int)blockDim.x, n - (int)(blockIdx.x * blockDim.x)) - 1) range[1] = src;
  __syncthreads();
  // the block's first cells, in sorted order (a misplaced particle, flagged above, can be anywhere)
  const int c0 = range[0];
  const int span = c0 >= 0 && range[1] >= c0 ? min(range[1] - c0 + 1, kAltCells) : 0;
  const AltStage st(lds + (threadIdx.x >> 6) * kAltWaveBytes);
  // moments that are not finite go alone: in the group's sums they would reach other cells
  double all = 0.0;
#pragma unroll
  for (int q = 0; q < 12; ++q) all += val[2 + q];
  if (dep && !isfinite(all)) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double w = ((c & 1) ? val[0] : 1.0 - val[0]) * ((c & 2) ? val[1] : 1.0 - val[1]);
      const uint32_t n = stay ? node_src[c] : node_dst[c];
#pragma unroll
      for (int q = 0; q < kAltVals; ++q)
        unsafeAtomicAdd(a.M + (int64_t)(q < 12 ? q : 12 + s) * g.nnodes + n, w * val[2 + q]);
    }
    dep = false;
  }
  alt_deposit(st, act, dep, stay, head || (act && (lane & 15) == 0), src, dst, node_src, node_dst, val,
              a.M, g.nnodes, 12 + s, acc, c0, span);
  if (span == 0) return;  // (the same for the whole block)
  __syncthreads();
  // Node column l lies between the cells c0 + l - 1 and c0 + l: the left corners of the second
  // and the right ones of the first, one node each where the cells are neighbours in a row.
  for (int e = threadIdx.x; e < (span + 1) * 2 * kAltVals; e += blockDim.x) {
    const int v = e % kAltVals, up = e / kAltVals % 2, l = e / (2 * kAltVals);
    double left = l < span ? acc[(l * 4 + 2 * up) * kAltVals + v] : 0.0;
    const double right = l > 0 ? acc[((l - 1) * 4 + 2 * up + 1) * kAltVals + v] : 0.0;
    double *M = a.M + (int64_t)(v < 12 ? v : 12 + s) * g.nnodes;
    const int cr = c0 + l - 1;  // the cell with the right corners
    const bool joined = l > 0 && l < span && (cr + 1) % g.nx != 0;
    if (joined) left += right;
    if (left != 0.0) {
      const int k = (c0 + l) / g.nx, i = c0 + l - k * g.nx;
      unsafeAtomicAdd(M + (int64_t)(up ? wrap1(k + 1, g.nz) : k) * g.nxn + i, left);
    }
    if (!joined && right != 0.0) {
      const int k = cr / g.nx, i = cr - k * g.nx;
      const int i1 = g.bc_x == PIC_BC_PERIODIC ? wrap1(i + 1, g.nx) : i + 1;
      unsafeAtomicAdd(M + (int64_t)(up ? wrap1(k + 1, g.nz) : k) * g.nxn + i1, right);
    }
  }
}

// Energies: out[0] field, out[1 + s] kinetic of species s (both times dx dz), summed over
// blocks with FP64 atomics.
__device__ __forceinline__ double block_sum(double v, double *sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
  __syncthreads();
  return t;
}

__global__ __launch_bounds__(kBlock) void k_energy(const StepArgs a, const double *E,
                                                   const double *H, double *out) {
  __shared__ double sh[kBlock / 64];
  const GridArgs &g = a.g;
  const double area = g.dx * g.dz;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  double f = 0.0;
  for (int64_t e = tid; e < 3 * g.nnodes; e += stride) f += E[e] * E[e];
  for (int64_t e = tid; e < 3 * g.ncells; e += stride) f += H[e] * H[e];
  const double fs = block_sum(f, sh);
  if (threadIdx.x == 0) unsafeAtomicAdd(&out[0], 0.5 * fs * area);
  for (int s = 0; s < a.nsp; ++s) {
    const SpeciesArgs &sp = a.sp[s];
    if (!sp.active) continue;
    const int n = sp.cs[g.ncells];
    double kin = 0.0;
    for (int64_t j = tid; j < n; j += stride) {
      const int p = sp.perm[j];
      double u0, u1, u2;
      if (a.mixed) {
        u0 = (double)sp.msrc[2][p];
        u1 = (double)sp.msrc[3][p];
        u2 = (double)sp.msrc[4][p];
      } else {
        u0 = sp.src[2][p];
        u1 = sp.src[3][p];
        u2 = sp.src[4][p];
      }
      // the particle's density (one per species unless carried per particle)
      double wp = 1.0;
      if (sp.w_stride) wp = a.mixed ? (double)sp.msrc_w[p] : sp.src_w[p];
      kin += wp * (sqrt(1.0 + u0 * u0 + u1 * u1 + u2 * u2) - 1.0);
    }
    const double ks = block_sum(kin, sh);
    const double wsp = sp.w_stride ? 1.0 : sp.w;
    if (threadIdx.x == 0) unsafeAtomicAdd(&out[1 + s], ks * wsp * sp.m * area);
  }
}

// ---- energy without device allocation ----------------------------------------------------
// The same sums as k_energy, reduced in a fixed order: every block writes its partial sums
// (field, then each species slot) to its own row of a fixed buffer, and one block adds the rows
// in block order.  Every value is written before it is read, so nothing needs clearing, and
// the result does not depend on the timing of the blocks.

__global__ __launch_bounds__(kBlock) void k_energy_partials(const StepArgs a, const double *E,
                                                            const double *H, double *part) {
  __shared__ double sh[kBlock / 64];
  const GridArgs &g = a.g;
  const double area = g.dx * g.dz;
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  double *row = part + (size_t)blockIdx.x * kEnergyVals;
  double f = 0.0;
  for (int64_t e = tid; e < 3 * g.nnodes; e += stride) f += E[e] * E[e];
  for (int64_t e = tid; e < 3 * g.ncells; e += stride) f += H[e] * H[e];
  const double fs = block_sum(f, sh);
  if (threadIdx.x == 0) row[0] = 0.5 * fs * area;
  for (int s = 0; s < kMaxSpecies; ++s) {
    if (s >= a.nsp || !a.sp[s].active) {
      if (threadIdx.x == 0) row[1 + s] = 0.0;
      continue;
    }
    const SpeciesArgs &sp = a.sp[s];
    const int n = sp.cs[g.ncells];
    double kin = 0.0;
    for (int64_t j = tid; j < n; j += stride) {
      const int p = sp.perm[j];
      double u0, u1, u2, wp = 1.0;
      if (a.mixed) {
        u0 = (double)sp.msrc[2][p];
        u1 = (double)sp.msrc[3][p];
        u2 = (double)sp.msrc[4][p];
        if (sp.w_stride) wp = (double)sp.msrc_w[p];
      } else {
        u0 = sp.src[2][p];
        u1 = sp.src[3][p];
        u2 = sp.src[4][p];
        if (sp.w_stride) wp = sp.src_w[p];
      }
      kin += wp * (sqrt(1.0 + u0 * u0 + u1 * u1 + u2 * u2) - 1.0);
    }
    const double ks = block_sum(kin, sh);
    const double wsp = sp.w_stride ? 1.0 : sp.w;
    if (threadIdx.x == 0) row[1 + s] = ks * wsp * sp.m * area;
  }
}

// Totals: thread v adds column v of the kEnergyBlocks rows in row order.
__global__ void k_energy_total(const double *part, double *total) {
  const int v = threadIdx.x;
  if (v >= kEnergyVals) return;
  double t = 0.0;
  for (int b = 0; b < kEnergyBlocks; ++b) t += part[(size_t)b * kEnergyVals + v];
  total[v] = t;
}

// The fixed buffer: kEnergyBlocks rows of partial sums, then the kEnergyVals totals.  One copy
// per GPU, kept until the process ends; every call on a GPU uses that GPU's copy.
static __device__ __align__(256) double scratch[kEnergyScratchDoubles];

std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxScratchDevices] = {};

}  // namespace

hipError_t energy_scratch(int32_t device, double **ptr) {
  *ptr = nullptr;
  if (device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    // the address of this device's copy, looked up once with the device current (the array's
    // name in host code is not a device address)
    int cur = 0;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = static_cast<double *>(p);
  }
  *ptr = g_scratch_ptr[device];
  return hipSuccess;
}

hipError_t launch_energy_scratch(const StepArgs &a, const double *E, const double *H,
                                 double *scratch_ptr, hipStream_t s) {
  hipLaunchKernelGGL(k_energy_partials, dim3(kEnergyBlocks), dim3(kBlock), 0, s, a, E, H,
                     scratch_ptr);
  hipLaunchKernelGGL(k_energy_total, dim3(1), dim3(64), 0, s, scratch_ptr,
                     scratch_ptr + kEnergyBlocks * kEnergyVals);
  return hipGetLastError();
}

hipError_t launch_particles_alt(const StepArgs &a, bool push, int mover, bool sparse, int32_t max_n,
                                hipStream_t s) {
  const unsigned nb = (unsigned)std::max<int64_t>(
      1, std::max<int64_t>((max_n + kBlock - 1) / kBlock, (a.t.ntiles + kBlock - 1) / kBlock));
  const dim3 grid(nb, (unsigned)a.nsp);
  if (push && sparse)
    hipLaunchKernelGGL((k_particles_alt<true, true>), grid, dim3(kBlock), 0, s, a, mover);
  else if (push)
    hipLaunchKernelGGL((k_particles_alt<true, false>), grid, dim3(kBlock), 0, s, a, mover);
  else if (sparse)
    hipLaunchKernelGGL((k_particles_alt<false, true>), grid, dim3(kBlock), 0, s, a, mover);
  else
    hipLaunchKernelGGL((k_particles_alt<false, false>), grid, dim3(kBlock), 0, s, a, mover);
  return hipGetLastError();
}

hipError_t launch_energy(const StepArgs &a, const double *E, const double *H, double *out,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_energy, dim3(1024), dim3(kBlock), 0, s, a, E, H, out);
  return hipGetLastError();
}

}  // namespace pic
