// The mixed-precision particle kernel's form of lane runs, above a few particles per cell: lanes walk
// runs of a tile row and sum their deposits in FP32 registers.  The grouped form (pic_kernels.hip)
// is faster there (21M particles at 128 per cell: 340 against 470 us), but adds the same FP32
// moments in FP64: the sums then differ by 1e-8, the last bits of E-bar by one rounding here and
// there, and after 20 cycles of 21M particles some particle next to a cell's face falls on its other
// side and takes another cell's B: single field values differ by up to 3e-3 of their scale from
// earlier results, although neither is nearer to the 64-bit ones (5e-6 both).  Results of such runs
// are kept.
#pragma once

#include "pic_device.h"

namespace pic {
namespace {

// The value of the lane above (lane 63 gets its own), by DPP wave shifts of 32-bit halves.
__device__ __forceinline__ int lane_after(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x130 /* wave_shl:1 */, 0xf, 0xf, false);
}
__device__ __forceinline__ float lane_after(float v) {
  return __int_as_float(lane_after(__float_as_int(v)));
}
// Per-lane running sum of the compact moments of consecutive particles that stay in one
// cell, per corner (order (i,k), (i+1,k), (i,k+1), (i+1,k+1)).
struct CellAcc {
  float A0[4], A1[4], A2[4], J0[4], J1[4], J2[4], D[4];
  int cell;  // tile-local column of the cell being accumulated, -1 when empty

  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int c = 0; c < 4; ++c) A0[c] = A1[c] = A2[c] = J0[c] = J1[c] = J2[c] = D[c] = 0.0f;
  }
  __device__ __forceinline__ void add(float fx, float fz, const Compact<float> &m, float w) {
    const float one = 1.0f;
    const float W[4] = {(one - fx) * (one - fz), fx * (one - fz), (one - fx) * fz, fx * fz};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      A0[c] = fmaf(W[c], m.a0, A0[c]);
      A1[c] = fmaf(W[c], m.a1, A1[c]);
      A2[c] = fmaf(W[c], m.a2, A2[c]);
      J0[c] = fmaf(W[c], m.j0, J0[c]);
      J1[c] = fmaf(W[c], m.j1, J1[c]);
      J2[c] = fmaf(W[c], m.j2, J2[c]);
      D[c] = fmaf(W[c], w, D[c]);
    }
  }
  // The accumulated cell is (cell, lz - 1) of the tile: ring cell (cell + 1, lz), whose
  // lower-left node is (cell + 1, lz) locally (the layout with the ring).
  __device__ __forceinline__ void flush(const AccLds &acc, int lz, int dplane) {
    const int b = lz * acc.LW + cell + 1, rc = lz * acc.NW + cell + 1;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      corner_add(acc, b + (c & 1) + (c >> 1) * acc.LW, rc, c, A0[c], A1[c], A2[c], J0[c], J1[c],
                 J2[c], D[c], dplane);
  }
  // End of a row: every lane flushes at once, and the lanes whose runs end in one cell are
  // neighbours.  Their sums are first added up across lanes (a segmented reduction with
  // shuffles towards the first lane of each cell), so that one lane per cell issues the LDS
  // atomics; same-address atomics from many lanes of one instruction are serialised.  All 64
  // lanes must be active.
  __device__ __forceinline__ void flush_row_end(const AccLds &acc, int lz, int dplane, int lane) {
    const int prev = lane_before(cell);
    const bool head = lane == 0 || prev != cell;
    const uint64_t heads = __ballot(head);
    const uint64_t above = heads & ~((2ull << lane) - 1ull);
    const int seg_end = above ? __ffsll((unsigned long long)above) - 1 : 64;
    {
      // first step (neighbour one lane up) by DPP; the wider steps go through the LDS crossbar
      const bool take = lane + 1 < seg_end;
      if (!__any(take)) {
        if (head && cell >= 0) flush(acc, lz, dplane);
        return;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float v;
        v = lane_after(A0[c]); A0[c] += take ? v : 0.0f;
        v = lane_after(A1[c]); A1[c] += take ? v : 0.0f;
        v = lane_after(A2[c]); A2[c] += take ? v : 0.0f;
        v = lane_after(J0[c]); J0[c] += take ? v : 0.0f;
        v = lane_after(J1[c]); J1[c] += take ? v : 0.0f;
        v = lane_after(J2[c]); J2[c] += take ? v : 0.0f;
        v = lane_after(D[c]); D[c] += take ? v : 0.0f;
      }
    }
    for (int d = 2; d < 64; d <<= 1) {
      const bool take = lane + d < seg_end;
      if (!__any(take)) break;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float v;
        v = __shfl_down(A0[c], d); A0[c] += take ? v : 0.0f;
        v = __shfl_down(A1[c], d); A1[c] += take ? v : 0.0f;
        v = __shfl_down(A2[c], d); A2[c] += take ? v : 0.0f;
        v = __shfl_down(J0[c], d); J0[c] += take ? v : 0.0f;
        v = __shfl_down(J1[c], d); J1[c] += take ? v : 0.0f;
        v = __shfl_down(J2[c], d); J2[c] += take ? v : 0.0f;
        v = __shfl_down(D[c], d); D[c] += take ? v : 0.0f;
      }
    }
    if (head && cell >= 0) flush(acc, lz, dplane);
  }
};

// Particles that change cell deposit into a different cell (and field) from the lane's run,
// so they are queued per wavefront in LDS and deposited 64 at a time, one per lane.
constexpr int kMqCap = 64;
// fx fz a0 a1 a2 j0 j1 j2, and the particle's density when densities are per particle
__host__ __device__ constexpr int mq_words(bool pw) { return pw ? 9 : 8; }

struct MoverQ {
  float *v;      // [mq_words][kMqCap]
  int *idx;  // [2][kMqCap]: lower-left accumulator node, ring cell of the destination
};

template <bool PW>
__device__ __forceinline__ void drain_movers(const MoverQ &q, int count, int lane,
                                             const AccLds &acc, int dplane, float w_uniform) {
  if (lane < count) {
    const float fx = q.v[0 * kMqCap + lane], fz = q.v[1 * kMqCap + lane];
    const float a0 = q.v[2 * kMqCap + lane], a1 = q.v[3 * kMqCap + lane];
    const float a2 = q.v[4 * kMqCap + lane], j0 = q.v[5 * kMqCap + lane];
    const float j1 = q.v[6 * kMqCap + lane], j2 = q.v[7 * kMqCap + lane];
    const float w = PW ? q.v[8 * kMqCap + lane] : w_uniform;
    const int o = q.idx[lane], rc = q.idx[kMqCap + lane];
#pragma unroll 1
    for (int c = 0; c < 4; ++c) {
      const int cx = c & 1, cz = c >> 1;
      const float W = (cx ? fx : 1.0f - fx) * (cz ? fz : 1.0f - fz);
      corner_add(acc, o + cx + cz * acc.LW, rc, c, W * a0, W * a1, W * a2, W * j0, W * j1, W * j2,
                 W * w, dplane);
    }
  }
}

// LDS layout of the lane-run form (byte offsets): the FP64 moment accumulators over the tile and its
// ring (delta-j and density per node, S-hat scalars per cell corner), the FP32 fields the tile's
// particles read (E-bar on the tile's nodes, H^{n+1/2} on its cells, H^{n+3/2} on its cells plus the
// one-cell ring a particle can move into), the per-wave mover queues, per species the move
// counters of the tile's cells and the arrival counts of the tile's cells and their ring, and the
// first and end slot of every tile row of every species slot.
struct RunsLds {
  int LW, LH, plane;          // accumulator node grid (tx + 3) x (tz + 3)
  int EW, EPL;                // E-bar node grid (tx + 1) x (tz + 1)
  int HPL;                    // H^{n+1/2} cells tx x tz
  int NW, NPL, CPL;           // H^{n+3/2} and S-hat corner cells (tx + 2) x (tz + 2)
  int n_node;                 // node accumulator planes: 3 + species
  size_t acc, accc, eb, ho, hn, mq, cnt, arr, rows;  // byte offsets
  size_t bytes;
  __host__ __device__ RunsLds(int n_planes, int tx, int tz, bool pw) {
    LW = tx + 3;
    LH = tz + 3;
    plane = LW * LH;
    EW = tx + 1;
    EPL = EW * (tz + 1);
    HPL = tx * tz;
    NW = tx + 2;
    NPL = CPL = NW * (tz + 2);
    n_node = 3 + (n_planes - 12);
    acc = 0;
    accc = acc + (size_t)n_node * plane * sizeof(double);
    eb = accc + (size_t)12 * CPL * sizeof(double);
    ho = eb + 3 * (size_t)EPL * sizeof(float);
    hn = ho + 3 * (size_t)HPL * sizeof(float);
    mq = (hn + 3 * (size_t)NPL * sizeof(float) + 7) & ~(size_t)7;
    cnt = mq + (size_t)(kBlock / 64) * kMqCap * (mq_words(pw) * sizeof(float) + 2 * sizeof(int));
    arr = cnt + (size_t)(n_node - 3) * tx * tz * kMoveCodes * sizeof(int);
    rows = arr + (size_t)(n_node - 3) * (tx + 2) * (tz + 2) * sizeof(int);
    bytes = rows + (size_t)(n_node - 3) * tz * 2 * sizeof(int);
  }
};

// One block of four wavefronts per tile of cells, one wavefront per tile row (or per part of a row
// when the tile has fewer rows than wavefronts).  The row's particles (a contiguous range of the
// cell-sorted order) are split into 64 contiguous runs, one per lane; run lengths differ by at most
// one.  A lane accumulates the deposits of particles that stay in their cell in registers and adds
// them to the LDS tile when its run enters the next cell, so LDS atomics are issued once per (lane,
// cell) instead of once per particle; particles changing cell go through a per-wave queue.  The
// pushed state of the particle at iteration `it` of lane `l` is written to location
// row_start + 64 it + l, which makes the stores (and next cycle's loads through the permutation)
// coalesced.  The register sums take about 150 VGPRs: three wavefronts per SIMD.  IDS adds the copy
// of particle ids (tests only).  PW selects per-particle densities: each particle's moments are
// those of unit density times its own density, which is read with the state and written with the
// pushed state (a species with one density reads it from a one-element array with stride 0).
template <bool PUSH, bool IDS, bool PW>
__device__ __forceinline__ void runs_body(const StepArgs &a, int tile) {
  const GridArgs &g = a.g;
  const TileArgs &t = a.t;
  const int tzi = tile / t.ntx, txi = tile - tzi * t.ntx;
  const int i0 = txi * t.tx, k0 = tzi * t.tz;
  const int i1 = min(i0 + t.tx, g.nx), k1 = min(k0 + t.tz, g.nz);
  const int ntc = t.tx * t.tz;
  const int64_t nn = g.nnodes, nc = g.ncells;

  extern __shared__ double lds[];
  char *ldsb = reinterpret_cast<char *>(lds);
  constexpr int kQw = mq_words(PW);
  const RunsLds Lo(g.n_planes, t.tx, t.tz, PW);
  const AccLds acc{reinterpret_cast<double *>(ldsb + Lo.acc),
                   reinterpret_cast<double *>(ldsb + Lo.accc), Lo.plane, Lo.CPL, Lo.LW, Lo.NW};
  float *Eb = reinterpret_cast<float *>(ldsb + Lo.eb);
  float *Ho = reinterpret_cast<float *>(ldsb + Lo.ho);
  float *Hn = reinterpret_cast<float *>(ldsb + Lo.hn);
  int *cntL = reinterpret_cast<int *>(ldsb + Lo.cnt);  // [species][cells of the tile][9 codes]
  int *arrL = reinterpret_cast<int *>(ldsb + Lo.arr);
  const int LW = Lo.LW;
  const int n_acc = Lo.n_node * Lo.plane + 12 * Lo.CPL;  // node planes, then cell-corner planes

  for (int e = threadIdx.x; e < n_acc; e += blockDim.x) acc.node[e] = 0.0;
  const int AW = t.tx + 2, AH = t.tz + 2;  // arrival counts: the tile's cells and their ring
  if (PUSH) {
    const int nsl = Lo.n_node - 3;
    for (int e = threadIdx.x; e < nsl * ntc * kMoveCodes; e += blockDim.x) cntL[e] = 0;
    for (int e = threadIdx.x; e < nsl * AW * AH; e += blockDim.x) arrL[e] = 0;
  }
  const int cw = i1 - i0, chh = k1 - k0;  // the tile's cells inside the grid
  // a tile and its two-cell ring fit in the grid along an axis: wraps need one compare there
  const bool nearx = g.nx >= t.tx + 3, nearz = g.nz >= t.tz + 3;
  // Stage the fields of the tile and the slot range of every tile row of every species in one
  // pass: a thread issues all its loads (at clamped, valid addresses) before it stores any, so
  // the block waits for one memory round trip instead of one per array.
  const int nrows_t = k1 - k0;
  int *rowsL = reinterpret_cast<int *>(ldsb + Lo.rows);  // [species][row]: first, end slot
  const int n_stage = max(max(Lo.HPL, nrows_t), PUSH ? max(Lo.EPL, Lo.NPL) : 0);
  for (int e = threadIdx.x; e < n_stage; e += blockDim.x) {
    // H^{n+1/2} on the tile's cells
    const int eh = min(e, Lo.HPL - 1);
    const int hk = SmallDiv(t.tx).q(eh), hi = eh - hk * t.tx;
    const bool h_in = e < Lo.HPL && i0 + hi < g.nx && k0 + hk < g.nz;
    const int64_t ch = (int64_t)min(k0 + hk, g.nz - 1) * g.nx + min(i0 + hi, g.nx - 1);
    double ho[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) ho[q] = a.Hold[q * nc + ch];
    // first and end slot of tile row e of every species (threads e < rows of the tile)
    const bool r_th = e < nrows_t;
    const int64_t rowc = (int64_t)(k0 + min(e, nrows_t - 1)) * g.nx;
    int rbv[kMaxSpecies], rev[kMaxSpecies];
#pragma unroll
    for (int q = 0; q < kMaxSpecies; ++q) {
      rbv[q] = 0;
      rev[q] = 0;
      if (q < a.nsp && a.sp[q].active && r_th) {
        rbv[q] = a.sp[q].cs[rowc + i0];
        rev[q] = a.sp[q].cs[rowc + i1];
      }
    }
    double eo[3], en[3], hn[3];
    bool e_in = false, n_in = false;
    if (PUSH) {
      // E-bar on the tile's nodes
      const int ee = min(e, Lo.EPL - 1);
      const int ek = SmallDiv(Lo.EW).q(ee), ei = ee - ek * Lo.EW;
      int gi = i0 + ei;
      const int gk = wrap_t(k0 + ek, g.nz, nearz);
      e_in = e < Lo.EPL;
      if (g.bc_x == PIC_BC_PERIODIC) gi = wrap_t(gi, g.nx, nearx); else e_in = e_in && gi <= g.nx;
      const int64_t n = (int64_t)gk * g.nxn + min(gi, g.nxn - 1);
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        eo[q] = a.Eold[q * nn + n];
        en[q] = a.Enew[q * nn + n];
      }
      // H^{n+3/2} on the tile's cells and their ring
      const int en_ = min(e, Lo.NPL - 1);
      const int nk = SmallDiv(Lo.NW).q(en_), ni = en_ - nk * Lo.NW;
      int gi2 = i0 - 1 + ni;
      const int gk2 = wrap_t(k0 - 1 + nk, g.nz, nearz);
      n_in = e < Lo.NPL;
      if (g.bc_x == PIC_BC_PERIODIC) gi2 = wrap_t(gi2, g.nx, nearx); else n_in = n_in && gi2 >= 0 && gi2 < g.nx;
      const int64_t c2 = (int64_t)gk2 * g.nx + min(max(gi2, 0), g.nx - 1);
#pragma unroll
      for (int q = 0; q < 3; ++q) hn[q] = a.Hnew[q * nc + c2];
    }
    if (e < Lo.HPL) {
#pragma unroll
      for (int q = 0; q < 3; ++q) Ho[q * Lo.HPL + e] = h_in ? (float)ho[q] : 0.0f;
    }
    if (r_th) {
#pragma unroll
      for (int q = 0; q < kMaxSpecies; ++q) {
        if (q < a.nsp) {
          rowsL[2 * (q * nrows_t + e)] = rbv[q];
          rowsL[2 * (q * nrows_t + e) + 1] = rev[q];
        }
      }
    }
    if (PUSH && e < Lo.EPL) {
#pragma unroll
      for (int q = 0; q < 3; ++q) Eb[q * Lo.EPL + e] = e_in ? (float)(0.5 * (eo[q] + en[q])) : 0.0f;
    }
    if (PUSH && e < Lo.NPL) {
#pragma unroll
      for (int q = 0; q < 3; ++q) Hn[q * Lo.NPL + e] = n_in ? (float)hn[q] : 0.0f;
    }
  }
  __syncthreads();

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  // the tile touches the grid's border: its particles may wrap or leave
  const bool edge = i0 == 0 || i1 == g.nx || k0 == 0 || k1 == g.nz;
  MoverQ mq;
  {
    char *qb = ldsb + Lo.mq + (size_t)wave * kMqCap * ((size_t)kQw * sizeof(float) + 2 * sizeof(int));
    mq.v = reinterpret_cast<float *>(qb);
    mq.idx = reinterpret_cast<int *>(qb + (size_t)kMqCap * kQw * sizeof(float));
  }

  for (int s = 0; s < a.nsp; ++s) {
    const SpeciesArgs &sp = a.sp[s];
    if (!sp.active) continue;
    int *const cntS = cntL + s * ntc * kMoveCodes;  // the species' move counters
    // (a species with one density keeps its own constants, also in a kernel with densities per
    // particle: its moments are then the same bits in both)
    const bool own_w = PW && sp.w_stride != 0;
    const SpConst<float> K{(float)sp.beta, (float)(own_w ? sp.cS1 : sp.cS), (float)(own_w ? sp.kJ1 : sp.kJ), (float)sp.w};
    const Pstate<true>::Src src(sp);
    // per-particle densities: index p * wstride (stride 0 reads a species' single density)
    const float *wsrc = sp.msrc_w;
    float *wdst = sp.mdst_w;
    const int wstride = sp.w_stride;
    const int32_t *perm = sp.perm;
    const int dplane = 3 + s;  // density plane of the species in the node accumulators
    // A tile with fewer rows than wavefronts splits each row's particles into wpr contiguous
    // parts, one per wavefront, so short tiles keep every wavefront busy.
    const int nrows = k1 - k0;
    const int wpr = nrows < nwaves ? nwaves / nrows : 1;  // 1, 2 or 4 (four wavefronts)
    const int wsh = wpr == 4 ? 2 : (wpr == 2 ? 1 : 0);
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
      const int lk = r - k0, lz = lk + 1;
      CellAcc ca;
      ca.clear();
      ca.cell = -1;
      int nq = 0;  // movers queued by this wavefront (uniform)
      // fields of the cell the lane's run is in, kept in registers while the run stays in it:
      // H^{n+1/2} (fB) and E-bar at its 4 nodes (fE, the push)
      float fB[3] = {0.0f, 0.0f, 0.0f}, fE[12];
      // The run is processed in chunks of kChunk particles: the chunk's state loads are issued
      // together (with the next chunk's permutation entries), then its particles are pushed
      // from registers in an unrolled sequence.  Global stores share the vector-memory counter
      // with loads, so a load whose value is still in flight across a loop iteration makes
      // the compiler wait for all earlier stores too; keeping every loaded value inside one
      // iteration lets it wait for the loads alone.  Loads are issued unconditionally (slots
      // past a lane's run read a location inside the state arrays, and their values go
      // unused): a load under a divergent branch also forces a full wait.
      constexpr int kChunk = 4;
      Pstate<true> cb[kChunk];
      int cp_[kChunk], np_[kChunk];
      float cw_[kChunk];
      // A chunk's permutation entries come in one 16-byte load per lane (the array is padded
      // so the load stays inside it); entries past the lane's run are clamped to a location
      // inside the state arrays and their particles go unused.
      static_assert(kPermPad >= 2 * kChunk, "one int4 of entries per chunk");
      const uint32_t loc_max = (uint32_t)(sp.cap - 1);
      auto perm4 = [&](int first, int out[kChunk]) {
        int4 v;
        __builtin_memcpy(&v, perm + first, sizeof(v));
        out[0] = (int)min((uint32_t)v.x, loc_max);
        out[1] = (int)min((uint32_t)v.y, loc_max);
        out[2] = (int)min((uint32_t)v.z, loc_max);
        out[3] = (int)min((uint32_t)v.w, loc_max);
      };
      perm4(start, np_);
      // all lanes run the same number of iterations so the mover queue stays wave-uniform
      for (int c0 = 0; c0 < iters; c0 += kChunk) {
#pragma unroll
        for (int kk = 0; kk < kChunk; ++kk) {
          cp_[kk] = np_[kk];
          cb[kk].load(src, cp_[kk]);
          if constexpr (PW) cw_[kk] = wsrc[cp_[kk] * wstride];
        }
        perm4(start + c0 + kChunk, np_);
#pragma unroll
        for (int kk = 0; kk < kChunk; ++kk) {
          const int it = c0 + kk;
          if (it >= iters) break;
          const bool act = it < my_n;
          const int j = start + it;
          const int p = cp_[kk];
          const Pstate<true> &ps = cb[kk];
          const int k = r, i = ps.cell - r * g.nx;
          const float fx = ps.x, fz = ps.z;
          const float wp = PW ? cw_[kk] : K.w;  // the particle's density
          const bool ok = act && i >= i0 && i < i1;
          const int loc = jb + it * 64 + lane;
          if (act && !ok) {
            atomicOr(a.flags, kFlagOrder);
            if (PUSH) sp.locode[j] = ((uint32_t)loc << 4) | kAbsorbed;
          }
          // Lanes without a valid particle run the arithmetic on a valid cell of the tile and
          // discard the results, so the main path has no branches around it.
          const int li = ok ? i - i0 : max(ca.cell, 0);
          const int hc = lk * t.tx + li;
          // On entering a new cell: read its fields, use them, and only then flush the previous
          // cell's accumulator.  LDS operations complete in order, so a read issued after the
          // flush's atomics (or consumed while they are in flight) would wait for all of them.
          const bool newcell = ok && li != ca.cell;
          if (newcell) {
#pragma unroll
            for (int qq = 0; qq < 3; ++qq) fB[qq] = Ho[qq * Lo.HPL + hc];
            if (PUSH) {
              const int e00 = lk * Lo.EW + li;
#pragma unroll
              for (int qq = 0; qq < 3; ++qq) {
                const float *f = Eb + qq * Lo.EPL + e00;
                fE[4 * qq] = f[0];
                fE[4 * qq + 1] = f[1];
                fE[4 * qq + 2] = f[Lo.EW];
                fE[4 * qq + 3] = f[Lo.EW + 1];
              }
            }
          }
          if constexpr (!PUSH) {
            const float ginv = rsqT(fmaf(ps.u2, ps.u2, fmaf(ps.u1, ps.u1, fmaf(ps.u0, ps.u0, 1.0f))));
            Compact<float> m0 = compact_moments(K, ginv, ps.u0, ps.u1, ps.u2, fB[0], fB[1], fB[2]);
            if constexpr (PW) scale_compact(m0, own_w ? wp : float(1));
            if (newcell) {
              if (ca.cell >= 0) ca.flush(acc, lz, dplane);
              ca.clear();
              ca.cell = li;
            }
            if (ok) ca.add(fx, fz, m0, wp);
          } else {
            Pushed<float> o;
            push_one<true>(g, K, ps, i, k, fx, fz, fE, fB, edge, ok, o);
            if (ok && !o.finite) atomicOr(a.flags, kFlagNonFinite);
            if (o.jump) atomicOr(a.flags, kFlagJump);
            const uint32_t code = o.alive ? (uint32_t)((o.dk + 1) * 3 + (o.di + 1)) : kAbsorbed;
            // moments M^{n+3/2} at x^{n+3/2} with u^{n+1}, 1/gamma(u^{n+1}) and H^{n+3/2}
            // of the new cell (read before any LDS atomic of this particle is issued)
            const int hn = (lk + o.dk + 1) * Lo.NW + (li + o.di + 1);
            Compact<float> m = compact_moments(K, o.rg1, o.n0, o.n1, o.n2, Hn[hn], Hn[Lo.NPL + hn], Hn[2 * Lo.NPL + hn]);
            if constexpr (PW) scale_compact(m, own_w ? wp : float(1));
            if (newcell) {
              if (ca.cell >= 0) ca.flush(acc, lz, dplane);
              ca.clear();
              ca.cell = li;
            }
            if (ok) {
              sp.mdst_cell[loc] = o.k2 * g.nx + o.i2;
              sp.mdst[0][loc] = o.xn;
              sp.mdst[1][loc] = o.zn;
              sp.mdst[2][loc] = o.n0;
              sp.mdst[3][loc] = o.n1;
              sp.mdst[4][loc] = o.n2;
              if (PW && wstride) wdst[loc] = wp;
              sp.locode[j] = ((uint32_t)loc << 4) | code;
              // particle ids (tests only): a separate instantiation, so that its load, which
              // is waited for at once, does not enter the wait counts of the kernel without ids
              if (IDS && sp.dst_id) sp.dst_id[loc] = sp.src_id[p];
              if (code != kAbsorbed) atomicAdd(&cntS[hc * kMoveCodes + code], 1);
            }
            // stayers add to the lane's accumulator, movers go through the queue
            if (o.alive && code == 4u) ca.add(o.fx, o.fz, m, wp);
            const bool mover = o.alive && code != 4u;
            // queue this iteration's movers; drain first if they would not fit
            const uint64_t mmask = __ballot(mover);
            const int nm = __popcll(mmask);
            if (nq + nm > kMqCap) {
              wave_sync();
              drain_movers<PW>(mq, nq, lane, acc, dplane, K.w);
              wave_sync();
              nq = 0;
            }
            if (mover) {
              const int e = nq + __popcll(mmask & lt_mask);
              mq.v[0 * kMqCap + e] = o.fx;
              mq.v[1 * kMqCap + e] = o.fz;
              mq.v[2 * kMqCap + e] = m.a0;
              mq.v[3 * kMqCap + e] = m.a1;
              mq.v[4 * kMqCap + e] = m.a2;
              mq.v[5 * kMqCap + e] = m.j0;
              mq.v[6 * kMqCap + e] = m.j1;
              mq.v[7 * kMqCap + e] = m.j2;
              if constexpr (PW) mq.v[8 * kMqCap + e] = wp;
              mq.idx[e] = (lz + o.dk) * LW + (li + 1 + o.di);
              mq.idx[kMqCap + e] = hn;
            }
            nq += nm;
          }
        }
      }
      ca.flush_row_end(acc, lz, dplane, lane);
      if (PUSH && nq > 0) {
        wave_sync();
        drain_movers<PW>(mq, nq, lane, acc, dplane, K.w);
        wave_sync();
      }
    }
  }
  __syncthreads();
  // Move counts of the tile's cells, for the ranking, and the arrivals.  The counts of every species
  // are kept until here, so the species need no barriers between them.
  if constexpr (PUSH) {
    const SmallDiv div_cw(cw);
    for (int s = 0; s < a.nsp; ++s) {
      const SpeciesArgs &sp = a.sp[s];
      if (!sp.active) continue;
      const int *cntS = cntL + s * ntc * kMoveCodes;
      int *arrS = arrL + s * AW * AH;
      for (int e = threadIdx.x; e < chh * cw; e += blockDim.x) {
        const int lkk = div_cw.q(e), li = e - lkk * cw;
        const int64_t cg = (int64_t)(k0 + lkk) * g.nx + (i0 + li);
        const int *cl = cntS + (lkk * t.tx + li) * kMoveCodes;
        uint32_t mask = 0;
#pragma unroll
        for (int d = 0; d < kMoveCodes; ++d) {
          const int v = cl[d];
          // with code masks only the nonzero counts are written (most cells send all their
          // particles with one code)
          if (!a.count_masks || v) sp.cnt[(int64_t)d * nc + cg] = v;
          if (v) {
            mask |= 1u << d;
            atomicAdd(&arrS[(lkk + d / 3) * AW + (li + d % 3)], v);
          }
        }
        if (a.count_masks) sp.cmask[cg] = (uint16_t)mask;
      }
    }
  }
  fold_tile<PUSH, false>(a, Lo, acc, Ho, Hn, i0, k0, nearx, nearz);
  if constexpr (PUSH) {
    __syncthreads();
    add_arrivals<false>(a, arrL, i0, k0);  // (block sums: see StepArgs::block_sums)
  }
}

}  // namespace
}  // namespace pic
