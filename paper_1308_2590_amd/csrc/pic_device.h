// Device code shared by the particle kernels: wrapping, arithmetic, compact moments, the push, the
// fold of a tile's accumulators and the arrivals.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include "pic_internal.h"

namespace pic {
namespace {

constexpr uint32_t kFlagOrder = PIC_FLAG_ORDER;
constexpr uint32_t kFlagNonFinite = PIC_FLAG_NONFINITE;
constexpr uint32_t kFlagJump = PIC_FLAG_JUMP;
constexpr uint32_t kFlagSlot = PIC_FLAG_SLOT;

__device__ __forceinline__ int wrap1(int i, int n) {
  if (i < 0) return i + n;
  if (i >= n) return i - n;
  return i;
}

__device__ __forceinline__ int wrap_any(int i, int n) {
  i %= n;
  return i < 0 ? i + n : i;
}

// Wrap onto [0, n): one conditional add or subtract when i is known to lie in [-n, 2n) (near:
// a tile and its ring fit in the grid), the general remainder otherwise (grids smaller than a
// tile).  near is the same for the whole block.
__device__ __forceinline__ int wrap_t(int i, int n, bool near) {
  return near ? wrap1(i, n) : wrap_any(i, n);
}

// Quotient e / d of integers (0 <= e < 2^22, d > 0) from one multiply:
// (e + 1/2) / d lies at least 1 / (2 d) away from every integer, and the float product is
// within a relative 2^-23 of it, i.e. within (e + 1/2) / d 2^-23 < 1 / (2 d) absolutely, so
// truncating it gives the exact quotient.  Grid coordinates (below 2^22 by the grid's limits)
// and tile-local indices both qualify.
struct SmallDiv {
  float r;
  __device__ __forceinline__ explicit SmallDiv(int d) : r(1.0f / (float)d) {}
  __device__ __forceinline__ int q(int e) const { return (int)(((float)e + 0.5f) * r); }
};

constexpr int kNoBandTiles = 512;

// The tile handled by this block, taken from the ordered list of tiles that hold particles:
// blocks are dealt round-robin to the 8 XCDs, so each XCD gets a contiguous band of the list
// (neighbouring tiles share halo nodes and field cache lines).  Surplus blocks return.
__device__ __forceinline__ int block_tile(const TileArgs &t, const int32_t *list) {
  const int count = list[t.ntiles];
  const int b = blockIdx.x;
  // few tiles: the entry's load does not wait for the count's
  if (t.ntiles <= kNoBandTiles) {
    const int e = b < t.ntiles ? list[b] : -1;
    return b < count ? e : -1;
  }
  const int per = (count + 7) >> 3;
  if ((b >> 3) >= per) return -1;
  const int idx = (b & 7) * per + (b >> 3);
  return idx < count ? list[idx] : -1;
}

__device__ __forceinline__ double fmaT(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float fmaT(float a, float b, float c) { return fmaf(a, b, c); }

// Reciprocal and reciprocal square root.  FP64: the hardware estimate refined by two
// Newton-Raphson steps (each squares the relative error), which leaves an error of about one
// unit in the last place.  FP32: the hardware results, accurate to about one unit in the last
// place, are used as they are.  Arguments here are >= 1, far from denormals and overflow.
__device__ __forceinline__ double rcpT(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  r = fma(r, fma(-x, r, 1.0), r);
  return r;
}
__device__ __forceinline__ float rcpT(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rsqT(double x) {
  // y' = y + (y / 2)(1 - x y^2)
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return y;
}
__device__ __forceinline__ float rsqT(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float floorT(float a) { return floorf(a); }  // the mixed carry (FP64 uses floor)

// The value of the lane below (lane 0 gets its own): a DPP wave shift by one lane, which
// stays in the VALU instead of the LDS crossbar.
__device__ __forceinline__ int lane_before(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}

// Inclusive sums over the wavefront (all lanes active), by DPP: along rows of 16, then the rows.
__device__ __forceinline__ int wave_sums(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111 /* row_shr:1 */, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142 /* row_bcast:15 */, 0xa, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143 /* row_bcast:31 */, 0xc, 0xf, false);
  return v;
}

// Arrivals v of a cell per lane (all lanes active), added per scan block of cells: the last lane of
// each run of cells in one block adds the run's sum (a tile's rows lie in a few blocks).
__device__ __forceinline__ void add_block_sums(int32_t *bsum, int v, int cell, int lane) {
  const int blk = (int)((uint32_t)cell / (uint32_t)kScanBlock);
  const int before = lane_before(blk), inc = wave_sums(v);
  const uint64_t heads = __ballot(lane == 0 || before != blk);
  const int first = 63 - __clzll((long long)(heads & (~0ull >> (63 - lane))));
  const int sum = inc - __shfl(inc - v, first, 64);
  if ((((heads >> 1) | 1ull << 63) >> lane & 1ull) && sum) atomicAdd(&bsum[blk], sum);
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Compact moments of one particle in the field B of its cell.  With s = beta / gamma and
// b = s B, R = (I + s [B]x + s^2 B B^T) / (1 + s^2 B.B), so
//   S-hat = a0 I + a1 [B]x + a2 B B^T,  a0 = w q^2 dt^2 / (4 m gamma (1 + s^2 B.B)),
//   a1 = a0 s, a2 = a1 s,
//   delta-j = (w q / gamma) R u = (w q / (gamma (1 + s^2 B.B))) (u + s u x B + s^2 (B.u) B).
// Particles sharing a cell share B, so their S-hat deposits add up through three scalars.
template <typename T>
struct Compact {
  T a0, a1, a2, j0, j1, j2;
};

// Species constants in the arithmetic type of the kernel.
template <typename T>
struct SpConst {
  T beta, cS, kJ, w;
};

template <typename T>
__device__ __forceinline__ Compact<T> compact_moments(const SpConst<T> &k, T ginv, T u0, T u1,
                                                      T u2, T B0, T B1, T B2) {
  const T s = k.beta * ginv;
  const T BB = fmaT(B2, B2, fmaT(B1, B1, B0 * B0));
  const T inv = rcpT(fmaT(s * s, BB, T(1)));
  Compact<T> m;
  m.a0 = k.cS * ginv * inv;
  m.a1 = m.a0 * s;
  m.a2 = m.a1 * s;
  const T kk = k.kJ * ginv * inv;
  const T bu = fmaT(B2, u2, fmaT(B1, u1, B0 * u0));
  const T s2bu = s * s * bu;
  m.j0 = kk * fmaT(s2bu, B0, fmaT(s, fmaT(u1, B2, -(u2 * B1)), u0));
  m.j1 = kk * fmaT(s2bu, B1, fmaT(s, fmaT(u2, B0, -(u0 * B2)), u1));
  m.j2 = kk * fmaT(s2bu, B2, fmaT(s, fmaT(u0, B1, -(u1 * B0)), u2));
  return m;
}

// The compact moments of unit density scaled to a particle's density w.
template <typename T>
__device__ __forceinline__ void scale_compact(Compact<T> &m, T w) {
  m.a0 *= w;
  m.a1 *= w;
  m.a2 *= w;
  m.j0 *= w;
  m.j1 *= w;
  m.j2 *= w;
}

// Add one corner's share of compact moments (one particle's, weighted, or a lane's sum):
// delta-j and the density to the node planes at node o, and the three S-hat scalars to the
// planes of that corner of cell rc.  S-hat is expanded with each cell's B only when the tile is
// folded, so a flush does no arithmetic.  The LDS accumulators are FP64 in both precisions
// (FP32 LDS atomic adds are far slower than FP64 ones on gfx950).
struct AccLds {
  double *node;  // [3 + species][plane]: delta-j x, y, z, then one density plane per species
  double *cell;  // [3 scalars][4 corners][npl]: S-hat scalars a0, a1, a2 per cell corner
  int plane, npl, LW, NW;
};

template <typename T>
__device__ __forceinline__ void corner_add(const AccLds &A, int o, int rc, int corner, T A0, T A1,
                                           T A2, T J0, T J1, T J2, T D, int dplane) {
  atomicAdd(&A.node[0 * A.plane + o], (double)J0);
  atomicAdd(&A.node[1 * A.plane + o], (double)J1);
  atomicAdd(&A.node[2 * A.plane + o], (double)J2);
  atomicAdd(&A.node[dplane * A.plane + o], (double)D);
  atomicAdd(&A.cell[(0 * 4 + corner) * A.npl + rc], (double)A0);
  atomicAdd(&A.cell[(1 * 4 + corner) * A.npl + rc], (double)A1);
  atomicAdd(&A.cell[(2 * 4 + corner) * A.npl + rc], (double)A2);
}

// Particle state in either form, as the kernel's arithmetic type: cell (i, k), in-cell offsets
// (fx, fz) and momentum.  FP64 keeps positions in cell units; the mixed form keeps the cell key
// and FP32 offsets.  Src holds the species' source arrays in registers for the whole species.
template <typename T>
__device__ __forceinline__ T at(const T *p, int i) {  // i >= 0; byte offsets fit 32 bits
  return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) + (uint32_t)i * (uint32_t)sizeof(T));
}
template <bool MIXED>
struct Pstate;
template <>
struct Pstate<false> {
  double x, z, u0, u1, u2;
  struct Src {
    const double *a[5];
    __device__ __forceinline__ explicit Src(const SpeciesArgs &sp) {
#pragma unroll
      for (int v = 0; v < 5; ++v) a[v] = sp.src[v];
    }
  };
  __device__ __forceinline__ void load(const Src &s, int p) {
    x = at(s.a[0], p);
    z = at(s.a[1], p);
    u0 = at(s.a[2], p);
    u1 = at(s.a[3], p);
    u2 = at(s.a[4], p);
  }
};
template <>
struct Pstate<true> {
  int cell;
  float x, z, u0, u1, u2;  // x, z: in-cell offsets
  struct Src {
    const int32_t *c;
    const float *a[5];
    __device__ __forceinline__ explicit Src(const SpeciesArgs &sp) {
      c = sp.msrc_cell;
#pragma unroll
      for (int v = 0; v < 5; ++v) a[v] = sp.msrc[v];
    }
  };
  __device__ __forceinline__ void load(const Src &s, int p) {
    cell = at(s.c, p);
    x = at(s.a[0], p);
    z = at(s.a[1], p);
    u0 = at(s.a[2], p);
    u1 = at(s.a[3], p);
    u2 = at(s.a[4], p);
  }
};

// A particle after the push: momentum u^{n+1}, position as stored (FP64: cell units; mixed:
// in-cell offsets), in-cell offsets, new cell (grid coordinates and offset from the old one).
template <typename T>
struct Pushed {
  T n0, n1, n2, rg1;  // u^{n+1}, 1 / gamma(u^{n+1})
  T xn, zn, fx, fz;
  int i2, k2, di, dk;
  bool alive, finite, jump;
};

// Gather, implicit push and position advance of one particle of cell (i, k) with in-cell offsets
// (fx, fz): E-bar at the cell's corner nodes in fE, its B in fB.  edge: the tile touches the
// grid's border, so positions may need the periodic wrap or leave the grid (elsewhere a
// particle, moving less than a cell, stays inside).  ok: the lane holds a particle.
template <bool MIXED, typename T>
__device__ __forceinline__ void push_one(const GridArgs &g, const SpConst<T> &K,
                                         const Pstate<MIXED> &ps, int i, int k, T fx, T fz,
                                         const T fE[12], const T fB[3], bool edge, bool ok,
                                         Pushed<T> &o) {
  const T one = T(1);
  const T u0 = ps.u0, u1 = ps.u1, u2 = ps.u2;
  const T ginv = rsqT(fmaT(u2, u2, fmaT(u1, u1, fmaT(u0, u0, one))));  // 1 / gamma(u^n)
  // gather E-bar at x^{n+1/2} from the 4 corner nodes (linear weights)
  const T W0 = (one - fx) * (one - fz), W1 = fx * (one - fz);
  const T W2 = (one - fx) * fz, W3 = fx * fz;
  T Ep[3];
#pragma unroll
  for (int qq = 0; qq < 3; ++qq)
    Ep[qq] = fmaT(W3, fE[4 * qq + 3],
                  fmaT(W2, fE[4 * qq + 2], fmaT(W1, fE[4 * qq + 1], W0 * fE[4 * qq])));
  // implicit push: with a = u + beta E and b = beta B / gamma,
  // u-bar = R a = (a + a x b + (a.b) b) / (1 + b.b), and u' = 2 u-bar - u
  const T bg = K.beta * ginv;
  const T bx = bg * fB[0], by = bg * fB[1], bz = bg * fB[2];
  const T a0 = fmaT(K.beta, Ep[0], u0), a1 = fmaT(K.beta, Ep[1], u1);
  const T a2 = fmaT(K.beta, Ep[2], u2);
  const T inv = rcpT(fmaT(bz, bz, fmaT(by, by, fmaT(bx, bx, one))));
  const T ab = fmaT(a2, bz, fmaT(a1, by, a0 * bx));
  o.n0 = fmaT(T(2), fmaT(ab, bx, a0 + fmaT(a1, bz, -(a2 * by))) * inv, -u0);
  o.n1 = fmaT(T(2), fmaT(ab, by, a1 + fmaT(a2, bx, -(a0 * bz))) * inv, -u1);
  o.n2 = fmaT(T(2), fmaT(ab, bz, a2 + fmaT(a0, by, -(a1 * bx))) * inv, -u2);
  const T g1sq = fmaT(o.n2, o.n2, fmaT(o.n1, o.n1, fmaT(o.n0, o.n0, one)));
  o.rg1 = rsqT(g1sq);  // 1 / gamma(u^{n+1})
  const T vx = o.n0 * o.rg1, vz = o.n2 * o.rg1;
  // position advance: FP64 in cell units; mixed as FP32 offset with integer carry
  bool alive = ok;
  if constexpr (MIXED) {
    T xn = fx + (T)g.cx * vx;
    T zn = fz + (T)g.cz * vz;
    o.finite = isfinite(g1sq) && isfinite(xn) && isfinite(zn);
    const int cxi = o.finite ? (int)floorT(xn) : 0, czi = o.finite ? (int)floorT(zn) : 0;
    xn -= (T)cxi;
    zn -= (T)czi;
    int ci = i + cxi, ck = k + czi;
    if (xn >= one) { xn = T(0); ci += 1; }
    if (zn >= one) { zn = T(0); ck += 1; }
    if (edge) {
      if (g.bc_x == PIC_BC_PERIODIC) {
        ci = wrap1(ci, g.nx);
      } else if (ci < 0 || ci >= g.nx) {
        alive = false;
      }
      ck = wrap1(ck, g.nz);
    }
    o.xn = xn;
    o.zn = zn;
    o.i2 = ci;
    o.k2 = ck;
    o.fx = xn;
    o.fz = zn;
  } else {
    T xn = ps.x + g.cx * vx;
    T zn = ps.z + g.cz * vz;
    if (edge) {
      if (g.bc_x == PIC_BC_PERIODIC) {
        if (xn < 0.0) xn += (double)g.nx;
        if (xn >= (double)g.nx) xn -= (double)g.nx;
      } else if (xn < 0.0 || xn >= (double)g.nx) {
        alive = false;
      }
      if (zn < 0.0) zn += (double)g.nz;
      if (zn >= (double)g.nz) zn -= (double)g.nz;
    }
    o.finite = isfinite(g1sq) && isfinite(xn) && isfinite(zn);
    const double xf = floor(xn), zf = floor(zn);
    o.i2 = o.finite ? (int)xf : i;
    o.k2 = o.finite ? (int)zf : k;
    o.xn = xn;
    o.zn = zn;
    o.fx = xn - xf;
    o.fz = zn - zf;
  }
  alive = alive && o.finite;
  int di = o.i2 - i, dk = o.k2 - k;
  if (edge) {
    if (di > 1) di -= g.nx;
    if (di < -1) di += g.nx;
    if (dk > 1) dk -= g.nz;
    if (dk < -1) dk += g.nz;
  }
  const bool in3 = (unsigned)(di + 1) <= 2u && (unsigned)(dk + 1) <= 2u;
  o.jump = alive && !in3;
  alive = alive && in3;
  o.di = alive ? di : 0;
  o.dk = alive ? dk : 0;
  o.alive = alive;
}

// Fold a tile's accumulators into the global FP64 moment planes, one node per thread:
// delta-j and the densities as they are; S-hat from the S-hat scalars of the (up to) four
// cells around the node, each expanded with its cell's B (H^{n+3/2} after a push, H^{n+1/2}
// for a deposit of the current state): S-hat = a0 I + a1 [B]x + a2 B B^T.  Lo: the kernel's LDS
// layout; TILE_ONLY: accumulators over the tile's own nodes and cells, without the ring.
template <bool PUSH, bool TILE_ONLY, typename T, typename Layout>
__device__ __forceinline__ void fold_tile(const StepArgs &a, const Layout &Lo, const AccLds &acc, const T *Ho,
                                          const T *Hn, int i0, int k0, bool nearx, bool nearz) {
  const GridArgs &g = a.g;
  const TileArgs &t = a.t;
  const int64_t nn = g.nnodes;
  const int LW = Lo.LW, plane = Lo.plane;
  const SmallDiv div_lw(LW);
  for (int idx = threadIdx.x; idx < LW * Lo.LH; idx += blockDim.x) {
    const int lzz = div_lw.q(idx), lx = idx - lzz * LW;
    constexpr int kOff = TILE_ONLY ? 0 : 1;  // the ring's column and row before the tile
    int gx = i0 - kOff + lx;
    bool in = true;
    if (g.bc_x == PIC_BC_PERIODIC) gx = wrap_t(gx, g.nx, nearx); else in = gx >= 0 && gx <= g.nx;
    const int gz = wrap_t(k0 - kOff + lzz, g.nz, nearz);
    const int64_t node = (int64_t)gz * g.nxn + gx;
    // the field solve reads and clears the moment planes only under a set deposit flag: set
    // the flag of every node this fold adds to
    bool wrote = false;
    for (int pp = 0; pp < Lo.n_node; ++pp) {
      const double v = acc.node[pp * plane + idx];
      const int gp = pp < 3 ? 9 + pp : 12 + (pp - 3);
      if (in && v != 0.0) {
        unsafeAtomicAdd(&a.M[(int64_t)gp * nn + node], v);
        wrote = true;
      }
    }
    double S[9] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    bool any = false;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      // the cell whose corner c is this node, tile-local (-1 and tx, tz: the ring)
      const int cx = lx - kOff - (c & 1), cz = lzz - kOff - (c >> 1);
      if (cx < -kOff || cx >= t.tx + kOff || cz < -kOff || cz >= t.tz + kOff) continue;
      const int rc = (cz + 1) * Lo.NW + (cx + 1);                 // in the ring's numbering
      const int ac = TILE_ONLY ? cz * t.tx + cx : rc;             // in the corner planes
      const double A0 = acc.cell[(0 * 4 + c) * Lo.CPL + ac];
      const double A1 = acc.cell[(1 * 4 + c) * Lo.CPL + ac];
      const double A2 = acc.cell[(2 * 4 + c) * Lo.CPL + ac];
      if (A0 == 0.0 && A1 == 0.0 && A2 == 0.0) continue;
      double B0 = 0.0, B1 = 0.0, B2 = 0.0;
      if (PUSH) {
        B0 = (double)Hn[rc];
        B1 = (double)Hn[Lo.NPL + rc];
        B2 = (double)Hn[2 * Lo.NPL + rc];
      } else if (cx >= 0 && cx < t.tx && cz >= 0 && cz < t.tz) {
        const int hc = cz * t.tx + cx;
        B0 = (double)Ho[hc];
        B1 = (double)Ho[Lo.HPL + hc];
        B2 = (double)Ho[2 * Lo.HPL + hc];
      }
      S[0] += fma(A2, B0 * B0, A0);
      S[1] += fma(A2, B0 * B1, A1 * B2);
      S[2] += fma(A2, B0 * B2, -A1 * B1);
      S[3] += fma(A2, B1 * B0, -A1 * B2);
      S[4] += fma(A2, B1 * B1, A0);
      S[5] += fma(A2, B1 * B2, A1 * B0);
      S[6] += fma(A2, B2 * B0, A1 * B1);
      S[7] += fma(A2, B2 * B1, -A1 * B0);
      S[8] += fma(A2, B2 * B2, A0);
      any = true;
    }
    if (any && in) {
#pragma unroll
      for (int r = 0; r < 9; ++r) {
        if (S[r] != 0.0) {
          unsafeAtomicAdd(&a.M[(int64_t)r * nn + node], S[r]);
          wrote = true;
        }
      }
    }
    if (wrote && a.mflag) a.mflag[node / kFlagNodes] = 1;
  }
}

// The particles the tile's cells send to each cell of the tile and its ring, summed in LDS (arrL
// [species][AH][AW]), added to the per-cell arrival counts: the sort's scan reads those instead of
// gathering nine counts per cell, and (BLOCK_SUMS) to the sums per scan block.
template <bool BLOCK_SUMS>
__device__ __forceinline__ void add_arrivals(const StepArgs &a, const int *arrL, int i0, int k0) {
  const GridArgs &g = a.g;
  const int AW = a.t.tx + 2, AH = a.t.tz + 2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
  // 64 cells per wavefront, the species dealt to the wavefronts too: with every thread doing one
  // species after the other most wavefronts stood idle, 1.5 us of the 8 x 4 tiles' time on a foil.
  const int n_part = (AW * AH + 63) >> 6;
  const SmallDiv div_part(n_part), div_aw(AW);
  for (int u = wave; u < a.nsp * n_part; u += nwaves) {
    const int s = __builtin_amdgcn_readfirstlane(div_part.q(u));
    const SpeciesArgs &sp = a.sp[s];
    if (!sp.active) continue;
    const int *arrS = arrL + s * AW * AH;
    const int e1 = (u - s * n_part) * 64 + lane, e = min(e1, AW * AH - 1);
    const int az = div_aw.q(e), ax = e - az * AW;
    int v = arrS[e];
    if (e1 != e) v = 0;
    int gi = i0 - 1 + ax;
    const int gk = wrap1(k0 - 1 + az, g.nz);
    if (g.bc_x == PIC_BC_PERIODIC) gi = wrap1(gi, g.nx);
    const int cell = gk * g.nx + gi;
    if (v) atomicAdd(&sp.arr[cell], v);
    if constexpr (BLOCK_SUMS) add_block_sums(sp.bsum, v, cell, lane);
  }
}

}  // namespace
}  // namespace pic
