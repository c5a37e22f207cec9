// The mixed-precision particle kernel of single runs above a few particles per cell: lanes walk
// runs of a tile row and sum their deposits in FP32 registers.  The grouped kernel (pic_kernels.hip)
// is faster there (21M particles at 128 per cell: 340 against 470 us), but adds the same FP32
// moments in FP64: the sums then differ by 1e-8, the last bits of E-bar by one rounding here and
// there, and after 20 cycles of 21M particles some particle next to a cell's face falls on its other
// side and takes another cell's B: single field values differ by 2e-3 of their scale from earlier
// results, although neither is nearer to the 64-bit ones (5e-6 both).  Results of such runs are kept.
#include <type_traits>

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

// Quotient e / d of non-negative integers (e < 2^22, 0 < d < 2^12) from one multiply:
// (e + 1/2) / d lies at least 1 / (2 d) away from every integer, and the float product is
// within a relative 2^-23 of it, i.e. within (e + 1/2) / d 2^-23 < 1 / (2 d) absolutely, so
// truncating it gives the exact quotient.  Grid coordinates (below 2^22 by the grid's limits)
// and tile-local indices both qualify.
struct SmallDiv {
  float r;
  __device__ __forceinline__ explicit SmallDiv(int d) : r(1.0f / (float)d) {}
  __device__ __forceinline__ int q(int e) const { return (int)(((float)e + 0.5f) * r); }
};

// The tile handled by this block, taken from the ordered list of tiles that hold particles:
// blocks are dealt round-robin to the 8 XCDs, so each XCD gets a contiguous band of the list
// (neighbouring tiles share halo nodes and field cache lines).  Surplus blocks return.
__device__ __forceinline__ int block_tile(const TileArgs &t, const int32_t *list) {
  const int count = list[t.ntiles];
  const int per = (count + 7) >> 3;
  const int b = blockIdx.x;
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

// ------------------------------------------------------------------------------------------
// Particles
// ------------------------------------------------------------------------------------------

// The value of the lane below (lane 0 gets its own): a DPP wave shift by one lane, which
// stays in the VALU instead of the LDS crossbar.
__device__ __forceinline__ int lane_before(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}

// The value of the lane above (lane 63 gets its own), by DPP wave shifts of 32-bit halves.
__device__ __forceinline__ int lane_after(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x130 /* wave_shl:1 */, 0xf, 0xf, false);
}
__device__ __forceinline__ float lane_after(float v) {
  return __int_as_float(lane_after(__float_as_int(v)));
}
__device__ __forceinline__ double lane_after(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = lane_after((int)(b & 0xffffffffll)), hi = lane_after((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

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
__device__ __forceinline__ void store_or_drop(uint32_t *p, int i, bool on, uint32_t v) {
  __builtin_amdgcn_raw_buffer_store_b32(v, store_rsrc(p), on ? i * 4 : kStoreDrop, 0, 0);
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

// Per-lane running sum of the compact moments of consecutive particles that stay in one
// cell, per corner (order (i,k), (i+1,k), (i,k+1), (i+1,k+1)).
template <typename T>
struct CellAcc {
  T A0[4], A1[4], A2[4], J0[4], J1[4], J2[4], D[4];
  int cell;  // tile-local column of the cell being accumulated, -1 when empty

  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int c = 0; c < 4; ++c) A0[c] = A1[c] = A2[c] = J0[c] = J1[c] = J2[c] = D[c] = T(0);
  }
  __device__ __forceinline__ void add(T fx, T fz, const Compact<T> &m, T w) {
    const T one = T(1);
    const T W[4] = {(one - fx) * (one - fz), fx * (one - fz), (one - fx) * fz, fx * fz};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      A0[c] = fmaT(W[c], m.a0, A0[c]);
      A1[c] = fmaT(W[c], m.a1, A1[c]);
      A2[c] = fmaT(W[c], m.a2, A2[c]);
      J0[c] = fmaT(W[c], m.j0, J0[c]);
      J1[c] = fmaT(W[c], m.j1, J1[c]);
      J2[c] = fmaT(W[c], m.j2, J2[c]);
      D[c] = fmaT(W[c], w, D[c]);
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
        T v;
        v = lane_after(A0[c]); A0[c] += take ? v : T(0);
        v = lane_after(A1[c]); A1[c] += take ? v : T(0);
        v = lane_after(A2[c]); A2[c] += take ? v : T(0);
        v = lane_after(J0[c]); J0[c] += take ? v : T(0);
        v = lane_after(J1[c]); J1[c] += take ? v : T(0);
        v = lane_after(J2[c]); J2[c] += take ? v : T(0);
        v = lane_after(D[c]); D[c] += take ? v : T(0);
      }
    }
    for (int d = 2; d < 64; d <<= 1) {
      const bool take = lane + d < seg_end;
      if (!__any(take)) break;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        T v;
        v = __shfl_down(A0[c], d); A0[c] += take ? v : T(0);
        v = __shfl_down(A1[c], d); A1[c] += take ? v : T(0);
        v = __shfl_down(A2[c], d); A2[c] += take ? v : T(0);
        v = __shfl_down(J0[c], d); J0[c] += take ? v : T(0);
        v = __shfl_down(J1[c], d); J1[c] += take ? v : T(0);
        v = __shfl_down(J2[c], d); J2[c] += take ? v : T(0);
        v = __shfl_down(D[c], d); D[c] += take ? v : T(0);
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

template <typename T>
struct MoverQ {
  T *v;      // [mq_words][kMqCap]
  int *idx;  // [2][kMqCap]: lower-left accumulator node, ring cell of the destination
};

template <typename T, bool PW>
__device__ __forceinline__ void drain_movers(const MoverQ<T> &q, int count, int lane,
                                             const AccLds &acc, int dplane, T w_uniform) {
  if (lane < count) {
    const T fx = q.v[0 * kMqCap + lane], fz = q.v[1 * kMqCap + lane];
    const T a0 = q.v[2 * kMqCap + lane], a1 = q.v[3 * kMqCap + lane];
    const T a2 = q.v[4 * kMqCap + lane], j0 = q.v[5 * kMqCap + lane];
    const T j1 = q.v[6 * kMqCap + lane], j2 = q.v[7 * kMqCap + lane];
    const T w = PW ? q.v[8 * kMqCap + lane] : w_uniform;
    const int o = q.idx[lane], rc = q.idx[kMqCap + lane];
#pragma unroll 1
    for (int c = 0; c < 4; ++c) {
      const int cx = c & 1, cz = c >> 1;
      const T W = (cx ? fx : T(1) - fx) * (cz ? fz : T(1) - fz);
      corner_add(acc, o + cx + cz * acc.LW, rc, c, W * a0, W * a1, W * a2, W * j0, W * j1, W * j2,
                 W * w, dplane);
    }
  }
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

// Chunk-of-2 form: a particle whose new cell (gi, gk) lies outside the tile adds its moments to
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

// LDS layout of the particle kernel (byte offsets): the moment accumulators (delta-j and
// density per node, S-hat scalars per cell corner), the fields the tile's particles read (E-bar
// on the tile's nodes, H^{n+1/2} on its cells, H^{n+3/2} on its cells plus the one-cell ring a
// particle can move into), the per-wave mover queues, per species the int move counters of the
// tile's cells and the arrival counts of the tile's cells and their ring, and the first and
// end slot of every tile row of every species slot.  Two layouts: with mover queues
// (qwords > 0) the accumulators cover the tile and its ring; without (the chunk-of-2 form) they
// cover the tile's own nodes and cells, particles leaving the tile deposit to the global
// planes, and the arrivals are summed from the move counters (no arrival array), which brings
// a 32 x 4 tile of two species to 40 KB: four blocks per CU.  Accumulators are FP64; fields
// and queues use the kernel's arithmetic type.
struct TileLds {
  int LW, LH, plane;          // accumulator node grid (tx + 3) x (tz + 3), or (tx + 1) x (tz + 1)
  int EW, EPL;                // E-bar node grid (tx + 1) x (tz + 1)
  int HPL;                    // H^{n+1/2} cells tx x tz
  int NW, NPL;                // H^{n+3/2} cells (tx + 2) x (tz + 2)
  int CPL;                    // pitch of the S-hat corner planes: NPL, or HPL padded
  int n_node;                 // node accumulator planes: 3 + species
  size_t acc, accc, eb, ho, hn, mq, cnt, arr, rows;  // byte offsets
  size_t bytes;
  __host__ __device__ TileLds(int n_planes, int tx, int tz, int tsize, int qwords) {
    const int ring = qwords ? 1 : 0;
    LW = tx + 1 + 2 * ring;
    LH = tz + 1 + 2 * ring;
    plane = LW * LH;
    EW = tx + 1;
    EPL = EW * (tz + 1);
    HPL = tx * tz;
    NW = tx + 2;
    NPL = NW * (tz + 2);
    // without the ring the corner-plane pitch is padded to 4 (mod 8) doubles: the two lanes of
    // one cell, whose corners are two planes apart, then use complementary LDS banks
    CPL = ring ? NPL : HPL + ((4 - HPL % 8) + 8) % 8;
    n_node = 3 + (n_planes - 12);
    acc = 0;
    accc = acc + (size_t)n_node * plane * sizeof(double);
    eb = accc + (size_t)12 * CPL * sizeof(double);
    ho = eb + 3 * (size_t)EPL * tsize;
    hn = ho + 3 * (size_t)HPL * tsize;
    mq = (hn + 3 * (size_t)NPL * tsize + 7) & ~(size_t)7;
    cnt = mq + (qwords ? (size_t)(kBlock / 64) * kMqCap * ((size_t)qwords * tsize + 2 * sizeof(int)) : 0);
    arr = cnt + (size_t)(n_node - 3) * tx * tz * kMoveCodes * sizeof(int);
    rows = arr + (ring ? (size_t)(n_node - 3) * (tx + 2) * (tz + 2) * sizeof(int) : 0);
    bytes = rows + (size_t)(n_node - 3) * tz * 2 * sizeof(int);
  }
};

// Particle state in either form, as the kernel's arithmetic type: cell (i, k), in-cell offsets
// (fx, fz) and momentum.  FP64 keeps positions in cell units; the mixed form keeps the cell key
// and FP32 offsets.  Src holds the species' source arrays in registers for the whole species.
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
    x = s.a[0][p];
    z = s.a[1][p];
    u0 = s.a[2][p];
    u1 = s.a[3][p];
    u2 = s.a[4][p];
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
    cell = s.c[p];
    x = s.a[0][p];
    z = s.a[1][p];
    u0 = s.a[2][p];
    u1 = s.a[3][p];
    u2 = s.a[4][p];
  }
};

// One block per tile of cells (tile rows are cell rows), one wavefront per tile row (or per
// part of a row when the tile has fewer rows than wavefronts).  The row's particles (a
// contiguous range of the cell-sorted order) are split into 64 contiguous runs, one per lane;
// run lengths differ by at most one.  A lane accumulates the deposits of
// particles that stay in their cell in registers and adds them to the LDS tile when its run
// enters the next cell, so LDS atomics are issued once per (lane, cell) instead of once per
// particle; particles changing cell go through a per-wave queue.  The pushed state of the
// particle at iteration `it` of lane `l` is written to location row_start + 64 it + l, which
// makes the stores (and next cycle's loads through the permutation) coalesced.
// MIXED selects the mixed-precision form: FP32 state, gather, push and per-lane partial sums,
// added into FP64 LDS accumulators and the FP64 moment planes.  With chunks of 4 the FP64 form
// needs about 230 VGPRs (two waves per SIMD) and the FP32 form about 150 (three); the
// chunk-of-2 form needs about 120 and 105 (four).  IDS adds the copy of particle ids
// (tests only).  PW selects per-particle densities: each particle's moments are those of unit
// density times its own density, which is read with the state and written with the pushed
// state (a species with one density reads it from a one-element array with stride 0).  CH is
// the chunk of particles a lane loads at once: 4, or 2 where a lane holds about two particles
// per row.  The chunk-of-2 form deposits each particle into LDS at once (no register sums or
// mover queue), reads the fields for every particle, keeps accumulators for the tile's own
// nodes and cells only and sends the moments of a particle that leaves the tile to the global
// planes: about 120 VGPRs (FP64) and 40 KB of LDS at 32 x 4, four blocks per CU.
template <bool PUSH, bool MIXED, bool IDS, bool PW, int CH = 4>
__device__ __forceinline__ void particles_body(const StepArgs &a, int tile) {
  using T = typename std::conditional<MIXED, float, double>::type;
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
  const TileLds Lo(g.n_planes, t.tx, t.tz, (int)sizeof(T), (PUSH && CH == 2) ? 0 : kQw);
  const AccLds acc{reinterpret_cast<double *>(ldsb + Lo.acc),
                   reinterpret_cast<double *>(ldsb + Lo.accc), Lo.plane, Lo.CPL, Lo.LW, Lo.NW};
  T *Eb = reinterpret_cast<T *>(ldsb + Lo.eb);
  T *Ho = reinterpret_cast<T *>(ldsb + Lo.ho);
  T *Hn = reinterpret_cast<T *>(ldsb + Lo.hn);
  int *cntL = reinterpret_cast<int *>(ldsb + Lo.cnt);
  int *arrL = reinterpret_cast<int *>(ldsb + Lo.arr);  // the layout with the ring
  const int LW = Lo.LW, plane = Lo.plane;
  const int n_acc = Lo.n_node * plane + 12 * Lo.CPL;  // node planes, then cell-corner planes

  for (int e = threadIdx.x; e < n_acc; e += blockDim.x) acc.node[e] = 0.0;
  // the chunk-of-2 form: accumulators over the tile's own nodes and cells (no ring)
  constexpr bool kTileOnly = PUSH && CH == 2;
  const int AW = t.tx + 2, AH = t.tz + 2;  // arrival counts: the tile's cells and their ring
  if (PUSH) {
    const int nsl = Lo.n_node - 3;
    for (int e = threadIdx.x; e < nsl * ntc * kMoveCodes; e += blockDim.x) cntL[e] = 0;
    if constexpr (!kTileOnly)
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
      for (int q = 0; q < 3; ++q) Ho[q * Lo.HPL + e] = h_in ? (T)ho[q] : T(0);
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
      for (int q = 0; q < 3; ++q) Eb[q * Lo.EPL + e] = e_in ? (T)(0.5 * (eo[q] + en[q])) : T(0);
    }
    if (PUSH && e < Lo.NPL) {
#pragma unroll
      for (int q = 0; q < 3; ++q) Hn[q * Lo.NPL + e] = n_in ? (T)hn[q] : T(0);
    }
  }
  __syncthreads();

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  MoverQ<T> mq;
  {
    char *qb = ldsb + Lo.mq + (size_t)wave * kMqCap * ((size_t)kQw * sizeof(T) + 2 * sizeof(int));
    mq.v = reinterpret_cast<T *>(qb);
    mq.idx = reinterpret_cast<int *>(qb + (size_t)kMqCap * kQw * sizeof(T));
  }
  const T cxT = (T)g.cx, czT = (T)g.cz;

  for (int s = 0; s < a.nsp; ++s) {
    const SpeciesArgs &sp = a.sp[s];
    if (!sp.active) continue;
    int *const cntS = cntL + s * ntc * kMoveCodes;  // the species' move counters
    const SpConst<T> K{(T)sp.beta, (T)(PW ? sp.cS1 : sp.cS), (T)(PW ? sp.kJ1 : sp.kJ), (T)sp.w};
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
      const int lz = r - k0 + 1;
      const int lk = r - k0;
      CellAcc<T> ca;
      ca.clear();
      ca.cell = -1;
      int nq = 0;  // movers queued by this wavefront (uniform)
      // fields of the cell the lane's run is in, kept in registers while the run stays in it:
      // H^{n+1/2} (fB) and E-bar at its 4 nodes (fE, the push)
      T fB0 = T(0), fB1 = T(0), fB2 = T(0), fE[12];
      // The run is processed in chunks of kChunk particles: the chunk's state loads are issued
      // together (with the next chunk's permutation entries), then its particles are pushed
      // from registers in an unrolled sequence.  Global stores share the vector-memory counter
      // with loads, so a load whose value is still in flight across a loop iteration makes
      // the compiler wait for all earlier stores too; keeping every loaded value inside one
      // iteration lets it wait for the loads alone.  Loads are issued unconditionally (slots
      // past a lane's run read a location inside the state arrays, and their values go
      // unused): a load under a divergent branch also forces a full wait.
      constexpr int kChunk = CH;
      // two particles per chunk: the form for about two particles per lane and row, where a
      // lane's register sums would hold one or two particles; it deposits each particle into
      // LDS directly (no register sums, row-end reduction or mover queue: fewer registers)
      constexpr bool kDirect = PUSH && CH == 2;
      Pstate<MIXED> cb[kChunk];
      int cp_[kChunk], np_[kChunk];
      T cw_[kChunk];
      // A chunk's permutation entries come in one 16-byte load per lane (the array is padded
      // so the load stays inside it); entries past the lane's run are clamped to a location
      // inside the state arrays and their particles go unused.
      static_assert((kChunk == 4 || kChunk == 2) && kPermPad >= 2 * kChunk,
                    "one int4 or int2 of entries per chunk");
      const uint32_t loc_max = (uint32_t)(sp.cap - 1);
      auto perm4 = [&](int first, int out[kChunk]) {
        if constexpr (kChunk == 4) {
          int4 v;
          __builtin_memcpy(&v, perm + first, sizeof(v));
          out[0] = (int)min((uint32_t)v.x, loc_max);
          out[1] = (int)min((uint32_t)v.y, loc_max);
          out[2] = (int)min((uint32_t)v.z, loc_max);
          out[3] = (int)min((uint32_t)v.w, loc_max);
        } else {
          int2 v;
          __builtin_memcpy(&v, perm + first, sizeof(v));
          out[0] = (int)min((uint32_t)v.x, loc_max);
          out[1] = (int)min((uint32_t)v.y, loc_max);
        }
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
          const Pstate<MIXED> &ps = cb[kk];
          int i, k;
          T fx, fz;
          if constexpr (MIXED) {
            k = r;
            i = ps.cell - r * g.nx;
            fx = ps.x;
            fz = ps.z;
          } else {
            i = (int)floor(ps.x);
            k = (int)floor(ps.z);
            fx = ps.x - (double)i;
            fz = ps.z - (double)k;
          }
          const T u0 = ps.u0, u1 = ps.u1, u2 = ps.u2;
          const T wp = PW ? cw_[kk] : K.w;  // the particle's density
          const bool ok = act && k == r && i >= i0 && i < i1;
          if (act && !ok) {
            atomicOr(a.flags, kFlagOrder);
            if (PUSH) sp.locode[j] = ((uint32_t)(jb + it * 64 + lane) << 4) | kAbsorbed;
          }
          // Lanes without a valid particle run the arithmetic on a valid cell of the tile and
          // discard the results, so the main path has no branches around it.
          const int li = ok ? i - i0 : max(ca.cell, 0);
          const int hc = lk * t.tx + li;
          // On entering a new cell: read its fields, use them, and only then flush the previous
          // cell's accumulator.  LDS operations complete in order, so a read issued after the
          // flush's atomics (or consumed while they are in flight) would wait for all of them.
          // The chunk-of-2 form reads them for every particle (a lane holds about two per row,
          // and fields kept across particles would hold about 30 registers).
          const bool newcell = kDirect || (ok && li != ca.cell);
          if (newcell) {
            fB0 = Ho[hc];
            fB1 = Ho[Lo.HPL + hc];
            fB2 = Ho[2 * Lo.HPL + hc];
            if (PUSH) {
              const int e00 = lk * Lo.EW + li;
#pragma unroll
              for (int qq = 0; qq < 3; ++qq) {
                const T *f = Eb + qq * Lo.EPL + e00;
                fE[4 * qq] = f[0];
                fE[4 * qq + 1] = f[1];
                fE[4 * qq + 2] = f[Lo.EW];
                fE[4 * qq + 3] = f[Lo.EW + 1];
              }
            }
          }
          const T one = T(1);
          const T ginv = rsqT(fmaT(u2, u2, fmaT(u1, u1, fmaT(u0, u0, one))));  // 1 / gamma(u^n)
          if (!PUSH) {
            Compact<T> m0 = compact_moments(K, ginv, u0, u1, u2, fB0, fB1, fB2);
            if constexpr (PW) scale_compact(m0, wp);
            if (newcell) {
              if (ca.cell >= 0) ca.flush(acc, lz, dplane);
              ca.clear();
              ca.cell = li;
            }
            if (ok) ca.add(fx, fz, m0, wp);
          } else {
            bool mover = false;
            int mo = 0, mh = 0;
            T fx2, fz2;
            Compact<T> m;
            {
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
              const T bx = bg * fB0, by = bg * fB1, bz = bg * fB2;
              const T a0 = fmaT(K.beta, Ep[0], u0), a1 = fmaT(K.beta, Ep[1], u1);
              const T a2 = fmaT(K.beta, Ep[2], u2);
              const T inv = rcpT(fmaT(bz, bz, fmaT(by, by, fmaT(bx, bx, one))));
              const T ab = fmaT(a2, bz, fmaT(a1, by, a0 * bx));
              const T n0 = fmaT(T(2), fmaT(ab, bx, a0 + fmaT(a1, bz, -(a2 * by))) * inv, -u0);
              const T n1 = fmaT(T(2), fmaT(ab, by, a1 + fmaT(a2, bx, -(a0 * bz))) * inv, -u1);
              const T n2 = fmaT(T(2), fmaT(ab, bz, a2 + fmaT(a0, by, -(a1 * bx))) * inv, -u2);
              const T g1sq = fmaT(n2, n2, fmaT(n1, n1, fmaT(n0, n0, one)));
              const T rg1 = rsqT(g1sq);  // 1 / gamma(u^{n+1})
              const T vx = n0 * rg1, vz = n2 * rg1;
              // position advance: FP64 in cell units; mixed as FP32 offset with integer carry
              T xn, zn;
              int i2, k2;
              bool alive = ok;
              bool finite;
              if constexpr (MIXED) {
                xn = fx + cxT * vx;
                zn = fz + czT * vz;
                finite = isfinite(g1sq) && isfinite(xn) && isfinite(zn);
                const int cxi = finite ? (int)floorT(xn) : 0, czi = finite ? (int)floorT(zn) : 0;
                xn -= (T)cxi;
                zn -= (T)czi;
                int ci = i + cxi, ck = k + czi;
                if (xn >= one) { xn = T(0); ci += 1; }
                if (zn >= one) { zn = T(0); ck += 1; }
                if (g.bc_x == PIC_BC_PERIODIC) {
                  ci = wrap1(ci, g.nx);
                } else if (ci < 0 || ci >= g.nx) {
                  alive = false;
                }
                ck = wrap1(ck, g.nz);
                i2 = ci;
                k2 = ck;
              } else {
                xn = ps.x + g.cx * vx;
                zn = ps.z + g.cz * vz;
                if (g.bc_x == PIC_BC_PERIODIC) {
                  if (xn < 0.0) xn += (double)g.nx;
                  if (xn >= (double)g.nx) xn -= (double)g.nx;
                } else if (xn < 0.0 || xn >= (double)g.nx) {
                  alive = false;
                }
                if (zn < 0.0) zn += (double)g.nz;
                if (zn >= (double)g.nz) zn -= (double)g.nz;
                finite = isfinite(g1sq) && isfinite(xn) && isfinite(zn);
                i2 = finite ? (int)floor(xn) : i;
                k2 = finite ? (int)floor(zn) : k;
              }
              if (ok && !finite) atomicOr(a.flags, kFlagNonFinite);
              alive = alive && finite;
              int di = i2 - i, dk = k2 - k;
              if (di > 1) di -= g.nx;
              if (di < -1) di += g.nx;
              if (dk > 1) dk -= g.nz;
              if (dk < -1) dk += g.nz;
              const bool jump = di < -1 || di > 1 || dk < -1 || dk > 1;
              if (alive && jump) atomicOr(a.flags, kFlagJump);
              alive = alive && !jump;
              if (!alive) {
                di = 0;
                dk = 0;
              }
              const uint32_t code = alive ? (uint32_t)((dk + 1) * 3 + (di + 1)) : kAbsorbed;
              // moments M^{n+3/2} at x^{n+3/2} with u^{n+1}, 1/gamma(u^{n+1}) and H^{n+3/2}
              // of the new cell (read before any LDS atomic of this particle is issued)
              const int hn = (lk + dk + 1) * Lo.NW + (li + di + 1);
              m = compact_moments(K, rg1, n0, n1, n2, Hn[hn], Hn[Lo.NPL + hn], Hn[2 * Lo.NPL + hn]);
              // the new cell, tile-local (a dead particle stays, unused)
              const int ldx = li + di, ldz = lk + dk;
              const bool inside = ldx >= 0 && ldx < cw && ldz >= 0 && ldz < chh;
              if constexpr (PW) scale_compact(m, wp);
              if constexpr (MIXED) {
                fx2 = xn;
                fz2 = zn;
              } else {
                fx2 = xn - (double)i2;
                fz2 = zn - (double)k2;
              }
              if (newcell) {
                if constexpr (!kDirect) {
                  if (ca.cell >= 0) ca.flush(acc, lz, dplane);
                  ca.clear();
                }
                ca.cell = li;
              }
              if constexpr (MIXED) {
                if (ok) {
                  const int loc = jb + it * 64 + lane;
                  sp.mdst_cell[loc] = k2 * g.nx + i2;
                  sp.mdst[0][loc] = xn;
                  sp.mdst[1][loc] = zn;
                  sp.mdst[2][loc] = n0;
                  sp.mdst[3][loc] = n1;
                  sp.mdst[4][loc] = n2;
                  if (PW && wstride) wdst[loc] = wp;
                  sp.locode[j] = ((uint32_t)loc << 4) | code;
                }
              } else {
                // FP64: every lane issues the stores, without a branch (a lane without a
                // particle passes an offset the hardware drops), so the compiler knows how many
                // stores each particle issues and waits for the next particle's loads alone.
                // (The mixed form measured no gain from this and keeps plain stores.)
                const int loc = jb + it * 64 + lane;
                store_or_drop(sp.dst[0], loc, ok, xn);
                store_or_drop(sp.dst[1], loc, ok, zn);
                store_or_drop(sp.dst[2], loc, ok, n0);
                store_or_drop(sp.dst[3], loc, ok, n1);
                store_or_drop(sp.dst[4], loc, ok, n2);
                if constexpr (PW) store_or_drop(wdst, loc, ok && wstride != 0, wp);
                store_or_drop(sp.locode, j, ok, ((uint32_t)loc << 4) | code);
              }
              if (ok) {
                // particle ids (tests only): a separate instantiation, so that its load, which
                // is waited for at once, does not enter the wait counts of the kernel without ids
                if (IDS && sp.dst_id) sp.dst_id[jb + it * 64 + lane] = sp.src_id[p];
                if (code != kAbsorbed) atomicAdd(&cntS[hc * kMoveCodes + code], 1);
              }
              // stayers add to the lane's accumulator, movers go through the queue (with few
              // particles per lane every particle goes to the LDS accumulators at once, or to
              // the global planes if it leaves the tile)
              if constexpr (kDirect) {
                if (alive && inside)
                  deposit_one(acc, ldz * LW + ldx, ldz * t.tx + ldx, fx2, fz2, m, wp, dplane);
                if (alive && !inside)
                  deposit_global(a, i2, k2, fx2, fz2, m, wp, Hn[hn], Hn[Lo.NPL + hn],
                                 Hn[2 * Lo.NPL + hn], dplane);
              } else if (alive && code == 4u) {
                ca.add(fx2, fz2, m, wp);
              } else if (alive) {
                mover = true;
                mo = (lz + dk) * LW + (li + 1 + di);
                mh = hn;
              }
            }
            // queue this iteration's movers; drain first if they would not fit
            const uint64_t mmask = __ballot(mover);
            const int nm = __popcll(mmask);
            if (nq + nm > kMqCap) {
              wave_sync();
              drain_movers<T, PW>(mq, nq, lane, acc, dplane, K.w);
              wave_sync();
              nq = 0;
            }
            if (mover) {
              const int e = nq + __popcll(mmask & lt_mask);
              mq.v[0 * kMqCap + e] = fx2;
              mq.v[1 * kMqCap + e] = fz2;
              mq.v[2 * kMqCap + e] = m.a0;
              mq.v[3 * kMqCap + e] = m.a1;
              mq.v[4 * kMqCap + e] = m.a2;
              mq.v[5 * kMqCap + e] = m.j0;
              mq.v[6 * kMqCap + e] = m.j1;
              mq.v[7 * kMqCap + e] = m.j2;
              if constexpr (PW) mq.v[8 * kMqCap + e] = wp;
              mq.idx[e] = mo;
              mq.idx[kMqCap + e] = mh;
            }
            nq += nm;
          }
        }
      }
      if constexpr (!kDirect) ca.flush_row_end(acc, lz, dplane, lane);
      if (PUSH && nq > 0) {
        wave_sync();
        drain_movers<T, PW>(mq, nq, lane, acc, dplane, K.w);
        wave_sync();
      }
    }
  }
  __syncthreads();
  // Move counts of the tile's cells, for the ranking.  The counts of every species are kept
  // until here, so the species need no barriers between them.
  for (int s = 0; s < a.nsp; ++s) {
    const SpeciesArgs &sp = a.sp[s];
    if (!PUSH || !sp.active) continue;
    const int *cntS = cntL + s * ntc * kMoveCodes;
    int *arrS = arrL + s * AW * AH;
    {
      const SmallDiv div_cw(cw);
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
            if constexpr (!kTileOnly) atomicAdd(&arrS[(lkk + d / 3) * AW + (li + d % 3)], v);
          }
        }
        if (a.count_masks) sp.cmask[cg] = (uint16_t)mask;
      }
    }
  }
  // Fold the tile's accumulators into the global FP64 moment planes, one node per thread:
  // delta-j and the densities as they are; S-hat from the S-hat scalars of the (up to) four
  // cells around the node, each expanded with its cell's B (H^{n+3/2} after a push, H^{n+1/2}
  // for a deposit of the current state): S-hat = a0 I + a1 [B]x + a2 B B^T.
  const SmallDiv div_lw(LW);
  for (int idx = threadIdx.x; idx < plane; idx += blockDim.x) {
    const int lzz = div_lw.q(idx), lx = idx - lzz * LW;
    constexpr int kOff = kTileOnly ? 0 : 1;  // the ring's column and row before the tile
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
      const int ac = kTileOnly ? cz * t.tx + cx : rc;             // in the corner planes
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
  if (PUSH) {
    // The particles the tile's cells send to each cell of the tile and its ring (the cell
    // (x - dx, z - dz) sends count[code (dx, dz)]), added to the per-cell arrival counts: the
    // sort's scan reads those instead of gathering nine counts per cell.
    // (the layout with the ring sums them in LDS during the count pass)
    if constexpr (!kTileOnly) __syncthreads();
    for (int s = 0; s < a.nsp; ++s) {
      const SpeciesArgs &sp = a.sp[s];
      if (!sp.active) continue;
      const int *cntS = cntL + s * ntc * kMoveCodes;
      const int *arrS = arrL + s * AW * AH;
      for (int e = threadIdx.x; e < AW * AH; e += blockDim.x) {
        const int az = SmallDiv(AW).q(e), ax = e - az * AW;
        int v = 0;
        if constexpr (kTileOnly) {
#pragma unroll
          for (int d = 0; d < kMoveCodes; ++d) {
            const int sx = ax - d % 3, sz = az - d / 3;  // the source cell, tile-local
            if (sx >= 0 && sx < cw && sz >= 0 && sz < chh) v += cntS[(sz * t.tx + sx) * kMoveCodes + d];
          }
        } else {
          v = arrS[e];
        }
        if (v == 0) continue;
        int gi = i0 - 1 + ax;
        const int gk = wrap1(k0 - 1 + az, g.nz);
        if (g.bc_x == PIC_BC_PERIODIC) gi = wrap1(gi, g.nx);
        atomicAdd(&sp.arr[(int64_t)gk * g.nx + gi], v);
      }
    }
  }
}

// Three waves per SIMD: the register sums take about 150 VGPRs.
template <bool PUSH, bool IDS, bool PW>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3, 3)))
void k_particles_runs(const StepArgs a) {
  // clear the next order's tile flags (set by the scan of this cycle's sort); the grid has a
  // block for every tile index
  if (threadIdx.x == 0 && (int)blockIdx.x < a.t.ntiles) a.tile_active_next[blockIdx.x] = 0;
  const int tile = block_tile(a.t, a.tile_list);
  if (tile < 0) return;
  particles_body<PUSH, true, IDS, PW>(a, tile);
}

}  // namespace

size_t runs_lds_bytes(const GridArgs &g, const TileArgs &t, bool pw) {
  return TileLds(g.n_planes, t.tx, t.tz, (int)sizeof(float), mq_words(pw)).bytes;
}

hipError_t launch_particles_runs(const StepArgs &a, bool push, hipStream_t s) {
  bool ids = false, pw = false;
  for (int q = 0; q < a.nsp; ++q) {
    ids = ids || a.sp[q].dst_id != nullptr;
    pw = pw || (a.sp[q].active && a.sp[q].w_stride != 0);
  }
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
  return hipGetLastError();
}

}  // namespace pic
