// stage_tile.hpp -- one stage of the MHD update in a single kernel.
//
// Each workgroup (34 x 15 threads, 8 wave64s, or one of the smaller tiles of
// stage_args.hpp) owns a tile of 32 x 13 active columns in (x1, x2) plus a
// one-cell ring, and marches along x3 over a segment of kz planes.  Per plane
// everything stays on chip:
//   * every thread owns one column of the region; it converts its column's
//     conserved state to primitives (Sec. 3.1) one plane ahead of use and keeps
//     a short window of planes in registers for the reconstruction along x3;
//   * the primitives of the current plane, plus LA extra rings, go to LDS for
//     the reconstructions along x1 and x2 (DC / PLM / PPM, Sec. 3.2.1);
//   * each thread solves the Riemann problems (HLLD / HLLE, Sec. 3.2.2) on the
//     lower x1-face and x2-face of its column in this plane and on the lower
//     x3-face of its column's cell;
//   * face fluxes, face EMFs, upwind weights and cell-centred EMFs are
//     exchanged through LDS to form the upwind-CT corner EMFs (Sec. 3.1);
//   * the flux divergence and the CT curl accumulate in registers and the
//     plane below is written out once its upper x3 fluxes / EMFs exist
//     (2S stage update, Eq. (rk-2s)).
// Two barriers per plane: after the primitives are in LDS, and after the face
// results are (and two more where cell edges are shared through LDS).  The face-field update that reads a plane's corner EMFs runs
// after the next plane's first barrier, and the exchange slots read by the
// corner EMFs are written after that barrier too, so no third barrier is
// needed to keep one plane's reads apart from the next plane's writes.
// HBM traffic per stage is the input state (with the halo overlap of
// neighbouring tiles), U^n where the stage needs it, and the output state.
//
// Bound by the issue and latency of FP64 VALU instructions at two waves per
// SIMD (registers and LDS allow no more), so no wave may also wait for memory:
//   * one raw-cell buffer per thread holds the look-ahead plane's loads while
//     the x1- and x2-faces are solved and the ring cell's loads while the
//     x3-face is, each converted only after the Riemann problems in between;
//   * the output's stored terms are read without a branch before the second
//     barrier and used after the corner EMFs;
//   * planes are addressed by a scalar base and a 32-bit vector offset.
// Before, a plane exposed three to five memory latencies one after the other
// (loads waited for inside the branch that issued them).  That and the later
// changes to this kernel together, sustained steps of a smooth 256^3 state without
// the CFL pass: VL2+PLM+HLLD 3.00 -> 2.66 ms, RK2+DC 2.72 -> 2.32 ms, RK3+PPM
// 16.0 -> 9.9 ms.
#pragma once

#include "stage_args.hpp"

namespace athmhd {

namespace {

// Arrays of one block: stage input (periodic images are read by index wrap,
// ghost entries are not used), U^n (the u^(1) register), stage output (active
// cells and their lower faces).
struct BlockPtrs {
  const double* xc;
  const double* xb;
  const double* unc;
  const double* unb;
  double* oc;
  double* ob;
  double* fm = nullptr;  // optional: mass fluxes through the lower faces of the active cells (3 face arrays)
};

// z-frame primitive vector of a cell: (rho, v3, v1, v2, P, B1cc, B2cc) plus
// B3cc kept alongside
struct ZCell {
  double q[7];
  double b3;
};

// Raw data of one cell needed to form its primitives.
struct Raw {
  double u[5];
  double b1lo, b1hi, b2lo, b2hi, b3lo, b3hi;
};

// How a block's neighbours are read (MESH):
//   0  the block is its own periodic neighbour: at the periodic images directly,
//      so its ghost entries are never needed;
//   1  the stored ghost entries, which an exchange filled before the stage
//      (coupled batches, meshes with passive scalars);
//   2  the blocks of a coupled mesh as one periodic domain: the tiles cover the
//      domain, not the blocks, and every column and plane is read and written
//      in the block that owns it, so no exchange is needed and tiles are not
//      cut at block edges.
// Column: byte offsets inside one x3 plane of its cell (a cell array) and of
// its lower faces, its upper x1 face and its upper x2 face (a face array); with
// MESH 2 they include the block's offset in its layer of blocks.
// A plane's base address is the same for the whole workgroup (scalar
// registers), so an access is one instruction with a 32-bit vector offset and
// no vector address arithmetic.  A plane's offsets fit 32 bits: a face array
// holds fewer than 2^31 entries in at least 6 planes (MESH 2: checked when the
// launch is chosen).
struct Col {
  unsigned c, f, f1, f2;
};

// Stored index read for position idx (cell, or face when hi = N) along a
// direction with n active cells: its periodic image (MESH 0), or the stored
// entry itself (MESH 1), clamped into the array for the columns of a ragged
// tile past the block edge, whose results are never written out.
template <int MESH>
__device__ __forceinline__ int read_index(const Geo& g, int idx, int n, int hi) {
  if (MESH == 0) return wrap_index(idx, n, g.ng);
  return idx < 0 ? 0 : (idx > hi ? hi : idx);
}

// Plane cursor: the stored plane (and layer of blocks) read for an unwrapped
// plane index, clamped where it is used with MESH 1.  Advancing it costs a
// compare, no division, in every plane.
struct Pos {
  int k, b;
};
template <int MESH>
__device__ __forceinline__ Pos pos_at(const Geo& g, int k) {
  if (MESH == 0) return Pos{wrap_index(k, g.n3, g.ng), 0};
  if (MESH == 1) return Pos{k, 0};
  const int d = wrap_index(k, g.mesh[2] * g.n3, g.ng) - g.ng;
  return Pos{g.ng + d % g.n3, d / g.n3};
}
template <int MESH>
__device__ __forceinline__ Pos pos_next(const Geo& g, Pos q) {
  ++q.k;
  if (MESH != 1 && q.k == g.ng + g.n3) {
    q.k = g.ng;
    if (MESH == 2) q.b = q.b + 1 == g.mesh[2] ? 0 : q.b + 1;
  }
  return q;
}
template <int MESH>
__device__ __forceinline__ Pos pos_read(Pos q, int hi) {
  if (MESH == 1) q.k = min(max(q.k, 0), hi);
  return q;
}

template <int MESH>
__device__ __forceinline__ Col make_col(const Geo& g, int i, int j) {
  Col c;
  if (MESH == 2) {
    const int D1 = g.mesh[0] * g.n1, D2 = g.mesh[1] * g.n2;
    const int i0 = wrap_index(i, D1, g.ng) - g.ng, i1 = wrap_index(i + 1, D1, g.ng) - g.ng;
    const int j0 = wrap_index(j, D2, g.ng) - g.ng, j1 = wrap_index(j + 1, D2, g.ng) - g.ng;
    const int a0 = i0 / g.n1, a1 = i1 / g.n1, b0 = j0 / g.n2, b1 = j1 / g.n2;
    const unsigned x0 = (unsigned)(g.ng + i0 - a0 * g.n1), x1 = (unsigned)(g.ng + i1 - a1 * g.n1);
    const unsigned y0 = (unsigned)(g.ng + j0 - b0 * g.n2), y1 = (unsigned)(g.ng + j1 - b1 * g.n2);
    const unsigned cb = (unsigned)g.cblock, fb = (unsigned)g.fblock, m0 = (unsigned)g.mesh[0];
    c.c = 8u * ((a0 + m0 * b0) * cb + y0 * g.N1 + x0);
    c.f = 8u * ((a0 + m0 * b0) * fb + y0 * g.F1 + x0);
    c.f1 = 8u * ((a1 + m0 * b0) * fb + y0 * g.F1 + x1);
    c.f2 = 8u * ((a0 + m0 * b1) * fb + y1 * g.F1 + x0);
    return c;
  }
  const int i0 = read_index<MESH>(g, i, g.n1, g.N1 - 1), i1 = read_index<MESH>(g, i + 1, g.n1, g.N1);
  const int j0 = read_index<MESH>(g, j, g.n2, g.N2 - 1), j1 = read_index<MESH>(g, j + 1, g.n2, g.N2);
  c.c = 8u * (unsigned)(j0 * g.N1 + i0);
  c.f = 8u * (unsigned)(j0 * g.F1 + i0);
  c.f1 = 8u * (unsigned)(j0 * g.F1 + i1);
  c.f2 = 8u * (unsigned)(j1 * g.F1 + i0);
  return c;
}

// base addresses of plane q of cell array v and of face array d
typedef const char* Plane;
template <int MESH>
__device__ __forceinline__ Plane cell_plane(const Geo& g, const double* x, int v, Pos q) {
  int64_t o = v * g.cvar + (int64_t)q.k * (g.N1 * g.N2);
  if (MESH == 2) o += q.b * (g.cblock * (g.mesh[0] * g.mesh[1]));
  return reinterpret_cast<const char*>(x + o);
}
template <int MESH>
__device__ __forceinline__ Plane face_plane(const Geo& g, const double* x, int d, Pos q) {
  int64_t o = d * g.fvar + (int64_t)q.k * (g.F1 * g.F2);
  if (MESH == 2) o += q.b * (g.fblock * (g.mesh[0] * g.mesh[1]));
  return reinterpret_cast<const char*>(x + o);
}
__device__ __forceinline__ double at(Plane pl, unsigned off) { return *reinterpret_cast<const double*>(pl + off); }
__device__ __forceinline__ void put(Plane pl, unsigned off, double v) {
  *reinterpret_cast<double*>(const_cast<char*>(pl) + off) = v;
}
// The offsets, made opaque where they are used: otherwise the compiler hoists
// the sum of base and offset out of the plane loop as 64-bit vector pointers,
// one per array.
__device__ __forceinline__ Col here(Col c) {
  asm("" : "+v"(c.c), "+v"(c.f), "+v"(c.f1), "+v"(c.f2));
  return c;
}
__device__ __forceinline__ unsigned here(unsigned o) {
  asm("" : "+v"(o));
  return o;
}

// Conserved state and the six bounding face fields of the cell of column c in
// the plane of cursor k.
template <int MESH>
__device__ __forceinline__ void load_raw(const Geo& g, const double* xc, const double* xb, const Col& col, Pos k,
                                         Raw& r) {
  const Col c = here(col);
  const Pos k0 = pos_read<MESH>(k, g.N3 - 1), k1 = pos_read<MESH>(pos_next<MESH>(g, k), g.N3);
#pragma unroll
  for (int v = 0; v < 5; ++v) r.u[v] = at(cell_plane<MESH>(g, xc, v, k0), c.c);
  const Plane b1 = face_plane<MESH>(g, xb, 0, k0), b2 = face_plane<MESH>(g, xb, 1, k0);
  r.b1lo = at(b1, c.f);
  r.b1hi = at(b1, c.f1);
  r.b2lo = at(b2, c.f);
  r.b2hi = at(b2, c.f2);
  r.b3lo = at(face_plane<MESH>(g, xb, 2, k0), c.f);
  r.b3hi = at(face_plane<MESH>(g, xb, 2, k1), c.f);
}

// cons -> prim: w = (rho, v1, v2, v3, P, B1cc, B2cc, B3cc); returns the flags
// of cell_prim (bit 0 non-physical, bit 1 floored).  The same cell is
// converted at several places (the register window along x3, the primitive
// plane, the extra rings, and again by the neighbouring tile or x3 segment);
// cell_prim computes without contraction, so all of them get the same bits.
// Fluxes and EMFs on tile and segment boundaries are computed twice and must
// agree exactly, or the CT update no longer preserves div B (reconstruction
// limiters can turn an ulp of difference into an O(1) one).
template <bool FL>
__device__ __forceinline__ int to_prim(const Raw& r, double gm1, const Floors& fl, double* w) {
  double b[3];
  {
#pragma clang fp contract(off)
    b[0] = 0.5 * (r.b1lo + r.b1hi);
    b[1] = 0.5 * (r.b2lo + r.b2hi);
    b[2] = 0.5 * (r.b3lo + r.b3hi);
  }
  const int flags = cell_prim(r.u, b, gm1, FL ? fl : Floors{0.0, 0.0}, w);
  w[5] = b[0];
  w[6] = b[1];
  w[7] = b[2];
  return flags;
}

__device__ __forceinline__ void to_zcell(const double* w, ZCell& z) {
  z.q[0] = w[0]; z.q[1] = w[3]; z.q[2] = w[1]; z.q[3] = w[2]; z.q[4] = w[4]; z.q[5] = w[5]; z.q[6] = w[6];
  z.b3 = w[7];
}

__device__ __forceinline__ FaceState make_state(const double* q) {
  FaceState s;
  s.rho = q[0]; s.vn = q[1]; s.vt1 = q[2]; s.vt2 = q[3]; s.p = q[4]; s.bt1 = q[5]; s.bt2 = q[6];
  return s;
}

template <int RS, bool FL>
__device__ __forceinline__ void riemann(const double* ql, const double* qr, double bn, const Gas& gas, double ct_eps,
                                        const Floors& fl, int& nfl, FaceFlux& F, double& w) {
  FaceState L = make_state(ql), R = make_state(qr);
  if (FL) nfl += floor_state(L, fl) + floor_state(R, fl);
  double smax;
  riemann_flux<RS>(L, R, bn, gas, F, smax);
  w = ct_weight(F.rho, 0.5 * (L.rho + R.rho), smax, ct_eps);
}

// LDS layout: the primitive plane (with LA extra rings), the per-thread
// exchange slots and the corner EMFs are separate, so a thread can publish
// each Riemann result as soon as it has it.
template <int LA, class T>
struct Smem {
  static constexpr int PW = T::BX + 2 * LA;  // width of the primitive plane incl. extra rings
  static constexpr int PH = T::BY + 2 * LA;
  static constexpr int PL = PW * PH;
};

enum {
  X_FX = 0, X_FY = 5, X_E3X = 10, X_WX, X_E3Y, X_WY, X_E3C, X_E1Z, X_E2Z, X_WZ, X_E1C, X_E2C, X_E1CP, X_E2CP,
  // the previous plane's x1-face E2 and weight, x2-face E1 and (DC, PLM) weight:
  // read only by the own thread, kept here rather than in registers
  X_E2XP, X_WXP, X_E1YP, X_WYP, X_N
};
// exchange slots of a stage: PPM's wider primitive plane leaves room for all
// but the last (its x2-face weight stays in a register)
template <int RECON>
constexpr int exchange_slots() { return RECON >= 2 ? X_N - 1 : X_N; }

// Face-field update of plane q from its corner EMFs in sc (E1, E2, E3 of the
// own column's edges; the neighbours' at tid + 1 and tid + BX): completes B1
// and B2 on the lower faces of cell q-1, writes B3 on the face q-1/2, and
// leaves the partial B1, B2 of plane q in bacc[5], bacc[6].  pwb holds the
// pointwise terms (g1 U^n + g0 X) of B1, B2 at q-1 and B3 at q.
template <int MESH>
__device__ __forceinline__ void face_update(const Geo& g, const double* sc, int tid, int BX, int NT,
                                            unsigned f, int q, Pos at_q, Pos below, int k0, int kend, double i1,
                                            double i2, double i3,
                                            double bdt, const double* pwb, double* bacc, double* ob) {
  const int tE = tid + 1, tN = tid + BX;
  const double e1 = sc[0 * NT + tid], e2 = sc[1 * NT + tid], e3 = sc[2 * NT + tid];
  // B1(i-1/2, j): -(E3(j+1/2) - E3(j-1/2))/dx2 + (E2(k+1/2) - E2(k-1/2))/dx3
  const double a5 = -(sc[2 * NT + tN] - e3) * i2 - e2 * i3;
  bacc[5] += e2 * i3;
  // B2(i, j-1/2): -(E1(k+1/2) - E1(k-1/2))/dx3 + (E3(i+1/2) - E3(i-1/2))/dx1
  const double a6 = (sc[2 * NT + tE] - e3) * i1 + e1 * i3;
  bacc[6] -= e1 * i3;
  // B3(i, j, q-1/2): -(E2(i+1/2) - E2(i-1/2))/dx1 + (E1(j+1/2) - E1(j-1/2))/dx2
  const double db3 = -(sc[1 * NT + tE] - e2) * i1 + (sc[0 * NT + tN] - e1) * i2;
  if (q < kend) put(face_plane<MESH>(g, ob, 2, at_q), f, pwb[2] + bdt * db3);
  if (q - 1 >= k0) {
    put(face_plane<MESH>(g, ob, 0, below), f, pwb[0] + bdt * bacc[5]);
    put(face_plane<MESH>(g, ob, 1, below), f, pwb[1] + bdt * bacc[6]);
  }
  bacc[5] = a5;
  bacc[6] = a6;
}

// Reconstructed states of a cell and a face along one direction of the primitive
// plane (row: the cell, st: stride of the direction), in the face's frame (map;
// nrm: slot of the cell-centred normal field).
// own_edges: left and right edge of the own cell.
template <int RECON, bool FLAT>
__device__ __forceinline__ void own_edges(const double* sp, int PL, int row, int st, const int (&map)[7],
                                          double* lo, double* hi) {
  constexpr int NW = 2 * RECON + 1;
#pragma unroll
  for (int v = 0; v < 7; ++v) {
    double line[NW];
#pragma unroll
    for (int o = 0; o < NW; ++o) line[o] = sp[map[v] * PL + row + (o - RECON) * st];
    cell_edges<RECON, FLAT>(line, lo[v], hi[v]);
    if (FLAT) {
      // one variable at a time: all masks of 14 limiters at once spill scalar registers
      asm volatile("" : "+v"(lo[v]), "+v"(hi[v]));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// face_states: right edge of the cell below and left edge of the own cell.
template <int RECON, bool CHAR>
__device__ __forceinline__ void face_states(const double* sp, int PL, int row, int st,
                                            const int (&map)[7], int nrm, double gamma, double* ql, double* qr) {
  constexpr int NW = 2 * RECON + 1;
  if constexpr (CHAR) {
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      double line[NW][7];
#pragma unroll
      for (int o = 0; o < NW; ++o)
#pragma unroll
        for (int v = 0; v < 7; ++v) line[o][v] = sp[map[v] * PL + row + (o - RECON - 1 + side) * st];
      char_edges<RECON>(line, sp[nrm * PL + row + (side - 1) * st], gamma, side == 1 ? qr : nullptr,
                        side == 0 ? ql : nullptr);
    }
  } else {
#pragma unroll
    for (int v = 0; v < 7; ++v) {
      const double* s = sp + map[v] * PL + row;
      double lineL[NW], lineR[NW];
#pragma unroll
      for (int o = 0; o < NW; ++o) {
        lineL[o] = s[(o - RECON - 1) * st];
        lineR[o] = s[(o - RECON) * st];
      }
      double a0, a1, b0, b1;
      cell_edges<RECON>(lineL, a0, a1);
      cell_edges<RECON>(lineR, b0, b1);
      ql[v] = a1;
      qr[v] = b0;
    }
  }
}

// One tile (tile_x, tile_y) of a block over the active planes [k0, kend).
// MF: also store the mass flux through the lower faces of the active cells,
// which passive scalars are carried by.
// SAME (donor cell only): the stage input is U^n itself (the first stage of
// every scheme), so the output's pointwise terms come from the raw cell read
// for the window one plane earlier, carried, instead of being read again.
// CHAR: PLM on characteristic variables.  Every face takes the edges of its two
// cells from their own waves (about 320 operations a cell, no face shares one
// with its neighbour through LDS, which is full), 58 registers spilled; the
// five-kernel pipeline with 7 x 7 eliminations it replaces took 5.97 ms per
// VL2+HLLD step at 192^3, of which the donor-cell predictor 1.6 ms; now 1.97 ms.
template <int RECON, int RS, class T, bool FL, int MESH = 0, bool MF = false, bool SAME = false, bool CHAR = false,
          bool LONE = false>
__device__ __forceinline__ void stage_tile(const Geo& g, const BlockPtrs& bp, const StageArgs& sa, int tile_x,
                                           int tile_y, int k0, int kend, double* sp,
                                           double* sx, double* sc) {
  constexpr int LA = RECON;  // cells of look-ahead / extra LDS rings: DC 0, PLM 1, PPM 2
  constexpr int NW = 2 * LA + 1;
  constexpr int BX = T::BX, BY = T::BY, NT = T::NT, TX = T::TX, TY = T::TY;
  using S = Smem<LA, T>;
  constexpr int PW = S::PW, PL = S::PL;
  // the last stage's output is U^n's own array, and the first stage's input is
  // U^n: nothing here may be called unaliased
  const double* const xc = bp.xc;
  const double* const xb = bp.xb;
  const double* const unc = bp.unc;
  const double* const unb = bp.unb;
  double* const oc = bp.oc;
  double* const ob = bp.ob;
  const double bdt = sa.dt_dev ? sa.beta * *sa.dt_dev : sa.cf.bdt;

  const int tid = threadIdx.x;
  const int tx = tid % BX, ty = tid / BX;
  const int x0 = g.ng + tile_x * TX, y0 = g.ng + tile_y * TY;
  // own column (columns of a ragged tile past the block edge only feed values
  // that are never written out); reads use the periodic images
  const int gi = x0 - 1 + tx, gj = y0 - 1 + ty;
  const Col own = make_col<MESH>(g, gi, gj);
  const bool act = tx >= 1 && tx <= TX && ty >= 1 && ty <= TY && 
                   gi < g.ng + (MESH == 2 ? g.mesh[0] * g.n1 : g.n1) &&
                   gj < g.ng + (MESH == 2 ? g.mesh[1] * g.n2 : g.n2);

  // ---- extra LDS rings (LA per side): left and right columns (BY cells per
  // depth), bottom and top rows (BX cells per depth), one cell per thread
  constexpr int NRING = 2 * LA * (BX + BY);
  static_assert(NRING <= NT, "ring cells must fit the workgroup");
  const bool ring = tid < NRING;
  int rl = 0;
  Col rcol{0u, 0u, 0u, 0u};
  if (ring) {
    constexpr int LD = LA > 0 ? LA : 1;  // no ring cells when LA = 0
    int rlx, rly;
    if (tid < 2 * LA * BY) {
      const int side = tid / (LD * BY), e = tid % (LD * BY), d = e / BY, pos = e % BY;
      rly = LA + pos;
      rlx = side == 0 ? LA - 1 - d : LA + BX + d;
    } else {
      const int u = tid - 2 * LA * BY;
      const int side = u / (LD * BX), e = u % (LD * BX), d = e / BX, pos = e % BX;
      rlx = LA + pos;
      rly = side == 0 ? LA - 1 - d : LA + BY + d;
    }
    rl = rly * PW + rlx;
    rcol = make_col<MESH>(g, x0 - 1 - LA + rlx, y0 - 1 - LA + rly);
  }

  const double i1 = 1.0 / g.dx1, i2 = 1.0 / g.dx2, i3 = 1.0 / g.dx3;
  const double gm1 = sa.gas.gm1;
  // bit 30: a non-physical cell was met; below it the floor activations: each
  // active cell (in its own column and segment) and each lower face of one counts
  // once, whatever the tiles and segments
  constexpr int kBad = 1 << 30;
  int seen = 0;

  // ---- z window: planes p-LA .. p+LA of the own column
  ZCell win[NW];
  // normal fields (lower x1, x2, x3 faces of the own cell) of planes
  // p .. p+LA, carried from the look-ahead loads; with PPM's five-plane window
  // they are read again from the cache each plane instead (fewer registers
  // live through the plane: 4.6 % faster for PPM, 2.2 % slower for PLM)
  constexpr bool RELOAD_BN = LA >= 2;
  constexpr int NBQ = RELOAD_BN ? 1 : LA + 1;
  double bnq[NBQ][3];
  // next own plane to load, and planes p, p - 1 and p - 2 (the last two: not with MESH 0)
  Pos ka = pos_at<MESH>(g, k0 - 1 - LA), kr = pos_at<MESH>(g, k0 - 1), kr1 = kr, kr2 = kr;
  {
    double w[8];
    Raw raw;
#pragma unroll
    for (int o = 0; o < NW - 1; ++o) {
      load_raw<MESH>(g, xc, xb, own, ka, raw);
      ka = pos_next<MESH>(g, ka);
      const int f = to_prim<FL>(raw, gm1, sa.fl, w);
      if (f & 1) seen |= kBad;
      if (FL && o > LA) seen += f >> 1;
      to_zcell(w, win[o + 1]);
      if (!RELOAD_BN && o >= LA) {
        bnq[o - LA][0] = raw.b1lo;
        bnq[o - LA][1] = raw.b2lo;
        bnq[o - LA][2] = raw.b3lo;
      }
    }
  }
  Raw pre;   // raw data of the next look-ahead plane
  load_raw<MESH>(g, xc, xb, own, ka, pre);

  double qz_carry[7];  // left state of the next x3-face (right edge of the cell below)
  constexpr bool WY_REG = exchange_slots<RECON>() < X_N;
  double wy_prev = 0.5;  // PPM: the previous plane's x2-face weight
  double acc_prev[7];  // partial update of the plane below: 5 conserved, B1, B2
  static_assert(!SAME || LA == 0, "the raw cell of the output plane is carried with the donor-cell window only");
  // SAME: conserved state and lower B1, B2 of the previous plane's cell, and
  // of the current plane's (from its look-ahead load, until the output step)
  double ucar[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  double unext[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  // where the look-ahead plane's loads are issued: before the x1-face (DC),
  // between the x1- and the x2-face (PLM), after the x2-face (PPM).  Earlier
  // hides more of their latency, later keeps 22 registers free through a
  // Riemann problem.  Sustained steps of a smooth 256^3 state without the CFL
  // pass, with each of the three places: RK2+DC 2.33 / 2.33 / 2.39 ms, VL2+PLM 2.68 /
  // 2.65 / 2.67 ms, RK3+PPM (18 x 14 threads) 11.10 / 10.14 / 9.92 ms.
  constexpr int PF = RECON;
  double pwb[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int v = 0; v < 7; ++v) { acc_prev[v] = 0.0; qz_carry[v] = 0.0; }

  for (int p = k0 - 1; p <= kend; ++p) {
    const bool zface = p >= k0;
    // the segment's planes p, p - 1, p - 2: plain indices for periodic blocks (the
    // cursors kept for them cost the batch 48 bytes of spill, 4 %), the cursors
    // elsewhere (coupled batch 4.50 ms with them, 4.60 without)
    const Pos w0 = MESH ? kr : Pos{p, 0}, w1 = MESH ? kr1 : Pos{p - 1, 0}, w2 = MESH ? kr2 : Pos{p - 2, 0};
    // ---- 1-2. shift the window and convert the look-ahead plane p+LA
#pragma unroll
    for (int o = 0; o < NW - 1; ++o) win[o] = win[o + 1];
    {
      double w[8];
      const int f = to_prim<FL>(pre, gm1, sa.fl, w);
      if (f & 1) seen |= kBad;
      if (FL && p + LA >= k0 && p + LA < kend) seen += f >> 1;
      to_zcell(w, win[NW - 1]);
      if (SAME) {
#pragma unroll
        for (int v = 0; v < 5; ++v) unext[v] = pre.u[v];
        unext[5] = pre.b1lo;
        unext[6] = pre.b2lo;
      }
      if (RELOAD_BN) {
        const Pos kp = pos_read<MESH>(kr, g.N3 - 1);
#pragma unroll
        for (int d = 0; d < 3; ++d) bnq[0][d] = at(face_plane<MESH>(g, xb, d, kp), own.f);
      } else {
        bnq[NBQ - 1][0] = pre.b1lo;
        bnq[NBQ - 1][1] = pre.b2lo;
        bnq[NBQ - 1][2] = pre.b3lo;
      }
    }

    // ---- 3. own cell of plane p: primitives to LDS, cell EMFs
    double e1c, e2c, e3c;
    {
      const ZCell& cur = win[LA];
      const int l = (ty + LA) * PW + tx + LA;
      sp[0 * PL + l] = cur.q[0];
      sp[1 * PL + l] = cur.q[2];
      sp[2 * PL + l] = cur.q[3];
      sp[3 * PL + l] = cur.q[1];
      sp[4 * PL + l] = cur.q[4];
      sp[5 * PL + l] = cur.q[5];
      sp[6 * PL + l] = cur.q[6];
      sp[7 * PL + l] = cur.b3;
      // E = -v x B at the cell centre
      const double v1 = cur.q[2], v2 = cur.q[3], v3 = cur.q[1];
      const double b1c = cur.q[5], b2c = cur.q[6], b3c = cur.b3;
      e1c = -(v2 * b3c - v3 * b2c);
      e2c = -(v3 * b1c - v1 * b3c);
      e3c = -(v1 * b2c - v2 * b1c);
    }

    // ---- 4. the ring cell's loads, used after the x3-face (the raw buffer is
    // free between the look-ahead plane's conversion and its next load)
    if (ring) load_raw<MESH>(g, xc, xb, rcol, kr, pre);

    // ---- 5. reconstruction along x3 and the Riemann problem on the lower
    // x3-face (p-1/2) of the own cell
    double fz_cons[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    double wz = 0.5, e1z = 0.0, e2z = 0.0;
    {
      double zl[7], zr[7];
      if constexpr (CHAR) {
        double line[NW][7], right[7];
#pragma unroll
        for (int o = 0; o < NW; ++o)
#pragma unroll
          for (int v = 0; v < 7; ++v) line[o][v] = win[o].q[v];
        char_edges<RECON>(line, win[LA].b3, sa.gas.gamma, zr, right);
#pragma unroll
        for (int v = 0; v < 7; ++v) {
          zl[v] = qz_carry[v];
          qz_carry[v] = right[v];
        }
      } else {
#pragma unroll
      for (int v = 0; v < 7; ++v) {
        double line[NW];
#pragma unroll
        for (int o = 0; o < NW; ++o) line[o] = win[o].q[v];
        double left, right;
        cell_edges<RECON, LONE>(line, left, right);
        zl[v] = qz_carry[v];
        zr[v] = left;
        qz_carry[v] = right;
      }
      }
      if (zface) {
        const double bn3 = bnq[0][2];
        FaceFlux fz;
        int hit = 0;
        riemann<RS, FL>(zl, zr, bn3, sa.gas, sa.ct_eps, sa.fl, hit, fz, wz);
        if (FL && p < kend) seen += hit;
        // z-frame -> (rho, M1, M2, M3, E); x3-face E2 = -F(B1), E1 = +F(B2)
        fz_cons[0] = fz.rho; fz_cons[1] = fz.mt1; fz_cons[2] = fz.mt2; fz_cons[3] = fz.mn; fz_cons[4] = fz.e;
        e2z = -fz.bt1;
        e1z = fz.bt2;
        if (MF && act && p < kend) put(face_plane<MESH>(g, bp.fm, 2, w0), own.f, fz.rho);
      }
    }
    if (ring) {
      double w[8];
      to_prim<FL>(pre, gm1, sa.fl, w);
#pragma unroll
      for (int v = 0; v < 8; ++v) sp[v * PL + rl] = w[v];
    }
    __syncthreads();

    // exchange values read only after the next barrier (writing them here, not
    // before the barrier above, lets the previous plane's corner EMFs read the
    // same slots without a third barrier per plane)
    sx[X_E3C * NT + tid] = e3c;
    // the previous plane's cell EMFs move to their own slots first (the slots
    // of the current plane still hold them: nobody reads these between the
    // previous plane's corner EMFs and here)
    sx[X_E1CP * NT + tid] = sx[X_E1C * NT + tid];
    sx[X_E2CP * NT + tid] = sx[X_E2C * NT + tid];
    sx[X_E1C * NT + tid] = e1c;
    sx[X_E2C * NT + tid] = e2c;
    sx[X_E1Z * NT + tid] = e1z;
    sx[X_E2Z * NT + tid] = e2z;
    sx[X_WZ * NT + tid] = wz;
    // ---- 8, for plane p-1: its face-field updates from the corner EMFs that
    // the previous iteration left in sc
    if (act && p - 1 >= k0)
      face_update<MESH>(g, sc, tid, BX, NT, own.f, p - 1, w1, w2, k0, kend, i1, i2, i3, bdt, pwb, acc_prev, ob);

    if (PF == 0) {
      ka = pos_next<MESH>(g, ka);
      load_raw<MESH>(g, xc, xb, own, ka, pre);
    }
    // ---- 6. Riemann problems on the lower x1-face and x2-face in plane p.
    // EDGES (PPM, and PLM on the 4-wave tiles): every thread reconstructs its own cell along x1 and x2 once;
    // the left edge is its own face's right state, the right edge goes to the
    // next thread through the slots that the face's results take afterwards.
    // Two more barriers a plane, for a quarter of the loop's instructions
    // (6171 -> 4682): 200x150x131 RK3+PPM+HLLE 2.81 -> 2.36 ms per chained step,
    // 512^3 blast 81.5 -> 76.8 ms.  With PLM a slope is cheap, and it pays less:
    // 1024 batched blocks, where the other workgroup of the CU fills the barriers,
    // 3.70 -> 3.61 ms; on the 8-wave tile 256^3 takes 3.03 ms either way and 512
    // blocks of 32^3 as one mesh 3.59 ms, or 3.51 with edges through LDS.
    constexpr bool EDGES = RECON >= 2 || (RECON == 1 && !CHAR && NT != TileU::NT);
    const int row = (ty + LA) * PW + tx + LA;  // own cell in the primitive plane
    // x-frame order: rho, v1, v2, v3, P, B2, B3; y-frame order: rho, v2, v3, v1, P, B3, B1
    constexpr int mapx[7] = {0, 1, 2, 3, 4, 6, 7}, mapy[7] = {0, 2, 3, 1, 4, 7, 5};
    constexpr int slotx[7] = {X_FX, X_FX + 1, X_FX + 2, X_FX + 3, X_FX + 4, X_E3X, X_WX};
    constexpr int sloty[7] = {X_FY, X_FY + 1, X_FY + 2, X_FY + 3, X_FY + 4, X_E3Y, X_WY};
    double xr[7], yr[7];  // right states of the own faces
    if constexpr (EDGES) {
      double hi[7];
      own_edges<RECON, LONE>(sp, PL, row, 1, mapx, xr, hi);
#pragma unroll
      for (int v = 0; v < 7; ++v) sx[slotx[v] * NT + tid] = hi[v];
      own_edges<RECON, LONE>(sp, PL, row, PW, mapy, yr, hi);
#pragma unroll
      for (int v = 0; v < 7; ++v) sx[sloty[v] * NT + tid] = hi[v];
      __syncthreads();
    }
    double e2x = 0.0, wx = 0.5, e1y = 0.0, wy = 0.5, e3x = 0.0, e3y = 0.0;
    FaceFlux fx{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (tx >= 1) {
      double ql[7];
      if constexpr (EDGES) {
#pragma unroll
        for (int v = 0; v < 7; ++v) ql[v] = sx[slotx[v] * NT + tid - 1];
      } else {
        face_states<RECON, CHAR>(sp, PL, row, 1, mapx, 5, sa.gas.gamma, ql, xr);
      }
      int hit = 0;
      riemann<RS, FL>(ql, xr, bnq[0][0], sa.gas, sa.ct_eps, sa.fl, hit, fx, wx);
      if (FL && zface && p < kend) seen += hit;
      if (MF && act && p >= k0 && p < kend) put(face_plane<MESH>(g, bp.fm, 0, w0), own.f, fx.rho);
      // x1-face E3 = -F(B2), E2 = +F(B3)
      e3x = -fx.bt1;
      e2x = fx.bt2;
    }
    double yl[7];
    if constexpr (EDGES) {
      if (ty >= 1) {
#pragma unroll
        for (int v = 0; v < 7; ++v) yl[v] = sx[sloty[v] * NT + tid - BX];
      }
      __syncthreads();  // every edge read: the slots take the results
    }
    sx[(X_FX + 0) * NT + tid] = fx.rho;
    sx[(X_FX + 1) * NT + tid] = fx.mn;   // M1
    sx[(X_FX + 2) * NT + tid] = fx.mt1;  // M2
    sx[(X_FX + 3) * NT + tid] = fx.mt2;  // M3
    sx[(X_FX + 4) * NT + tid] = fx.e;
    sx[X_E3X * NT + tid] = e3x;
    sx[X_WX * NT + tid] = wx;
    if (PF == 1) {
      ka = pos_next<MESH>(g, ka);
      load_raw<MESH>(g, xc, xb, own, ka, pre);
    }
    if (ty >= 1) {
      if constexpr (!EDGES) face_states<RECON, CHAR>(sp, PL, row, PW, mapy, 6, sa.gas.gamma, yl, yr);
      FaceFlux fy;
      int hit = 0;
      riemann<RS, FL>(yl, yr, bnq[0][1], sa.gas, sa.ct_eps, sa.fl, hit, fy, wy);
      if (FL && zface && p < kend) seen += hit;
      if (MF && act && p >= k0 && p < kend) put(face_plane<MESH>(g, bp.fm, 1, w0), own.f, fy.rho);
      sx[(X_FY + 0) * NT + tid] = fy.rho;
      sx[(X_FY + 1) * NT + tid] = fy.mt2;  // M1
      sx[(X_FY + 2) * NT + tid] = fy.mn;   // M2
      sx[(X_FY + 3) * NT + tid] = fy.mt1;  // M3
      sx[(X_FY + 4) * NT + tid] = fy.e;
      // x2-face E1 = -F(B3), E3 = +F(B1)
      e1y = -fy.bt1;
      e3y = fy.bt2;
    }
    sx[X_E3Y * NT + tid] = e3y;
    sx[X_WY * NT + tid] = wy;
    if (PF == 2) {
      ka = pos_next<MESH>(g, ka);
      load_raw<MESH>(g, xc, xb, own, ka, pre);
    }
    // the stored terms of this iteration's output (U^n, and the stage input
    // where g0 != 0): cell p-1 (5 values), B1, B2 at p-1, B3 at p.  Read by
    // every thread, without a branch, so that nothing waits for them before
    // they are used, after the corner EMFs (planes clamped into the segment).
    const bool out_cell = act && zface && p - 1 >= k0;
    double un[8], xg[8];
    if constexpr (!SAME) {
      const Pos first = MESH ? pos_at<MESH>(g, k0) : Pos{k0, 0};
      const Pos qc = MESH == 0 ? Pos{max(p - 1, k0), 0} : p > k0 ? kr1 : first;
      const Pos qf = MESH == 0 ? Pos{min(max(p, k0), kend - 1), 0} : p < k0 ? first : (p < kend ? kr : kr1);
      const Col c = here(own);
#pragma unroll
      for (int v = 0; v < 5; ++v) un[v] = at(cell_plane<MESH>(g, unc, v, qc), c.c);
#pragma unroll
      for (int d = 0; d < 3; ++d) un[5 + d] = at(face_plane<MESH>(g, unb, d, d < 2 ? qc : qf), c.f);
      if (sa.cf.g0 != 0.0) {
#pragma unroll
        for (int v = 0; v < 5; ++v) xg[v] = at(cell_plane<MESH>(g, xc, v, qc), c.c);
#pragma unroll
        for (int d = 0; d < 3; ++d) xg[5 + d] = at(face_plane<MESH>(g, xb, d, d < 2 ? qc : qf), c.f);
      } else {
#pragma unroll
        for (int v = 0; v < 8; ++v) xg[v] = 0.0;
      }
    }
    __syncthreads();

    // ---- 7. corner EMFs of the own edges and the conserved update
    const int tW = tid - 1, tS = tid - BX, tSW = tid - BX - 1, tE = tid + 1, tN = tid + BX;
    double c1 = 0.0, c2 = 0.0, c3 = 0.0;
    if (tx >= 1 && ty >= 1 && p >= k0 && p < kend) {
      // E3 at (i-1/2, j-1/2, p): a = x1, b = x2
      c3 = corner_emf(sx[X_E3X * NT + tid], sx[X_E3X * NT + tS], sx[X_E3Y * NT + tid], sx[X_E3Y * NT + tW],
                      sx[X_E3C * NT + tid], sx[X_E3C * NT + tW], sx[X_E3C * NT + tS], sx[X_E3C * NT + tSW], wx,
                      sx[X_WX * NT + tS], wy, sx[X_WY * NT + tW]);
    }
    if (ty >= 1 && zface) {
      // E1 at (i, j-1/2, p-1/2): a = x2, b = x3
      double wyp = wy_prev;
      if constexpr (!WY_REG) wyp = sx[X_WYP * NT + tid];
      c1 = corner_emf(e1y, sx[X_E1YP * NT + tid], sx[X_E1Z * NT + tid], sx[X_E1Z * NT + tS],
                      sx[X_E1C * NT + tid], sx[X_E1C * NT + tS], sx[X_E1CP * NT + tid], sx[X_E1CP * NT + tS], wy, wyp,
                      sx[X_WZ * NT + tid], sx[X_WZ * NT + tS]);
    }
    if (tx >= 1 && zface) {
      // E2 at (i-1/2, j, p-1/2): a = x3, b = x1
      c2 = corner_emf(sx[X_E2Z * NT + tid], sx[X_E2Z * NT + tW], e2x, sx[X_E2XP * NT + tid],
                      sx[X_E2C * NT + tid], sx[X_E2CP * NT + tid], sx[X_E2C * NT + tW], sx[X_E2CP * NT + tW],
                      sx[X_WZ * NT + tid], sx[X_WZ * NT + tW], wx, sx[X_WXP * NT + tid]);
    }
    sc[0 * NT + tid] = c1;
    sc[1 * NT + tid] = c2;
    sc[2 * NT + tid] = c3;

    double acc[7];
    if (act && zface) {
      // flux divergence of plane p (x1, x2) and the x3 flux through p-1/2
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const double dfx = sx[(X_FX + v) * NT + tE] - sx[(X_FX + v) * NT + tid];
        const double dfy = sx[(X_FY + v) * NT + tN] - sx[(X_FY + v) * NT + tid];
        acc[v] = -(dfx * i1 + dfy * i2) + fz_cons[v] * i3;
        acc_prev[v] -= fz_cons[v] * i3;
      }
      // g1 U^n + g0 X; for the first stage from the carried raw values of cell
      // p-1 and the lower B3 of plane p (its look-ahead load)
      double pw[8];
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const double u = SAME ? (v < 7 ? ucar[v] : bnq[0][2]) : un[v], x = SAME ? u : xg[v];
        pw[v] = sa.cf.g1 * u;
        if (sa.cf.g0 != 0.0) pw[v] += sa.cf.g0 * x;
      }
      if (out_cell) {
#pragma unroll
        for (int v = 0; v < 5; ++v) put(cell_plane<MESH>(g, oc, v, w1), own.c, pw[v] + bdt * acc_prev[v]);
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) acc_prev[v] = acc[v];
      // the face fields of this plane are updated after the next barrier
      pwb[0] = pw[5];
      pwb[1] = pw[6];
      pwb[2] = pw[7];
    }
    if (SAME) {
#pragma unroll
      for (int v = 0; v < 7; ++v) ucar[v] = unext[v];
    }

    // ---- 9. carry this plane's face EMFs / weights / cell EMFs upward
#pragma unroll
    for (int o = 0; o < NBQ - 1; ++o) {
      bnq[o][0] = bnq[o + 1][0];
      bnq[o][1] = bnq[o + 1][1];
      bnq[o][2] = bnq[o + 1][2];
    }
    sx[X_E2XP * NT + tid] = e2x;
    sx[X_WXP * NT + tid] = wx;
    sx[X_E1YP * NT + tid] = e1y;
    if constexpr (WY_REG) wy_prev = wy;
    else sx[X_WYP * NT + tid] = wy;
    kr2 = kr1;
    kr1 = kr;
    kr = pos_next<MESH>(g, kr);
  }
  __syncthreads();
  if (act && kend >= k0)
    face_update<MESH>(g, sc, tid, BX, NT, own.f, kend, MESH ? kr1 : Pos{kend, 0},
                      MESH ? kr2 : Pos{kend - 1, 0}, k0, kend, i1, i2, i3, bdt, pwb, acc_prev, ob);
  if ((seen & kBad) && act) atomicAdd(sa.bad, 1);
  if (FL && (seen & ~kBad) && act) add_floor_count(sa.bad, (unsigned long long)(seen & ~kBad));
}

// Uniform blocks: one workgroup per (tile, x3 segment, block), XCD-aware:
// consecutive logical tiles land on the same XCD so that halo overlap hits its
// L2.
// LONE (PPM on the 4-wave tile, launches with no more workgroups than CUs): a
// wave has its SIMD to itself, 512 registers and nobody to fill its waits, so
// PPM's limiters run without branches.  64x32x32 stage 56 -> 48 us; with two waves
// per SIMD the branches win (256^3: 0.79x without).
template <int RECON, int RS, class T, bool FL, int MESH, bool MF, bool SAME = false, bool CHAR = false, bool LONE = false>
__global__ void __launch_bounds__(T::NT) __attribute__((amdgpu_waves_per_eu(LONE ? 1 : 2)))
k_stage_fused(UniformArgs a) {
  using S = Smem<RECON, T>;
  __shared__ double sp[8 * S::PL];      // primitives of the current plane
  __shared__ double sx[exchange_slots<RECON>() * T::NT];  // exchange slots
  __shared__ double sc[3 * T::NT];      // corner EMFs E1, E2, E3 of the current (half-)plane
  const int64_t bid = blockIdx.x;
  const int64_t logical = (bid % 8) * a.per_xcd + bid / 8;
  if (logical >= a.total) return;
  const Geo& g = a.g;
  int64_t r = logical;
  const int tile_x = (int)(r % a.ntx); r /= a.ntx;
  const int tile_y = (int)(r % a.nty); r /= a.nty;
  const int seg = (int)(r % a.nseg); r /= a.nseg;
  const int64_t blk = r;
  BlockPtrs bp{a.xc + blk * g.cblock, a.xb + blk * g.fblock, a.unc + blk * g.cblock,
               a.unb + blk * g.fblock, a.oc + blk * g.cblock, a.ob + blk * g.fblock,
               MF ? a.fm + blk * 3 * g.fvar : nullptr};
  const int k0 = g.ng + seg * a.kz;
  const int kend = min(k0 + a.kz, g.ng + (MESH == 2 ? g.mesh[2] * g.n3 : g.n3));
  stage_tile<RECON, RS, T, FL, MESH, MF, SAME, CHAR, LONE>(g, bp, a.sa, tile_x, tile_y, k0, kend, sp, sx, sc);
}

// Batched blocks of uneven sizes: a persistent grid whose workgroups pull
// (block, tile, x3 segment) items from a device queue until it is drained.
// MESH 1: the blocks tile one domain and read their exchanged ghost entries.
template <int RECON, int RS, class T, bool FL, bool MF, bool SAME = false, int MESH = 0>
__global__ void __launch_bounds__(T::NT) __attribute__((amdgpu_waves_per_eu(2))) k_stage_batch(BatchArgs a) {
  using S = Smem<RECON, T>;
  __shared__ double sp[8 * S::PL];
  __shared__ double sx[exchange_slots<RECON>() * T::NT];
  __shared__ double sc[3 * T::NT];
  __shared__ int s_item;
  for (;;) {
    if (threadIdx.x == 0) s_item = (int)atomicAdd(a.queue, 1u);
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(s_item);
    __syncthreads();
    if (it >= a.nitems) {
      // the last workgroup to find the queue empty clears it for the next launch
      if (threadIdx.x == 0 && atomicAdd(a.queue + 1, 1u) == gridDim.x - 1) {
        atomicExch(a.queue, 0u);
        atomicExch(a.queue + 1, 0u);
      }
      break;
    }
    const WorkItem w = a.items[it];
    const BatchDesc& d = a.desc[w.block];
    BlockPtrs bp{a.xc + d.coff, a.xb + d.foff, a.unc + d.coff, a.unb + d.foff, a.oc + d.coff, a.ob + d.foff,
                 MF ? a.fm + d.foff : nullptr};
    stage_tile<RECON, RS, T, FL, MESH, MF, SAME>(d.g, bp, a.sa, w.tile_x, w.tile_y, w.k0, w.kend, sp, sx, sc);
    __syncthreads();
  }
}

// MESH: how neighbours are read; MF: the face mass fluxes are stored for
// passive scalars.  Compile-time switches,
// so that the plain periodic-block kernels keep their code.
template <int RECON, int RS, class T, int MESH, bool MF>
hipError_t uniform_fl(const UniformArgs& fa, hipStream_t s) {
  const dim3 grid((unsigned)(8 * fa.per_xcd)), wg(T::NT);
  if constexpr (RECON == 0) {
    // the first stage of a scheme reads U^n as its input: carry its raw cells
    if (fa.xc == fa.unc && fa.xb == fa.unb) {
      if (fa.sa.fl.on())
        hipLaunchKernelGGL((k_stage_fused<RECON, RS, T, true, MESH, MF, true>), grid, wg, 0, s, fa);
      else
        hipLaunchKernelGGL((k_stage_fused<RECON, RS, T, false, MESH, MF, true>), grid, wg, 0, s, fa);
      return hipGetLastError();
    }
  }
  if constexpr (RECON == 2 && T::NT <= 256 && MESH == 0 && !MF) {
    if (fa.lone) {
      if (fa.sa.fl.on())
        hipLaunchKernelGGL((k_stage_fused<RECON, RS, T, true, 0, false, false, false, true>), grid, wg, 0, s, fa);
      else
        hipLaunchKernelGGL((k_stage_fused<RECON, RS, T, false, 0, false, false, false, true>), grid, wg, 0, s, fa);
      return hipGetLastError();
    }
  }
  if (fa.sa.fl.on()) hipLaunchKernelGGL((k_stage_fused<RECON, RS, T, true, MESH, MF>), grid, wg, 0, s, fa);
  else hipLaunchKernelGGL((k_stage_fused<RECON, RS, T, false, MESH, MF>), grid, wg, 0, s, fa);
  return hipGetLastError();
}

template <int RECON, class T, int MESH, bool MF>
hipError_t uniform_rs(int rs, const UniformArgs& fa, hipStream_t s) {
  if (rs == 1) return uniform_fl<RECON, 1, T, MESH, MF>(fa, s);
  if (rs == 2) return uniform_fl<RECON, 2, T, MESH, MF>(fa, s);
  return uniform_fl<RECON, 0, T, MESH, MF>(fa, s);
}

template <int RS, class T>
hipError_t charac_fl(const UniformArgs& fa, hipStream_t s) {
  const dim3 grid((unsigned)(8 * fa.per_xcd)), wg(T::NT);
  if (fa.sa.fl.on()) hipLaunchKernelGGL((k_stage_fused<1, RS, T, true, 0, false, false, true>), grid, wg, 0, s, fa);
  else hipLaunchKernelGGL((k_stage_fused<1, RS, T, false, 0, false, false, true>), grid, wg, 0, s, fa);
  return hipGetLastError();
}

template <class T, int RECON, int RS, bool MF, bool SAME>
hipError_t batch_fl(const BatchArgs& ba, int grid, hipStream_t s) {
  if (ba.sa.fl.on())
    hipLaunchKernelGGL((k_stage_batch<RECON, RS, T, true, MF, SAME>), dim3(grid), dim3(T::NT), 0, s, ba);
  else
    hipLaunchKernelGGL((k_stage_batch<RECON, RS, T, false, MF, SAME>), dim3(grid), dim3(T::NT), 0, s, ba);
  return hipGetLastError();
}

template <class T, int RECON, int RS, bool SAME>
hipError_t batch_kind(const BatchArgs& ba, int grid, hipStream_t s, bool mesh) {
  if (mesh) {  // blocks that tile one domain (no floors, no mass fluxes)
    hipLaunchKernelGGL((k_stage_batch<RECON, RS, T, false, false, SAME, 1>), dim3(grid), dim3(T::NT), 0, s, ba);
    return hipGetLastError();
  }
  return ba.fm ? batch_fl<T, RECON, RS, true, SAME>(ba, grid, s) : batch_fl<T, RECON, RS, false, SAME>(ba, grid, s);
}

}  // namespace

template <int RECON, class T>
hipError_t launch_uniform(int rs, const UniformArgs& fa, hipStream_t s) {
  if (fa.fm) return fa.g.mesh[0] ? uniform_rs<RECON, T, 1, true>(rs, fa, s) : uniform_rs<RECON, T, 0, true>(rs, fa, s);
  if (fa.domain) return uniform_rs<RECON, T, 2, false>(rs, fa, s);
  return fa.g.mesh[0] ? uniform_rs<RECON, T, 1, false>(rs, fa, s) : uniform_rs<RECON, T, 0, false>(rs, fa, s);
}

template <class T>
hipError_t launch_charac(int rs, const UniformArgs& fa, hipStream_t s) {
  if (rs == 1) return charac_fl<1, T>(fa, s);
  if (rs == 2) return charac_fl<2, T>(fa, s);
  return charac_fl<0, T>(fa, s);
}

template <class T, int RECON>
hipError_t launch_batch(int rs, const BatchArgs& ba, int grid, hipStream_t s, bool mesh) {
  // the first stage of a scheme reads U^n as its input: carry its raw cells
  if constexpr (RECON == 0) {
    if (ba.xc == ba.unc && ba.xb == ba.unb)
      return rs == 1 ? batch_kind<T, RECON, 1, true>(ba, grid, s, mesh) : batch_kind<T, RECON, 0, true>(ba, grid, s, mesh);
  }
  return rs == 1 ? batch_kind<T, RECON, 1, false>(ba, grid, s, mesh) : batch_kind<T, RECON, 0, false>(ba, grid, s, mesh);
}

}  // namespace athmhd
