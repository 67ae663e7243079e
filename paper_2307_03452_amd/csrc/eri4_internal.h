// eri4_internal.h -- constants and parameter blocks shared by the host side and
// the gfx950 kernels of liberi4.  Not part of the public ABI.
#pragma once
#include <stdint.h>

namespace eri4 {

// Largest l per shell the index tables are sized for, and the largest total
// Hermite order L = la+lb+lc+ld (Boys orders 0..L).
constexpr int kTableLMax = 7;
constexpr int kMaxL = 4 * kTableLMax;  // 28

// Boys-function interpolation grid (Sec. 2, eq. (boys)): F_k(T_i) at
// T_i = i * kBoysH for i < kBoysRows, k < kBoysCols, used as a Taylor expansion
// F_m(T_i + d) = sum_j F_{m+j}(T_i) (-d)^j / j!, j <= kBoysJ.  kBoysH is a
// power of two so that T_i and d = T - T_i are exact.  Beyond kBoysTMax the
// asymptotic form F_m(T) = (2m-1)!! / 2^(m+1) sqrt(pi / T^(2m+1)) is used; its
// neglected part is below 1e-20 relative there for m <= kMaxL.
constexpr double kBoysH = 1.0 / 32.0;
constexpr double kBoysInvH = 32.0;
constexpr int kBoysJ = 7;
constexpr double kBoysTMax = 120.0;
constexpr int kBoysRows = 120 * 32 + 2;
constexpr int kBoysCols = kMaxL + kBoysJ + 2;  // 37
// Row kBoysRows of the uploaded table holds the asymptotic coefficients
// (2m-1)!! sqrt(pi) / 2^(m+1) = Gamma(m+1/2)/2, so F_m(T) = c_m / (T^m sqrt(T)).
constexpr int kBoysAsymRow = kBoysRows;

// Strides of the R box used for total order L: offset(t,u,v) = t*S2 + u*S1 + v.
// S1 is the even number >= L+1 so that entries of one total order, which sit
// S1-1 doubles apart, spread over the LDS banks; S2 = S1*(L+1).
__host__ __device__ constexpr int box_s1(int L) { return ((L + 1) & 1) ? L + 2 : L + 1; }
__host__ __device__ constexpr int box_s2(int L) { return box_s1(L) * (L + 1); }
// Odd row length >= n for the 1-d E tables (rows of one table read by the
// lanes of a wave then fall in different LDS banks).
__host__ __device__ constexpr int odd_row(int n) { return n | 1; }

// Pyramidal number: Hermite functions with total order <= n.
__host__ __device__ constexpr int nherm(int n) { return (n + 1) * (n + 2) * (n + 3) / 6; }
__host__ __device__ constexpr int ncart(int l) { return (l + 1) * (l + 2) / 2; }

// Two LDS layouts of the Hermite integrals [r] with t+u+v <= L:
//   box  (L+1)^3 cells:   offset = t*S2 + u*S1 + v,        S2 = S1*(L+1)
//   slab t-slabs of (L+1-t) rows: offset = slab_base(t) + u*S1 + v
// The box makes the index p+q of eq. (pq) an address sum; the slab needs one
// more term (slab_base of the summed t) but about half the space, which is
// what lets L = 26, 28 fit in LDS.
__host__ __device__ constexpr int slab_base(int t, int L, int S1) { return S1 * (t * (2 * L + 3 - t) / 2); }
__host__ __device__ constexpr int r_cells(bool slab, int L) {
  return slab ? box_s1(L) * (L + 1) * (L + 2) / 2 : (L + 1) * box_s2(L);
}
__host__ __device__ constexpr int r_offset(bool slab, int L, int t, int u, int v) {
  return (slab ? slab_base(t, L, box_s1(L)) : t * box_s2(L)) + u * box_s1(L) + v;
}

// Hermite recursion tables (box layout): for each L in 0..kMaxL, the nherm(L) triples (t,u,v) with t+u+v <= L ordered by total
// order, each as two 32-bit words
//   x: offset of (t,u,v) | offset of (t,u,v) - 1_i << 16
//   y: offset of (t,u,v) - 2*1_i (or of -1_i when r_i < 2) | i << 16 | r_i << 18
// where i is the axis eq. (md1) raises to reach (t,u,v) (the last non-zero of
// t, u, v).  The first entry of each table is (0,0,0) with all fields 0.

// Solid-harmonic coefficient table (make_solid_table): per (l, m) one entry of
// kSolidEntry doubles, the count and up to kSolidTerms (Cartesian index,
// coefficient) pairs; kSolidRows = 2 * kTableLMax + 1 rows per l.
constexpr int kSolidTerms = 16;
constexpr int kSolidEntry = 1 + 2 * kSolidTerms;
constexpr int kSolidRows = 2 * kTableLMax + 1;
// Hermite functions of one side (total order <= 2 * kTableLMax), padded to 4,
// and the doubles of that side's three 1-d E tables.
constexpr int kMaxHerm = (nherm(2 * kTableLMax) + 3) & ~3;
constexpr int kMaxEtab = 3 * ((kTableLMax + 1) * (kTableLMax + 1) + 1) * odd_row(2 * kTableLMax + 2);

// Units of 16 rows (bra) or columns (ket) of the H matrices of one pair-list
// entry: bra rows are padded to 64, a whole tile of any height.
__host__ __device__ constexpr int solid_pair_units(int l1, int l2, bool ket) {
  return ket ? ((2 * l1 + 1) * (2 * l2 + 1) + 15) / 16 : 4 * (((2 * l1 + 1) * (2 * l2 + 1) + 63) / 64);
}

// Dynamic LDS (bytes) of the H-matrix builder for shells l1, l2 with nk4
// Hermite indices: one chunk of P[2 l1 + 1][ncart(l2)][16], the three 1-d E
// tables, the Hermite index table.
__host__ __device__ constexpr int solid_h_lds(int l1, int l2, int nk4) {
  return (2 * l1 + 1) * ncart(l2) * 16 * 8 + 3 * ((l1 + 1) * (l2 + 1) + 1) * odd_row(l1 + l2 + 2) * 8 + nk4 * 8;
}

// Layout of W (one value per [r]) in the Cartesian integral kernels
// (eri4_tile.h): nherm(L) values, rows of t = 0..L-s for each (u, v), the rows in order of
// increasing s = u + v and then u.  Row (u, v) starts at tile_r_base(L, s) +
// u (L + 1 - s), so that the row of a sum of two (u, v) follows from the sums
// of their s and u.
__host__ __device__ constexpr int tile_r_base(int L, int s) { return s * (s + 1) * (3 * (L + 1) - 2 * (s - 1)) / 6; }
// (u, v) with u + v <= n.
__host__ __device__ constexpr int nuv(int n) { return (n + 1) * (n + 2) / 2; }
// Layout of F (eri4_tile.h) of a row group with u + v <= m0 in the bra: rows
// (u, v) as in [r], s = u + v <= m0 + Lk, of t = 0..min(Lk, m0 + Lk - s).  With s
// = m0 + Lk + 1 and u = 0: the number of values.
__host__ __device__ constexpr int tile_f_row(int m0, int Lk, int s, int u) {
  return s <= m0 ? (Lk + 1) * (nuv(s - 1) + u)
                 : (Lk + 1) * nuv(m0) + tile_r_base(m0 + Lk, s) - tile_r_base(m0 + Lk, m0 + 1) + u * (m0 + Lk + 1 - s);
}
// Steps of 64 of the per-axis tables (eri4_tile.h): rows 0..15, and from 16 to L.
__host__ __device__ constexpr int h_steps(int L) { return L < 16 ? (L >> 2) + 1 : (L >> 2) + 3; }
// Row blocks moved to the LDS tile at a time: with five or more column blocks
// per wave over eight waves (lc + ld >= 13) 32 rows of [ab|q] do not fit.
__host__ __device__ constexpr int tile_xb(int cw, int nc) { return cw == 8 && nc >= 5 ? 1 : 2; }
// Units whose rows it holds: both of a tile where they fit (lc + ld <= 9).
__host__ __device__ constexpr int tile_xu(int cw, int nc) { return cw == 4 && nc <= 4 ? 2 : 1; }

// LDS of one compute unit (gfx950).
constexpr int kMaxLdsBytes = 160 * 1024;

// One-wave kernel for classes whose shells all have l <= kSmallLMax
// (eri4_small.hip): its largest dynamic LDS.
constexpr int kSmallLMax = 3;
constexpr int kSmallLdsMax = 64 * 1024;

// One workgroup computes a tile of 16 or 32 bra rows (ab) of one quartet.
constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;
constexpr int kBoxLMax = 24;  // box layout only up to here
constexpr int kDenseSolid = 0, kDenseExch = 1, kDenseCart = 2;  // what a tile of eri4_dense.h computes
constexpr int kWaveL = 8;  // total orders whose recursion one wave runs (eri4_dense.h)
constexpr int kMaxC1 = 6;  // first-transform column blocks per wave (L_ket <= 14)
// Layouts of [r] that a tile choice may name: kLayBox, kLaySlab, and kLayBox2, the box
// where LDS had room for two of them (total order up to kBox2LMax): the recursion
// needs one, so that it is the box layout with that condition.
constexpr int kLayBox = 0, kLaySlab = 1, kLayBox2 = 2;
constexpr int kBox2LMax = 19;

// Everything the fused kernel needs to know about one class (la lb|lc ld).
struct ClassParams {
  int la, lb, lc, ld;
  int na, nb, nc, nd;
  int nab, ncd;
  int Lb, Lk, L;
  int np, nq;      // Hermite functions of the bra and the ket
  int np4, nq4;    // padded to a multiple of 4 (MFMA K step)
  int nqb;         // 16-wide column blocks of [ab|q]
  int ncdb;        // 16-wide column blocks of (ab|cd)
  int nrt;         // row tiles per quartet
  int S1, S2;      // strides of the R box: u -> S1, t -> S2 (box_s1, box_s2)
  int tbrow, tkrow;    // 1-d E table row lengths (Lb+2, Lk+2); last entry is 0
  int tbaxis, tkaxis;  // doubles per axis of the bra / ket tables (incl. zero row)
  int xs;              // row stride (doubles) of the [ab|q] tile in LDS
  int kmax;
  int rtab_off;        // first entry (uint2 units) of the recursion table for this layout and L
  int slab;            // R layout: 0 box, 1 slab
  int rb;              // 16-row blocks per tile (1, 2, or 4 with a box layout)
  int lay;             // kLayBox, kLaySlab or kLayBox2 (slab == (lay == kLaySlab))
  // LDS layout (byte offsets)
  int o_union;   // phase 1: R box then bra tables; phase 2: [ab|q] tile then ket tables
  int o_brae;    // bra tables (phase 1)
  int o_kete;    // ket tables (phase 2)
  int o_ptab, o_qtab, o_base, o_shell;
  int o_rowt, o_rs, o_rv, o_zt, o_h;        // recursion of the solid and exchange kernels (eri4_dense.h)
  int ntask, o_uv, o_task;                  // and its tables (make_tile_tables), in words
  int lds_bytes;
};

// The same for the Cartesian integral kernels (eri4_tile.h).  Table offsets
// o_uv..o_klist are in words of the tile tables (make_tile_tables).
struct TileParams {
  int la, lb, lc, ld;
  int nab, ncd;
  int Lb, Lk, L;
  int nq;              // Hermite functions of the ket
  int nqb;             // 16-wide column blocks of [ab|q]
  int kb, kk;          // (u, v) of the bra and the ket: nuv(Lb), nuv(Lk)
  int nr, nzt;         // values of W and of zt (eri4_tile.h)
  int nks;             // steps of G, at most
  int tbrow, tkrow;    // 1-d E table row lengths
  int tbaxis, tkaxis;  // doubles per axis of the bra / ket tables (incl. zero row)
  int xs;              // row stride (doubles) of the [ab|q] tile in LDS
  int kmax;
  int shape;           // kernel shape (tile_shape)
  int nunits, ntiles;  // bra units, and tiles of them
  int nkblk;           // 16-wide column blocks of (ab|cd), grouped by (cx, dx)
  int ntask;           // wave tasks of W
  int o_uv, o_qcol, o_task;
  int o_bunit, o_brows, o_kunit, o_kcols, o_klist;
  // LDS layout (byte offsets)
  int o_row1;   // row tables of the second unit of a tile
  int o_union;  // two buffers of buf bytes (bra tables; W), F, then zt, the per-axis tables and G; or the [ab|q]
                // tile and, past F too, the ket tables
  int o_f, o_zt, o_h, o_g, o_kete, buf;
  int fsize;  // doubles of F per unit, at most
  int lds_bytes;
};

// LDS of the Cartesian integral kernels: the small tables sit at fixed places,
// sized for the largest class (scalar registers for their offsets would spill).
constexpr int kTileShell = 0;                                             // centres, exponents, coefficients, lengths
constexpr int kTileBase = kTileShell + (12 + 8 * 16) * 8 + 16;            // [0]^(m) (32), ket pair (16), output rows
constexpr int kTileRowfSize = ((kMaxL + 1) * (kMaxL + 1) * 2 + 15) / 16 * 16;
constexpr int kTileRfSize = (nuv(kMaxL) * 4 + 15) / 16 * 16;
constexpr int kTileRowt = kTileBase + 80 * 8;              // row starts of W by (u, v)
constexpr int kTileRowf = kTileRowt + kTileRowfSize;       // and of F
constexpr int kTileRf = kTileRowf + kTileRowfSize;         // rows of F in order
constexpr int kTileRs = kTileRf + kTileRfSize;             // rows of W in order
constexpr int kTileRv = kTileRs + kTileRfSize;             // their u, v
constexpr int kTileBtab = kTileRv + (nuv(kMaxL) * 2 + 15) / 16 * 16;  // (u, v) of the bra
constexpr int kTileKtab = kTileBtab + (nuv(2 * kTableLMax) + 1) * 16;  // (u, v) of the ket
constexpr int kTileKcol = kTileKtab + (nuv(2 * kTableLMax) + 1) * 16;  // columns of the ket

// Kernel shapes by the number of [ab|q] column blocks: waves per row of column
// blocks, bra row blocks per unit, column blocks per wave, limits of a unit
// (kTileUnitLimits).  Four waves per row (two units of bra rows per tile) where
// eight would leave more of them without a column block; units of two row blocks
// where three would need more than 96 accumulator registers (four blocks of four
// columns, 128 registers, spilled 350 and saved one unit of 34 for (ii|)).
struct TileShapeInfo { int cw, rb, nc, lim; };
constexpr TileShapeInfo kTileShapes[9] = {{4, 3, 1, 0}, {4, 3, 2, 0}, {4, 3, 3, 0}, {4, 3, 4, 1}, {4, 2, 5, 2},
                                          {8, 3, 3, 3}, {8, 3, 4, 3}, {8, 2, 5, 4}, {8, 2, 6, 4}};
// What a unit of bra rows may hold, for kets up to order Lk: blocks, and doubles of
// F of its groups together (LDS).
struct TileUnitLimits { int Lk, rb, fmax; };
constexpr int kTileLimits = 5;
constexpr TileUnitLimits kTileUnitLimits[kTileLimits] = {{8, 3, 3200}, {9, 3, 3200}, {10, 2, 3600}, {12, 3, 5200},
                                                         {14, 2, 4400}};
constexpr int tile_shape(int nqb) {
  return nqb <= 16 ? (nqb + 3) / 4 - 1 : (nqb <= 20 ? 4 : (nqb + 7) / 8 + 2);
}

// Where the tables of the Cartesian integral kernels start (make_tile_tables),
// in words: per order n, and per shell pair (l1, l2) as bra or ket.
struct TileTableIndex {
  int uv;
  int qcol[2 * kTableLMax + 1], task[kMaxL + 1], ntask[kMaxL + 1];
  int chunk[2 * kTableLMax + 1], nchunk[2 * kTableLMax + 1];
  int item[2 * kTableLMax + 1], nitem[2 * kTableLMax + 1], dsize[2 * kTableLMax + 1], qpos[2 * kTableLMax + 1];
  struct Side {
    int nunits, nblocks, units, rows, list;
  } bra[kTileLimits][kTableLMax + 1][kTableLMax + 1], ket[kTableLMax + 1][kTableLMax + 1];
};

// The same for the kernels of eri4_quad.hip: of t, what does not concern LDS.
struct QuadParams {
  TileParams t;
  int fsize, fsize1;  // doubles of F of a wave's first and second group
  int nkunits;   // units of the ket
  int o_base, o_rowt, o_rs, o_rv, o_btab, o_ktab, o_kcol, o_orow;
  int o_kete, o_brae, o_h, o_zt, o_w, o_f;
  int lds_bytes;
};

// The same for the Coulomb (J-engine) kernels (eri4_coulomb.hip).
struct JParams {
  int la, lb, lc, ld;
  int nab, ncd;
  int Lb, Lk, L;
  int nq;              // Hermite functions of the ket
  int nzt;             // values of zt: nuv(L)
  int ntask;           // wave tasks of W and of [r]
  int nchunk, ncp, ncps;  // chunks of the bra's Hermite functions, the power of two above (>= 8) and its exponent
  int nitems;          // items of the ket's
  int tbrow, tbaxis;   // bra 1-d tables
  int kmax;
  int ds;              // doubles of dket per ket primitive pair
  int rsize, dsize;    // doubles of [r] (with kJPad before and after it) and of dket in LDS
  int o_uv, o_task, o_chunk, o_item, o_qpos;
  // LDS (byte offsets): fixed part (kJ..), dket, [r] (or parts of w), then W, zt
  // and the per-axis tables; or the bra tables, w and the folded w
  int o_d, o_r, o_w, o_zt, o_h, o_wp, o_wf;
  int lds_bytes;
};

constexpr int kJShell = 0;                                             // shells, lengths
constexpr int kJBase = kJShell + (12 + 8 * 16) * 8 + 16;               // [0]^(m)
constexpr int kJRowt = kJBase + 32 * 8;                                // row starts of W by (u, v)
constexpr int kJRs = kJRowt + kTileRowfSize;                           // rows of W in order
constexpr int kJRv = kJRs + kTileRfSize;                               // their u, v
constexpr int kJVrow = kJRv + (nuv(kMaxL) * 2 + 15) / 16 * 16;         // [r] by v
constexpr int kJItem = kJVrow + 32 * 4;                                // items of the ket
constexpr int kJEnd = kJItem + 64 * 8;
// Reads of [r] past its rows: at most 3 rows of S <= 29 and a few values.
constexpr int kJPad = 112;
// The Coulomb kernels of low orders (eri4_coulomb_low.hip): total orders up to kWaveL
// with at most kLowHerm Hermite functions on either side.
constexpr int kLowHerm = 84;  // l1 + l2 <= 6
constexpr int kLowAb = 100;   // (ff|: the most rows
constexpr int kLowWaves = 8;  // waves of a workgroup, at most
struct JLowParams {
  int la, lb, lc, ld;
  int nab, ncd, nb, nd;
  int Lb, Lk, L;
  int np, nq;
  int S1, S2;
  int tbrow, tbaxis, tkrow, tkaxis;
  int kmax, ds;
  int rtab_off, o_uv;
  // LDS (byte offsets): shells, Hermite tables and the recursion's table, then per wave
  // (wsize bytes from o_wave): [0]^(m), [r], dket, w, bra tables; and J (over [r])
  int o_ptab, o_qtab, o_entl, o_wave, wsize, o_r, o_d, o_w, o_e;
  int lds_bytes;  // of one wave; + wsize for each more
};

// Values of w, or of a density block, folded over the groups (x1, x2) of a shell
// pair: the (u, v) of each group.
__host__ __device__ constexpr int nfold(int l1, int l2) {
  int n = 0;
  for (int x1 = 0; x1 <= l1; ++x1)
    for (int x2 = 0; x2 <= l2; ++x2) n += nuv(l1 + l2 - x1 - x2);
  return n;
}

}  // namespace eri4
