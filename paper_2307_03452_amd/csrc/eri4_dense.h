// eri4_dense.h -- gfx950 device code of the solid-harmonic integrals, of the
// exchange contraction and of small classes of Cartesian integrals (FP64): one
// workgroup computes one tile of bra rows of one quartet by a dense first transform,
// [ab|q] += sum_p A_ab^p [p+q], whose operand [p+q] is read from [r] in LDS as the sum
// of two offsets.  (The rows of a solid harmonic mix all x exponents, and a tile of
// the exchange contraction holds all a of one b, so that the grouping of eri4_tile.h
// does not apply; of small classes it leaves groups of a few rows in blocks of 16, and
// a recursion for every two or three of them.)
#pragma once
#include "eri4_tile.h"

namespace eri4 {
namespace {

// First transform over one bra primitive pair for NR row blocks x NC column
// blocks of this wave (both fixed per wave):
//   acc[r][c] += sum_p E_ab[row block r][p] * box[off(p) + off(q in block c)]
// E_ab is the product of three bra-table entries.  The operands of a k step are
// read before the MFMAs of the step before it.
// gemm1_e runs the k steps kbeg..kend-1 (multiples of 4) only.
template <int NR, int NC, bool SLAB>
__device__ __forceinline__ void gemm1_e(typename Acc<false>::type (&acc)[NR][NC], const double* __restrict__ brae,
                                            const double* __restrict__ R, const int2* __restrict__ ptab,
                                            const int (&rowx)[NR], const int (&rowy)[NR], const int (&rowz)[NR],
                                            const int (&offq)[NC], const int (&tq)[NC], int kbeg, int kend, int L,
                                            int S1, int lane) {
  if (kbeg >= kend) return;
  const int g = lane >> 4;
  double ex[NR], ey[NR], ez[NR], b[NC];
  auto fetch = [&](int2 pt) {
    const int tp = pt.x & 0xff, up = (pt.x >> 8) & 0xff, vp = (pt.x >> 16) & 0xff;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      ex[r] = brae[rowx[r] + tp];
      ey[r] = brae[rowy[r] + up];
      ez[r] = brae[rowz[r] + vp];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)  // t of p+q selects the slab
      b[c] = R[(SLAB ? slab_base((pt.x >> 24) + tq[c], L, S1) : 0) + pt.y + offq[c]];
  };
  fetch(ptab[kbeg + g]);
  int2 pt = ptab[min(kbeg + 4, kend - 4) + g];
#pragma unroll 1
  for (int kk = kbeg; kk < kend; kk += 4) {
    double a[NR], bb[NC];
#pragma unroll
    for (int r = 0; r < NR; ++r) a[r] = ex[r] * ey[r] * ez[r];
#pragma unroll
    for (int c = 0; c < NC; ++c) bb[c] = b[c];
    fetch(pt);
    pt = ptab[min(kk + 8, kend - 4) + g];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[r][c] = mfma16<false>(a[r], bb[c], acc[r][c]);
  }
}

// Solid harmonics: the transform matrices H = (C_a x C_b) E of one
// primitive pair come from device memory (solid_h_kernel), stored in the
// operand order of the matrix cores: for row (or column) block u and k step s,
// 64 doubles, lane l holding H[16u + (l & 15)][4s + (l >> 4)].  A wave's load of
// one operand is one contiguous 512-byte read.

// First transform, A operand from H: acc[r][c] += sum_p H[row block r][p] [p|q].
// H points at this lane's element of row block 0, k step 0.  Its operands come
// from the last cache level or memory: four steps are requested while the four
// before them run (requested two steps ahead, the products waited for them);
// [p|q] is read one step ahead.
template <int NR, int NC, bool SLAB>
__device__ __forceinline__ void gemm1_h(typename Acc<false>::type (&acc)[NR][NC], const double* __restrict__ H,
                                        const double* __restrict__ R, const int2* __restrict__ ptab,
                                        const int (&offq)[NC], const int (&tq)[NC], int np4, int L, int S1,
                                        int lane) {
  constexpr int U = 4;
  const int g = lane >> 4;
  const int rs = np4 * 16;  // doubles per row block
  double a[U][NR], an[U][NR], b[NC];
  auto fetch_a = [&](double (&x)[U][NR], int kk) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < NR; ++r) x[u][r] = H[r * rs + min(kk + 4 * u, np4 - 4) * 16];
  };
  auto fetch_b = [&](int2 pt) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      b[c] = R[(SLAB ? slab_base((pt.x >> 24) + tq[c], L, S1) : 0) + pt.y + offq[c]];
  };
  fetch_a(a, 0);
  fetch_b(ptab[g]);
  int2 pt = ptab[min(4, np4 - 4) + g];
#pragma unroll 1
  for (int k0 = 0; k0 < np4; k0 += 4 * U) {
    fetch_a(an, k0 + 4 * U);
    asm volatile("" ::: "memory");  // keep the requests ahead of the products
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = k0 + 4 * u;
      if (kk < np4) {
        double bb[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) bb[c] = b[c];
        fetch_b(pt);
        pt = ptab[min(kk + 8, np4 - 4) + g];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int c = 0; c < NC; ++c) acc[r][c] = mfma16<false>(a[u][r], bb[c], acc[r][c]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < NR; ++r) a[u][r] = an[u][r];
  }
}

// Second transform for one group of NC output column blocks, B operand from
// H_cd (Hk: this lane's element of column block 0, k step 0), then the output
// write, as gemm2_group.  The operands of eight steps are requested while the eight
// before them run: requested one step ahead, a tile of (ii|ii) waited 75 000 of the
// 120 000 cycles of this transform
// (U; four of low orders).
template <int NR, int NC, int U>
__device__ __forceinline__ void gemm2_group_h(const ClassParams& cp, const double* __restrict__ X,
                                              const double* __restrict__ Hk, int cb0, int row0,
                                              double* __restrict__ outq, bool first, double unscale,
                                              int lane) {
  const int g = lane >> 4, n = lane & 15;
  const int cs = cp.nq4 * 16;  // doubles per column block
  typename Acc<false>::type acc[NR][NC];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[r][c] = acc_zero<false>();
  const int xs = cp.xs, nq4 = cp.nq4;
  double b[U][NC], bn[U][NC];
  auto fetch = [&](double (&x)[U][NC], int kk) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) x[u][c] = Hk[(cb0 + 8 * c) * cs + min(kk + 4 * u, nq4 - 4) * 16];
  };
  fetch(b, 0);
#pragma unroll 1
  for (int k0 = 0; k0 < nq4; k0 += 4 * U) {
    fetch(bn, k0 + 4 * U);
    asm volatile("" ::: "memory");  // keep the requests ahead of the products
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + 4 * u < nq4) {
        double a[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) a[r] = X[(r * 16 + n) * xs + k0 + 4 * u + g];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int r = 0; r < NR; ++r) acc[r][c] = mfma16<false>(a[r], b[u][c], acc[r][c]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) b[u][c] = bn[u][c];
  }
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int cd = (cb0 + 8 * c) * 16 + n;
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int ab = row0 + r * 16 + acc_row<false>(jj, g);
        if (ab < cp.nab && cd < cp.ncd) {
          double* o = outq + (int64_t)ab * cp.ncd + cd;
          const double v = acc[r][c][jj] * unscale;
          if (first)
            __builtin_nontemporal_store(v, o);
          else
            *o += v;
        }
      }
    }
}

// Exchange contraction: bra row order.  Padded row pr of a quartet is shell-b
// component pr / P and shell-a component pr % P, with P = 16 * ceil(na / 16)
// rows per b (components a >= na are padding).
__device__ __forceinline__ int exch_rows_per_b(const ClassParams& cp) { return 16 * ((cp.na + 15) / 16); }
__device__ __forceinline__ void exch_row(const ClassParams& cp, int pr, int& ia, int& ib) {
  const int P = exch_rows_per_b(cp);
  ib = pr / P;
  ia = pr - ib * P;
}

// y blocks of one ket pair: NR * ncc blocks of row block r = blk / ncc and column
// block cc = blk % ncc (c = 16 cc + lane % 16),
//   y[r][cc] += sum_q X[row block r][q] F^b[q][cc],  b the row block's shell-b component.
// Up to eight blocks of many k: 8 / blocks waves share the k of one (exch_split; of few
// steps, adding the parts took longer than the steps: 4000 (ss|ss) 114 us, 92 without);
// else wave w takes blocks w and w + 8.  F^b of this ket pair at F + (b * ncc + cc) * nq4 * 16
// in operand order (k step s, lane l: F^b[4 s + l / 16][16 cc + l % 16]); U
// steps of it are requested while the U before them run.
__device__ __forceinline__ int exch_split(int nblk, int nq4) { return nblk <= kWaves && nq4 > 64 ? kWaves / nblk : 1; }

template <int NR, int U>
__device__ __forceinline__ void exch_gemm(const ClassParams& cp, const double* __restrict__ X,
                                          const double* __restrict__ F, int row0, int wave, int lane, d4 (&yacc)[2]) {
  const int g = lane >> 4, n = lane & 15;
  const int ncc = (cp.nc + 15) / 16, nblk = NR * ncc, split = exch_split(nblk, cp.nq4);
  const int P = exch_rows_per_b(cp);
  const int64_t fs = (int64_t)cp.nq4 * 16;
  const int steps = cp.nq4 >> 2;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int part = nblk <= kWaves ? wave / nblk : 0;
    const int blk = nblk <= kWaves ? wave - part * nblk + kWaves * i : wave + kWaves * i;
    if (blk >= nblk || part >= split) break;
    const int r = blk / ncc, cc = blk - (blk / ncc) * ncc;
    const int ib = (row0 + r * 16) / P;  // one b per row block
    if (ib >= cp.nb) continue;           // padding rows past the last b
    const int s0 = steps * part / split, s1 = steps * (part + 1) / split;
    const double* __restrict__ Fb = F + ((int64_t)ib * ncc + cc) * fs + lane;
    const double* __restrict__ Xr = X + (r * 16 + n) * cp.xs + g;
    d4 acc = yacc[i];
    double b[U], bn[U];
    auto fetch = [&](double (&x)[U], int st) {
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = Fb[min(st + u, steps - 1) * 64];
    };
    fetch(b, s0);
#pragma unroll 1
    for (int st = s0; st < s1; st += U) {
      fetch(bn, st + U);
      double a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) a[u] = Xr[4 * min(st + u, steps - 1)];
      asm volatile("" ::: "memory");  // keep the requests ahead of the products
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (st + u < s1) acc = mfma16<false>(a[u], b[u], acc);
#pragma unroll
      for (int u = 0; u < U; ++u) b[u] = bn[u];
    }
    yacc[i] = acc;
  }
}

// y of the blocks, the parts added in order, to outq[(b * na + a) * nc + c] (valid a,
// b, c only).  part: LDS for kWaves blocks; called by all threads.
template <int NR>
__device__ __forceinline__ void exch_store(const ClassParams& cp, const d4 (&yacc)[2], double scale,
                                           double* __restrict__ outq, double* parts, int row0, int wave, int lane) {
  const int g = lane >> 4, n = lane & 15;
  const int ncc = (cp.nc + 15) / 16, nblk = NR * ncc, split = exch_split(nblk, cp.nq4);
  if (split > 1) {
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) parts[(wave * 4 + jj) * 64 + lane] = yacc[0][jj];
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int blk = wave + kWaves * i;
    if (blk >= nblk) break;
    const int r = blk / ncc, cc = blk - (blk / ncc) * ncc;
    const int ic = 16 * cc + n;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      double y = yacc[i][jj];
      for (int p = 1; p < split; ++p) y += parts[((wave + p * nblk) * 4 + jj) * 64 + lane];
      int ia, ib;
      exch_row(cp, row0 + r * 16 + acc_row<false>(jj, g), ia, ib);
      if (ia < cp.na && ib < cp.nb && ic < cp.nc) outq[((int64_t)ib * cp.na + ia) * cp.nc + ic] = y * scale;
    }
  }
}

// LDS regions of a tile (see dense_layout).
struct DenseLds {
  TileLds t;  // shells, [0]^(m) and what the recursion's steps share with eri4_tile.h
  double *box, *brae, *kete, *X;
  int2 *ptab, *qtab;
  uint2* entl;  // recursion table of total orders up to kWaveL, in the place of rowt
};

// Tables of row (u, v) of W, the k-th, of L+1-u-v values: it lies in the tail of the
// k-th longest of [r]'s row tails (S1 - (L+1-n) values behind row (t, u) of n = t+u;
// the (t, u) of largest n come last in the list uvs).  Without spare columns (S1 ==
// L+1) the first row is one longer than any tail and goes behind the box.
template <bool SLAB>
__device__ __forceinline__ void w_row(const TileLds& s, const uint32_t* __restrict__ uvs, int L, int S1, int k) {
  const uint32_t w = uvs[k];
  const int u = (int)(w & 0xff), v = (int)((w >> 8) & 0xff), sum = (int)(w >> 24);
  const int shift = S1 == L + 1;
  int at = r_cells(SLAB, L);
  if (k >= shift) {
    const uint32_t e = uvs[nuv(L) - 1 - (k - shift)];
    at = r_offset(SLAB, L, (int)(e & 0xff), (int)((e >> 8) & 0xff), L + 1 - (int)(e >> 24));
  }
  s.rowt[u * (L + 1) + v] = (uint16_t)at;
  s.rs[k] = (uint32_t)(at | (sum << 16));
  s.rv[k] = (uint16_t)(u | (v << 8));
}

// [r] into the box or slab layout from W: 16 rows (u, v) (the columns of the
// product) by 16 t at a time.
template <bool SLAB>
__device__ __forceinline__ void build_box(const DenseLds& s, int L, int S1, int S2, int task, int ntask, int lane) {
  const int g = lane >> 4;
  for (int i = 0; i < ntask; ++i) {
    const int w = __builtin_amdgcn_readlane(task, i);
    const int tb = w >> 12, r = (w & 0xfff) + (lane & 15), rc = min(r, nuv(L) - 1);
    const uint32_t e = s.t.rs[rc], uv = s.t.rv[rc];
    const int u = (int)(uv & 0xff), v = (int)(uv >> 8);
    const int last = r < nuv(L) ? L - u - v : -1;  // largest t
    const double* src = s.box + (e & 0xffff);
    double* o = s.box + u * S1 + v;
    // the block's first row is its longest
    const int tm = min(16 * tb + 15, __builtin_amdgcn_readfirstlane(last));
    const d4 acc = small_product(
        (tm >> 2) + 1 - 2 * tb, [&](int k) { return s.t.h[(4 * tb + k) * 64 + lane]; },
        [&](int k) { return src[min(8 * tb + 4 * k + g, max(last, 0))]; });
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int t = 16 * tb + 4 * jj + g;
      if (t <= last) o[SLAB ? slab_base(t, L, S1) : t * S2] = acc[jj];
    }
  }
}

// Everything a workgroup does after its prologue, for NR valid row blocks and
// NC1 first-transform column blocks of this wave.  [r] comes from one wave
// (hermite_r_wave; LOW: total orders up to kWaveL) or from three products
// (eri4_tile.h); W sits in the tails of [r]'s rows, so that the box needs no room
// beside it.  Bound by the first transform's products: of a tile of (ii|ii), 216 000
// cycles for solid harmonics, they take 143 000 (117 000 at the matrix cores' rate),
// the second transform 58 000, the steps before them 15 000.  512 (ii|ii) quartets
// of single primitives took 2172 us (solid) and 256 of them 3434 us (exchange) with
// the recursion level by level and operands requested one or two steps ahead; 1620
// and 2690 us so.
// kDenseSolid: rows and columns are real solid harmonics and both
// transforms read their H matrices from hb / hk (this quartet's, hbs / hks doubles
// per primitive pair, pair (i, j) of shells with K1, K2 primitives at slot
// i * K2 + j).
// kDenseCart: E as products of 1-d tables in both transforms (gemm1_e, gemm2_group).
// kDenseExch: no second transform; bra rows are ordered (b, a) with a padded
// to a multiple of 16 (exch_row), so each 16-row block has one b, and [ab|q]
// is contracted on the matrix cores with F^b[q][c] = sum_d E_cd^q D_bd of ket
// pair (k, l) (exchange_f_kernel, at hk + (k * kmax + l) * hks in operand
// order), accumulated over the ket pairs into y[a][c] = sum_d (ab|cd) D_bd,
// written to outq[(b * na + a) * nc + c] for the tile's b (Cartesian).  A row
// block holds no a with ax above that of its first, and E_ab^tuv = 0 for t > ax+bx:
// its first transform ends with that t (of (ii|ii)'s products 23% fall away).  Of few
// values of p, or of p and column blocks together, the separate ends of the row blocks
// cost more than the products: 300 (pp|pp) 35 us cut, 34 whole, (gg|ss) 131 and 115,
// (hh|dp) 407 and 412, (kk|ss) 1578 and 1638.
constexpr int kCutP = 84, kCutPq = 200;
template <int NR, int NC1, bool SLAB, int MODE, bool LOW>
__device__ __forceinline__ void dense_body(const ClassParams& cp, const DenseLds& s, const Tables& tb,
                                           double* __restrict__ outq, int row0, int Ka, int Kb, int Kc, int Kd,
                                           int task, int ntask, int tid, int wave, int lane,
                                           const double* __restrict__ hb, const double* __restrict__ hk, int64_t hbs,
                                           int64_t hks) {
  constexpr bool EXCH = MODE == kDenseExch, CART = MODE == kDenseCart;
  const int kmax = cp.kmax, L = cp.L;
  const double* A = s.t.sh;
  const double* B = s.t.sh + 3;
  const double* C = s.t.sh + 6;
  const double* D = s.t.sh + 9;
  const double* ex = s.t.sh + 12;
  const double* co = s.t.sh + 12 + 4 * kmax;
  constexpr int NC1A = NC1 > 0 ? NC1 : 1;

  // bra rows of this lane (A operand of the first transform) and where the p of
  // each row block end
  int rowx[NR], rowy[NR], rowz[NR], kend[NR], kmin = cp.np4;
#pragma unroll
  for (int r = 0; r < NR && (EXCH || CART); ++r) {
    int ia, ib, ax, ay, az, bx, by, bz;
    if constexpr (EXCH) {
      exch_row(cp, row0 + r * 16 + (lane & 15), ia, ib);
    } else {
      ia = (row0 + r * 16 + (lane & 15)) / cp.nb;
      ib = row0 + r * 16 + (lane & 15) - ia * cp.nb;
    }
    if (ia < cp.na && ib < cp.nb) {
      cart_of(cp.la, ia, ax, ay, az);
      cart_of(cp.lb, ib, bx, by, bz);
      rowx[r] = (ax * (cp.lb + 1) + bx) * cp.tbrow;
      rowy[r] = cp.tbaxis + (ay * (cp.lb + 1) + by) * cp.tbrow;
      rowz[r] = 2 * cp.tbaxis + (az * (cp.lb + 1) + bz) * cp.tbrow;
    } else {
      const int zr = (cp.la + 1) * (cp.lb + 1) * cp.tbrow;
      rowx[r] = zr;
      rowy[r] = cp.tbaxis + zr;
      rowz[r] = 2 * cp.tbaxis + zr;
    }
    kend[r] = cp.np4;
    if (CART || cp.np4 <= kCutP || cp.np4 * cp.nqb <= kCutPq) continue;
    exch_row(cp, row0 + r * 16, ia, ib);  // the block's first row: the largest ax
    kend[r] = 0;
    if (ib < cp.nb) {
      cart_of(cp.la, ia, ax, ay, az);
      cart_of(cp.lb, ib, bx, by, bz);
      const int rest = cp.Lb - ax - bx;  // p with t <= ax+bx: the first of the table
      kend[r] = (cp.np - (rest > 0 ? nherm(rest - 1) : 0) + 3) & ~3;
    }
    kmin = min(kmin, kend[r]);
  }
  // [ab|q] columns of this lane (B operand of the first transform)
  int offq[NC1A], tq[NC1A];
#pragma unroll
  for (int c = 0; c < NC1A; ++c) {
    const int2 e = (c < NC1) ? s.qtab[(wave + 8 * c) * 16 + (lane & 15)] : make_int2(0, 0);
    offq[c] = e.y;
    tq[c] = (int)((unsigned)e.x >> 24);
  }
  const int ncbw = (wave < cp.ncdb) ? (cp.ncdb - wave + 7) / 8 : 0;  // output column blocks of this wave

  const int hs = 64 * h_steps(L);
  const bool over = !LOW && cp.o_brae == cp.o_zt;
  // (of low orders the transforms amplify little, and it would be a tenth of a tile's time)
  int eb = 0, ek = 0;
  if constexpr (!LOW) tiny_exponents(s.t.sh, kmax, Ka, Kb, Kc, Kd, eb, ek);
  const double scaleb = ldexp(1.0, -eb), scalek = ldexp(1.0, -ek), unscale = ldexp(1.0, eb + ek);
  // EXCH: y blocks (row block, 16 columns c) of this wave, kept over the ket pairs
  d4 yacc[2] = {acc_zero<false>(), acc_zero<false>()};

  for (int kl = 0; kl < Kc * Kd; ++kl) {
    const int k = kl / Kd, l = kl - (kl / Kd) * Kd;
    typename Acc<false>::type acc1[NR][NC1A];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int c = 0; c < NC1A; ++c) acc1[r][c] = acc_zero<false>();

    for (int ij = 0; ij < Ka * Kb; ++ij) {
      const int i = ij / Kb, j = ij - (ij / Kb) * Kb;
      int ti = tid;  // opaque, as in tile_body
      asm volatile("" : "+v"(ti));
      const int la_ = ti & 63;
      // [0]^(m), of low orders [r] (wave 0) and the per-axis tables, with room the bra
      // tables too, and for kDenseCart at first the ket tables (the other waves)
      {
        const double za = ex[i], zb = ex[kmax + j], zc = ex[2 * kmax + k], zd = ex[3 * kmax + l];
        double pq[3];
        if constexpr (!LOW) {
          const double iz = 1.0 / (za + zb), iq = 1.0 / (zc + zd);
#pragma unroll
          for (int x = 0; x < 3; ++x) pq[x] = (za * A[x] + zb * B[x]) * iz - (zc * C[x] + zd * D[x]) * iq;
          if (wave == 0 && la_ <= L) {
            double ab2 = 0.0, cd2 = 0.0, r2 = 0.0;
#pragma unroll
            for (int x = 0; x < 3; ++x) {
              ab2 += (A[x] - B[x]) * (A[x] - B[x]);
              cd2 += (C[x] - D[x]) * (C[x] - D[x]);
              r2 += pq[x] * pq[x];
            }
            const double wb = co[i] * co[kmax + j] * exp(-za * zb * iz * ab2);
            const double wk = co[2 * kmax + k] * co[3 * kmax + l] * exp(-zc * zd * iq * cd2);
            s.t.baseM[la_] = hermite_base_m(la_, za + zb, zc + zd, r2, (wb * scaleb) * (wk * scalek), tb.boys);
          }
        } else if (wave == 0) {
          // the bra pair in lanes 0..31, the ket pair in the others
          const int ket = la_ >> 5;
          const double z1 = ket ? zc : za, z2 = ket ? zd : zb, z = z1 + z2, iz = 1.0 / z;
          const double c = ket ? co[2 * kmax + k] * co[3 * kmax + l] : co[i] * co[kmax + j];
          double p[3], d2 = 0.0, r2 = 0.0;
#pragma unroll
          for (int x = 0; x < 3; ++x) {
            const double s1 = A[6 * ket + x], s2 = A[6 * ket + 3 + x];
            p[x] = (z1 * s1 + z2 * s2) * iz;
            d2 += (s1 - s2) * (s1 - s2);
          }
          const double w = c * exp(-z1 * z2 * iz * d2), zo = __shfl_xor(z, 32), wo = __shfl_xor(w, 32);
#pragma unroll
          for (int x = 0; x < 3; ++x) {
            const double o = __shfl_xor(p[x], 32);
            pq[x] = ket ? o - p[x] : p[x] - o;
            r2 += pq[x] * pq[x];
          }
          if (la_ <= L) s.t.baseM[la_] = hermite_base_m(la_, z, zo, r2, w * wo, tb.boys);
          hermite_r_wave(s.box, s.t.baseM, L, pq[0], pq[1], pq[2], s.entl, la_);
        }
        if (wave != 0) {
          if constexpr (!LOW)
            build_htables(s.t.h, hs, tb.hcoef, pq[0], pq[1], pq[2], ti - 64, kThreads - 64);
          if (MODE != kDenseSolid && !over) {
            build_etab_rows(s.brae, cp.la, cp.lb, cp.tbrow, cp.tbaxis, za, zb, A, B, false, (ti >> 4) - 4,
                            kWaves * 4 - 4, la_ & 15);
            if (wave == kWaves - 1) zero_rows(s.brae, cp.la, cp.lb, cp.tbrow, cp.tbaxis, la_, 64);
          }
          if (CART && ij == 0) {
            build_etab_rows(s.kete, cp.lc, cp.ld, cp.tkrow, cp.tkaxis, zc, zd, C, D, true, (ti >> 4) - 4,
                            kWaves * 4 - 4, la_ & 15);
            if (wave == kWaves - 1) zero_rows(s.kete, cp.lc, cp.ld, cp.tkrow, cp.tkaxis, la_, 64);
          }
        }
      }
      __syncthreads();
      if constexpr (!LOW) {
        if (wave < 3) {
          const int jb = wave == 2, ub = wave == 1;
          if (L >= 16 * (jb + ub)) build_zt(s.t, s.t.h + 2 * hs, L, jb, ub, la_);
        }
        __syncthreads();
        build_w(s.t, s.box, s.t.h + hs, L, task, ntask, la_);
        __syncthreads();
        build_box<SLAB>(s, L, cp.S1, cp.S2, task, ntask, la_);
        __syncthreads();
      }
      // first transform, accumulated over ij: [ab|q] += A_ab^p [p|q]
      if constexpr (EXCH) {
        if (over) {  // the bra tables over zt and the per-axis tables
          build_etab_rows(s.brae, cp.la, cp.lb, cp.tbrow, cp.tbaxis, ex[i], ex[kmax + j], A, B, false, ti >> 4,
                          kThreads / 16, la_ & 15);
          zero_rows(s.brae, cp.la, cp.lb, cp.tbrow, cp.tbaxis, ti, kThreads);
          __syncthreads();
        }
        if constexpr (NC1 > 0) {
          gemm1_e<NR, NC1, SLAB>(acc1, s.brae, s.box, s.ptab, rowx, rowy, rowz, offq, tq, 0, kmin, L,
                                            cp.S1, lane);
          if (kmin < cp.np4) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
              typename Acc<false>::type a[1][NC1];
              const int x[1] = {rowx[r]}, y[1] = {rowy[r]}, z[1] = {rowz[r]};
#pragma unroll
              for (int c = 0; c < NC1; ++c) a[0][c] = acc1[r][c];
              gemm1_e<1, NC1, SLAB>(a, s.brae, s.box, s.ptab, x, y, z, offq, tq, kmin, kend[r], L, cp.S1, lane);
#pragma unroll
              for (int c = 0; c < NC1; ++c) acc1[r][c] = a[0][c];
            }
          }
        }
      } else if constexpr (CART && NC1 > 0) {
        gemm1_e<NR, NC1, SLAB>(acc1, s.brae, s.box, s.ptab, rowx, rowy, rowz, offq, tq, 0, cp.np4, L, cp.S1, lane);
      } else if constexpr (NC1 > 0) {
        gemm1_h<NR, NC1, SLAB>(acc1, hb + (i * Kb + j) * hbs + (row0 / 16) * (cp.np4 * 16) + lane, s.box, s.ptab,
                               offq, tq, cp.np4, L, cp.S1, lane);
      }
      __syncthreads();
    }

    // [ab_tile|q] -> LDS (over [r])
    if constexpr (NC1 > 0) {
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int c = 0; c < NC1; ++c) {
          const int cb = wave + 8 * c;
#pragma unroll
          for (int jj = 0; jj < 4; ++jj)
            s.X[(r * 16 + acc_row<false>(jj, lane >> 4)) * cp.xs + cb * 16 + (lane & 15)] = acc1[r][c][jj];
        }
    }
    __syncthreads();
    if constexpr (EXCH) {
      // y[a][c] += sum_q [ab|q] F^b[q][c] for this ket pair
      const double* f = hk + (k * kmax + l) * hks;
      if (LOW && cp.nq4 <= 32)
        exch_gemm<NR, 2>(cp, s.X, f, row0, wave, lane, yacc);
      else
        exch_gemm<NR, 8>(cp, s.X, f, row0, wave, lane, yacc);
    } else {
      // second transform, written to HBM (accumulated over kl); groups of four
      // column blocks (2 with four row blocks, for the accumulators)
      constexpr int G2 = NR >= 4 ? 2 : 4;
      const double* hkp = CART ? nullptr : hk + (k * Kd + l) * hks + lane;
      for (int g0 = 0; g0 < ncbw; g0 += G2) {
        const int ng = min(G2, ncbw - g0);
        const int cb0 = wave + 8 * g0;
        const bool first = kl == 0;
        auto group = [&](auto nc, int cb) {
          if constexpr (CART)
            gemm2_group<NR, decltype(nc)::value, 8>(cp, s.X, s.kete, s.qtab, cb, row0, outq, first, lane, unscale);
          else if (LOW)
            gemm2_group_h<NR, decltype(nc)::value, 4>(cp, s.X, hkp, cb, row0, outq, first, unscale, lane);
          else
            gemm2_group_h<NR, decltype(nc)::value, 8>(cp, s.X, hkp, cb, row0, outq, first, unscale, lane);
        };
        const std::integral_constant<int, 1> one;
        const std::integral_constant<int, 2> two;
        if (ng >= 2)
          group(two, cb0);
        else
          group(one, cb0);
        if (ng == 3) group(one, cb0 + 16);
        if (ng == 4) group(two, cb0 + 16);
      }
    }
    __syncthreads();
  }
  if constexpr (EXCH) exch_store<NR>(cp, yacc, unscale, outq, s.X, row0, wave, lane);
}

// All the work of one tile: quartet q, bra rows rt*RB*16.., whose integrals
// start at outq.  Called by every thread of the workgroup; ends with a barrier.
// PAIRS and the shell arrays: as load_shells.  MODE, hb, hk: as dense_body.
template <int RB, bool SLAB, bool PAIRS, int MODE, bool LOW>
__device__ __forceinline__ void dense_tile(const ClassParams& cp, unsigned char* lds, const Tables& tb,
                                           const double* __restrict__ centers, const double* __restrict__ exps,
                                           const double* __restrict__ coefs, const int32_t* __restrict__ nprim,
                                           double* __restrict__ outq, int64_t q, int rt, int tid, int wave, int lane,
                                           const double* __restrict__ kcenters, const double* __restrict__ kexps,
                                           const double* __restrict__ kcoefs, int64_t nket,
                                           const double* __restrict__ hb, const double* __restrict__ hk, int64_t hbs,
                                           int64_t hks) {
  constexpr bool EXCH = MODE == kDenseExch;
  const int kmax = cp.kmax, L = cp.L;
  DenseLds s;
  s.t.sh = (double*)(lds + cp.o_shell);
  s.t.baseM = (double*)(lds + cp.o_base);
  s.t.rowt = (uint16_t*)(lds + cp.o_rowt);
  s.t.rs = (uint32_t*)(lds + cp.o_rs);
  s.t.rv = (uint16_t*)(lds + cp.o_rv);
  s.t.zt = (double*)(lds + cp.o_zt);
  s.t.h = (double*)(lds + cp.o_h);
  s.ptab = (int2*)(lds + cp.o_ptab);
  s.qtab = (int2*)(lds + cp.o_qtab);
  s.box = (double*)(lds + cp.o_union);
  s.brae = (double*)(lds + cp.o_brae);
  s.kete = (double*)(lds + cp.o_kete);
  s.entl = (uint2*)(lds + cp.o_rowt);
  s.X = (double*)(lds + cp.o_union);
  int* shn = (int*)(s.t.sh + 12 + 8 * kmax);
  load_shells<PAIRS>(s.t.sh, shn, kmax, centers, exps, coefs, nprim, q, kcenters, kexps, kcoefs, nket, tid);
  build_htab(s.ptab, cp.Lb, cp.np, cp.np4, cp.S1, cp.S2, SLAB, tid);
  build_htab(s.qtab, cp.Lk, cp.nq, 16 * cp.nqb, cp.S1, cp.S2, SLAB, tid);
  // tables of the recursion; this wave's tasks of W and [r], one per lane
  int ntask = 0, task = 0;
  if constexpr (LOW) {
    if (tid < nherm(L)) s.entl[tid] = tb.rtab[cp.rtab_off + tid];
  } else {
    if (tid < nuv(L)) w_row<SLAB>(s.t, tb.ttab + cp.o_uv, L, cp.S1, tid);
    ntask = (cp.ntask - wave + kWaves - 1) / kWaves;
    task = lane < ntask ? (int)tb.ttab[cp.o_task + wave + kWaves * lane] : 0;
  }
  __syncthreads();

  const int Ka = shn[0], Kb = shn[1], Kc = shn[2], Kd = shn[3];
  const int row0 = rt * RB * 16;
  if (Ka < 1 || Ka > kmax || Kb < 1 || Kb > kmax || Kc < 1 || Kc > kmax || Kd < 1 || Kd > kmax) {
    if constexpr (EXCH) {
      // this tile's rows (b, a) of y
      for (int i = tid; i < RB * 16 * cp.nc; i += kThreads) {
        int ia, ib;
        exch_row(cp, row0 + i / cp.nc, ia, ib);
        if (ia < cp.na && ib < cp.nb) outq[((int64_t)ib * cp.na + ia) * cp.nc + i % cp.nc] = __builtin_nan("");
      }
    } else {
      const int nrows = min(RB * 16, cp.nab - row0);
      const int ncols = cp.ncd;
      double* o = outq + (int64_t)row0 * ncols;
      for (int i = tid; i < nrows * ncols; i += kThreads) o[i] = __builtin_nan("");
    }
    __syncthreads();
    return;
  }
  const int nc1 = (wave < cp.nqb) ? min(kMaxC1, (cp.nqb - wave + 7) / 8) : 0;  // [ab|q] column blocks of this wave
  const int nrows_all = EXCH ? cp.nb * 16 * ((cp.na + 15) / 16) : cp.nab;           // (padded) bra rows
  const int nrv = min(RB, (nrows_all - row0 + 15) / 16);                          // valid row blocks of this tile
#define BODY(NR, NC1)                                                                                          \
  dense_body<NR, NC1, SLAB, MODE, LOW>(cp, s, tb, outq, row0, Ka, Kb, Kc, Kd, task, ntask, tid, wave, lane, hb, hk, \
                                  hbs, hks)
  constexpr int NR2 = RB >= 2 ? 2 : 1;
  if constexpr (RB == 4) {
    // 64-row tiles (kets with at most 2 column blocks per wave): the last tile
    // of a quartet runs with padding rows, whose outputs are not written
    switch (nc1) {
      case 0: BODY(4, 0); break;
      case 1: BODY(4, 1); break;
      default: BODY(4, 2); break;
    }
  } else if (nrv == NR2 && NR2 == 2) {
    switch (nc1) {
      case 0: BODY(NR2, 0); break;
      case 1: BODY(NR2, 1); break;
      case 2: BODY(NR2, 2); break;
      case 3: BODY(NR2, 3); break;
      default: BODY(NR2, 4); break;
    }
  } else if constexpr (SLAB) {
    switch (nc1) {
      case 0: BODY(1, 0); break;
      case 1: BODY(1, 1); break;
      case 2: BODY(1, 2); break;
      case 3: BODY(1, 3); break;
      case 4: BODY(1, 4); break;
      case 5: BODY(1, 5); break;
      default: BODY(1, 6); break;
    }
  } else {
    switch (nc1) {
      case 0: BODY(1, 0); break;
      case 1: BODY(1, 1); break;
      case 2: BODY(1, 2); break;
      case 3: BODY(1, 3); break;
      default: BODY(1, 4); break;
    }
  }
#undef BODY
}

}  // namespace
}  // namespace eri4
