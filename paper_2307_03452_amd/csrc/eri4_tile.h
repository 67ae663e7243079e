// eri4_tile.h -- gfx950 device code of the Cartesian integral kernels: one
// workgroup computes one tile of bra rows of one quartet.
//
// (ab|cd) over contracted Cartesian Gaussians by the matrix form of the
// McMurchie-Davidson scheme (Asadchev & Valeev, Sec. 2 and Sec. 3):
//
//   [p|q] = (-1)^|q| [p+q]^(0)                                       eq. (pq)
//   [ab|q] = sum_p E_ab^p [p|q]                                      eq. (ab_to_hermite)
//   (ab|cd) = sum_q E_cd^q [ab|q]                                    eq. (cd_to_hermite)
//
// E is a product of one 1-d table per axis, E_ab^tuv = X^t Y^u Z^v with X
// depending on (ax, bx) only, and zero above t = ax+bx, u = ay+by, v = az+bz.
// Both transforms use that: rows are grouped by (ax, bx), and for one group
//
//   [ab|q] = sum_uv Y^u Z^v ( sum_t X^t [tuv|q] )
//
// the inner sum, over ax+bx+1 values of t, is the same for every pair of p and
// q with the same u+uq, v+vq, so it is formed once per (ax, bx) for all of them
// (F below, at most as many values as [r] has); the outer sum runs over u+v <=
// Lb-ax-bx only, as a product on the matrix cores (16 rows of the group x 16
// columns q) that gathers its operand from F.  For (ii|ii) that is 813 (16-row x
// 4-k) steps per 16 columns where the dense product of the same rows takes 5586,
// for (gg|gg) 146 against 630, for (kk|kk) 1573 against 13770.  The second
// transform is the same with columns (cd) grouped by (cx, dx); its inner sum is
// formed while the operand is read, since no two products share it.
#pragma once
#include <type_traits>

#include "eri4_device.h"

namespace eri4 {
namespace {

// Shapes of the kernels: CW waves share the columns of [ab|q] (NC blocks of 16
// each), the 8 / CW groups of waves take one unit of bra row blocks each (at
// most RB blocks of 16 rows), XB blocks of XU units go through the LDS tile at a time.
template <int CW_, int RB_, int NC_>
struct TileShape {
  static constexpr int CW = CW_, RB = RB_, NC = NC_;
  static constexpr int UG = kWaves / CW_;
  static constexpr int XB = tile_xb(CW_, NC_), XU = tile_xu(CW_, NC_);
};

// LDS regions of one tile (byte offsets in TileParams).
struct TileLds {
  double *sh, *baseM, *kpair, *h, *zt, *g, *X, *kete;
  uint32_t* orow;      // byte offset in the output of each row of X
  uint16_t* rowt;      // where row (u, v) of W starts, at u (L+1) + v
  uint32_t* rs;        // rows of W in order: start | (u + v) << 16
  uint16_t* rv;        // and their u | v << 8
  uint16_t* rowf;      // where row (u, v) of F of this wave's unit starts
  uint32_t* rf;        // rows of that F in order: start | last t << 16
  int4 *btab, *ktab;   // (u, v) of the bra / ket: byte offsets into the y and z tables, rowf / X
  uint32_t* kcol;
};

// Value of the lane below (CTRL 0x111) or above (0x101) in its row of 16
// lanes; 0 past the end of the row.
template <int CTRL>
__device__ __forceinline__ double dpp_row(double x) {
  const long long v = __double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(v & 0xffffffffll), CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ double ipow(double x, int e) {  // x^e, 0 <= e < 32
  double r = 1.0;
#pragma unroll
  for (int b = 0; b < 5; ++b) {
    if (e & (1 << b)) r *= x;
    x *= x;
  }
  return r;
}

// The rows (axis, a, 0..l2) of the 1-d tables of one primitive pair by the two
// recursions after eq. (cart2herm-2), one row of 16 lanes per (axis, a): lane t
// holds E^t, a step moves t-1 and t+1 across lanes.  (A lane per (axis, a) with
// all t in its registers takes la + lb steps of la + lb + 1 dependent updates;
// here each step is three multiply-adds.)  Layout as build_etab: row (a, b) at
// axis * taxis + (a * (l2+1) + b) * trow.  g0: this row of lanes, of ng.
__device__ __forceinline__ void build_etab_rows(double* E, int l1, int l2, int trow, int taxis, double za, double zb,
                                                const double* A, const double* B, bool alt_sign, int g0, int ng,
                                                int t) {
  const int na = l1 + 1, nb = l2 + 1;
  const double iz = 1.0 / (za + zb);
  const double h = 0.5 * iz;
  const double t1 = (double)(t + 1);
  const bool neg = alt_sign && (t & 1);
  for (int c = g0; c < 3 * na; c += ng) {
    const int axis = c / na, a = c - (c / na) * na;
    const double dd = A[axis] - B[axis];
    const double pa = -zb * iz * dd, pb = za * iz * dd;
    double e = t == 0 ? 1.0 : 0.0;
    for (int s = 0; s < a; ++s) e = h * dpp_row<0x111>(e) + pa * e + t1 * dpp_row<0x101>(e);
    double* row = E + axis * taxis + a * nb * trow + t;
    for (int b = 0; b < nb; ++b) {
      if (t < trow) row[b * trow] = neg ? -e : e;
      if (b + 1 < nb) e = h * dpp_row<0x111>(e) + pb * e + t1 * dpp_row<0x101>(e);
    }
  }
}

// The all-zero row of each axis (padding rows and columns).
__device__ __forceinline__ void zero_rows(double* E, int l1, int l2, int trow, int taxis, int i, int n) {
  for (; i < 3 * trow; i += n) E[(i / trow) * taxis + (l1 + 1) * (l2 + 1) * trow + i % trow] = 0.0;
}

// x^e with the rounding of one operation: each product carries its error term.
__device__ __forceinline__ double ipow_exact(double x, int e) {  // 0 <= e < 32
  double rh = 1.0, rl = 0.0, xh = x, xl = 0.0;
#pragma unroll
  for (int b = 0; b < 5; ++b) {
    if (e & (1 << b)) {
      const double p = rh * xh;
      rl = fma(rh, xh, -p) + (rh * xl + rl * xh);
      rh = p;
    }
    const double p = xh * xh;
    xl = fma(2.0 * xh, xl, fma(xh, xh, -p));
    xh = p;
  }
  const double r = rh + rl;
  return fabs(rh) <= 0x1p1000 ? r : rh;  // (beyond, the error terms may be infinite)
}

// [0]^(m) = (-2 rho)^m 2 pi^(5/2) / (zp zq sqrt(zp + zq)) w F_m(rho |PQ|^2) of
// one lane m.  Above the table F_m(T) = c_m / (T^m sqrt(T)), so the powers
// join: (-2 rho / T)^m = (-2 / |PQ|^2)^m.  The rounding of a power's base counts m
// times and the sums that follow amplify it, so that the base is one operation where
// it can be and the power adds none: error of [r], relative to its largest terms, 1.02
// to 1.07 times that of eq. (md1) level by level with plain powers of -2 rho / T (800
// points per order 8..28, geometric mean), 0.99 to 1.03 so.
__device__ __forceinline__ double hermite_base_m(int m, double zp, double zq, double r2, double w,
                                                 const double* __restrict__ tab) {
  const double zs = zp + zq;
  const double rho = zp * zq / zs;
  const double T = rho * r2;
  const double pref = 2.0 * 17.493418327624862846 / (zp * zq * sqrt(zs));  // pi^(5/2)
  double F, x = -2.0 * rho;
  if (T < kBoysTMax) {
    F = boys_fm(m, T, tab);
  } else if (T >= kBoysTMax) {
    F = tab[(size_t)kBoysAsymRow * kBoysCols + m] / sqrt(T);
    x = -2.0 / r2;
  } else {
    F = __builtin_nan("");
  }
  return ipow_exact(x, m) * F * pref * w;  // w last: it may be subnormal
}

// The Hermite integrals and F.  Eq. (md1) applied along one axis is
//   [t] = sum_j H[t][j] [0]^(j),  H[t][t-a] = t! / (a! (t-2a)! 2^a) x^(t-2a), a = 0..t/2
// (each application of eq. (md1) either multiplies by x and raises m or lowers
// the index), so the whole recursion is three sums, one per axis, with a
// barrier after each, where applying eq. (md1) level by level takes L levels
// with one or two barriers each:
//   zt[v][m]    = sum_k HZ[v][k] [0]^(m+k)        m = 0..L-v
//   W[u][v][j]  = sum_k HY[u][k] zt[v][j+k]       j = 0..L-u-v
//   [tuv]       = sum_j HX[t][j] W[u][v][j]
// and F follows from W without forming [tuv]:
//   F_p[u][v][tq] = sum_t X_p^t [tq+t, u, v] = sum_j G_p[j][tq] W[u][v][j],
//   G_p[j][tq] = sum_t X_p^t HX[tq+t][j].
// All are products on the matrix cores (16 x 16 blocks, the padding of the
// triangles costs less than the lanes' own sums did: (ii|ii) took 19 000 cycles
// of a primitive quartet and tile in those).  H is kept per axis in operand
// order (h_steps(L) steps of 64): step s < 4: rows t = 0..15, k = 4 s + ..;
// above: t = 16.., k = 4 (s - 2) + ..

// A B of nk (1..8) steps of 4: the operands of all steps are read first.
template <class FA, class FB>
__device__ __forceinline__ d4 small_product(int nk, FA fa, FB fb) {
  d4 acc = acc_zero<false>();
  auto steps = [&](auto n) {
    constexpr int N = decltype(n)::value;
    double a[N], b[N];
#pragma unroll
    for (int k = 0; k < N; ++k) b[k] = fb(k);
#pragma unroll
    for (int k = 0; k < N; ++k) a[k] = fa(k);
#pragma unroll
    for (int k = 0; k < N; ++k) acc = mfma16<false>(a[k], b[k], acc);
  };
  switch (nk) {
#define T(N) \
  case N: steps(std::integral_constant<int, N>{}); break;
    T(1) T(2) T(3) T(4) T(5) T(6) T(7)
    default: steps(std::integral_constant<int, 8>{}); break;
#undef T
  }
  return acc;
}

// Limit of the distances P - Q (build_htables).  None where the bra's shells are more
// than 2^30 apart: their Gaussian product prefactor is zero, and the powers of P - Q
// and of A - B in G could have an infinite product.
__device__ __forceinline__ double far_limit(const double* A, const double* B) {
  double r2 = 0.0;
#pragma unroll
  for (int x = 0; x < 3; ++x) r2 += (A[x] - B[x]) * (A[x] - B[x]);
  return r2 > 0x1p60 ? 0.0 : 0x1p54;
}

// Per-axis tables h of P - Q by threads i, i + n, ...: hcoef * (P-Q)_axis^e, entry (row
// t, column j) with e = 2 j - t (hcoef is 0 where that is no exponent).  A distance above
// 2^54 counts as infinite and an entry above 2^250 as nothing: what they multiply, [0]^(j)
// with j >= e, is then below 2^-250 of [0]^(0) or has long been rounded to 0, and 0
// times an infinite power would be NaN.  Of total orders up to 12 no entry is infinite
// without the second (CUT false).
template <bool CUT = true>
__device__ __forceinline__ void build_htables(double* h, int hs, const double* __restrict__ hcoef, double px,
                                              double py, double pz, int i, int n, double lim = 0x1p54) {
  px = fabs(px) > lim ? 0.0 : px;
  py = fabs(py) > lim ? 0.0 : py;
  pz = fabs(pz) > lim ? 0.0 : pz;
  auto entry = [](double c, double x, int e) {
    const double v = c * ipow(x, e);
    return !CUT || fabs(v) <= 0x1p250 ? v : 0.0;  // (an infinite power times 0, too)
  };
  for (; i < hs; i += n) {
    const double c = hcoef[i];
    const int s = i >> 6;
    int e = max(0, (s < 4 ? 8 * s : 8 * s - 32) + 2 * ((i >> 4) & 3) - (i & 15));
    if (!CUT) e = min(e, 15);  // (past the rows below 16, whose coefficients are 0)
    h[i] = entry(c, px, e);
    h[hs + i] = entry(c, py, e);
    h[2 * hs + i] = entry(c, pz, e);
  }
}

// G of the np row groups of a unit, in operand order (step s: j = 4 s .., tq): one
// step of one group at a time, by the waves cw, cw + cws, .. of the unit.  bu: the
// unit's record.
__device__ __forceinline__ void build_g(const TileLds& s, const double* brae, const uint32_t* __restrict__ bu, int np,
                                        int xdeg, int L, int nks, int cw, int cws, int lane) {
  const int base = (lane >> 4) * 16, tq = lane & 15;
  for (int i = cw; i < np * nks; i += cws) {
    const int p = i / nks, ks = i - p * nks;
    const double* e = brae + (int)bu[2 + p];
    double acc = 0.0;
#pragma unroll 4
    for (int t = 0; t <= xdeg; ++t) {
      const int u = min(tq + t, L);
      // k = 4 ks .. of row u: steps 0..3 of rows below 16, steps from k = 8 above
      const bool ok = u < 16 ? ks < 4 : ks >= 2;
      const double hv = s.h[ok ? (ks + (u < 16 ? 0 : 2)) * 64 + base + (u & 15) : 0];
      acc = fma(ok ? hv : 0.0, e[t], acc);
    }
    s.g[i * 64 + lane] = acc;
  }
}

// F of the np row groups of a unit from W: 16 rows (the columns of the product) of
// one group at a time, by the waves cw, cw + cws, .. of the unit.  nrow: rows of
// F; fsize: doubles per group.
__device__ __forceinline__ void build_f(const TileLds& s, const double* W, double* F, int fsize, int nrow, int np,
                                        int L, int nks, int cw, int cws, int lane) {
  const int g = lane >> 4, nb = (nrow + 15) >> 4;
  int p = 0, b = cw;  // block b of group p
  for (; b >= nb && p < np; b -= nb) ++p;
  int r = min(16 * b + (lane & 15), nrow - 1);
  uint32_t e = s.rs[r], f = s.rf[r];
  while (p < np) {
    const int last = L - (int)(e >> 16);  // last value of this lane's row of W
    const double* w = W + (e & 0xffff);
    double* o = F + p * fsize + (f & 0xffff) + g;
    const int ft = 16 * b + (lane & 15) < nrow ? (int)(f >> 16) : -1;
    const double* gp = s.g + p * nks * 64 + lane;
    // the block's first row is its longest
    const int nk = min(nks, (__builtin_amdgcn_readfirstlane(last) >> 2) + 1);
    for (b += cws; b >= nb && p < np; b -= nb) ++p;
    r = min(16 * b + (lane & 15), nrow - 1);
    e = s.rs[r];
    f = s.rf[r];
    const d4 acc = small_product(
        nk, [&](int k) { return gp[k * 64]; }, [&](int k) { return w[min(4 * k + g, last)]; });
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
      if (4 * jj + g <= ft) o[4 * jj] = acc[jj];
  }
}

// W from zt, 16 pairs (v, j) (the columns of the product, in the order of the
// rows of W) by 16 rows u at a time; ntask tasks of this wave, one per lane of
// task: first pair | ub << 12.
__device__ __forceinline__ void build_w(const TileLds& s, double* W, const double* h, int L, int task, int ntask,
                                        int lane) {
  const int g = lane >> 4;
  for (int i = 0; i < ntask; ++i) {
    const int w = __builtin_amdgcn_readlane(task, i);
    const int ub = w >> 12, r = (w & 0xfff) + (lane & 15);
    const uint32_t e = s.rv[min(r, nuv(L) - 1)];
    const int v = (int)(e & 0xff), j = (int)(e >> 8);
    const int last = r < nuv(L) ? L - v - j : -1;  // largest u
    const double* src = s.zt + v * (L + 1) - ((v * (v - 1)) >> 1) + j;
    // the block's first pair has the most u
    const int um = min(16 * ub + 15, __builtin_amdgcn_readfirstlane(last));
    const uint16_t* row = s.rowt + (16 * ub + g) * (L + 1) + v;
    const d4 acc = small_product(
        (um >> 2) + 1 - 2 * ub, [&](int k) { return h[(4 * ub + k) * 64 + lane]; },
        [&](int k) { return src[min(8 * ub + 4 * k + g, max(last, 0))]; });
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
      if (16 * ub + 4 * jj + g <= last) W[row[4 * jj * (L + 1)] + j] = acc[jj];
  }
}

// zt from [0]^(m): block (rows v = 16 ub .., columns m = 16 jb ..).
__device__ __forceinline__ void build_zt(const TileLds& s, const double* h, int L, int jb, int ub, int lane) {
  const int g = lane >> 4, m = 16 * jb + (lane & 15);
  const int um = min(16 * ub + 15, L - 16 * jb);
  const d4 acc = small_product(
      (um >> 2) + 1 - 2 * ub, [&](int k) { return h[(4 * ub + k) * 64 + lane]; },
      [&](int k) { return s.baseM[min(m + 8 * ub + 4 * k + g, L)]; });
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) {
    const int v = 16 * ub + 4 * jj + g;
    if (m + v <= L) s.zt[v * (L + 1) - ((v * (v - 1)) >> 1) + m] = acc[jj];
  }
}

// acc[r] += sum over i < 4 of X^(T0+i) x[i][r], X^t in lane t of each row of 16
// lanes of exv.  The coefficient comes in through the row broadcast of the
// multiply-add itself: reading it into scalar registers costs two instructions
// more per multiply-add, which made the sums as long as the products that use
// them.  The leading wait states are those between a vector write of exv and
// its use across lanes, the trailing ones those before the matrix cores may read
// a vector result (the compiler does not count them for assembly).
template <int NR, int T0>
__device__ __forceinline__ void fold4(double (&acc)[NR], const double (&x)[4][NR], double exv) {
#define F_(D, S, I) "v_fmac_f64_dpp %" D ", %[e], %[" S "] row_newbcast:%[" I "] row_mask:0xf bank_mask:0xf\n\t"
  if constexpr (NR == 2)
    asm("s_nop 1\n\t" F_("0", "a", "i") F_("1", "p", "i") F_("0", "b", "j") F_("1", "q", "j") F_("0", "c", "k")
            F_("1", "r", "k") F_("0", "d", "l") F_("1", "s", "l") "s_nop 1"
        : "+v"(acc[0]), "+v"(acc[1])
        : [e] "v"(exv), [a] "v"(x[0][0]), [b] "v"(x[1][0]), [c] "v"(x[2][0]), [d] "v"(x[3][0]), [p] "v"(x[0][1]),
          [q] "v"(x[1][1]), [r] "v"(x[2][1]), [s] "v"(x[3][1]), [i] "n"(T0), [j] "n"(T0 + 1), [k] "n"(T0 + 2),
          [l] "n"(T0 + 3));
  else
    asm("s_nop 1\n\t" F_("0", "a", "i") F_("0", "b", "j") F_("0", "c", "k") F_("0", "d", "l") "s_nop 1"
        : "+v"(acc[0])
        : [e] "v"(exv), [a] "v"(x[0][0]), [b] "v"(x[1][0]), [c] "v"(x[2][0]), [d] "v"(x[3][0]), [i] "n"(T0),
          [j] "n"(T0 + 1), [k] "n"(T0 + 2), [l] "n"(T0 + 3));
#undef F_
}

__device__ __forceinline__ double lds_at(const double* p, int bytes) {
  return *(const double*)((const char*)p + bytes);
}

// One unit of the first transform: NP row groups (ax, bx) of equal ax + bx,
// NB blocks of 16 rows each, by NC column blocks of this wave:
//   acc[R0 + p * NB + r][c] += sum_uv Y^u Z^v F_p[u + uq][v + vq][tq]
// rowf gives where the row (u + uq, v + vq) of F starts.  The table entries and
// row starts of the next steps and the E factors of the next one are read
// before the products of this one.
template <class S, int NP, int NB, int R0, bool F32>
__device__ __forceinline__ void gemm1_unit(typename Acc<F32>::type (&acc)[S::RB][S::NC], const TileLds& s,
                                           const double* brae, const double* F, int fsize, const TileParams& cp,
                                           int K, const uint32_t (&brow)[S::RB], const uint32_t (&qcol)[S::NC],
                                           int lane) {
  constexpr int NC = S::NC, NBK = NP * NB;
  const int g = lane >> 4, pad = cp.kb;
  int rowy[NBK], rowz[NBK], tq[NC], iq[NC];
#pragma unroll
  for (int r = 0; r < NBK; ++r) {
    rowy[r] = 8 * (cp.tbaxis + (int)(brow[R0 + r] & 0x7f) * cp.tbrow);
    rowz[r] = 8 * (2 * cp.tbaxis + (int)((brow[R0 + r] >> 7) & 0x7f) * cp.tbrow);
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int u = (int)((qcol[c] >> 8) & 0xff);
    tq[c] = (int)(qcol[c] & 0xff);
    iq[c] = 2 * (u * cp.L + (int)(qcol[c] >> 16));  // u (L + 1) + v
  }
  int4 w = s.btab[g < K ? g : pad];
  int row[NC];
  double y[NBK], z[NBK], b[NP][NC];
  auto fetch_rows = [&]() {
#pragma unroll
    for (int c = 0; c < NC; ++c) row[c] = *(const uint16_t*)((const char*)s.rowf + w.z + iq[c]);
  };
  auto fetch = [&]() {
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int c = 0; c < NC; ++c) b[p][c] = F[p * fsize + row[c] + tq[c]];
  };
  auto fetch_e = [&]() {
#pragma unroll
    for (int r = 0; r < NBK; ++r) {
      y[r] = lds_at(brae, rowy[r] + w.x);
      z[r] = lds_at(brae, rowz[r] + w.y);
    }
  };
  fetch_rows();
  fetch_e();
  w = s.btab[4 + g < K ? 4 + g : pad];
  fetch();
  fetch_rows();
#pragma unroll 1
  for (int kk = 0; kk < K; kk += 4) {
    double a[NBK], bb[NP][NC];
#pragma unroll
    for (int r = 0; r < NBK; ++r) a[r] = y[r] * z[r];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int c = 0; c < NC; ++c) bb[p][c] = b[p][c];
    fetch_e();
    fetch();
    w = s.btab[kk + 8 + g < K ? kk + 8 + g : pad];
    fetch_rows();
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int r = 0; r < NB; ++r)
#pragma unroll
        for (int c = 0; c < NC; ++c)
          acc[R0 + p * NB + r][c] = mfma16<F32>(a[p * NB + r], bb[p][c], acc[R0 + p * NB + r][c]);
  }
}

// The quartet's block of the output as a buffer resource: stores past its end
// (padding rows and columns, whose offsets are made large) are dropped and
// loads return 0, so that the write needs no masks.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t out_rsrc(double* outq, int n) {
  return __builtin_amdgcn_make_buffer_rsrc(outq, 0, n * 8, 0x00027000);
}
constexpr uint32_t kNoRow = 0x80000000u, kNoCol = 0x40000000u;

// One unit of the second transform: NBK blocks of 16 columns, each of one group
// (cx, dx), all of equal cx + dx < 4 NCH, by NR blocks of 16 rows of the [ab|q]
// tile, then the output write:
//   out[ab][cd] (+)= sum_uv Y^u Z^v (sum_t X^t [ab|tuv])
// X holds the columns q in (u, v) order of increasing u + v, t fastest, and three
// zero columns: the sums run over 4 NCH values of t, with zero coefficients past
// cx + dx.  The reads of the next step go out before the products of this one, so
// that its sums need not wait: while one wave of a SIMD sums, the other's
// products run.
template <int NBK, int NCH, int NR, bool F32>
__device__ __forceinline__ void gemm2_loop(typename Acc<F32>::type (&acc)[NBK][NR], const TileParams& cp,
                                           const TileLds& s, const uint32_t* __restrict__ unit, int lane) {
  const int g = lane >> 4, n = lane & 15;
  const int xdeg = (int)(unit[0] & 0xff), K = (int)unit[1], pad = cp.kk;
  double exv[NBK];
  int ky[NBK], kz[NBK];
  const int blk0 = (int)unit[6];
#pragma unroll
  for (int j = 0; j < NBK; ++j) {
    const uint32_t w = s.kcol[(blk0 + j) * 16 + n];
    exv[j] = s.kete[(int)unit[2 + j] + min(n, xdeg)];
    if (n > xdeg) exv[j] = 0.0;
    ky[j] = 8 * (cp.tkaxis + (int)(w & 0x7f) * cp.tkrow);
    kz[j] = 8 * (2 * cp.tkaxis + (int)((w >> 7) & 0x7f) * cp.tkrow);
  }
#pragma unroll
  for (int j = 0; j < NBK; ++j)
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[j][r] = acc_zero<F32>();
  const double* xr[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) xr[r] = s.X + (r * 16 + n) * cp.xs;
  double x[NCH][4][NR], y[NBK], z[NBK], a[NBK][NR], b[NBK];
  auto fetch = [&](int4 w) {
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int t = 0; t < 4; ++t) x[c][t][r] = lds_at(xr[r], w.z + 8 * (4 * c + t));
#pragma unroll
    for (int j = 0; j < NBK; ++j) {
      y[j] = lds_at(s.kete, ky[j] + w.x);
      z[j] = lds_at(s.kete, kz[j] + w.y);
    }
  };
  auto sums = [&]() {
#pragma unroll
    for (int j = 0; j < NBK; ++j) {
#pragma unroll
      for (int r = 0; r < NR; ++r) a[j][r] = 0.0;
      fold4<NR, 0>(a[j], x[0], exv[j]);
      if constexpr (NCH > 1) fold4<NR, 4>(a[j], x[1], exv[j]);
      if constexpr (NCH > 2) fold4<NR, 8>(a[j], x[2], exv[j]);
      if constexpr (NCH > 3) fold4<NR, 12>(a[j], x[3], exv[j]);
      b[j] = y[j] * z[j];
    }
  };
  fetch(s.ktab[g < K ? g : pad]);
  int4 w = s.ktab[4 + g < K ? 4 + g : pad];
#pragma unroll 1
  for (int kk = 0; kk < K; kk += 4) {
    sums();
    fetch(w);
    w = s.ktab[kk + 8 + g < K ? kk + 8 + g : pad];
#pragma unroll
    for (int j = 0; j < NBK; ++j)
#pragma unroll
      for (int r = 0; r < NR; ++r) acc[j][r] = mfma16<F32>(a[j][r], b[j], acc[j][r]);
  }
}

template <int NBK, int NR, bool F32>
__device__ __forceinline__ void gemm2_unit(const TileParams& cp, const TileLds& s, const uint32_t* __restrict__ unit,
                                           __amdgpu_buffer_rsrc_t outq, bool first, double unscale, int lane) {
  const int g = lane >> 4, n = lane & 15;
  typename Acc<F32>::type acc[NBK][NR];
  switch ((unit[0] & 0xff) >> 2) {
    case 0: gemm2_loop<NBK, 1, NR, F32>(acc, cp, s, unit, lane); break;
    case 1: gemm2_loop<NBK, 2, NR, F32>(acc, cp, s, unit, lane); break;
    case 2:
      if constexpr (NBK == 2) gemm2_loop<NBK, 3, NR, F32>(acc, cp, s, unit, lane);
      break;
    default:
      if constexpr (NBK == 2) gemm2_loop<NBK, 4, NR, F32>(acc, cp, s, unit, lane);
      break;
  }
  uint32_t cd[NBK];
#pragma unroll
  for (int j = 0; j < NBK; ++j) {
    const uint32_t c = s.kcol[((int)unit[6] + j) * 16 + n] >> 14;
    cd[j] = (int)c < cp.ncd ? c * 8u : kNoCol;
  }
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    uint32_t row[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) row[jj] = s.orow[r * 16 + acc_row<F32>(jj, g)];
#pragma unroll
    for (int j = 0; j < NBK; ++j) {
      double v[4];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) v[jj] = acc[j][r][jj] * unscale;
      if (!first) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
          v[jj] += __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(outq, row[jj] + cd[j], 0, 0));
      }
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v[jj]), outq, row[jj] + cd[j], 0, 0);
    }
  }
}

// The second transform of the rows in X (NR blocks of 16): each wave takes its
// list of the ket's units.
template <int NR, bool F32>
__device__ __forceinline__ void gemm2_all(const TileParams& cp, const TileLds& s, const uint32_t* __restrict__ ttab,
                                          __amdgpu_buffer_rsrc_t outq, bool first, double unscale, int wave, int lane) {
  const uint32_t* lst = ttab + cp.o_klist;
  const int i1 = (int)lst[wave + 1];
#pragma unroll 1
  for (int i = (int)lst[wave]; i < i1; ++i) {
    const uint32_t* unit = ttab + cp.o_kunit + 8 * lst[9 + i];
    if ((unit[0] >> 8) == 4)
      gemm2_unit<4, NR, F32>(cp, s, unit, outq, first, unscale, lane);
    else
      gemm2_unit<2, NR, F32>(cp, s, unit, outq, first, unscale, lane);
  }
}

// All the work of one tile: quartet q, tile rt (the S::UG units UG * rt ... of
// the bra's unit list), whose integrals start at outq.  Called by every thread
// of the workgroup; ends with a barrier.  PAIRS and the shell arrays: as
// load_shells.
template <class S, bool F32, bool PAIRS>
__device__ __forceinline__ void tile_body(const TileParams& cp, unsigned char* lds, const Tables& tb,
                                          const double* __restrict__ centers, const double* __restrict__ exps,
                                          const double* __restrict__ coefs, const int32_t* __restrict__ nprim,
                                          double* __restrict__ outq, int64_t q, int rt, int tid, int wave, int lane,
                                          const double* __restrict__ kcenters, const double* __restrict__ kexps,
                                          const double* __restrict__ kcoefs, int64_t nket) {
  constexpr int RB = S::RB, NC = S::NC, XB = S::XB;
  const uint32_t* __restrict__ ttab = tb.ttab;
  const int kmax = cp.kmax, L = cp.L;
  TileLds s;
  s.sh = (double*)(lds + kTileShell);
  s.baseM = (double*)(lds + kTileBase);
  s.kpair = s.baseM + 32;
  s.orow = (uint32_t*)(s.kpair + 16);
  s.rowt = (uint16_t*)(lds + kTileRowt);
  s.rs = (uint32_t*)(lds + kTileRs);
  s.rv = (uint16_t*)(lds + kTileRv);
  s.btab = (int4*)(lds + kTileBtab);
  s.ktab = (int4*)(lds + kTileKtab);
  s.kcol = (uint32_t*)(lds + kTileKcol);
  s.kete = (double*)(lds + cp.o_kete);
  s.X = (double*)(lds + cp.o_union);
  s.zt = (double*)(lds + cp.o_zt);
  s.h = (double*)(lds + cp.o_h);
  s.g = (double*)(lds + cp.o_g);
  // two buffers in turn: the bra tables of one primitive pair; W, whose place the
  // bra tables of the next pair take
  double* const buf0 = (double*)(lds + cp.o_union);
  auto buf = [&](int i) { return (double*)((char*)buf0 + i * cp.buf); };
  // this wave's unit of rows
  const int ug = wave / S::CW, cw = wave - (wave / S::CW) * S::CW;
  const int unit0 = rt * S::UG;
  const bool active = unit0 + ug < cp.nunits;
  const uint32_t* __restrict__ bu = ttab + cp.o_bunit + 8 * (active ? unit0 + ug : unit0);
  const int ushape = (int)(bu[0] >> 8), xdeg = (int)(bu[0] & 0xff), bK = (int)bu[1];
  // the second unit's tables and F have places of their own
  s.rowf = (uint16_t*)(lds + (ug ? cp.o_row1 : kTileRowf));
  s.rf = (uint32_t*)(lds + (ug ? cp.o_row1 + kTileRowfSize : kTileRf));
  s.g += ug * RB * 64 * cp.nks;
  double* const F = (double*)(lds + cp.o_f) + ug * cp.fsize;
  int* shn = (int*)(s.sh + 12 + 8 * kmax);
  load_shells<PAIRS>(s.sh, shn, kmax, centers, exps, coefs, nprim, q, kcenters, kexps, kcoefs, nket, tid);
  // tables of this class: (u, v) of the bra and the ket in order of increasing
  // u + v, ending with a padding entry (the zero of the y table, a valid place
  // in R or X); where the rows of R start; the ket's columns
  if (tid < cp.nzt) {
    const uint32_t w = ttab[cp.o_uv + tid];
    const int u = (int)(w & 0xff), v = (int)((w >> 8) & 0xff), sum = (int)(w >> 24);
    const int at = tile_r_base(L, sum) + u * (L + 1 - sum);
    s.rowt[u * (L + 1) + v] = (uint16_t)at;
    s.rs[tid] = (uint32_t)(at | (sum << 16));
    s.rv[tid] = (uint16_t)(u | (v << 8));
    if (tid < cp.kb) s.btab[tid] = make_int4(8 * u, 8 * v, 2 * (u * (L + 1) + v), 0);
    if (tid < cp.kk) s.ktab[tid] = make_int4(8 * u, 8 * v, 8 * (tile_r_base(cp.Lk, sum) + u * (cp.Lk + 1 - sum)), 0);
#pragma unroll
    for (int x = 0; x < S::UG; ++x)
      if (unit0 + x < cp.nunits) {
        const int m0 = cp.Lb - (int)(ttab[cp.o_bunit + 8 * (unit0 + x)] & 0xff);
        if (sum <= m0 + cp.Lk) {
          const int f = tile_f_row(m0, cp.Lk, sum, u);
          ((uint16_t*)(lds + (x ? cp.o_row1 : kTileRowf)))[u * (L + 1) + v] = (uint16_t)f;
          ((uint32_t*)(lds + (x ? cp.o_row1 + kTileRowfSize : kTileRf)))[tid] =
              (uint32_t)(f | (min(cp.Lk, m0 + cp.Lk - sum) << 16));
        }
      }
  }
  if (tid == 0) s.btab[cp.kb] = make_int4(8 * (cp.Lb + 1), 0, 0, 0);
  if (tid == 64) s.ktab[cp.kk] = make_int4(8 * (cp.Lk + 1), 0, 0, 0);
  for (int i = tid; i < 16 * cp.nkblk; i += kThreads) s.kcol[i] = ttab[cp.o_kcols + i];
  // this wave's tasks of W, one per lane
  const int ntask = (cp.ntask - wave + kWaves - 1) / kWaves;
  const int task = lane < ntask ? (int)ttab[cp.o_task + wave + kWaves * lane] : 0;
  // F of this wave's unit
  const int fm = cp.Lb - xdeg + cp.Lk;
  const int fsize = tile_f_row(cp.Lb - xdeg, cp.Lk, fm + 1, 0);
  const int nks = ((xdeg + cp.Lk) >> 2) + 1;
  __syncthreads();

  const int Ka = shn[0], Kb = shn[1], Kc = shn[2], Kd = shn[3];
  if (Ka < 1 || Ka > kmax || Kb < 1 || Kb > kmax || Kc < 1 || Kc > kmax || Kd < 1 || Kd > kmax) {
    for (int ug = 0; ug < S::UG && unit0 + ug < cp.nunits; ++ug) {
      const uint32_t* bu = ttab + cp.o_bunit + 8 * (unit0 + ug);
      const int nr = 16 * (int)(((bu[0] >> 8) & 0xff) * (bu[0] >> 16));
      for (int r = wave; r < nr; r += kWaves) {
        const int ab = (int)(ttab[cp.o_brows + 16 * bu[6] + r] >> 14);
        if (ab < cp.nab)
          for (int cd = lane; cd < cp.ncd; cd += 64) outq[(int64_t)ab * cp.ncd + cd] = __builtin_nan("");
      }
    }
    __syncthreads();
    return;
  }
  // its lanes' rows
  uint32_t brow[RB], qcol[NC];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    const int nblk = (ushape & 0xff) * (ushape >> 8);
    brow[r] = ttab[cp.o_brows + 16 * ((int)bu[6] + min(r, nblk - 1)) + (lane & 15)];
  }
  // this lane's columns q
#pragma unroll
  for (int c = 0; c < NC; ++c) qcol[c] = ttab[cp.o_qcol + min(cw + S::CW * c, cp.nqb - 1) * 16 + (lane & 15)];
  const double* A = s.sh;
  const double* B = s.sh + 3;
  const double* C = s.sh + 6;
  const double* D = s.sh + 9;
  const double* ex = s.sh + 12;
  const double* co = s.sh + 12 + 4 * kmax;
  const int hs = 64 * h_steps(L);
  const double flim = far_limit(A, B);
  int eb = 0, ek = 0;
  if constexpr (!F32) tiny_exponents(s.sh, kmax, Ka, Kb, Kc, Kd, eb, ek);
  constexpr int NG = kWaves * 4 - 4;  // rows of 16 lanes outside wave 0
  const __amdgpu_buffer_rsrc_t rsrc = out_rsrc(outq, cp.nab * cp.ncd);

  StageClock clk;
  clk.start();
  for (int kl = 0; kl < Kc * Kd; ++kl) {
    const int k = kl / Kd, l = kl - (kl / Kd) * Kd;
    if (wave == 0) {
      // every lane the same values
      make_pair(s.kpair, ex[2 * kmax + k], ex[3 * kmax + l], co[2 * kmax + k], co[3 * kmax + l], C, D);
      if constexpr (F32) {
        fp32_scale(s.sh, s.kpair, kmax, Ka, Kb);
      } else {
        s.kpair[13] = ldexp(1.0, -eb);
        s.kpair[11] = ldexp(1.0, -ek);
        s.kpair[12] = ldexp(1.0, eb + ek);
      }
    }
    // What the recursion and the first transform of bra pair ij read: [0]^(m)
    // (wave 0), the 1-d tables and the per-axis tables (the other waves).
    // Runs ahead, beside the first transform of the pair before.
    auto prepare = [&](int ij, double* E, int tid, int lane) {
      const int i = ij / Kb, j = ij - (ij / Kb) * Kb;
      const double za = ex[i], zb = ex[kmax + j], zc = ex[2 * kmax + k], zd = ex[3 * kmax + l];
      const double iz = 1.0 / (za + zb), iq = 1.0 / (zc + zd);
      double pq[3];
#pragma unroll
      for (int x = 0; x < 3; ++x) pq[x] = (za * A[x] + zb * B[x]) * iz - (zc * C[x] + zd * D[x]) * iq;
      if (wave == 0) {
        if (lane <= L) {
          double ab2 = 0.0, r2 = 0.0;
#pragma unroll
          for (int x = 0; x < 3; ++x) {
            ab2 += (A[x] - B[x]) * (A[x] - B[x]);
            r2 += pq[x] * pq[x];
          }
          const double wb = co[i] * co[kmax + j] * exp(-za * zb * iz * ab2);
          s.baseM[lane] = hermite_base_m(lane, za + zb, zc + zd, r2, (wb * s.kpair[13]) * (s.kpair[1] * s.kpair[11]),
                                          tb.boys);
        }
      } else {
        build_etab_rows(E, cp.la, cp.lb, cp.tbrow, cp.tbaxis, za, zb, A, B, false, (tid >> 4) - 4, NG, lane & 15);
        build_htables(s.h, hs, tb.hcoef, pq[0], pq[1], pq[2], tid - 64, kThreads - 64, flim);
        if (wave == kWaves - 1) zero_rows(E, cp.la, cp.lb, cp.tbrow, cp.tbaxis, lane, 64);
      }
    };
    typename Acc<F32>::type acc[RB][NC];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[r][c] = acc_zero<F32>();
    ERI4_STAGE(kStPair);

#pragma unroll 1
    for (int ij = -1; ij < Ka * Kb; ++ij) {
      // an opaque thread number: what follows from it is computed where it is
      // used (the compiler would otherwise take all of it out of the loop, into
      // registers that the accumulators need)
      int ti = tid;
      asm volatile("" : "+v"(ti));
      const int la_ = ti & 63;
      double* const brae = buf(ij & 1);
      double* const W = buf((ij & 1) ^ 1);
      if (ij >= 0) {
        // zt (three blocks at most, waves 0..2) and G
        if (wave < 3) {
          const int jb = wave == 2, ub = wave == 1;
          if (L >= 16 * (jb + ub)) build_zt(s, s.h + 2 * hs, L, jb, ub, la_);
        }
        if (active) build_g(s, brae, bu, ushape & 0xff, xdeg, L, nks, cw, S::CW, la_);
        __syncthreads();
        build_w(s, W, s.h + hs, L, task, ntask, la_);
        __syncthreads();
        if (active) build_f(s, W, F, fsize, nuv(fm), ushape & 0xff, L, nks, cw, S::CW, la_);
        __syncthreads();
        ERI4_STAGE(kStR);
      }
      if (ij + 1 < Ka * Kb) {
        prepare(ij + 1, W, ti, la_);
      } else if (wave != 0) {
        // the ket tables, beside the last first transform
        build_etab_rows(s.kete, cp.lc, cp.ld, cp.tkrow, cp.tkaxis, ex[2 * kmax + k], ex[3 * kmax + l], C, D,
                        true, (ti >> 4) - 4, NG, la_ & 15);
        if (wave == kWaves - 1) zero_rows(s.kete, cp.lc, cp.ld, cp.tkrow, cp.tkaxis, la_, 64);
      }
      ERI4_STAGE(kStBoysE);
      if (ij >= 0 && active) {
        switch (ushape) {
#define U(NP, NB) \
  case (NP) | ((NB) << 8): gemm1_unit<S, NP, NB, 0, F32>(acc, s, brae, F, fsize, cp, bK, brow, qcol, la_); break;
          U(1, 1) U(1, 2)
#undef U
          default:
            gemm1_unit<S, 2, 1, 0, F32>(acc, s, brae, F, fsize, cp, bK, brow, qcol, la_);
            break;
        }
        // a third group on its own (with the first two it needs more registers than there are)
        if constexpr (RB > 2)
          if ((ushape & 0xff) == 3)
            gemm1_unit<S, 1, 1, 2, F32>(acc, s, brae, F + 2 * fsize, fsize, cp, bK, brow, qcol, la_);
      }
      __syncthreads();
      ERI4_STAGE(kStGemm1);
    }

    // [ab|q] -> LDS (over the tables and F), then the second transform: the rows
    // of a unit without the padding rows between its blocks, 32 at most, or (XB
    // == 1) one block at a time.
    const double unscale = s.kpair[12];
    int tj = tid;  // opaque, as above
    asm volatile("" : "+v"(tj));
    const int lj = tj & 63;
    auto pass = [&](auto r0c, auto r1c, int u0) {
      constexpr int R0 = decltype(r0c)::value, R1 = decltype(r1c)::value;
      if (ug >= u0 && ug < u0 + S::XU && active) {  // this wave's unit is among them
        const uint32_t vrows = bu[7];
        double* const X = s.X + (ug - u0) * 16 * XB * cp.xs;
        int first = 0;
#pragma unroll
        for (int r = R0; r < R1; ++r) {
          const int valid = (int)(vrows >> (8 * r)) & 0xff;
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const int col = (cw + S::CW * c) * 16 + (lj & 15);
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
              const int row = acc_row<F32>(jj, lj >> 4);
              if (row < valid && col < cp.nq) X[(first + row) * cp.xs + col] = acc[r][c][jj];
            }
          }
          first += valid;
        }
      }
      // zero columns; where each row goes in the output
      if (tj < 16 * XB * S::XU) {
        const int u = u0 + tj / (16 * XB), row = tj % (16 * XB);
        uint32_t to = kNoRow;
        if (unit0 + u < cp.nunits) {
          const uint32_t* xu = ttab + cp.o_bunit + 8 * (unit0 + u);
          int at = 16 * R0 + row, first = 0;  // this row's place in the unit's blocks
#pragma unroll
          for (int r = R0; r < R1; ++r) {
            if (row >= first) at = 16 * r + row - first;
            first += (int)(xu[7] >> (8 * r)) & 0xff;
          }
          if (row < first) to = (ttab[cp.o_brows + 16 * xu[6] + at] >> 14) * (8u * cp.ncd);
        }
        s.orow[tj] = to;
        for (int c = 0; c < 3; ++c) s.X[tj * cp.xs + cp.nq + c] = 0.0;
      }
      __syncthreads();
      ERI4_STAGE(kStMove);
#pragma unroll 1
      for (int u = u0; u < u0 + S::XU && unit0 + u < cp.nunits; ++u) {
        const uint32_t vrows = ttab[cp.o_bunit + 8 * (unit0 + u) + 7];
        int nrows = 0;
#pragma unroll
        for (int r = R0; r < R1; ++r) nrows += (int)(vrows >> (8 * r)) & 0xff;
        TileLds x = s;
        x.X += (u - u0) * 16 * XB * cp.xs;
        x.orow += (u - u0) * 16 * XB;
        if (XB == 2 && nrows > 16)
          gemm2_all<XB, F32>(cp, x, ttab, rsrc, kl == 0, unscale, wave, lj);
        else if (nrows > 0)
          gemm2_all<1, F32>(cp, x, ttab, rsrc, kl == 0, unscale, wave, lj);
      }
      __syncthreads();
      ERI4_STAGE(kStGemm2);
    };
    std::integral_constant<int, 0> c0;
    std::integral_constant<int, 1> c1;
    std::integral_constant<int, 2> c2;
    for (int u = 0; u < S::UG && unit0 + u < cp.nunits; u += S::XU) {
      if constexpr (XB == 2) {
        pass(c0, std::integral_constant<int, RB>{}, u);
      } else {
        pass(c0, c1, u);
        pass(c1, c2, u);
      }
    }
  }
  clk.flush(tid);
}

// Runs BODY(shape) for the class's shape (TileParams::shape).
#define ERI4_TILE_SHAPES(BODY) \
  BODY(0, 4, 3, 1) BODY(1, 4, 3, 2) BODY(2, 4, 3, 3) BODY(3, 4, 3, 4) BODY(4, 4, 2, 5) BODY(5, 8, 3, 3) \
  BODY(6, 8, 3, 4) BODY(7, 8, 2, 5) BODY(8, 8, 2, 6)

}  // namespace
}  // namespace eri4
