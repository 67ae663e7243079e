// eri4_device.h -- gfx950 device code of liberi4 (kernels and their helpers).
//
// (ab|cd) over contracted Cartesian Gaussians by the matrix form of the
// McMurchie-Davidson scheme (Asadchev & Valeev, Sec. 2 and Sec. 3):
//
//   [0]^(m) = (-2 rho)^m 2 pi^(5/2) / (zp zq sqrt(zp+zq)) F_m(rho |P-Q|^2)
//   [r + 1_i]^(m) = r_i [r - 1_i]^(m+1) + (P_i - Q_i) [r]^(m+1)      eq. (md1)
//   [p|q] = (-1)^|q| [p+q]^(0)                                       eq. (pq)
//   [ab|q] = sum_p E_ab^p [p|q]                                      eq. (ab_to_hermite)
//   (ab|cd) = sum_q E_cd^q [ab|q]                                    eq. (cd_to_hermite)
//
// Here: what several kernels share (matrix products, Boys function, 1-d tables,
// Hermite index tables, shell data), the recursion of low orders, and the
// dense transforms of the low-l kernels.  The contraction is folded into the product dimension (Sec. 3),
// [p|q] is gathered from [r] in LDS and never stored, the sign (-1)^|q| is part of
// the ket tables, and the Gaussian-product prefactors and contraction coefficients
// are part of [0]^(m).  eri4_tile.h holds the grouped scheme of the larger
// classes, eri4_dense.h the solid-harmonic and exchange tiles.
//
// Everything here has internal linkage: each translation unit that launches
// one of the kernels compiles its own copy, in parallel.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <stdint.h>

#include "eri4_internal.h"
#include "eri4_launch.h"

namespace eri4 {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// device helpers
// ---------------------------------------------------------------------------

// D[16x16] += A[16x4] B[4x16] on the matrix cores, in FP64 or (F32 = true)
// with both operands rounded to FP32 and an FP32 accumulator.  Lane l holds
// A[l%16][l/16] and B[l/16][l%16]; element j of its accumulator is column l%16
// of row acc_row<F32>(j, l/16).
template <bool F32>
struct Acc {
  using type = d4;
};
template <>
struct Acc<true> {
  using type = f4;
};

template <bool F32>
__device__ __forceinline__ typename Acc<F32>::type mfma16(double a, double b, typename Acc<F32>::type c) {
  if constexpr (F32)
    return __builtin_amdgcn_mfma_f32_16x16x4f32((float)a, (float)b, c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <bool F32>
__device__ __forceinline__ int acc_row(int j, int g) {
  return F32 ? 4 * g + j : 4 * j + g;
}

template <bool F32>
__device__ __forceinline__ typename Acc<F32>::type acc_zero() {
  return typename Acc<F32>::type{0, 0, 0, 0};
}

// Stage timers (compile-time, ERI4_STAGE_TIMERS): wave 0 of each workgroup of
// the Cartesian kernels reads the shader clock after every barrier that ends a
// stage and adds the cycles since the previous read to that stage; the sums of
// all workgroups go to g_stage_cycles at the end of each tile.  The stages
// follow the paper's per-kernel breakdown (Table 2): pair data, Boys function
// and bra 1-d tables ([0]^(m) of eq. (boys)), the recursion of eq. (md1), the
// first transform (eq. (ab_to_hermite)), the tile move and ket tables, and
// the second transform with the output write (eq. (cd_to_hermite)).
enum { kStPair = 0, kStBoysE, kStR, kStGemm1, kStMove, kStGemm2, kStTiles, kStCount };
#ifdef ERI4_STAGE_TIMERS
__device__ unsigned long long g_stage_cycles[kStCount];
struct StageClock {
  unsigned long long t, acc[kStCount];
  __device__ __forceinline__ void start() {
    t = __builtin_readcyclecounter();
    for (int i = 0; i < kStCount; ++i) acc[i] = 0;
  }
  __device__ __forceinline__ void mark(int st) {
    const unsigned long long n = __builtin_readcyclecounter();
    acc[st] += n - t;
    t = n;
  }
  __device__ __forceinline__ void flush(int tid) {
    if (tid == 0) {
      acc[kStTiles] = 1;
      for (int i = 0; i < kStCount; ++i) atomicAdd(&g_stage_cycles[i], acc[i]);
    }
  }
};
#define ERI4_STAGE(st) clk.mark(st)
#else
struct StageClock {
  __device__ __forceinline__ void start() {}
  __device__ __forceinline__ void flush(int) {}
};
#define ERI4_STAGE(st) ((void)0)
#endif

// F_m(T), eq. (boys): Taylor expansion on the grid below kBoysTMax, asymptotic
// form above.  Negative T gives NaN.
__device__ double boys_fm(int m, double T, const double* __restrict__ tab) {
  if (T >= 0.0 && T < kBoysTMax) {
    const int i = (int)(T * kBoysInvH + 0.5);
    const double x = (double)i * kBoysH - T;  // -(T - T_i), exact
    const double* r = tab + (size_t)i * kBoysCols + m;
    double s = r[kBoysJ];
#pragma unroll
    for (int j = kBoysJ - 1; j >= 0; --j) s = fma(s * x, 1.0 / (double)(j + 1), r[j]);
    return s;
  }
  if (!(T >= 0.0)) return __builtin_nan("");
  // F_m(T) = Gamma(m+1/2) / (2 T^(m+1/2)); the neglected incomplete-gamma part
  // is below 1e-20 relative for T >= kBoysTMax and m <= kMaxL.
  return tab[(size_t)kBoysAsymRow * kBoysCols + m] / (pow(T, (double)m) * sqrt(T));
}

// One step of the E recursions that follow eq. (cart2herm-2):
//   E^t <- (1/(2 zp)) E^(t-1) + c E^t + (t+1) E^(t+1),  c = P-A or P-B.
template <int NT>
__device__ __forceinline__ void etab_step(double (&e)[NT], double h, double c) {
  double prev = 0.0;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const double cur = e[t];
    const double nxt = (t + 1 < NT) ? e[t + 1] : 0.0;
    e[t] = h * prev + c * cur + (double)(t + 1) * nxt;
    prev = cur;
  }
}

// Three 1-d tables (x, y, z) of one primitive pair into LDS, one wave:
// row (a,b) of axis i at E + i*taxis + (a*(lb+1)+b)*trow, entries t < trow
// (t > a+b are 0, in particular the last one).  Each axis ends with an all-zero
// row at row index (la+1)*(lb+1), used for padding rows.  alt_sign multiplies
// entry t by (-1)^t (the ket side of eq. (pq)).
// TMAX (at least la+lb+1) entries of each recursion are kept in registers.
template <int TMAX = 16>
__device__ void build_etab(double* E, int la, int lb, int trow, int taxis, double h,
                           const double* PA, const double* PB, bool alt_sign, int lane) {
  const int na = la + 1;
  for (int j = lane; j < 3 * trow; j += 64) {  // the all-zero padding rows
    const int axis = j / trow;
    E[axis * taxis + na * (lb + 1) * trow + (j - axis * trow)] = 0.0;
  }
  if (lane < 3 * na) {
    const int axis = lane / na;
    const int a = lane - axis * na;
    const double pa = PA[axis], pb = PB[axis];
    double e[TMAX];
#pragma unroll
    for (int t = 0; t < TMAX; ++t) e[t] = (t == 0) ? 1.0 : 0.0;
    for (int s = 0; s < a; ++s) etab_step(e, h, pa);
    double* base = E + axis * taxis + a * (lb + 1) * trow;
    for (int b = 0; b <= lb; ++b) {
      double* row = base + b * trow;
#pragma unroll
      for (int t = 0; t < TMAX; ++t)
        if (t < trow) row[t] = (alt_sign && (t & 1)) ? -e[t] : e[t];
      for (int t = TMAX; t < trow; ++t) row[t] = 0.0;  // beyond a+b
      if (b < lb) etab_step(e, h, pb);
    }
  }
}

// Hermite index table: ordinal -> (t,u,v) in lexicographic order over
// t+u+v <= Lh, packed t | u<<8 | v<<16 | t<<24 together with its part of the R
// offset (box: t*S2 + u*S1 + v; slab: u*S1 + v, the slab of the summed t,
// taken from bits 24.., is added per gather).  Entries n..n_alloc-1 are
// padding: E index (Lh+1, 0, 0), whose value is 0, and R index (0,0,0).
template <int NT = kThreads>
__device__ void build_htab(int2* tab, int Lh, int n, int n_alloc, int S1, int S2, bool slab, int tid) {
  const int ncol = (Lh + 1) * (Lh + 2) / 2;
  for (int c = tid; c < ncol; c += NT) {
    int t = 0, rem = c;
    while (rem >= Lh - t + 1) {
      rem -= Lh - t + 1;
      ++t;
    }
    const int u = rem;
    // triples before column (t,u): all with a smaller t, then columns u' < u of this t
    const int first = (nherm(Lh) - nherm(Lh - t)) + u * (2 * (Lh - t) + 3 - u) / 2;
    for (int v = 0; v <= Lh - t - u; ++v)
      tab[first + v] = make_int2(t | (u << 8) | (v << 16) | (t << 24), (slab ? 0 : t * S2) + u * S1 + v);
  }
  for (int i = n + tid; i < n_alloc; i += NT) tab[i] = make_int2(Lh + 1, 0);
}

// Cartesian component index -> (x, y, z) for shell l (order ax = l..0, ay = l-ax..0).
__device__ __forceinline__ void cart_of(int l, int i, int& x, int& y, int& z) {
  int n = 0;
  while ((n + 1) * (n + 2) / 2 <= i) ++n;
  z = i - n * (n + 1) / 2;
  y = n - z;
  x = l - n;
}

// [r] of total order L <= kWaveL by eq. (md1) for decreasing m, by one wave (entries e =
// lane + 64 k of the table): the waves of a workgroup need no barrier until it is done,
// where the three products of higher orders take one each.  Measured, 300 quartets of
// 81 primitive quartets of solid (ps|ps): 454 us with all waves level by level, 572
// with the products, 211 so (with 16 rows to a tile for 9).
constexpr int kWaveRE = (nherm(kWaveL) + 63) / 64;
__device__ __forceinline__ void hermite_r_wave(double* R, const double* baseM, int L, double px, double py, double pz,
                                               const uint2* entl, int lane) {
  uint2 en[kWaveRE];
#pragma unroll
  for (int k = 0; k < kWaveRE; ++k) en[k] = entl[min(lane + 64 * k, nherm(L) - 1)];
  // (memory operations of one wave on LDS run in order; the compiler keeps theirs)
  auto order = []() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  };
  order();
  if (lane == 0) R[0] = baseM[L];
  order();
#pragma unroll 1
  for (int m = L - 1; m >= 0; --m) {
    const int nact = nherm(L - m);
    double nv[kWaveRE];
#pragma unroll
    for (int k = 0; k < kWaveRE; ++k) {
      const int o1 = (int)(en[k].x >> 16), o2 = (int)(en[k].y & 0xffffu);
      const int dir = (int)((en[k].y >> 16) & 3u), ri = (int)(en[k].y >> 18);
      const double c1 = dir == 0 ? px : (dir == 1 ? py : pz);
      nv[k] = lane + 64 * k < nact ? c1 * R[o1] + (double)max(ri - 1, 0) * R[o2] : 0.0;
    }
    const double b = baseM[m];
    order();
#pragma unroll
    for (int k = 0; k < kWaveRE; ++k)
      if (lane + 64 * k < nact) R[en[k].x & 0xffffu] = k == 0 && lane == 0 ? b : nv[k];
    order();
  }
}

// Primitive-pair data, stored in LDS as 11 doubles:
//   [0] z = za + zb, [1] w = ca cb exp(-za zb / z |A-B|^2) (Gaussian product
//   prefactor times the two contraction coefficients), [2..4] P, [5..7] P-A, [8..10] P-B.
// The ket pair's slots [13] and [11] hold the power-of-two scales of the bra's and
// the ket's weights, [12] the inverse of their product (1 mostly, see tiny_exponents).

__device__ __forceinline__ void make_pair(double* out, double za, double zb, double ca, double cb,
                                          const double* A, const double* B) {
  const double z = za + zb;
  const double iz = 1.0 / z;
  double ab2 = 0.0;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    // P - A = zb (B - A) / z and P - B = za (A - B) / z, formed without the
    // cancellation of subtracting two absolute positions
    const double dd = A[i] - B[i];
    out[2 + i] = (za * A[i] + zb * B[i]) * iz;
    out[5 + i] = -zb * iz * dd;
    out[8 + i] = za * iz * dd;
    ab2 += dd * dd;
  }
  out[0] = z;
  out[1] = ca * cb * exp(-za * zb * iz * ab2);
}

// First transform over one bra primitive pair for NR row blocks x NC column
// blocks of this wave (both fixed per wave):
//   acc[r][c] += sum_p E_ab[row block r][p] * box[off(p) + off(q in block c)]
// E_ab is the product of three bra-table entries.  All LDS reads of a k step
// are issued before its MFMAs; the next p index is fetched one step ahead.
template <int NR, int NC>
__device__ __forceinline__ void gemm1_range(d4 (&acc)[NR][NC], const double* __restrict__ brae,
                                            const double* __restrict__ R, const int2* __restrict__ ptab,
                                            const int (&rowx)[NR], const int (&rowy)[NR], const int (&rowz)[NR],
                                            const int (&offq)[NC], int np4, int lane) {
  const int g = lane >> 4;
  int2 pt = ptab[g];
  for (int kk = 0; kk < np4; kk += 4) {
    const int tp = pt.x & 0xff, up = (pt.x >> 8) & 0xff, vp = (pt.x >> 16) & 0xff;
    double ex[NR], ey[NR], ez[NR], b[NC];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      ex[r] = brae[rowx[r] + tp];
      ey[r] = brae[rowy[r] + up];
      ez[r] = brae[rowz[r] + vp];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) b[c] = R[pt.y + offq[c]];
    pt = ptab[min(kk + 4, np4 - 4) + g];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const double a = ex[r] * ey[r] * ez[r];
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[r][c] = mfma16<false>(a, b[c], acc[r][c]);
    }
  }
}

// Second transform for one group of NC output column blocks (cb0, cb0+CSTRIDE, ...)
// and NR row blocks, then the output write:
//   out[ab][cd] (+)= sum_q X[ab][q] E_cd[cd][q]
// E_cd is the product of three ket-table entries (sign of eq. (pq) folded in).
template <int NR, int NC, int CSTRIDE>
__device__ __forceinline__ void gemm2_group(const ClassParams& cp, const double* __restrict__ X,
                                            const double* __restrict__ kete, const int2* __restrict__ qtab,
                                            int cb0, int row0, double* __restrict__ outq, bool first, int lane,
                                            double unscale = 1.0) {
  const int g = lane >> 4, n = lane & 15;
  int kx[NC], ky[NC], kz[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int cd = (cb0 + CSTRIDE * c) * 16 + n;
    if (cd < cp.ncd) {
      const int ic = cd / cp.nd, id = cd - (cd / cp.nd) * cp.nd;
      int cx, cy, cz, dx, dy, dz;
      cart_of(cp.lc, ic, cx, cy, cz);
      cart_of(cp.ld, id, dx, dy, dz);
      kx[c] = (cx * (cp.ld + 1) + dx) * cp.tkrow;
      ky[c] = cp.tkaxis + (cy * (cp.ld + 1) + dy) * cp.tkrow;
      kz[c] = 2 * cp.tkaxis + (cz * (cp.ld + 1) + dz) * cp.tkrow;
    } else {
      const int zr = (cp.lc + 1) * (cp.ld + 1) * cp.tkrow;
      kx[c] = zr;
      ky[c] = cp.tkaxis + zr;
      kz[c] = 2 * cp.tkaxis + zr;
    }
  }
  d4 acc[NR][NC];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[r][c] = acc_zero<false>();
  const int xs = cp.xs, nq4 = cp.nq4;
  auto load = [&](int kk, int pk, double (&aa)[NR], double (&xx)[NC], double (&yy)[NC], double (&zz)[NC]) {
    const int tq = pk & 0xff, uq = (pk >> 8) & 0xff, vq = (pk >> 16) & 0xff;
#pragma unroll
    for (int r = 0; r < NR; ++r) aa[r] = X[(r * 16 + n) * xs + kk + g];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      xx[c] = kete[kx[c] + tq];
      yy[c] = kete[ky[c] + uq];
      zz[c] = kete[kz[c] + vq];
    }
  };
  auto step = [&](const double (&aa)[NR], const double (&xx)[NC], const double (&yy)[NC], const double (&zz)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double b = xx[c] * yy[c] * zz[c];
#pragma unroll
      for (int r = 0; r < NR; ++r) acc[r][c] = mfma16<false>(aa[r], b, acc[r][c]);
    }
  };
  if constexpr (NR <= 2) {
    // the operands of step k+4 are read before the MFMAs of step k are issued
    // (measured: 1-2% on tiles of up to 32 rows; not kept for 64-row tiles,
    // whose doubled operand registers cost more than it gains)
    double a[NR], fx[NC], fy[NC], fz[NC];
    load(0, qtab[g].x, a, fx, fy, fz);
    int pk = qtab[min(4, nq4 - 4) + g].x;
    for (int kk = 0; kk < nq4; kk += 4) {
      double an[NR], fxn[NC], fyn[NC], fzn[NC];
      load(min(kk + 4, nq4 - 4), pk, an, fxn, fyn, fzn);
      pk = qtab[min(kk + 8, nq4 - 4) + g].x;
      asm volatile("" ::: "memory");  // keep the prefetch ahead of the MFMAs
      step(a, fx, fy, fz);
#pragma unroll
      for (int r = 0; r < NR; ++r) a[r] = an[r];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        fx[c] = fxn[c];
        fy[c] = fyn[c];
        fz[c] = fzn[c];
      }
    }
  } else {
    int pk = qtab[g].x;
    for (int kk = 0; kk < nq4; kk += 4) {
      double a[NR], fx[NC], fy[NC], fz[NC];
      load(kk, pk, a, fx, fy, fz);
      pk = qtab[min(kk + 4, nq4 - 4) + g].x;
      step(a, fx, fy, fz);
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int cd = (cb0 + CSTRIDE * c) * 16 + n;
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

// Power-of-two scales of the bra's and the ket's pair weights (coefficients times
// Gaussian product prefactor), whose product [0]^(m) carries.  One scale for the
// product would overflow where one side's weight is large and the other's tiny.
__device__ __forceinline__ int weight_exponent(double w) {
  return w > 0.0 && w < INFINITY ? max(-1000, min(1000, ilogb(w))) : 0;
}

// FP32 transforms: the scales that bring the largest weight of either side near 1,
// for the ket pair in kpair, so that the FP32 operands of both transforms stay
// inside FP32's exponent range for quartets with tiny integrals; into kpair[13]
// (bra) and kpair[11] (ket), what the output write multiplies by into kpair[12].
// sh: shell data (load_shells).
__device__ __forceinline__ void fp32_scale(const double* sh, double* kpair, int kmax, int Ka, int Kb) {
  const double* A = sh;
  const double* B = sh + 3;
  const double* ex = sh + 12;
  const double* co = sh + 12 + 4 * kmax;
  double ab2 = 0.0;
  for (int x = 0; x < 3; ++x) ab2 += (A[x] - B[x]) * (A[x] - B[x]);
  double wmax = 0.0;
  for (int ij = 0; ij < Ka * Kb; ++ij) {
    const int i = ij / Kb, j = ij - (ij / Kb) * Kb;
    const double za = ex[i], zb = ex[kmax + j];
    wmax = fmax(wmax, fabs(co[i] * co[kmax + j]) * exp(-za * zb / (za + zb) * ab2));
  }
  const int eb = weight_exponent(wmax), ek = weight_exponent(fabs(kpair[1]));
  kpair[13] = ldexp(1.0, -eb);
  kpair[11] = ldexp(1.0, -ek);
  kpair[12] = ldexp(1.0, eb + ek);
}

// FP64 transforms: the binary exponents of the largest weights of both sides where
// their Gaussian product prefactors are below 2^-600 together, else 0.  [0]^(m) carries
// their inverses and the output write restores them, so that the steps between work
// on normal numbers: subnormal values carry few bits, and the transforms amplify what
// their rounding loses by up to 1e6.  The largest prefactor of a pair is that of its
// smallest exponents.
__device__ __forceinline__ void tiny_exponents(const double* sh, int kmax, int Ka, int Kb, int Kc, int Kd, int& eb,
                                               int& ek) {
  const double* ex = sh + 12;
  double e[2];
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const int n1 = side ? Kc : Ka, n2 = side ? Kd : Kb;
    const double* e1 = ex + 2 * side * kmax;
    double z1 = e1[0], z2 = e1[kmax], r2 = 0.0;
    for (int i = 1; i < n1; ++i) z1 = fmin(z1, e1[i]);
    for (int i = 1; i < n2; ++i) z2 = fmin(z2, e1[kmax + i]);
    for (int x = 0; x < 3; ++x) {
      const double d = sh[6 * side + x] - sh[6 * side + 3 + x];
      r2 += d * d;
    }
    e[side] = -1.4426950408889634 * (z1 * z2 * __builtin_amdgcn_rcp(z1 + z2) * r2);  // log2 (seven digits will do)
  }
  eb = ek = 0;
  if (e[0] + e[1] < -600.0) {
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      for (int shell = 2 * side; shell < 2 * side + 2; ++shell) {
        const int n = shell == 0 ? Ka : shell == 1 ? Kb : shell == 2 ? Kc : Kd;
        double w = 0.0;
        for (int i = 0; i < n; ++i) w = fmax(w, fabs(ex[(4 + shell) * kmax + i]));
        e[side] += weight_exponent(w);
      }
    }
    eb = (int)fmax(fmin(e[0], 900.0), -900.0);
    ek = (int)fmax(fmin(e[1], 900.0), -900.0);
  }
}

// Shell data of quartet q into LDS: centres A B C D in sh[0..11], then the
// exponents and the coefficients of shells a b c d (kmax each), and the four
// contraction lengths in shn[0..3].  PAIRS: the bra pair is entry q / nket of
// the bra list (centers, exps, coefs as [n][2][...]) and the ket pair entry
// q % nket of the ket list.  Called by all threads; the caller synchronises.
template <bool PAIRS>
__device__ __forceinline__ void load_shells(double* sh, int* shn, int kmax, const double* __restrict__ centers,
                                            const double* __restrict__ exps, const double* __restrict__ coefs,
                                            const int32_t* __restrict__ nprim, int64_t q,
                                            const double* __restrict__ kcenters, const double* __restrict__ kexps,
                                            const double* __restrict__ kcoefs, int64_t nket, int tid) {
  if constexpr (!PAIRS) {
    if (tid < 12) {
      sh[tid] = centers[q * 12 + tid];
    } else if (tid < 12 + 8 * kmax) {
      const int j = tid - 12;
      sh[tid] = (j < 4 * kmax) ? exps[q * 4 * kmax + j] : coefs[q * 4 * kmax + (j - 4 * kmax)];
    } else if (tid >= 256 && tid < 260) {
      shn[tid - 256] = nprim[q * 4 + (tid - 256)];
    }
  } else {
    const int64_t ib = q / nket, ik = q - ib * nket;
    if (tid < 12) {
      sh[tid] = tid < 6 ? centers[ib * 6 + tid] : kcenters[ik * 6 + (tid - 6)];
    } else if (tid < 12 + 8 * kmax) {
      const int j = tid - 12;
      const bool ex = j < 4 * kmax;
      const int jj = ex ? j : j - 4 * kmax;  // shell jj / kmax, primitive jj % kmax
      if (jj < 2 * kmax)
        sh[tid] = (ex ? exps : coefs)[ib * 2 * kmax + jj];
      else
        sh[tid] = (ex ? kexps : kcoefs)[ik * 2 * kmax + (jj - 2 * kmax)];
    } else if (tid >= 256 && tid < 260) {
      shn[tid - 256] = nprim[q * 4 + (tid - 256)];
    }
  }
}

}  // namespace
}  // namespace eri4
