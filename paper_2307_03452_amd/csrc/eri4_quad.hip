// eri4_quad.hip -- (ab|cd) for classes whose four shells all have l <= 3, where few
// quartets or large bras leave the kernels of eri4_small.hip behind (quad_route):
// one workgroup of eight waves computes a whole quartet by the scheme of
// eri4_tile.h.
//
// With l <= 3 a group (ax, bx) of the bra has at most 16 rows, and there are at most
// 16 groups: each wave keeps the accumulators of two of them (all columns q) over
// the bra primitive pairs, so that a quartet has one recursion per primitive
// quartet.  A wave forms F of its groups and multiplies from it without waiting for
// the others; only zt and W are shared.  Of a primitive quartet of (ff|ff), 28 000
// cycles, F takes about 8 000, the first transform 6 500, the steps before them
// 6 000 and the second transform 7 000 (5 ket of 25 pairs); matrix products at their
// full rate would take 9 000: it is bound by the latency of LDS and products, with
// two waves per SIMD (a wave holds 96 accumulator registers).  1024 quartets of
// (ff|ff) with 25 primitive quartets each: 1960 -> 1205 us; 64 of them 1030 -> 300 us.
#include "eri4_tile.h"

namespace eri4 {
namespace {

// Group gi of the bra in order of increasing X = x1 + x2, then x1 (the largest
// first): x1, x2 and the number of its first row.
__device__ __forceinline__ void quad_group(int la, int lb, int gi, int& x1, int& x2, int& first) {
  first = 0;
  for (int X = 0; X <= la + lb; ++X)
    for (int a = max(0, X - lb); a <= min(la, X); ++a) {
      x1 = a;
      x2 = X - a;
      if (gi-- == 0) return;
      first += (la - x1 + 1) * (lb - x2 + 1);
    }
}

// F of the two groups of this wave, F[u][v][tq] at F0 / F1 + u su + v sv + tq: tq <= 6
// takes half of a product's rows, so that rows 0..7 are those of the first group
// and 8..15 those of the second; columns: the rows of W, 32 at a time.  G^T = HX^T
// T^T with T[tq][u] = X^(u-tq) is a product too (ht: HX^T in operand order), whose
// result comes out as the operand that F needs.  The operands of the next rows are
// read before the products of these.  e0, e1: the groups' rows of the x table; X0 <=
// X1.  one: there is no second group.
__device__ __forceinline__ void quad_f(const TileLds& s, const double* W, double* F0, double* F1, int su, int sv,
                                       const double (&ht)[4], const double* e0, const double* e1, int X0, int X1,
                                       bool one, int Lk, int L, int lane) {
  const int g = lane >> 4, n = lane & 15;
  const int nks = (((one ? X0 : X1) + Lk) >> 2) + 1, nrow = nuv(L - X0);
  const int X = n < 8 ? X0 : X1;
  const double* ex = n < 8 ? e0 : e1;
  double x[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int t = 4 * k + g - (n & 7);
    const double v = ex[max(0, min(t, X))];
    x[k] = t >= 0 && t <= X ? v : 0.0;
  }
  uint32_t e[2], uv[2];
  double bn[2][4];
  auto fetch = [&](int r0) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = min(r0 + 16 * h + n, nrow - 1);
      e[h] = s.rs[r];
      uv[h] = s.rv[r];
    }
  };
  auto fetch_w = [&]() {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int last = L - (int)(e[h] >> 16);
      const double* w = W + (e[h] & 0xffff);
#pragma unroll
      for (int k = 0; k < 4; ++k) bn[h][k] = w[min(4 * k + g, last)];
    }
  };
  fetch(0);
  d4 a = acc_zero<false>();
#pragma unroll
  for (int k = 0; k < 4; ++k) a = mfma16<false>(ht[k], x[k], a);
  fetch_w();
#pragma unroll 1
  for (int r0 = 0; r0 < nrow; r0 += 32) {
    double b[2][4];
    int f0[2], f1[2], o[2], nk = 0;  // last tq of either group
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int sum = (int)(e[h] >> 16);
      f0[h] = r0 + 16 * h + n < nrow ? min(Lk, L - X0 - sum) : -1;
      f1[h] = r0 + 16 * h + n < nrow && !one ? min(Lk, L - X1 - sum) : -1;
      o[h] = (int)(uv[h] & 0xff) * su + (int)(uv[h] >> 8) * sv + g;
      // the first row is the longest
      if (h == 0) nk = min(nks, (__builtin_amdgcn_readfirstlane(L - sum) >> 2) + 1);
#pragma unroll
      for (int k = 0; k < 4; ++k) b[h][k] = bn[h][k];
    }
    fetch(r0 + 32);
    d4 acc[2] = {acc_zero<false>(), acc_zero<false>()};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k < nk) {
        acc[0] = mfma16<false>(a[k], b[0][k], acc[0]);
        acc[1] = mfma16<false>(a[k], b[1][k], acc[1]);
      }
    fetch_w();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        if (4 * jj + g <= f0[h]) F0[o[h] + 4 * jj] = acc[h][jj];
        if (4 * jj + g <= f1[h]) F1[o[h] + 4 * jj] = acc[h][jj + 2];
      }
  }
}

// acc[c] += sum_uv Y^u Z^v F[u + uq][v + vq][tq] of one group's 16 rows, K values of
// (u, v); offq: bytes of the lane's columns q in F, rowy, rowz: of its row in the
// tables.  As gemm1_unit, with F in linear places.
template <int NC>
__device__ __forceinline__ void quad_gemm1(d4 (&acc)[NC], const TileLds& s, const double* brae, const double* F,
                                           int rowy, int rowz, const int (&offq)[NC], int K, int pad, int lane) {
  const int g = lane >> 4;
  double y, z, b[NC];
  auto fetch = [&](int4 w) {
    y = lds_at(brae, rowy + w.x);
    z = lds_at(brae, rowz + w.y);
#pragma unroll
    for (int c = 0; c < NC; ++c) b[c] = lds_at(F, w.z + offq[c]);
  };
  fetch(s.btab[g < K ? g : pad]);
  int4 w = s.btab[4 + g < K ? 4 + g : pad];
#pragma unroll 1
  for (int kk = 0; kk < K; kk += 4) {
    const double a = y * z;
    double bb[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) bb[c] = b[c];
    fetch(w);
    w = s.btab[kk + 8 + g < K ? kk + 8 + g : pad];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = mfma16<false>(a, bb[c], acc[c]);
  }
}

// One quartet (q0 + blockIdx.x) per workgroup; NC: 16-wide column blocks of [ab|q].
template <int NC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void eri4_quad_kernel(
    const QuadParams qp, const Tables tb, const double* __restrict__ centers, const double* __restrict__ exps,
    const double* __restrict__ coefs, const int32_t* __restrict__ nprim, double* __restrict__ out, int64_t q0) {
  extern __shared__ __align__(16) unsigned char lds[];
  const TileParams& cp = qp.t;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t q = q0 + blockIdx.x;
  const int kmax = cp.kmax, L = cp.L, Lb = cp.Lb, Lk = cp.Lk, la = cp.la, lb = cp.lb;
  double* outq = out + q * (int64_t)cp.nab * cp.ncd;
  const uint32_t* __restrict__ ttab = tb.ttab;
  TileLds s;
  s.sh = (double*)lds;
  s.baseM = (double*)(lds + qp.o_base);
  s.rowt = (uint16_t*)(lds + qp.o_rowt);
  s.rs = (uint32_t*)(lds + qp.o_rs);
  s.rv = (uint16_t*)(lds + qp.o_rv);
  s.btab = (int4*)(lds + qp.o_btab);
  s.ktab = (int4*)(lds + qp.o_ktab);
  s.kcol = (uint32_t*)(lds + qp.o_kcol);
  s.orow = (uint32_t*)(lds + qp.o_orow);
  s.kete = (double*)(lds + qp.o_kete);
  s.zt = (double*)(lds + qp.o_zt);
  s.X = (double*)(lds + qp.o_f);
  double* const W = (double*)(lds + qp.o_w);
  double* const F = (double*)(lds + qp.o_f) + wave * (qp.fsize + qp.fsize1);
  const int hs = 64 * h_steps(L);
  const int sv = odd_row(Lk + 1), su = sv * (L + 1);  // strides of F
  auto brae_of = [&](int i) { return (double*)(lds + qp.o_brae) + (i & 1) * 3 * cp.tbaxis; };
  auto h_of = [&](int i) { return (double*)(lds + qp.o_h) + (i & 1) * 3 * hs; };
  int* shn = (int*)(s.sh + 12 + 8 * kmax);
  load_shells<false>(s.sh, shn, kmax, centers, exps, coefs, nprim, q, nullptr, nullptr, nullptr, 0, tid);
  if (tid < cp.nzt) {
    const uint32_t w = ttab[cp.o_uv + tid];
    const int u = (int)(w & 0xff), v = (int)((w >> 8) & 0xff), sum = (int)(w >> 24);
    const int at = tile_r_base(L, sum) + u * (L + 1 - sum);
    s.rowt[u * (L + 1) + v] = (uint16_t)at;
    s.rs[tid] = (uint32_t)(at | (sum << 16));
    s.rv[tid] = (uint16_t)(u | (v << 8));
    if (tid < cp.kb) s.btab[tid] = make_int4(8 * u, 8 * v, 8 * (u * su + v * sv), 0);
    if (tid < cp.kk) s.ktab[tid] = make_int4(8 * u, 8 * v, 8 * (tile_r_base(Lk, sum) + u * (Lk + 1 - sum)), 0);
  }
  if (tid == 0) s.btab[cp.kb] = make_int4(8 * (Lb + 1), 0, 0, 0);
  if (tid == 64) s.ktab[cp.kk] = make_int4(8 * (Lk + 1), 0, 0, 0);
  for (int i = tid; i < 16 * cp.nkblk; i += kThreads) s.kcol[i] = ttab[cp.o_kcols + i];
  // where each row goes in the output, rows by groups
  const int ng = (la + 1) * (lb + 1);
  if (tid < 16 * ng) {
    int x1, x2, first;
    quad_group(la, lb, tid >> 4, x1, x2, first);
    const int m1 = la - x1, m2 = lb - x2, i = tid & 15;
    if (i < (m1 + 1) * (m2 + 1)) {
      const int z1 = i / (m2 + 1), z2 = i - z1 * (m2 + 1);
      s.orow[first + i] = (uint32_t)(((m1 * (m1 + 1) / 2 + z1) * ncart(lb) + m2 * (m2 + 1) / 2 + z2) * 8 * cp.ncd);
    }
  }
  if (tid >= cp.nab && tid < (cp.nab + 31) / 32 * 32) s.orow[tid] = kNoRow;
  zero_rows(brae_of(0), la, lb, cp.tbrow, cp.tbaxis, tid, kThreads);
  zero_rows(brae_of(1), la, lb, cp.tbrow, cp.tbaxis, tid, kThreads);
  zero_rows(s.kete, cp.lc, cp.ld, cp.tkrow, cp.tkaxis, tid, kThreads);
  __syncthreads();
  const int Ka = shn[0], Kb = shn[1], Kc = shn[2], Kd = shn[3];
  if (Ka < 1 || Ka > kmax || Kb < 1 || Kb > kmax || Kc < 1 || Kc > kmax || Kd < 1 || Kd > kmax) {
    for (int i = tid; i < cp.nab * cp.ncd; i += kThreads) outq[i] = __builtin_nan("");
    return;
  }
  // this wave's groups: the w-th largest and the w-th of the other end
  int rowy[2], rowz[2], offq[NC];
  int gX[2], grow[2], gfirst[2], gn[2];  // X, row of the x table, first row, rows (0: none)
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int gi = r ? 2 * kWaves - 1 - wave : wave;
    int x1, x2, first;
    quad_group(la, lb, min(gi, ng - 1), x1, x2, first);
    const int n2 = lb - x2 + 1, m = (la - x1 + 1) * n2, i = lane & 15, z1 = i / n2, z2 = i - z1 * n2;
    const int zero = (la + 1) * (lb + 1);
    rowy[r] = 8 * (cp.tbaxis + (i < m ? (la - x1 - z1) * (lb + 1) + lb - x2 - z2 : zero) * cp.tbrow);
    rowz[r] = 8 * (2 * cp.tbaxis + (i < m ? z1 * (lb + 1) + z2 : zero) * cp.tbrow);
    gX[r] = x1 + x2;
    grow[r] = (x1 * (lb + 1) + x2) * cp.tbrow;
    gfirst[r] = first;
    gn[r] = gi < ng ? m : 0;
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const uint32_t w = ttab[cp.o_qcol + c * 16 + (lane & 15)];
    const int u = (int)((w >> 8) & 0xff), v = (int)(w >> 16) - u;
    offq[c] = 8 * ((int)(w & 0xff) + u * su + v * sv);
  }
  const int ntask = wave < cp.ntask ? 1 : 0;  // of W (six at most)
  const int task = ntask ? (int)ttab[cp.o_task + wave] : 0;
  const double* A = s.sh;
  const double* B = s.sh + 3;
  const double* C = s.sh + 6;
  const double* D = s.sh + 9;
  const double* ex = s.sh + 12;
  const double* co = s.sh + 12 + 4 * kmax;
  const double flim = far_limit(A, B);
  int eb, ek;
  tiny_exponents(s.sh, kmax, Ka, Kb, Kc, Kd, eb, ek);
  eb = __builtin_amdgcn_readfirstlane(eb), ek = __builtin_amdgcn_readfirstlane(ek);
  const double unscale = ldexp(1.0, eb + ek);
  const __amdgpu_buffer_rsrc_t rsrc = out_rsrc(outq, cp.nab * cp.ncd);
  const int nij = Ka * Kb;
  int step = 0;  // primitive quartets so far: which of the two buffers

  // [0]^(m) (the last wave, whose groups are the smallest), the bra and the
  // per-axis tables (the others) of primitive quartet (ij, kl)
  auto prepare = [&](int ij, int kl, int st, int ti) {
    const int i = ij / Kb, j = ij - (ij / Kb) * Kb, k = kl / Kd, l = kl - (kl / Kd) * Kd;
    const double za = ex[i], zb = ex[kmax + j], zc = ex[2 * kmax + k], zd = ex[3 * kmax + l];
    const double iz = 1.0 / (za + zb), iq = 1.0 / (zc + zd);
    double pq[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) pq[x] = (za * A[x] + zb * B[x]) * iz - (zc * C[x] + zd * D[x]) * iq;
    if (wave == kWaves - 1) {
      if ((ti & 63) <= L) {
        double ab2 = 0.0, cd2 = 0.0, r2 = 0.0;
#pragma unroll
        for (int x = 0; x < 3; ++x) {
          ab2 += (A[x] - B[x]) * (A[x] - B[x]);
          cd2 += (C[x] - D[x]) * (C[x] - D[x]);
          r2 += pq[x] * pq[x];
        }
        const double wb = co[i] * co[kmax + j] * exp(-za * zb * iz * ab2);
        const double wk = co[2 * kmax + k] * co[3 * kmax + l] * exp(-zc * zd * iq * cd2);
        s.baseM[ti & 63] = hermite_base_m(ti & 63, za + zb, zc + zd, r2, ldexp(wb, -eb) * ldexp(wk, -ek), tb.boys);
      }
    } else {
      build_htables<false>(h_of(st), hs, tb.hcoef, pq[0], pq[1], pq[2], ti, kThreads - 64, flim);
      build_etab_rows(brae_of(st), la, lb, cp.tbrow, cp.tbaxis, za, zb, A, B, false, ti >> 4, kWaves * 4 - 4, ti & 15);
    }
  };
  prepare(0, 0, 0, tid);

#pragma unroll 1
  for (int kl = 0; kl < Kc * Kd; ++kl) {
    d4 acc[2][NC];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[r][c] = acc_zero<false>();
#pragma unroll 1
    for (int ij = 0; ij < nij; ++ij, ++step) {
      int ti = tid;  // opaque, as in tile_body
      asm volatile("" : "+v"(ti));
      const int la_ = ti & 63;
      s.h = h_of(step);
      __syncthreads();
      if (wave == 0) build_zt(s, s.h + 2 * hs, L, 0, 0, la_);
      __syncthreads();
      build_w(s, W, s.h + hs, L, task, ntask, la_);
      __syncthreads();
      if (ij + 1 < nij) {
        prepare(ij + 1, kl, step + 1, ti);
      } else {
        if (kl + 1 < Kc * Kd) prepare(0, kl + 1, step + 1, ti);
        if (wave != kWaves - 1)
          build_etab_rows(s.kete, cp.lc, cp.ld, cp.tkrow, cp.tkaxis, ex[2 * kmax + kl / Kd],
                          ex[3 * kmax + kl - (kl / Kd) * Kd], C, D, true, ti >> 4, kWaves * 4 - 4, la_ & 15);
      }
      const double* brae = brae_of(step);
      // HX^T: row j of lane % 16, u = 4 k + lane / 16 (zero above L: j <= u)
      double ht[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int j = la_ & 15, u = 4 * k + (la_ >> 4);
        const double h = s.h[(min(j, L) >> 2) * 64 + (j & 3) * 16 + min(u, 15)];
        ht[k] = j <= L && u <= L ? h : 0.0;
      }
      if (gn[0] > 0) {
        quad_f(s, W, F, F + qp.fsize, su, sv, ht, brae + grow[0], brae + grow[1], gX[0], gX[1], gn[1] == 0, Lk, L,
               la_);
        quad_gemm1<NC>(acc[0], s, brae, F, rowy[0], rowz[0], offq, nuv(Lb - gX[0]), cp.kb, la_);
        if (gn[1] > 0)
          quad_gemm1<NC>(acc[1], s, brae, F + qp.fsize, rowy[1], rowz[1], offq, nuv(Lb - gX[1]), cp.kb, la_);
      }
    }
    __syncthreads();
    // [ab|q] -> LDS (over F), rows by groups; then the second transform: the ket's
    // units by blocks of 32 rows, dealt to the waves in order of decreasing cost
    int tj = tid;
    asm volatile("" : "+v"(tj));
    const int lj = tj & 63;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int i = acc_row<false>(jj, lj >> 4);
        if (i < gn[r]) {
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const int col = c * 16 + (lj & 15);
            if (col < cp.nq) s.X[(gfirst[r] + i) * cp.xs + col] = acc[r][c][jj];
          }
        }
      }
    const int nrp = (cp.nab + 31) >> 5;
    for (int i = tj; i < 96 * nrp; i += kThreads) s.X[(i / 3) * cp.xs + cp.nq + i % 3] = 0.0;
    __syncthreads();
#pragma unroll 1
    for (int i = wave; i < qp.nkunits * nrp; i += kWaves) {
      const int unit = i / nrp, row0 = 32 * (i - unit * nrp);
      const uint32_t* u = ttab + cp.o_kunit + 8 * unit;
      TileLds x = s;
      x.X += row0 * cp.xs;
      x.orow += row0;
      const bool four = (u[0] >> 8) == 4;
      if (cp.nab - row0 > 16) {
        if (four)
          gemm2_unit<4, 2, false>(cp, x, u, rsrc, kl == 0, unscale, lj);
        else
          gemm2_unit<2, 2, false>(cp, x, u, rsrc, kl == 0, unscale, lj);
      } else {
        if (four)
          gemm2_unit<4, 1, false>(cp, x, u, rsrc, kl == 0, unscale, lj);
        else
          gemm2_unit<2, 1, false>(cp, x, u, rsrc, kl == 0, unscale, lj);
      }
    }
    __syncthreads();
  }
}

template <int NC>
hipError_t quad_launch_t(const QuadParams& p, int64_t nq, hipStream_t s, const Tables& t, const double* centers,
                         const double* exps, const double* coefs, const int32_t* nprim, double* out, int64_t q0) {
  hipLaunchKernelGGL(eri4_quad_kernel<NC>, dim3((unsigned)nq), dim3(kThreads), p.lds_bytes, s, p, t, centers, exps,
                     coefs, nprim, out, q0);
  return hipGetLastError();
}

}  // namespace

hipError_t quad_set_attrs() {
  const void* k[6] = {(const void*)eri4_quad_kernel<1>, (const void*)eri4_quad_kernel<2>,
                      (const void*)eri4_quad_kernel<3>, (const void*)eri4_quad_kernel<4>,
                      (const void*)eri4_quad_kernel<5>, (const void*)eri4_quad_kernel<6>};
  for (const void* f : k) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t quad_launch(const QuadParams& p, int64_t nq, hipStream_t s, const Tables& t, const double* centers,
                       const double* exps, const double* coefs, const int32_t* nprim, double* out, int64_t q0) {
  switch (p.t.nqb) {
#define L(NC) \
  case NC: return quad_launch_t<NC>(p, nq, s, t, centers, exps, coefs, nprim, out, q0);
    L(1) L(2) L(3) L(4) L(5) L(6)
#undef L
    default: return hipErrorInvalidValue;
  }
}

}  // namespace eri4
