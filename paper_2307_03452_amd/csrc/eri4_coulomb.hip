// eri4_coulomb.hip -- Coulomb contraction without forming (ab|cd) (FP64,
// Cartesian): J_ab = sum_cd (ab|cd) D_cd per quartet.  The ket density is first
// taken to Hermite space per ket primitive pair, dket^kl_q = sum_cd E_cd^q D_cd
// (sign of eq. (pq) included).  Since (ab|cd) = sum_pq E_ab^p [p+q] E_cd^q
// (eqs. (abcd_to_hermite), (pq)), J_ab = sum_p E_ab^p w_p with
// w_p = sum_kl sum_q [p+q]^kl dket^kl_q: the density is carried through the
// Hermite integrals as a matrix-vector product per primitive quartet, and the
// bra transform is a matrix-vector product per bra primitive pair, instead of
// the matrix-matrix products that form [ab|q] (a J-engine).
//
// Per primitive quartet the recursion runs as in eri4_tile.h (three products).
// The matrix-vector product is then a correlation over three indices,
//   w[t,u,v] = sum_q [t+tq, u+uq, v+vq] dket[tq,uq,vq],
// bound by its LDS reads (one of [r] per multiply-add where a thread forms one
// w): a thread forms 4 t x 3 u of w and takes 3 uq at a time (jengine_mv).
// Measured, both against a recursion level by level with one w per thread:
// 512 (ii|ii) quartets of single primitives 289 -> 84 us, a 96 x 80 pair list
// of mixed classes and lengths 18.3 -> 3.88 ms.
#include "eri4_tile.h"

namespace eri4 {
namespace {

// dket of ket primitives (z1, w1) of shell lc and (z2, w2) of shell ld at
// centres c[0..5], for the density block D[Nc][Nd], in the order of W (nq
// doubles at out; eri4_internal.h).  By groups (cx, dx), as the integrals'
// second transform: over the y and z exponents of each group, then over the
// groups,
//   dket[t,u,v] = sum_(cx,dx) X^t sum_(cd in group) Y^u Z^v D_cd.
// uv: the list of (u, v).  Called by all threads of a workgroup.
__device__ __forceinline__ void build_dket(int lc, int ld, const double* __restrict__ c, double z1, double z2,
                                           const double* __restrict__ D, const uint32_t* __restrict__ uv,
                                           double* __restrict__ out, int tid) {
  __shared__ double tabs[kMaxEtab];
  __shared__ double dens[ncart(kTableLMax) * ncart(kTableLMax)];
  __shared__ double fold[nfold(kTableLMax, kTableLMax)];
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Lk = lc + ld, nd = ncart(ld), ncd = ncart(lc) * nd;
  const int trow = odd_row(Lk + 2), taxis = ((lc + 1) * (ld + 1) + 1) * trow;
  for (int i = tid; i < ncd; i += kThreads) dens[i] = D[i];
  build_etab_rows(tabs, lc, ld, trow, taxis, z1, z2, c, c + 3, true, tid >> 4, kThreads / 16, tid & 15);
  __syncthreads();
  int g = 0, off = 0;
  for (int X = 0; X <= Lk; ++X) {
    const int n = nuv(Lk - X);
    for (int x1 = max(0, X - ld); x1 <= min(lc, X); ++x1, off += n) {
      if ((g++ & (kWaves - 1)) != wave) continue;
      const int m1 = lc - x1, m2 = ld - X + x1;  // y + z of either shell
      const double* d1 = dens + (m1 * (m1 + 1) / 2) * nd + m2 * (m2 + 1) / 2;
      for (int r = lane; r < n; r += 64) {
        const int u = (int)(uv[r] & 0xff), v = (int)((uv[r] >> 8) & 0xff);
        double a = 0.0;
        for (int zc = 0; zc <= m1; ++zc) {
          const double* ey = tabs + taxis + ((m1 - zc) * (ld + 1) + m2) * trow + u;
          const double* ez = tabs + 2 * taxis + zc * (ld + 1) * trow + v;
#pragma unroll 4
          for (int zd = 0; zd <= m2; ++zd) a += d1[zc * nd + zd] * (ey[-zd * trow] * ez[zd * trow]);
        }
        fold[off + r] = a;
      }
    }
  }
  __syncthreads();
  for (int r = tid; r < nuv(Lk) * (Lk + 1); r += kThreads) {
    const int i = r / (Lk + 1), t = r - (r / (Lk + 1)) * (Lk + 1);
    const int u = (int)(uv[i] & 0xff), sum = (int)(uv[i] >> 24);
    if (t > Lk - sum) continue;
    double a = 0.0;
    int at = i;
    for (int X = 0; X <= Lk - sum; ++X) {  // E^t is zero for X < t
      const int n = nuv(Lk - X);
      for (int x1 = max(0, X - ld); x1 <= min(lc, X); ++x1, at += n)
        if (X >= t) a += tabs[(x1 * (ld + 1) + X - x1) * trow + t] * fold[at];
    }
    out[tile_r_base(Lk, sum) + u * (Lk + 1 - sum) + t] = a;
  }
}

// Batch form: one workgroup per (quartet q0 + blockIdx.x, ket pair slot
// blockIdx.y = k * kmax + l), dket at dket + (blockIdx.x * kmax^2 + slot) * cp.ds.
__global__ __launch_bounds__(kThreads, 1) void coulomb_dket_kernel(
    const JParams cp, const uint32_t* __restrict__ ttab, const double* __restrict__ centers,
    const double* __restrict__ exps, const int32_t* __restrict__ nprim, const double* __restrict__ dens,
    double* __restrict__ dket, int64_t q0) {
  const int tid = threadIdx.x;
  const int64_t iq = blockIdx.x;
  const int64_t q = q0 + iq;
  const int slot = blockIdx.y, kmax = cp.kmax;
  const int k = slot / kmax, l = slot - (slot / kmax) * kmax;
  const int Kc = nprim[q * 4 + 2], Kd = nprim[q * 4 + 3];
  if (Kc < 1 || Kc > kmax || Kd < 1 || Kd > kmax || k >= Kc || l >= Kd) return;
  const double* e = exps + (q * 4 + 2) * kmax;
  build_dket(cp.lc, cp.ld, centers + q * 12 + 6, e[k], e[kmax + l], dens + q * cp.ncd, ttab + cp.o_uv,
             dket + (iq * kmax * kmax + slot) * cp.ds, tid);
}

// List form: one workgroup per (ket list entry blockIdx.x, slot blockIdx.y);
// pl / pn hold (lc, ld) and the contraction lengths per entry, its density
// block starts at dens + doff[entry], its dket slots at dket + dkoff[entry]
// (16 * nqb doubles each).
__global__ __launch_bounds__(kThreads, 1) void coulomb_dket_pairs_kernel(
    int kmax, const uint32_t* __restrict__ uv, const int32_t* __restrict__ pl, const int32_t* __restrict__ pn,
    const double* __restrict__ kcenters, const double* __restrict__ kexps, const double* __restrict__ dens,
    const int64_t* __restrict__ doff, const int64_t* __restrict__ dkoff, double* __restrict__ dket) {
  const int tid = threadIdx.x;
  const int64_t jk = blockIdx.x;
  const int slot = blockIdx.y;
  const int k = slot / kmax, l = slot - (slot / kmax) * kmax;
  const int Kc = pn[2 * jk], Kd = pn[2 * jk + 1];
  if (Kc < 1 || Kc > kmax || Kd < 1 || Kd > kmax || k >= Kc || l >= Kd) return;
  const int lc = pl[2 * jk], ld = pl[2 * jk + 1];
  const int ds = 16 * ((nherm(lc + ld) + 15) / 16);
  const double* e = kexps + jk * 2 * kmax;
  build_dket(lc, ld, kcenters + jk * 6, e[k], e[kmax + l], dens + doff[jk], uv,
             dket + dkoff[jk] + (int64_t)slot * ds, tid);
}

// LDS of the J-engine kernels (JParams).
struct JLds {
  TileLds t;             // what the recursion's steps share with eri4_tile.h
  int* vrow;             // [r] by v: start | row stride << 16
  uint2* item;           // the ket's items: v | u << 8 | length << 16, place of its first dket
  double *d, *R, *E, *w, *wf;
};

// [r] in LDS for the matrix-vector product: the cells (u, t) of v = 2k fill the
// lower triangle of n x n cells, n = L+1-2k, those of v = 2k+1 the upper one from
// its far corner, so that u, t of one v are steps of +-S, +-1 (S = n | 1: the rows
// fall in different banks) and nothing is left empty.
__device__ __forceinline__ int jrow_start(int L, int v) {
  const int k = v >> 1;
  int base = kJPad;
  for (int j = 0; j < k; ++j) base += (L + 1 - 2 * j) * ((L + 1 - 2 * j) | 1);
  const int n = L + 1 - 2 * k;
  return (v & 1) ? base + (n - 1) * ((n | 1) + 1) : base;
}

// [r] from W: 16 rows (u, v) (the columns of the product) by 16 t at a time.
__device__ __forceinline__ void build_r(const JLds& s, const double* W, const double* h, int L, int task, int ntask,
                                        int lane) {
  const int g = lane >> 4;
  for (int i = 0; i < ntask; ++i) {
    const int w = __builtin_amdgcn_readlane(task, i);
    const int tb = w >> 12, r = (w & 0xfff) + (lane & 15), rc = min(r, nuv(L) - 1);
    const uint32_t e = s.t.rs[rc], uv = s.t.rv[rc];
    const int u = (int)(uv & 0xff), v = (int)(uv >> 8);
    const int last = r < nuv(L) ? L - u - v : -1;  // largest t
    const double* src = W + (e & 0xffff);
    const int vr = s.vrow[v], sg = (v & 1) ? -1 : 1;
    double* o = s.R + (vr & 0xffff) + sg * (u * (vr >> 16) + 16 * tb + g);
    // the block's first row is its longest
    const int tm = min(16 * tb + 15, __builtin_amdgcn_readfirstlane(last));
    const d4 acc = small_product(
        (tm >> 2) + 1 - 2 * tb, [&](int k) { return h[(4 * tb + k) * 64 + lane]; },
        [&](int k) { return src[min(8 * tb + 4 * k + g, max(last, 0))]; });
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
      if (16 * tb + 4 * jj + g <= last) o[4 * jj * sg] = acc[jj];
  }
}

// One step of jengine_mv: tq of three uq, the window of t+tq starting at PH.
template <int PH>
__device__ __forceinline__ void mv_step(double (&acc)[3][4], double (&x)[5][4], const double* (&a)[5], int sg,
                                        const double* d) {
  double dd[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) dd[j] = d[j];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    x[i][(PH + 3) & 3] = *a[i];
    a[i] += sg;
  }
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int j = 0; j < 3; ++j) acc[b][t] = fma(x[b + j][(PH + t) & 3], dd[j], acc[b][t]);
}

// acc[b][i] += w of Hermite functions (t0 + i, u0 + b, v) over the ket's items
// g, g + G, ...: an item is one vq and three uq, its dket three to a tq, zero past
// the end of a row.  A value of [r] (row u + uq of vq + v, one of five) is read
// once for the up to 3 x 4 products that use it, where a thread with one w reads
// one per product; reads past the rows (those products are with zero or of w that
// nobody reads) stay within kJPad of [r].
__device__ __forceinline__ void jengine_mv(double (&acc)[3][4], const JLds& s, int u0, int v, int t0, int g, int G,
                                           int nitems) {
#pragma unroll 1
  for (; g < nitems; g += G) {
    const uint2 it = s.item[g];
    const int V = v + (int)(it.x & 0xff), U = u0 + (int)((it.x >> 8) & 0xff);
    int n = (int)(it.x >> 16);
    const int vr = s.vrow[V], sg = (V & 1) ? -1 : 1;
    const double* a[5];
    a[0] = s.R + (vr & 0xffff) + sg * (U * (vr >> 16) + t0);
#pragma unroll
    for (int i = 1; i < 5; ++i) a[i] = a[i - 1] + sg * (vr >> 16);
    const double* d = s.d + it.y;
    double x[5][4];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        x[i][j] = *a[i];
        a[i] += sg;
      }
#pragma unroll 1
    for (; n >= 4; n -= 4, d += 12) {
      mv_step<0>(acc, x, a, sg, d);
      mv_step<1>(acc, x, a, sg, d + 3);
      mv_step<2>(acc, x, a, sg, d + 6);
      mv_step<3>(acc, x, a, sg, d + 9);
    }
    if (n > 0) mv_step<0>(acc, x, a, sg, d);
    if (n > 1) mv_step<1>(acc, x, a, sg, d + 3);
    if (n > 2) mv_step<2>(acc, x, a, sg, d + 6);
  }
}

// J of quartet q (shells from the quartet arrays, or PAIRS: from the bra and ket
// lists): all: summed over its bra primitive pairs into outJ[ab]; else that of
// bra pair (i0, j0), at outJ + (i0 Kb + j0) nab.  For each bra pair ij:
//   w_p  = sum over ket pairs kl, sum_q [p+q]^(0) dket^kl_q
//   J_ab += sum_p E_ab^p w_p
// with dket^kl at dket + (k * kmax + l) * cp.ds.  Threads: 4 t x 3 u of w (a chunk
// of the bra) by a part of the ket's items; ncp chunks (a power of two >= the
// bra's) side by side, the 512 / ncp parts are added at the end.  The bra
// transform goes by groups (ax, bx): wf[u,v] = sum_t X^t w[t,u,v] per group, then
// J_ab = sum_uv Y^u Z^v wf[u,v].  Returns without writing when the contraction
// lengths are out of range or (i0, j0) is not a pair of the quartet.  Called by all
// threads; ends with a barrier.
constexpr int kJAb = (ncart(kTableLMax) * ncart(kTableLMax) + kThreads - 1) / kThreads;  // J rows per thread

template <bool PAIRS>
__device__ __forceinline__ void jengine_quartet(
    const JParams& cp, unsigned char* lds, const Tables& tb, const double* __restrict__ centers,
    const double* __restrict__ exps, const double* __restrict__ coefs, const int32_t* __restrict__ nprim, int64_t q,
    const double* __restrict__ kcenters, const double* __restrict__ kexps, const double* __restrict__ kcoefs,
    int64_t nket, int i0, int j0, bool all, const double* __restrict__ dket, double* __restrict__ outJ, int tid,
    int wave, int lane) {
  const uint32_t* __restrict__ ttab = tb.ttab;
  const int kmax = cp.kmax, L = cp.L, Lb = cp.Lb, Lk = cp.Lk;
  JLds s;
  s.t.sh = (double*)(lds + kJShell);
  s.t.baseM = (double*)(lds + kJBase);
  s.t.rowt = (uint16_t*)(lds + kJRowt);
  s.t.rs = (uint32_t*)(lds + kJRs);
  s.t.rv = (uint16_t*)(lds + kJRv);
  s.vrow = (int*)(lds + kJVrow);
  s.item = (uint2*)(lds + kJItem);
  s.d = (double*)(lds + cp.o_d);
  s.R = (double*)(lds + cp.o_r);
  double* const W = (double*)(lds + cp.o_w);
  s.t.zt = (double*)(lds + cp.o_zt);
  s.t.h = (double*)(lds + cp.o_h);
  s.E = (double*)(lds + cp.o_w);
  s.w = (double*)(lds + cp.o_wp);
  s.wf = (double*)(lds + cp.o_wf);
  int* shn = (int*)(s.t.sh + 12 + 8 * kmax);
  load_shells<PAIRS>(s.t.sh, shn, kmax, centers, exps, coefs, nprim, q, kcenters, kexps, kcoefs, nket, tid);
  if (tid < cp.nzt) {
    const uint32_t w = ttab[cp.o_uv + tid];
    const int u = (int)(w & 0xff), v = (int)((w >> 8) & 0xff), sum = (int)(w >> 24);
    const int at = tile_r_base(L, sum) + u * (L + 1 - sum);
    s.t.rowt[u * (L + 1) + v] = (uint16_t)at;
    s.t.rs[tid] = (uint32_t)(at | (sum << 16));
    s.t.rv[tid] = (uint16_t)(u | (v << 8));
  }
  if (tid <= L) s.vrow[tid] = jrow_start(L, tid) | (((L + 1 - 2 * (tid >> 1)) | 1) << 16);
  if (tid < cp.nitems) s.item[tid] = make_uint2(ttab[cp.o_item + 2 * tid], ttab[cp.o_item + 2 * tid + 1]);
  // places between the rows of [r] and of dket are read too; what they add is 0 times
  // a value of dket or of [r], or goes to w that nobody reads
  for (int i = tid; i < cp.rsize; i += kThreads) s.R[i] = 0.0;
  for (int i = tid; i < cp.dsize; i += kThreads) s.d[i] = 0.0;
  // this wave's tasks of W and [r], one per lane
  const int ntask = (cp.ntask - wave + kWaves - 1) / kWaves;
  const int task = lane < ntask ? (int)ttab[cp.o_task + wave + kWaves * lane] : 0;
  // this thread's chunk of w and part of the items
  const int ncp = cp.ncp, chunk = tid & (ncp - 1), part = tid >> cp.ncps;
  const uint32_t cw = ttab[cp.o_chunk + min(chunk, cp.nchunk - 1)];
  const int u0 = (int)(cw & 0xff), v0 = (int)((cw >> 8) & 0xff), t0 = (int)(cw >> 16);
  __syncthreads();
  const int Ka = shn[0], Kb = shn[1], Kc = shn[2], Kd = shn[3];
  const bool ok = Ka >= 1 && Ka <= kmax && Kb >= 1 && Kb <= kmax && Kc >= 1 && Kc <= kmax && Kd >= 1 && Kd <= kmax;
  if (!ok || (!all && (i0 >= Ka || j0 >= Kb))) {
    __syncthreads();
    return;
  }
  const int ij0 = all ? 0 : i0 * Kb + j0, ij1 = all ? Ka * Kb : ij0 + 1;
  if (!all) outJ += (int64_t)ij0 * cp.nab;
  const double* A = s.t.sh;
  const double* B = s.t.sh + 3;
  const double* C = s.t.sh + 6;
  const double* D = s.t.sh + 9;
  const double* ex = s.t.sh + 12;
  const double* co = s.t.sh + 12 + 4 * kmax;
  const int hs = 64 * h_steps(L), nkl = Kc * Kd;
  int eb, ek;
  tiny_exponents(s.t.sh, kmax, Ka, Kb, Kc, Kd, eb, ek);
  eb = __builtin_amdgcn_readfirstlane(eb), ek = __builtin_amdgcn_readfirstlane(ek);
  // [0]^(m) (wave 0) and the per-axis tables (the other waves)
  auto prepare = [&](int ij, int kl, int ti) {
    const int i = ij / Kb, j = ij - (ij / Kb) * Kb, k = kl / Kd, l = kl - (kl / Kd) * Kd;
    const double za = ex[i], zb = ex[kmax + j], zc = ex[2 * kmax + k], zd = ex[3 * kmax + l];
    const double iz = 1.0 / (za + zb), iq = 1.0 / (zc + zd);
    double pq[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) pq[x] = (za * A[x] + zb * B[x]) * iz - (zc * C[x] + zd * D[x]) * iq;
    if (wave == 0) {
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
        s.t.baseM[ti & 63] = hermite_base_m(ti & 63, za + zb, zc + zd, r2, ldexp(wb, -eb) * ldexp(wk, -ek), tb.boys);
      }
    } else {
      build_htables(s.t.h, hs, tb.hcoef, pq[0], pq[1], pq[2], ti - 64, kThreads - 64);
    }
  };
  double J[kJAb];
#pragma unroll
  for (int r = 0; r < kJAb; ++r) J[r] = 0.0;
#pragma unroll 1
  for (int ij = ij0; ij < ij1; ++ij) {
    double acc[3][4];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[b][t] = 0.0;
    int ti = tid;  // opaque, as in tile_body
    asm volatile("" : "+v"(ti));
    prepare(ij, 0, ti);
    __syncthreads();
#pragma unroll 1
    for (int kl = 0; kl < nkl; ++kl) {
      int ti = tid;
      asm volatile("" : "+v"(ti));
      const int la_ = ti & 63;
      // dket to its items; zt (three blocks at most)
      const double* __restrict__ dq = dket + (int64_t)((kl / Kd) * kmax + kl - (kl / Kd) * Kd) * cp.ds;
      for (int i = ti; i < cp.nq; i += kThreads) s.d[ttab[cp.o_qpos + i]] = dq[i];
      if (L == 0) {
        if (ti == 0) s.R[s.vrow[0] & 0xffff] = s.t.baseM[0];
      } else {
        if (wave < 3) {
          const int jb = wave == 2, ub = wave == 1;
          if (L >= 16 * (jb + ub)) build_zt(s.t, s.t.h + 2 * hs, L, jb, ub, la_);
        }
        __syncthreads();
        build_w(s.t, W, s.t.h + hs, L, task, ntask, la_);
        __syncthreads();
        build_r(s, W, s.t.h, L, task, ntask, la_);
      }
      __syncthreads();
      if (kl + 1 < nkl)
        prepare(ij, kl + 1, ti);
      else if (wave != 0)  // the bra tables, over W
        build_etab_rows(s.E, cp.la, cp.lb, cp.tbrow, cp.tbaxis, ex[ij / Kb], ex[kmax + ij - (ij / Kb) * Kb], A, B,
                        false, (ti >> 4) - 4, kWaves * 4 - 4, la_ & 15);
      jengine_mv(acc, s, u0, v0, t0, part, kThreads >> cp.ncps, cp.nitems);
      __syncthreads();
    }
    // the parts of w: those within a wave, then halves of the rest (over [r])
    for (int m = ncp; m < 64; m <<= 1)
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[b][t] += __shfl_xor(acc[b][t], m);
    const int np = max(ncp, 64), col = tid & (np - 1), grp = tid / np;
    for (int h = kThreads / np / 2; h >= 1; h >>= 1) {
      if (grp >= h && grp < 2 * h) {
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
          for (int t = 0; t < 4; ++t) s.R[kJPad + ((grp - h) * 12 + b * 4 + t) * np + col] = acc[b][t];
      }
      __syncthreads();
      if (grp < h) {
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[b][t] += s.R[kJPad + (grp * 12 + b * 4 + t) * np + col];
      }
      __syncthreads();
    }
    // the places the parts took, for the next bra pair: zero again between [r]'s rows
    // (a value left there would reach w that nobody reads, be left there in turn, and
    // grow by the density with every bra pair until it is infinite, and 0 times that
    // reaches w that is read)
    if (ij + 1 < ij1)
      for (int i = tid; i < 12 * kThreads / 2; i += kThreads) s.R[kJPad + i] = 0.0;
    if (tid < cp.nchunk) {
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const int sum = u0 + b + v0;
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (sum + t0 + t <= Lb) s.w[tile_r_base(Lb, sum) + (u0 + b) * (Lb + 1 - sum) + t0 + t] = acc[b][t];
      }
    }
    __syncthreads();
    // wf[u,v] = sum_t X^t w[t,u,v] of each group (ax, bx)
    {
      int g = 0, off = 0;
      for (int X = 0; X <= Lb; ++X) {
        const int n = nuv(Lb - X);
        for (int x1 = max(0, X - cp.lb); x1 <= min(cp.la, X); ++x1, off += n) {
          if ((g++ & (kWaves - 1)) != wave) continue;
          const double* e = s.E + (x1 * (cp.lb + 1) + X - x1) * cp.tbrow;
          for (int r = lane; r < n; r += 64) {
            const int u = s.t.rv[r] & 0xff, sum = u + (s.t.rv[r] >> 8);
            const double* w = s.w + tile_r_base(Lb, sum) + u * (Lb + 1 - sum);
            double a = 0.0;
            for (int t = 0; t <= X; ++t) a += e[t] * w[t];
            s.wf[off + r] = a;
          }
        }
      }
    }
    __syncthreads();
    // J_ab += sum_uv Y^u Z^v wf[u,v], u <= ay+by, v <= az+bz
#pragma unroll 1
    for (int r = 0; r < kJAb; ++r) {
      const int ab = ti + r * kThreads;
      if (ab >= cp.nab) break;
      const int nb = ncart(cp.lb), ia = ab / nb, ib = ab - (ab / nb) * nb;
      int ax, ay, az, bx, by, bz;
      cart_of(cp.la, ia, ax, ay, az);
      cart_of(cp.lb, ib, bx, by, bz);
      int off = 0;
      for (int X = 0; X < ax + bx; ++X)
        off += nuv(Lb - X) * (min(cp.la, X) - max(0, X - cp.lb) + 1);
      off += nuv(Lb - ax - bx) * (ax - max(0, ax + bx - cp.lb));
      const double* ey = s.E + cp.tbaxis + (ay * (cp.lb + 1) + by) * cp.tbrow;
      const double* ez = s.E + 2 * cp.tbaxis + (az * (cp.lb + 1) + bz) * cp.tbrow;
      double a = 0.0;
      for (int u = 0; u <= ay + by; ++u) {
        double b = 0.0;
        int at = off + u * (u + 1) / 2 + u;  // (u, v): s (s + 1) / 2 + u, s = u + v
#pragma unroll 4
        for (int v = 0; v <= az + bz; ++v) {
          b += ez[v] * s.wf[at];
          at += u + v + 1;
        }
        a += ey[u] * b;
      }
      // (a constant index for J)
#pragma unroll
      for (int rr = 0; rr < kJAb; ++rr)
        if (rr == r) J[rr] += a;
    }
    __syncthreads();  // the tables and wf are overwritten for the next bra pair
  }
#pragma unroll
  for (int r = 0; r < kJAb; ++r)
    if (tid + r * kThreads < cp.nab) outJ[tid + r * kThreads] = ldexp(J[r], eb + ek);
}

// Batch form: one workgroup per (quartet q0 + blockIdx.x / kmax^2, bra
// primitive pair (i, j) = divmod(blockIdx.x % kmax^2, kmax)); its J^ij goes to
// part + ((blockIdx.x / kmax^2) * kmax^2 + i * Kb + j) * nab.
__global__ __launch_bounds__(kThreads, 4) void eri4_coulomb_kernel(
    const JParams cp, const Tables tb, const double* __restrict__ centers, const double* __restrict__ exps,
    const double* __restrict__ coefs, const int32_t* __restrict__ nprim, double* __restrict__ part, int64_t q0,
    const double* __restrict__ dket) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t kk2 = (int64_t)cp.kmax * cp.kmax;
  const int64_t iq = blockIdx.x / kk2;
  const int slot = (int)(blockIdx.x - iq * kk2);
  const int i = slot / cp.kmax, j = slot - (slot / cp.kmax) * cp.kmax;
  jengine_quartet<false>(cp, lds, tb, centers, exps, coefs, nprim, q0 + iq, nullptr, nullptr, nullptr, 0, i, j, false,
                         dket + iq * kk2 * cp.ds, part + iq * kk2 * cp.nab, tid, wave, lane);
}

// J of quartet q0 + blockIdx.x: the sum over its bra primitive pairs s = 0 ..
// Ka*Kb-1, in that order, of part[(blockIdx.x * kmax^2 + s) * nab ..]; NaN for
// a quartet whose contraction lengths are out of range.
__global__ void coulomb_pairsum_kernel(const JParams cp, const int32_t* __restrict__ nprim,
                                       const double* __restrict__ part, double* __restrict__ out, int64_t q0) {
  const int64_t iq = blockIdx.x, q = q0 + iq;
  const int kmax = cp.kmax;
  const int Ka = nprim[q * 4], Kb = nprim[q * 4 + 1], Kc = nprim[q * 4 + 2], Kd = nprim[q * 4 + 3];
  const bool ok = Ka >= 1 && Ka <= kmax && Kb >= 1 && Kb <= kmax && Kc >= 1 && Kc <= kmax && Kd >= 1 && Kd <= kmax;
  const int64_t kk2 = (int64_t)kmax * kmax;
  const double* p = part + iq * kk2 * cp.nab;
  for (int ab = threadIdx.x; ab < cp.nab; ab += blockDim.x) {
    double a = ok ? 0.0 : __builtin_nan("");
    if (ok)
      for (int s = 0; s < Ka * Kb; ++s) a += p[(int64_t)s * cp.nab + ab];
    out[q * cp.nab + ab] = a;
  }
}

// Persistent kernel of a Coulomb pair-list plan: work items are whole quartets
// (largest first); each sums J over all its bra primitive pairs with the dket
// of its ket entry (dket + dkoff[q % nket]) and writes it to jpart + qoff[q].
__global__ __launch_bounds__(kThreads, 4) void eri4_plan_coulomb_kernel(
    const JParams* __restrict__ classes, const int2* __restrict__ items, int nitems,
    const int64_t* __restrict__ qoff, int* __restrict__ counter, const Tables tb,
    const double* __restrict__ centers, const double* __restrict__ exps, const double* __restrict__ coefs,
    const int32_t* __restrict__ nprim, double* __restrict__ jpart, const double* __restrict__ kcenters,
    const double* __restrict__ kexps, const double* __restrict__ kcoefs, int64_t nket,
    const int64_t* __restrict__ dkoff, const double* __restrict__ dket) {
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ int next_item;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (;;) {
    if (tid == 0) next_item = atomicAdd(counter, 1);
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(next_item);
    __syncthreads();
    if (it >= nitems) break;
    const int2 w = items[it];
    const int q = __builtin_amdgcn_readfirstlane(w.x);
    const int rc = __builtin_amdgcn_readfirstlane(w.y);
    const JParams cp = classes[rc >> 16];
    const int64_t ik = q - (q / nket) * nket;
    jengine_quartet<true>(cp, lds, tb, centers, exps, coefs, nprim, q, kcenters, kexps, kcoefs, nket, 0, 0, true,
                          dket + dkoff[ik], jpart + qoff[q], tid, wave, lane);
  }
}

// J of bra entry blockIdx.x: the sum over ket entries j = 0..nket-1, in that
// order, of the J rows of quartet (i, j) (jpart + qoff[i * nket + j]), into
// out + joff[i]; nab rows from the entry's (la, lb) in pl.
__global__ void coulomb_reduce_kernel(int64_t nket, const int32_t* __restrict__ pl, const int64_t* __restrict__ qoff,
                                      const double* __restrict__ jpart, const int64_t* __restrict__ joff,
                                      double* __restrict__ out) {
  const int64_t i = blockIdx.x;
  const int nab = ncart(pl[2 * i]) * ncart(pl[2 * i + 1]);
  for (int ab = threadIdx.x; ab < nab; ab += blockDim.x) {
    double a = 0.0;
    for (int64_t j = 0; j < nket; ++j) a += jpart[qoff[i * nket + j] + ab];
    out[joff[i] + ab] = a;
  }
}

}  // namespace

hipError_t plan_coulomb_set_attrs() {
  return hipFuncSetAttribute((const void*)eri4_plan_coulomb_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                             kMaxLdsBytes - 64);
}

hipError_t plan_coulomb_occupancy(int lds_bytes, int* per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, (const void*)eri4_plan_coulomb_kernel, kThreads,
                                                      lds_bytes);
}

// The steps of a Coulomb pair-list plan (after the caller reset the work counter):
// dket of every ket entry, the persistent kernel and that of low orders, the reduction.
hipError_t plan_coulomb_launch(dim3 grid, int lds_bytes, hipStream_t s, const Tables& t, const PlanArgs& a,
                               int nbra, int kmax, int uv, const int32_t* pl, const int32_t* pn, const double* ket_dens,
                               const int64_t* doff, const int64_t* dkoff, const int64_t* joff, double* dket,
                               double* jpart, double* out, const LowItems& low) {
  const Shells& x = a.shells;
  hipLaunchKernelGGL(coulomb_dket_pairs_kernel, dim3((unsigned)x.nket, (unsigned)(kmax * kmax)), dim3(kThreads), 0, s,
                     kmax, t.ttab + uv, pl + 2 * nbra, pn + 2 * nbra, x.kcenters, x.kexps, ket_dens, doff, dkoff, dket);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.nitems > 0) {
    hipLaunchKernelGGL(eri4_plan_coulomb_kernel, grid, dim3(kThreads), lds_bytes, s, (const JParams*)a.classes, a.items,
                       a.nitems, a.qoff, a.counter, t, x.centers, x.exps, x.coefs, a.nprim, jpart, x.kcenters, x.kexps,
                       x.kcoefs, x.nket, dkoff, dket);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (low.n > 0) {
    e = plan_coulomb_low_launch(low.n, low.waves, low.lds_bytes, s, t, low.classes, low.items, a.qoff, a.nprim, x,
                                dkoff, dket, jpart);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(coulomb_reduce_kernel, dim3((unsigned)nbra), dim3(256), 0, s, x.nket, pl, a.qoff, jpart, joff,
                     out);
  return hipGetLastError();
}

hipError_t coulomb_set_attrs() {
  return hipFuncSetAttribute((const void*)eri4_coulomb_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                             kMaxLdsBytes);
}

hipError_t coulomb_dket_launch(const JParams& p, int64_t nq, hipStream_t s, const Tables& t, const double* centers,
                               const double* exps, const int32_t* nprim, const double* dens, double* dket,
                               int64_t q0) {
  const dim3 grid((unsigned)nq, (unsigned)(p.kmax * p.kmax));
  hipLaunchKernelGGL(coulomb_dket_kernel, grid, dim3(kThreads), 0, s, p, t.ttab, centers, exps, nprim, dens, dket,
                     q0);
  return hipGetLastError();
}

// J of quartets q0..q0+nq-1: the J^ij of every bra primitive pair into part
// (kmax^2 * nab doubles per quartet), then their sum per quartet into out.
hipError_t coulomb_launch(const JParams& p, int64_t nq, hipStream_t s, const Tables& t, const double* centers,
                          const double* exps, const double* coefs, const int32_t* nprim, double* part, double* out,
                          int64_t q0, const double* dket) {
  hipLaunchKernelGGL(eri4_coulomb_kernel, dim3((unsigned)(nq * p.kmax * p.kmax)), dim3(kThreads), p.lds_bytes, s, p,
                     t, centers, exps, coefs, nprim, part, q0, dket);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(coulomb_pairsum_kernel, dim3((unsigned)nq), dim3(256), 0, s, p, nprim, part, out, q0);
  return hipGetLastError();
}

}  // namespace eri4
