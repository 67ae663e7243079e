// eri4_coulomb_low.hip -- the Coulomb contraction of eri4_coulomb.hip for low orders
// (JLowParams): a wave takes a bra primitive pair of a quartet on its own, so that
// nothing between the recursions needs a barrier and a compute unit runs many quartets
// at once.  With one p of [p+q] dket_q per lane, in the box layout of [r].  In the
// workgroups of eri4_coulomb.hip, eight waves for every bra primitive pair, the set-up
// and the barriers of a primitive quartet took longer than its products: 4000 (ps|ss)
// of single primitives 115 us with them (80 before their recursion by products), 300 of
// three primitives per shell 229 (146); here 16 and 44.
#include "eri4_tile.h"

namespace eri4 {
namespace {

__device__ __forceinline__ void wave_order() {  // memory operations of one wave run in order; the compiler keeps theirs
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// dket of ket primitives k, l of quartet q0 + blockIdx.x (slot blockIdx.y = k kmax + l),
// one wave: dket_q = sum_cd E_cd^q D_cd, one q per lane; layout as build_dket.
__global__ __launch_bounds__(64) void coulomb_low_dket_kernel(
    const JLowParams cp, const uint32_t* __restrict__ ttab, const double* __restrict__ centers,
    const double* __restrict__ exps, const int32_t* __restrict__ nprim, const double* __restrict__ dens,
    double* __restrict__ dket, int64_t q0) {
  __shared__ double tabs[3 * 17 * 9];  // (ff|: 3 axes of 17 rows of 9, the most for l1 + l2 <= 6
  __shared__ double D[kLowAb];
  __shared__ int4 rows[kLowAb];
  const int lane = threadIdx.x;
  const int64_t iq = blockIdx.x, q = q0 + iq;
  const int kmax = cp.kmax, slot = blockIdx.y, k = slot / kmax, l = slot - (slot / kmax) * kmax;
  const int Kc = nprim[q * 4 + 2], Kd = nprim[q * 4 + 3];
  if (Kc < 1 || Kc > kmax || Kd < 1 || Kd > kmax || k >= Kc || l >= Kd) return;
  const double* e = exps + (q * 4 + 2) * kmax;
  const double* c = centers + q * 12 + 6;
  build_etab_rows(tabs, cp.lc, cp.ld, cp.tkrow, cp.tkaxis, e[k], e[kmax + l], c, c + 3, true, lane >> 4, 4, lane & 15);
  for (int i = lane; i < cp.ncd; i += 64) {
    D[i] = dens[q * cp.ncd + i];
    const int ic = i / cp.nd, id = i - (i / cp.nd) * cp.nd;
    int cx, cy, cz, dx, dy, dz;
    cart_of(cp.lc, ic, cx, cy, cz);
    cart_of(cp.ld, id, dx, dy, dz);
    rows[i] = make_int4((cx * (cp.ld + 1) + dx) * cp.tkrow, cp.tkaxis + (cy * (cp.ld + 1) + dy) * cp.tkrow,
                        2 * cp.tkaxis + (cz * (cp.ld + 1) + dz) * cp.tkrow, 0);
  }
  __syncthreads();
  double* out = dket + (iq * kmax * kmax + slot) * cp.ds;
  const int Lk = cp.Lk;
  for (int r = lane; r < nuv(Lk) * (Lk + 1); r += 64) {
    const int i = r / (Lk + 1), t = r - (r / (Lk + 1)) * (Lk + 1);
    const uint32_t w = ttab[cp.o_uv + i];
    const int u = (int)(w & 0xff), v = (int)((w >> 8) & 0xff), sum = (int)(w >> 24);
    if (t > Lk - sum) continue;
    double a = 0.0;
#pragma unroll 4
    for (int cd = 0; cd < cp.ncd; ++cd) {
      const int4 x = rows[cd];
      a = fma(tabs[x.x + t] * tabs[x.y + u] * tabs[x.z + v], D[cd], a);
    }
    out[tile_r_base(Lk, sum) + u * (Lk + 1 - sum) + t] = a;
  }
}

// J of quartet q into outJ: its bra primitive pairs dealt to the waves of the workgroup
// (wave, wave + waves, ...), whose sums are added in order.  dket: that of the quartet's
// ket pairs (slot k kmax + l).  Lengths out of range: NaN.
template <bool PAIRS>
__device__ __forceinline__ void jlow_quartet(const JLowParams& cp, unsigned char* lds, const Tables& tb,
                                             const double* __restrict__ centers, const double* __restrict__ exps,
                                             const double* __restrict__ coefs, const int32_t* __restrict__ nprim,
                                             int64_t q, const double* __restrict__ kcenters,
                                             const double* __restrict__ kexps, const double* __restrict__ kcoefs,
                                             int64_t nket, const double* __restrict__ dket,
                                             double* __restrict__ outJ, int tid, int nthreads) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = nthreads >> 6;
  const int kmax = cp.kmax, L = cp.L, Lb = cp.Lb;
  double* sh = (double*)lds;
  int* shn = (int*)(sh + 12 + 8 * kmax);
  int2* ptab = (int2*)(lds + cp.o_ptab);  // t | u << 8 | v << 16, place in [r]; (t, u, v) order
  int* qtab = (int*)(lds + cp.o_qtab);    // place in [r], in the order of dket
  uint2* entl = (uint2*)(lds + cp.o_entl);
  unsigned char* own = lds + cp.o_wave + wave * cp.wsize;
  double* baseM = (double*)own;
  double* R = (double*)(own + cp.o_r);
  double* dl = (double*)(own + cp.o_d);
  double* wl = (double*)(own + cp.o_w);
  double* E = (double*)(own + cp.o_e);
  // shells (load_shells deals them to 512 threads; here there may be 64)
  {
    const int64_t ib = PAIRS ? q / nket : q, ik = PAIRS ? q - ib * nket : q;
    for (int i = tid; i < 12 + 8 * kmax; i += nthreads) {
      if (i < 12) {
        sh[i] = PAIRS ? (i < 6 ? centers[ib * 6 + i] : kcenters[ik * 6 + i - 6]) : centers[q * 12 + i];
      } else {
        const int j = i - 12;
        const bool ex = j < 4 * kmax;
        const int jj = ex ? j : j - 4 * kmax;  // shell jj / kmax, primitive jj % kmax
        if (PAIRS)
          sh[i] = jj < 2 * kmax ? (ex ? exps : coefs)[ib * 2 * kmax + jj]
                                : (ex ? kexps : kcoefs)[ik * 2 * kmax + jj - 2 * kmax];
        else
          sh[i] = (ex ? exps : coefs)[q * 4 * kmax + jj];
      }
    }
    for (int i = tid; i < 4; i += nthreads) shn[i] = nprim[q * 4 + i];
  }
  for (int i = tid; i < nherm(L); i += nthreads) entl[i] = tb.rtab[cp.rtab_off + i];
  for (int c = tid; c < nuv(Lb); c += nthreads) {
    int t = 0, rem = c;
    while (rem >= Lb - t + 1) {
      rem -= Lb - t + 1;
      ++t;
    }
    const int u = rem, first = nherm(Lb) - nherm(Lb - t) + u * (2 * (Lb - t) + 3 - u) / 2;
    for (int v = 0; v <= Lb - t - u; ++v)
      ptab[first + v] = make_int2(t | (u << 8) | (v << 16), t * cp.S2 + u * cp.S1 + v);
  }
  for (int r = tid; r < nuv(cp.Lk) * (cp.Lk + 1); r += nthreads) {
    const int i = r / (cp.Lk + 1), t = r - (r / (cp.Lk + 1)) * (cp.Lk + 1);
    const uint32_t w = tb.ttab[cp.o_uv + i];
    const int u = (int)(w & 0xff), v = (int)((w >> 8) & 0xff), sum = (int)(w >> 24);
    if (t <= cp.Lk - sum) qtab[tile_r_base(cp.Lk, sum) + u * (cp.Lk + 1 - sum) + t] = t * cp.S2 + u * cp.S1 + v;
  }
  __syncthreads();
  const int Ka = shn[0], Kb = shn[1], Kc = shn[2], Kd = shn[3];
  if (Ka < 1 || Ka > kmax || Kb < 1 || Kb > kmax || Kc < 1 || Kc > kmax || Kd < 1 || Kd > kmax) {
    for (int i = tid; i < cp.nab; i += nthreads) outJ[i] = __builtin_nan("");
    return;
  }
  const double* ex = sh + 12;
  const double* co = sh + 12 + 4 * kmax;
  const int p0 = ptab[min(lane, cp.np - 1)].y, p1 = ptab[min(lane + 64, cp.np - 1)].y;
  double J[2] = {0.0, 0.0};
  const int nkl = Kc * Kd;
#pragma unroll 1
  for (int ij = wave; ij < Ka * Kb; ij += waves) {
    const int i = ij / Kb, j = ij - (ij / Kb) * Kb;
    build_etab_rows(E, cp.la, cp.lb, cp.tbrow, cp.tbaxis, ex[i], ex[kmax + j], sh, sh + 3, false, lane >> 4, 4,
                    lane & 15);
    double w0 = 0.0, w1 = 0.0;
#pragma unroll 1
    for (int kl = 0; kl < nkl; ++kl) {
      const int k = kl / Kd, l = kl - (kl / Kd) * Kd;
      const double* __restrict__ dq = dket + (int64_t)(k * kmax + l) * cp.ds;
      const double d0 = dq[min(lane, cp.nq - 1)], d1 = cp.nq > 64 ? dq[min(lane + 64, cp.nq - 1)] : 0.0;
      // the bra pair in lanes 0..31, the ket pair in the others
      const int ket = lane >> 5;
      const double z1 = ket ? ex[2 * kmax + k] : ex[i], z2 = ket ? ex[3 * kmax + l] : ex[kmax + j];
      const double c = ket ? co[2 * kmax + k] * co[3 * kmax + l] : co[i] * co[kmax + j];
      const double z = z1 + z2, iz = 1.0 / z;
      double p[3], pq[3], d2 = 0.0, r2 = 0.0;
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        const double s1 = sh[6 * ket + x], s2 = sh[6 * ket + 3 + x];
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
      wave_order();
      if (lane <= L) baseM[lane] = hermite_base_m(lane, z, zo, r2, w * wo, tb.boys);
      dl[lane] = d0;
      if (cp.nq > 64 && lane + 64 < cp.nq) dl[lane + 64] = d1;
      hermite_r_wave(R, baseM, L, pq[0], pq[1], pq[2], entl, lane);
#pragma unroll 4
      for (int x = 0; x < cp.nq; ++x) {
        const double dx = dl[x];
        const int at = qtab[x];
        w0 = fma(R[p0 + at], dx, w0);
        if (cp.np > 64) w1 = fma(R[p1 + at], dx, w1);
      }
      wave_order();
    }
    if (lane < cp.np) wl[lane] = w0;
    if (lane + 64 < cp.np) wl[lane + 64] = w1;
    wave_order();
    // J_ab += sum_p E_ab^p w_p, E zero above t = ax+bx, u = ay+by, v = az+bz
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int ab = lane + 64 * r;
      if (ab >= cp.nab) continue;
      const int ia = ab / cp.nb, ib = ab - (ab / cp.nb) * cp.nb;
      int ax, ay, az, bx, by, bz;
      cart_of(cp.la, ia, ax, ay, az);
      cart_of(cp.lb, ib, bx, by, bz);
      const double* ex_ = E + (ax * (cp.lb + 1) + bx) * cp.tbrow;
      const double* ey = E + cp.tbaxis + (ay * (cp.lb + 1) + by) * cp.tbrow;
      const double* ez = E + 2 * cp.tbaxis + (az * (cp.lb + 1) + bz) * cp.tbrow;
      double a = 0.0;
      for (int t = 0; t <= ax + bx; ++t) {
        const int first = nherm(Lb) - nherm(Lb - t);
        for (int u = 0; u <= ay + by; ++u) {
          const double* wt = wl + first + u * (2 * (Lb - t) + 3 - u) / 2;
          double b = 0.0;
          for (int v = 0; v <= az + bz; ++v) b = fma(ez[v], wt[v], b);
          a = fma(ex_[t] * ey[u], b, a);
        }
      }
      J[r] += a;
    }
    wave_order();
  }
  // the waves' sums, over their [r]
#pragma unroll
  for (int r = 0; r < 2; ++r)
    if (lane + 64 * r < cp.nab) R[lane + 64 * r] = J[r];
  __syncthreads();
  for (int ab = tid; ab < cp.nab; ab += nthreads) {
    double a = 0.0;
    for (int x = 0; x < waves; ++x) a += ((const double*)(lds + cp.o_wave + x * cp.wsize + cp.o_r))[ab];
    outJ[ab] = a;
  }
}

__global__ __launch_bounds__(64 * kLowWaves) void eri4_coulomb_low_kernel(
    const JLowParams cp, const Tables tb, const double* __restrict__ centers, const double* __restrict__ exps,
    const double* __restrict__ coefs, const int32_t* __restrict__ nprim, const double* __restrict__ dket,
    double* __restrict__ out, int64_t q0) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int64_t iq = blockIdx.x, q = q0 + iq;
  jlow_quartet<false>(cp, lds, tb, centers, exps, coefs, nprim, q, nullptr, nullptr, nullptr, 0,
                      dket + iq * cp.kmax * cp.kmax * cp.ds, out + q * cp.nab, threadIdx.x, blockDim.x);
}

__global__ __launch_bounds__(64 * kLowWaves) void eri4_plan_coulomb_low_kernel(
    const JLowParams* __restrict__ classes, const int2* __restrict__ items, const int64_t* __restrict__ qoff,
    const Tables tb, const double* __restrict__ centers, const double* __restrict__ exps,
    const double* __restrict__ coefs, const int32_t* __restrict__ nprim, const double* __restrict__ kcenters,
    const double* __restrict__ kexps, const double* __restrict__ kcoefs, int64_t nket,
    const int64_t* __restrict__ dkoff, const double* __restrict__ dket, double* __restrict__ jpart) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int2 it = items[blockIdx.x];
  const int64_t q = it.x;
  const JLowParams cp = classes[it.y];
  jlow_quartet<true>(cp, lds, tb, centers, exps, coefs, nprim, q, kcenters, kexps, kcoefs, nket,
                     dket + dkoff[q - (q / nket) * nket], jpart + qoff[q], threadIdx.x, blockDim.x);
}

}  // namespace

hipError_t coulomb_low_set_attrs() {
  const void* k[2] = {(const void*)eri4_coulomb_low_kernel, (const void*)eri4_plan_coulomb_low_kernel};
  for (const void* f : k) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t coulomb_low_launch(const JLowParams& p, int waves, int64_t nq, hipStream_t s, const Tables& t,
                              const double* centers, const double* exps, const double* coefs, const int32_t* nprim,
                              const double* dens, double* dket, double* out, int64_t q0) {
  hipLaunchKernelGGL(coulomb_low_dket_kernel, dim3((unsigned)nq, (unsigned)(p.kmax * p.kmax)), dim3(64), 0, s, p, t.ttab,
                     centers, exps, nprim, dens, dket, q0);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(eri4_coulomb_low_kernel, dim3((unsigned)nq), dim3(64 * waves), p.lds_bytes + (waves - 1) * p.wsize,
                     s, p, t, centers, exps, coefs, nprim, dket, out, q0);
  return hipGetLastError();
}

hipError_t plan_coulomb_low_launch(int nitems, int waves, int lds_bytes, hipStream_t s, const Tables& t,
                                   const JLowParams* classes, const int2* items, const int64_t* qoff,
                                   const int32_t* nprim, const Shells& x, const int64_t* dkoff, const double* dket,
                                   double* jpart) {
  hipLaunchKernelGGL(eri4_plan_coulomb_low_kernel, dim3((unsigned)nitems), dim3(64 * waves), lds_bytes, s, classes,
                     items, qoff, t, x.centers, x.exps, x.coefs, nprim, x.kcenters, x.kexps, x.kcoefs, x.nket, dkoff,
                     dket, jpart);
  return hipGetLastError();
}

}  // namespace eri4
