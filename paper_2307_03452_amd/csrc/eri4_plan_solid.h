// eri4_plan_solid.h -- the persistent kernel of solid-harmonic plans, compiled once per
// source of the shells (eri4_plan_solid.hip, eri4_plan_solidp.hip).
#pragma once
#include "eri4_dense.h"

namespace eri4 {
namespace {

// Persistent kernel of a solid-harmonic plan: the work loop of
// eri4_plan_kernel, both transforms reading the H matrices built by
// solid_hpairs_kernel.  PAIRS: shells from the bra and ket lists, H of the
// quartet's bra entry at h + hoff[q / nket] and of its ket entry at h +
// hoff[nbra + q % nket]; otherwise shells from the quartet arrays and H at h +
// hoff[2q] (bra) and h + hoff[2q + 1] (ket).
template <bool PAIRS>
__global__ __launch_bounds__(kThreads, 1) void eri4_plan_solid_kernel(
    const ClassParams* __restrict__ classes, const int2* __restrict__ items, int nitems,
    const int64_t* __restrict__ qoff, const int32_t* __restrict__ nprim, int* __restrict__ counter,
    const Tables tb, const double* __restrict__ centers, const double* __restrict__ exps, const double* __restrict__ coefs, double* __restrict__ out,
    const double* __restrict__ kcenters, const double* __restrict__ kexps, const double* __restrict__ kcoefs,
    int64_t nket, int64_t nbra, const int64_t* __restrict__ hoff, const double* __restrict__ h) {
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
    const ClassParams cp = classes[rc >> 16];
    const int rt = rc & 0xffff;
    double* oq = out + qoff[q];
    const double* hb;
    const double* hk;
    if constexpr (PAIRS) {
      const int64_t ib = q / nket, ik = q - ib * nket;
      hb = h + hoff[ib];
      hk = h + hoff[nbra + ik];
    } else {
      hb = h + hoff[2 * (int64_t)q];
      hk = h + hoff[2 * (int64_t)q + 1];
    }
    const int64_t hbs = (int64_t)solid_pair_units(cp.la, cp.lb, false) * 16 * cp.np4;
    const int64_t hks = (int64_t)cp.ncdb * 16 * cp.nq4;
#define T(RB, SLAB, LOW)                                                                                           \
  dense_tile<RB, SLAB, PAIRS, kDenseSolid, LOW>(cp, lds, tb, centers, exps, coefs, nprim, oq, q, rt, tid, wave, lane, kcenters, \
                                     kexps, kcoefs, nket, hb, hk, hbs, hks)
    if (cp.slab) {
      if (cp.rb == 2) T(2, true, false); else T(1, true, false);
    } else if (cp.L <= kWaveL) {
      if (cp.rb == 4) T(4, false, true); else if (cp.rb == 2) T(2, false, true); else T(1, false, true);
    } else {
      if (cp.rb == 4) T(4, false, false); else if (cp.rb == 2) T(2, false, false); else T(1, false, false);
    }
#undef T
  }
}

template <bool PAIRS>
hipError_t plan_solid_set_attrs_t() {
  return hipFuncSetAttribute((const void*)eri4_plan_solid_kernel<PAIRS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             kMaxLdsBytes - 64);
}

template <bool PAIRS>
hipError_t plan_solid_occupancy_t(int lds_bytes, int* per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, (const void*)eri4_plan_solid_kernel<PAIRS>, kThreads,
                                                      lds_bytes);
}

template <bool PAIRS>
hipError_t plan_solid_launch_t(dim3 grid, int lds_bytes, hipStream_t s, const Tables& t, const PlanArgs& a, int64_t nbra,
                                 const int64_t* hoff, const double* h) {
  const Shells& x = a.shells;
  hipLaunchKernelGGL(eri4_plan_solid_kernel<PAIRS>, grid, dim3(kThreads), lds_bytes, s, (const ClassParams*)a.classes,
                     a.items, a.nitems, a.qoff, a.nprim, a.counter, t, x.centers, x.exps, x.coefs, a.out, x.kcenters,
                     x.kexps, x.kcoefs, x.nket, nbra, hoff, h);
  return hipGetLastError();
}

}  // namespace
}  // namespace eri4
