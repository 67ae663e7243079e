// eri4_plan_cart.h -- the persistent kernel of the quartets of Cartesian plans whose
// classes run as dense tiles (FP64, in plans of either precision), compiled once per
// source of the shells (eri4_plan_cart.hip, eri4_plan_cartp.hip).
#pragma once
#include "eri4_dense.h"

namespace eri4 {
namespace {

// As eri4_plan_kernel (eri4_plan.h), over the items of the classes that run dense.
template <bool PAIRS>
__global__ __launch_bounds__(kThreads, 1) void eri4_plan_cart_kernel(
    const ClassParams* __restrict__ classes, const int2* __restrict__ items, int nitems,
    const int64_t* __restrict__ qoff, const int32_t* __restrict__ nprim, int* __restrict__ counter, const Tables tb,
    const double* __restrict__ centers, const double* __restrict__ exps, const double* __restrict__ coefs,
    double* __restrict__ out, const double* __restrict__ kcenters, const double* __restrict__ kexps,
    const double* __restrict__ kcoefs, int64_t nket) {
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
    double* oq = out + qoff[q];
#define T(RB, LOW)                                                                                                \
  dense_tile<RB, false, PAIRS, kDenseCart, LOW>(cp, lds, tb, centers, exps, coefs, nprim, oq, q, rc & 0xffff, tid, wave, lane, \
                                      kcenters, kexps, kcoefs, nket, nullptr, nullptr, 0, 0)
    if (cp.L <= kWaveL) {
      if (cp.rb == 4) T(4, true); else if (cp.rb == 2) T(2, true); else T(1, true);
    } else {
      if (cp.rb == 4) T(4, false); else if (cp.rb == 2) T(2, false); else T(1, false);
    }
#undef T
  }
}

template <bool PAIRS>
hipError_t plan_cart_launch_t(dim3 grid, int lds_bytes, hipStream_t s, const Tables& t, const PlanArgs& a) {
  const Shells& h = a.shells;
  hipLaunchKernelGGL(eri4_plan_cart_kernel<PAIRS>, grid, dim3(kThreads), lds_bytes, s, (const ClassParams*)a.classes,
                     a.items, a.nitems, a.qoff, a.nprim, a.counter, t, h.centers, h.exps, h.coefs, a.out, h.kcenters,
                     h.kexps, h.kcoefs, h.nket);
  return hipGetLastError();
}

template <bool PAIRS>
hipError_t plan_cart_set_attrs_t() {
  return hipFuncSetAttribute((const void*)eri4_plan_cart_kernel<PAIRS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             kMaxLdsBytes - 64);
}

template <bool PAIRS>
hipError_t plan_cart_occupancy_t(int lds_bytes, int* per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, (const void*)eri4_plan_cart_kernel<PAIRS>, kThreads,
                                                      lds_bytes);
}

}  // namespace
}  // namespace eri4
