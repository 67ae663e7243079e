// eri4_plan.h -- the persistent kernel of Cartesian plans, compiled once per
// arithmetic of the transforms and source of the shells (eri4_plan64.hip and
// its siblings).
#pragma once
#include "eri4_tile.h"

namespace eri4 {
namespace {

// Work items {quartet, tile | class << 16}, largest first, taken from a device
// counter until none are left (every workgroup exits once the counter passes
// nitems).  qoff[q] is where quartet q's integrals start in out.  Each class
// brings its own shape.  F32: both transforms on FP32 matrix cores.
template <bool F32, bool PAIRS>
__global__ __launch_bounds__(kThreads, 1) void eri4_plan_kernel(
    const TileParams* __restrict__ classes, const int2* __restrict__ items, int nitems,
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
    const TileParams cp = classes[rc >> 16];
    double* oq = out + qoff[q];
    switch (cp.shape) {
#define B(I, CW, RB, NC)                                                                                            \
  case I:                                                                                                           \
    tile_body<TileShape<CW, RB, NC>, F32, PAIRS>(cp, lds, tb, centers, exps, coefs, nprim, oq, q, rc & 0xffff, tid, \
                                                 wave, lane, kcenters, kexps, kcoefs, nket);                        \
    break;
      ERI4_TILE_SHAPES(B)
#undef B
    }
  }
}

template <bool F32, bool PAIRS>
hipError_t plan_set_attrs_t() {
  return hipFuncSetAttribute((const void*)eri4_plan_kernel<F32, PAIRS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             kMaxLdsBytes - 64);
}

template <bool F32, bool PAIRS>
hipError_t plan_occupancy_t(int lds_bytes, int* per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, (const void*)eri4_plan_kernel<F32, PAIRS>, kThreads,
                                                      lds_bytes);
}

template <bool F32, bool PAIRS>
hipError_t plan_launch_t(dim3 grid, int lds_bytes, hipStream_t s, const Tables& t, const PlanArgs& a) {
  const Shells& h = a.shells;
  hipLaunchKernelGGL((eri4_plan_kernel<F32, PAIRS>), grid, dim3(kThreads), lds_bytes, s, (const TileParams*)a.classes, a.items, a.nitems,
                     a.qoff, a.nprim, a.counter, t, h.centers, h.exps, h.coefs, a.out, h.kcenters, h.kexps, h.kcoefs,
                     h.nket);
  return hipGetLastError();
}

}  // namespace
}  // namespace eri4
