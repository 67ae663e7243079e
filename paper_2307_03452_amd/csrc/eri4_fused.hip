// eri4_fused.hip -- the single-class Cartesian kernels (FP64), one instance per
// kernel shape.
#include "eri4_tile.h"

namespace eri4 {

namespace {

// One workgroup = one quartet x one tile of bra rows; 8 waves.  Tiles come in
// order of decreasing work, so the grid runs over the quartets first.
template <class S>
__global__ __launch_bounds__(kThreads, 1) void eri4_fused_kernel(
    const TileParams cp, const Tables tb, const double* __restrict__ centers, const double* __restrict__ exps,
    const double* __restrict__ coefs, const int32_t* __restrict__ nprim, double* __restrict__ out, int64_t q0,
    unsigned nq) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform (SGPR)
  const int rt = (int)(blockIdx.x / nq);
  const int64_t q = q0 + (blockIdx.x - rt * nq);
  tile_body<S, false, false>(cp, lds, tb, centers, exps, coefs, nprim, out + q * (int64_t)cp.nab * cp.ncd, q, rt, tid,
                             wave, lane, nullptr, nullptr, nullptr, 0);
}

template <class S>
hipError_t launch_one(const TileParams& p, int64_t nq, hipStream_t s, const Tables& t, const double* centers,
                      const double* exps, const double* coefs, const int32_t* nprim, double* out, int64_t q0) {
  hipLaunchKernelGGL((eri4_fused_kernel<S>), dim3((unsigned)(nq * p.ntiles)), dim3(kThreads), p.lds_bytes, s, p, t,
                     centers, exps, coefs, nprim, out, q0, (unsigned)nq);
  return hipGetLastError();
}
}  // namespace

hipError_t fused_set_attrs() {
#define B(I, CW, RB, NC) (const void*)eri4_fused_kernel<TileShape<CW, RB, NC>>,
  const void* k[] = {ERI4_TILE_SHAPES(B)};
#undef B
  for (const void* f : k) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t fused_launch(const TileParams& p, int64_t nq, hipStream_t s, const Tables& t, const double* centers,
                        const double* exps, const double* coefs, const int32_t* nprim, double* out, int64_t q0) {
  switch (p.shape) {
#define B(I, CW, RB, NC) \
  case I: return launch_one<TileShape<CW, RB, NC>>(p, nq, s, t, centers, exps, coefs, nprim, out, q0);
    ERI4_TILE_SHAPES(B)
#undef B
  }
  return hipErrorInvalidValue;
}

#ifdef ERI4_STAGE_TIMERS
// Stage-timer build only: the per-stage cycle sums of the Cartesian fused
// kernels (kStCount counters in the order of the stage enum; the last one
// counts tiles), then zeroed if reset.  Returns 0, or 4 on a HIP error.
extern "C" int eri4_stage_cycles(unsigned long long* out, int reset) {
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpyFromSymbol(out, HIP_SYMBOL(g_stage_cycles), sizeof(unsigned long long) * kStCount);
  if (e == hipSuccess && reset) {
    const unsigned long long z[kStCount] = {0};
    e = hipMemcpyToSymbol(HIP_SYMBOL(g_stage_cycles), z, sizeof z);
  }
  return e == hipSuccess ? 0 : 4;
}
#endif

}  // namespace eri4
