// eri4_dense.hip -- Cartesian integrals of small classes by the dense tiles of
// eri4_dense.h (FP64; cart_route): single-class kernels, one instance per tile
// height and form of the recursion.
#include "eri4_dense.h"

namespace eri4 {
namespace {

// One workgroup = one quartet (q0 + blockIdx.x / nrt) x one tile of RB*16 bra rows.
template <int RB, bool LOW>
__global__ __launch_bounds__(kThreads, 1) void eri4_cart_kernel(
    const ClassParams cp, const Tables tb, const double* __restrict__ centers, const double* __restrict__ exps,
    const double* __restrict__ coefs, const int32_t* __restrict__ nprim, double* __restrict__ out, int64_t q0) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t q = q0 + blockIdx.x / cp.nrt;
  dense_tile<RB, false, false, kDenseCart, LOW>(cp, lds, tb, centers, exps, coefs, nprim,
                                      out + q * (int64_t)cp.nab * cp.ncd, q, blockIdx.x % cp.nrt, tid, wave, lane,
                                      nullptr, nullptr, nullptr, 0, nullptr, nullptr, 0, 0);
}

}  // namespace

hipError_t cart_set_attrs() {
#define K(RB, LOW) (const void*)eri4_cart_kernel<RB, LOW>
  const void* k[6] = {K(1, false), K(2, false), K(4, false), K(1, true), K(2, true), K(4, true)};
#undef K
  for (const void* f : k) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes - 64);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t cart_launch(const ClassParams& p, int64_t nq, hipStream_t s, const Tables& t, const double* centers,
                       const double* exps, const double* coefs, const int32_t* nprim, double* out, int64_t q0) {
  const dim3 grid((unsigned)(nq * p.nrt));
#define L(RB, LOW)                                                                                                   \
  hipLaunchKernelGGL((eri4_cart_kernel<RB, LOW>), grid, dim3(kThreads), p.lds_bytes, s, p, t, centers, exps, coefs, \
                     nprim, out, q0)
  if (p.L <= kWaveL) {
    if (p.rb == 4) L(4, true); else if (p.rb == 2) L(2, true); else L(1, true);
  } else {
    if (p.rb == 4) L(4, false); else if (p.rb == 2) L(2, false); else L(1, false);
  }
#undef L
  return hipGetLastError();
}

}  // namespace eri4
