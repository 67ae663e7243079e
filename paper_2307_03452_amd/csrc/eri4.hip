// eri4.hip -- host side of liberi4's C ABI (gfx950), and the small stage
// kernels.  The integral and contraction kernels are compiled in units of their
// own (eri4_launch.h).
//
// (ab|cd) over contracted Cartesian Gaussians by the matrix form of the
// McMurchie-Davidson scheme (Asadchev & Valeev, Sec. 2 and Sec. 3).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "eri4.h"
#include "eri4_dense.h"
#include "eri4_internal.h"
#include "eri4_launch.h"

namespace eri4 {
void make_boys_table(std::vector<double>& tab);
void make_rtabs(std::vector<uint32_t>& tab, std::vector<int>& start);
void make_solid_table(std::vector<double>& tab);
void make_tile_tables(std::vector<uint32_t>& tab, std::vector<double>& hcoef, TileTableIndex& ix);
void solid_dense(int l, double* C);

__global__ void reset_counter_kernel(int* counter) {
  if (threadIdx.x < 2) counter[threadIdx.x] = 0;
}

// out[0..n) = 0 (a kernel rather than a memset, so that graph captures of the
// calls that use it stay correct on replay)
__global__ void zero_fill_kernel(double* __restrict__ out, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = 0.0;
}

// ---------------------------------------------------------------------------
// stage kernels: the device code of the integral kernels for one stage each
// ---------------------------------------------------------------------------

__global__ void boys_kernel(int mmax, int64_t n, const double* __restrict__ T, double* __restrict__ F,
                            const double* __restrict__ tab) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = n * (mmax + 1);
  if (g >= total) return;
  const int64_t i = g / (mmax + 1);
  const int m = (int)(g - i * (mmax + 1));
  F[g] = boys_fm(m, T[i], tab);
}

// Places in LDS (bytes) of the stage kernel of the recursion.
struct StageR {
  int L, ntask, o_uv, o_task, rtab_off;
  int o_rowt, o_rs, o_rv, o_box, o_zt, o_h, lds_bytes;
};

// [r] of one primitive quartet as the tiles of eri4_dense.h form it: of orders up to
// kWaveL by one wave, above by the three products.
template <bool SLAB>
__global__ __launch_bounds__(kThreads, 1) void hermite_r_kernel(
    const StageR sp, const Tables tb, const double* __restrict__ zp, const double* __restrict__ zq,
    const double* __restrict__ P, const double* __restrict__ Q, double* __restrict__ R) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t it = blockIdx.x;
  const int L = sp.L, n1 = L + 1, S1 = box_s1(L), S2 = box_s2(L);
  DenseLds s;
  s.t.baseM = (double*)lds;
  s.t.rowt = (uint16_t*)(lds + sp.o_rowt);
  s.t.rs = (uint32_t*)(lds + sp.o_rs);
  s.t.rv = (uint16_t*)(lds + sp.o_rv);
  s.t.zt = (double*)(lds + sp.o_zt);
  s.t.h = (double*)(lds + sp.o_h);
  s.box = (double*)(lds + sp.o_box);
  s.entl = (uint2*)(lds + sp.o_rowt);
  const bool low = L <= kWaveL;
  double pq[3], r2 = 0.0;
  for (int x = 0; x < 3; ++x) {
    pq[x] = P[it * 3 + x] - Q[it * 3 + x];
    r2 += pq[x] * pq[x];
  }
  if (tid <= L) s.t.baseM[tid] = hermite_base_m(tid, zp[it], zq[it], r2, 1.0, tb.boys);
  const int hs = 64 * h_steps(L);
  int ntask = 0, task = 0;
  if (low) {
    if (tid < nherm(L)) s.entl[tid] = tb.rtab[sp.rtab_off + tid];
  } else {
    if (tid < nuv(L)) w_row<SLAB>(s.t, tb.ttab + sp.o_uv, L, S1, tid);
    ntask = (sp.ntask - wave + kWaves - 1) / kWaves;
    task = lane < ntask ? (int)tb.ttab[sp.o_task + wave + kWaves * lane] : 0;
    if (wave > 0) build_htables(s.t.h, hs, tb.hcoef, pq[0], pq[1], pq[2], tid - 64, kThreads - 64);
  }
  __syncthreads();
  if (low) {
    if (wave == 0) hermite_r_wave(s.box, s.t.baseM, L, pq[0], pq[1], pq[2], s.entl, lane);
  } else {
    if (wave < 3) {
      const int jb = wave == 2, ub = wave == 1;
      if (L >= 16 * (jb + ub)) build_zt(s.t, s.t.h + 2 * hs, L, jb, ub, lane);
    }
    __syncthreads();
    build_w(s.t, s.box, s.t.h + hs, L, task, ntask, lane);
    __syncthreads();
    build_box<SLAB>(s, L, S1, S2, task, ntask, lane);
  }
  __syncthreads();
  double* o = R + it * (int64_t)n1 * n1 * n1;
  for (int e = tid; e < n1 * n1 * n1; e += kThreads) {
    const int t = e / (n1 * n1), u = (e / n1) % n1, v = e % n1;
    o[e] = (t + u + v <= L) ? s.box[r_offset(SLAB, L, t, u, v)] : 0.0;
  }
}

__global__ void hermite_e_kernel(int la, int lb, const double* __restrict__ za, const double* __restrict__ zb,
                                 const double* __restrict__ A, const double* __restrict__ B,
                                 double* __restrict__ E) {
  extern __shared__ __align__(16) unsigned char lds[];
  double* tabs = (double*)lds;
  const int lane = threadIdx.x;
  const int64_t it = blockIdx.x;
  const int trow = odd_row(la + lb + 2);
  const int taxis = ((la + 1) * (lb + 1) + 1) * trow;
  build_etab_rows(tabs, la, lb, trow, taxis, za[it], zb[it], A + it * 3, B + it * 3, false, lane >> 4, 4, lane & 15);
  __syncthreads();
  const int nt = la + lb + 1;
  const int per_axis = (la + 1) * (lb + 1) * nt;
  double* o = E + it * 3 * per_axis;
  for (int e = lane; e < 3 * per_axis; e += blockDim.x) {
    const int axis = e / per_axis, rem = e - axis * per_axis;
    const int ab = rem / nt, t = rem - ab * nt;
    o[e] = tabs[axis * taxis + ab * trow + t];
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

namespace {

thread_local std::string g_err;

eri4_status fail(eri4_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

// Device scratch of the no-allocation Coulomb call (eri4_batch_coulomb_static):
// the Hermite-space ket densities of one pass of quartets.  Each device holds
// its own copy until the process ends.  Host code must never pass this name to
// a kernel or a copy (on the host it is only a stand-in, not a device address):
// it uses the address that hipGetSymbolAddress returned for the current device
// (DeviceState::scratch), taken once per device in ensure_device.
constexpr int64_t kStaticScratchDoubles = (int64_t)4 << 20;  // 32 MiB
static __device__ __align__(256) double scratch[kStaticScratchDoubles];

struct DeviceState {
  bool ready = false;
  double* scratch = nullptr;  // this device's address of `scratch`
  double* boys = nullptr;
  uint2* rtab = nullptr;
  double* stab = nullptr;  // solid-harmonic coefficients (make_solid_table)
  int rstart[kMaxL + 1] = {0};  // per total order, in uint2 entries
  uint32_t* ttab = nullptr;  // tables of the Cartesian integral kernels (make_tile_tables)
  double* hcoef = nullptr;
  int cus = 0;  // compute units
  Tables tables() const { return Tables{boys, rtab, ttab, hcoef}; }
};

// Host copies of the tile tables (built once, read by the plans' cost estimate).
std::vector<uint32_t> g_ttab;
TileTableIndex g_tix;

std::mutex g_mu;
std::deque<DeviceState> g_dev;  // a deque: growing it keeps pointers to existing entries valid

#define HIP_TRY(call)                                                                     \
  do {                                                                                    \
    hipError_t e_ = (call);                                                               \
    if (e_ != hipSuccess) return fail(ERI4_ERROR_HIP, "%s: %s", #call, hipGetErrorString(e_)); \
  } while (0)

eri4_status set_attrs() {
  HIP_TRY(fused_set_attrs());
  HIP_TRY(cart_set_attrs());
  HIP_TRY(small_set_attrs());
  HIP_TRY(quad_set_attrs());
  HIP_TRY(solid_set_attrs());
  HIP_TRY(plan_set_attrs_solid());
  HIP_TRY(plan_set_attrs_solidp());
  HIP_TRY(plan_set_attrs_cart());
  HIP_TRY(plan_set_attrs_cartp());
  HIP_TRY(coulomb_set_attrs());
  HIP_TRY(coulomb_low_set_attrs());
  HIP_TRY(exchange_set_attrs());
  HIP_TRY(plan_coulomb_set_attrs());
  HIP_TRY(plan_set_attrs_f64());
  HIP_TRY(plan_set_attrs_f32());
  HIP_TRY(plan_set_attrs_f64p());
  HIP_TRY(plan_set_attrs_f32p());
  HIP_TRY(hipFuncSetAttribute((const void*)hermite_r_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              kMaxLdsBytes));
  HIP_TRY(hipFuncSetAttribute((const void*)hermite_r_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              kMaxLdsBytes));
  return ERI4_SUCCESS;
}

eri4_status ensure_device(DeviceState** st) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_mu);
  if ((int)g_dev.size() <= dev) g_dev.resize(dev + 1);
  DeviceState& d = g_dev[dev];
  if (!d.ready) {
    static std::vector<double> boys;
    static std::vector<uint32_t> rt;
    static std::vector<int> rs;
    static std::vector<double> st;
    static std::vector<double> hc;
    if (boys.empty()) {
      make_tile_tables(g_ttab, hc, g_tix);
      make_boys_table(boys);
      make_rtabs(rt, rs);
      make_solid_table(st);
    }
    if (hipMalloc(&d.boys, boys.size() * sizeof(double)) != hipSuccess)
      return fail(ERI4_ERROR_OUT_OF_MEMORY, "device allocation of the Boys table failed");
    if (hipMalloc(&d.rtab, rt.size() * sizeof(uint32_t)) != hipSuccess)
      return fail(ERI4_ERROR_OUT_OF_MEMORY, "device allocation of the recursion tables failed");
    HIP_TRY(hipMemcpy(d.boys, boys.data(), boys.size() * sizeof(double), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(d.rtab, rt.data(), rt.size() * sizeof(uint32_t), hipMemcpyHostToDevice));
    if (hipMalloc(&d.stab, st.size() * sizeof(double)) != hipSuccess)
      return fail(ERI4_ERROR_OUT_OF_MEMORY, "device allocation of the solid-harmonic table failed");
    HIP_TRY(hipMemcpy(d.stab, st.data(), st.size() * sizeof(double), hipMemcpyHostToDevice));
    if (hipMalloc(&d.ttab, g_ttab.size() * sizeof(uint32_t)) != hipSuccess ||
        hipMalloc(&d.hcoef, hc.size() * sizeof(double)) != hipSuccess)
      return fail(ERI4_ERROR_OUT_OF_MEMORY, "device allocation of the tile tables failed");
    HIP_TRY(hipMemcpy(d.ttab, g_ttab.data(), g_ttab.size() * sizeof(uint32_t), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(d.hcoef, hc.data(), hc.size() * sizeof(double), hipMemcpyHostToDevice));
    for (int i = 0; i <= kMaxL; ++i) d.rstart[i] = rs[i];
    HIP_TRY(hipGetSymbolAddress((void**)&d.scratch, HIP_SYMBOL(scratch)));
    HIP_TRY(hipDeviceGetAttribute(&d.cus, hipDeviceAttributeMultiprocessorCount, dev));
    eri4_status s = set_attrs();
    if (s != ERI4_SUCCESS) return s;
    d.ready = true;
  }
  *st = &d;
  return ERI4_SUCCESS;
}

int align16(int x) { return (x + 15) & ~15; }

// Class parameters and LDS layout for a tile of rb*16 bra rows.  xs: row
// stride of the [ab|q] staging area in doubles (0: 16 * nqb + 2, every column
// the first transform's accumulators hold).
ClassParams make_params(int la, int lb, int lc, int ld, int kmax, int rb, bool slab, bool box2, int xs = 0) {
  ClassParams p{};
  p.rb = rb;
  p.slab = slab ? 1 : 0;
  p.la = la; p.lb = lb; p.lc = lc; p.ld = ld;
  p.na = ncart(la); p.nb = ncart(lb); p.nc = ncart(lc); p.nd = ncart(ld);
  p.nab = p.na * p.nb; p.ncd = p.nc * p.nd;
  p.Lb = la + lb; p.Lk = lc + ld; p.L = p.Lb + p.Lk;
  p.np = nherm(p.Lb); p.nq = nherm(p.Lk);
  p.np4 = (p.np + 3) & ~3; p.nq4 = (p.nq + 3) & ~3;
  p.nqb = (p.nq + 15) / 16;
  p.ncdb = (p.ncd + 15) / 16;
  p.nrt = (p.nab + 16 * rb - 1) / (16 * rb);
  p.S1 = box_s1(p.L); p.S2 = box_s2(p.L);
  p.tbrow = odd_row(p.Lb + 2); p.tkrow = odd_row(p.Lk + 2);
  p.tbaxis = ((la + 1) * (lb + 1) + 1) * p.tbrow;
  p.tkaxis = ((lc + 1) * (ld + 1) + 1) * p.tkrow;
  p.xs = xs > 0 ? xs : 16 * p.nqb + 2;
  p.kmax = kmax;
  int off = 0;
  p.o_shell = off; off = align16(off + (12 + 8 * kmax) * 8 + 4 * 4);
  p.o_base = off;  off = align16(off + 96 * 8);  // [0]^(m), ket pair, bra pair, P-Q
  p.o_ptab = off;  off = align16(off + p.np4 * 8);
  p.o_qtab = off;  off = align16(off + 16 * p.nqb * 8);
  p.o_union = off;
  const int box_b = r_cells(slab, p.L) * 8;
  p.lay = slab ? kLaySlab : (box2 ? kLayBox2 : kLayBox);
  // phase 1: R box, bra tables (two-box layout: room for a second box)
  const int ph1 = align16(box_b) + (box2 ? align16(3 * p.tbaxis * 8) + box_b : 3 * p.tbaxis * 8);
  const int xb = align16(rb * 16 * p.xs * 8);
  const int ph2 = xb + 3 * p.tkaxis * 8;
  p.o_brae = off + align16(box_b);
  p.o_kete = off + xb;
  off = align16(off + (ph1 > ph2 ? ph1 : ph2));
  p.lds_bytes = off;
  return p;
}

// Class parameters for one tile height and R layout, if they fit (limit:
// bytes of LDS available for the dynamic area; column blocks per wave within
// what the kernel bodies are instantiated for).  The sizes and orders tested here are
// those of make_params, an upper bound of what the kernels take (dense_layout): a tile
// choice is accepted or refused as it always was.
bool try_params(int la, int lb, int lc, int ld, int kmax, int rb, int lay, const DeviceState* d, int limit,
                ClassParams* out) {
  const bool slab = lay == kLaySlab, two = lay == kLayBox2;
  if ((rb != 1 && rb != 2 && rb != 4) || lay < kLayBox || lay > kLayBox2) return false;
  if (rb == 4 && slab) return false;  // 64-row tiles are built for the box layouts
  if (two && la + lb + lc + ld > kBox2LMax) return false;
  ClassParams p = make_params(la, lb, lc, ld, kmax, rb, slab, two);
  const int maxc = rb == 4 ? 2 : (slab && rb == 1 ? kMaxC1 : 4);
  if (p.lds_bytes > limit || p.L > kMaxL || (p.nqb + 7) / 8 > maxc) return false;
  if (!slab && p.L > kBoxLMax) return false;
  p.rtab_off = d ? d->rstart[p.L] : 0;
  *out = p;
  return true;
}

// The library's own choice: the first that fits of two boxes (64-row tiles,
// then 32, then 16), box (the same), slab (32, 16).
bool pick_params(int la, int lb, int lc, int ld, int kmax, const DeviceState* d, int limit, ClassParams* out) {
  static const int order[8][2] = {{4, kLayBox2}, {2, kLayBox2}, {1, kLayBox2}, {4, kLayBox},
                                  {2, kLayBox},  {1, kLayBox},  {2, kLaySlab}, {1, kLaySlab}};
  for (const auto& o : order)
    if (try_params(la, lb, lc, ld, kmax, o[0], o[1], d, limit, out)) return true;
  return false;
}

// Parameters of the Cartesian integral kernels for a class (after
// ensure_device).  Every class with l <= ERI4_MAX_L fits: 159 616 bytes
// at most, of the 163 776 that a persistent kernel's own variables leave.
TileParams tile_params(int la, int lb, int lc, int ld, int kmax) {
  TileParams p{};
  p.la = la; p.lb = lb; p.lc = lc; p.ld = ld;
  p.nab = ncart(la) * ncart(lb); p.ncd = ncart(lc) * ncart(ld);
  p.Lb = la + lb; p.Lk = lc + ld; p.L = p.Lb + p.Lk;
  p.nq = nherm(p.Lk); p.nqb = (p.nq + 15) / 16;
  p.kb = nuv(p.Lb); p.kk = nuv(p.Lk);
  p.nr = nherm(p.L); p.nzt = nuv(p.L);
  p.tbrow = odd_row(p.Lb + 2); p.tkrow = odd_row(p.Lk + 2);
  p.tbaxis = ((la + 1) * (lb + 1) + 1) * p.tbrow;
  p.tkaxis = ((lc + 1) * (ld + 1) + 1) * p.tkrow;
  p.xs = (p.nq + 3) | 1;  // three zero columns; odd: the 16 rows of an operand read fall in different banks
  p.kmax = kmax;
  p.shape = tile_shape(p.nqb);
  const TileShapeInfo sh = kTileShapes[p.shape];
  const TileTableIndex& ix = g_tix;
  const TileTableIndex::Side& b = ix.bra[sh.lim][la][lb];
  const TileTableIndex::Side& k = ix.ket[lc][ld];
  p.nunits = b.nunits;
  p.ntiles = (b.nunits + kWaves / sh.cw - 1) / (kWaves / sh.cw);
  p.nkblk = k.nblocks;
  p.o_uv = ix.uv; p.o_qcol = ix.qcol[p.Lk]; p.o_task = ix.task[p.L]; p.ntask = ix.ntask[p.L];
  p.o_bunit = b.units; p.o_brows = b.rows;
  p.o_kunit = k.units; p.o_kcols = k.rows; p.o_klist = k.list;
  p.nks = 0;
  for (int i = 0; i < b.nunits; ++i) {
    const uint32_t w = g_ttab[b.units + 8 * i];
    const int X = (int)(w & 0xff), m0 = p.Lb - X;
    p.fsize = std::max(p.fsize, (int)((w >> 8) & 0xff) * tile_f_row(m0, p.Lk, m0 + p.Lk + 1, 0));
    p.nks = std::max(p.nks, ((X + p.Lk) >> 2) + 1);
  }
  const int ug = kWaves / sh.cw;  // units per tile
  int off = kTileKcol + 16 * p.nkblk * 4;
  p.o_row1 = off;
  if (ug > 1) off += kTileRowfSize + kTileRfSize;
  p.o_union = off;
  p.buf = align16(std::max(p.nr, 3 * p.tbaxis) * 8);
  p.o_f = off + 2 * p.buf;
  const int xbytes = align16(16 * tile_xb(sh.cw, sh.nc) * tile_xu(sh.cw, sh.nc) * p.xs * 8);
  p.o_zt = p.o_f + align16(ug * p.fsize * 8);
  p.o_kete = std::max(off + xbytes, p.o_zt);
  p.o_h = p.o_zt + align16(p.nzt * 8);
  p.o_g = p.o_h + 3 * 64 * h_steps(p.L) * 8;
  const int ph1 = p.o_g + ug * sh.rb * 64 * p.nks * 8;
  const int ph2 = p.o_kete + 3 * p.tkaxis * 8;
  p.lds_bytes = align16(std::max(ph1, ph2));
  return p;
}

// Estimated cycles of each tile of a quartet, per primitive quartet (products,
// reads over t, and the steps before them) and per ket primitive pair: f(quartet, ket).
template <class F>
void each_tile_cost(const TileParams& p, F f) {
  const TileShapeInfo sh = kTileShapes[p.shape];
  const int ug = kWaves / sh.cw;
  auto steps = [](const uint32_t* w) { return (double)((w[1] + 3) / 4); };
  double ket = 0.0;
  for (int i = 0; i < g_tix.ket[p.lc][p.ld].nunits; ++i) {  // for one row block
    const uint32_t* w = g_ttab.data() + p.o_kunit + 8 * i;
    ket += steps(w) * (w[0] >> 8) * (64.0 + 16.0 * ((w[0] & 0xff) / 4 + 1)) / 4.0;
  }
  for (int rt = 0; rt < p.ntiles; ++rt) {
    double g1 = 0.0, g2 = 0.0;
    for (int i = 0; i < ug && rt * ug + i < p.nunits; ++i) {
      const uint32_t* w = g_ttab.data() + p.o_bunit + 8 * (rt * ug + i);
      const double np = (w[0] >> 8) & 0xff, nb = w[0] >> 16, X = w[0] & 0xff;
      g1 = std::max(g1, steps(w) * sh.nc * (128.0 * np * nb + 12.0 * (X + 1)));
      const uint32_t v = w[7];
      g2 += (((v & 0xff) + ((v >> 8) & 0xff) + ((v >> 16) & 0xff) + (v >> 24)) + 15) / 16;
    }
    f(g1 + 5000.0 + 2.0 * p.nr, g2 * ket + 3000.0);
  }
}
struct TileCost { double quartet, ket; };
std::vector<TileCost> tile_costs(const TileParams& p) {
  std::vector<TileCost> cost;
  each_tile_cost(p, [&](double q, double k) { cost.push_back({q, k}); });
  return cost;
}

// The low-l kernels: one wave per quartet for kets of at most four [ab|q]
// column blocks, four waves for more.
bool small_four_waves(const ClassParams& p) { return p.nqb > 4; }

// The low-l kernels' parameters for classes whose shells all have l <=
// kSmallLMax: box layout, rb = bra row blocks per pass (at most 3, with at
// most 12 first-transform accumulator blocks of 16 x 16, spread evenly over
// the passes: (fd|fd)'s 4 row blocks run as 2 + 2, not 3 + 1).  The [ab|q]
// rows hold only the nq4 columns the second transform reads (the kernels
// store no others).
bool small_params(int la, int lb, int lc, int ld, int kmax, const DeviceState* d, ClassParams* out) {
  if (la > kSmallLMax || lb > kSmallLMax || lc > kSmallLMax || ld > kSmallLMax) return false;
  const int nrb = (ncart(la) * ncart(lb) + 15) / 16, nqb = (nherm(lc + ld) + 15) / 16;
  int rg = std::min(nrb, 3);
  while (rg > 1 && rg * nqb > 12) --rg;
  const int passes = (nrb + rg - 1) / rg;
  rg = (nrb + passes - 1) / passes;
  const int nq4 = (nherm(lc + ld) + 3) & ~3;
  ClassParams p = make_params(la, lb, lc, ld, kmax, rg, false, false, nq4 + 2);
  if (!small_four_waves(p)) {
    // [r] and W, the bra tables, zt and the per-axis tables; or the [ab|q] rows and
    // the ket tables
    const int nzt = nuv(p.L), xb = p.o_kete - p.o_union;
    p.o_rowt = p.o_union;
    p.o_rs = p.o_rowt + align16((p.L + 1) * (p.L + 1) * 2);
    p.o_rv = p.o_rs + align16(nzt * 4);
    p.o_union = p.o_rv + align16(nzt * 2);
    p.o_kete = p.o_union + xb;
    p.o_brae = p.o_union + align16((r_cells(false, p.L) + (p.S1 == p.L + 1 ? p.L + 1 : 0)) * 8);
    p.o_zt = p.o_brae + align16(3 * p.tbaxis * 8);
    p.o_h = p.o_zt + align16(nzt * 8);
    p.lds_bytes = align16(std::max(p.o_h + 3 * 64 * h_steps(p.L) * 8, p.o_kete + 3 * p.tkaxis * 8));
    p.o_uv = g_tix.uv;
  }
  if (p.lds_bytes > kSmallLdsMax || p.nqb > 6) return false;
  p.rtab_off = d ? d->rstart[p.L] : 0;
  *out = p;
  return true;
}

// Parameters of the kernels of eri4_quad.hip (l <= kSmallLMax; after
// ensure_device).  At most 153 KB of LDS: (ff|ff).
QuadParams quad_params(int la, int lb, int lc, int ld, int kmax) {
  QuadParams p{};
  p.t = tile_params(la, lb, lc, ld, kmax);
  const TileParams& t = p.t;
  const int n2 = (t.L + 1) * (t.L + 1);
  int off = 0;
  auto take = [&](int bytes) { const int o = off; off += align16(bytes); return o; };
  take((12 + 8 * kmax) * 8 + 4 * 4);
  p.o_base = take(32 * 8);
  p.o_rowt = take(n2 * 2);
  p.o_rs = take(t.nzt * 4);
  p.o_rv = take(t.nzt * 2);
  p.o_btab = take((t.kb + 1) * 16);
  p.o_ktab = take((t.kk + 1) * 16);
  p.o_kcol = take(16 * t.nkblk * 4);
  p.o_orow = take((t.nab + 31) / 32 * 32 * 4);
  p.o_kete = take(3 * t.tkaxis * 8);
  p.o_brae = take(2 * 3 * t.tbaxis * 8);
  p.o_h = take(2 * 3 * 64 * h_steps(t.L) * 8);
  p.o_zt = take(t.nzt * 8);
  p.o_w = take(t.nr * 8);
  // (u, v) of F: u su + v sv for u + v <= L - X; X = 0, and the least X of a second
  // group (the ninth group's)
  int x9 = 0;
  for (int X = 0, n = 0; X <= t.Lb && n <= kWaves; ++X) {
    n += std::min(la, X) - std::max(0, X - lb) + 1;
    x9 = X;
  }
  const int sv = odd_row(t.Lk + 1), su = sv * (t.L + 1);
  p.fsize = t.L * su + sv;
  p.fsize1 = (la + 1) * (lb + 1) > kWaves ? (t.L - x9) * su + sv : 0;
  p.nkunits = g_tix.ket[lc][ld].nunits;
  p.o_f = take(std::max(kWaves * (p.fsize + p.fsize1), (t.nab + 31) / 32 * 32 * t.xs) * 8);
  p.lds_bytes = off;
  return p;
}

// Whether nq quartets of a class with l <= kSmallLMax run on the kernels of
// eri4_quad.hip (one workgroup per compute unit, one recursion per primitive
// quartet) or on those of eri4_small.hip (many waves per compute unit, but a
// recursion per 32 or 48 bra rows).  Measured, quad : small in us, single
// primitives and 5151 (K = 5 in shells a and c):
//   256 quartets  (dd|dd) 19 : 25 and 157 : 305 (64 quartets), (ff|ss) 16 : 45 and 137
//                 : 808 (64), (pp|ff) 16 : 19; below L = 6 ((dp|ss) 14 : 12) no gain
//   512           (ff|ss) 29 : 46, (ff|ff) 65 : 111, (fd|dd) 38 : 44, (dd|dd) 35 : 26
//   768           (ff|ss) 42 : 47, (ff|fp) 64 : 78, (fd|dd) 55 : 45
//   4096          (ff|ff) 458 : 584 and 4804 : 7342, (ff|fd) 388 : 475 and 3993 : 7091,
//                 (ff|dd) 330 : 296 and 3445 : 5069, (ff|ss) 213 : 113
bool quad_route(int la, int lb, int lc, int ld, int kmax, int64_t nq, int cus) {
  const int Lb = la + lb, Lk = lc + ld;
  if (std::max(std::max(la, lb), std::max(lc, ld)) > kSmallLMax || Lb + Lk < 6) return false;
  if (Lb == 6 && (Lk >= 5 || (Lk == 4 && kmax > 1))) return true;
  return nq <= (int64_t)cus * (Lb == 6 ? 3 : Lb == 5 ? 2 : 1);
}

// LDS layout of the kernels of eri4_dense.h (mode: what they compute) and the
// tables of their recursion (whose places need d, an initialised device): [r], whose
// unused cells hold W, then zt and the per-axis tables, then but for solid harmonics the bra tables (behind or over them) and
// for Cartesian integrals the ket tables; or the [ab|q] tile.  For solid harmonics and
// exchange it fits wherever the layout of make_params does (checked over all classes,
// tiles and layouts), without the second box that the two-box layout once held.
void dense_layout(ClassParams* p, int mode, const DeviceState* d) {
  if (d) {
    const TileTableIndex& ix = g_tix;
    p->ntask = ix.ntask[p->L]; p->o_uv = ix.uv; p->o_task = ix.task[p->L];
  }
  const int nzt = nuv(p->L);
  p->o_rowt = p->o_qtab + align16(16 * p->nqb * 8);
  p->o_rs = p->o_rowt + align16((p->L + 1) * (p->L + 1) * 2);
  p->o_rv = p->o_rs + align16(nzt * 4);
  p->o_union = p->o_rv + align16(nzt * 2);
  if (p->L <= kWaveL) p->o_union = p->o_rowt + align16(nherm(p->L) * 8);  // (or, of low orders, the recursion's table)
  p->o_zt = p->o_union + align16((r_cells(p->slab, p->L) + (p->S1 == p->L + 1 ? p->L + 1 : 0)) * 8);
  p->o_h = p->o_zt + align16(nzt * 8);
  int end = p->o_h + 3 * 64 * h_steps(p->L) * 8;
  const int etab = mode != kDenseSolid ? align16(3 * p->tbaxis * 8) : 0;
  // the bra tables in a place of their own where there is room (one workgroup runs
  // per compute unit in any case), else over zt and the per-axis tables
  p->o_brae = end + etab <= kMaxLdsBytes ? end : p->o_zt;
  end = std::max(end, p->o_brae + etab);
  // over the tile at the end: the exchange blocks of every wave (exch_store)
  const int tile = std::max(p->rb * 16 * p->xs, mode == kDenseExch ? kWaves * 4 * 64 : 0);
  p->o_kete = align16(std::max(end, p->o_union + tile * 8));
  p->lds_bytes = p->o_kete + (mode == kDenseCart ? align16(3 * p->tkaxis * 8) : 0);
}

// Parameters of the dense Cartesian kernels for a class, if it fits: the tile height
// that holds its rows, 64 at most.
bool cart_params(int la, int lb, int lc, int ld, int kmax, const DeviceState* d, int limit, ClassParams* out) {
  if (la + lb + lc + ld > kBoxLMax) return false;
  const int nrb = (ncart(la) * ncart(lb) + 15) / 16;
  for (int rb = nrb > 2 ? 4 : nrb; rb >= 1; rb >>= 1) {
    ClassParams p = make_params(la, lb, lc, ld, kmax, rb, false, false);
    dense_layout(&p, kDenseCart, d);
    if (p.lds_bytes > limit || (p.nqb + 7) / 8 > (rb == 4 ? 2 : 4)) continue;
    p.rtab_off = d->rstart[p.L];
    *out = p;
    return true;
  }
  return false;
}

// Whether the Cartesian integrals of nq quartets of a class run as dense tiles (p,
// eri4_dense.h) or as grouped ones (t, eri4_tile.h): kb * kk and kk primitive quartets
// and ket pairs of a quartet.  Grouped tiles have fewer products, but leave groups of
// a few rows in blocks of 16 and repeat the recursion for every two or three blocks.
// The times below (us) were fitted to 1004 calls: all classes with l <= 3 and la >=
// lb, lc >= ld as plans, 110 higher ones as batches, 16 to 2048 quartets of one and
// three primitives per shell (to 9% and 12%; the margin takes the forms' own tie).  Of
// those calls, dense : grouped in us, 300 quartets:
//   (ss|ss) 18 : 31, (pp|pp) 22 : 47, (dd|dd) 34 : 70, (ff|ff) 91 : 123, (hp|ss) 31 : 62,
//   (fd|hp) 44 : 69, (gf|ss) 66 : 106, (gg|gg) 297 : 210, (kd|gd) 210 : 186
double grouped_us(double kbkk, double kk, double tq, double tk) { return kbkk * 7.9e-4 * tq + kk * 8.1e-4 * tk + 6.9; }
double dense_us(const ClassParams& p, double kbkk, double kk) {
  const double s1 = p.np4 / 4 * ((p.nqb + 7) / 8) * p.rb, s2 = p.nq4 / 4 * ((p.ncdb + 7) / 8) * p.rb;
  return kbkk * (1.9 + 0.062 * s1 + 0.0063 * nherm(p.L)) + kk * 0.079 * s2 + 5.1;
}
constexpr double kGroupedLaunch = 4.5, kDenseLaunch = 4.1;
bool cart_route(const TileParams& t, const ClassParams& p, double nq, double kbkk, double kk, int cus) {
#ifdef ROUTE_ALL
  return ROUTE_ALL;
#endif
  double tq = 0.0, tk = 0.0;
  each_tile_cost(t, [&](double q, double k) { tq += q; tk += k; });
  const double grouped =
      std::ceil(nq * t.ntiles / cus) * grouped_us(kbkk, kk, tq / t.ntiles, tk / t.ntiles) + kGroupedLaunch;
  const double dense = std::ceil(nq * p.nrt / cus) * dense_us(p, kbkk, kk) + kDenseLaunch;
  return dense < (p.L <= 13 ? 0.95 : 0.85) * grouped;
}

// Solid-harmonic output: the library's tile for the class, with rows and
// columns over the 2l+1 real solid harmonics of each shell; hbs / hks doubles
// of H per bra / ket primitive pair (rows padded to whole tiles, columns to
// whole 16-column blocks, k to the padded Hermite counts).
void to_solid(ClassParams* p, const DeviceState* d) {
  p->na = 2 * p->la + 1; p->nb = 2 * p->lb + 1; p->nc = 2 * p->lc + 1; p->nd = 2 * p->ld + 1;
  p->nab = p->na * p->nb;
  p->ncd = p->nc * p->nd;
  p->nrt = (p->nab + 16 * p->rb - 1) / (16 * p->rb);
  p->ncdb = (p->ncd + 15) / 16;
  dense_layout(p, kDenseSolid, d);
}

// The library's own tile of solid harmonics, no taller than the rows there are: 4000
// (ss|ss) 177 -> 160 us with 16 rows for one instead of 64.
void fit_rows(ClassParams* p, const DeviceState* d) {
  const int nrb = (p->nab + 15) / 16;
  if (nrb > 2 || nrb >= p->rb) return;
  p->rb = nrb;
  p->nrt = 1;
  dense_layout(p, kDenseSolid, d);
}

bool solid_params(int la, int lb, int lc, int ld, int kmax, const DeviceState* d, ClassParams* p, int64_t* hbs,
                  int64_t* hks) {
  if (!pick_params(la, lb, lc, ld, kmax, d, kMaxLdsBytes, p)) return false;
  to_solid(p, d);
  *hbs = (int64_t)p->nrt * p->rb * 16 * p->np4;
  *hks = (int64_t)p->ncdb * 16 * p->nq4;
  fit_rows(p, d);
  return true;
}

}  // namespace
}  // namespace eri4

using namespace eri4;

extern "C" {

int eri4_ncart(int l) { return l < 0 ? -1 : ncart(l); }

int64_t eri4_quartet_size(int la, int lb, int lc, int ld) {
  if (la < 0 || lb < 0 || lc < 0 || ld < 0) return -1;
  return (int64_t)ncart(la) * ncart(lb) * ncart(lc) * ncart(ld);
}

const char* eri4_last_error(void) { return g_err.c_str(); }

const char* eri4_version(void) { return "eri4 0.1 (gfx950, FP64 MFMA matrix McMurchie-Davidson)"; }

eri4_status eri4_init(void) {
  g_err.clear();
  DeviceState* d;
  return ensure_device(&d);
}

eri4_status eri4_batch(int la, int lb, int lc, int ld, int64_t nquartets, const double* centers,
                       const double* exponents, const double* coeffs, const int32_t* nprim, int kmax,
                       double* out, hipStream_t stream) {
  g_err.clear();
  if (la < 0 || lb < 0 || lc < 0 || ld < 0)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "angular momenta must be >= 0 (got %d %d %d %d)", la, lb, lc, ld);
  if (la > ERI4_MAX_L || lb > ERI4_MAX_L || lc > ERI4_MAX_L || ld > ERI4_MAX_L)
    return fail(ERI4_ERROR_UNSUPPORTED, "angular momentum above %d is not supported (got %d %d %d %d)",
                ERI4_MAX_L, la, lb, lc, ld);
  if (nquartets < 0) return fail(ERI4_ERROR_INVALID_ARGUMENT, "nquartets must be >= 0");
  if (kmax < 1 || kmax > ERI4_MAX_K)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "kmax must be in 1..%d (got %d)", ERI4_MAX_K, kmax);
  if (nquartets == 0) return ERI4_SUCCESS;
  if (!centers || !exponents || !coeffs || !nprim || !out)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
  DeviceState* d;
  eri4_status s = ensure_device(&d);
  if (s != ERI4_SUCCESS) return s;
  ClassParams p;
  if (quad_route(la, lb, lc, ld, kmax, nquartets, d->cus)) {
    const QuadParams qp = quad_params(la, lb, lc, ld, kmax);
    const int64_t qchunk = (int64_t)1 << 22;  // grid below 2^32 work-items
    for (int64_t q0 = 0; q0 < nquartets; q0 += qchunk) {
      const int64_t nq = std::min(qchunk, nquartets - q0);
      const hipError_t e = quad_launch(qp, nq, stream, d->tables(), centers, exponents, coeffs, nprim, out, q0);
      if (e != hipSuccess) return fail(ERI4_ERROR_HIP, "kernel launch: %s", hipGetErrorString(e));
    }
    return ERI4_SUCCESS;
  }
  if (small_params(la, lb, lc, ld, kmax, d, &p)) {
    const int64_t qchunk = (int64_t)1 << 24;  // grid of qchunk workgroups of at most 256 threads
    for (int64_t q0 = 0; q0 < nquartets; q0 += qchunk) {
      const int64_t nq = std::min(qchunk, nquartets - q0);
      // four waves per quartet for kets with more than four [ab|q] column
      // blocks, one wave otherwise (measured: (ff|ff) 10-16% faster on four
      // waves at K_bra K_ket = 1, 5 and 25; (dd|dd) faster on one wave)
      const bool four = small_four_waves(p);
      const Tables tb = d->tables();
      const hipError_t e = four ? small4_launch(p, nq, stream, tb, centers, exponents, coeffs, nprim, out, q0)
                                : small_launch(p, nq, stream, tb, centers, exponents, coeffs, nprim, out, q0);
      if (e != hipSuccess) return fail(ERI4_ERROR_HIP, "kernel launch: %s", hipGetErrorString(e));
    }
    return ERI4_SUCCESS;
  }
  const TileParams t = tile_params(la, lb, lc, ld, kmax);
  const double kk = (double)kmax * kmax;
  if (cart_params(la, lb, lc, ld, kmax, d, kMaxLdsBytes - 64, &p) &&
      cart_route(t, p, (double)nquartets, kk * kk, kk, d->cus)) {
    const int64_t qchunk = ((int64_t)1 << 22) / p.nrt;  // grid below 2^32 work-items
    for (int64_t q0 = 0; q0 < nquartets; q0 += qchunk) {
      const int64_t nq = std::min(qchunk, nquartets - q0);
      const hipError_t e = cart_launch(p, nq, stream, d->tables(), centers, exponents, coeffs, nprim, out, q0);
      if (e != hipSuccess) return fail(ERI4_ERROR_HIP, "kernel launch: %s", hipGetErrorString(e));
    }
    return ERI4_SUCCESS;
  }
  const int64_t qchunk = ((int64_t)1 << 22) / t.ntiles;  // grid below 2^32 work-items
  for (int64_t q0 = 0; q0 < nquartets; q0 += qchunk) {
    const int64_t nq = std::min(qchunk, nquartets - q0);
    const hipError_t e =
        fused_launch(t, nq, stream, d->tables(), centers, exponents, coeffs, nprim, out, q0);
    if (e != hipSuccess) return fail(ERI4_ERROR_HIP, "kernel launch: %s", hipGetErrorString(e));
  }
  return ERI4_SUCCESS;
}

static eri4_status check_class(int la, int lb, int lc, int ld, int64_t nquartets, int kmax) {
  if (la < 0 || lb < 0 || lc < 0 || ld < 0)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "angular momenta must be >= 0 (got %d %d %d %d)", la, lb, lc, ld);
  if (la > ERI4_MAX_L || lb > ERI4_MAX_L || lc > ERI4_MAX_L || ld > ERI4_MAX_L)
    return fail(ERI4_ERROR_UNSUPPORTED, "angular momentum above %d is not supported (got %d %d %d %d)",
                ERI4_MAX_L, la, lb, lc, ld);
  if (nquartets < 0) return fail(ERI4_ERROR_INVALID_ARGUMENT, "nquartets must be >= 0");
  if (kmax < 1 || kmax > ERI4_MAX_K)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "kmax must be in 1..%d (got %d)", ERI4_MAX_K, kmax);
  return ERI4_SUCCESS;
}

eri4_status eri4_solid_coefficients(int l, double* C) {
  g_err.clear();
  if (l < 0 || l > ERI4_MAX_L) return fail(ERI4_ERROR_INVALID_ARGUMENT, "l must be in 0..%d (got %d)", ERI4_MAX_L, l);
  if (!C) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL output array");
  solid_dense(l, C);
  return ERI4_SUCCESS;
}

int64_t eri4_solid_work_size(int la, int lb, int lc, int ld, int kmax, int64_t nquartets) {
  if (check_class(la, lb, lc, ld, nquartets, kmax) != ERI4_SUCCESS) return -1;
  ClassParams p;
  int64_t hbs, hks;
  if (!solid_params(la, lb, lc, ld, kmax, nullptr, &p, &hbs, &hks)) return -1;
  return nquartets * kmax * kmax * (hbs + hks);
}

eri4_status eri4_batch_solid(int la, int lb, int lc, int ld, int64_t nquartets, const double* centers,
                             const double* exponents, const double* coeffs, const int32_t* nprim, int kmax,
                             double* work, int64_t work_size, double* out, hipStream_t stream) {
  g_err.clear();
  eri4_status st = check_class(la, lb, lc, ld, nquartets, kmax);
  if (st != ERI4_SUCCESS) return st;
  if (nquartets == 0) return ERI4_SUCCESS;
  if (!centers || !exponents || !coeffs || !nprim || !out || !work)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
  ClassParams p;
  int64_t hbs, hks;
  if (!solid_params(la, lb, lc, ld, kmax, nullptr, &p, &hbs, &hks))
    return fail(ERI4_ERROR_UNSUPPORTED, "class (%d %d|%d %d) does not fit in LDS", la, lb, lc, ld);
  // quartets per pass: what the workspace holds (H of every primitive pair),
  // within the grid limits
  const int64_t perq = (int64_t)kmax * kmax * (hbs + hks);
  int64_t chunk = work_size / perq;
  if (chunk < 1)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "workspace of %lld doubles is below one quartet's %lld",
                (long long)work_size, (long long)perq);
  DeviceState* d;
  st = ensure_device(&d);
  if (st != ERI4_SUCCESS) return st;
  (void)solid_params(la, lb, lc, ld, kmax, d, &p, &hbs, &hks);  // the same tile, with the device's table offsets
  chunk = std::min<int64_t>(chunk, std::min<int64_t>(((int64_t)1 << 30) / p.nrt, INT32_MAX));
  double* hbra = work;
  for (int64_t q0 = 0; q0 < nquartets; q0 += chunk) {
    const int64_t nq = std::min(chunk, nquartets - q0);
    double* hket = hbra + nq * kmax * kmax * hbs;
    hipError_t e = solid_h_launch(p, nq, stream, centers, exponents, coeffs, nprim, d->stab, hbra, hket, q0, hbs, hks);
    if (e == hipSuccess)
      e = solid_launch(p, dim3((unsigned)(nq * p.nrt)), stream, d->tables(), centers, exponents, coeffs,
                       nprim, out, q0, hbra, hket, hbs, hks);
    if (e != hipSuccess) return fail(ERI4_ERROR_HIP, "kernel launch: %s", hipGetErrorString(e));
  }
  return ERI4_SUCCESS;
}

// Parameters and LDS layout of the Coulomb (J-engine) kernels (after
// ensure_device).  Every class with l <=
// ERI4_MAX_L fits: at most 103 KB, 75 KB for (ii|ii): two workgroups per compute unit.
JParams jengine_params(int la, int lb, int lc, int ld, int kmax) {
  JParams p{};
  p.la = la; p.lb = lb; p.lc = lc; p.ld = ld;
  p.nab = ncart(la) * ncart(lb); p.ncd = ncart(lc) * ncart(ld);
  p.Lb = la + lb; p.Lk = lc + ld; p.L = p.Lb + p.Lk;
  p.nq = nherm(p.Lk); p.nzt = nuv(p.L);
  p.tbrow = odd_row(p.Lb + 2);
  p.tbaxis = ((la + 1) * (lb + 1) + 1) * p.tbrow;
  p.kmax = kmax;
  p.ds = 16 * ((p.nq + 15) / 16);
  const TileTableIndex& ix = g_tix;
  p.ntask = ix.ntask[p.L]; p.nchunk = ix.nchunk[p.Lb]; p.nitems = ix.nitem[p.Lk];
  for (p.ncps = 3; (1 << p.ncps) < p.nchunk;) ++p.ncps;
  p.ncp = 1 << p.ncps;
  p.o_uv = ix.uv; p.o_task = ix.task[p.L]; p.o_chunk = ix.chunk[p.Lb];
  p.o_item = ix.item[p.Lk]; p.o_qpos = ix.qpos[p.Lk];
  p.dsize = ix.dsize[p.Lk];
  int cells = 0;
  for (int n = p.L + 1; n >= 1; n -= 2) cells += n * (n | 1);
  // the parts of w over [r]: twelve values of half the threads
  p.rsize = kJPad + std::max(cells + kJPad, 12 * kThreads / 2);
  p.o_d = kJEnd;
  p.o_r = p.o_d + align16(p.dsize * 8);
  p.o_w = p.o_r + align16(p.rsize * 8);
  p.o_zt = p.o_w + align16(nherm(p.L) * 8);
  p.o_h = p.o_zt + align16(p.nzt * 8);
  p.o_wp = p.o_w + align16(3 * p.tbaxis * 8);
  p.o_wf = p.o_wp + align16(nherm(p.Lb) * 8);
  p.lds_bytes = align16(std::max(p.o_h + 3 * 64 * h_steps(p.L) * 8, p.o_wf + nfold(la, lb) * 8));
  return p;
}

// Parameters of the Coulomb kernels of low orders (after ensure_device); false where
// they do not apply: above kWaveL, or with a side of l1 + l2 > 6.
bool jlow_params(int la, int lb, int lc, int ld, int kmax, const DeviceState* d, JLowParams* out) {
  JLowParams p{};
  p.la = la; p.lb = lb; p.lc = lc; p.ld = ld;
  p.Lb = la + lb; p.Lk = lc + ld; p.L = p.Lb + p.Lk;
  if (p.L > kWaveL || p.Lb > 6 || p.Lk > 6) return false;
  p.nb = ncart(lb); p.nd = ncart(ld);
  p.nab = ncart(la) * p.nb; p.ncd = ncart(lc) * p.nd;
  p.np = nherm(p.Lb); p.nq = nherm(p.Lk);
  p.S1 = box_s1(p.L); p.S2 = box_s2(p.L);
  p.tbrow = odd_row(p.Lb + 2); p.tkrow = odd_row(p.Lk + 2);
  p.tbaxis = ((la + 1) * (lb + 1) + 1) * p.tbrow;
  p.tkaxis = ((lc + 1) * (ld + 1) + 1) * p.tkrow;
  p.kmax = kmax;
  p.ds = 16 * ((p.nq + 15) / 16);
  p.rtab_off = d->rstart[p.L];
  p.o_uv = g_tix.uv;
  int off = 0;
  auto take = [&](int bytes) { const int o = off; off += align16(bytes); return o; };
  take((12 + 8 * kmax) * 8 + 4 * 4);
  p.o_ptab = take(p.np * 8);
  p.o_qtab = take(p.nq * 4);
  p.o_entl = take(nherm(p.L) * 8);
  p.o_wave = off;
  off = 0;
  take(16 * 8);
  p.o_r = take(std::max(r_cells(false, p.L), p.nab) * 8);
  p.o_d = take(std::max(64, p.nq) * 8);
  p.o_w = take(p.np * 8);
  p.o_e = take(3 * p.tbaxis * 8);
  p.wsize = off;
  p.lds_bytes = p.o_wave + p.wsize;
  *out = p;
  return true;
}
// Waves of their workgroups: one per bra primitive pair, kLowWaves at most.
int jlow_waves(int kmax) { return std::min(kLowWaves, kmax * kmax); }

// Workspace doubles per primitive pair slot: dket of the ket pair, J of the bra's.
static int64_t coulomb_slot(int la, int lb, int lc, int ld) {
  return 16 * ((nherm(lc + ld) + 15) / 16) + ncart(la) * ncart(lb);
}

int64_t eri4_coulomb_work_size(int la, int lb, int lc, int ld, int kmax, int64_t nquartets) {
  if (check_class(la, lb, lc, ld, nquartets, kmax) != ERI4_SUCCESS) return -1;
  return nquartets * kmax * kmax * coulomb_slot(la, lb, lc, ld);
}

// J for nquartets quartets in passes of as many as the workspace (work_size
// doubles) holds the Hermite-space densities and per-bra-pair J of: per pass,
// the density kernel, the J-engine kernel and the sum over bra pairs.
// Arguments already checked; d is initialised.
static eri4_status coulomb_passes(int la, int lb, int lc, int ld, int64_t nquartets, const double* centers,
                                  const double* exponents, const double* coeffs, const int32_t* nprim, int kmax,
                                  const double* dens, double* work, int64_t work_size, double* out,
                                  hipStream_t stream, const DeviceState* d) {
  const JParams p = jengine_params(la, lb, lc, ld, kmax);
  const int64_t kk2 = (int64_t)kmax * kmax;
  const int64_t perq = kk2 * (p.ds + p.nab);
  int64_t chunk = work_size / perq;
  if (chunk < 1)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "workspace of %lld doubles is below one quartet's %lld",
                (long long)work_size, (long long)perq);
  chunk = std::min<int64_t>(chunk, ((int64_t)1 << 22) / kk2);  // grid of chunk * kmax^2 workgroups
  JLowParams low;
  const bool is_low = jlow_params(la, lb, lc, ld, kmax, d, &low);
  for (int64_t q0 = 0; q0 < nquartets; q0 += chunk) {
    const int64_t nq = std::min(chunk, nquartets - q0);
    if (is_low) {
      const hipError_t e = coulomb_low_launch(low, jlow_waves(kmax), nq, stream, d->tables(), centers, exponents,
                                              coeffs, nprim, dens, work, out, q0);
      if (e != hipSuccess) return fail(ERI4_ERROR_HIP, "kernel launch: %s", hipGetErrorString(e));
      continue;
    }
    double* part = work + nq * kk2 * p.ds;
    hipError_t e = coulomb_dket_launch(p, nq, stream, d->tables(), centers, exponents, nprim, dens, work, q0);
    if (e == hipSuccess)
      e = coulomb_launch(p, nq, stream, d->tables(), centers, exponents, coeffs, nprim, part, out, q0, work);
    if (e != hipSuccess) return fail(ERI4_ERROR_HIP, "kernel launch: %s", hipGetErrorString(e));
  }
  return ERI4_SUCCESS;
}

eri4_status eri4_batch_coulomb(int la, int lb, int lc, int ld, int64_t nquartets, const double* centers,
                               const double* exponents, const double* coeffs, const int32_t* nprim, int kmax,
                               const double* dens, double* work, int64_t work_size, double* out, hipStream_t stream) {
  g_err.clear();
  eri4_status st = check_class(la, lb, lc, ld, nquartets, kmax);
  if (st != ERI4_SUCCESS) return st;
  if (nquartets == 0) return ERI4_SUCCESS;
  if (!centers || !exponents || !coeffs || !nprim || !dens || !out || !work)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
  if (work_size < (int64_t)kmax * kmax * coulomb_slot(la, lb, lc, ld))
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "workspace of %lld doubles is below one quartet's %lld",
                (long long)work_size, (long long)kmax * kmax * coulomb_slot(la, lb, lc, ld));
  DeviceState* d;
  st = ensure_device(&d);
  if (st != ERI4_SUCCESS) return st;
  return coulomb_passes(la, lb, lc, ld, nquartets, centers, exponents, coeffs, nprim, kmax, dens, work, work_size,
                        out, stream, d);
}

// Exchange contraction: the library's tile for the class, with the bra rows
// ordered (b, a) and a padded to whole 16-row blocks (one b per block); fbs
// doubles of F^b per ket primitive pair and b, ps doubles of partial rows
// y^b per quartet.
static bool exchange_params(int la, int lb, int lc, int ld, int kmax, const DeviceState* d, ClassParams* p,
                            int64_t* fbs, int64_t* ps) {
  if (!pick_params(la, lb, lc, ld, kmax, d, kMaxLdsBytes, p)) return false;
  const int blocks = p->nb * ((p->na + 15) / 16);
  // no taller than the rows there are
  if (blocks <= 2 && blocks < p->rb) {
    const int lay = p->lay;
    if (!try_params(la, lb, lc, ld, kmax, blocks, lay, d, kMaxLdsBytes, p)) return false;
  }
  p->nrt = (blocks + p->rb - 1) / p->rb;
  dense_layout(p, kDenseExch, d);
  *fbs = (int64_t)((p->nc + 15) / 16) * 16 * p->nq4;
  *ps = (int64_t)p->nb * p->na * p->nc;
  return true;
}

int64_t eri4_exchange_work_size(int la, int lb, int lc, int ld, int kmax, int64_t nquartets) {
  if (check_class(la, lb, lc, ld, nquartets, kmax) != ERI4_SUCCESS) return -1;
  ClassParams p;
  int64_t fbs, ps;
  if (!exchange_params(la, lb, lc, ld, kmax, nullptr, &p, &fbs, &ps)) return -1;
  return nquartets * ((int64_t)kmax * kmax * p.nb * fbs + ps);
}

eri4_status eri4_batch_exchange(int la, int lb, int lc, int ld, int64_t nquartets, const double* centers,
                                const double* exponents, const double* coeffs, const int32_t* nprim, int kmax,
                                const double* dens, double* work, int64_t work_size, double* out,
                                hipStream_t stream) {
  g_err.clear();
  eri4_status st = check_class(la, lb, lc, ld, nquartets, kmax);
  if (st != ERI4_SUCCESS) return st;
  if (nquartets == 0) return ERI4_SUCCESS;
  if (!centers || !exponents || !coeffs || !nprim || !dens || !out || !work)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
  ClassParams p;
  int64_t fbs, ps;
  if (!exchange_params(la, lb, lc, ld, kmax, nullptr, &p, &fbs, &ps))
    return fail(ERI4_ERROR_UNSUPPORTED, "class (%d %d|%d %d) does not fit in LDS", la, lb, lc, ld);
  const int64_t perq = (int64_t)kmax * kmax * p.nb * fbs + ps;
  int64_t chunk = work_size / perq;
  if (chunk < 1)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "workspace of %lld doubles is below one quartet's %lld",
                (long long)work_size, (long long)perq);
  DeviceState* d;
  st = ensure_device(&d);
  if (st != ERI4_SUCCESS) return st;
  (void)exchange_params(la, lb, lc, ld, kmax, d, &p, &fbs, &ps);
  chunk = std::min<int64_t>(chunk, std::min<int64_t>(((int64_t)1 << 30) / p.nrt, INT32_MAX));
  for (int64_t q0 = 0; q0 < nquartets; q0 += chunk) {
    const int64_t nq = std::min(chunk, nquartets - q0);
    double* fb = work;
    double* part = work + nq * (int64_t)kmax * kmax * p.nb * fbs;
    const hipError_t e = exchange_launch(p, nq, stream, d->tables(), centers, exponents, coeffs, nprim,
                                         dens, fb, fbs, part, out, q0);
    if (e != hipSuccess) return fail(ERI4_ERROR_HIP, "kernel launch: %s", hipGetErrorString(e));
  }
  return ERI4_SUCCESS;
}

int64_t eri4_static_scratch_bytes(void) { return kStaticScratchDoubles * (int64_t)sizeof(double); }

eri4_status eri4_batch_coulomb_static(int la, int lb, int lc, int ld, int64_t nquartets, const double* centers,
                                      const double* exponents, const double* coeffs, const int32_t* nprim, int kmax,
                                      const double* dens, double* out, hipStream_t stream) {
  g_err.clear();
  eri4_status st = check_class(la, lb, lc, ld, nquartets, kmax);
  if (st != ERI4_SUCCESS) return st;
  if (nquartets == 0) return ERI4_SUCCESS;
  if (!centers || !exponents || !coeffs || !nprim || !dens || !out)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
  if (kmax * kmax * coulomb_slot(la, lb, lc, ld) > kStaticScratchDoubles)
    return fail(ERI4_ERROR_UNSUPPORTED, "one quartet's Hermite-space densities and partial J (%lld doubles) exceed "
                "the %lld-double static scratch", (long long)kmax * kmax * coulomb_slot(la, lb, lc, ld),
                (long long)kStaticScratchDoubles);
  // no initialisation here: that allocates the tables (eri4_init must have run)
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  const DeviceState* d = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (dev < (int)g_dev.size() && g_dev[dev].ready) d = &g_dev[dev];
  }
  if (!d)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "the library is not initialised on device %d: call eri4_init there "
                "first (it allocates; this call does not)", dev);
  return coulomb_passes(la, lb, lc, ld, nquartets, centers, exponents, coeffs, nprim, kmax, dens, d->scratch,
                        kStaticScratchDoubles, out, stream, d);
}

// ---------------------------------------------------------------------------
// plans: many classes and contraction lengths in one persistent launch, or two
// ---------------------------------------------------------------------------

struct eri4_plan_s {
  int device = 0;
  int64_t nq = 0;
  int kmax = 1;
  int nitems = 0;
  int nclasses = 0;
  int lds_bytes = 0;
  int grid = 0;
  // Cartesian plans: the items of classes that run as dense tiles, behind the others
  int ncart_items = 0, cart_lds = 0, cart_grid = 0;
  ClassParams* d_cart = nullptr;
  // Coulomb plans: the same for the kernel of low orders
  int nlow = 0, low_lds = 0;
  JLowParams* d_low = nullptr;
  bool f32 = false;  // ERI4_PREC_FP32
  bool pairs = false;  // made from a bra and a ket list of shell pairs
  int64_t nbra = 0, nket = 0;
  bool solid = false;  // solid-harmonic output
  int64_t work = 0;    // doubles of caller workspace for the H matrices
  int64_t nentries = 0;      // solid plans: list entries whose H is built (2 per quartet for quartet plans)
  int hlds = 0;              // solid plans: dynamic LDS of the H builder (its largest entry)
  int32_t* d_pl = nullptr;   // per list entry: l of its two shells (bra entries first)
  int32_t* d_pn = nullptr;   // per list entry: contraction lengths
  int64_t* d_hoff = nullptr; // per list entry: where its H matrices start in the workspace
  bool coul = false;         // Coulomb contraction over the lists (eri4_plan_create_coulomb)
  int64_t dket_size = 0;     // doubles of the workspace holding the ket entries' dket
  int64_t ket_dens_size = 0; // doubles of ket_dens (all ket entries' blocks)
  std::vector<int64_t> ooff; // output offsets per bra entry (Coulomb plans)
  int64_t* d_doff = nullptr;   // per ket entry: its density block in ket_dens
  int64_t* d_dkoff = nullptr;  // per ket entry: its dket in the workspace
  int64_t* d_joff = nullptr;   // per bra entry: its J block in out
  int64_t out_size = 0;
  std::vector<int64_t> qoff;
  void* d_classes = nullptr;  // TileParams (Cartesian plans), ClassParams (solid) or JParams (Coulomb) per class
  int2* d_items = nullptr;
  int64_t* d_qoff = nullptr;
  int32_t* d_nprim = nullptr;
  int* d_counter = nullptr;
};

static void plan_free(eri4_plan_s* p) {
  if (!p) return;
  if (p->d_classes) (void)hipFree(p->d_classes);
  if (p->d_items) (void)hipFree(p->d_items);
  if (p->d_cart) (void)hipFree(p->d_cart);
  if (p->d_low) (void)hipFree(p->d_low);
  if (p->d_qoff) (void)hipFree(p->d_qoff);
  if (p->d_nprim) (void)hipFree(p->d_nprim);
  if (p->d_counter) (void)hipFree(p->d_counter);
  if (p->d_pl) (void)hipFree(p->d_pl);
  if (p->d_pn) (void)hipFree(p->d_pn);
  if (p->d_hoff) (void)hipFree(p->d_hoff);
  if (p->d_doff) (void)hipFree(p->d_doff);
  if (p->d_dkoff) (void)hipFree(p->d_dkoff);
  if (p->d_joff) (void)hipFree(p->d_joff);
  delete p;
}

eri4_status eri4_plan_create(eri4_plan* plan, int64_t nquartets, const int32_t* l, const int32_t* nprim, int kmax,
                             eri4_precision precision) {
  return eri4_plan_create_tuned(plan, nquartets, l, nprim, kmax, precision, nullptr, 0);
}

static_assert(ERI4_LAYOUT_BOX == kLayBox && ERI4_LAYOUT_SLAB == kLaySlab && ERI4_LAYOUT_BOX2 == kLayBox2,
              "public and internal layout codes agree");

// items by decreasing cost, equal ones in order: three passes of 11 bits over the
// costs as floats, whose bits order as positive numbers do (30 000 tiles of a pair
// list took a comparison sort longer than the rest of a plan's creation).
static std::vector<int2> largest_first(const std::vector<int2>& items, const std::vector<double>& cost) {
  struct Entry { uint32_t key; int2 item; };
  std::vector<Entry> a(items.size()), b(items.size());
  for (size_t i = 0; i < items.size(); ++i) {
    const float c = (float)cost[i];
    std::memcpy(&a[i].key, &c, sizeof c);
    a[i].key = ~a[i].key;
    a[i].item = items[i];
  }
  for (int shift = 0; shift < 33; shift += 11) {
    std::vector<size_t> at(2049, 0);
    for (const Entry& e : a) ++at[((e.key >> shift) & 2047) + 1];
    for (int i = 0; i < 2048; ++i) at[i + 1] += at[i];
    for (const Entry& e : a) b[at[(e.key >> shift) & 2047]++] = e;
    a.swap(b);
  }
  std::vector<int2> sorted(items.size());
  for (size_t i = 0; i < a.size(); ++i) sorted[i] = a[i].item;
  return sorted;
}

// Plan over quartets given by l / nprim; pairs: the shells will come from a
// bra and a ket list (quartet q = bra pair q / nket with ket pair q % nket).
static eri4_status plan_create(eri4_plan* plan, int64_t nquartets, const int32_t* l, const int32_t* nprim, int kmax,
                               eri4_precision precision, const eri4_tile_choice* choices, int nchoices, bool pairs,
                               int64_t nbra, int64_t nket, bool solid, bool coul = false) {
  if (!plan) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL plan pointer");
  *plan = nullptr;
  if (precision != ERI4_PREC_FP64 && precision != ERI4_PREC_FP32)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "unknown precision %d", (int)precision);
  if (nquartets < 0 || nquartets > ((int64_t)1 << 31) - 1)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "nquartets must be in 0..2^31-1");
  if (kmax < 1 || kmax > ERI4_MAX_K)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "kmax must be in 1..%d (got %d)", ERI4_MAX_K, kmax);
  if (nquartets > 0 && (!l || !nprim)) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL host array");
  for (int64_t i = 0; i < 4 * nquartets; ++i) {
    if (l[i] < 0) return fail(ERI4_ERROR_INVALID_ARGUMENT, "negative angular momentum at quartet %lld", (long long)(i / 4));
    if (l[i] > ERI4_MAX_L)
      return fail(ERI4_ERROR_UNSUPPORTED, "angular momentum %d above %d at quartet %lld", l[i], ERI4_MAX_L,
                  (long long)(i / 4));
    if (nprim[i] < 1 || nprim[i] > kmax)
      return fail(ERI4_ERROR_INVALID_ARGUMENT, "contraction length %d outside 1..%d at quartet %lld", nprim[i], kmax,
                  (long long)(i / 4));
  }
  if (nchoices < 0 || (nchoices > 0 && !choices))
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "tile choices: NULL array or negative count");
  // entries of the choice table per class, in table order
  std::vector<std::vector<int>> choices_of(8 * 8 * 8 * 8);
  for (int i = 0; i < nchoices; ++i) {
    const eri4_tile_choice& c = choices[i];
    if (c.rows16 != 1 && c.rows16 != 2 && c.rows16 != 4)
      return fail(ERI4_ERROR_INVALID_ARGUMENT, "tile choice %d: rows16 must be 1, 2 or 4 (got %d)", i, c.rows16);
    if (c.layout < ERI4_LAYOUT_BOX || c.layout > ERI4_LAYOUT_BOX2)
      return fail(ERI4_ERROR_INVALID_ARGUMENT, "tile choice %d: unknown layout %d", i, c.layout);
    if (c.kq_min > c.kq_max)
      return fail(ERI4_ERROR_INVALID_ARGUMENT, "tile choice %d: kq_min %d above kq_max %d", i, c.kq_min, c.kq_max);
    for (int x = 0; x < 4; ++x)
      if (c.l[x] < 0 || c.l[x] > ERI4_MAX_L)
        return fail(ERI4_ERROR_INVALID_ARGUMENT, "tile choice %d: angular momentum %d out of range", i, c.l[x]);
    choices_of[((c.l[0] * 8 + c.l[1]) * 8 + c.l[2]) * 8 + c.l[3]].push_back(i);
  }
  int device = 0;
  HIP_TRY(hipGetDevice(&device));
  DeviceState* d;
  eri4_status st = ensure_device(&d);
  if (st != ERI4_SUCCESS) return st;
  eri4_plan_s* p = new (std::nothrow) eri4_plan_s();
  if (!p) return fail(ERI4_ERROR_OUT_OF_MEMORY, "host allocation failed");
  p->device = device;
  p->nq = nquartets;
  p->kmax = kmax;
  p->f32 = precision == ERI4_PREC_FP32;
  p->pairs = pairs;
  p->nbra = nbra;
  p->nket = nket;
  p->solid = solid;
  p->coul = coul;
  // dynamic LDS available next to the persistent kernel's static LDS
  const int limit = kMaxLdsBytes - 64;

  // groups of quartets with the same class and tile choice (the first matching
  // entry of the table, or none), keyed by class * (nchoices + 1) + entry + 1
  std::map<int64_t, int> group_of;
  std::vector<int> qcls(nquartets);
  std::vector<std::array<int, 5>> keys;  // la, lb, lc, ld, entry (-1: none)
  for (int64_t q = 0; q < nquartets; ++q) {
    const int key = ((l[4 * q] * 8 + l[4 * q + 1]) * 8 + l[4 * q + 2]) * 8 + l[4 * q + 3];
    const int64_t kq = (int64_t)nprim[4 * q] * nprim[4 * q + 1] * nprim[4 * q + 2] * nprim[4 * q + 3];
    int entry = -1;
    for (int i : choices_of[key])
      if (kq >= choices[i].kq_min && kq <= choices[i].kq_max) {
        entry = i;
        break;
      }
    const int64_t gkey = (int64_t)key * (nchoices + 1) + entry + 1;
    auto it = group_of.find(gkey);
    if (it == group_of.end()) {
      it = group_of.emplace(gkey, (int)keys.size()).first;
      keys.push_back({l[4 * q], l[4 * q + 1], l[4 * q + 2], l[4 * q + 3], entry});
    }
    qcls[q] = it->second;
  }
  if (keys.size() > 32767) {
    plan_free(p);
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "too many (class, tile choice) groups");
  }
  // per group: tile height and R layout (the table's, or see pick_params)
  std::vector<ClassParams> cps(coul ? 0 : keys.size());
  std::vector<JParams> jps;
  std::vector<JLowParams> lps;
  std::vector<char> is_low;
  for (size_t c = 0; c < keys.size(); ++c) {
    const auto& k = keys[c];
    if (coul) {
      jps.push_back(jengine_params(k[0], k[1], k[2], k[3], kmax));
      JLowParams lp{};
      is_low.push_back(jlow_params(k[0], k[1], k[2], k[3], kmax, d, &lp));
      lps.push_back(lp);
    } else if (k[4] >= 0) {
      const eri4_tile_choice& ch = choices[k[4]];
      if (!try_params(k[0], k[1], k[2], k[3], kmax, ch.rows16, ch.layout, d, limit, &cps[c])) {
        plan_free(p);
        return fail(ERI4_ERROR_INVALID_ARGUMENT, "tile choice %d (rows16 %d, layout %d) does not fit class (%d %d|%d %d)",
                    k[4], ch.rows16, ch.layout, k[0], k[1], k[2], k[3]);
      }
    } else if (!pick_params(k[0], k[1], k[2], k[3], kmax, d, limit, &cps[c])) {
      plan_free(p);
      return fail(ERI4_ERROR_UNSUPPORTED, "class (%d %d|%d %d) does not fit in LDS", k[0], k[1], k[2], k[3]);
    }
  }
  if (solid)
    for (size_t c = 0; c < keys.size(); ++c) {  // rows and columns over solid functions; same tile
      to_solid(&cps[c], d);
      if (keys[c][4] < 0) fit_rows(&cps[c], d);
    }
  // Cartesian plans run the kernels of eri4_tile.h, or those of eri4_dense.h (cart_route:
  // dense[c]), whose tilings follow from the class; a tile choice is checked and changes
  // nothing
  std::vector<TileParams> tps;
  std::vector<ClassParams> dps;
  std::vector<char> dense;
  std::vector<std::vector<TileCost>> tcs;
  if (!solid && !coul) {
    std::vector<std::array<double, 3>> work(keys.size(), {0.0, 0.0, 0.0});  // quartets, primitive quartets, ket pairs
    for (int64_t q = 0; q < nquartets; ++q) {
      const double kk = (double)nprim[4 * q + 2] * nprim[4 * q + 3];
      auto& w = work[qcls[q]];
      w[0] += 1.0, w[1] += (double)nprim[4 * q] * nprim[4 * q + 1] * kk, w[2] += kk;
    }
    for (size_t c = 0; c < keys.size(); ++c) {
      const auto& k = keys[c];
      ClassParams dp{};
      tps.push_back(tile_params(k[0], k[1], k[2], k[3], kmax));
      // as if all quartets were of this class: they share the compute units
      dense.push_back(cart_params(k[0], k[1], k[2], k[3], kmax, d, limit, &dp) &&
                      cart_route(tps.back(), dp, (double)nquartets, work[c][1] / work[c][0], work[c][2] / work[c][0],
                                 d->cus));
      dps.push_back(dp);
      tcs.push_back(tile_costs(tps.back()));
    }
    // The two kernels of a plan of both kinds run one after the other, each for as long
    // as its longest tile takes: where few quartets make that the time, all take one
    // (60 quartets of f and g, 2 primitives at most: 420 us in both, 253 in one).
    const auto any = [&](char x) { return std::find(dense.begin(), dense.end(), x) != dense.end(); };
    if (any(0) && any(1)) {
      double sum[3] = {}, most[3] = {};  // both kinds: grouped, dense; all grouped
      for (int64_t q = 0; q < nquartets; ++q) {
        const int c = qcls[q];
        const double kk = (double)nprim[4 * q + 2] * nprim[4 * q + 3], kbkk = kk * nprim[4 * q] * nprim[4 * q + 1];
        for (const TileCost& t : tcs[c]) {
          const double us = grouped_us(kbkk, kk, t.quartet, t.ket);
          for (int x : {0, 2})
            if (x == 2 || !dense[c]) sum[x] += us, most[x] = std::max(most[x], us);
        }
        if (dense[c]) {
          const double us = dense_us(dps[c], kbkk, kk);
          sum[1] += us * dps[c].nrt, most[1] = std::max(most[1], us);
        }
      }
      double us[3];
      for (int x = 0; x < 3; ++x) us[x] = std::max(most[x], sum[x] / d->cus + 0.5 * most[x]);
      if (us[2] + kGroupedLaunch < us[0] + us[1] + kGroupedLaunch + kDenseLaunch)
        std::fill(dense.begin(), dense.end(), (char)0);
    }
  }
  p->nclasses = (int)keys.size();
  // A Coulomb plan of both kinds runs two kernels one after the other: a gain where there
  // are quartets enough to fill the chip many times (3969 of s to f: 195 us in one, 111 in
  // two), a loss where the longest quartet is the time (225: 39 and 51; of three primitives
  // per shell 435 and 575)
  if (std::find(is_low.begin(), is_low.end(), (char)0) != is_low.end() && nquartets <= 4 * (int64_t)d->cus)
    std::fill(is_low.begin(), is_low.end(), (char)0);
  if (coul)
    for (size_t c = 0; c < keys.size(); ++c) {
      if (is_low[c])
        p->low_lds = std::max(p->low_lds, lps[c].lds_bytes + (jlow_waves(kmax) - 1) * lps[c].wsize);
      else
        p->lds_bytes = std::max(p->lds_bytes, jps[c].lds_bytes);
    }
  else if (solid)
    for (const ClassParams& c : cps) p->lds_bytes = std::max(p->lds_bytes, c.lds_bytes);
  else
    for (size_t c = 0; c < keys.size(); ++c) {
      int& lds = dense[c] ? p->cart_lds : p->lds_bytes;
      lds = std::max(lds, dense[c] ? dps[c].lds_bytes : tps[c].lds_bytes);
    }

  // output offsets in input order, and work items with their cost
  p->qoff.resize(nquartets);
  int64_t off = 0;
  std::vector<int2> items, cart_items, low_items;
  std::vector<double> cost, cart_cost, low_cost;
  for (int64_t q = 0; q < nquartets; ++q) {
    const double kb = (double)nprim[4 * q] * nprim[4 * q + 1], kk = (double)nprim[4 * q + 2] * nprim[4 * q + 3];
    p->qoff[q] = off;
    if (coul) {
      // one item per quartet (J-engine): per primitive quartet the recursion
      // and the matrix-vector product, per bra pair the bra transform
      const JParams& j = jps[qcls[q]];
      off += j.nab;  // J rows per quartet
      if (is_low[qcls[q]]) {
        low_cost.push_back(kb * kk * (4000.0 + nherm(j.L) + 10.0 * j.nq) + kb * 2000.0);
        low_items.push_back(make_int2((int)q, qcls[q]));
        continue;
      }
      cost.push_back(kb * kk * (5000.0 + 2.0 * nherm(j.L) + nherm(j.Lb) * (double)j.nq / 16.0) +
                     kb * (4000.0 + 8.0 * j.nab) + 4000.0);
      items.push_back(make_int2((int)q, qcls[q] << 16));
      continue;
    }
    const ClassParams& c = cps[qcls[q]];
    off += (int64_t)c.nab * c.ncd;
    if (!solid && !dense[qcls[q]]) {
      const std::vector<TileCost>& t = tcs[qcls[q]];
      for (size_t rt = 0; rt < t.size(); ++rt) {
        cost.push_back(kb * kk * t[rt].quartet + kk * t[rt].ket + 4000.0);
        items.push_back(make_int2((int)q, (int)rt | (qcls[q] << 16)));
      }
      continue;
    }
    const ClassParams& dc = solid ? c : dps[qcls[q]];
    for (int rt = 0; rt < dc.nrt; ++rt) {
      const int rows = 16 * std::min(dc.rb, (dc.nab - rt * dc.rb * 16 + 15) / 16);
      // MFMA cycles of the two transforms at 128 FLOP/clk per CU, plus a
      // latency-bound estimate for Boys and the recursion per primitive quartet
      const double g1 = 2.0 * rows * dc.np4 * 16.0 * dc.nqb * kb * kk;
      const double g2 = 2.0 * rows * dc.nq4 * 16.0 * dc.ncdb * kk;
      (solid ? cost : cart_cost).push_back((g1 + g2) / 128.0 + kb * kk * (8000.0 + 4.0 * nherm(dc.L)) + 4000.0);
      (solid ? items : cart_items).push_back(make_int2((int)q, rt | (qcls[q] << 16)));
    }
  }
  p->out_size = off;
  std::vector<int2> sorted = largest_first(items, cost);
  const std::vector<int2> cart_sorted = largest_first(cart_items, cart_cost);
  if (sorted.size() + cart_sorted.size() > (size_t)INT32_MAX) {
    plan_free(p);
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "too many work items");
  }
  p->ncart_items = (int)cart_sorted.size();
  const std::vector<int2> low_sorted = largest_first(low_items, low_cost);
  p->nlow = (int)low_sorted.size();
  p->nitems = (int)sorted.size();

  int ncu = 0, per_cu = 0;
  HIP_TRY(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, p->device));
  const hipError_t oe = p->coul ? plan_coulomb_occupancy(p->lds_bytes, &per_cu)
                        : p->solid ? (p->pairs ? plan_occupancy_solidp(p->lds_bytes, &per_cu)
                                              : plan_occupancy_solid(p->lds_bytes, &per_cu))
                        : p->pairs ? (p->f32 ? plan_occupancy_f32p(p->lds_bytes, &per_cu)
                                           : plan_occupancy_f64p(p->lds_bytes, &per_cu))
                                 : (p->f32 ? plan_occupancy_f32(p->lds_bytes, &per_cu)
                                           : plan_occupancy_f64(p->lds_bytes, &per_cu));
  if (oe != hipSuccess || per_cu < 1) per_cu = 1;
  p->grid = (int)std::min<int64_t>(std::max(p->nitems, 1), (int64_t)ncu * per_cu);

  if (p->ncart_items > 0) {
    if ((p->pairs ? plan_occupancy_cartp(p->cart_lds, &per_cu) : plan_occupancy_cart(p->cart_lds, &per_cu)) != hipSuccess ||
        per_cu < 1)
      per_cu = 1;
    p->cart_grid = (int)std::min<int64_t>(p->ncart_items, (int64_t)ncu * per_cu);
    sorted.insert(sorted.end(), cart_sorted.begin(), cart_sorted.end());
  }
  sorted.insert(sorted.end(), low_sorted.begin(), low_sorted.end());

  const void* params = coul ? (const void*)jps.data() : solid ? (const void*)cps.data() : (const void*)tps.data();
  const size_t params_size = keys.size() * (coul ? sizeof(JParams) : solid ? sizeof(ClassParams) : sizeof(TileParams));
  const bool ok = hipMalloc(&p->d_classes, std::max<size_t>(1, params_size)) == hipSuccess &&
                  hipMalloc(&p->d_items, std::max<size_t>(1, sorted.size()) * sizeof(int2)) == hipSuccess &&
                  hipMalloc(&p->d_qoff, std::max<int64_t>(1, nquartets) * sizeof(int64_t)) == hipSuccess &&
                  hipMalloc(&p->d_nprim, std::max<int64_t>(1, 4 * nquartets) * sizeof(int32_t)) == hipSuccess &&
                  hipMalloc(&p->d_counter, 64) == hipSuccess &&
                  (p->ncart_items == 0 || hipMalloc(&p->d_cart, keys.size() * sizeof(ClassParams)) == hipSuccess) &&
                  (p->nlow == 0 || hipMalloc(&p->d_low, keys.size() * sizeof(JLowParams)) == hipSuccess);
  if (!ok) {
    plan_free(p);
    return fail(ERI4_ERROR_OUT_OF_MEMORY, "device allocation for the plan failed");
  }
  hipError_t e = hipSuccess;
  if (params_size) e = hipMemcpy(p->d_classes, params, params_size, hipMemcpyHostToDevice);
  if (e == hipSuccess && p->nlow > 0)
    e = hipMemcpy(p->d_low, lps.data(), keys.size() * sizeof(JLowParams), hipMemcpyHostToDevice);
  if (e == hipSuccess && p->ncart_items > 0)
    e = hipMemcpy(p->d_cart, dps.data(), keys.size() * sizeof(ClassParams), hipMemcpyHostToDevice);
  if (e == hipSuccess && !sorted.empty())
    e = hipMemcpy(p->d_items, sorted.data(), sorted.size() * sizeof(int2), hipMemcpyHostToDevice);
  if (e == hipSuccess && nquartets > 0)
    e = hipMemcpy(p->d_qoff, p->qoff.data(), nquartets * sizeof(int64_t), hipMemcpyHostToDevice);
  if (e == hipSuccess && nquartets > 0)
    e = hipMemcpy(p->d_nprim, nprim, 4 * nquartets * sizeof(int32_t), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    plan_free(p);
    return fail(ERI4_ERROR_HIP, "plan upload: %s", hipGetErrorString(e));
  }
  *plan = p;
  return ERI4_SUCCESS;
}

eri4_status eri4_plan_create_tuned(eri4_plan* plan, int64_t nquartets, const int32_t* l, const int32_t* nprim,
                                   int kmax, eri4_precision precision, const eri4_tile_choice* choices,
                                   int nchoices) {
  g_err.clear();
  return plan_create(plan, nquartets, l, nprim, kmax, precision, choices, nchoices, false, 0, 0, false);
}

// Tile table file (format in eri4.h) -> choices; checks the arch line against
// the current device.
static eri4_status read_tile_table(const char* path, std::vector<eri4_tile_choice>* out) {
  FILE* f = std::fopen(path, "r");
  if (!f) return fail(ERI4_ERROR_INVALID_ARGUMENT, "tile table %s: cannot open it", path);
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
    std::fclose(f);
    return fail(ERI4_ERROR_HIP, "tile table %s: no device properties", path);
  }
  std::string devarch(prop.gcnArchName);
  devarch = devarch.substr(0, devarch.find(':'));
  char line[512];
  int lineno = 0;
  bool have_arch = false;
  eri4_status st = ERI4_SUCCESS;
  while (st == ERI4_SUCCESS && std::fgets(line, sizeof line, f)) {
    ++lineno;
    char* p = line;
    while (*p == ' ' || *p == '\t') ++p;
    if (*p == '#' || *p == '\n' || *p == '\r' || *p == 0) continue;
    char word[64];
    if (std::sscanf(p, "arch %63s", word) == 1 && std::strncmp(p, "arch", 4) == 0) {
      if (devarch != word)
        st = fail(ERI4_ERROR_INVALID_ARGUMENT, "tile table %s is for %s, the device is %s", path, word,
                  devarch.c_str());
      have_arch = true;
      continue;
    }
    eri4_tile_choice c{};
    char lay[16];
    int n = 0;
    if (std::sscanf(p, "%d %d %d %d %d %d %d %15s %n", &c.l[0], &c.l[1], &c.l[2], &c.l[3], &c.kq_min, &c.kq_max,
                    &c.rows16, lay, &n) != 8 || p[n] != 0) {
      st = fail(ERI4_ERROR_INVALID_ARGUMENT, "tile table %s line %d: expected 'la lb lc ld kq_min kq_max rows16 "
                "layout'", path, lineno);
      break;
    }
    if (!have_arch) {
      st = fail(ERI4_ERROR_INVALID_ARGUMENT, "tile table %s line %d: entry before the arch line", path, lineno);
      break;
    }
    if (!std::strcmp(lay, "box")) c.layout = ERI4_LAYOUT_BOX;
    else if (!std::strcmp(lay, "slab")) c.layout = ERI4_LAYOUT_SLAB;
    else if (!std::strcmp(lay, "box2")) c.layout = ERI4_LAYOUT_BOX2;
    else {
      st = fail(ERI4_ERROR_INVALID_ARGUMENT, "tile table %s line %d: unknown layout %s", path, lineno, lay);
      break;
    }
    out->push_back(c);
  }
  std::fclose(f);
  if (st == ERI4_SUCCESS && !have_arch) st = fail(ERI4_ERROR_INVALID_ARGUMENT, "tile table %s: no arch line", path);
  return st;
}

eri4_status eri4_plan_create_tunefile(eri4_plan* plan, int64_t nquartets, const int32_t* l, const int32_t* nprim,
                                      int kmax, eri4_precision precision, const char* tune_file) {
  g_err.clear();
  if (!plan) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL plan pointer");
  *plan = nullptr;
  std::vector<eri4_tile_choice> choices;
  if (tune_file) {
    const eri4_status st = read_tile_table(tune_file, &choices);
    if (st != ERI4_SUCCESS) return st;
  }
  return plan_create(plan, nquartets, l, nprim, kmax, precision, choices.data(), (int)choices.size(), false, 0, 0,
                     false);
}

int64_t eri4_plan_output_size(eri4_plan plan) { return plan ? plan->out_size : -1; }

eri4_status eri4_plan_output_offsets(eri4_plan plan, int64_t* offsets) {
  g_err.clear();
  if (!plan) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL plan");
  const std::vector<int64_t>& o = plan->coul ? plan->ooff : plan->qoff;
  if (!o.empty() && !offsets) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL offsets array");
  std::copy(o.begin(), o.end(), offsets);
  return ERI4_SUCCESS;
}

// Enqueue the counter reset and the persistent kernel of a plan.
static eri4_status plan_launch(eri4_plan plan, const Shells& shl, double* work, int64_t work_size, double* out,
                               hipStream_t stream) {
  if (plan->nitems + plan->ncart_items == 0) return ERI4_SUCCESS;
  if (!shl.centers || !shl.exps || !shl.coefs || !out || (plan->pairs && (!shl.kcenters || !shl.kexps || !shl.kcoefs)))
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
  if (plan->solid && (!work || work_size < plan->work))
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "workspace of %lld doubles is below the plan's %lld",
                (long long)(work ? work_size : 0), (long long)plan->work);
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev != plan->device)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "plan was made for device %d, current device is %d", plan->device, dev);
  DeviceState* d;
  eri4_status st = ensure_device(&d);
  if (st != ERI4_SUCCESS) return st;
  if (plan->solid)
    HIP_TRY(solid_hpairs_launch(plan->pairs ? plan->nbra : -1, plan->nentries, plan->kmax, plan->hlds, stream, plan->d_pl,
                                plan->d_pn, shl, plan->d_hoff, d->stab, work));
  hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, stream, plan->d_counter);
  HIP_TRY(hipGetLastError());
  const PlanArgs a{plan->d_classes, plan->d_items, plan->nitems, plan->d_qoff, plan->d_nprim, plan->d_counter, shl,
                   out};
  const Tables t = d->tables();
  const dim3 grid(plan->grid);
  if (plan->ncart_items > 0) {
    const PlanArgs c{plan->d_cart, plan->d_items + plan->nitems, plan->ncart_items, plan->d_qoff, plan->d_nprim,
                     plan->d_counter + 1, shl, out};
    HIP_TRY(plan->pairs ? plan_launch_cartp(dim3(plan->cart_grid), plan->cart_lds, stream, t, c)
                        : plan_launch_cart(dim3(plan->cart_grid), plan->cart_lds, stream, t, c));
    if (plan->nitems == 0) return ERI4_SUCCESS;
  }
  if (plan->solid)
    HIP_TRY(plan->pairs ? plan_launch_solidp(grid, plan->lds_bytes, stream, t, a, plan->nbra, plan->d_hoff, work)
                        : plan_launch_solid(grid, plan->lds_bytes, stream, t, a, plan->nbra, plan->d_hoff, work));
  else if (plan->pairs)
    HIP_TRY(plan->f32 ? plan_launch_f32p(grid, plan->lds_bytes, stream, t, a)
                      : plan_launch_f64p(grid, plan->lds_bytes, stream, t, a));
  else
    HIP_TRY(plan->f32 ? plan_launch_f32(grid, plan->lds_bytes, stream, t, a)
                      : plan_launch_f64(grid, plan->lds_bytes, stream, t, a));
  return ERI4_SUCCESS;
}

eri4_status eri4_plan_execute(eri4_plan plan, const double* centers, const double* exponents, const double* coeffs,
                              double* out, hipStream_t stream) {
  g_err.clear();
  if (!plan) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL plan");
  if (plan->pairs)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "plan made from pair lists: use eri4_plan_execute_pairs");
  if (plan->solid) return fail(ERI4_ERROR_INVALID_ARGUMENT, "solid-harmonic plan: use eri4_plan_execute_solid");
  return plan_launch(plan, Shells{centers, exponents, coeffs, nullptr, nullptr, nullptr, 0}, nullptr, 0, out, stream);
}

// Workspace layout of a solid plan's H matrices: entry e (l and contraction
// lengths pl[2e..2e+1], pn[2e..2e+1]; a ket pair if e >= nbra, or for nbra < 0
// if e is odd) holds K1 * K2 slots from hoff[e] (solid_hpairs_kernel); uploads
// pl, pn and hoff into the plan and sets its workspace size.  Frees the plan
// and clears *plan on error.
static eri4_status solid_entries(eri4_plan* plan, int64_t ne, int64_t nbra, const int32_t* pl, const int32_t* pn) {
  eri4_plan_s* p = *plan;
  std::vector<int64_t> hoff(ne);
  int64_t off = 0;
  for (int64_t e = 0; e < ne; ++e) {
    hoff[e] = off;
    const int l1 = pl[2 * e], l2 = pl[2 * e + 1];
    const int nk4 = (nherm(l1 + l2) + 3) & ~3;
    off += (int64_t)pn[2 * e] * pn[2 * e + 1] * solid_pair_units(l1, l2, nbra < 0 ? (e & 1) != 0 : e >= nbra) * 16 *
           nk4;
    p->hlds = std::max(p->hlds, solid_h_lds(l1, l2, nk4));
  }
  p->work = off;
  p->nentries = ne;
  const bool ok = hipMalloc(&p->d_pl, std::max<int64_t>(1, 2 * ne) * sizeof(int32_t)) == hipSuccess &&
                  hipMalloc(&p->d_pn, std::max<int64_t>(1, 2 * ne) * sizeof(int32_t)) == hipSuccess &&
                  hipMalloc(&p->d_hoff, std::max<int64_t>(1, ne) * sizeof(int64_t)) == hipSuccess;
  hipError_t e = ok ? hipSuccess : hipErrorOutOfMemory;
  if (e == hipSuccess && ne > 0) e = hipMemcpy(p->d_pl, pl, 2 * ne * sizeof(int32_t), hipMemcpyHostToDevice);
  if (e == hipSuccess && ne > 0) e = hipMemcpy(p->d_pn, pn, 2 * ne * sizeof(int32_t), hipMemcpyHostToDevice);
  if (e == hipSuccess && ne > 0) e = hipMemcpy(p->d_hoff, hoff.data(), ne * sizeof(int64_t), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    plan_free(p);
    *plan = nullptr;
    return ok ? fail(ERI4_ERROR_HIP, "plan upload: %s", hipGetErrorString(e))
              : fail(ERI4_ERROR_OUT_OF_MEMORY, "device allocation for the plan failed");
  }
  return ERI4_SUCCESS;
}

eri4_status eri4_plan_create_solid(eri4_plan* plan, int64_t nquartets, const int32_t* l, const int32_t* nprim,
                                   int kmax, const char* tune_file) {
  g_err.clear();
  if (!plan) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL plan pointer");
  *plan = nullptr;
  std::vector<eri4_tile_choice> choices;
  if (tune_file) {
    const eri4_status st = read_tile_table(tune_file, &choices);
    if (st != ERI4_SUCCESS) return st;
  }
  eri4_status st = plan_create(plan, nquartets, l, nprim, kmax, ERI4_PREC_FP64, choices.data(), (int)choices.size(),
                               false, 0, 0, true);
  if (st != ERI4_SUCCESS) return st;
  // entries 2q (bra pair) and 2q + 1 (ket pair): the quartet arrays as they are
  return solid_entries(plan, 2 * nquartets, -1, l, nprim);
}

eri4_status eri4_plan_execute_solid(eri4_plan plan, const double* centers, const double* exponents,
                                    const double* coeffs, double* work, int64_t work_size, double* out,
                                    hipStream_t stream) {
  g_err.clear();
  if (!plan) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL plan");
  if (plan->pairs) return fail(ERI4_ERROR_INVALID_ARGUMENT, "plan made from pair lists: use eri4_plan_execute_pairs");
  if (!plan->solid) return fail(ERI4_ERROR_INVALID_ARGUMENT, "Cartesian plan: use eri4_plan_execute");
  return plan_launch(plan, Shells{centers, exponents, coeffs, nullptr, nullptr, nullptr, 0}, work, work_size, out,
                     stream);
}

eri4_status eri4_plan_create_pairs(eri4_plan* plan, int64_t nbra, const int32_t* bra_l, const int32_t* bra_nprim,
                                   int64_t nket, const int32_t* ket_l, const int32_t* ket_nprim, int kmax,
                                   eri4_precision precision, eri4_functions functions,
                                   const eri4_tile_choice* choices, int nchoices) {
  g_err.clear();
  if (!plan) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL plan pointer");
  *plan = nullptr;
  if (functions != ERI4_CARTESIAN && functions != ERI4_SOLID)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "unknown functions %d", (int)functions);
  const bool solid = functions == ERI4_SOLID;
  if (solid && precision != ERI4_PREC_FP64)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "solid-harmonic output runs FP64 transforms only");
  if (nbra < 0 || nket < 0) return fail(ERI4_ERROR_INVALID_ARGUMENT, "negative list length");
  if (nbra > 0 && nket > (((int64_t)1 << 31) - 1) / nbra)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "nbra * nket must be below 2^31");
  if ((nbra > 0 && (!bra_l || !bra_nprim)) || (nket > 0 && (!ket_l || !ket_nprim)))
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL host array");
  // quartet (i, j) = bra pair i with ket pair j, at q = i * nket + j
  const int64_t nq = nbra * nket;
  std::vector<int32_t> l(4 * nq), np(4 * nq);
  for (int64_t i = 0; i < nbra; ++i)
    for (int64_t j = 0; j < nket; ++j) {
      const int64_t q = i * nket + j;
      l[4 * q] = bra_l[2 * i], l[4 * q + 1] = bra_l[2 * i + 1];
      l[4 * q + 2] = ket_l[2 * j], l[4 * q + 3] = ket_l[2 * j + 1];
      np[4 * q] = bra_nprim[2 * i], np[4 * q + 1] = bra_nprim[2 * i + 1];
      np[4 * q + 2] = ket_nprim[2 * j], np[4 * q + 3] = ket_nprim[2 * j + 1];
    }
  eri4_status st = plan_create(plan, nq, l.data(), np.data(), kmax, precision, choices, nchoices, true, nbra, nket, solid);
  if (st != ERI4_SUCCESS || !solid) return st;
  // H matrices of every list entry, bra entries first
  const int64_t ne = nbra + nket;
  std::vector<int32_t> pl(2 * ne), pn(2 * ne);
  for (int64_t e = 0; e < ne; ++e) {
    const bool ket = e >= nbra;
    const int64_t i = ket ? e - nbra : e;
    const int32_t* lsrc = ket ? ket_l : bra_l;
    const int32_t* nsrc = ket ? ket_nprim : bra_nprim;
    pl[2 * e] = lsrc[2 * i], pl[2 * e + 1] = lsrc[2 * i + 1];
    pn[2 * e] = nsrc[2 * i], pn[2 * e + 1] = nsrc[2 * i + 1];
  }
  return solid_entries(plan, ne, nbra, pl.data(), pn.data());
}

int64_t eri4_plan_work_size(eri4_plan plan) { return plan ? plan->work : -1; }

eri4_status eri4_plan_create_coulomb(eri4_plan* plan, int64_t nbra, const int32_t* bra_l, const int32_t* bra_nprim,
                                     int64_t nket, const int32_t* ket_l, const int32_t* ket_nprim, int kmax) {
  g_err.clear();
  if (!plan) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL plan pointer");
  *plan = nullptr;
  if (nbra < 0 || nket < 0) return fail(ERI4_ERROR_INVALID_ARGUMENT, "negative list length");
  if (nbra > 0 && nket > (((int64_t)1 << 31) - 1) / nbra)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "nbra * nket must be below 2^31");
  if ((nbra > 0 && (!bra_l || !bra_nprim)) || (nket > 0 && (!ket_l || !ket_nprim)))
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL host array");
  const int64_t nq = nbra * nket;
  std::vector<int32_t> l(4 * nq), np(4 * nq);
  for (int64_t i = 0; i < nbra; ++i)
    for (int64_t j = 0; j < nket; ++j) {
      const int64_t q = i * nket + j;
      l[4 * q] = bra_l[2 * i], l[4 * q + 1] = bra_l[2 * i + 1];
      l[4 * q + 2] = ket_l[2 * j], l[4 * q + 3] = ket_l[2 * j + 1];
      np[4 * q] = bra_nprim[2 * i], np[4 * q + 1] = bra_nprim[2 * i + 1];
      np[4 * q + 2] = ket_nprim[2 * j], np[4 * q + 3] = ket_nprim[2 * j + 1];
    }
  eri4_status st = plan_create(plan, nq, l.data(), np.data(), kmax, ERI4_PREC_FP64, nullptr, 0, true, nbra, nket,
                               false, true);
  if (st != ERI4_SUCCESS) return st;
  eri4_plan_s* p = *plan;
  // workspace: dket of every ket entry (kmax^2 slots), then the quartets' J rows
  const int64_t ne = nbra + nket;
  std::vector<int32_t> pl(2 * ne), pn(2 * ne);
  std::vector<int64_t> doff(std::max<int64_t>(1, nket)), dkoff(std::max<int64_t>(1, nket)), joff(nbra);
  for (int64_t e = 0; e < ne; ++e) {
    const bool ket = e >= nbra;
    const int64_t i = ket ? e - nbra : e;
    pl[2 * e] = (ket ? ket_l : bra_l)[2 * i], pl[2 * e + 1] = (ket ? ket_l : bra_l)[2 * i + 1];
    pn[2 * e] = (ket ? ket_nprim : bra_nprim)[2 * i], pn[2 * e + 1] = (ket ? ket_nprim : bra_nprim)[2 * i + 1];
  }
  int64_t od = 0, ok_ = 0, oj = 0;
  for (int64_t j = 0; j < nket; ++j) {
    const int lc = ket_l[2 * j], ld = ket_l[2 * j + 1];
    doff[j] = od;
    od += (int64_t)ncart(lc) * ncart(ld);
    dkoff[j] = ok_;
    ok_ += (int64_t)kmax * kmax * 16 * ((nherm(lc + ld) + 15) / 16);
  }
  for (int64_t i = 0; i < nbra; ++i) {
    joff[i] = oj;
    oj += (int64_t)ncart(bra_l[2 * i]) * ncart(bra_l[2 * i + 1]);
  }
  p->dket_size = ok_;
  p->work = ok_ + p->out_size;  // out_size so far: the quartets' J rows
  p->out_size = oj;
  p->ooff = joff;
  p->ket_dens_size = od;
  const bool ok = hipMalloc(&p->d_pl, std::max<int64_t>(1, 2 * ne) * sizeof(int32_t)) == hipSuccess &&
                  hipMalloc(&p->d_pn, std::max<int64_t>(1, 2 * ne) * sizeof(int32_t)) == hipSuccess &&
                  hipMalloc(&p->d_doff, doff.size() * sizeof(int64_t)) == hipSuccess &&
                  hipMalloc(&p->d_dkoff, dkoff.size() * sizeof(int64_t)) == hipSuccess &&
                  hipMalloc(&p->d_joff, std::max<int64_t>(1, nbra) * sizeof(int64_t)) == hipSuccess;
  hipError_t e = ok ? hipSuccess : hipErrorOutOfMemory;
  if (e == hipSuccess && ne > 0) e = hipMemcpy(p->d_pl, pl.data(), 2 * ne * sizeof(int32_t), hipMemcpyHostToDevice);
  if (e == hipSuccess && ne > 0) e = hipMemcpy(p->d_pn, pn.data(), 2 * ne * sizeof(int32_t), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(p->d_doff, doff.data(), doff.size() * sizeof(int64_t), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(p->d_dkoff, dkoff.data(), dkoff.size() * sizeof(int64_t), hipMemcpyHostToDevice);
  if (e == hipSuccess && nbra > 0) e = hipMemcpy(p->d_joff, joff.data(), nbra * sizeof(int64_t), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    plan_free(p);
    *plan = nullptr;
    return ok ? fail(ERI4_ERROR_HIP, "plan upload: %s", hipGetErrorString(e))
              : fail(ERI4_ERROR_OUT_OF_MEMORY, "device allocation for the plan failed");
  }
  return ERI4_SUCCESS;
}

eri4_status eri4_plan_execute_coulomb(eri4_plan plan, const double* bra_centers, const double* bra_exponents,
                                      const double* bra_coeffs, const double* ket_centers,
                                      const double* ket_exponents, const double* ket_coeffs, const double* ket_dens,
                                      double* work, int64_t work_size, double* out, hipStream_t stream) {
  g_err.clear();
  if (!plan) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL plan");
  if (!plan->coul) return fail(ERI4_ERROR_INVALID_ARGUMENT, "not a Coulomb plan (eri4_plan_create_coulomb)");
  if (plan->nitems + plan->nlow == 0) {
    // an empty ket list: every J_i is an empty sum
    if (plan->out_size == 0) return ERI4_SUCCESS;
    if (!out) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
    const int64_t nb = std::min<int64_t>((plan->out_size + 255) / 256, 4096);
    hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)nb), dim3(256), 0, stream, out, plan->out_size);
    HIP_TRY(hipGetLastError());
    return ERI4_SUCCESS;
  }
  if (!bra_centers || !bra_exponents || !bra_coeffs || !ket_centers || !ket_exponents || !ket_coeffs || !ket_dens ||
      !out)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
  if (!work || work_size < plan->work)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "workspace of %lld doubles is below the plan's %lld",
                (long long)(work ? work_size : 0), (long long)plan->work);
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev != plan->device)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "plan was made for device %d, current device is %d", plan->device, dev);
  DeviceState* d;
  eri4_status st = ensure_device(&d);
  if (st != ERI4_SUCCESS) return st;
  hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, stream, plan->d_counter);
  HIP_TRY(hipGetLastError());
  const Shells shl{bra_centers, bra_exponents, bra_coeffs, ket_centers, ket_exponents, ket_coeffs, plan->nket};
  const PlanArgs a{plan->d_classes, plan->d_items, plan->nitems, plan->d_qoff, plan->d_nprim, plan->d_counter, shl,
                   nullptr};
  HIP_TRY(plan_coulomb_launch(dim3(plan->grid), plan->lds_bytes, stream, d->tables(), a,
                              (int)plan->nbra, plan->kmax, g_tix.uv, plan->d_pl, plan->d_pn, ket_dens, plan->d_doff,
                              plan->d_dkoff, plan->d_joff, work, work + plan->dket_size, out,
                              LowItems{plan->d_low, plan->d_items + plan->nitems, plan->nlow, jlow_waves(plan->kmax),
                                       plan->low_lds}));
  return ERI4_SUCCESS;
}

eri4_status eri4_plan_execute_pairs(eri4_plan plan, const double* bra_centers, const double* bra_exponents,
                                    const double* bra_coeffs, const double* ket_centers,
                                    const double* ket_exponents, const double* ket_coeffs, double* work,
                                    int64_t work_size, double* out, hipStream_t stream) {
  g_err.clear();
  if (!plan) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL plan");
  if (!plan->pairs) return fail(ERI4_ERROR_INVALID_ARGUMENT, "plan made from quartets: use eri4_plan_execute");
  if (plan->coul) return fail(ERI4_ERROR_INVALID_ARGUMENT, "Coulomb plan: use eri4_plan_execute_coulomb");
  return plan_launch(plan,
                     Shells{bra_centers, bra_exponents, bra_coeffs, ket_centers, ket_exponents, ket_coeffs,
                            plan->nket},
                     work, work_size, out, stream);
}

eri4_status eri4_plan_destroy(eri4_plan plan) {
  g_err.clear();
  plan_free(plan);
  return ERI4_SUCCESS;
}

eri4_status eri4_boys(int mmax, int64_t n, const double* T, double* F, hipStream_t stream) {
  g_err.clear();
  if (mmax < 0 || mmax > ERI4_MAX_BOYS_M)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "mmax must be in 0..%d", ERI4_MAX_BOYS_M);
  if (n < 0) return fail(ERI4_ERROR_INVALID_ARGUMENT, "n must be >= 0");
  if (n == 0) return ERI4_SUCCESS;
  if (!T || !F) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
  DeviceState* d;
  eri4_status s = ensure_device(&d);
  if (s != ERI4_SUCCESS) return s;
  const int64_t total = n * (mmax + 1);
  const int64_t nb = (total + 255) / 256;
  if (nb > ((int64_t)1 << 31) - 1) return fail(ERI4_ERROR_INVALID_ARGUMENT, "n too large");
  hipLaunchKernelGGL(boys_kernel, dim3((unsigned)nb), dim3(256), 0, stream, mmax, n, T, F, d->boys);
  HIP_TRY(hipGetLastError());
  return ERI4_SUCCESS;
}

eri4_status eri4_hermite_r(int L, int64_t n, const double* zp, const double* zq, const double* P,
                           const double* Q, double* R, hipStream_t stream) {
  g_err.clear();
  if (L < 0 || L > 4 * ERI4_MAX_L)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "L must be in 0..%d", 4 * ERI4_MAX_L);
  if (n < 0) return fail(ERI4_ERROR_INVALID_ARGUMENT, "n must be >= 0");
  if (n == 0) return ERI4_SUCCESS;
  if (!zp || !zq || !P || !Q || !R) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
  if (n > ((int64_t)1 << 31) - 1) return fail(ERI4_ERROR_INVALID_ARGUMENT, "n too large");
  DeviceState* d;
  eri4_status s = ensure_device(&d);
  if (s != ERI4_SUCCESS) return s;
  const bool slab = L > kBoxLMax;
  StageR p{};
  p.L = L;
  p.ntask = g_tix.ntask[L]; p.o_uv = g_tix.uv; p.o_task = g_tix.task[L]; p.rtab_off = d->rstart[L];
  p.o_rowt = 32 * 8;
  p.o_rs = p.o_rowt + align16((L + 1) * (L + 1) * 2);
  p.o_rv = p.o_rs + align16(nuv(L) * 4);
  p.o_box = L <= kWaveL ? p.o_rowt + align16(nherm(L) * 8) : p.o_rv + align16(nuv(L) * 2);
  p.o_zt = p.o_box + align16((r_cells(slab, L) + (box_s1(L) == L + 1 ? L + 1 : 0)) * 8);
  p.o_h = p.o_zt + align16(nuv(L) * 8);
  p.lds_bytes = p.o_h + 3 * 64 * h_steps(L) * 8;
  const auto kernel = slab ? hermite_r_kernel<true> : hermite_r_kernel<false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(kThreads), p.lds_bytes, stream, p, d->tables(), zp, zq, P, Q, R);
  HIP_TRY(hipGetLastError());
  return ERI4_SUCCESS;
}

eri4_status eri4_hermite_e(int la, int lb, int64_t n, const double* za, const double* zb, const double* A,
                           const double* B, double* E, hipStream_t stream) {
  g_err.clear();
  if (la < 0 || lb < 0 || la > kTableLMax || lb > kTableLMax)
    return fail(ERI4_ERROR_INVALID_ARGUMENT, "la, lb must be in 0..%d", kTableLMax);
  if (n < 0) return fail(ERI4_ERROR_INVALID_ARGUMENT, "n must be >= 0");
  if (n == 0) return ERI4_SUCCESS;
  if (!za || !zb || !A || !B || !E) return fail(ERI4_ERROR_INVALID_ARGUMENT, "NULL buffer pointer");
  if (n > ((int64_t)1 << 31) - 1) return fail(ERI4_ERROR_INVALID_ARGUMENT, "n too large");
  DeviceState* d;
  eri4_status s = ensure_device(&d);
  if (s != ERI4_SUCCESS) return s;
  const int trow = odd_row(la + lb + 2);
  const int lds = 3 * ((la + 1) * (lb + 1) + 1) * trow * 8;
  hipLaunchKernelGGL(hermite_e_kernel, dim3((unsigned)n), dim3(64), lds, stream, la, lb, za, zb, A, B, E);
  HIP_TRY(hipGetLastError());
  return ERI4_SUCCESS;
}

}  // extern "C"
