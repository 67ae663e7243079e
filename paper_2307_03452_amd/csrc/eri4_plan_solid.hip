// eri4_plan_solid.hip -- the persistent kernel of solid-harmonic plans, shells read from per-quartet arrays.
#include "eri4_plan_solid.h"

namespace eri4 {
hipError_t plan_set_attrs_solid() { return plan_solid_set_attrs_t<false>(); }
hipError_t plan_occupancy_solid(int lds_bytes, int* per_cu) { return plan_solid_occupancy_t<false>(lds_bytes, per_cu); }
hipError_t plan_launch_solid(dim3 grid, int lds_bytes, hipStream_t s, const Tables& t, const PlanArgs& a, int64_t nbra,
                                 const int64_t* hoff, const double* h) {
  return plan_solid_launch_t<false>(grid, lds_bytes, s, t, a, nbra, hoff, h);
}
}  // namespace eri4
