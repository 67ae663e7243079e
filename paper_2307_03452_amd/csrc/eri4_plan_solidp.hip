// eri4_plan_solidp.hip -- the persistent kernel of solid-harmonic plans, shells read from a bra and a ket list of shell pairs.
#include "eri4_plan_solid.h"

namespace eri4 {
hipError_t plan_set_attrs_solidp() { return plan_solid_set_attrs_t<true>(); }
hipError_t plan_occupancy_solidp(int lds_bytes, int* per_cu) { return plan_solid_occupancy_t<true>(lds_bytes, per_cu); }
hipError_t plan_launch_solidp(dim3 grid, int lds_bytes, hipStream_t s, const Tables& t, const PlanArgs& a, int64_t nbra,
                                 const int64_t* hoff, const double* h) {
  return plan_solid_launch_t<true>(grid, lds_bytes, s, t, a, nbra, hoff, h);
}
}  // namespace eri4
