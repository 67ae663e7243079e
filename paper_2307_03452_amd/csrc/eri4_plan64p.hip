// eri4_plan64p.hip -- the persistent plan kernel with FP64 transforms, shells read from a bra and a ket list of shell pairs.
#include "eri4_plan.h"

namespace eri4 {
hipError_t plan_set_attrs_f64p() { return plan_set_attrs_t<false, true>(); }
hipError_t plan_occupancy_f64p(int lds_bytes, int* per_cu) {
  return plan_occupancy_t<false, true>(lds_bytes, per_cu);
}
hipError_t plan_launch_f64p(dim3 grid, int lds_bytes, hipStream_t s, const Tables& t, const PlanArgs& a) {
  return plan_launch_t<false, true>(grid, lds_bytes, s, t, a);
}
}  // namespace eri4
