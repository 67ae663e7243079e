// eri4_plan_cartp.hip -- the persistent kernel of dense Cartesian tiles, shells read from a bra and a ket list of shell pairs.
#include "eri4_plan_cart.h"

namespace eri4 {
hipError_t plan_set_attrs_cartp() { return plan_cart_set_attrs_t<true>(); }
hipError_t plan_occupancy_cartp(int lds_bytes, int* per_cu) { return plan_cart_occupancy_t<true>(lds_bytes, per_cu); }
hipError_t plan_launch_cartp(dim3 grid, int lds_bytes, hipStream_t s, const Tables& t, const PlanArgs& a) {
  return plan_cart_launch_t<true>(grid, lds_bytes, s, t, a);
}
}  // namespace eri4
