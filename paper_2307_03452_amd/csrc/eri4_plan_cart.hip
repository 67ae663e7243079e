// eri4_plan_cart.hip -- the persistent kernel of dense Cartesian tiles, shells read from per-quartet arrays.
#include "eri4_plan_cart.h"

namespace eri4 {
hipError_t plan_set_attrs_cart() { return plan_cart_set_attrs_t<false>(); }
hipError_t plan_occupancy_cart(int lds_bytes, int* per_cu) { return plan_cart_occupancy_t<false>(lds_bytes, per_cu); }
hipError_t plan_launch_cart(dim3 grid, int lds_bytes, hipStream_t s, const Tables& t, const PlanArgs& a) {
  return plan_cart_launch_t<false>(grid, lds_bytes, s, t, a);
}
}  // namespace eri4
