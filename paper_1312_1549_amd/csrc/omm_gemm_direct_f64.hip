// FP64 instantiations of the small tiles (omm_gemm_direct.h), single and grouped launches.
#include "omm_gemm_direct.h"

namespace omm {
namespace gemm_detail {

gemm_fn pick_direct_f64(const GemmDesc& d) {
  if (d.la == KC && d.lb == KC) return pick_direct<CF64, double, double, double, double, KC, KC>(d.tile);
  if (d.la == KC && d.lb == RC) return pick_direct<CF64, double, double, double, double, KC, RC>(d.tile);
  if (d.la == RC && d.lb == RC) return pick_direct<CF64, double, double, double, double, RC, RC>(d.tile);
  return nullptr;
}

grouped_fn pick_grouped_f64(const GemmDesc& d) {
  if (d.ta != T_F64 || d.tb != T_F64 || d.tc != T_F64 || d.tx != T_F64) return nullptr;
  if (d.la == KC && d.lb == KC)
    return pick_direct_grouped<CF64, double, double, double, double, KC, KC>(d.tile);
  if (d.la == RC && d.lb == RC)
    return pick_direct_grouped<CF64, double, double, double, double, RC, RC>(d.tile);
  return nullptr;
}

}  // namespace gemm_detail
}  // namespace omm
