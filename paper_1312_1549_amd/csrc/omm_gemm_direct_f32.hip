// FP32 instantiations of the small tiles (omm_gemm_direct.h), single and grouped launches.
#include "omm_gemm_direct.h"

namespace omm {
namespace gemm_detail {

gemm_fn pick_direct_f32(const GemmDesc& d) {
  const bool kk = d.la == KC && d.lb == KC, rr = d.la == RC && d.lb == RC;
  if (kk && d.ta == T_F32 && d.tb == T_F32 && d.tc == T_F32 && d.tx == T_F32)
    return pick_direct<CF32, float, float, float, float, KC, KC>(d.tile);
  if (kk && d.ta == T_F32 && d.tb == T_F32 && d.tc == T_F64 && d.tx == T_F64)
    return pick_direct<CF32, float, float, double, double, KC, KC>(d.tile);
  if (rr && d.ta == T_F64 && d.tb == T_F32 && d.tc == T_F32 && d.tx == T_F32)
    return pick_direct<CF32, double, float, float, float, RC, RC>(d.tile);
  return nullptr;
}

grouped_fn pick_grouped_f32(const GemmDesc& d) {
  const bool kk = d.la == KC && d.lb == KC, rr = d.la == RC && d.lb == RC;
  if (kk && d.ta == T_F32 && d.tb == T_F32 && d.tc == T_F32 && d.tx == T_F32)
    return pick_direct_grouped<CF32, float, float, float, float, KC, KC>(d.tile);
  if (kk && d.ta == T_F32 && d.tb == T_F32 && d.tc == T_F64 && d.tx == T_F64)
    return pick_direct_grouped<CF32, float, float, double, double, KC, KC>(d.tile);
  if (rr && d.ta == T_F64 && d.tb == T_F32 && d.tc == T_F32 && d.tx == T_F32)
    return pick_direct_grouped<CF32, double, float, float, float, RC, RC>(d.tile);
  return nullptr;
}

}  // namespace gemm_detail
}  // namespace omm
