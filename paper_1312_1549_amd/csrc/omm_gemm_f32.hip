// FP32 MFMA GEMM instantiations (v_mfma_f32_16x16x4f32), staged tiles. Operands: FP32, with FP32 or
// FP64 output, or (the gradient) an FP64 A.
#include "omm_gemm_impl.h"

namespace omm {
namespace gemm_detail {

gemm_fn pick_direct_f32(const GemmDesc& d);

gemm_fn pick_f32(const GemmDesc& d) {
  if (tile_direct(d.tile)) return pick_direct_f32(d);
  const bool kk = d.la == KC && d.lb == KC, rr = d.la == RC && d.lb == RC;
  if (kk && d.ta == T_F32 && d.tb == T_F32 && d.tc == T_F32 && d.tx == T_F32)
    return pick_tile<CF32, float, float, float, float, KC, KC>(d.tile);
  if (kk && d.ta == T_F32 && d.tb == T_F32 && d.tc == T_F64 && d.tx == T_F64)
    return pick_tile<CF32, float, float, double, double, KC, KC>(d.tile);
  if (rr && d.ta == T_F64 && d.tb == T_F32 && d.tc == T_F32 && d.tx == T_F32)
    return pick_tile<CF32, double, float, float, float, RC, RC>(d.tile);
  return nullptr;
}

}  // namespace gemm_detail
}  // namespace omm
