// The separate kernels' bfloat16 instances, and the EMA update (which reads no 16-bit data).
#include "prr_sep.h"

namespace prr {

template hipError_t launch_score_topk_t<true>(ScoreLaunch, hipStream_t);
template hipError_t launch_spec_attn_t<true>(const SpecLaunch&, hipStream_t);
template hipError_t launch_select_spec_t<true>(ScoreLaunch, const SpecLaunch&, hipStream_t);
template hipError_t launch_repair_t<true>(const RepairLaunch&, hipStream_t);
template hipError_t launch_repair_predict_t<true>(const RepairLaunch&, PredictLaunch, hipStream_t);

hipError_t launch_ema_topk(PredictLaunch a, hipStream_t stream) {
  if (!predict_spread(a)) return launch_predict(a, stream);
  plan_predict(a);
  return launch((const void*)ema_topk_kernel, dim3(a.nblk, a.num_kv_heads), stream, a);
}

}  // namespace prr
