// The separate kernels' float16 instances.
#include "prr_sep.h"

namespace prr {

template hipError_t launch_score_topk_t<false>(ScoreLaunch, hipStream_t);
template hipError_t launch_spec_attn_t<false>(const SpecLaunch&, hipStream_t);
template hipError_t launch_select_spec_t<false>(ScoreLaunch, const SpecLaunch&, hipStream_t);
template hipError_t launch_repair_t<false>(const RepairLaunch&, hipStream_t);
template hipError_t launch_repair_predict_t<false>(const RepairLaunch&, PredictLaunch, hipStream_t);

}  // namespace prr
