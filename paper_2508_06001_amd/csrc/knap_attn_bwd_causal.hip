// The backward's kernels under the causal mask.
#include "knap_attn_joint.h"

namespace knap {

hipError_t launch_dq_causal(const BwdArgs& a, int d, int cus, int wg_per_cu, hipStream_t stream) {
  return launch_dq_m<true>(a, d, cus, wg_per_cu, stream);
}

hipError_t launch_dkdv_causal(const BwdArgs& a, int d, int pairs, int cus, hipStream_t stream) {
  return launch_dkdv_m<true>(a, d, pairs, cus, stream);
}

hipError_t launch_joint_causal(const BwdArgs& a, int d, int cus, hipStream_t stream) {
  return launch_joint_m<true>(a, d, cus, stream);
}

}  // namespace knap
