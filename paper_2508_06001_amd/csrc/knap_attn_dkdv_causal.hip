// dK/dV kernel, causal mask.
#include "knap_attn_dkdv.h"

namespace knap {

hipError_t launch_dkdv_causal(const DkdvArgs& a, int d, int pairs, int cus, hipStream_t stream) {
  return launch_dkdv_m<true>(a, d, pairs, cus, stream);
}

}  // namespace knap
