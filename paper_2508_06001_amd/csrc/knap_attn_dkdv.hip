// dK/dV kernel, bidirectional mask.
#include "knap_attn_dkdv.h"

namespace knap {

hipError_t launch_dkdv(const DkdvArgs& a, int d, int pairs, int cus, hipStream_t stream) {
  return launch_dkdv_m<false>(a, d, pairs, cus, stream);
}

}  // namespace knap
