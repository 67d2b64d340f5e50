// Internal launch interface between the C-ABI layer and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "knap_dispatch.h"

namespace knap {

// the forward without the mask (knap_attn_fwd_full.hip) and the causal one (knap_attn_fwd.hip)
hipError_t launch_fwd_full(const void* q, const void* k, const void* v, const int32_t* cu, int n_seq, int H, int d, float scale,
                           void* out, float* lse, unsigned* counters, int grid, hipStream_t stream);
hipError_t launch_fwd_causal(const void* q, const void* k, const void* v, const int32_t* cu, int n_seq, int H, int d, float scale,
                             void* out, float* lse, unsigned* counters, int grid, hipStream_t stream);

// Device address (on the current device) of the forward's work-queue counters: kQueueSets sets of 8, at zero
// whenever no kernel uses them; nullptr on failure.
unsigned* queue_base();
hipError_t clear_queue_sets(unsigned* first, unsigned sets, hipStream_t stream);

struct BwdArgs {
  const void *q, *k, *v, *out, *dout;
  const float* lse;
  const int32_t* cu;
  int n_seq, H;
  float scale;
  void *dq, *dk, *dv;
  float *delta, *lse2;      // (H, T) each, -delta and the base-2 LSE, handed from the dQ kernel to the dK/dV kernel
  unsigned* counters;       // 8 for the dQ kernel, 8 for the dK/dV kernel; the launches clear them, they may hold anything
};
// `dkdv_pairs`: wave pairs (2 or 4) per workgroup of the dK/dV kernel
hipError_t launch_bwd(const BwdArgs& a, int d, bool causal, int dkdv_pairs, int cus, int dq_wg_per_cu, hipStream_t stream,
                      hipEvent_t ev_start, hipEvent_t ev_stop);
// both kinds of items in one launch, T tokens, behind the kernel that forms delta: tiles of 128 rows (knap_attn_joint.h) or, `small`, of 64
// (knap_attn_bwd_small.hip)
constexpr int kSmallPays = 8;      // behind the counters of the launch's queues: whether items of 64 rows pay, where that is decided on the device
hipError_t launch_joint(const BwdArgs& a, int d, bool causal, bool small, int T, int cus, hipStream_t stream, hipEvent_t ev_start,
                        hipEvent_t ev_stop);
hipError_t launch_small(const BwdArgs& a, int d, bool causal, bool sure, int cus, hipStream_t stream);
hipError_t launch_joint_causal(const BwdArgs& a, int d, int cus, hipStream_t stream);
hipError_t launch_dq_causal(const BwdArgs& a, int d, int cus, int wg_per_cu, hipStream_t stream);
hipError_t launch_dkdv_causal(const BwdArgs& a, int d, int pairs, int cus, hipStream_t stream);

// Ulysses layout switch, local data movement; rows of U 16-byte units.
hipError_t launch_ulysses_heads(const void* src, void* dst, uint32_t T, uint32_t U, uint32_t g, bool pack,
                                hipStream_t stream);
hipError_t launch_ulysses_rows(const void* src, void* dst, const int32_t* row_map, uint32_t T, uint32_t U,
                               bool gather, hipStream_t stream);
hipError_t launch_ulysses_plan(const int32_t* cu, int n_seq, int g, int T, int32_t* row_map, hipStream_t stream);

// resident workgroups per compute unit of the persistent kernels
int fwd_workgroups_per_cu(int d);
int bwd_dq_workgroups_per_cu(int d);

}  // namespace knap
