// Backward kernels: gradients of sum(dout * out) with respect to q, k, v for
// packed block-diagonal attention, recomputing the probabilities from q, k and
// the forward's log-sum-exp (the training loop of Sec. 4 backpropagates through
// the attention of Sec. 3.4; Sec. 4.2 counts the backward as twice the forward).
//
//   delta_i = sum_c dO_ic O_ic
//   S = Q K^T, P = exp(scale S - LSE), dP = dO V^T, dS = P (dP - delta)
//   dQ = scale dS K                                    (by query tiles)
//   dV = P^T dO, dK = scale dS^T Q                     (by key tiles)
//
// dQ sums over keys and dK, dV sum over queries.  Doing all three in one pass
// needs a cross-workgroup reduction of one of them; on MI355X fp32 atomics into
// HBM-resident accumulators cap that design far below the MFMA rate (every
// atomic is a read-modify-write that leaves the XCD).  The backward therefore has
// two kinds of work items that each keep their accumulators in registers and recompute S and
// dP: seven contractions are issued for the five the mathematics needs, nothing
// is reduced across workgroups, and the result is bitwise reproducible.
//
// dK/dV items (knap_attn_dkdv.h): a workgroup of 8 or 4 waves owns a 256- or 128-row key/value tile of
// one (sequence, head) and walks over that sequence's queries 32 rows at a time; wave pairs split the work by
// output (one wave S, P, dV; its partner dP, dS, dK, one tile behind) so that each wave holds a
// single accumulator and two waves fit on a SIMD.  Details there.
//
// dQ items (knap_attn_dq.h): the forward kernel's structure.
//
// Bags that fill the GPU up to a dozen times hand out both kinds in one launch (knap_attn_joint.h; the smallest ones in items of half the
// rows, knap_attn_bwd_small.hip), with delta from a kernel in front of it; larger ones in two, dQ first, which forms delta on the way.
// bwd_joint() and bwd_small() in knap_dispatch.h choose.  This file holds the bidirectional kernels and the launches of both masks.
#include "knap_attn_joint.h"

namespace knap {

constexpr int kQueueCounters = 16;    // one work-queue counter per XCD for the dQ kernel, then one for the dK/dV kernel

// The work queues of the kernels that follow on the stream start at zero.  The counters lie in the call's workspace, as delta
// does: whatever else runs, no other call draws from them.
__global__ void bwd_queue_reset_kernel(unsigned* __restrict__ counters) {
  if (threadIdx.x < kQueueCounters) counters[threadIdx.x] = 0u;
}

hipError_t launch_bwd(const BwdArgs& a, int d, bool causal, int dkdv_pairs, int cus, int dq_wg_per_cu, hipStream_t stream,
                      hipEvent_t ev_start, hipEvent_t ev_stop) {
  hipLaunchKernelGGL(bwd_queue_reset_kernel, dim3(1), dim3(64), 0, stream, a.counters);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the dQ kernel also produces delta, which the dK/dV kernel needs: it goes first
  e = causal ? launch_dq_causal(a, d, cus, dq_wg_per_cu, stream) : launch_dq_m<false>(a, d, cus, dq_wg_per_cu, stream);
  if (e != hipSuccess) return e;
  if (ev_start && ev_stop && (e = hipEventRecord(ev_start, stream)) != hipSuccess) return e;
  e = causal ? launch_dkdv_causal(a, d, dkdv_pairs, cus, stream) : launch_dkdv_m<false>(a, d, dkdv_pairs, cus, stream);
  if (e != hipSuccess) return e;
  if (ev_start && ev_stop && (e = hipEventRecord(ev_stop, stream)) != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_joint(const BwdArgs& a, int d, bool causal, bool small, int T, int cus, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  hipError_t e = hipSuccess;
  if (ev_start && ev_stop && (e = hipEventRecord(ev_start, stream)) != hipSuccess) return e;
  if ((e = launch_delta(a, d, T, stream)) != hipSuccess) return e;
  e = small ? launch_small(a, d, causal, cus, stream) : causal ? launch_joint_causal(a, d, cus, stream) : launch_joint_m<false>(a, d, cus, stream);
  if (e != hipSuccess) return e;
  if (ev_start && ev_stop && (e = hipEventRecord(ev_stop, stream)) != hipSuccess) return e;
  return hipSuccess;
}

int bwd_dq_workgroups_per_cu(int d) {
  int n = 0;
  const void* fn = d == 64 ? (const void*)attn_bwd_dq_kernel<64, false> : (const void*)attn_bwd_dq_kernel<128, false>;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, kThreads, 0) != hipSuccess || n < 1) {
    (void)hipGetLastError();
    n = 1;
  }
  return n;
}

}  // namespace knap
