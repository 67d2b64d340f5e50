// Backward of bags whose items fill the GPU only a few times: the items of the dK/dV kernel (128 keys, two wave pairs) and of
// the dQ kernel (128 queries) in one launch, so that there is one thin last round instead of two and the second kind starts
// where the first one runs out.  delta and the LSE in base 2, which both need, come from a kernel of their own in front
// (otherwise the dQ kernel forms them on the way; 3 us where out is still in the caches).  bwd_joint() chooses, and has both
// sides measured.  One text, compiled for either mask in a translation unit of its own.
#pragma once

#include "knap_attn_dkdv.h"
#include "knap_attn_dq.h"

namespace knap {

// LDS of the launch.  Four arrays that hold a K or V tile each for one kind, and a tile of Q and of dO (or the P of the pairs) for the
// other: whatever is copied into while another is read is an array of its own, so that the reads are known not to depend on it.
template <int D>
struct JointLds {
  static constexpr int HALF = Bwd2Cfg<D, 2>::TILE_ELEMS, P_ELEMS = 2 * DkdvLane<D, 2>::P_PAIR / (int)sizeof(__bf16);
  static_assert(DqCfg<D>::TILE_ELEMS == 2 * HALF && P_ELEMS >= 2 * HALF, "the arrays serve both kinds");
  __bf16 *a0, *a1, *a2, *a3;       // 2 HALF each, P_ELEMS the last
  float *lse0, *delta0, *lse1, *delta1, *lse2, *delta2, *sink;      // 64 each
  int* ticket;
  int *order, *start;              // of the schedule, n_seq and n_seq + 1
};

#define KNAP_JOINT_LDS(D, lds)                                                                                                   \
  extern __shared__ int s_dyn[];                                                                                                 \
  __shared__ __attribute__((aligned(1024))) __bf16 sA0[2 * JointLds<D>::HALF];                                                   \
  __shared__ __attribute__((aligned(1024))) __bf16 sA1[2 * JointLds<D>::HALF];                                                   \
  __shared__ __attribute__((aligned(1024))) __bf16 sA2[2 * JointLds<D>::HALF];                                                   \
  __shared__ __attribute__((aligned(1024))) __bf16 sA3[JointLds<D>::P_ELEMS];                                                    \
  __shared__ __attribute__((aligned(256))) float sLse0[64], sDelta0[64], sLse1[64], sDelta1[64], sLse2[64], sDelta2[64], sSink[64]; \
  __shared__ int s_ticket;                                                                                                       \
  const JointLds<D> lds = {sA0, sA1, sA2, sA3, sLse0, sDelta0, sLse1, sDelta1, sLse2, sDelta2, sSink, &s_ticket, s_dyn, s_dyn + n_seq}

// all items of a launch, tiles of 128 rows, behind their schedule
template <int D, bool CAUSAL>
__device__ __forceinline__ void joint_items(const BwdPtrs& g, const JointLds<D>& lds, const int32_t* __restrict__ cu, int n_seq, int H,
                                            unsigned* __restrict__ counters) {
  using KV = Bwd2Cfg<D, 2>;
  constexpr int BM = 128;                          // rows of a tile of either kind
  static_assert(KV::BN == BM && DqCfg<D>::BM == BM, "one schedule serves both");
  constexpr int HALF = JointLds<D>::HALF;
  int *const s_order = lds.order, *const s_start = lds.start;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int role = (wave >> 1) ^ ((int)(blockIdx.x * dkdv_workgroups_per_cu(D, 2) / gridDim.x) & 1);
  const uint32_t row_bytes = (uint32_t)((size_t)H * D * sizeof(__bf16));
  const DkdvLds kv_lds = {lds.a0, lds.a0 + HALF, lds.a1, lds.a1 + HALF, lds.a2, lds.a2 + HALF, lds.lse0, lds.delta0, lds.lse1, lds.delta1,
                          lds.lse2, lds.delta2, lds.sink, reinterpret_cast<u32x4*>(lds.a3)};
  const DqLds q_lds = {lds.a0, lds.a1, lds.a2, lds.a3};

  // the first kind are the key tiles (the dearer ones), the second the query tiles
  constexpr int SPLIT = CAUSAL ? 4 : 2;     // narrow items (64 queries) of a query tile, or of a pair of them
  EvenQueue<SPLIT, 2> queue;
  queue.init(counters);
  if (wave == 0) even_shares(queue, n_seq, s_start, lane);
  __syncthreads();
  deal_even<BM, CAUSAL>(queue, cu, n_seq, s_order, s_start);
  // item i of this queue's, of either kind
  auto take = [&](int i) {
    WorkItem it = decode_even<BM, CAUSAL>(i, queue, cu, n_seq, H, s_order, s_start);
    it.head = __builtin_amdgcn_readfirstlane(it.head);
    it.tile = __builtin_amdgcn_readfirstlane(it.tile);
    return it;
  };
  int ticket = queue.first_ticket();
  while (ticket < queue.wide + queue.parts) {
    const bool whole = ticket < queue.wide, keys = whole && queue.first_kind(ticket);
    const int part = ticket - queue.wide;
    const WorkItem it = take(whole ? queue.item(ticket) : queue.item_of_part(part));
    // The next ticket is drawn in front of the item's stores, under which it arrives.  Drawn at the item's start, the items
    // behind the first round went to the workgroups that had started first, with the longest ones.  Forward and backward in
    // us, start -> end: 7250 tokens and 24 short sequences, 6 x 128, 842 -> 713; 4292, 24 x 128, 964 -> 923; 10000 and 33
    // short ones, 12 x 128, 2660 -> 2498; 10 of 310..6795, 48 x 64, 5760 -> 5692; but 9000 and 30, 6 x 128, 1143 -> 1175.
    unsigned next_ticket;      // thread 0 only; no initial value, which would be merged in (and waited for) at once
    auto draw = [&] { if (tid == 0 && queue.draws) next_ticket = atomicAdd(queue.ctr, 1u); };
    // CAUSAL: the item is the pair of tiles {p, tiles - 1 - p}, the dearer one first; the middle tile of an odd count stands alone
    const int other = (it.len + BM - 1) / BM - 1 - it.tile;
    const int n_sub = CAUSAL && other != it.tile ? 2 : 1;
    int ln = lane;
    asm volatile("" : "+v"(ln));      // what follows from the lane is formed per item, not kept through the other kind's
    if (keys) {
      DkdvLane<D, 2> me;
      me.init(ln, wave, role, row_bytes);
#pragma unroll 1
      for (int sub = 0; sub < n_sub; ++sub)
        dkdv_tile<D, 2, CAUSAL>(g, kv_lds, me, it, sub == 0 ? it.tile : other, [] {}, [] {}, [&] { if (sub == n_sub - 1) draw(); });
    } else {
      const int from = whole ? 0 : (part % SPLIT) >> 1, to = whole ? n_sub : from + 1;
#pragma unroll 1
      for (int sub = from; sub < to; ++sub) {
        const int q_tile = CAUSAL && sub == 0 ? other : it.tile;
        const int q0 = q_tile * BM + (whole ? 0 : 64 * (part & 1));
        asm volatile("" : "+v"(ln));
        DqLane<D> me;
        me.init(ln, wave);
        auto ending = [&] { if (sub == to - 1) draw(); };
        if (whole && !dq_narrow(it.len, q_tile)) dq_tile<D, CAUSAL, false>(g, q_lds, me, it, q_tile, [] {}, ending);
        else if (q0 < it.len && sub < n_sub) dq_part<D, CAUSAL, false>(g, q_lds, me, it, q0, [] {}, ending);
        else ending();
      }
    }
    if (!queue.draws) return;
    if (tid == 0) *lds.ticket = queue.later_ticket(next_ticket);
    lds_barrier();                    // (and the partial sums of a narrow tile are no longer read)
    ticket = __builtin_amdgcn_readfirstlane(*lds.ticket);
    if (ticket >= queue.wide) lds_barrier();        // every wave has the ticket before the next one is put down: a part may have no rows
  }
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_bwd_joint_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v, const __bf16* __restrict__ dout,
    float* __restrict__ lse2, float* __restrict__ delta, const int32_t* __restrict__ cu, int n_seq, int H, float scale,
    __bf16* __restrict__ dq, __bf16* __restrict__ dk, __bf16* __restrict__ dv, unsigned* __restrict__ counters) {
  KNAP_JOINT_LDS(D, lds);
  const BwdPtrs g = {q, k, v, nullptr, dout, nullptr, lse2, delta, dq, dk, dv, cu[n_seq], H, scale};
  build_schedule<128, kThreads, CAUSAL>(cu, n_seq, H, lds.order, lds.start, reinterpret_cast<int*>(sA0));
  joint_items<D, CAUSAL>(g, lds, cu, n_seq, H, counters);
}

template <bool CAUSAL>
static hipError_t launch_joint_m(const BwdArgs& a, int d, int cus, hipStream_t stream) {
  const size_t dyn = (size_t)(2 * a.n_seq + 1) * sizeof(int);
  auto* joint = d == 64 ? attn_bwd_joint_kernel<64, CAUSAL> : attn_bwd_joint_kernel<128, CAUSAL>;
  hipLaunchKernelGGL(joint, dim3(cus * dkdv_workgroups_per_cu(d, 2)), dim3(kThreads), dyn, stream, (const __bf16*)a.q,
                     (const __bf16*)a.k, (const __bf16*)a.v, (const __bf16*)a.dout, a.lse2, a.delta, a.cu, a.n_seq, a.H, a.scale,
                     (__bf16*)a.dq, (__bf16*)a.dk, (__bf16*)a.dv, a.counters);
  return hipGetLastError();
}

}  // namespace knap
