// Backward of bags whose items fill the GPU only a few times: the items of the dK/dV kernel (128 keys, two wave pairs) and of
// the dQ kernel (128 queries) in one launch, so that there is one thin last round instead of two and the second kind starts
// where the first one runs out.  delta and the LSE in base 2, which both need, come from a kernel of their own in front
// (otherwise the dQ kernel forms them on the way; 3 us where out is still in the caches).  bwd_joint() chooses, and has both
// sides measured.  One text, compiled for either mask in a translation unit of its own.
#pragma once

#include "knap_attn_dkdv.h"
#include "knap_attn_dq.h"

namespace knap {

// What items of 64 rows need of the LDS
template <int D>
struct SmallLds {
  __bf16 *a0, *a1, *a2, *a3;                       // a tile of 64 rows each
  float *lse0, *delta0, *lse1, *delta1, *sink;     // 64 each
  int* ticket;
};

// All items of a launch in tiles of 64 rows, behind their schedule (knap_attn_bwd_small.hip)
template <int D, bool CAUSAL>
__device__ __forceinline__ void small_items(const BwdPtrs g, const SmallLds<D> s, const int32_t* __restrict__ cu, int n_seq, int H,
                                            const int* s_order, int* s_start, unsigned* __restrict__ counters);

// EITHER: the kernel in front has decided, by the lengths, whether the items are of 64 rows (small_pays()).
template <int D, bool CAUSAL, bool EITHER>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_bwd_joint_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v, const __bf16* __restrict__ dout,
    float* __restrict__ lse2, float* __restrict__ delta, const int32_t* __restrict__ cu, int n_seq, int H, float scale,
    __bf16* __restrict__ dq, __bf16* __restrict__ dk, __bf16* __restrict__ dv, unsigned* __restrict__ counters) {
  using KV = Bwd2Cfg<D, 2>;
  constexpr int BM = 128;                          // rows of a tile of either kind
  static_assert(KV::BN == BM && DqCfg<D>::BM == BM, "one schedule serves both");
  extern __shared__ int s_dyn[];
  int* s_order = s_dyn;
  int* s_start = s_dyn + n_seq;
  // Four arrays that hold a K or V tile each for one kind, and a tile of Q and of dO (or the P of the pairs) for the other:
  // whatever is copied into while another is read is an array of its own, so that the reads are known not to depend on it.
  constexpr int HALF = KV::TILE_ELEMS, P_ELEMS = 2 * DkdvLane<D, 2>::P_PAIR / (int)sizeof(__bf16);
  static_assert(DqCfg<D>::TILE_ELEMS == 2 * HALF && P_ELEMS >= 2 * HALF, "the arrays serve both kinds");
  __shared__ __attribute__((aligned(1024))) __bf16 sA0[2 * HALF];
  __shared__ __attribute__((aligned(1024))) __bf16 sA1[2 * HALF];
  __shared__ __attribute__((aligned(1024))) __bf16 sA2[2 * HALF];
  __shared__ __attribute__((aligned(1024))) __bf16 sA3[P_ELEMS];
  __shared__ __attribute__((aligned(256))) float sLse0[64], sDelta0[64], sLse1[64], sDelta1[64], sLse2[64], sDelta2[64], sSink[64];
  __shared__ int s_ticket;

  const int T = cu[n_seq];
  if constexpr (EITHER) {
    const unsigned pays = counters[kSmallPays];    // (arrives with the lengths)
    build_schedule_of(cu, n_seq, [&](int len) {
      const int wide = items_per_head<CAUSAL>((len + BM - 1) / BM), tiles = (len + 63) / 64;
      return (pays ? tiles : wide) * H;
    }, s_order, s_start, reinterpret_cast<int*>(&sA0[0]));
    if (__builtin_amdgcn_readfirstlane(pays)) {
      const BwdPtrs all = {q, k, v, nullptr, dout, nullptr, lse2, delta, dq, dk, dv, T, H, scale};
      const SmallLds<D> lds = {sA0, sA1, sA2, sA3, sLse0, sDelta0, sLse1, sDelta1, sSink, &s_ticket};
      small_items<D, CAUSAL>(all, lds, cu, n_seq, H, s_order, s_start, counters);
      return;
    }
  } else {
    build_schedule<BM, kThreads, CAUSAL>(cu, n_seq, H, s_order, s_start, reinterpret_cast<int*>(&sA0[0]));
  }
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int role = (wave >> 1) ^ ((int)(blockIdx.x * dkdv_workgroups_per_cu(D, 2) / gridDim.x) & 1);
  const uint32_t row_bytes = (uint32_t)((size_t)H * D * sizeof(__bf16));
  const BwdPtrs g = {q, k, v, nullptr, dout, nullptr, lse2, delta, dq, dk, dv, T, H, scale};
  const DkdvLds kv_lds = {sA0, sA0 + HALF, sA1, sA1 + HALF, sA2, sA2 + HALF, sLse0, sDelta0, sLse1, sDelta1, sLse2, sDelta2, sSink,
                          reinterpret_cast<u32x4*>(sA3)};
  const DqLds q_lds = {sA0, sA1, sA2, sA3};

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
    if (tid == 0) s_ticket = queue.later_ticket(next_ticket);
    lds_barrier();                    // (and the partial sums of a narrow tile are no longer read)
    ticket = __builtin_amdgcn_readfirstlane(s_ticket);
    if (ticket >= queue.wide) lds_barrier();        // every wave has the ticket before the next one is put down: a part may have no rows
  }
}

template <bool CAUSAL>
static hipError_t launch_joint_m(const BwdArgs& a, int d, int cus, hipStream_t stream) {
  const size_t dyn = (size_t)(2 * a.n_seq + 1) * sizeof(int);
  auto* joint = d == 64 ? attn_bwd_joint_kernel<64, CAUSAL, false> : attn_bwd_joint_kernel<128, CAUSAL, false>;
  hipLaunchKernelGGL(joint, dim3(cus * dkdv_workgroups_per_cu(d, 2)), dim3(kThreads), dyn, stream, (const __bf16*)a.q,
                     (const __bf16*)a.k, (const __bf16*)a.v, (const __bf16*)a.dout, a.lse2, a.delta, a.cu, a.n_seq, a.H, a.scale,
                     (__bf16*)a.dq, (__bf16*)a.dk, (__bf16*)a.dv, a.counters);
  return hipGetLastError();
}

}  // namespace knap
