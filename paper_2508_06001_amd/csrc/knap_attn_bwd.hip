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

#include <type_traits>

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

// -delta and the LSE in base 2 of 128 rows of one head; bound by reading out and dout once (31464 tokens,
// 24 x 128: 67 us, 5.8 TB/s; 79 before).  The D / 8 lanes of a row hold 8 columns each, so that a load takes whole rows, and add up
// over the lanes.  With 32 bytes of 32 rows to a load, as the dQ kernel takes its rows, backward in us:
// 4 sequences of up to 311 tokens, 2 x 64, 11.5 against 11.0; 4 of 400, 24 x 128, 55.2 against 53.9; 17 of 328..4533 3228 against 3219.  out
// is not read again, and past the caches where it is large (32 of 1024, 12 x 64, 378 -> 374; 40 of 600, 24 x 128, 762 -> 753; but
// 4 of 400 54.2 -> 54.9).  It also clears the counters of the queues of the launch behind it, which therefore may hold
// anything (a caller's workspace) and need no launch of their own.
constexpr size_t kOutPastCaches = 20u << 20;        // elements

// One workgroup beside those with rows: which items the launch behind this one takes (small_pays()).
template <int D>
__device__ __forceinline__ void decide_small(const int32_t* __restrict__ cu, int n_seq, int H, unsigned* __restrict__ counters, int slots, bool causal) {
  __shared__ int s_tiles[kThreads / 64], s_longest[kThreads / 64];
  int tiles = 0, longest = 0;
  for (int i = threadIdx.x; i < n_seq; i += kThreads) {
    const int n = (cu[i + 1] - cu[i] + 63) / 64;
    tiles += n;
    longest = max(longest, n);
  }
  tiles = wave_scan(tiles);
  longest = wave_max(longest);
  if ((threadIdx.x & 63) == 63) {
    s_tiles[threadIdx.x >> 6] = tiles;
    s_longest[threadIdx.x >> 6] = longest;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    tiles = longest = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) {
      tiles += s_tiles[w];
      longest = max(longest, s_longest[w]);
    }
    counters[kSmallPays] = small_pays(tiles, longest, H, slots, D, causal) ? 1u : 0u;
  }
}

template <int D>
__global__ __launch_bounds__(kThreads) void attn_bwd_delta_kernel(
    const __bf16* __restrict__ out, const __bf16* __restrict__ dout, const float* __restrict__ lse,
    float* __restrict__ delta, float* __restrict__ lse2, const int32_t* __restrict__ cu, int n_seq, int H,
    unsigned* __restrict__ counters, int slots, bool causal) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 8) counters[threadIdx.x] = 0u;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t0 = blockIdx.x * 128, head = blockIdx.y, T = cu[n_seq];
  if (t0 >= T) {
    if (slots > 0 && head == 0 && blockIdx.x == gridDim.x - 1) decide_small<D>(cu, n_seq, H, counters, slots, causal);
    return;
  }
  const uint32_t row_bytes = (uint32_t)((size_t)H * D * sizeof(__bf16));
  const size_t at = ((size_t)t0 * H + head) * D;
  const uint32_t bytes = (uint32_t)min(T - t0, 128) * row_bytes;
  const auto ro = make_rsrc(out + at, bytes);
  const auto rd = make_rsrc(dout + at, bytes);
  constexpr int LANES = D / 8, ROWS = 64 / LANES, N = 32 / ROWS;      // lanes of a row, rows of a load, loads of a wave
  bf16x8 of[N], dof[N];
  const uint32_t off = (uint32_t)(wave * 32 + lane / LANES) * row_bytes + (uint32_t)(lane % LANES) * 16u;
  if ((size_t)T * H * D > kOutPastCaches) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      of[i] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(ro, (int)(off + (uint32_t)(i * ROWS) * row_bytes), 0, 2 /* nt */));
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) of[i] = __builtin_bit_cast(bf16x8, buffer_load16(ro, off + (uint32_t)(i * ROWS) * row_bytes));
  }
#pragma unroll
  for (int i = 0; i < N; ++i) dof[i] = __builtin_bit_cast(bf16x8, buffer_load16(rd, off + (uint32_t)(i * ROWS) * row_bytes));
  KNAP_SCHED_FENCE();
  float mine = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    float x = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) x = __builtin_fmaf((float)dof[i][e], (float)of[i][e], x);
    auto add = [&](auto ctrl) {
      x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    add(std::integral_constant<int, 0xb1>{});         // quad_perm 1, 0, 3, 2
    add(std::integral_constant<int, 0x4e>{});         // quad_perm 2, 3, 0, 1
    add(std::integral_constant<int, 0x141>{});        // row_half_mirror: the other four of eight
    if constexpr (D == 128) add(std::integral_constant<int, 0x140>{});        // row_mirror: the other eight of sixteen
    mine = lane % LANES == i ? x : mine;              // row ROWS i + lane / LANES of the wave's 32, kept by lane i of its row
  }
  const int t = t0 + wave * 32 + ROWS * (lane % LANES) + lane / LANES;
  if (lane % LANES < N && t < T) {
    const size_t row_at = (size_t)head * T + t;
    delta[row_at] = -mine;
    lse2[row_at] = lse[row_at] * kLog2e;
  }
}

// slots: of the workgroups of a launch behind it that asks for the decision on its items, else 0
static hipError_t launch_delta(const BwdArgs& a, int d, int T, int slots, bool causal, hipStream_t stream) {
  const dim3 rows((T + 127) / 128 + (slots > 0 ? 1 : 0), a.H);
  auto* delta = d == 64 ? attn_bwd_delta_kernel<64> : attn_bwd_delta_kernel<128>;
  hipLaunchKernelGGL(delta, rows, dim3(kThreads), 0, stream, (const __bf16*)a.out, (const __bf16*)a.dout, a.lse, a.delta, a.lse2, a.cu,
                     a.n_seq, a.H, a.counters, slots, causal);
  return hipGetLastError();
}

hipError_t launch_joint(const BwdArgs& a, int d, bool causal, bool small, int T, int cus, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  hipError_t e = hipSuccess;
  if (ev_start && ev_stop && (e = hipEventRecord(ev_start, stream)) != hipSuccess) return e;
  const bool sure = !small || small_sure(T, a.n_seq, a.H, d, causal, cus);
  if ((e = launch_delta(a, d, T, sure ? 0 : cus * dkdv_workgroups_per_cu(d, 2), causal, stream)) != hipSuccess) return e;
  e = small ? launch_small(a, d, causal, sure, cus, stream) : causal ? launch_joint_causal(a, d, cus, stream) : launch_joint_m<false>(a, d, cus, stream);
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
