// Backward of bags whose tiles of 128 rows would leave most of the GPU idle, either mask: both kinds of items in one launch, as in
// knap_attn_joint.h, but of 64 rows each, so that there are twice as many and each walks half as far in time.  What bounds such a bag is
// its longest item, one workgroup alone on a CU: a 128-key item takes a step of 32 queries after the other, 1.0 to 1.2 us each, and no part of it
// could go to an idle CU.  Under the mask the items are single tiles, the dearest first, and not pairs of equal cost.  bwd_small() and
// small_pays() in knap_dispatch.h choose and have both sides measured.
#include "knap_attn_joint.h"

namespace knap {

// dK and dV of 64 keys, from kv0 on.  Wave w holds 32 of them (w & 1), K and V rows and both accumulators, and takes every other 32
// queries (w >> 1): the walk over the sequence has half as many steps as that of a 128-key tile, and no wave waits for another's
// probabilities.  What bounds it is the latency of a step (a CU has one workgroup, a SIMD one wave): two chains of MFMAs, the
// exponentials, the other products, the barrier.  LDS operands are requested two MFMA groups ahead in fenced groups, so that nothing is
// spilled in the loops (one value of the causal kernel at d = 128 outside of them; with the order left to the compiler 46 were, reloaded in every step behind the tile copies: one of 1300 tokens, 3 x 128, backward
// 51 us, 48 with 128-key items, 32 so).  The two halves of the queries are added through LDS at the end.  `ending` is called
// in front of the stores.
template <int D, bool CAUSAL, class Ending>
__device__ __forceinline__ void dkdv_part(const BwdPtrs& g, const DqLds& lds, float* const (&scalars)[2][2], float* sink, const WorkItem& it,
                                          int kv0, int lane, int wave, Ending ending) {
  constexpr int KC = D / 16, DB = D / 32, BM = 64;       // queries of a step
  const int L = it.len, T = g.T, l32 = lane & 31, hh = lane >> 5;
  const int kb = __builtin_amdgcn_readfirstlane(wave & 1), half = __builtin_amdgcn_readfirstlane(wave >> 1);
  const float c = g.scale * kLog2e;
  const size_t row_stride = (size_t)g.H * D;
  const uint32_t row_bytes = (uint32_t)(row_stride * sizeof(__bf16));
  const size_t head_off = (size_t)it.head * D;
  __bf16 *const sQ0 = lds.k0, *const sQ1 = lds.k1, *const sdO0 = lds.v0, *const sdO1 = lds.v1;
  // the queries that these keys meet; steps count from the first of them
  const int q_first = CAUSAL ? kv0 : 0;
  const int Lq = L - q_first;
  const int n_steps = (Lq + BM - 1) / BM;
  const __bf16* q_base = g.q + (size_t)(it.row0 + q_first) * row_stride + head_off;
  const __bf16* do_base = g.dout + (size_t)(it.row0 + q_first) * row_stride + head_off;
  const size_t row_at = (size_t)it.head * T + it.row0 + q_first;
  constexpr int ROWS_PER_INSTR = 512 / D, COPIES = BM / (4 * ROWS_PER_INSTR);     // of a wave's share of a tile
  const int cp_row = wave * COPIES * ROWS_PER_INSTR + lane / Tile<D>::CPR;
  const uint32_t cp_off = (uint32_t)cp_row * row_bytes + (uint32_t)Tile<D>::chunk_pos(cp_row, lane % Tile<D>::CPR) * 16u;
  // rows past the end arrive as zeros in all four: P = exp2(0 - 0) = 1, but dO = 0 and dP - delta = 0
  auto load_step = [&](int t, __bf16* dQ, __bf16* ddO, float* dLse, float* dDelta) __attribute__((always_inline)) {
    const int q0 = t * BM, n_rows = max(0, min(Lq - q0, BM));
    const auto rq = make_rsrc(q_base + (size_t)q0 * row_stride, (uint32_t)n_rows * row_bytes);
    const auto rd = make_rsrc(do_base + (size_t)q0 * row_stride, (uint32_t)n_rows * row_bytes);
#pragma unroll
    for (int i = 0; i < COPIES; ++i) {
      uint32_t off = cp_off;
      if (i) asm volatile("" : "+v"(off));     // formed here, not kept in a register of its own through the loop
      // 4 i (D = 128) or 8 i (D = 64) rows further on the chunk's position differs by an exclusive or with i or 4 i
      off = (off ^ (uint32_t)((D == 128 ? i : 4 * i) * 16)) + (uint32_t)(i * ROWS_PER_INSTR) * row_bytes;
      const int at = (wave * COPIES + i) * ROWS_PER_INSTR * Tile<D>::LD;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rq, (__attribute__((address_space(3))) void*)(dQ + at), 16, (int)off, 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rd, (__attribute__((address_space(3))) void*)(ddO + at), 16, (int)off, 0, 0, 0);
    }
    const float* src = wave == 0 ? g.lse2 + row_at + q0 : g.delta + row_at + q0;
    float* dst = wave == 0 ? dLse : wave == 1 ? dDelta : sink;
    const auto rs = make_rsrc(src, wave < 2 ? (uint32_t)n_rows * 4u : 0u);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)dst, 4, 4 * lane_id(), 0, 0, 0);
  };
  bf16x8 kf[KC], vf[KC];
  {
    const uint32_t kv_bytes = (uint32_t)min(L - kv0, 64) * row_bytes;
    const size_t at = (size_t)(it.row0 + kv0) * row_stride + head_off;
    const auto rk = make_rsrc(g.k + at, kv_bytes), rv = make_rsrc(g.v + at, kv_bytes);
    const uint32_t off = (uint32_t)(32 * kb + l32) * row_bytes + (uint32_t)(16 * hh);
#pragma unroll
    for (int cc = 0; cc < KC; ++cc) kf[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rk, off + 32u * cc));
    KNAP_SCHED_FENCE();
#pragma unroll
    for (int cc = 0; cc < KC; ++cc) vf[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rv, off + 32u * cc));
    KNAP_SCHED_FENCE();
  }
  load_step(0, sQ0, sdO0, scalars[0][0], scalars[0][1]);
  RowReaderX<D> rows;
  ColReaderX<D> cols;
  rows.init(lane);
  cols.init(lane);
  f32x16 dk[DB], dv[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) dk[db] = dv[db] = zero16();
  wait_async_loads();
  lds_barrier();

  auto step = [&](int t, const __bf16* stepQ, const __bf16* stepdO, const float* tLse, const float* tDelta, __bf16* nQ, __bf16* ndO, float* nLse,
                  float* nDelta) __attribute__((always_inline)) {
    load_step(t + 1, nQ, ndO, nLse, nDelta);
    const __bf16 *tQ = stepQ + 32 * half * Tile<D>::LD, *tdO = stepdO + 32 * half * Tile<D>::LD;
    const int rb = rows.fresh(), cb = cols.fresh(), ln = lane_id(), l32 = ln & 31, hh = ln >> 5;
    f32x16 s = zero16(), dp;
#pragma unroll
    for (int j = 0; j < 4; ++j) {          // dP starts from -delta
      const f32x4 x = *reinterpret_cast<const f32x4*>(tDelta + 32 * half + 8 * j + 4 * hh);
#pragma unroll
      for (int e = 0; e < 4; ++e) dp[4 * j + e] = x[e];
    }
    constexpr int AHEAD = 2;
    bf16x8 aq[KC], ao[KC];
#pragma unroll
    for (int cc = 0; cc < AHEAD; ++cc) {
      aq[cc] = rows.get(tQ, rb, cc);
      ao[cc] = rows.get(tdO, rb, cc);
    }
    KNAP_SCHED_FENCE();
#pragma unroll
    for (int cc = 0; cc < KC; ++cc) {
      s = mfma32(aq[cc], kf[cc], s);
      if (cc + AHEAD < KC) aq[cc + AHEAD] = rows.get(tQ, rb, cc + AHEAD);
      dp = mfma32(ao[cc], vf[cc], dp);
      if (cc + AHEAD < KC) ao[cc + AHEAD] = rows.get(tdO, rb, cc + AHEAD);
      KNAP_SCHED_FENCE();
    }
    // register r: query 8 (r / 4) + 4 hh + r % 4 of the wave's 32; chunk cq holds registers 8 cq .. 8 cq + 7
    const int before = CAUSAL && t == 0 ? 32 * kb + l32 - 32 * half - 4 * hh : 0;      // queries of the 32 in front of the lane's key
    bf16x8 pa[2], da[2];
    uint32_t pw[2][4], dw[2][4];
    f32x4 lq[2][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) lq[0][j] = *reinterpret_cast<const f32x4*>(tLse + 32 * half + 8 * j + 4 * hh);
    // registers 8 cq + 2 i and the one behind it
    auto slice = [&](int cq, int i) __attribute__((always_inline)) {
      bf16x2 x, y;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int r = 8 * cq + 2 * i + e;
        float p = fast_exp2(__builtin_fmaf(s[r], c, -lq[cq][i >> 1][2 * (i & 1) + e]));
        if constexpr (CAUSAL) p = 8 * (r >> 2) + (r & 3) < before ? 0.f : p;
        x[e] = (__bf16)p;
        y[e] = (__bf16)(p * dp[r]);
      }
      pw[cq][i] = __builtin_bit_cast(uint32_t, x);
      dw[cq][i] = __builtin_bit_cast(uint32_t, y);
      if (i == 3) {
        const u32x4 u = {pw[cq][0], pw[cq][1], pw[cq][2], pw[cq][3]}, w = {dw[cq][0], dw[cq][1], dw[cq][2], dw[cq][3]};
        pa[cq] = __builtin_bit_cast(bf16x8, u);
        da[cq] = __builtin_bit_cast(bf16x8, w);
      }
    };
    bf16x8 of[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) of[i] = cols.get(tdO, cb, 0, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) slice(0, i);
#pragma unroll
    for (int j = 0; j < 2; ++j) lq[1][j] = *reinterpret_cast<const f32x4*>(tLse + 32 * half + 16 + 8 * j + 4 * hh);
    KNAP_SCHED_FENCE();
#pragma unroll
    for (int i = 0; i < 2 * DB; ++i) {
      f32x16& x = i < DB ? dv[i % DB] : dk[i % DB];
      x = mfma32(of[i & 1], i < DB ? pa[0] : da[0], x);
      if (i + 2 < 2 * DB) of[i & 1] = cols.get(i + 2 < DB ? tdO : tQ, cb, 0, (i + 2) % DB);
      if (i < 4) slice(1, i);
      KNAP_SCHED_FENCE();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) of[i] = cols.get(tdO, cb, 16, i);
    KNAP_SCHED_FENCE();
#pragma unroll
    for (int i = 0; i < 2 * DB; ++i) {
      f32x16& x = i < DB ? dv[i % DB] : dk[i % DB];
      x = mfma32(of[i & 1], i < DB ? pa[1] : da[1], x);
      if (i + 2 < 2 * DB) of[i & 1] = cols.get(i + 2 < DB ? tdO : tQ, cb, 16, (i + 2) % DB);
      KNAP_SCHED_FENCE();
    }
    wait_async_loads();
    lds_barrier();
  };
  for (int t = 0; t < n_steps; t += 2) {
    step(t, sQ0, sdO0, scalars[0][0], scalars[0][1], sQ1, sdO1, scalars[1][0], scalars[1][1]);
    if (t + 1 < n_steps) step(t + 1, sQ1, sdO1, scalars[1][0], scalars[1][1], sQ0, sdO0, scalars[0][0], scalars[0][1]);
  }

  ending();
  // The waves of the same keys trade halves: those of the first queries finish dK, those of the second dV.  A wave's 2 D bytes per
  // lane fill one of the four tile buffers.
  float* const mine = reinterpret_cast<float*>(half == 0 ? (kb == 0 ? sQ0 : sQ1) : (kb == 0 ? sdO0 : sdO1));
  const float* const other = reinterpret_cast<const float*>(half == 0 ? (kb == 0 ? sdO0 : sdO1) : (kb == 0 ? sQ0 : sQ1));
  const auto rg = make_rsrc((half == 0 ? g.dk : g.dv) + (size_t)(it.row0 + kv0) * row_stride + head_off, (uint32_t)min(L - kv0, 64) * row_bytes);
  const float out_scale = half == 0 ? g.scale : 1.0f;
  const int ln = lane_id();
  auto put = [&](const f32x16 (&x)[DB]) __attribute__((always_inline)) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 y = {x[db][4 * j], x[db][4 * j + 1], x[db][4 * j + 2], x[db][4 * j + 3]};
        *reinterpret_cast<f32x4*>(mine + ((4 * db + j) * 64 + ln) * 4) = y;
      }
  };
  auto finish = [&](f32x16 (&x)[DB]) __attribute__((always_inline)) {
    const uint32_t off = (uint32_t)(32 * kb + (ln & 31)) * row_bytes + (uint32_t)(16 * (ln >> 5));
#pragma unroll
    for (int db = 0; db < DB; ++db) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 y = *reinterpret_cast<const f32x4*>(other + ((4 * db + j) * 64 + ln) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[db][4 * j + e] += y[e];
      }
      store_block(rg, off + 64u * db, x[db], out_scale);
    }
  };
  if (half == 0) put(dv); else put(dk);
  lds_barrier();
  if (half == 0) finish(dk); else finish(dv);
}

template <int D, bool CAUSAL>
__device__ __forceinline__ void small_items(const BwdPtrs g, const SmallLds<D> s, const int32_t* __restrict__ cu, int n_seq, int H,
                                            const int* s_order, int* s_start, unsigned* __restrict__ counters) {
  constexpr int BM = 64;                           // rows of an item of either kind
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const DqLds lds = {s.a0, s.a1, s.a2, s.a3};
  float* const scalars[2][2] = {{s.lse0, s.delta0}, {s.lse1, s.delta1}};

  EvenQueue<0, 2> queue;          // key items, then query items, all of them whole
  queue.init(counters);
  if (wave == 0) even_shares(queue, n_seq, s_start, lane);
  __syncthreads();
  deal_even<BM, false>(queue, cu, n_seq, s_order, s_start);
  int ticket = queue.first_ticket();
  while (ticket < queue.wide) {
    const bool keys = queue.first_kind(ticket);
    const WorkItem it = decode_even<BM, false>(queue.item(ticket), queue, cu, n_seq, H, s_order, s_start);
    const int tile = __builtin_amdgcn_readfirstlane(it.tile), tiles = (it.len + BM - 1) / BM;
    const WorkItem x = {it.row0, it.len, __builtin_amdgcn_readfirstlane(it.head), tile};
    unsigned next_ticket;      // thread 0 only; no initial value, which would be merged in (and waited for) at once
    auto draw = [&] { if (tid == 0 && queue.draws) next_ticket = atomicAdd(queue.ctr, 1u); };
    int ln = lane;
    asm volatile("" : "+v"(ln));      // what follows from the lane is formed per item, not kept through the other kind's
    if (keys) {
      dkdv_part<D, CAUSAL>(g, lds, scalars, s.sink, x, tile * BM, ln, wave, draw);
    } else {
      DqLane<D> me;
      me.init(ln, wave);
      // under the mask the last queries see the most keys: they go first
      dq_part<D, CAUSAL, false>(g, lds, me, x, (CAUSAL ? tiles - 1 - tile : tile) * BM, [] {}, draw);
    }
    if (!queue.draws) return;
    if (tid == 0) *s.ticket = queue.later_ticket(next_ticket);
    lds_barrier();                    // (and the partial sums are no longer read)
    ticket = __builtin_amdgcn_readfirstlane(*s.ticket);
  }
}

// Items of 64 rows whatever the lengths are: the host knows that they pay (small_sure()).
template <int D, bool CAUSAL>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_bwd_small_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v, const __bf16* __restrict__ dout,
    float* __restrict__ lse2, float* __restrict__ delta, const int32_t* __restrict__ cu, int n_seq, int H, float scale,
    __bf16* __restrict__ dq, __bf16* __restrict__ dk, __bf16* __restrict__ dv, unsigned* __restrict__ counters) {
  extern __shared__ int s_dyn[];
  int* s_order = s_dyn;
  int* s_start = s_dyn + n_seq;
  constexpr int TILE = DqCfg<D>::TILE_ELEMS;
  __shared__ __attribute__((aligned(1024))) __bf16 sA0[TILE];
  __shared__ __attribute__((aligned(1024))) __bf16 sA1[TILE];
  __shared__ __attribute__((aligned(1024))) __bf16 sA2[TILE];
  __shared__ __attribute__((aligned(1024))) __bf16 sA3[TILE];
  __shared__ __attribute__((aligned(256))) float sLse0[64], sDelta0[64], sLse1[64], sDelta1[64], sSink[64];
  __shared__ int s_ticket;
  const int T = cu[n_seq];
  build_schedule<64, kThreads, false>(cu, n_seq, H, s_order, s_start, reinterpret_cast<int*>(&sA0[0]));
  const BwdPtrs g = {q, k, v, nullptr, dout, nullptr, lse2, delta, dq, dk, dv, T, H, scale};
  const SmallLds<D> lds = {sA0, sA1, sA2, sA3, sLse0, sDelta0, sLse1, sDelta1, sSink, &s_ticket};
  small_items<D, CAUSAL>(g, lds, cu, n_seq, H, s_order, s_start, counters);
}

template <int D>
static hipError_t launch_small_d(const BwdArgs& a, bool causal, bool sure, int cus, hipStream_t stream) {
  const size_t dyn = (size_t)(2 * a.n_seq + 1) * sizeof(int);
  auto* kernel = causal ? (sure ? attn_bwd_small_kernel<D, true> : attn_bwd_joint_kernel<D, true, true>)
                        : (sure ? attn_bwd_small_kernel<D, false> : attn_bwd_joint_kernel<D, false, true>);
  hipLaunchKernelGGL(kernel, dim3(cus * dkdv_workgroups_per_cu(D, 2)), dim3(kThreads), dyn, stream, (const __bf16*)a.q, (const __bf16*)a.k,
                     (const __bf16*)a.v, (const __bf16*)a.dout, a.lse2, a.delta, a.cu, a.n_seq, a.H, a.scale, (__bf16*)a.dq, (__bf16*)a.dk,
                     (__bf16*)a.dv, a.counters);
  return hipGetLastError();
}

hipError_t launch_small(const BwdArgs& a, int d, bool causal, bool sure, int cus, hipStream_t stream) {
  return d == 64 ? launch_small_d<64>(a, causal, sure, cus, stream) : launch_small_d<128>(a, causal, sure, cus, stream);
}

}  // namespace knap
