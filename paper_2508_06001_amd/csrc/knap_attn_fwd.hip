// Forward kernel: out = softmax(scale q k^T) v per (sequence, head) of a packed
// bag, with the row log-sum-exp (Sec. 3.4 / the attention listing of Sec. 3.5:
// full bidirectional attention inside each sequence, none across sequences).
// CAUSAL is the other mask the paper admits inside a datum (Limitations
// paragraph): query i sees keys 0..i of its own sequence.
//
// One persistent workgroup (4 waves) takes work items (sequence, head, 128-row
// query tile) from the longest-first schedule.  Wave w owns 32 query rows and
// streams the sequence's keys and values through LDS in tiles of 64 rows; the
// next tile is copied global -> LDS asynchronously (no staging registers) into
// the other buffer while the current one is used, behind one barrier per tile.
//
// Orientation: the scores are computed transposed, S^T = K Q^T, so that in the
// MFMA result layout a lane holds ONE query (column l % 32) and its registers
// run over keys.  Row max and row sum are then in-register reductions plus one
// exchange between lanes l and l ^ 32, the rescale factor is a per-lane scalar,
// and P^T in that layout is, unchanged, the B operand of O^T += V^T P^T.  V^T
// fragments come from the row-major V tile through transposing LDS reads.
//
// Softmax bookkeeping: P of a half tile (32 keys) is formed against the exponent reference m_ref as it
// stands, and the row sums that come out of it decide whether the reference has to move: only when a
// lane's 16 probabilities sum to more than 2^8 (the first half always does: the reference starts at
// -inf), in which case the maximum is taken (of the tile, or of the half if it is the tile's second), the accumulators
// are rescaled and P is formed again.  So no maximum is taken per tile (a fifth of the loop's vector instructions: 4.2 -> 3.4
// per MFMA);
// P <= 256 all the same, and the final division by the row sum removes the reference exactly as in
// the textbook recurrence.  The row sum is taken over the bf16-rounded P that the MFMA multiplies, so the
// effective weights of a row sum to one exactly (a one-hot row returns its v bit for bit); the stored
// log-sum-exp inherits at most a 2^-8 relative change of that sum.
//
// What bounds it: MFMA and softmax arithmetic share the issue slots, at the clock the power limit leaves.
// The arithmetic of a half therefore runs in the slot of the next half's MFMAs, and an item's first loads
// go out under the previous item's epilogue.  Measured at 24 heads of 128 when both came in
// (before -> after, us): 32 sequences of 256..648 tokens 172 -> 144, one of 4292 tokens 305 -> 283, 17 of 328..4533 tokens
// 1104 -> 1040, one of 65536 and 200 short ones 47500 -> 46600.  Now: 136, 254, 1025 and 45500.
#include "knap_attn_fwd_part.h"

namespace knap {

template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_fwd_causal_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
    const int32_t* __restrict__ cu, int n_seq, int H, float scale,
    __bf16* __restrict__ out, float* __restrict__ lse, unsigned* __restrict__ counters) {
  using C = FwdCfg<D>;
  extern __shared__ int s_dyn[];
  int* s_order = s_dyn;
  int* s_start = s_dyn + n_seq;
  // separate arrays (not one indexed array) so that reads of one buffer are known not to
  // depend on the asynchronous copy into the other
  __shared__ __attribute__((aligned(1024))) __bf16 sK0[C::TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) __bf16 sK1[C::TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) __bf16 sV0[C::TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) __bf16 sV1[C::TILE_ELEMS];
  static_assert(sizeof(__bf16) * C::TILE_ELEMS >= sizeof(int) * kThreads, "scan scratch must fit in a tile");

  // the scan scratch of the schedule lives in the first K buffer, which is not in use yet
  const int T = cu[n_seq];
  build_schedule<C::BM, kThreads, true>(cu, n_seq, H, s_order, s_start, reinterpret_cast<int*>(&sK0[0]));
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  // known to be wave-uniform: the LDS address of each of a tile's eight copies otherwise goes through a vector register (dQ
  // kernel: there)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31;
  const int hh = lane >> 5;
  const float c = scale * kLog2e;
  const size_t row_stride = (size_t)H * D;
  const uint32_t row_bytes = (uint32_t)(row_stride * sizeof(__bf16));
  RowReader<D> k_rows;   // K tile rows -> A operands of S^T
  ColReader<D> v_cols;   // V tile columns -> A operands of O^T += V^T P^T
  k_rows.init(lane);
  v_cols.init(lane);

  // Work items come from this XCD's queue.  The ticket for the NEXT item is drawn in front of the item's last two tiles and
  // looked at behind them, so that the counter's latency is covered (vector-memory operations complete in issue order: in
  // front of the first loads it would hold up the whole prologue) and the items go to the workgroups that end first.  Drawn at
  // the item's start, what is left behind a full round went to those that had started first, with the longest items.  Drawn at
  // the start -> at the end, us: 8192 and 3 of 4096 and one of 2048 tokens, 3 x 128, 214 -> 182; 2 of 8192 and 2 of 4096 271 ->
  // 244; 4096, 2 of 2048 and 3 of 1024, 6 x 128, 110 -> 93; one round, or many, the same within 0.5 %.
  __shared__ int s_ticket;
  constexpr int SPLIT = 4;     // narrow items (64 queries) of a wide one
  EvenQueue<SPLIT, 1> queue;
  queue.init(counters);
  if (tid < 64) even_shares(queue, n_seq, s_start, lane);
  __syncthreads();
  deal_even<C::BM, true>(queue, cu, n_seq, s_order, s_start);
  auto take = [&](int i) { return decode_even<C::BM, true>(i, queue, cu, n_seq, H, s_order, s_start); };
  int ticket = queue.first_ticket();
  WorkItem it;
  unsigned next_ticket;      // thread 0 only; no initial value, which would be merged in (and waited for) at once
  int sub = 0;               // the item is the pair of query tiles {q_tiles - 1 - p, p}, the long one first

  bf16x8 qf[C::KC];          // this lane's query row as the B operand of S^T = K Q^T
  auto q_tile_of = [&]() {
    return sub == 0 ? (it.len + C::BM - 1) / C::BM - 1 - it.tile : it.tile;
  };
  // asynchronous copy of tile t (keys 64 t ..) of the item; rows at or past kv_end arrive as zeros
  auto load_tile = [&](int t, int kv_end, __bf16* dK, __bf16* dV) {
    const int kv0 = t * C::BN;
    const uint32_t bytes = (uint32_t)max(0, min(kv_end - kv0, C::BN)) * row_bytes;
    const size_t off = (size_t)(it.row0 + kv0) * row_stride + (size_t)it.head * D;
    tile_load_async<D>(dK, make_rsrc(k + off, bytes), row_bytes, C::BN, wave, lane);
    tile_load_async<D>(dV, make_rsrc(v + off, bytes), row_bytes, C::BN, wave, lane);
  };
  const uint32_t q_off = (uint32_t)(wave * 32 + l32) * row_bytes + (uint32_t)(8 * hh) * 2u;
  // what an item needs before its first product: tile 0 and the query rows (rows past the end read as zero)
  auto load_first = [&]() {
    const int q0 = q_tile_of() * C::BM;
    load_tile(0, min(it.len, q0 + C::BM), sK0, sV0);
    const auto rq = make_rsrc(q + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D,
                              (uint32_t)min(it.len - q0, C::BM) * row_bytes);
#pragma unroll
    for (int cc = 0; cc < C::KC; ++cc) qf[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rq, q_off + 32u * cc));
  };
  if (ticket < queue.wide) {
  it = take(ticket);
  load_first();
  wait_async_loads();
  lds_barrier();

  for (;;) {
    const int L = it.len;
    const int q_tile = q_tile_of();
    const int q0 = q_tile * C::BM;
    const int q_row = q0 + wave * 32 + l32;      // row inside the sequence
    // keys this query tile sees at all
    const int kv_end = min(L, q0 + C::BM);
    const int n_tiles = (kv_end + C::BN - 1) / C::BN;
    // the last pair of tiles of the item's second query tile
    const int t_draw = queue.draws && !(sub == 0 && it.tile != q_tile) ? (n_tiles - 1) & ~1 : -1;

    f32x16 o[C::DB];
#pragma unroll
    for (int db = 0; db < C::DB; ++db) o[db] = zero16();
    float m_ref = -INFINITY;   // exponent reference (raw score units)
    float mc = -INFINITY;      // m_ref * c
    float l_run = 0.f;         // this lane's share of the row sum (its 32 of the 64 keys per tile)

    // the first tile in which some key of this item's queries is masked: after a query (which covers the ragged end for the
    // rows of the sequence)
    const int first_masked = 2 * q_tile;
    const int kv_lim = q_row + 1;

    // One tile: 64 keys as two halves of 32.  A wave whose 32 queries all precede the tile's first key has
    // nothing to do in it.
    auto process_tile = [&](int t, const __bf16* tK, const __bf16* tV, __bf16* nK, __bf16* nV) {
      load_tile(t + 1, kv_end, nK, nV);
      const bool masked = t >= first_masked;
      if (t * C::BN <= q0 + 32 * wave + 31) {

      bf16x8 ak0[C::KC], ak1[C::KC];
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) ak0[cc] = k_rows.get(tK, 0, cc);
      KNAP_SCHED_FENCE();

      f32x16 s0 = zero16(), s1 = zero16();
      // slot 1: S^T of keys 0..31 | K fragments of keys 32..63
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) s0 = mfma32(ak0[cc], qf[cc], s0);
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) ak1[cc] = k_rows.get(tK, 32, cc);
#pragma unroll
      for (int i = 0; i < C::KC; ++i) { KNAP_SGB(KNAP_SG_MFMA, 1); KNAP_SGB(KNAP_SG_DS_READ, 1); }
      KNAP_SCHED_FENCE();

      if (masked) mask_half(s0, kv_lim - t * C::BN, hh);
      KNAP_SCHED_FENCE();
      // slot 2: S^T of keys 32..63 | P^T of keys 0..31, V^T fragments of keys 0..15
      bf16x8 vt0[2][C::DB], vt1[2][C::DB];
      bf16x8 pb0[2], pb1[2];
      float l0 = l_run;
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) s1 = mfma32(ak1[cc], qf[cc], s1);
      half_exps(s0, c, mc, pb0, l0);
#pragma unroll
      for (int db = 0; db < C::DB; ++db) vt0[0][db] = v_cols.get(tV, 0, db);
#pragma unroll
      for (int i = 0; i < C::KC; ++i) { KNAP_SGB(KNAP_SG_MFMA, 1); KNAP_SGB(KNAP_SG_DS_READ, 1); KNAP_SGB(KNAP_SG_VALU, 48 / C::KC); }
      KNAP_SCHED_FENCE();
      half_settle<C::DB>(s0, c, [&] { return fmaxf(half_max(s0, C::BN, hh), half_max(s1, kv_lim - t * C::BN - 32, hh)); }, pb0, l0, m_ref, mc, l_run, o);
      if (masked) mask_half(s1, kv_lim - t * C::BN - 32, hh);
      KNAP_SCHED_FENCE();

      // slot 3: O^T += V^T P^T over keys 0..31 | P^T of keys 32..63, V^T fragments of keys 16..47
#pragma unroll
      for (int db = 0; db < C::DB; ++db) vt0[1][db] = v_cols.get(tV, 16, db);
#pragma unroll
      for (int ck = 0; ck < 2; ++ck)
#pragma unroll
        for (int db = 0; db < C::DB; ++db) o[db] = mfma32(vt0[ck][db], pb0[ck], o[db]);
      float l1 = l_run;
      half_exps(s1, c, mc, pb1, l1);
#pragma unroll
      for (int db = 0; db < C::DB; ++db) vt1[0][db] = v_cols.get(tV, 32, db);
#pragma unroll
      for (int i = 0; i < 2 * C::DB; ++i) { KNAP_SGB(KNAP_SG_DS_READ, 2); KNAP_SGB(KNAP_SG_MFMA, 1); KNAP_SGB(KNAP_SG_VALU, 24 / C::DB); }
      KNAP_SCHED_FENCE();
      half_settle<C::DB>(s1, c, [&] { return half_max(s1, C::BN, hh); }, pb1, l1, m_ref, mc, l_run, o);
      KNAP_SCHED_FENCE();

      // slot 4: O^T += V^T P^T over keys 32..63 | V^T fragments of keys 48..63
#pragma unroll
      for (int db = 0; db < C::DB; ++db) vt1[1][db] = v_cols.get(tV, 48, db);
#pragma unroll
      for (int ck = 0; ck < 2; ++ck)
#pragma unroll
        for (int db = 0; db < C::DB; ++db) o[db] = mfma32(vt1[ck][db], pb1[ck], o[db]);
#pragma unroll
      for (int i = 0; i < C::DB; ++i) { KNAP_SGB(KNAP_SG_DS_READ, 2); KNAP_SGB(KNAP_SG_MFMA, 1); }
      KNAP_SCHED_FENCE();
      }
      wait_async_loads();
      __syncthreads();     // next tile visible; this tile no longer read
    };

    for (int t = 0; t < n_tiles; t += 2) {
      if (t == t_draw && tid == 0) next_ticket = atomicAdd(queue.ctr, 1u);
      process_tile(t, sK0, sV0, sK1, sV1);
      if (t + 1 < n_tiles) process_tile(t + 1, sK1, sV1, sK0, sV0);
    }

    // The next item's first loads go out before this one's results are stored, so that they travel under
    // the epilogue; both tile buffers are free (the last tile ended with a barrier).
    const auto ro = make_rsrc(out + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D,
                              (uint32_t)min(L - q0, C::BM) * row_bytes);
    const auto rl = make_rsrc(lse + (size_t)it.head * T + it.row0 + q0, (uint32_t)min(L - q0, C::BM) * 4u);
    bool more = true;
    if (sub == 0 && it.tile != q_tile) {   // not the middle tile of an odd count
      sub = 1;
    } else if (!queue.draws) {
      more = false;
    } else {
      if (tid == 0) {
        s_ticket = drawn_ticket(queue, next_ticket);   // every wave read the old one many barriers ago
      }
      lds_barrier();
      ticket = __builtin_amdgcn_readfirstlane(s_ticket);
      more = ticket < queue.wide;
      if (more) it = take(ticket);
      sub = 0;
    }
    if (more) load_first();
    KNAP_SCHED_FENCE();

    // epilogue: normalise, store lse (natural log) and out (bf16)
    const float l_tot = l_run + xor32(l_run);
    const float inv = 1.0f / l_tot;
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, m_ref * scale + __logf(l_tot)), rl,
                                          hh == 0 ? (wave * 32 + l32) * 4 : 4 * C::BM, 0, 0);
#pragma unroll
    for (int db = 0; db < C::DB; ++db) store_block(ro, q_off + 64u * db, o[db], inv);
    if (!more) break;
    // the loads have landed: all but the 2 DB stores of the output, which are younger (in-order completion)
    wait_vm<2 * C::DB>();
    lds_barrier();
  }
  }

  // Narrow items: 64 queries.  Where the items are few, or the last round is thin, each is cut in two that run on two CUs (a
  // CU's matrix units are nearly as busy with one workgroup as with two: an item of 4096 keys beside another of twice
  // the length 145 us, alone 67).
  if (queue.parts > 0) lds_barrier();     // every wave has the ticket before the next one is put down
  const FwdPtrs g = {q, k, v, out, lse, T, H, scale};
  const FwdLds lds = {sK0, sK1, sV0, sV1};
  for (int part = ticket - queue.wide; part >= 0 && part < queue.parts;) {
    it = take(queue.item_of_part(part));
    const int q_tiles = (it.len + C::BM - 1) / C::BM;
    const int member = (part % SPLIT) >> 1;
    const int q0 = __builtin_amdgcn_readfirstlane((member == 0 ? q_tiles - 1 - it.tile : it.tile) * C::BM + 64 * (part & 1));
    const bool exists = q0 < it.len && !(member == 1 && it.tile == q_tiles - 1 - it.tile);
    if (exists) fwd_part<D, true>(g, lds, it, q0, lane, wave);
    if (!queue.draws) return;         // every part was a first ticket
    if (tid == 0) {
      const unsigned drawn = atomicAdd(queue.ctr, 1u);
      s_ticket = drawn_ticket(queue, drawn);
    }
    lds_barrier();                    // (and the tile buffers are no longer read)
    part = __builtin_amdgcn_readfirstlane(s_ticket) - queue.wide;
    lds_barrier();                    // everyone has the ticket before it is drawn again
  }
}

// Counters of the work queues, in the library's device image (512 KB that start at zero): sets of 8, one counter per XCD,
// handed out by the host (eager_set(), captured_set()).  The kernel leaves its counters at zero, so no launch has to clear
// them in front of it.
static __device__ __align__(256) unsigned g_queues[kQueueSets * 8];

__global__ __launch_bounds__(kThreads) void queue_clear_kernel(unsigned* __restrict__ counters, unsigned n) {
  const unsigned i = blockIdx.x * kThreads + threadIdx.x;
  if (i < n) counters[i] = 0u;
}

hipError_t clear_queue_sets(unsigned* first, unsigned sets, hipStream_t stream) {
  hipLaunchKernelGGL(queue_clear_kernel, dim3((8 * sets + kThreads - 1) / kThreads), dim3(kThreads), 0, stream, first, 8 * sets);
  return hipGetLastError();
}

unsigned* queue_base() {
  unsigned* p = nullptr;
  if (hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(g_queues)) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return p;
}

template <int D>
static hipError_t launch_causal_t(const void* q, const void* k, const void* v, const int32_t* cu, int n_seq, int H, float scale, void* out,
                                  float* lse, unsigned* counters, int grid, hipStream_t stream) {
  const size_t dyn = (size_t)(2 * n_seq + 1) * sizeof(int);
  hipLaunchKernelGGL((attn_fwd_causal_kernel<D>), dim3(grid), dim3(kThreads), dyn, stream, (const __bf16*)q, (const __bf16*)k,
                     (const __bf16*)v, cu, n_seq, H, scale, (__bf16*)out, lse, counters);
  return hipGetLastError();
}

hipError_t launch_fwd_causal(const void* q, const void* k, const void* v, const int32_t* cu, int n_seq, int H, int d, float scale,
                             void* out, float* lse, unsigned* counters, int grid, hipStream_t stream) {
  return d == 64 ? launch_causal_t<64>(q, k, v, cu, n_seq, H, scale, out, lse, counters, grid, stream)
                 : launch_causal_t<128>(q, k, v, cu, n_seq, H, scale, out, lse, counters, grid, stream);
}

}  // namespace knap
