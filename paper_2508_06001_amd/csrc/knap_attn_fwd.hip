// Forward kernel under the causal mask: out = softmax(scale q k^T) v per (sequence, head) of a packed bag, with the row log-sum-exp.
// It is the other mask the paper admits inside a datum (Limitations paragraph): query i sees keys 0..i of its own sequence.
//
// One persistent workgroup (4 waves) takes work items (sequence, head, pair of 128-row query tiles) from the longest-first schedule,
// the long tile of a pair first.  Wave w owns 32 query rows and streams the sequence's keys and values through LDS in tiles of 64 rows
// (fwd_tile() in knap_attn_fwd_part.h, which the forward without the mask shares).
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
// are rescaled and P is formed again.  So no maximum is taken per tile; P <= 256 all the same, and the final division by the row sum
// removes the reference exactly as in the textbook recurrence.  The row sum is taken over the bf16-rounded P that the MFMA multiplies, so
// the effective weights of a row sum to one exactly (a one-hot row returns its v bit for bit); the stored
// log-sum-exp inherits at most a 2^-8 relative change of that sum.
//
// What bounds it: MFMA and softmax arithmetic share the issue slots, at the clock the power limit leaves.  Three halves of 32 keys are in
// work at a time, and the waves whose queries precede the whole last tile leave its turn to the others.  A half's arithmetic between
// its own two products -> this, forward in us, 24 x 128: 17 sequences of 328..4533 tokens 602 -> 583, 14 of 406..14415 3315 -> 3202, 2 of up to
// 4173 258 -> 246, 32 of 450 110 -> 108; 6 x 128, one of 8000 141 -> 133; 12 x 64, one of 8000 144 -> 138, of 30000 1578 -> 1548, but 32 of 450
// 30.9 -> 32.2; 80 bags 1.019 in the geometric mean.  With those waves in the last turn as well: 1.011.
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
  // asynchronous copy of this wave's share of tile t (keys 64 t ..) of K or V; rows past the last that the query tile sees arrive as zeros
  auto copy_rows = [&](const __bf16* __restrict__ src, int t, __bf16* dst) __attribute__((always_inline)) {
    const int kv0 = t * C::BN, kv_end = min(it.len, (q_tile_of() + 1) * C::BM);
    const uint32_t bytes = (uint32_t)max(0, min(kv_end - kv0, C::BN)) * row_bytes;
    tile_load_async<D>(dst, make_rsrc(src + (size_t)(it.row0 + kv0) * row_stride + (size_t)it.head * D, bytes), row_bytes, C::BN, wave, lane);
  };
  const uint32_t q_off = (uint32_t)(wave * 32 + l32) * row_bytes + (uint32_t)(8 * hh) * 2u;
  // what a query tile needs before its first product, the keys of tile 0 and the query rows (rows past the end read as zero), and
  // behind it what its first turn of the loop reads: the values of tile 0 and the keys of tile 1
  auto load_first = [&]() __attribute__((always_inline)) {
    const int q0 = q_tile_of() * C::BM;
    copy_rows(k, 0, sK0);
    const auto rq = make_rsrc(q + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D,
                              (uint32_t)min(it.len - q0, C::BM) * row_bytes);
#pragma unroll
    for (int cc = 0; cc < C::KC; ++cc) qf[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rq, q_off + 32u * cc));
    KNAP_SCHED_FENCE();
    copy_rows(v, 0, sV0);
    copy_rows(k, 1, sK1);
    KNAP_SCHED_FENCE();
  };
  constexpr int COPIES = C::BN * D / 2048;      // copies of a wave's share of a tile
  const FwdLds lds = {sK0, sK1, sV0, sV1};
  if (ticket < queue.wide) {
  it = take(ticket);
  load_first();
  wait_vm<2 * COPIES>();
  lds_barrier();

  for (;;) {
    const int L = it.len;
    const int q_tile = q_tile_of();
    const int q0 = q_tile * C::BM;
    const int q_row = q0 + wave * 32 + l32;      // row inside the sequence
    // keys this query tile sees at all
    const int kv_end = min(L, q0 + C::BM);
    const int n_tiles = (kv_end + C::BN - 1) / C::BN;
    // the next ticket is drawn in the last turn of the item's second query tile
    const bool draws = queue.draws && !(sub == 0 && it.tile != q_tile);
    // From tile 2 q_tile on some key of this item's queries is masked: after a query (which covers the ragged end for the rows of the
    // sequence).
    f32x16 o[C::DB];
    float m_ref, l_run;
    fwd_tile<D, true>(lds, qf, k_rows, v_cols, c, n_tiles,
                q0 + 32 * wave < L ? min(n_tiles, (q0 + 32 * wave + 31) / C::BN + 1) : 0, (wave & 1) != 0, 2 * q_tile, q_row + 1, hh,
                [&](int t, __bf16* dst) __attribute__((always_inline)) { copy_rows(k, t, dst); },
                [&](int t, __bf16* dst) __attribute__((always_inline)) { copy_rows(v, t, dst); },
                [&] { if (draws && tid == 0) next_ticket = atomicAdd(queue.ctr, 1u); }, o, m_ref, l_run);

    // The next item's first loads go out before this one's results are stored, so that they travel under the epilogue.
    const auto ro = make_rsrc(out + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D,
                              (uint32_t)min(L - q0, C::BM) * row_bytes);
    const auto rl = make_rsrc(lse + (size_t)it.head * T + it.row0 + q0, (uint32_t)min(L - q0, C::BM) * 4u);
    bool more = true;
    if (draws && tid == 0) s_ticket = drawn_ticket(queue, next_ticket);   // every wave read the old one many barriers ago
    lds_barrier();          // nobody reads a tile any longer
    if (sub == 0 && it.tile != q_tile) {   // not the middle tile of an odd count
      sub = 1;
    } else if (!queue.draws) {
      more = false;
    } else {
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
    // the keys and the query rows have landed: all but the copies behind them and the stores, which are younger (in-order completion)
    wait_vm<2 * COPIES + 1 + 2 * C::DB>();
    lds_barrier();
  }
  }

  // Narrow items: 64 queries.  Where the items are few, or the last round is thin, each is cut in two that run on two CUs (a
  // CU's matrix units are nearly as busy with one workgroup as with two: an item of 4096 keys beside another of twice
  // the length 145 us, alone 67).
  if (queue.parts > 0) lds_barrier();     // every wave has the ticket before the next one is put down
  const FwdPtrs g = {q, k, v, out, lse, T, H, scale};
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
