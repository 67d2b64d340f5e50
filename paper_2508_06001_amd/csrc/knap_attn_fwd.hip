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
#include "knap_device.h"
#include "knap_kernels.h"

namespace knap {

template <int D>
struct FwdCfg {
  static constexpr int BM = 128;         // query rows per work item
  static constexpr int BN = 64;          // key/value rows per LDS tile
  static constexpr int KC = D / 16;      // contraction chunks over d
  static constexpr int DB = D / 32;      // 32-wide blocks of d
  static constexpr int TILE_ELEMS = BN * Tile<D>::LD;
};

constexpr float kMaxHalfSum = 256.f;        // of a lane's 16 probabilities against the present reference

template <int D, bool CAUSAL>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_fwd_kernel(
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
  build_schedule<C::BM, kThreads, CAUSAL>(cu, n_seq, H, s_order, s_start, reinterpret_cast<int*>(&sK0[0]));
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
  constexpr int SPLIT = CAUSAL ? 4 : 2;     // narrow items (64 queries) of a wide one
  EvenQueue<SPLIT, 1> queue;
  queue.init(counters);
  if (tid < 64) even_shares(queue, n_seq, s_start, lane);
  __syncthreads();
  deal_even<C::BM, CAUSAL>(queue, cu, n_seq, s_order, s_start);
  auto take = [&](int i) { return decode_even<C::BM, CAUSAL>(i, queue, cu, n_seq, H, s_order, s_start); };
  int ticket = queue.first_ticket();
  WorkItem it;
  unsigned next_ticket;      // thread 0 only; no initial value, which would be merged in (and waited for) at once
  int sub = 0;               // CAUSAL: the item is the pair of query tiles {q_tiles - 1 - p, p}, the long one first

  bf16x8 qf[C::KC];          // this lane's query row as the B operand of S^T = K Q^T
  auto q_tile_of = [&]() {
    return !CAUSAL ? it.tile : sub == 0 ? (it.len + C::BM - 1) / C::BM - 1 - it.tile : it.tile;
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
    load_tile(0, CAUSAL ? min(it.len, q0 + C::BM) : it.len, sK0, sV0);
    const auto rq = make_rsrc(q + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D,
                              (uint32_t)min(it.len - q0, C::BM) * row_bytes);
#pragma unroll
    for (int cc = 0; cc < C::KC; ++cc) qf[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rq, q_off + 32u * cc));
  };
  auto mask_half = [&](f32x16& s, int seen) {     // `seen`: keys of the half, from its first, that this lane's query sees
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 8 * (r >> 2) + (r & 3) < seen - 4 * hh ? s[r] : -INFINITY;
  };

  // P^T of a half, packed, against the reference as it stands (mc = m_ref c): element e of chunk ck is key
  // 16 ck + 8 (e / 4) + 4 hh + e % 4; the lane's 16 rounded probabilities are added to `l`
  auto half_exps = [&](const f32x16& s, float mc, bf16x8 (&pb)[2], float& l) {
    float p[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = fast_exp2(__builtin_fmaf(s[r], c, -mc));
#pragma unroll
    for (int ck = 0; ck < 2; ++ck) {
      const int r0 = 8 * ck;
      pb[ck] = pack8_sum(p[r0], p[r0 + 1], p[r0 + 2], p[r0 + 3], p[r0 + 4], p[r0 + 5], p[r0 + 6], p[r0 + 7], l);
    }
  };
  // `l_new` is l_run with the half's probabilities added.  The reference moves only when they are too large (always
  // on the first half, where it is -inf and the sum inf or NaN): up to the maximum, with what is accumulated rescaled
  // and the half's probabilities formed again.  The first half of a tile takes the maximum of the whole tile, so that
  // the largest probability of an item's first 64 keys is exactly 1 and carries no rounding error (taken over 32
  // keys, the error of lse against 64 bits grew by up to 6 %, that of out by up to 1.7 %).
  auto half_max = [&](const f32x16& s, int seen) {
    float m = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) m = fmaxf(m, 8 * (r >> 2) + (r & 3) < seen - 4 * hh ? s[r] : -INFINITY);
    return m;
  };
  auto half_settle = [&](const f32x16& s, auto maximum, bf16x8 (&pb)[2], float l_new, float& m_ref, float& mc, float& l_run, f32x16 (&o)[C::DB]) {
    if (__builtin_amdgcn_ballot_w64(!(l_new - l_run <= kMaxHalfSum)) != 0) {
      const float m_loc = maximum();
      const float m_new = fmaxf(m_ref, fmaxf(m_loc, xor32(m_loc)));
      const float alpha = m_new == m_ref ? 1.f : fast_exp2((m_ref - m_new) * c);
      m_ref = m_new;
      mc = m_new == -INFINITY ? 0.f : m_new * c;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < C::DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      l_new = l_run;
      half_exps(s, mc, pb, l_new);
      if (m_new == -INFINITY) mc = -INFINITY;   // scores of -inf alone set no reference: the next half has to settle too
    }
    l_run = l_new;
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
    const int kv_end = CAUSAL ? min(L, q0 + C::BM) : L;
    const int n_tiles = (kv_end + C::BN - 1) / C::BN;
    // the last pair of tiles of the item; of both its query tiles under the mask
    const int t_draw = queue.draws && !(CAUSAL && sub == 0 && it.tile != q_tile) ? (n_tiles - 1) & ~1 : -1;

    f32x16 o[C::DB];
#pragma unroll
    for (int db = 0; db < C::DB; ++db) o[db] = zero16();
    float m_ref = -INFINITY;   // exponent reference (raw score units)
    float mc = -INFINITY;      // m_ref * c
    float l_run = 0.f;         // this lane's share of the row sum (its 32 of the 64 keys per tile)

    // the first tile in which some key of this item's queries is masked: past the end of the sequence, or (CAUSAL)
    // after a query (which covers the ragged end for the rows of the sequence)
    const int first_masked = CAUSAL ? 2 * q_tile : L / C::BN;
    const int kv_lim = CAUSAL ? q_row + 1 : L;

    // One tile: 64 keys as two halves of 32.  A wave whose 32 queries all precede the tile's first key has
    // nothing to do in it.
    auto process_tile = [&](int t, const __bf16* tK, const __bf16* tV, __bf16* nK, __bf16* nV) {
      load_tile(t + 1, kv_end, nK, nV);
      const bool masked = t >= first_masked;
      if (!(CAUSAL && t * C::BN > q0 + 32 * wave + 31)) {

      bf16x8 ak0[C::KC], ak1[C::KC];
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) ak0[cc] = k_rows.get(tK, 0, cc);
      if constexpr (D == 128 && !CAUSAL) {   // the reads between the eight copies: all behind them costs three heads of
        KNAP_SGB(KNAP_SG_DS_READ, 2);        // 131072 keys 1.4 %, all in front of them 1.7 %
        KNAP_SGB(KNAP_SG_VMEM_READ, 3);
        KNAP_SGB(KNAP_SG_DS_READ, 1);
        KNAP_SGB(KNAP_SG_VMEM_READ, 4);
        KNAP_SGB(KNAP_SG_DS_READ, 1);
        KNAP_SGB(KNAP_SG_VMEM_READ, 1);
        KNAP_SGB(KNAP_SG_DS_READ, 4);
      }
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

      if (masked) mask_half(s0, kv_lim - t * C::BN);
      KNAP_SCHED_FENCE();
      // slot 2: S^T of keys 32..63 | P^T of keys 0..31, V^T fragments of keys 0..15
      bf16x8 vt0[2][C::DB], vt1[2][C::DB];
      bf16x8 pb0[2], pb1[2];
      float l0 = l_run;
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) s1 = mfma32(ak1[cc], qf[cc], s1);
      half_exps(s0, mc, pb0, l0);
#pragma unroll
      for (int db = 0; db < C::DB; ++db) vt0[0][db] = v_cols.get(tV, 0, db);
#pragma unroll
      for (int i = 0; i < C::KC; ++i) { KNAP_SGB(KNAP_SG_MFMA, 1); KNAP_SGB(KNAP_SG_DS_READ, 1); KNAP_SGB(KNAP_SG_VALU, 48 / C::KC); }
      KNAP_SCHED_FENCE();
      half_settle(s0, [&] { return fmaxf(half_max(s0, C::BN), half_max(s1, kv_lim - t * C::BN - 32)); }, pb0, l0, m_ref, mc, l_run, o);
      if (masked) mask_half(s1, kv_lim - t * C::BN - 32);
      KNAP_SCHED_FENCE();

      // slot 3: O^T += V^T P^T over keys 0..31 | P^T of keys 32..63, V^T fragments of keys 16..47
#pragma unroll
      for (int db = 0; db < C::DB; ++db) vt0[1][db] = v_cols.get(tV, 16, db);
#pragma unroll
      for (int ck = 0; ck < 2; ++ck)
#pragma unroll
        for (int db = 0; db < C::DB; ++db) o[db] = mfma32(vt0[ck][db], pb0[ck], o[db]);
      float l1 = l_run;
      half_exps(s1, mc, pb1, l1);
#pragma unroll
      for (int db = 0; db < C::DB; ++db) vt1[0][db] = v_cols.get(tV, 32, db);
#pragma unroll
      for (int i = 0; i < 2 * C::DB; ++i) { KNAP_SGB(KNAP_SG_DS_READ, 2); KNAP_SGB(KNAP_SG_MFMA, 1); KNAP_SGB(KNAP_SG_VALU, 24 / C::DB); }
      KNAP_SCHED_FENCE();
      half_settle(s1, [&] { return half_max(s1, C::BN); }, pb1, l1, m_ref, mc, l_run, o);
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
    if (CAUSAL && sub == 0 && it.tile != q_tile) {   // not the middle tile of an odd count
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
  // Waves w and w + 2 share 32 queries, one taking the first 32 keys of every tile, the other the second 32; the two
  // halves of the softmax are merged through LDS at the end.
  if (queue.parts > 0) lds_barrier();     // every wave has the ticket before the next one is put down
  const int rb = wave & 1, kh = wave >> 1;
  const int kh_u = __builtin_amdgcn_readfirstlane(kh), rb_u = __builtin_amdgcn_readfirstlane(rb);
  for (int part = ticket - queue.wide; part >= 0 && part < queue.parts;) {
    it = take(queue.item_of_part(part));
    const int L = it.len;
    const int q_tiles = (L + C::BM - 1) / C::BM;
    const int member = (part % SPLIT) >> 1;
    const int q0 = __builtin_amdgcn_readfirstlane((!CAUSAL ? it.tile : member == 0 ? q_tiles - 1 - it.tile : it.tile) * C::BM + 64 * (part & 1));
    const bool exists = q0 < L && !(CAUSAL && member == 1 && it.tile == q_tiles - 1 - it.tile);
    if (exists) {
      const int q_row = q0 + 32 * rb + l32;
      const int kv_end = CAUSAL ? min(L, q0 + 64) : L;
      const int n_tiles = (kv_end + C::BN - 1) / C::BN;
      const int first_masked = CAUSAL ? q0 / C::BN : L / C::BN;
      const int kv_lim = CAUSAL ? q_row + 1 : L;
      const uint32_t off = (uint32_t)(32 * rb + l32) * row_bytes + (uint32_t)(8 * hh) * 2u;
      load_tile(0, kv_end, sK0, sV0);
      const auto rq = make_rsrc(q + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D,
                                (uint32_t)min(L - q0, 64) * row_bytes);
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) qf[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rq, off + 32u * cc));
      wait_async_loads();
      lds_barrier();

      f32x16 o[C::DB];
#pragma unroll
      for (int db = 0; db < C::DB; ++db) o[db] = zero16();
      float m_ref = -INFINITY, mc = -INFINITY, l_run = 0.f;

      auto half_tile = [&](int t, const __bf16* tK, const __bf16* tV, __bf16* nK, __bf16* nV) {
        load_tile(t + 1, kv_end, nK, nV);
        if (!(CAUSAL && t * C::BN + 32 * kh_u > q0 + 32 * rb_u + 31)) {
          f32x16 s = zero16();
#pragma unroll
          for (int cc = 0; cc < C::KC; ++cc) s = mfma32(k_rows.get(tK, 32 * kh, cc), qf[cc], s);
          bf16x8 vt[2][C::DB];
#pragma unroll
          for (int ck = 0; ck < 2; ++ck)
#pragma unroll
            for (int db = 0; db < C::DB; ++db) vt[ck][db] = v_cols.get(tV, 32 * kh + 16 * ck, db);
          if (t >= first_masked) mask_half(s, kv_lim - t * C::BN - 32 * kh);
          bf16x8 pb[2];
          float l_new = l_run;
          half_exps(s, mc, pb, l_new);
          half_settle(s, [&] { return half_max(s, C::BN); }, pb, l_new, m_ref, mc, l_run, o);
#pragma unroll
          for (int ck = 0; ck < 2; ++ck)
#pragma unroll
            for (int db = 0; db < C::DB; ++db) o[db] = mfma32(vt[ck][db], pb[ck], o[db]);
        }
        wait_async_loads();
        lds_barrier();
      };
      // The loop starts on a multiple of 32 bytes whatever stands in front of it (d = 64: six instructions on).  2280 tokens, 2 x
      // 64, 19.1 us; at 12 past one 19.6, at 24 past 19.25.  At d = 128, and under the mask, the same anywhere.
      asm volatile(".p2align 6\n\ts_nop 0\n\ts_nop 0");
      for (int t = 0; t < n_tiles; t += 2) {
        half_tile(t, sK0, sV0, sK1, sV1);
        if (t + 1 < n_tiles) half_tile(t + 1, sK1, sV1, sK0, sV0);
      }

      // merge: the waves of the second keys put down reference, sum and output, those of the first take them up
      // (in the tile buffers, which are free)
      float* part_o = reinterpret_cast<float*>(rb_u == 0 ? sK1 : sV1);
      float* part_ml = reinterpret_cast<float*>(sV0) + 128 * rb_u;
      if (kh_u == 1) {
        part_ml[lane] = m_ref;
        part_ml[64 + lane] = l_run;
#pragma unroll
        for (int db = 0; db < C::DB; ++db)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 x = {o[db][4 * g], o[db][4 * g + 1], o[db][4 * g + 2], o[db][4 * g + 3]};
            *reinterpret_cast<f32x4*>(part_o + ((4 * db + g) * 64 + lane) * 4) = x;
          }
      }
      lds_barrier();
      if (kh_u == 0) {
        const float m_other = part_ml[lane], l_other = part_ml[64 + lane];
        const float m_new = fmaxf(m_ref, m_other);
        const float a_own = m_new == m_ref ? 1.f : fast_exp2((m_ref - m_new) * c);
        const float a_other = m_new == m_other ? 1.f : fast_exp2((m_other - m_new) * c);
        const float l_half = l_run * a_own + l_other * a_other;
        const float l_tot = l_half + xor32(l_half);
        const float inv = 1.0f / l_tot;
        const auto ro = make_rsrc(out + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D,
                                  (uint32_t)min(L - q0, 64) * row_bytes);
        const auto rl = make_rsrc(lse + (size_t)it.head * T + it.row0 + q0, (uint32_t)min(L - q0, 64) * 4u);
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, m_new * scale + __logf(l_tot)), rl,
                                              hh == 0 ? (32 * rb + l32) * 4 : 4 * 64, 0, 0);
#pragma unroll
        for (int db = 0; db < C::DB; ++db) {
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(part_o + ((4 * db + g) * 64 + lane) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[db][4 * g + e] = o[db][4 * g + e] * a_own + x[e] * a_other;
          }
          store_block(ro, off + 64u * db, o[db], inv);
        }
      }
    }
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

// instantiated in this order (the bidirectional kernels first)
#define KNAP_FWD_INSTANCE(D, CAUSAL)                                                                    \
  template __global__ void attn_fwd_kernel<D, CAUSAL>(const __bf16*, const __bf16*, const __bf16*,      \
                                                      const int32_t*, int, int, float, __bf16*, float*, \
                                                      unsigned*);
KNAP_FWD_INSTANCE(64, false)
KNAP_FWD_INSTANCE(128, false)
KNAP_FWD_INSTANCE(64, true)
KNAP_FWD_INSTANCE(128, true)
#undef KNAP_FWD_INSTANCE

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

template <int D, bool CAUSAL>
static hipError_t launch_fwd_t(const void* q, const void* k, const void* v, const int32_t* cu, int n_seq,
                               int H, float scale, void* out, float* lse, unsigned* counters, int grid,
                               hipStream_t stream) {
  const size_t dyn = (size_t)(2 * n_seq + 1) * sizeof(int);
  hipLaunchKernelGGL((attn_fwd_kernel<D, CAUSAL>), dim3(grid), dim3(kThreads), dyn, stream,
                     (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, cu, n_seq, H, scale,
                     (__bf16*)out, lse, counters);
  return hipGetLastError();
}

hipError_t launch_fwd(const void* q, const void* k, const void* v, const int32_t* cu, int n_seq,
                      int H, int d, float scale, bool causal, void* out, float* lse, unsigned* counters, int grid,
                      hipStream_t stream) {
  if (!causal) {
    if (d == 64) return launch_fwd_t<64, false>(q, k, v, cu, n_seq, H, scale, out, lse, counters, grid, stream);
    return launch_fwd_t<128, false>(q, k, v, cu, n_seq, H, scale, out, lse, counters, grid, stream);
  }
  if (d == 64) return launch_fwd_t<64, true>(q, k, v, cu, n_seq, H, scale, out, lse, counters, grid, stream);
  return launch_fwd_t<128, true>(q, k, v, cu, n_seq, H, scale, out, lse, counters, grid, stream);
}

int fwd_workgroups_per_cu(int d) {
  int n = 0;
  hipError_t e = (d == 64)
      ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, attn_fwd_kernel<64, false>, kThreads, 0)
      : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, attn_fwd_kernel<128, false>, kThreads, 0);
  if (e != hipSuccess || n < 1) { (void)hipGetLastError(); n = 1; }
  return n;
}

}  // namespace knap
