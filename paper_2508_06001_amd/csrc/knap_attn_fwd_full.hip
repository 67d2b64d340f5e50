// Forward kernel without the mask: out = softmax(scale q k^T) v per (sequence, head) of a packed bag, with the row log-sum-exp
// (Sec. 3.4 / the attention listing of Sec. 3.5: full bidirectional attention inside each sequence, none across sequences).
//
// Orientation, LDS tiles and queues are those of knap_attn_fwd.hip (the causal kernel): S^T = K Q^T, so that a lane holds one
// query, O^T += V^T P^T, keys and values in tiles of 64 rows, copied global -> LDS asynchronously, two buffers of each.  Items come
// in three sizes, and a workgroup of 4 waves does all of them:
//
//  * Pairs of query tiles that follow each other, 256 rows, 64 per wave (two blocks of 32).  Every LDS operand feeds two MFMAs, one per
//    block, and every tile that is copied serves 256 queries: 512 bytes of LDS operands and half the copies per MFMA of the 32-row form.
//    What bounds the loop at the clock that the power limit leaves is the mix of MFMAs, operand reads, copies and arithmetic: a bare
//    loop of MFMAs alone (random operands) runs at 1750 TFLOP/s, with 1 KB of operands per MFMA at 1430, with the arithmetic of the
//    softmax as well at 1310, with the copies and a barrier per tile at 1130 to 1190; half the operands alone: 1640.  The registers
//    just allow it: 128 (O) + 64 (Q) + 32 (scores) + operands in flight, of the 256 of two waves per SIMD (168 of three at d = 64).
//    Three K operands in flight, not four, and what depends on the lane formed where it is used (lane_id()): with four, eight values
//    were reloaded in every turn, 12 % slower than the 32-row form.
//  * Single query tiles, 128 rows, 32 per wave, for the shorter sequences and the end of the list: see there.
//  * Parts of 64 rows (knap_attn_fwd_part.h) where the last round is thin.
//
// Softmax of the pairs: the exponent reference of a row is the maximum over its first 64 keys and stays (the accumulators are not
// rescaled: in this loop that cost 500 to 1500 spilled values, in whatever form).  Nothing is lost by that but rounding: the weight
// of a key far above the reference carries a relative error of 2^-9, as any other, where a reference that moves up to it would make
// its weight exactly one.  So where the probabilities of a half (32 keys) exceed kLargeSum, what rounding took from them goes through
// the MFMAs as a second bf16 term.  Errors against 64 bits, reference moving (as in the other forms) -> this, one key entry in
// a hundred eight times as large: 16000 keys, d = 128, out 1.93e-3 -> 1.88e-3, lse 7.2e-5 -> 6.4e-5; 4096, d = 64, out 1.90e-3 ->
// 1.89e-3, lse 1.80e-4 -> 1.71e-4; N(0,1) inputs the same bits.  An item whose sums or outputs leave the range all the same (keys e^69
// above the first 64; infinities) is done again in parts, whose reference moves.
//
// Forward in us, 24 x 128 where nothing else is said, one form of 32 rows -> this file: 65536 and 200 short 45500 -> 42600, 14 of
// 406..14415 tokens 6130 -> 5650, three heads of up to 131072 23950 -> 21900, 16 of 4096 2970 -> 2740, 17 of 328..4533 1045 -> 1000, 4173
// and 4096 410 -> 395, one of 4292 254 -> 241, 32 of 256..648 138 -> 134; 48 x 64, 8 of 4096 1760 -> 1630, 10 of 310..6795 1450 -> 1400.
#include "knap_attn_fwd_part.h"

#include <type_traits>

namespace knap {

constexpr float kLn2 = 0.6931471805599453f;

// a wave-uniform value whose uses cannot be moved in front of this: what a form derives from it is not formed ahead of all forms
__device__ __forceinline__ int uniform_here(int x) {
  asm volatile("" : "+s"(x));
  return x;
}

template <int D>
struct FwdFullCfg : FwdCfg<D> {
  static constexpr int QB = 2;                           // blocks of 32 queries of a wave, pairs of tiles
  static constexpr int AHEAD = D == 64 ? 2 : 3;          // K operands requested ahead of their MFMAs
  static constexpr int ROWS_PER_INSTR = 512 / D;         // rows that one instruction copies, and ...
  static constexpr int COPIES = FwdCfg<D>::BN / (4 * ROWS_PER_INSTR);     // ... those of a wave for its share of a tile of K or V
  // of a lane's 32 probabilities of a half, 16 of either of its two queries, against the reference.  Without the second term (2048) the error of out
  // grew by up to 5 % on the bags above, at 512 (d = 128) by up to 1.7 %; forward of 16 x 4096 of them, 48 x 64, us: 256 3584, 512 3408
  static constexpr float kLargeSum = D == 64 ? 512.f : 256.f;
};

template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_fwd_full_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
    const int32_t* __restrict__ cu, int n_seq, int H, float scale,
    __bf16* __restrict__ out, float* __restrict__ lse, unsigned* __restrict__ counters) {
  using C = FwdFullCfg<D>;
  constexpr int QB = C::QB, TAIL_ROUNDS = pair_tail_rounds(D);
  extern __shared__ int s_dyn[];
  int* s_order = s_dyn;
  int* s_start = s_dyn + n_seq;
  __shared__ __attribute__((aligned(1024))) __bf16 sK0[C::TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) __bf16 sK1[C::TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) __bf16 sV0[C::TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) __bf16 sV1[C::TILE_ELEMS];
  const int T = cu[n_seq];
  build_schedule<128, kThreads, false>(cu, n_seq, H, s_order, s_start, reinterpret_cast<int*>(&sK0[0]));
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float c = scale * kLog2e;
  __shared__ int s_ticket, s_redo, s_paired;
  EvenQueue<2, 1> queue;
  queue.init(counters);
  if (tid < 64) {
    // even_shares(), and beside it how many of the queue's items may be paired, where there are more than the tail
    const bool enough = s_start[n_seq] > TAIL_ROUNDS * (int)gridDim.x;
    auto items_of = [&](int r) { return r < n_seq ? s_start[r + 1] - s_start[r] : 0; };
    int behind = 0;
    if (enough)
      for (int r0 = 0; r0 < n_seq; r0 += 64) {
        const int items = items_of(r0 + lane);
        behind += __builtin_amdgcn_readlane(wave_scan(queue.share(items, r0 + lane) * item_work(items / H)), 63);
      }
    int before = 0, paired = 0;
    bool stop = !enough;
    for (int r0 = 0; r0 < n_seq; r0 += 64) {
      const int r = r0 + lane, items = items_of(r), n = queue.share(items, r);
      const int sum = wave_scan(n), all = __builtin_amdgcn_readlane(sum, 63);
      if (!stop) {
        const int tiles = items / H, work = max(1, item_work(tiles)), done = wave_scan(n * work);
        const int some = pairable(n, tiles, work, behind - done, TAIL_ROUNDS * queue.per);
        const unsigned long long less = __builtin_amdgcn_ballot_w64(some < n);
        stop = less != 0;
        const int first = stop ? __builtin_ctzll(less) : 63;
        paired = before + __builtin_amdgcn_readlane(sum - n + some, first);
        behind -= __builtin_amdgcn_readlane(done, 63);
      }
      if (r < n_seq) s_start[r] = before + sum - n;
      before += all;
    }
    if (lane == 0) {
      s_start[n_seq] = before;
      s_paired = paired;
      s_redo = -1;
    }
  }
  __syncthreads();
  deal_even<128, false>(queue, cu, n_seq, s_order, s_start);
  // tickets: pairs of items that follow each other, single ones, parts
  const int pairs = __builtin_amdgcn_readfirstlane(item_pairs(s_paired, queue.wide, TAIL_ROUNDS * queue.per, least_pairs(D, queue.per)));
  const int singles = queue.wide - pairs;         // tickets before the parts
  const int tickets = singles + queue.parts;
  const bool draws = tickets > queue.per;
  auto drawn_next = [&](unsigned n) {
    if ((int)n == tickets - 1) atomicExch(queue.ctr, 0u);     // the queue's last draw
    return queue.later_ticket(n);
  };
  bool is_pair = false;        // (where there are pairs somebody draws: the tail behind them is longer than a round)
  // item i of this queue's; is_pair: whether item i + 1 is the tile behind it
  auto take = [&](int i) {
    const int r = __builtin_amdgcn_readfirstlane(rank_of_item(s_start, n_seq, i));
    const int at = i - __builtin_amdgcn_readfirstlane(s_start[r]), end = __builtin_amdgcn_readfirstlane(s_start[r + 1]);
    WorkItem x = sequence_of_rank(r, cu, s_order);
    const int per_head = (x.len + 127) / 128;
    const int rem = queue.locate(per_head * H, r, at);
    x.head = __builtin_amdgcn_readfirstlane(rem / per_head);
    x.tile = __builtin_amdgcn_readfirstlane(rem - x.head * per_head);
    is_pair = i + 1 < end && x.tile + 1 < per_head && queue.locate(per_head * H, r, at + 1) == rem + 1;
    return x;
  };
  int ticket = queue.first_ticket();
  WorkItem it;
  unsigned next_ticket;
  const FwdPtrs g = {q, k, v, out, lse, T, H, scale};
  const FwdLds lds = {sK0, sK1, sV0, sV1};
  // A bag of so few items that all of them go out in parts, one for a workgroup: ahead of everything that the other forms keep in
  // registers, whose set-up costs 0.5 us (4 sequences of up to 311 tokens, 2 x 64: 8.6 -> 7.8 us).  The hint orders the code behind it so that
  // the first items of a launch fetch less of it, forward at 24 x 128 in us without -> with: 4 sequences of 256 12.44 -> 12.13, one of 300
  // 9.64 -> 9.30, 2 of 400 14.76 -> 14.32, one of 600 12.82 -> 12.52; larger bags and d = 64 the same.
  if (__builtin_expect_with_probability(singles == 0, 1, 0.99)) {
    if (ticket < tickets) {
      it = take(queue.item_of_part(ticket));
      const int q0 = it.tile * 128 + 64 * (ticket & 1);
      if (q0 < it.len) fwd_part<D, false>(g, lds, it, q0, lane, wave_id);
    }
    return;
  }

  bf16x2 ones;
  ones[0] = (__bf16)1.0f;
  ones[1] = (__bf16)1.0f;

  int whole = -1;               // first item of a pair that is done 64 rows after the other ...
  bool drawn = false;           // ... while the ticket after it has been drawn
  int single = -1, other = -1;  // items that are taken singly, one after the other
pairs_of_items:
  if (ticket < pairs) {
  it = take(2 * ticket);
  if (!is_pair) {
    single = 2 * ticket;
    other = single + 1;
  } else {
  const int H_pairs = uniform_here(H), wave = uniform_here(wave_id);
  const size_t row_stride = (size_t)H_pairs * D;
  const uint32_t row_bytes = (uint32_t)(row_stride * sizeof(__bf16));
  // This wave's 64 rows lie in the first or the second of the two tiles.  Descriptors of q and out cover one tile each, as those of
  // the other forms: 256 rows of 65536 heads of 128 are 2^32 bytes.
  const int own_tile = 128 * (wave >> 1), own_row = 64 * (wave & 1);
  RowReaderX<D> rows;
  ColReaderX<D> cols;
  const int ln = lane_id();
  rows.init(ln);
  cols.init(ln);
  bf16x8 qf[QB][C::KC];
  constexpr int ROWS_PER_INSTR = C::ROWS_PER_INSTR, COPIES = C::COPIES;
  // This wave's share of a tile of 64 rows of K or V, rows 16 wave + 4 i + lane / 16 of it (D = 128; 8 i + lane / 8 at D = 64): one
  // lane-dependent offset for all of them, the others formed where they are used
  const int cp_row = wave * COPIES * ROWS_PER_INSTR + ln / Tile<D>::CPR;
  const uint32_t cp_off = (uint32_t)cp_row * row_bytes + (uint32_t)Tile<D>::chunk_pos(cp_row, ln % Tile<D>::CPR) * 16u;
  auto load_rows = [&](const __bf16* __restrict__ src, int t, __bf16* dst) __attribute__((always_inline)) {
    const int kv0 = t * C::BN;
    const uint32_t bytes = (uint32_t)max(0, min(it.len - kv0, C::BN)) * row_bytes;
    const auto r = make_rsrc(src + (size_t)(it.row0 + kv0) * row_stride + (size_t)it.head * D, bytes);
#pragma unroll
    for (int i = 0; i < COPIES; ++i) {
      uint32_t off = cp_off;
      if (i) asm volatile("" : "+v"(off));
      // 4 i (D = 128) or 8 i (D = 64) rows further on the chunk's position differs by an exclusive or with i or 4 i
      off = (off ^ (uint32_t)((D == 128 ? i : 4 * i) * 16)) + (uint32_t)(i * ROWS_PER_INSTR) * row_bytes;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(dst + (wave * COPIES + i) * ROWS_PER_INSTR * Tile<D>::LD), 16, (int)off, 0, 0, 0);
    }
  };
  // what a pair needs before its first product: tile 0 and the query rows (rows past the end read as zero)
  auto load_wide = [&]() __attribute__((always_inline)) {
    load_rows(k, 0, sK0);
    load_rows(v, 0, sV0);
    const int q0 = it.tile * 128 + own_tile;
    const int ln = lane_id(), l32 = ln & 31, hh = ln >> 5;
    const uint32_t q_off = (uint32_t)(own_row + l32) * row_bytes + (uint32_t)(8 * hh) * 2u;
    const auto rq = make_rsrc(q + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D, (uint32_t)min(it.len - q0, 128) * row_bytes);
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) qf[b][cc] = __builtin_bit_cast(bf16x8, buffer_load16(rq, q_off + (uint32_t)(32 * b) * row_bytes + 32u * cc));
  };
  load_wide();
  wait_async_loads();
  lds_barrier();
  for (;;) {
    const int L = it.len;
    const int q0 = it.tile * 128;
    const int n_tiles = (L + C::BN - 1) / C::BN;
    const int t_draw = (n_tiles - 1) & ~1;
    f32x16 o[QB][C::DB];
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
      for (int db = 0; db < C::DB; ++db) o[b][db] = zero16();
    float mc[QB], l[QB];       // the reference, times c, and this lane's share of the row sums
    constexpr int AHEAD = C::AHEAD;
    bf16x8 af[C::KC];
    auto first_keys = [&](const __bf16* tK) __attribute__((always_inline)) {
      const int rb = rows.fresh();
#pragma unroll
      for (int cc = 0; cc < AHEAD; ++cc) af[cc] = rows.get(tK, rb, cc);
    };
    auto scores = [&](const __bf16* tK, f32x16 (&s)[QB]) {
      const int rb = rows.fresh();
      KNAP_SCHED_FENCE();
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) {
#pragma unroll
        for (int b = 0; b < QB; ++b) s[b] = mfma32(af[cc], qf[b][cc], cc == 0 ? zero16() : s[b]);
        if (cc + AHEAD < C::KC) af[cc + AHEAD] = rows.get(tK, rb, cc + AHEAD);
        KNAP_SCHED_FENCE();
      }
    };
    // The reference of the item's probabilities is the maximum of its first 64 keys: here of the second 32, in the loop's first turn of
    // the first 32, whose scores it needs anyway
    {
      f32x16 s[QB];
      first_keys(sK0 + 32 * Tile<D>::LD);
      scores(sK0 + 32 * Tile<D>::LD, s);
      const int hh = lane_id() >> 5;
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        mc[b] = half_max(s[b], L - 32, hh);
        l[b] = 0.f;
      }
    }
    // 32 keys, from k0 on: their scores (the first of their LDS operands stand in `af`), probabilities in two chunks of 16, and each
    // chunk's product with the values while the next one's probabilities are formed.  Whether they are large.
    auto half_step = [&](auto masked_tag, bool first, int k0, const __bf16* tK, const __bf16* tV, const __bf16* nextK) __attribute__((always_inline)) {
      f32x16 s[QB];
      scores(tK, s);
      if constexpr (decltype(masked_tag)::value) {
        const int hh = lane_id() >> 5;
#pragma unroll
        for (int b = 0; b < QB; ++b) mask_half(s[b], L - k0, hh);
        KNAP_SCHED_FENCE();
      }
      if (first) {
        const int hh = lane_id() >> 5;
#pragma unroll
        for (int b = 0; b < QB; ++b) {
          const float m = fmaxf(mc[b], half_max(s[b], C::BN, hh));
          mc[b] = fmaxf(m, xor32(m)) * c;
        }
      }
      KNAP_SCHED_FENCE();
      const int cb = cols.fresh(), rb = rows.fresh();
      uint32_t w[2][QB][4];
      const float before = l[0] + l[1];
      // probabilities 8 cq + 4 part .. + 3 of block b
      auto exp_slice = [&](int cq, int b, int part) __attribute__((always_inline)) {
        float p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] = fast_exp2(__builtin_fmaf(s[b][8 * cq + 4 * part + e], c, -mc[b]));
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          bf16x2 x;
          x[0] = (__bf16)p[2 * e];
          x[1] = (__bf16)p[2 * e + 1];
          l[b] = __builtin_amdgcn_fdot2_f32_bf16(x, ones, l[b], false);
          w[cq][b][2 * part + e] = __builtin_bit_cast(uint32_t, x);
        }
      };
      auto second_product = [&](int cq, auto between) __attribute__((always_inline)) {
        bf16x8 bf[C::DB];
        constexpr int AH2 = 2;
#pragma unroll
        for (int db = 0; db < AH2; ++db) bf[db] = cols.get(tV, cb, 16 * cq, db);
        bf16x8 pb[QB];
#pragma unroll
        for (int b = 0; b < QB; ++b) {
          const u32x4 x = {w[cq][b][0], w[cq][b][1], w[cq][b][2], w[cq][b][3]};
          pb[b] = __builtin_bit_cast(bf16x8, x);
        }
        KNAP_SCHED_FENCE();
#pragma unroll
        for (int db = 0; db < C::DB; ++db) {
#pragma unroll
          for (int b = 0; b < QB; ++b) o[b][db] = mfma32(bf[db], pb[b], o[b][db]);
          if (db + AH2 < C::DB) bf[db + AH2] = cols.get(tV, cb, 16 * cq, db + AH2);
          between(db);
          KNAP_SCHED_FENCE();
        }
      };
#pragma unroll
      for (int j = 0; j < 2 * QB; ++j) exp_slice(0, j >> 1, j & 1);
      KNAP_SCHED_FENCE();
      second_product(0, [&](int db) __attribute__((always_inline)) {
        if constexpr (C::DB == 4) exp_slice(1, db >> 1, db & 1);
        else { exp_slice(1, db, 0); exp_slice(1, db, 1); }
      });
      // l[0] + l[1] - before, the increase, plus 2^-16 of what was there: from 2^16 kLargeSum on every half counts as large, before one
      // row's sum hides the other's increase in its rounding
      const bool large = __builtin_amdgcn_ballot_w64(!(__builtin_fmaf(before, 0x1p-16f - 1.0f, l[0] + l[1]) <= C::kLargeSum)) != 0;
      // (8 bytes of code where a subtraction has 4; with the 4 of this behind it the loop goes on 8 bytes further and loses nothing:
      // 65536 tokens and 200 short, 24 x 128, us: 41250 with a subtraction, 41540 without this, 41330; 32 of 2048 1481, 1489, 1481)
      asm volatile("s_nop 0");
      second_product(1, [&](int db) __attribute__((always_inline)) {
        if (nextK) {
          constexpr int PER = (AHEAD + C::DB - 1) / C::DB;
#pragma unroll
          for (int e = 0; e < PER; ++e)
            if (db + C::DB * e < AHEAD) af[db + C::DB * e] = rows.get(nextK, rb, db + C::DB * e);
        }
      });
      return large;
    };
    // What rounding took from the probabilities of 32 keys, as a second term: P = bf16(P) + bf16(P - bf16(P)).  For halves with
    // probabilities far above one, whose rounding would otherwise dominate the error of their rows.
    auto add_rest = [&](auto masked_tag, int k0, const __bf16* tK, const __bf16* tV) __attribute__((always_inline)) {
      f32x16 s[QB];
      first_keys(tK);
      scores(tK, s);
      const int cb = cols.fresh();
      bf16x8 pb[QB][2];
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        if constexpr (decltype(masked_tag)::value) mask_half(s[b], L - k0, lane_id() >> 5);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = fast_exp2(__builtin_fmaf(s[b][r], c, -mc[b]));
          s[b][r] = p - (float)(__bf16)p;
        }
#pragma unroll
        for (int ck = 0; ck < 2; ++ck)
          pb[b][ck] = pack8_sum(s[b][8 * ck], s[b][8 * ck + 1], s[b][8 * ck + 2], s[b][8 * ck + 3], s[b][8 * ck + 4], s[b][8 * ck + 5],
                                s[b][8 * ck + 6], s[b][8 * ck + 7], l[b]);
        KNAP_SCHED_FENCE();
      }
#pragma unroll
      for (int i = 0; i < 2 * C::DB; ++i) {
        const bf16x8 bf = cols.get(tV, cb, 16 * (i / C::DB), i % C::DB);
#pragma unroll
        for (int b = 0; b < QB; ++b) o[b][i % C::DB] = mfma32(bf, pb[b][i / C::DB], o[b][i % C::DB]);
        KNAP_SCHED_FENCE();
      }
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    auto process_tile = [&](auto masked_tag, bool first, int t, const __bf16* tK, const __bf16* tV, __bf16* nK, __bf16* nV) __attribute__((always_inline)) {
      first_keys(tK);
      load_rows(k, t + 1, nK);
      load_rows(v, t + 1, nV);
      const bool large0 = half_step(masked_tag, first, t * C::BN, tK, tV, tK + 32 * Tile<D>::LD);
      const bool large1 = half_step(masked_tag, false, t * C::BN + 32, tK + 32 * Tile<D>::LD, tV + 32 * Tile<D>::LD, nullptr);
      if (__builtin_expect_with_probability(large0 || large1, 0, 0.9999)) {
#pragma unroll 1
        for (int half = large0 ? 0 : 1; half < (large1 ? 2 : 1); ++half)
          add_rest(masked_tag, t * C::BN + 32 * half, tK + 32 * half * Tile<D>::LD, tV + 32 * half * Tile<D>::LD);
      }
      wait_async_loads();
      lds_barrier();
    };
    const int n_full = L / C::BN;
    // Behind a multiple of 64 bytes whatever stands in front of it.  Of 16 places (11 bags, against code without this) the even instructions past
    // one, multiples of 8 bytes, are 0.998 to 1.003, the fourth the best, the odd ones 0.995 to 0.998.
    asm volatile(".p2align 6\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
    for (int t = 0; t < n_full; t += 2) {
      if (t == t_draw && tid == 0) next_ticket = atomicAdd(queue.ctr, 1u);
      process_tile(no, t == 0, t, sK0, sV0, sK1, sV1);
      if (t + 1 < n_full) process_tile(no, false, t + 1, sK1, sV1, sK0, sV0);
    }
    if (n_full < n_tiles) {       // the ragged last tile, whichever buffer it is in (the tile after it is never loaded)
      if (n_full == t_draw && tid == 0) next_ticket = atomicAdd(queue.ctr, 1u);
      const bool odd = n_full & 1;
      process_tile(yes, n_full == 0, n_full, odd ? sK1 : sK0, odd ? sV1 : sV0, odd ? sK0 : sK1, odd ? sV0 : sV1);
    }
    // A row whose sum or output left the range (a later key's score far above those of the first 64: 2^100, or infinities and NaN
    // among the inputs) sends the whole item through the narrow form, which moves its reference.
    float inv[QB];
    bool redo = false;
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      l[b] += xor32(l[b]);
      inv[b] = 1.0f / l[b];
      float none = 0.f;
#pragma unroll
      for (int db = 0; db < C::DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) none = __builtin_fmaf(o[b][db][r], 0.f, none);
      redo = redo || !(l[b] <= 0x1p100f) || none != 0.f;
    }
    if (__builtin_amdgcn_ballot_w64(redo) != 0 && lane == 0) s_redo = ticket;
    if (tid == 0) s_ticket = drawn_next(next_ticket);     // every wave read the old one many barriers ago
    lds_barrier();
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(s_redo) == ticket, 0)) {
      whole = 2 * ticket;
      drawn = true;
      ticket = __builtin_amdgcn_readfirstlane(s_ticket);
      break;
    }
    const auto ro = make_rsrc(out + (size_t)(it.row0 + q0 + own_tile) * row_stride + (size_t)it.head * D, (uint32_t)min(L - q0 - own_tile, 128) * row_bytes);
    const auto rl = make_rsrc(lse + (size_t)it.head * T + it.row0 + q0, (uint32_t)min(L - q0, 128 * QB) * 4u);
    // the next item's first loads go out before this one's results are stored, so that they travel under the epilogue
    ticket = __builtin_amdgcn_readfirstlane(s_ticket);
    bool more = ticket < pairs;
    if (more) {
      it = take(2 * ticket);
      if (!is_pair) {
        single = 2 * ticket;
        other = single + 1;
        more = false;
      }
    }
    if (more) load_wide();
    KNAP_SCHED_FENCE();
    const int ln = lane_id(), l32 = ln & 31, hh = ln >> 5;
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      const uint32_t q_off = (uint32_t)(own_row + l32) * row_bytes + (uint32_t)(8 * hh) * 2u;
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, mc[b] * kLn2 + __logf(l[b])), rl, hh == 0 ? (wave * 64 + 32 * b + l32) * 4 : 4 * 128 * QB, 0, 0);
#pragma unroll
      for (int db = 0; db < C::DB; ++db) store_block(ro, q_off + (uint32_t)(32 * b) * row_bytes + 64u * db, o[b][db], inv[b]);
    }
    if (!more) break;
    wait_vm<2 * QB * C::DB>();
    lds_barrier();
  }
  }
  }

  // Single items: 128 queries, 32 per wave (fwd_tile).
  if (single < 0 && ticket >= pairs && ticket < singles && whole < 0) single = ticket + pairs;
  if (single >= 0) {
    lds_barrier();            // every wave has the ticket; nobody reads a tile any longer
    const int H_single = uniform_here(H), wave = uniform_here(wave_id);
    const size_t row_stride = (size_t)H_single * D;
    const uint32_t row_bytes = (uint32_t)(row_stride * sizeof(__bf16));
    constexpr int COPIES = C::COPIES;
    const int ln = lane_id();
    const int l32 = ln & 31, hh = ln >> 5;
    RowReader<D> k_rows;   // K tile rows -> A operands of S^T
    ColReader<D> v_cols;   // V tile columns -> A operands of O^T += V^T P^T
    k_rows.init(ln);
    v_cols.init(ln);
    constexpr int KC = C::KC, DB = C::DB;
    const uint32_t q_off = (uint32_t)(wave * 32 + l32) * row_bytes + (uint32_t)(8 * hh) * 2u;
    bf16x8 qs[KC];
    auto copy_rows = [&](const __bf16* __restrict__ src, int t, __bf16* dst) __attribute__((always_inline)) {
      const int kv0 = t * C::BN;
      const uint32_t bytes = (uint32_t)max(0, min(it.len - kv0, C::BN)) * row_bytes;
      tile_load_async<D>(dst, make_rsrc(src + (size_t)(it.row0 + kv0) * row_stride + (size_t)it.head * D, bytes), row_bytes, C::BN, wave, ln);
    };
    // what an item needs before its first product, the keys of tile 0 and the query rows (rows past the end read as zero), and
    // behind it what its first turn of the loop reads: the values of tile 0 and the keys of tile 1
    auto load_first = [&]() __attribute__((always_inline)) {
      const int q0 = it.tile * 128;
      copy_rows(k, 0, sK0);
      const auto rq = make_rsrc(q + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D, (uint32_t)min(it.len - q0, 128) * row_bytes);
#pragma unroll
      for (int cc = 0; cc < KC; ++cc) qs[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rq, q_off + 32u * cc));
      KNAP_SCHED_FENCE();
      copy_rows(v, 0, sV0);
      copy_rows(k, 1, sK1);
      KNAP_SCHED_FENCE();
    };
    it = take(single);
    load_first();
    wait_vm<2 * COPIES>();
    lds_barrier();
    for (;;) {
      const int L = it.len;
      const int q0 = it.tile * 128;
      const int n_tiles = (L + C::BN - 1) / C::BN;
      const int first_masked = L / C::BN;
      // the next ticket is drawn in the last turn of the loop
      auto draw = [&] { if (draws && other < 0 && tid == 0) next_ticket = atomicAdd(queue.ctr, 1u); };
      f32x16 o[DB];
      float m_ref, l_run;
      // (a last half without keys is left out at d = 64 alone: at d = 128 20 of 350 to 450 tokens gain 1 %, 100 of 290 lose as much)
      fwd_tile<D, false>(lds, qs, k_rows, v_cols, c, n_tiles, q0 + 32 * wave < L ? n_tiles : 0, D == 128 || L > n_tiles * C::BN - 32, first_masked, L, hh, [&](int t, __bf16* dst) __attribute__((always_inline)) { copy_rows(k, t, dst); },
                  [&](int t, __bf16* dst) __attribute__((always_inline)) { copy_rows(v, t, dst); }, draw, o, m_ref, l_run);
      const auto ro = make_rsrc(out + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D, (uint32_t)min(L - q0, 128) * row_bytes);
      const auto rl = make_rsrc(lse + (size_t)it.head * T + it.row0 + q0, (uint32_t)min(L - q0, 128) * 4u);
      if (draws && other < 0 && tid == 0) s_ticket = drawn_next(next_ticket);     // every wave read the old one many barriers ago
      lds_barrier();          // nobody reads a tile any longer
      if (other >= 0) {
        single = other;
        other = -1;
      } else {
        if (draws) ticket = __builtin_amdgcn_readfirstlane(s_ticket);
        single = draws && ticket >= pairs && ticket < singles ? ticket + pairs : -1;
      }
      const bool more = single >= 0;
      if (more) {
        it = take(single);
        load_first();
      }
      KNAP_SCHED_FENCE();
      // epilogue: normalise, store lse (natural log) and out (bf16)
      const float l_tot = l_run + xor32(l_run);
      const float inv = 1.0f / l_tot;
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, m_ref * scale + __logf(l_tot)), rl, hh == 0 ? (wave * 32 + l32) * 4 : 4 * 128, 0, 0);
#pragma unroll
      for (int db = 0; db < DB; ++db) store_block(ro, q_off + 64u * db, o[db], inv);
      if (!more) break;
      // the keys and the query rows have landed: all but the copies behind them and the stores, which are younger (in-order completion)
      wait_vm<2 * COPIES + 1 + 2 * DB>();
      lds_barrier();
    }
    if (!draws) return;
    if (ticket < pairs) {
      lds_barrier();
      goto pairs_of_items;
    }
  }

  // Narrow items: parts, and pairs that have to be done again
  lds_barrier();                        // every wave has the tickets before the next ones are put down
  int done = 0;
  for (;;) {
    int q0;
    bool last = true;
    if (whole >= 0) {
      it = take(whole);
      q0 = it.tile * 128 + 64 * done;
      ++done;
      last = done == C::QB * 2 || q0 + 64 >= it.len;
    } else if (ticket >= singles && ticket < tickets) {
      const int part = ticket - singles;
      it = take(queue.item_of_part(part));
      q0 = it.tile * 128 + 64 * (part & 1);
    } else {
      return;
    }
    if (q0 < it.len) {
      const FwdPtrs here = {q, k, v, out, lse, T, uniform_here(H), scale};
      fwd_part<D, false>(here, lds, it, q0, lane_id(), uniform_here(wave_id));
    }
    if (last) {
      if (!draws) return;         // every ticket was a first one
      if (!drawn && tid == 0) {
        const unsigned n = atomicAdd(queue.ctr, 1u);
        s_ticket = drawn_next(n);
      }
      lds_barrier();
      if (!drawn) ticket = __builtin_amdgcn_readfirstlane(s_ticket);
      whole = -1;
      done = 0;
      drawn = false;
    }
    lds_barrier();                    // the tile buffers are no longer read, everyone has the ticket before it is drawn again
    if (last && ticket < singles) goto pairs_of_items;
  }
}
template <int D>
static hipError_t launch_full_t(const void* q, const void* k, const void* v, const int32_t* cu, int n_seq, int H, float scale, void* out,
                                float* lse, unsigned* counters, int grid, hipStream_t stream) {
  const size_t dyn = (size_t)(2 * n_seq + 1) * sizeof(int);
  hipLaunchKernelGGL((attn_fwd_full_kernel<D>), dim3(grid), dim3(kThreads), dyn, stream, (const __bf16*)q, (const __bf16*)k,
                     (const __bf16*)v, cu, n_seq, H, scale, (__bf16*)out, lse, counters);
  return hipGetLastError();
}

hipError_t launch_fwd_full(const void* q, const void* k, const void* v, const int32_t* cu, int n_seq, int H, int d, float scale,
                           void* out, float* lse, unsigned* counters, int grid, hipStream_t stream) {
  return d == 64 ? launch_full_t<64>(q, k, v, cu, n_seq, H, scale, out, lse, counters, grid, stream)
                 : launch_full_t<128>(q, k, v, cu, n_seq, H, scale, out, lse, counters, grid, stream);
}

int fwd_workgroups_per_cu(int d) {
  int n = 0;
  const void* fn = d == 64 ? (const void*)attn_fwd_full_kernel<64> : (const void*)attn_fwd_full_kernel<128>;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, kThreads, 0) != hipSuccess || n < 1) { (void)hipGetLastError(); n = 1; }
  return n;
}

}  // namespace knap
