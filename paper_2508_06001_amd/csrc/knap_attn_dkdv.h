// dK/dV kernel of the backward: one text, compiled for either mask in a translation unit of its own (see build.py).
#pragma once

#include "knap_device.h"
#include "knap_kernels.h"

namespace knap {

// ---------------------------------------------------------------------------
// dK/dV kernel.  A persistent workgroup of PAIRS pairs of waves owns a tile of 64 PAIRS key/value rows of one
// (sequence, head) and walks over that sequence's queries 32 rows at a time.  Pair i owns key rows
// [64 i, 64 i + 64) of the tile as two 32-row blocks; the two waves of a pair split the work by output:
//   dV wave: keeps its K rows in registers, S = Q K^T, P = exp2(c S - LSE2), dV += P^T dO, and hands
//            the packed bf16 P to its partner through LDS (one way, double buffered);
//   dK wave: keeps its V rows in registers and runs ONE TILE BEHIND: dP - delta = dO V^T - delta, dS = P (dP - delta)
//            with the partner's P, dK += dS^T Q.
// Each wave holds one accumulator, so two waves fit on a SIMD and each one's MFMAs run against the
// other's exponentials, LDS reads and waits.  With S = Q K^T in the MFMA result layout a lane holds one
// key and its registers run over queries, so P and dS are, unchanged, operands of the second
// products' key side (MFMA takes rows and columns alike); dO and Q enter those through transposing LDS reads.
//
// Every fragment of Q or dO that a wave reads from LDS, row-wise for S / dP and transposed for dV /
// dK, feeds TWO MFMAs, one per key block: 512 bytes of LDS operand per MFMA.  The registers just allow
// it because the accumulators sit on the key side: per wave 128 (dV or dK, 64 x d fp32) + 64 (its K or
// V rows) + 32 (scores of a step) + operands in flight, within the 256 of two waves per SIMD (every
// base address in scalar registers, every LDS address formed next to its read, and everything else that depends on the
// lane taken out of one register: see LaneWord).  Without a spilled register in a step: a reload there waits for the tile
// copy issued just before it (17 causal sequences of 328..4533 tokens, 24 x 128: 1216 -> 1139 us, 14 of 406..14415: 6.42 ->
// 6.27 ms).
//
// The second products are formed as dV^T += dO^T P and dK^T += Q^T dS, so that a lane holds one key and its registers run
// along the row of the result: 16 stores of 16 bytes per wave, where dV itself would take 128 of 2 bytes, predicated by
// row (32 sequences of 256..648 tokens, 24 x 128: 231 -> 215 us; the causal 17 of 328..4533: 1126 -> 1079 us).
//
// Query-side tiles (32 rows of Q and dO, their LSE in base 2 and -delta) go global -> LDS
// asynchronously, one tile ahead, into a ring of three buffers (being filled / dV role / dK
// role).  The buffers are separate arrays and the loop is unrolled once around the ring, so that every
// LDS read names its buffer at compile time and is known not to depend on the copies in flight into
// the others.  (Three tiles ahead in a ring of five measured the same within 0.6 %.)  Rows past the end of the sequence arrive as zeros in all four
// (empty buffer descriptor): P = exp2(0 - 0) = 1 there, but dO = 0 and dP - delta = 0, so they add
// nothing to dV or dK.
//
// CAUSAL (query i sees keys 0..i): a key tile starting at row kv0 only meets the queries from row kv0
// on.  The walk over them runs BACKWARDS, from the sequence's last query tile down to the tiles
// that cross the diagonal (which get the mask): workgroups on different key tiles of one (sequence,
// head) then read the same query tiles at the same time, as they do without the mask, instead of each
// starting at its own diagonal.  Work items are pairs of key tiles of equal total cost (see
// build_schedule).
//
// PAIRS = 4 (8 waves, 256 keys, one workgroup per CU) copies the fewest bytes into LDS per MFMA and is the faster
// one on long sequences.  PAIRS = 2 (4 waves, 128 keys, two workgroups per CU) hides the start and the end of
// an item (K / V rows, first tile and stores) under the other workgroup's loop,
// pads sequences to 128 keys instead of 256 and fills the GPU from half as many keys on; dkdv_pairs() chooses.
// At d = 64 the registers of two pairs (152 of them, 157 under the mask, without a spill) and their 43 KB of LDS leave room for a third
// workgroup on the CU, and a third wave on a SIMD has its MFMAs while the other two form exponentials, which are twice as
// many per MFMA there: 10 sequences of 310..6795 tokens, 48 x 64, 2760 -> 2631 us.
// ---------------------------------------------------------------------------
template <int D, int PAIRS_>
struct Bwd2Cfg {
  static constexpr int PAIRS = PAIRS_;
  static constexpr int THREADS = 128 * PAIRS;
  static constexpr int BM = 32;
  static constexpr int BN = 64 * PAIRS;
  static constexpr int KB = 2;
  static constexpr int NB = D / 32;
  static constexpr int KC = D / 16;
  static constexpr int TILE_ELEMS = BM * Tile<D>::LD;
};

// 16 times the lane's number, plus a multiple of 1024
struct LaneWord {
  int word;
  __device__ __forceinline__ int fresh() const { int w = word; asm volatile("" : "+v"(w)); return w; }
  __device__ static __forceinline__ int l32(int w) { return (w >> 4) & 31; }
  __device__ static __forceinline__ int hh16(int w) { return (w >> 5) & 16; }       // 16 for the upper 32 lanes
  __device__ static __forceinline__ int lane4(int w) { return (w >> 2) & 252; }
};

// LDS of a dK/dV workgroup: the ring (i: 0, 1, 2), the P of its pairs, and a place for copies that nobody needs
struct DkdvLds {
  __bf16 *q0, *do0, *q1, *do1, *q2, *do2;
  float *lse0, *delta0, *lse1, *delta1, *lse2, *delta2, *sink;
  u32x4* p;
};

// what a lane keeps between key tiles
template <int D, int PAIRS>
struct DkdvLane {
  using C = Bwd2Cfg<D, PAIRS>;
  static constexpr int ROWS_PER_INSTR = 512 / D;
  // one instruction copies 1 KB: ROWS_PER_INSTR rows; Q and dO of a tile are dealt to the waves in one or more passes
  static_assert(C::BM % (2 * PAIRS * ROWS_PER_INSTR) == 0, "a pass of the waves is whole rows of a tile");
  static constexpr int P_BLOCK = 64 * 16, P_TILE = 2 * C::KB * P_BLOCK, P_PAIR = 2 * P_TILE;     // bytes of sP
  RowReaderX<D> rows;
  ColReaderX<D> cols;
  // where this lane's 16 bytes of its pair's P lie; its number and its halves are bits of that word, taken out of it where
  // they are needed (a step has no register to spare for each of them)
  LaneWord at;
  uint32_t cp_off;
  int cp_row0, wave, pair, role;     // wave-uniform
  __device__ __forceinline__ void init(int lane, int wave_, int role_, uint32_t row_bytes) {
    wave = wave_;
    role = role_;
    pair = wave & (PAIRS - 1);
    rows.init(lane);
    cols.init(lane);
    at.word = P_PAIR * pair + 16 * lane;
    cp_row0 = wave * ROWS_PER_INSTR;
    const int cp_row = cp_row0 + lane / Tile<D>::CPR;
    cp_off = (uint32_t)cp_row * row_bytes + (uint32_t)Tile<D>::chunk_pos(cp_row, lane % Tile<D>::CPR) * 16u;
  }
};

// One key tile of an item.  `draw` is called behind its first loads, `drawn` when they have landed, `ending` in front of its
// stores.
template <int D, int PAIRS, bool CAUSAL, class Draw, class Drawn, class Ending>
__device__ __forceinline__ void dkdv_tile(const BwdPtrs& g, const DkdvLds& lds, const DkdvLane<D, PAIRS>& me, const WorkItem& it,
                                          int kv_tile, Draw draw, Drawn drawn, Ending ending) {
    using C = Bwd2Cfg<D, PAIRS>;
    using W = DkdvLane<D, PAIRS>;
    const auto *q = g.q, *k = g.k, *v = g.v, *dout = g.dout;
    const float *lse2 = g.lse2, *delta = g.delta;
    const int L = it.len, T = g.T;
    const float scale = g.scale, c = scale * kLog2e;
    const size_t row_stride = (size_t)g.H * D;
    const uint32_t row_bytes = (uint32_t)(row_stride * sizeof(__bf16));
    const size_t head_off = (size_t)it.head * D;
    const auto& rows = me.rows;
    const auto& cols = me.cols;
    const auto& at = me.at;
    const uint32_t cp_off = me.cp_off;
    const int cp_row0 = me.cp_row0, wave = me.wave, pair = me.pair, role = me.role;
    __bf16 *const sQ0 = lds.q0, *const sdO0 = lds.do0, *const sQ1 = lds.q1, *const sdO1 = lds.do1, *const sQ2 = lds.q2, *const sdO2 = lds.do2;
    float *const sLse0 = lds.lse0, *const sDelta0 = lds.delta0, *const sLse1 = lds.lse1, *const sDelta1 = lds.delta1,
          *const sLse2 = lds.lse2, *const sDelta2 = lds.delta2, *const sSink = lds.sink;
    const int kv0 = kv_tile * C::BN;
    // queries this key tile meets: rows q_first .. L - 1 of the sequence; tiles and rows below count from q_first
    const int q_first = CAUSAL ? kv0 : 0;
    const int Lq = L - q_first;
    const __bf16* q_base = q + (size_t)(it.row0 + q_first) * row_stride + head_off;
    const __bf16* do_base = dout + (size_t)(it.row0 + q_first) * row_stride + head_off;
    const float* lse_base = lse2 + (size_t)it.head * T + it.row0 + q_first;
    const float* delta_base = delta + (size_t)it.head * T + it.row0 + q_first;
    const int n_tiles = (Lq + C::BM - 1) / C::BM;
    // CAUSAL: step t works on query tile n_tiles - 1 - t: the walk runs BACKWARDS, from the sequence's last
    // query tile down to the tiles that cross the diagonal of this key tile (which get the mask), so
    // that workgroups on different key tiles of one (sequence, head) read the same query tiles at the same
    // time, as they do without the mask

    bf16x8 kvf[C::KB][C::KC];
    {
      const uint32_t kv_bytes = (uint32_t)min(L - kv0, C::BN) * row_bytes;
      const __bf16* src = (role == 0 ? k : v) + (size_t)(it.row0 + kv0) * row_stride + head_off;
      const auto r = make_rsrc(src, kv_bytes);
      const int w = at.fresh();
#pragma unroll
      for (int kb = 0; kb < C::KB; ++kb) {
        const uint32_t off = (uint32_t)(64 * pair + 32 * kb + LaneWord::l32(w)) * row_bytes + (uint32_t)LaneWord::hh16(w);
#pragma unroll
        for (int cc = 0; cc < C::KC; ++cc) kvf[kb][cc] = __builtin_bit_cast(bf16x8, buffer_load16(r, off + 32u * cc));
      }
    }

    f32x16 acc[C::KB][C::NB];
#pragma unroll
    for (int kb = 0; kb < C::KB; ++kb)
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb) acc[kb][nb] = zero16();

    auto issue_tile = [&](int t, __bf16* tQ, __bf16* tdO, float* tLse, float* tDelta) {
      int q0, n_rows;
      if constexpr (CAUSAL) {
        q0 = max(0, n_tiles - 1 - t) * C::BM;
        n_rows = t < n_tiles ? min(Lq - q0, C::BM) : 0;
      } else {
        q0 = t * C::BM;
        n_rows = max(0, min(L - q0, C::BM));
      }
      const auto rq = make_rsrc(q_base + (size_t)q0 * row_stride, (uint32_t)n_rows * row_bytes);
      const auto rd = make_rsrc(do_base + (size_t)q0 * row_stride, (uint32_t)n_rows * row_bytes);
#pragma unroll
      for (int r = 0; r < C::BM; r += 2 * PAIRS * W::ROWS_PER_INSTR) {
        uint32_t off = cp_off;
        if (r) asm volatile("" : "+v"(off));     // formed here, not kept in a register of its own through the loop
        off += (uint32_t)r * row_bytes;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rq, (__attribute__((address_space(3))) void*)(tQ + (cp_row0 + r) * Tile<D>::LD), 16, (int)off, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rd, (__attribute__((address_space(3))) void*)(tdO + (cp_row0 + r) * Tile<D>::LD), 16, (int)off, 0, 0, 0);
      }
      const float* src = wave == 0 ? lse_base + q0 : delta_base + q0;
      float* dst = wave == 0 ? tLse : wave == 1 ? tDelta : sSink;
      const auto rs = make_rsrc(src, wave < 2 ? (uint32_t)n_rows * 4u : 0u);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)dst, 4, LaneWord::lane4(at.fresh()), 0, 0, 0);
    };

    // End of a step: this wave's copies of the next tile have landed, its LDS writes (P) are done, then the
    // workgroup barrier (the empty asm statement keeps the compiler from moving LDS accesses across it).
    auto step_sync = [&]() {
      wait_async_loads();
      lds_barrier();
    };

    // Both roles share one shape of step, written as an explicit software pipeline (scheduling fences
    // between the groups, so that the order below is the order issued): LDS fragments are requested
    // AHEAD groups before the MFMAs that use them, and the arithmetic of the second half of the tile
    // (16 queries) is cut into slices that sit between the MFMAs of the first half.
    // (Four groups at four pairs: 65536 tokens and 200 short ones, 24 x 128, 82.8 -> 82.4 ms, three heads of up to 131072 44.4 ->
    // 44.1; at two pairs no gain, and up to 2 % worse on short sequences.)
    constexpr int AHEAD = PAIRS == 4 ? 4 : 2;
    // first product: x[kb] = sum over d of tile rows (A, from LDS) x this wave's K or V rows (B, registers / LDS)
    auto first_product = [&](const __bf16* tA, int rb, f32x16 (&x)[C::KB]) {
      bf16x8 af[C::KC];
#pragma unroll
      for (int cc = 0; cc < AHEAD; ++cc) af[cc] = rows.get(tA, rb, cc);
      KNAP_SCHED_FENCE();
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) {
#pragma unroll
        for (int kb = 0; kb < C::KB; ++kb) x[kb] = mfma32(af[cc], kvf[kb][cc], x[kb]);
        if (cc + AHEAD < C::KC) af[cc + AHEAD] = rows.get(tA, rb, cc + AHEAD);
        KNAP_SCHED_FENCE();
      }
    };
    // second product over the 16 queries of chunk cq: acc[kb][nb] += op[kb] (A, registers) x tile columns (B, LDS),
    // with `between(nb)` issued after the MFMAs of column block nb
    auto second_product = [&](const __bf16* tB, int cb, int cq, const bf16x8 (&op)[C::KB], auto between) {
      bf16x8 bf[C::NB];
      constexpr int AH2 = 2;
#pragma unroll
      for (int nb = 0; nb < AH2; ++nb) bf[nb] = cols.get(tB, cb, 16 * cq, nb);
      KNAP_SCHED_FENCE();
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb) {
#pragma unroll
        for (int kb = 0; kb < C::KB; ++kb) acc[kb][nb] = mfma32(bf[nb], op[kb], acc[kb][nb]);
        if (nb + AH2 < C::NB) bf[nb + AH2] = cols.get(tB, cb, 16 * cq, nb + AH2);
        between(nb);
        KNAP_SCHED_FENCE();
      }
    };

    // 16 bytes of this lane in block `b` of its pair's P of tile t
    auto p_at = [&](int w, int t, int b) {
      return reinterpret_cast<u32x4*>(reinterpret_cast<char*>(lds.p) + W::P_BLOCK * b + (w + (t & 1) * W::P_TILE));
    };
    // dV wave, tile t: S, P, hand P over, dV += P^T dO
    auto dv_step = [&](int t, const __bf16* tQ, const __bf16* tdO, const float* tLse) {
      const int rb = rows.fresh(), cb = cols.fresh(), w = at.fresh();
      f32x16 s[C::KB];
#pragma unroll
      for (int kb = 0; kb < C::KB; ++kb) s[kb] = zero16();
      first_product(tQ, rb, s);
      // P = exp2(c S - LSE2); register r of a key block is query 8 (r / 4) + 4 hh + r % 4, chunk cq holds
      // registers 8 cq .. 8 cq + 7, slice (kb, half) four of them
      bf16x8 pa[2][C::KB];
      bf16x4 ph[2][C::KB][2];
      f32x4 lq[2][2];
      auto lse_of = [&](int cq) {
        const char* row = reinterpret_cast<const char*>(tLse + 16 * cq) + LaneWord::hh16(w);
        lq[cq][0] = *reinterpret_cast<const f32x4*>(row);
        lq[cq][1] = *reinterpret_cast<const f32x4*>(row + 32);
      };
      // CAUSAL, tiles that cross the diagonal (the first BN / BM from q_first): a query before this lane's key
      // gets P = 0.  Counted from the tile's first query, the lane's key of block kb is the first one that
      // query `first_seen[kb]` sees.
      bool diag = false;
      int first_seen[C::KB];
      if constexpr (CAUSAL) {
        diag = n_tiles - 1 - t < C::BN / C::BM;
#pragma unroll
        for (int kb = 0; kb < C::KB; ++kb) first_seen[kb] = 64 * pair + 32 * kb + LaneWord::l32(w) - (n_tiles - 1 - t) * C::BM - LaneWord::hh16(w) / 4;
      }
      auto exp_slice = [&](int cq, int kb, int half) {
        float p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] = fast_exp2(__builtin_fmaf(s[kb][8 * cq + 4 * half + e], c, -lq[cq][half][e]));
        if constexpr (CAUSAL) {
          if (diag) {
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = 8 * (2 * cq + half) + e < first_seen[kb] ? 0.f : p[e];
          }
        }
        ph[cq][kb][half] = pack4(p[0], p[1], p[2], p[3]);
        if (half == 1) {
          pa[cq][kb] = join(ph[cq][kb][0], ph[cq][kb][1]);
          *p_at(w, t, 2 * kb + cq) = __builtin_bit_cast(u32x4, pa[cq][kb]);
        }
      };
      lse_of(0);
#pragma unroll
      for (int j = 0; j < 2 * C::KB; ++j) exp_slice(0, j >> 1, j & 1);
      lse_of(1);
      KNAP_SCHED_FENCE();
      second_product(tdO, cb, 0, pa[0], [&](int nb) {
        // 2 KB slices of the second chunk spread over NB groups
        if constexpr (C::NB == 4) exp_slice(1, nb >> 1, nb & 1);
        else { exp_slice(1, nb, 0); exp_slice(1, nb, 1); }
      });
      second_product(tdO, cb, 1, pa[1], [&](int) {});
    };
    // dK wave, tile u: dP - delta, dS = P (dP - delta) with the partner's P, dK += dS^T Q.  The product starts from -delta instead of
    // zero, which takes a subtraction per score out of the step (138 -> 106 vector instructions of a wave, beside 32 MFMAs):
    // dK/dV, us, images and videos, 24 x 128, 11080 -> 10850; three heads of up to 131072 43870 -> 42980; backward of 10 sequences
    // of up to 6795, 48 x 64, 4490 -> 4400.
    auto dk_step = [&](int u, const __bf16* tQ, const __bf16* tdO, const float* tDelta) {
      const int rb = rows.fresh(), w = at.fresh();
      f32x16 dp[C::KB];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(tDelta) + LaneWord::hh16(w) + 32 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int kb = 0; kb < C::KB; ++kb) dp[kb][4 * g + e] = x[e];
      }
      first_product(tdO, rb, dp);
      const int cb = cols.fresh();
      bf16x8 da[2][C::KB];
      bf16x4 dh[2][C::KB][2];
      u32x4 pw[2][C::KB];
      auto fetch_of = [&](int cq) {
#pragma unroll
        for (int kb = 0; kb < C::KB; ++kb) pw[cq][kb] = *p_at(w, u, 2 * kb + cq);
      };
      auto ds_slice = [&](int cq, int kb, int half) {
        float ds[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t word = pw[cq][kb][2 * half + (e >> 1)];
          const float p = __builtin_bit_cast(float, (e & 1) ? (word & 0xffff0000u) : (word << 16));
          ds[e] = p * dp[kb][8 * cq + 4 * half + e];
        }
        dh[cq][kb][half] = pack4(ds[0], ds[1], ds[2], ds[3]);
        if (half == 1) da[cq][kb] = join(dh[cq][kb][0], dh[cq][kb][1]);
      };
      fetch_of(0);
#pragma unroll
      for (int j = 0; j < 2 * C::KB; ++j) ds_slice(0, j >> 1, j & 1);
      fetch_of(1);
      KNAP_SCHED_FENCE();
      second_product(tQ, cb, 0, da[0], [&](int nb) {
        if constexpr (C::NB == 4) ds_slice(1, nb >> 1, nb & 1);
        else { ds_slice(1, nb, 0); ds_slice(1, nb, 1); }
      });
      second_product(tQ, cb, 1, da[1], [&](int) {});
    };

    // Steps that a pair has part in: none where the sequence ends in front of its keys, and under the mask none of those whose queries all
    // come before its keys (the last two, four or six, for the pairs behind the first); it leaves the SIMDs to the other waves.  Backward,
    // us: 100 sequences of 290 tokens, 24 x 128, 658 -> 642, 32 of 256..648 400 -> 395; under the mask, with the halves of tiles that dq_tile leaves out
    // likewise, 32 of 450 315 -> 309, 48 x 64, 334 -> 324, 17 of 328..4533 1902 -> 1886, 2038 -> 2013.
    const int n_own = 64 * pair >= L - kv0 ? 0 : CAUSAL ? n_tiles - 2 * pair : n_tiles;
    // Each role runs its own copy of the loop over the steps: with the roles as branches inside one
    // loop the accumulators would be merged at every step's join, and the register allocator then keeps
    // two sets.  Every wave still executes the same sequence of copies, waits and barriers.
#define KNAP_STEP(ROLE, t, cur, prev, nxt)                                                    \
    do {                                                                                      \
      issue_tile((t) + 1, sQ##nxt, sdO##nxt, sLse##nxt, sDelta##nxt);                  \
      if constexpr (ROLE == 0) {                                                              \
        if ((t) < n_own) dv_step((t), sQ##cur, sdO##cur, sLse##cur);                          \
      } else {                                                                                \
        if ((t) >= 1 && (t) <= n_own) dk_step((t) - 1, sQ##prev, sdO##prev, sDelta##prev); \
      }                                                                                       \
      step_sync();                                                                            \
    } while (0)
#define KNAP_ROLE_LOOP(ROLE)                                                                  \
    do {                                                                                      \
      int t = 0;                                                                              \
      for (; t + 2 <= n_tiles; t += 3) {                                                      \
        KNAP_STEP(ROLE, t, 0, 2, 1);                                                          \
        KNAP_STEP(ROLE, t + 1, 1, 0, 2);                                                      \
        KNAP_STEP(ROLE, t + 2, 2, 1, 0);                                                      \
      }                                                                                       \
      if (t <= n_tiles) {                                                                     \
        KNAP_STEP(ROLE, t, 0, 2, 1);                                                          \
        if (t + 1 <= n_tiles) KNAP_STEP(ROLE, t + 1, 1, 0, 2);                                \
      }                                                                                       \
    } while (0)

    issue_tile(0, sQ0, sdO0, sLse0, sDelta0);
    draw();
    step_sync();      // tile 0 has landed (and the K / V rows requested before it)
    drawn();

    if (role == 0) KNAP_ROLE_LOOP(0);
    else KNAP_ROLE_LOOP(1);
#undef KNAP_ROLE_LOOP
#undef KNAP_STEP

    ending();
    const auto rg = make_rsrc((role == 0 ? g.dv : g.dk) + (size_t)(it.row0 + kv0) * row_stride + head_off,
                              (uint32_t)min(L - kv0, C::BN) * row_bytes);
    const float out_scale = role == 0 ? 1.0f : scale;
    const int w_out = at.fresh();
#pragma unroll
    for (int kb = 0; kb < C::KB; ++kb) {
      const uint32_t off = (uint32_t)(64 * pair + 32 * kb + LaneWord::l32(w_out)) * row_bytes + (uint32_t)LaneWord::hh16(w_out);
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb) store_block(rg, off + 64u * nb, acc[kb][nb], out_scale);
    }
}

template <int D, int PAIRS, bool CAUSAL>
__global__ __launch_bounds__(128 * PAIRS, dkdv_waves_per_simd(D, PAIRS)) void attn_bwd_dkdv64_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
    const __bf16* __restrict__ dout, const float* __restrict__ lse2, const float* __restrict__ delta,
    const int32_t* __restrict__ cu, int n_seq, int H, float scale,
    __bf16* __restrict__ dk, __bf16* __restrict__ dv, unsigned* __restrict__ counters) {
  using C = Bwd2Cfg<D, PAIRS>;
  extern __shared__ int s_dyn[];
  int* s_order = s_dyn;
  int* s_start = s_dyn + n_seq;
#define KNAP_RING(i)                                                                    \
  __shared__ __attribute__((aligned(1024))) __bf16 sQ##i[C::TILE_ELEMS];                \
  __shared__ __attribute__((aligned(1024))) __bf16 sdO##i[C::TILE_ELEMS];               \
  __shared__ __attribute__((aligned(256))) float sLse##i[64];                           \
  __shared__ __attribute__((aligned(256))) float sDelta##i[64];
  KNAP_RING(0) KNAP_RING(1) KNAP_RING(2)
#undef KNAP_RING
  __shared__ __attribute__((aligned(256))) float sSink[64];
  __shared__ __attribute__((aligned(16))) u32x4 sP[C::PAIRS][2][2 * C::KB][64];

  const int T = cu[n_seq];
  const int n_items = build_schedule<C::BN, C::THREADS, CAUSAL>(cu, n_seq, H, s_order, s_start, reinterpret_cast<int*>(&sP[0][0][0][0]));
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // PAIRS = 2: the two waves of a pair sit on different SIMDs, each next to the waves of the CU's other workgroups; every
  // other one of those (a half or a third of the grid further on) has the roles the other way round, so that the SIMDs
  // get waves of either role
  const int role = (wave / PAIRS) ^ (PAIRS == 2 ? (int)(blockIdx.x * dkdv_workgroups_per_cu(D, PAIRS) / gridDim.x) & 1 : 0);
  const uint32_t row_bytes = (uint32_t)((size_t)H * D * sizeof(__bf16));
  DkdvLane<D, PAIRS> me;
  me.init(lane, wave, role, row_bytes);
  const BwdPtrs g = {q, k, v, nullptr, dout, nullptr, const_cast<float*>(lse2), const_cast<float*>(delta), nullptr, dk, dv, T, H, scale};
  const DkdvLds lds = {sQ0, sdO0, sQ1, sdO1, sQ2, sdO2, sLse0, sDelta0, sLse1, sDelta1, sLse2, sDelta2, sSink, &sP[0][0][0][0]};

  // work items from this XCD's queue, the next one's ticket drawn behind the item's first loads and put down after
  // the barrier that every wave reaches with its copy of the old one
  __shared__ int s_ticket;
  ItemQueue<0> queue;
  queue.init(counters, s_start, n_seq, n_items);
  for (int ticket = queue.first_ticket(); ticket < queue.wide;) {
    const int w = queue.item(ticket);
    unsigned next_ticket;      // thread 0 only; no initial value, which would be merged in (and waited for) at once
    WorkItem it = decode_item<C::BN, CAUSAL>(w, cu, n_seq, s_order, s_start);
    // head and tile come out of a division, i.e. of vector instructions: say that they are wave-uniform, so
    // that every base address below lives in scalar registers
    it.head = __builtin_amdgcn_readfirstlane(it.head);
    it.tile = __builtin_amdgcn_readfirstlane(it.tile);
    // CAUSAL: the item is the pair of key tiles {p, kv_tiles - 1 - p} (equal cost together, see build_schedule),
    // the one that meets more queries first; the middle tile of an odd count stands alone
    const int kv_tiles = (it.len + C::BN - 1) / C::BN;
    int sub = 0;
  second_tile_of_pair:;     // CAUSAL only: jumped back to once, from the end of the first tile
    dkdv_tile<D, PAIRS, CAUSAL>(g, lds, me, it, (!CAUSAL || sub == 0) ? it.tile : kv_tiles - 1 - it.tile,
        [&] { if (tid == 0 && sub == 0 && queue.draws) next_ticket = atomicAdd(queue.ctr, 1u); },
        [&] { if (tid == 0 && sub == 0 && queue.draws) s_ticket = queue.later_ticket(next_ticket); }, [] {});
    if constexpr (CAUSAL) {
      if (sub == 0 && it.tile != kv_tiles - 1 - it.tile) {   // not the middle tile of an odd count
        sub = 1;
        goto second_tile_of_pair;
      }
    }
    if (!queue.draws) break;
    ticket = __builtin_amdgcn_readfirstlane(s_ticket);
  }
}

template <int D, int PAIRS, bool CAUSAL>
static hipError_t launch_dkdv_t(const BwdArgs& a, int cus, hipStream_t stream) {
  const size_t dyn = (size_t)(2 * a.n_seq + 1) * sizeof(int);
  hipLaunchKernelGGL((attn_bwd_dkdv64_kernel<D, PAIRS, CAUSAL>), dim3(cus * dkdv_workgroups_per_cu(D, PAIRS)), dim3(128 * PAIRS),
                     dyn, stream, (const __bf16*)a.q, (const __bf16*)a.k, (const __bf16*)a.v, (const __bf16*)a.dout,
                     a.lse2, a.delta, a.cu, a.n_seq, a.H, a.scale, (__bf16*)a.dk, (__bf16*)a.dv, a.counters + 8);
  return hipGetLastError();
}

template <bool CAUSAL>
static hipError_t launch_dkdv_m(const BwdArgs& a, int d, int pairs, int cus, hipStream_t stream) {
  if (d == 64) return launch_dkdv_t<64, 2, CAUSAL>(a, cus, stream);
  return pairs == 2 ? launch_dkdv_t<128, 2, CAUSAL>(a, cus, stream) : launch_dkdv_t<128, 4, CAUSAL>(a, cus, stream);
}

}  // namespace knap
