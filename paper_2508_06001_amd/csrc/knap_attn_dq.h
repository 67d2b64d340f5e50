// dQ kernel of the backward: the forward kernel's structure.  S^T = K Q^T and dP^T = V dO^T put one query in each
// lane, LSE and delta are per-lane scalars, and dS^T is, unchanged, the B operand of dQ^T += K^T dS^T with K^T read
// transposed from LDS.  One text, compiled for either mask in a translation unit of its own (see build.py).
// d = 64: 168 registers (10 values spilled outside the loops, bidirectional) let three workgroups share a CU where 174 allowed two; the
// third wave of a SIMD fills the exponentials of the others (48 x 64, 10 sequences of 310..6795 tokens: 2077 -> 1988 us,
// 65536 tokens 77.6 -> 73.7 ms).
#pragma once

#include "knap_device.h"
#include "knap_kernels.h"

#include <type_traits>

namespace knap {

template <int D>
struct DqCfg {
  static constexpr int BM = 128;         // query rows per work item
  static constexpr int BN = 64;          // key/value rows per LDS tile
  static constexpr int KC = D / 16;
  static constexpr int DB = D / 32;
  static constexpr int TILE_ELEMS = BN * Tile<D>::LD;
};

struct DqLds {
  __bf16 *k0, *k1, *v0, *v1;
};

// what a lane keeps between query tiles
template <int D>
struct DqLane {
  RowReader<D> rows;     // K and V tile rows -> A operands of S^T and dP^T
  ColReader<D> cols;     // K tile columns -> A operands of dQ^T += K^T dS^T
  int lane, wave;        // the wave known to be wave-uniform
  __device__ __forceinline__ void init(int lane_, int wave_) {
    lane = lane_;
    wave = wave_;
    rows.init(lane);
    cols.init(lane);
  }
};

// delta = sum_c dO_c O_c of a lane's query: the lane holds half of the row's elements (8 of every 16),
// its partner at lane ^ 32 the other half
template <int D>
__device__ __forceinline__ float row_delta(const bf16x8 (&dof)[D / 16], const bf16x8 (&of)[D / 16]) {
  float dl = 0.f;
#pragma unroll
  for (int cc = 0; cc < D / 16; ++cc)
#pragma unroll
    for (int e = 0; e < 8; ++e) dl = __builtin_fmaf((float)dof[cc][e], (float)of[cc][e], dl);
  return dl + xor32(dl);
}

// Whether a whole query tile goes through the narrow form (dq_part): the last one of its sequence, of at most 64 rows, where
// two waves of four would have nothing but padding.  From the third tile on: the narrow form needs more than half of the time.
// (64 sequences, 24 x 128, us: of 448 tokens 339 -> 331, of 400 under the mask 286 -> 279, of 300, 48 x 64, 205 -> 199; but of
// 180 109 -> 115.)
__device__ __forceinline__ bool dq_narrow(int len, int q_tile) { return q_tile >= 2 && len - q_tile * 128 <= 64; }

// One query tile (128 rows) of an item.  DELTA: delta and the LSE in base 2 are formed here and handed on in memory; else
// they are read from there.  `draw` is called behind the first loads, `ending` in front of the stores.
template <int D, bool CAUSAL, bool DELTA, class Draw, class Ending>
__device__ __forceinline__ void dq_tile(const BwdPtrs& g, const DqLds& lds, const DqLane<D>& me, const WorkItem& it, int q_tile, Draw draw,
                                        Ending ending) {
    using C = DqCfg<D>;
    const auto *q = g.q, *k = g.k, *v = g.v, *out = g.out, *dout = g.dout;
    const float* lse = g.lse;
    float *delta = g.delta, *lse2_out = g.lse2;
    __bf16* dq = g.dq;
    const int L = it.len, T = g.T;
    const float scale = g.scale, c = scale * kLog2e;
    const size_t row_stride = (size_t)g.H * D;
    const uint32_t row_bytes = (uint32_t)(row_stride * sizeof(__bf16));
    const size_t head_off = (size_t)it.head * D;
    const auto& rows = me.rows;
    const auto& cols = me.cols;
    const int lane = me.lane, wave = me.wave, l32 = lane & 31, hh = lane >> 5;
    __bf16 *const sK0 = lds.k0, *const sK1 = lds.k1, *const sV0 = lds.v0, *const sV1 = lds.v1;
    const int q0 = q_tile * C::BM;
    const int q_row = q0 + wave * 32 + l32;
    const bool q_valid = q_row < L;
    // keys this query tile sees at all
    const int kv_end = CAUSAL ? min(L, q0 + C::BM) : L;

    const __bf16* k_base = k + (size_t)it.row0 * row_stride + head_off;
    const __bf16* v_base = v + (size_t)it.row0 * row_stride + head_off;
    const int n_tiles = (kv_end + C::BN - 1) / C::BN;

    // asynchronous; rows past the end arrive as zeros and add nothing to dQ
    auto load_tile = [&](int t, __bf16* dK, __bf16* dV) {
      const int kv0 = t * C::BN;
      const uint32_t bytes = (uint32_t)max(0, min(kv_end - kv0, C::BN)) * row_bytes;
      tile_load_async<D>(dK, make_rsrc(k_base + (size_t)kv0 * row_stride, bytes), row_bytes, C::BN, wave, lane);
      tile_load_async<D>(dV, make_rsrc(v_base + (size_t)kv0 * row_stride, bytes), row_bytes, C::BN, wave, lane);
    };

    // this lane's q and dO rows as B operands (rows past the end read as zero), and
    // delta = sum_c dO_c O_c of its query: the lane holds half of the row's elements (8 of every 16),
    // its partner at lane ^ 32 the other half.  The dK/dV kernel reads -delta from memory afterwards.
    // One tensor after the other: an access takes 32 bytes of each of 32 rows, and the four that share their 128-byte lines
    // find them in the L1 only if they follow each other (the three tensors of the CU's waves are several times its size).  Taken
    // in turn, dQ alone, us: 32 sequences of 256..648 tokens, 24 x 128, 201 against 192; 32 of 450, 48 x 64, 205 against 191.
    // The first tile is under way before delta is formed.
    // per-lane scalars of this lane's query; +inf LSE turns rows past the end into P = 0
    const size_t row_at = (size_t)it.head * T + it.row0 + (q_valid ? q_row : 0);
    float lse2 = DELTA ? lse[row_at] * kLog2e : lse2_out[row_at];
    bf16x8 qf[C::KC], dof[C::KC];
    float dl = DELTA ? 0.f : -delta[row_at];
    {
      const uint32_t bytes = (uint32_t)min(L - q0, C::BM) * row_bytes;
      const auto rq = make_rsrc(q + (size_t)(it.row0 + q0) * row_stride + head_off, bytes);
      const auto rd = make_rsrc(dout + (size_t)(it.row0 + q0) * row_stride + head_off, bytes);
      const auto ro = make_rsrc(out + (size_t)(it.row0 + q0) * row_stride + head_off, bytes);   // DELTA only
      const uint32_t off = (uint32_t)(wave * 32 + l32) * row_bytes + (uint32_t)(8 * hh) * 2u;
      bf16x8 of[C::KC];
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) qf[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rq, off + 32u * cc));
      KNAP_SCHED_FENCE();
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) dof[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rd, off + 32u * cc));
      KNAP_SCHED_FENCE();
      if constexpr (DELTA) {
#pragma unroll
        for (int cc = 0; cc < C::KC; ++cc) of[cc] = __builtin_bit_cast(bf16x8, buffer_load16(ro, off + 32u * cc));
        KNAP_SCHED_FENCE();
      }
      load_tile(0, sK0, sV0);    // a barrier stands between the last reads of either buffer (or the schedule build) and this
      KNAP_SCHED_FENCE();
      if constexpr (DELTA) dl = row_delta<D>(dof, of);
    }
    const float own = lse2;
    if (!q_valid) lse2 = INFINITY;
    f32x16 acc[C::DB];
#pragma unroll
    for (int db = 0; db < C::DB; ++db) acc[db] = zero16();

    // d = 64: dP^T starts from -delta, which sits in 16 registers through the loop, so that nothing is subtracted per score: 115
    // vector instructions per tile instead of 147, beside 24 MFMAs (48 x 64, forward and backward in us: 10 sequences of
    // 310..6795 tokens 5855 -> 5749, 16 of 4096 14010 -> 13746, 20 causal ones of 3000 5662 -> 5573; 32 of 450 the same).  At d =
    // 128 the 16 registers are not there: 54 to 129 values spilled around the loop, long sequences 0.8 to 1.4 % faster, 9 of
    // 1000 tokens, 12 heads, 2.3 % slower, 60 of 300, 24 heads, 2.2 %.
    constexpr bool SEEDED = D == 64;
    f32x16 dp_start;
    // One tile: 64 keys as two halves of 32, one after the other (the register file is full with
    // the q and dO fragments and the dQ accumulator; the second wave of the SIMD fills the gaps).
    // Within a half the LDS reads are streamed a few MFMAs ahead of their use.
    // MODE 2: the tile crosses the causal diagonal; keys after this lane's query get dS = 0, and a wave
    // whose 32 queries all precede a half's first key has nothing to do in it.
    // MODE 1: the ragged last tile; the scores of keys past the end of the sequence start (and stay) at
    // -inf, so P = 0 and dS = 0 there.  Their K and V rows arrive as zeros: left at score 0, P would be
    // exp2(-LSE2), which overflows for a query whose scores are all far below zero, and the product of
    // that dS with the zero K row would be NaN.  A second half without keys is left out, in the kernel of query tiles alone (64 sequences of
    // 450 tokens, 48 x 64, backward 827 -> 820 us, 32 of 24 x 128 404 -> 400; in the launch of both kinds it costs registers,
    // and one of 16384, 6 x 128, 0.9 %).
    auto process_tile = [&](auto mode_tag, int t, const __bf16* tK, const __bf16* tV, __bf16* nK, __bf16* nV) {
      constexpr int MODE = decltype(mode_tag)::value;
      constexpr bool DIAG = MODE == 2;
      load_tile(t + 1, nK, nV);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        if (DIAG && t * C::BN + 32 * half > q0 + 32 * wave + 31) break;
        if (MODE == 1 && DELTA && t * C::BN + 32 * half >= L) break;
        f32x16 s = zero16(), dp = SEEDED ? dp_start : zero16();
        if constexpr (MODE == 1) {
          const int first_past = L - t * C::BN - 32 * half - 4 * hh;   // counted from this half's first key
#pragma unroll
          for (int r = 0; r < 16; ++r) s[r] = 8 * (r >> 2) + (r & 3) >= first_past ? -INFINITY : 0.f;
        }
#pragma unroll
        for (int cc = 0; cc < C::KC; ++cc) {
          s = mfma32(rows.get(tK, 32 * half, cc), qf[cc], s);
          dp = mfma32(rows.get(tV, 32 * half, cc), dof[cc], dp);
        }
        // K^T fragments of the first 16 keys are requested before the arithmetic
        bf16x8 kt0[C::DB];
#pragma unroll
        for (int db = 0; db < C::DB; ++db) kt0[db] = cols.get(tK, 32 * half, db);
        KNAP_STREAM_READS(2 * C::KC, 1, 4);
        KNAP_SCHED_FENCE();
        // dS^T = P^T (dP^T - delta), P^T = exp2(c S^T - LSE2); element e of chunk ck is key
        // 32 half + 16 ck + 8 (e / 4) + 4 hh + e % 4
        float ds[16];
        const int last_seen = q_row - t * C::BN - 32 * half - 4 * hh;   // counted from this half's first key
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float x = fast_exp2(__builtin_fmaf(s[r], c, -lse2)) * (SEEDED ? dp[r] : dp[r] - dl);
          ds[r] = (DIAG && 8 * (r >> 2) + (r & 3) > last_seen) ? 0.f : x;
        }
        const bf16x8 d0 = pack8(ds[0], ds[1], ds[2], ds[3], ds[4], ds[5], ds[6], ds[7]);
        const bf16x8 d1 = pack8(ds[8], ds[9], ds[10], ds[11], ds[12], ds[13], ds[14], ds[15]);
        KNAP_SCHED_FENCE();
#pragma unroll
        for (int db = 0; db < C::DB; ++db) acc[db] = mfma32(kt0[db], d0, acc[db]);
#pragma unroll
        for (int db = 0; db < C::DB; ++db) acc[db] = mfma32(cols.get(tK, 32 * half + 16, db), d1, acc[db]);
        // the second chunk's K^T fragments between the first chunk's MFMAs (all of them in front: 65536 tokens and 200 short
        // ones, 24 x 128, 63.7 against 62.3 ms)
#pragma unroll
        for (int i = 0; i < C::DB; ++i) { KNAP_SGB(KNAP_SG_MFMA, 1); KNAP_SGB(KNAP_SG_DS_READ, 2); }
        KNAP_SGB(KNAP_SG_MFMA, C::DB);
        KNAP_SCHED_FENCE();
      }
      wait_async_loads();
      __syncthreads();     // next tile visible; this tile no longer read
    };

    wait_async_loads();
    draw();
    if constexpr (DELTA) {          // behind the wait, which would wait for these stores as well
      if (q_valid && hh == 0) {     // for the dK/dV kernel: -delta, and the LSE in base 2 (it copies both straight into LDS)
        delta[row_at] = -dl;
        lse2_out[row_at] = own;
      }
    }
    lds_barrier();
    if constexpr (SEEDED) {
#pragma unroll
      for (int r = 0; r < 16; ++r) dp_start[r] = -dl;
      asm volatile("" : "+v"(dp_start));         // 16 registers, not one that is copied 16 times per half tile
    }
    constexpr std::integral_constant<int, 0> plain{};
    constexpr std::integral_constant<int, 1> ragged_end{};
    constexpr std::integral_constant<int, 2> diagonal{};
    if constexpr (!CAUSAL) {
      const bool ragged = (L % C::BN) != 0;
      const int n_full = ragged ? n_tiles - 1 : n_tiles;
      for (int t = 0; t < n_full; t += 2) {
        process_tile(plain, t, sK0, sV0, sK1, sV1);
        if (t + 1 < n_full) process_tile(plain, t + 1, sK1, sV1, sK0, sV0);
      }
      if (ragged) {     // one instantiation for either buffer: the tile after the last is never loaded (empty descriptor)
        const bool odd = (n_tiles - 1) & 1;
        process_tile(ragged_end, n_tiles - 1, odd ? sK1 : sK0, odd ? sV1 : sV0, odd ? sK0 : sK1, odd ? sV0 : sV1);
      }
    } else {
      // tiles 0 .. 2 q_tile - 1 lie below the diagonal (an even count: the pair loop ends on buffer 0);
      // tiles 2 q_tile and, if the sequence reaches it, 2 q_tile + 1 cross it
      const int n_below = 2 * q_tile;
      for (int t = 0; t < n_below; t += 2) {
        process_tile(plain, t, sK0, sV0, sK1, sV1);
        process_tile(plain, t + 1, sK1, sV1, sK0, sV0);
      }
      process_tile(diagonal, n_below, sK0, sV0, sK1, sV1);
      if (n_below + 1 < n_tiles) process_tile(diagonal, n_below + 1, sK1, sV1, sK0, sV0);
    }

    ending();
    {
      const auto rg = make_rsrc(dq + (size_t)(it.row0 + q0) * row_stride + head_off,
                                (uint32_t)min(L - q0, C::BM) * row_bytes);
      const uint32_t off = (uint32_t)(wave * 32 + l32) * row_bytes + (uint32_t)(8 * hh) * 2u;
#pragma unroll
      for (int db = 0; db < C::DB; ++db) store_block(rg, off + 64u * db, acc[db], scale);
    }
}

// 64 query rows, from q0 on: waves w and w + 2 share 32 queries, one taking the first 32 keys of every tile, the other the
// second 32; the two gradients are added through LDS at the end.  `draw` and `ending` as above.
template <int D, bool CAUSAL, bool DELTA, class Draw, class Ending>
__device__ __forceinline__ void dq_part(const BwdPtrs& g, const DqLds& lds, const DqLane<D>& me, const WorkItem& it, int q0, Draw draw,
                                        Ending ending) {
    using C = DqCfg<D>;
    const auto *q = g.q, *k = g.k, *v = g.v, *out = g.out, *dout = g.dout;
    const float* lse = g.lse;
    float *delta = g.delta, *lse2_out = g.lse2;
    __bf16* dq = g.dq;
    const int L = it.len, T = g.T;
    const float scale = g.scale, c = scale * kLog2e;
    const size_t row_stride = (size_t)g.H * D;
    const uint32_t row_bytes = (uint32_t)(row_stride * sizeof(__bf16));
    const size_t head_off = (size_t)it.head * D;
    const auto& rows = me.rows;
    const auto& cols = me.cols;
    const int lane = me.lane, wave = me.wave, l32 = lane & 31, hh = lane >> 5;
    __bf16 *const sK0 = lds.k0, *const sK1 = lds.k1, *const sV0 = lds.v0, *const sV1 = lds.v1;
    const int rb = wave & 1;
    const int kh_u = __builtin_amdgcn_readfirstlane(wave >> 1), rb_u = __builtin_amdgcn_readfirstlane(rb);
    const int q_row = q0 + 32 * rb + l32;
    const bool q_valid = q_row < L;
    const int kv_end = CAUSAL ? min(L, q0 + 64) : L;
    const int n_tiles = (kv_end + C::BN - 1) / C::BN;
    const int first_masked = CAUSAL ? q0 / C::BN : L / C::BN;
    const int kv_lim = CAUSAL ? q_row + 1 : L;
    const __bf16* k_base = k + (size_t)it.row0 * row_stride + head_off;
    const __bf16* v_base = v + (size_t)it.row0 * row_stride + head_off;
    auto load_tile = [&](int t, __bf16* dK, __bf16* dV) {
      const int kv0 = t * C::BN;
      const uint32_t bytes = (uint32_t)max(0, min(kv_end - kv0, C::BN)) * row_bytes;
      tile_load_async<D>(dK, make_rsrc(k_base + (size_t)kv0 * row_stride, bytes), row_bytes, C::BN, wave, lane);
      tile_load_async<D>(dV, make_rsrc(v_base + (size_t)kv0 * row_stride, bytes), row_bytes, C::BN, wave, lane);
    };
    const uint32_t off = (uint32_t)(32 * rb + l32) * row_bytes + (uint32_t)(8 * hh) * 2u;
    const size_t q_at = (size_t)(it.row0 + q0) * row_stride + head_off;
    const uint32_t bytes = (uint32_t)min(L - q0, 64) * row_bytes;
    bf16x8 qf[C::KC], dof[C::KC];
    float dl = 0.f;
    {
      const auto rq = make_rsrc(q + q_at, bytes);
      const auto rd = make_rsrc(dout + q_at, bytes);
      const auto ro = make_rsrc(out + q_at, bytes);
      bf16x8 of[C::KC];
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) qf[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rq, off + 32u * cc));
      KNAP_SCHED_FENCE();
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) dof[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rd, off + 32u * cc));
      KNAP_SCHED_FENCE();
      if constexpr (DELTA) {
#pragma unroll
        for (int cc = 0; cc < C::KC; ++cc) of[cc] = __builtin_bit_cast(bf16x8, buffer_load16(ro, off + 32u * cc));
        KNAP_SCHED_FENCE();
      }
      load_tile(0, sK0, sV0);
      if constexpr (DELTA) dl = row_delta<D>(dof, of);
    }
    const size_t row_at = (size_t)it.head * T + it.row0 + (q_valid ? q_row : 0);
    float lse2;
    if constexpr (DELTA) {
      const float own = lse[row_at] * kLog2e;
      lse2 = q_valid ? own : INFINITY;
      if (q_valid && hh == 0 && kh_u == 0) {
        delta[row_at] = -dl;
        lse2_out[row_at] = own;
      }
    } else {
      dl = -delta[row_at];
      lse2 = q_valid ? lse2_out[row_at] : INFINITY;
    }
    f32x16 acc[C::DB];
#pragma unroll
    for (int db = 0; db < C::DB; ++db) acc[db] = zero16();
    wait_async_loads();
    draw();
    lds_barrier();

    auto half_tile = [&](int t, const __bf16* tK, const __bf16* tV, __bf16* nK, __bf16* nV) {
      load_tile(t + 1, nK, nV);
      const int k0 = t * C::BN + 32 * kh_u;
      if (!(CAUSAL && k0 > q0 + 32 * rb_u + 31)) {
        f32x16 s = zero16(), dp = zero16();
#pragma unroll
        for (int cc = 0; cc < C::KC; ++cc) {
          s = mfma32(rows.get(tK, 32 * kh_u, cc), qf[cc], s);
          dp = mfma32(rows.get(tV, 32 * kh_u, cc), dof[cc], dp);
        }
        bf16x8 kt0[C::DB];
#pragma unroll
        for (int db = 0; db < C::DB; ++db) kt0[db] = cols.get(tK, 32 * kh_u, db);
        KNAP_STREAM_READS(2 * C::KC, 1, 4);
        KNAP_SCHED_FENCE();
        float ds[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) ds[r] = fast_exp2(__builtin_fmaf(s[r], c, -lse2)) * (dp[r] - dl);
        if (t >= first_masked) {
          const int seen = kv_lim - k0 - 4 * hh;
#pragma unroll
          for (int r = 0; r < 16; ++r) ds[r] = 8 * (r >> 2) + (r & 3) < seen ? ds[r] : 0.f;
        }
        const bf16x8 d0 = pack8(ds[0], ds[1], ds[2], ds[3], ds[4], ds[5], ds[6], ds[7]);
        const bf16x8 d1 = pack8(ds[8], ds[9], ds[10], ds[11], ds[12], ds[13], ds[14], ds[15]);
        KNAP_SCHED_FENCE();
#pragma unroll
        for (int db = 0; db < C::DB; ++db) acc[db] = mfma32(kt0[db], d0, acc[db]);
#pragma unroll
        for (int db = 0; db < C::DB; ++db) acc[db] = mfma32(cols.get(tK, 32 * kh_u + 16, db), d1, acc[db]);
        KNAP_SGB(KNAP_SG_DS_READ, 2 * C::DB);          // the second chunk's K^T fragments go out first
        KNAP_SGB(KNAP_SG_MFMA, 2 * C::DB);
        KNAP_SCHED_FENCE();
      }
      wait_async_loads();
      lds_barrier();
    };
    for (int t = 0; t < n_tiles; t += 2) {
      half_tile(t, sK0, sV0, sK1, sV1);
      if (t + 1 < n_tiles) half_tile(t + 1, sK1, sV1, sK0, sV0);
    }

    ending();
    float* part_acc = reinterpret_cast<float*>(rb_u == 0 ? sK1 : sV1);
    if (kh_u == 1) {
#pragma unroll
      for (int db = 0; db < C::DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 x = {acc[db][4 * g], acc[db][4 * g + 1], acc[db][4 * g + 2], acc[db][4 * g + 3]};
          *reinterpret_cast<f32x4*>(part_acc + ((4 * db + g) * 64 + lane) * 4) = x;
        }
    }
    lds_barrier();
    if (kh_u == 0) {
      const auto rg = make_rsrc(dq + q_at, bytes);
#pragma unroll
      for (int db = 0; db < C::DB; ++db) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(part_acc + ((4 * db + g) * 64 + lane) * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[db][4 * g + e] += x[e];
        }
        store_block(rg, off + 64u * db, acc[db], scale);
      }
    }
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void attn_bwd_dq_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
    const __bf16* __restrict__ out, const __bf16* __restrict__ dout, const float* __restrict__ lse,
    float* __restrict__ delta, float* __restrict__ lse2_out, const int32_t* __restrict__ cu, int n_seq, int H, float scale,
    __bf16* __restrict__ dq, unsigned* __restrict__ counters) {
  using C = DqCfg<D>;
  extern __shared__ int s_dyn[];
  int* s_order = s_dyn;
  int* s_start = s_dyn + n_seq;
  // K is read row-wise (S^T) and transposed (dQ^T), V row-wise (dP^T); two buffers each, as
  // separate arrays so that reads of one are known not to depend on the copy into the other
  __shared__ __attribute__((aligned(1024))) __bf16 sK0[C::TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) __bf16 sK1[C::TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) __bf16 sV0[C::TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) __bf16 sV1[C::TILE_ELEMS];
  static_assert(sizeof(__bf16) * C::TILE_ELEMS >= sizeof(int) * kThreads, "scan scratch must fit in a tile");

  const int T = cu[n_seq];
  const int n_items = build_schedule<C::BM, kThreads, CAUSAL>(cu, n_seq, H, s_order, s_start, reinterpret_cast<int*>(&sK0[0]));
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  // known to be wave-uniform, also behind the barrier to the compiler below: the LDS address of each of a tile's eight copies
  // would go through a vector register, 8 to 16 of 155 vector instructions per tile (with the forward's alike, forward and
  // backward of 60 sequences of 300 tokens, 24 x 128: 582 -> 573 us; 60 causal ones of 400 717 -> 705)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const BwdPtrs g = {q, k, v, out, dout, lse, lse2_out, delta, dq, nullptr, nullptr, T, H, scale};
  const DqLds lds = {sK0, sK1, sV0, sV1};

  // Work items come from this XCD's queue.  The ticket for the NEXT item is requested right
  // after the item's first loads (vector-memory operations complete in issue order: requested
  // before them, the slow counter update would hold up the whole prologue) and only looked at
  // when the item is done, so the counter's latency is never waited for.
  __shared__ int s_ticket;
  constexpr int SPLIT = CAUSAL ? 4 : 2;     // narrow items (64 queries) of a wide one
  ItemQueue<SPLIT> queue;
  queue.init(counters, s_start, n_seq, n_items);
  int ticket = queue.first_ticket();
  while (ticket < queue.wide + queue.parts) {
    const bool whole = ticket < queue.wide;
    const int p = queue.part0 + ticket - queue.wide;       // of the parts
    const WorkItem it = decode_item<C::BM, CAUSAL>(whole ? queue.item(ticket) : queue.n_wide + p / SPLIT, cu, n_seq, s_order, s_start);
    unsigned next_ticket;      // thread 0 only; no initial value, which would be merged in (and waited for) at once
    // CAUSAL: the item is the pair of query tiles {q_tiles - 1 - p, p}, the long one first
    const int other = (it.len + C::BM - 1) / C::BM - 1 - it.tile;
    int sub = !CAUSAL || whole ? 0 : (p % SPLIT) >> 1;
    bool first = true;
  second_tile_of_pair:;     // CAUSAL only: jumped back to once, from the end of the first tile
    auto draw = [&] { if (tid == 0 && first && queue.draws) next_ticket = atomicAdd(queue.ctr, 1u); };
    const int q_tile = !CAUSAL ? it.tile : sub == 0 ? other : it.tile;
    const int q0 = __builtin_amdgcn_readfirstlane(q_tile * C::BM + (whole ? 0 : 64 * (p & 1)));
    int ln = lane, wv = wave;
    // what follows from them is formed per tile, not kept in registers through the other form's (45 values were spilled at d =
    // 128, now 10, none in a loop over keys: 32 sequences of 450 tokens, 24 x 128, 200 -> 195 us)
    asm volatile("" : "+v"(ln), "+s"(wv));
    DqLane<D> me;
    me.init(ln, wv);
    if (whole && !dq_narrow(it.len, q_tile)) dq_tile<D, CAUSAL, true>(g, lds, me, it, q_tile, draw, [] {});
    else if (q0 < it.len && !(CAUSAL && !whole && sub == 1 && it.tile == other)) dq_part<D, CAUSAL, true>(g, lds, me, it, q0, draw, [] {});
    else draw();
    if constexpr (CAUSAL) {
      if (whole && first && it.tile != other) {   // not the middle tile of an odd count
        first = false;
        sub = 1;
        goto second_tile_of_pair;
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
static hipError_t launch_dq_m(const BwdArgs& a, int d, int cus, int wg_per_cu, hipStream_t stream) {
  const size_t dyn = (size_t)(2 * a.n_seq + 1) * sizeof(int);
  auto* kernel = d == 64 ? attn_bwd_dq_kernel<64, CAUSAL> : attn_bwd_dq_kernel<128, CAUSAL>;
  hipLaunchKernelGGL(kernel, dim3(cus * wg_per_cu), dim3(kThreads), dyn, stream, (const __bf16*)a.q, (const __bf16*)a.k,
                     (const __bf16*)a.v, (const __bf16*)a.out, (const __bf16*)a.dout, a.lse, a.delta, a.lse2, a.cu,
                     a.n_seq, a.H, a.scale, (__bf16*)a.dq, a.counters);
  return hipGetLastError();
}

}  // namespace knap
