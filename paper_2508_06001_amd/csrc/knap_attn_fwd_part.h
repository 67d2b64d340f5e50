// Pieces of the forward that its kernels share: the softmax of half a tile (32 keys), the query tiles of 128 rows, and the narrow items.
#pragma once

#include "knap_device.h"
#include "knap_kernels.h"

#include <type_traits>

namespace knap {

template <int D>
struct FwdCfg {
  static constexpr int BM = 128;         // query rows per work item
  static constexpr int BN = 64;          // key/value rows per LDS tile
  static constexpr int KC = D / 16;      // contraction chunks over d
  static constexpr int DB = D / 32;      // 32-wide blocks of d
  static constexpr int TILE_ELEMS = BN * Tile<D>::LD;
};

struct FwdPtrs {
  const __bf16 *q, *k, *v;
  __bf16* out;
  float* lse;
  int T, H;
  float scale;
};

struct FwdLds {
  __bf16 *k0, *k1, *v0, *v1;
};

constexpr float kMaxHalfSum = 256.f;        // of a lane's 16 probabilities against the present reference

// `seen`: keys of the half, from its first, that this lane's query sees
__device__ __forceinline__ void mask_half(f32x16& s, int seen, int hh) {
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = 8 * (r >> 2) + (r & 3) < seen - 4 * hh ? s[r] : -INFINITY;
}

__device__ __forceinline__ float half_max(const f32x16& s, int seen, int hh) {
  float m = -INFINITY;
#pragma unroll
  for (int r = 0; r < 16; ++r) m = fmaxf(m, 8 * (r >> 2) + (r & 3) < seen - 4 * hh ? s[r] : -INFINITY);
  return m;
}

// P^T of a half, packed, against the reference as it stands (mc = m_ref c): element e of chunk ck is key
// 16 ck + 8 (e / 4) + 4 hh + e % 4; the lane's 16 rounded probabilities are added to `l`
__device__ __forceinline__ void half_exps(const f32x16& s, float c, float mc, bf16x8 (&pb)[2], float& l) {
  float p[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) p[r] = fast_exp2(__builtin_fmaf(s[r], c, -mc));
#pragma unroll
  for (int ck = 0; ck < 2; ++ck) {
    const int r0 = 8 * ck;
    pb[ck] = pack8_sum(p[r0], p[r0 + 1], p[r0 + 2], p[r0 + 3], p[r0 + 4], p[r0 + 5], p[r0 + 6], p[r0 + 7], l);
  }
}

// `l_new` is l_run with the half's probabilities added.  The reference moves only when they are too large (always
// on the first half, where it is -inf and the sum inf or NaN): up to the maximum, with what is accumulated rescaled
// and the half's probabilities formed again.  The first half of a tile takes the maximum of the whole tile, so that
// the largest probability of an item's first 64 keys is exactly 1 and carries no rounding error (taken over 32
// keys, the error of lse against 64 bits grew by up to 6 %, that of out by up to 1.7 %).  That it moves is rare behind the first keys: what it takes
// stands out of the loops' way (APART), but not under the mask.  Forward in us, with the start of fwd_tile: 6 sequences of 1536, 2 x 64, 19.7 -> 18.5, 1944,
// 12 x 64, 23.9 -> 22.7, 30 of 290, 3 x 128, 18.8 -> 18.1, 6 x 128 26.4 -> 27.1; 146 bags 1.009; under the mask 32 of 450, 12 x 128, 53.9 -> 57.9.
template <bool APART, int DB, class Maximum>
__device__ __forceinline__ void half_settle(const f32x16& s, float c, Maximum maximum, bf16x8 (&pb)[2], float l_new, float& m_ref, float& mc,
                                            float& l_run, f32x16 (&o)[DB]) {
  const bool moves = __builtin_amdgcn_ballot_w64(!(l_new - l_run <= kMaxHalfSum)) != 0;
  if (APART ? __builtin_expect(moves, 0) : moves) {
    const float m_loc = maximum();
    const float m_new = fmaxf(m_ref, fmaxf(m_loc, xor32(m_loc)));
    const float alpha = m_new == m_ref ? 1.f : fast_exp2((m_ref - m_new) * c);
    m_ref = m_new;
    mc = m_new == -INFINITY ? 0.f : m_new * c;
    l_run *= alpha;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    l_new = l_run;
    half_exps(s, c, mc, pb, l_new);
    if (m_new == -INFINITY) mc = -INFINITY;   // scores of -inf alone set no reference: the next half has to settle too
  }
  l_run = l_new;
}

// The loop over the keys of a query tile of 128 rows, 32 per wave.  Three halves of 32 keys that follow each other are in work at a time, in
// one slot of the pipeline: the scores of the last one, the probabilities of the middle one, the product with the values of the first one.
// No MFMA of a slot waits for its arithmetic, nor the other way round.  Against a loop in which a half's arithmetic stood between its two
// products, without the mask, us: 32 of 256..648 tokens 138 -> 133, one of 4292 259 -> 247, 20 of 1536 610 -> 571, 8 of 1024 119 -> 109, 64 of 450
// 263 -> 252 (24 x 128), the same bits.
//
// Results: o, its reference and this lane's share of the row sum (its 32 of the 64 keys per tile).  kv_lim: the first key that this
// lane's query does not see, in tiles from first_masked on.  copy_k(t, to) and copy_v copy this wave's share of tile t; the keys of tile 0
// have landed, the values of tile 0 and the keys of tile 1 are on their way.  draw() is called in the last turn.  A barrier has to stand
// behind it in front of whatever fills the tiles.
//
// n_own: the tiles that this wave's queries see (wave-uniform): under the mask one less than n_tiles for half of the waves, which leave
// the last turn to the others, and none for a wave whose rows lie past the end of the sequence, which leaves its SIMD to other
// workgroups (forward in us, 24 x 128: 100 of 290 tokens 216 -> 207, 32 of 256..648 130.5 -> 127, causal 102 -> 99).  last_half: whether
// they see keys of the second half of the last of these (left out where not: 64 of 450, 48 x 64, 276 -> 271, causal 211 -> 207).
template <int D, bool CAUSAL, class CopyK, class CopyV, class Draw>
__device__ __forceinline__ void fwd_tile(const FwdLds& lds, const bf16x8 (&qs)[D / 16], const RowReader<D>& k_rows, const ColReader<D>& v_cols, float c,
                                         int n_tiles, int n_own, bool last_half, int first_masked, int kv_lim, int hh, CopyK copy_k, CopyV copy_v, Draw draw,
                                         f32x16 (&o)[D / 32], float& m_ref, float& l_run) {
  using C = FwdCfg<D>;
  constexpr int KC = C::KC, DB = C::DB;
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = zero16();
  m_ref = -INFINITY;         // exponent reference (raw score units)
  float mc = -INFINITY;      // m_ref * c
  l_run = 0.f;
  if (n_own == 0) {         // no rows: nothing but this wave's copies
    for (int t = 0; t < n_tiles - 1; ++t) {
      wait_async_loads();
      lds_barrier();
      copy_k(t + 2, (t & 1) ? lds.k1 : lds.k0);
      copy_v(t + 1, (t & 1) ? lds.v0 : lds.v1);
    }
    wait_async_loads();
    lds_barrier();
    return;
  }
  bf16x2 ones;
  ones[0] = (__bf16)1.0f;
  ones[1] = (__bf16)1.0f;
  bf16x8 ak[KC];
  // One slot: the scores sn of a half (QK: its keys in `ak`), the probabilities pn of the half before (of scores s), the product of
  // the one before that (PV: its probabilities pb, its values at tV).  Cut into as many groups as it has MFMAs, fences between
  // them, so that the order below is the order issued; `behind(i)` goes into the groups of the second product.
  auto slot = [&](auto qk_tag, auto pv_tag, auto lead_tag, const f32x16& s, f32x16& sn, const bf16x8 (&pb)[2], bf16x8 (&pn)[2],
                  const __bf16* tV, float& l, auto behind) __attribute__((always_inline)) {
    constexpr bool QK = decltype(qk_tag)::value, PV = decltype(pv_tag)::value;
    constexpr int LEAD = decltype(lead_tag)::value;          // probabilities in front of the first MFMA
    constexpr int GROUPS = (QK ? KC : 0) + (PV ? 2 * DB : 0), PER = (16 + GROUPS - 1) / GROUPS;
    float p[16];
    uint32_t w[2][4];
    auto form = [&](int r) __attribute__((always_inline)) {          // probability r, and the pair that is complete
      if (r < 16) p[r] = fast_exp2(__builtin_fmaf(s[r], c, -mc));
      if (r >= 3 && (r & 1)) {
        const int j = (r - 3) >> 1;      // pair j: registers 2 j and 2 j + 1
        bf16x2 x;
        x[0] = (__bf16)p[2 * j];
        x[1] = (__bf16)p[2 * j + 1];
        l = __builtin_amdgcn_fdot2_f32_bf16(x, ones, l, false);
        w[j >> 2][j & 3] = __builtin_bit_cast(uint32_t, x);
      }
    };
#pragma unroll
    for (int r = 0; r < LEAD; ++r) form(r);
    KNAP_SCHED_FENCE();
    bf16x8 vt[2][DB];
    if constexpr (PV && !QK) {
#pragma unroll
      for (int i = 0; i < 2 * DB; ++i) vt[i / DB][i % DB] = v_cols.get(tV, 16 * (i / DB), i % DB);
      KNAP_SCHED_FENCE();
    }
    int r = LEAD;
    if constexpr (QK) {
#pragma unroll
      for (int i = 0; i < KC; ++i) {
        sn = mfma32(ak[i], qs[i], i == 0 ? zero16() : sn);
        if constexpr (PV) vt[i / DB][i % DB] = v_cols.get(tV, 16 * (i / DB), i % DB);
#pragma unroll
        for (int e = 0; e < PER; ++e) form(r++);
        KNAP_SCHED_FENCE();
      }
    }
    if constexpr (PV) {
#pragma unroll
      for (int i = 0; i < 2 * DB; ++i) {
        o[i % DB] = mfma32(vt[i / DB][i % DB], pb[i / DB], o[i % DB]);
        behind(i);
#pragma unroll
        for (int e = 0; e < PER; ++e) { if (r < 18) form(r); ++r; }
        KNAP_SCHED_FENCE();
      }
    }
    for (; r < 18; ++r) form(r);
#pragma unroll
    for (int ck = 0; ck < 2; ++ck) {
      u32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = w[ck][e];
      pn[ck] = __builtin_bit_cast(bf16x8, x);
    }
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  constexpr std::integral_constant<int, 0> at_once{};
  constexpr std::integral_constant<int, 4> some{};
  f32x16 s0, s1;            // scores of a tile's first and second half
  bf16x8 pb0[2], pb1[2];    // their probabilities
  auto keys_of = [&](const __bf16* tK, int row) __attribute__((always_inline)) {
#pragma unroll
    for (int cc = 0; cc < KC; ++cc) ak[cc] = k_rows.get(tK, row, cc);
  };
  auto nothing = [](int) {};
  auto mask_first = [&](int t) __attribute__((always_inline)) {
    if (t >= first_masked) mask_half(s0, kv_lim - t * C::BN, hh);
    KNAP_SCHED_FENCE();
  };
  auto settle_first = [&](int t, float l) __attribute__((always_inline)) {
    half_settle<!CAUSAL, DB>(s0, c, [&] { return fmaxf(half_max(s0, C::BN, hh), half_max(s1, kv_lim - t * C::BN - 32, hh)); }, pb0, l, m_ref, mc, l_run, o);
    KNAP_SCHED_FENCE();
  };
  auto mask_second = [&](int t) __attribute__((always_inline)) {
    if (t >= first_masked) mask_half(s1, kv_lim - t * C::BN - 32, hh);
    KNAP_SCHED_FENCE();
  };
  auto settle_second = [&](float l) __attribute__((always_inline)) {
    half_settle<!CAUSAL, DB>(s1, c, [&] { return half_max(s1, C::BN, hh); }, pb1, l, m_ref, mc, l_run, o);
    KNAP_SCHED_FENCE();
  };
  // One turn: the second half of tile t and the first of tile t + 1 go through the softmax.  Behind its barrier the keys of tile
  // t + 1 and the values of tile t are there, and nobody reads the keys of tile t or the values before it any longer.
  auto turn = [&](int t, const __bf16* tK, const __bf16* tV, __bf16* nK, __bf16* nV) __attribute__((always_inline)) {
    wait_async_loads();
    lds_barrier();
    if (t == n_tiles - 2) draw();
    keys_of(tK, 0);
    copy_k(t + 2, nK);
    copy_v(t + 1, nV);
    mask_second(t);
    float l = l_run;
    slot(yes, yes, some, s1, s0, pb0, pb1, tV, l, [&](int i) __attribute__((always_inline)) { if (i < KC) ak[i] = k_rows.get(tK, 32, i); });
    settle_second(l);
    mask_first(t + 1);
    l = l_run;
    slot(yes, yes, at_once, s0, s1, pb1, pb0, tV + 32 * Tile<D>::LD, l, nothing);
    settle_first(t + 1, l);
  };
  keys_of(lds.k0, 0);
#pragma unroll
  for (int cc = 0; cc < KC; ++cc) s0 = mfma32(ak[cc], qs[cc], cc == 0 ? zero16() : s0);
  keys_of(lds.k0, 32);
  KNAP_SCHED_FENCE();
  if (n_tiles == 1) draw();
  {
    mask_first(0);
    if constexpr (CAUSAL) {
      float l = l_run;
      slot(yes, no, at_once, s0, s1, pb1, pb0, lds.v0, l, nothing);
      settle_first(0, l);
    } else {
      // What the settling comes to here, without the probabilities against no reference: 30 of 600, 24 x 128, 185 -> 181 us.  Under the mask it loses
      // more than it gains: 32 of 450, 24 x 128, 104.6 -> 101, but 16 of 512 52.9 -> 58.3; at d = 64 5 % on 130 to 192 tokens, 3 % gained on 193 to 256.
#pragma unroll
      for (int cc = 0; cc < KC; ++cc) s1 = mfma32(ak[cc], qs[cc], cc == 0 ? zero16() : s1);
      const float m = fmaxf(half_max(s0, C::BN, hh), half_max(s1, kv_lim - 32, hh));
      m_ref = fmaxf(m, xor32(m));
      mc = m_ref == -INFINITY ? 0.f : m_ref * c;
      half_exps(s0, c, mc, pb0, l_run);
      if (m_ref == -INFINITY) mc = -INFINITY;
      KNAP_SCHED_FENCE();
    }
  }
  for (int t = 0; t < n_own - 1; t += 2) {
    turn(t, lds.k1, lds.v0, lds.k0, lds.v1);
    if (t + 2 < n_own) turn(t + 1, lds.k0, lds.v1, lds.k1, lds.v0);
  }
  wait_async_loads();
  lds_barrier();
  const bool early = CAUSAL && n_own < n_tiles;
  if (early) {              // the others' last turn: nothing but its copy
    draw();
    copy_v(n_own, (n_own & 1) ? lds.v1 : lds.v0);
  }
  const __bf16* tV = (n_own & 1) ? lds.v0 : lds.v1;
  if (last_half) {
    mask_second(n_own - 1);
    float l = l_run;
    slot(no, yes, at_once, s1, s0, pb0, pb1, tV, l, nothing);
    settle_second(l);
  }
  {       // the product of the last half with keys
    const bf16x8 (&pb)[2] = last_half ? pb1 : pb0;
    const int row = last_half ? 32 : 0;
    bf16x8 vt[2][DB];
#pragma unroll
    for (int ck = 0; ck < 2; ++ck)
#pragma unroll
      for (int db = 0; db < DB; ++db) vt[ck][db] = v_cols.get(tV + row * Tile<D>::LD, 16 * ck, db);
#pragma unroll
    for (int ck = 0; ck < 2; ++ck)
#pragma unroll
      for (int db = 0; db < DB; ++db) o[db] = mfma32(vt[ck][db], pb[ck], o[db]);
    KNAP_SCHED_FENCE();
  }
  if (early) {
    wait_async_loads();
    lds_barrier();
  }
}

// 64 query rows of an item's sequence and head, from q0 on.  Waves w and w + 2 share 32 of them, one taking the first 32 keys of
// every tile, the other the second 32; the two halves of the softmax are merged through LDS at the end.  A barrier has to stand
// between this and whatever reads or fills the tiles before or behind it.
template <int D, bool CAUSAL>
__device__ __forceinline__ void fwd_part(const FwdPtrs& g, const FwdLds& lds, const WorkItem& it, int q0, int lane, int wave) {
  using C = FwdCfg<D>;
  const int L = it.len, l32 = lane & 31, hh = lane >> 5, rb = wave & 1, kh = wave >> 1;
  const int kh_u = __builtin_amdgcn_readfirstlane(kh), rb_u = __builtin_amdgcn_readfirstlane(rb);
  const float c = g.scale * kLog2e;
  const size_t row_stride = (size_t)g.H * D;
  const uint32_t row_bytes = (uint32_t)(row_stride * sizeof(__bf16));
  // asynchronous copy of tile t (keys 64 t ..) of the item; rows at or past kv_end arrive as zeros
  auto load_tile = [&](int t, __bf16* dK, __bf16* dV) {
    const int kv_end = CAUSAL ? min(L, q0 + 64) : L;
    const int kv0 = t * C::BN;
    const uint32_t bytes = (uint32_t)max(0, min(kv_end - kv0, C::BN)) * row_bytes;
    const size_t off = (size_t)(it.row0 + kv0) * row_stride + (size_t)it.head * D;
    tile_load_async<D>(dK, make_rsrc(g.k + off, bytes), row_bytes, C::BN, wave, lane);
    tile_load_async<D>(dV, make_rsrc(g.v + off, bytes), row_bytes, C::BN, wave, lane);
  };
  const int q_row = q0 + 32 * rb + l32;
  const int kv_end = CAUSAL ? min(L, q0 + 64) : L;
  const int n_tiles = (kv_end + C::BN - 1) / C::BN;
  const int first_masked = CAUSAL ? q0 / C::BN : L / C::BN;
  const int kv_lim = CAUSAL ? q_row + 1 : L;
  const uint32_t off = (uint32_t)(32 * rb + l32) * row_bytes + (uint32_t)(8 * hh) * 2u;
  load_tile(0, lds.k0, lds.v0);
  bf16x8 qf[C::KC];          // this lane's query row as the B operand of S^T = K Q^T
  const auto rq = make_rsrc(g.q + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D,
                            (uint32_t)min(L - q0, 64) * row_bytes);
#pragma unroll
  for (int cc = 0; cc < C::KC; ++cc) qf[cc] = __builtin_bit_cast(bf16x8, buffer_load16(rq, off + 32u * cc));
  KNAP_SCHED_FENCE();
  RowReader<D> k_rows;       // K tile rows -> A operands of S^T (formed under the loads)
  ColReader<D> v_cols;       // V tile columns -> A operands of O^T += V^T P^T
  k_rows.init(lane);
  v_cols.init(lane);
  KNAP_SCHED_FENCE();
  wait_async_loads();
  lds_barrier();

  f32x16 o[C::DB];
#pragma unroll
  for (int db = 0; db < C::DB; ++db) o[db] = zero16();
  float m_ref = -INFINITY, mc = -INFINITY, l_run = 0.f;

  auto half_tile = [&](int t, const __bf16* tK, const __bf16* tV, __bf16* nK, __bf16* nV) {
    load_tile(t + 1, nK, nV);
    if (!(CAUSAL && t * C::BN + 32 * kh_u > q0 + 32 * rb_u + 31)) {
      f32x16 s = zero16();
#pragma unroll
      for (int cc = 0; cc < C::KC; ++cc) s = mfma32(k_rows.get(tK, 32 * kh, cc), qf[cc], s);
      bf16x8 vt[2][C::DB];
#pragma unroll
      for (int ck = 0; ck < 2; ++ck)
#pragma unroll
        for (int db = 0; db < C::DB; ++db) vt[ck][db] = v_cols.get(tV, 32 * kh + 16 * ck, db);
      if (t >= first_masked) mask_half(s, kv_lim - t * C::BN - 32 * kh, hh);
      bf16x8 pb[2];
      float l_new = l_run;
      half_exps(s, c, mc, pb, l_new);
      half_settle<!CAUSAL, C::DB>(s, c, [&] { return half_max(s, C::BN, hh); }, pb, l_new, m_ref, mc, l_run, o);
#pragma unroll
      for (int ck = 0; ck < 2; ++ck)
#pragma unroll
        for (int db = 0; db < C::DB; ++db) o[db] = mfma32(vt[ck][db], pb[ck], o[db]);
    }
    wait_async_loads();
    lds_barrier();
  };
  // The code here starts two instructions past a multiple of 32 bytes whatever stands in front of it.  Of 16 places, forward in us: 6
  // sequences of 1536 tokens, 2 x 64, 18.2 to 18.6 two and three past one, 19.1 to 19.6 elsewhere, 1944, 12 x 64, 22.6 to 22.9 and 23.4 to 23.8;
  // 2280, 2 x 64, 19.1 to 19.3 anywhere; d = 128 within 0.7 %; under the mask 1500, 12 x 64, 16.0 here (15.8 to 16.6), 5000, 2 x 64, 36.7 (35.4 to 37.0).
  asm volatile(".p2align 6\n\ts_nop 0\n\ts_nop 0");
  for (int t = 0; t < n_tiles; t += 2) {
    half_tile(t, lds.k0, lds.v0, lds.k1, lds.v1);
    if (t + 1 < n_tiles) half_tile(t + 1, lds.k1, lds.v1, lds.k0, lds.v0);
  }

  // merge: the waves of the second keys put down reference, sum and output, those of the first take them up
  // (in the tile buffers, which are free)
  float* part_o = reinterpret_cast<float*>(rb_u == 0 ? lds.k1 : lds.v1);
  float* part_ml = reinterpret_cast<float*>(lds.v0) + 128 * rb_u;
  if (kh_u == 1) {
    part_ml[lane] = m_ref;
    part_ml[64 + lane] = l_run;
#pragma unroll
    for (int db = 0; db < C::DB; ++db)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 x = {o[db][4 * j], o[db][4 * j + 1], o[db][4 * j + 2], o[db][4 * j + 3]};
        *reinterpret_cast<f32x4*>(part_o + ((4 * db + j) * 64 + lane) * 4) = x;
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
    const auto ro = make_rsrc(g.out + (size_t)(it.row0 + q0) * row_stride + (size_t)it.head * D,
                              (uint32_t)min(L - q0, 64) * row_bytes);
    const auto rl = make_rsrc(g.lse + (size_t)it.head * g.T + it.row0 + q0, (uint32_t)min(L - q0, 64) * 4u);
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, m_new * g.scale + __logf(l_tot)), rl,
                                          hh == 0 ? (32 * rb + l32) * 4 : 4 * 64, 0, 0);
#pragma unroll
    for (int db = 0; db < C::DB; ++db) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(part_o + ((4 * db + j) * 64 + lane) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[db][4 * j + e] = o[db][4 * j + e] * a_own + x[e] * a_other;
      }
      store_block(ro, off + 64u * db, o[db], inv);
    }
  }
}

}  // namespace knap
